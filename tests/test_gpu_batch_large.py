"""Batches of several grid groups on either side of the 100 MB of grid fields up to which the groups' FFT passes
are merged into one launch each: the first and the last problem of every group against the oracle.  FP64 1e-12,
mixed 2e-5, as the other applies."""
import numpy as np
import pytest
import torch

import paper_2210_07403_amd as ibdl

from test_gpu_batch_groups import _spec

from _helpers import make_oracle, relerr, to_np

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs an MI355X")]


@pytest.mark.parametrize("precision,large", [("fp64", 11), ("fp64", 12), ("mixed", 23), ("mixed", 24)])
def test_both_sides_of_the_limit(precision, large):
    sizes = [(512, 256)] + [(1024, 1024)] * large + [(256, 512)]
    mb = sum(a * b for a, b in sizes) * (8 if precision == "fp64" else 4) / 1e6
    assert abs(mb - 100.0) < 8.0
    specs = [_spec(n, k) for k, n in enumerate(sizes)]
    bt = ibdl.Batch([dict(dim=2, n=s.n, L=s.L, origin=s.origin, X=s.markers.X, nrm=s.markers.nrm, ds=s.markers.ds,
                          pde=s.pde, kappa=s.kappa, kernel=s.kernel) for s in specs], precision=precision)
    qs = [np.random.default_rng(50 + k).standard_normal(s.n_ib) for k, s in enumerate(specs)]
    tol = 1e-12 if precision == "fp64" else 2e-5
    for _ in range(2):
        ys = bt.apply(qs)
        for k in (0, 1, large, large + 1):
            assert relerr(to_np(ys[k]), make_oracle(specs[k]).apply(qs[k])) < tol, k
    bt.close()
