"""The FFT passes of a batch's grid groups merged into one launch per pass: every row length (64 to
1,024 points) and lines from the shortest to the longest, several problems to a group, against the
oracle; and the same problems with a grid that cannot be merged among them, where the passes run group
by group.  FP64 1e-12, mixed 2e-5, as the other applies."""
import numpy as np
import pytest
import torch

import paper_2210_07403_amd as ibdl
from workloads import geometry as geo
from workloads import problems as P

from _helpers import make_oracle, relerr, to_np

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs an MI355X")]

GRIDS = [(64, 64), (64, 1024), (128, 32), (128, 32), (256, 16), (256, 512), (512, 256), (512, 256), (512, 256),
         (1024, 16), (1024, 1024), (64, 64)]


def _spec(n, seed):
    rng = np.random.default_rng(seed)
    L = tuple(v / 64.0 for v in n)
    nib = 5 + seed % 7
    nrm = rng.standard_normal((nib, 2))
    nrm /= np.linalg.norm(nrm, axis=1, keepdims=True)
    ds = rng.uniform(0.5, 1.5, nib) / 64.0
    return P.ProblemSpec("group", 2, n, L, (0.0, 0.0), "screened", 2.0, 1.0, "dirichlet", 0.0, "peskin4", "fd2",
                         geo.Markers(rng.uniform(0, 1, (nib, 2)) * np.array(L), nrm, ds, float(ds.sum())),
                         np.zeros(nib), None)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("grids", [GRIDS, GRIDS + [(32, 64)]], ids=["merged", "apart"])
def test_groups(grids, precision):
    specs = [_spec(n, k) for k, n in enumerate(grids)]
    probs = [dict(dim=2, n=s.n, L=s.L, origin=s.origin, X=s.markers.X, nrm=s.markers.nrm, ds=s.markers.ds,
                  pde=s.pde, kappa=s.kappa, kernel=s.kernel) for s in specs]
    bt = ibdl.Batch(probs, precision=precision)
    qs = [np.random.default_rng(50 + k).standard_normal(s.n_ib) for k, s in enumerate(specs)]
    tol = 1e-12 if precision == "fp64" else 2e-5
    for _ in range(2):
        for s, q, y in zip(specs, qs, bt.apply(qs)):
            assert relerr(to_np(y), make_oracle(s).apply(q)) < tol, s.n
    bt.close()
