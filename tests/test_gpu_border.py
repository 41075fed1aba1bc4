"""The border rows' sums beside the interpolation (up to 16,384 markers: one more workgroup of its
launch; longer: a launch of their own) and the transposed operator combined in the interpolation's
launch, with one marker, at the limit and beyond it: the apply against the oracle and the transpose by
adjointness; FP64 1e-12, mixed 2e-5, as the other applies."""
import numpy as np
import pytest
import torch

from workloads import geometry as geo
from workloads import problems as P

from _helpers import make_oracle, make_problem, relerr, to_np

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs an MI355X")]

KINDS = {
    "fd": dict(dim=2, pde="poisson"),
    "spectral": dict(dim=2, pde="poisson", disc="spectral"),
    "bspline": dict(dim=2, pde="stokes", disc="spectral", kernel="bspline6"),
    "stokes": dict(dim=2, pde="stokes", disc="spectral"),
    "3d": dict(dim=3, pde="poisson", disc="spectral"),
}


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n_ib", [1, 16384, 16385])
@pytest.mark.parametrize("kind", list(KINDS))
def test_border_rows(kind, n_ib, precision):
    c = dict(disc="fd2", kernel="peskin4")
    c.update(KINDS[kind])
    dim, N = c["dim"], 64 if c["dim"] == 2 else 32
    rng = np.random.default_rng(n_ib)
    X = rng.uniform(0, 1, (n_ib, dim))
    nrm = rng.standard_normal((n_ib, dim))
    nrm /= np.linalg.norm(nrm, axis=1, keepdims=True)
    ds = rng.uniform(0.5, 1.5, n_ib) / n_ib
    spec = P.ProblemSpec("border", dim, (N,) * dim, (1.0,) * dim, (0.0,) * dim, c["pde"], 0.0, 1.0, "dirichlet", 3.0,
                         c["kernel"], c["disc"], geo.Markers(X, nrm, ds, float(ds.sum())), np.zeros(n_ib), None)
    tol = 1e-12 if precision == "fp64" else 2e-5
    with make_problem(spec, precision) as pr:
        q, p = rng.standard_normal(pr.n_aug), rng.standard_normal(pr.n_aug)
        Aq, Atp = to_np(pr.apply(q)), to_np(pr.apply_transpose(p))
        assert relerr(Aq, make_oracle(spec).apply(q)) < tol
        scale = np.linalg.norm(Atp) * np.linalg.norm(q) + np.linalg.norm(p) * np.linalg.norm(Aq)
        assert abs(Atp @ q - p @ Aq) < tol * scale
