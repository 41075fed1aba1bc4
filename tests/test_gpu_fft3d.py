"""The 3-D x passes at every row length, 16 to 1024: the operator apply against the oracle and its
transpose by adjointness, on grids of nx x 16 x 16 with twelve markers at random places (windows
across the seams; rows whose markers touch a few segments only).  FP64 1e-12, mixed 2e-5."""
import numpy as np
import pytest
import torch

from workloads import geometry as geo
from workloads import problems as P

from _helpers import make_oracle, make_problem, relerr, to_np

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs an MI355X")]

KINDS = {
    "fd": dict(pde="screened", kappa=2.0),
    "spectral-eta": dict(pde="poisson", kappa=0.0, eta=3.0, disc="spectral", kernel="bspline6"),
}


def _spec(n, kw, seed):
    c = dict(pde="screened", kappa=0.0, mu=1.0, eta=0.0, kernel="peskin4", disc="fd2")
    c.update(kw)
    L = tuple(v / 64.0 for v in n)
    rng = np.random.default_rng(seed)
    X = rng.uniform(0, 1, (12, 3)) * np.array(L)
    nrm = rng.standard_normal((12, 3))
    nrm /= np.linalg.norm(nrm, axis=1, keepdims=True)
    ds = rng.uniform(0.5, 1.5, 12) / 4096.0
    return P.ProblemSpec("rows", 3, n, L, (0.0, 0.0, 0.0), c["pde"], c["kappa"], c["mu"], "dirichlet", c["eta"],
                         c["kernel"], c["disc"], geo.Markers(X, nrm, ds, float(ds.sum())), np.zeros(12), None)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("kind", list(KINDS))
def test_every_row_length(kind, precision):
    tol = 1e-12 if precision == "fp64" else 2e-5
    for k in range(4, 11):
        spec = _spec((1 << k, 16, 16), KINDS[kind], k)
        print(f"# {kind} {precision} {1 << k}", flush=True)
        with make_problem(spec, precision) as pr:
            rng = np.random.default_rng(k)
            q, p = rng.standard_normal(pr.n_aug), rng.standard_normal(pr.n_aug)
            Aq = to_np(pr.apply(q))
            assert relerr(Aq, make_oracle(spec).apply(q)) < tol, k
            Atp = to_np(pr.apply_transpose(p))
            assert abs(Atp @ q - p @ Aq) < tol * np.linalg.norm(Atp) * np.linalg.norm(q) + tol * np.linalg.norm(p) * np.linalg.norm(Aq), k
