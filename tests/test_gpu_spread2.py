"""The 2-D spread where a wave's candidates end: one, an odd number, a round of 16 (double) or 32 (single
precision) and one more, several rounds; windows over the seams of the smallest grid, where a tile is the whole
axis.  Operator applies against the oracle, which evaluates the same sums in double: 1e-12 in FP64, 2e-5 on
float grids as the other applies."""
import numpy as np
import pytest
import torch

from workloads import geometry as geo
from workloads import problems as P

from _helpers import make_oracle, make_problem, relerr, to_np

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs an MI355X")]

KINDS = {
    "fd": dict(pde="screened", disc="fd2", eta=0.0),
    "spectral": dict(pde="screened", disc="spectral", eta=3.0),
    "stokes": dict(pde="stokes", disc="spectral", eta=3.0),
}


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("n,nib", [((16, 16), k) for k in (1, 2, 5, 13, 64, 65, 129, 260)] + [((64, 16), 515)])
def test_round_ends(n, nib, kind, precision):
    rng = np.random.default_rng(nib)
    L = np.array(n) / 16.0
    X = rng.uniform(0.0, 1.0, (nib, 2)) * L
    X[:: 3] = (rng.uniform(-2.0, 2.0, (len(X[:: 3]), 2)) / 16.0) % L      # across the seams
    nrm = rng.standard_normal((nib, 2))
    nrm /= np.linalg.norm(nrm, axis=1, keepdims=True)
    ds = rng.uniform(0.5, 1.5, nib) / nib
    kw = KINDS[kind]
    spec = P.ProblemSpec("rounds", 2, n, tuple(L), (0.0, 0.0), kw["pde"], 2.0, 1.0, "dirichlet", kw["eta"], "peskin4",
                         kw["disc"], geo.Markers(X, nrm, ds, float(ds.sum())), np.zeros(nib), None)
    o = make_oracle(spec)
    tol = 1e-12 if precision == "fp64" else 2e-5
    q = np.random.default_rng(1).standard_normal(o.n_aug)
    with make_problem(spec, precision) as pr:
        assert relerr(to_np(pr.apply(q)), o.apply(q)) < tol
        u = pr.spread(q[:nib * pr.nq].reshape(nib, pr.nq))
        assert relerr(to_np(u).reshape(pr.nq, -1), np.asarray(_spread(o, spec, q[:nib * pr.nq])).reshape(pr.nq, -1)) < tol


def _spread(o, spec, f):
    """S f: the oracle's weights, summed plainly."""
    nx, ny = spec.n
    h = spec.L[0] / nx
    m = spec.markers
    f = f.reshape(len(m.X), -1)
    out = np.zeros((f.shape[1], ny, nx))

    def phi(r):
        a = np.abs(r)
        lo = (3 - 2 * a + np.sqrt(np.maximum(1 + 4 * a - 4 * a * a, 0))) / 8
        hi = (5 - 2 * a - np.sqrt(np.maximum(-7 + 12 * a - 4 * a * a, 0))) / 8
        return np.where(a <= 1, lo, np.where(a < 2, hi, 0.0))

    for i, x in enumerate(m.X):
        w = []
        for d, n in enumerate((nx, ny)):
            t = x[d] / h
            k = int(np.floor(t)) + np.arange(-2, 4)
            wd = np.zeros(n)
            np.add.at(wd, k % n, phi(k - t))
            w.append(wd)
        out += (f[i] * m.ds[i] / h ** 2)[:, None, None] * np.outer(w[1], w[0])[None]
    return out
