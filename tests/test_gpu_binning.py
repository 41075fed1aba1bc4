"""Marker binning and the kernel-derivative gather where their work splits: candidate lists longer than
the 256 entries a sort stages at once, more busy tiles than one count trip, more tiles than one trip of
the scan (4,096), one marker, marker counts off the gather's sixteen per workgroup.

The apply reads every list, so it is compared with the oracle (FP64, 1e-12 as the other applies); moving
the markers and moving them back must give the first result bit for bit (the lists are sorted).
Gradients: 1e-8 against the oracle's dense ones, as the other backward tests."""
import numpy as np
import pytest
import torch

from oracle import Setup
from oracle import adjoint as ADJ
from workloads import geometry as geo
from workloads import problems as P

from _helpers import make_oracle, make_problem, relerr, to_np

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs an MI355X")]


def _spec(n, X, seed, eta=2.0, kernel="peskin4"):
    dim = len(n)
    rng = np.random.default_rng(seed)
    L = tuple(v / 64.0 for v in n)
    nrm = rng.standard_normal((len(X), dim))
    nrm /= np.linalg.norm(nrm, axis=1, keepdims=True)
    ds = rng.uniform(0.5, 1.5, len(X)) / 64.0 ** (dim - 1)
    return P.ProblemSpec("bins", dim, n, L, (0.0,) * dim, "screened", 2.0, 1.0, "dirichlet", eta, kernel,
                         "spectral" if kernel == "bspline6" else "fd2",
                         geo.Markers(np.asarray(X) * np.array(L), nrm, ds, float(ds.sum())), np.zeros(len(X)), None)


def _points(kind, dim, n):
    rng = np.random.default_rng(11)
    if kind == "one":
        return rng.uniform(0, 1, (1, dim))
    X = rng.uniform(0, 1, (3000 if dim == 2 else 900, dim))
    # 700 markers inside one tile: a list of three staged parts
    X[:700] = 0.5 + rng.uniform(0.1, 0.9, (700, dim)) * np.array([16, 4, 8][:dim]) / np.array(n)
    return X


@pytest.mark.parametrize("kind", ["one", "crowded"])
@pytest.mark.parametrize("n", [(64, 64), (2048, 1024), (32, 32, 32), (512, 64, 128)])
def test_lists(n, kind):
    spec = _spec(n, _points(kind, len(n), n), 3)
    q = np.random.default_rng(1).standard_normal(len(spec.markers.X))
    with make_problem(spec, "fp64") as pr:
        a = to_np(pr.apply(q))
        assert relerr(a, make_oracle(spec).apply(q)) < 1e-12
        m = spec.markers
        t = lambda v: torch.as_tensor(v, device="cuda")
        pr.set_markers(t(np.array(spec.L) - m.X), t(m.nrm), t(m.ds))
        pr.set_markers(t(m.X), t(m.nrm), t(m.ds))
        assert np.array_equal(to_np(pr.apply(q)), a)


@pytest.mark.parametrize("kernel", ["peskin4", "bspline6"])
@pytest.mark.parametrize("n,nib", [((32, 32), 17), ((16, 16, 16), 15), ((16, 16, 16), 33)])
def test_gather(n, nib, kernel):
    rng = np.random.default_rng(5)
    X = rng.uniform(0, 1, (nib, len(n)))
    spec = _spec(n, X, 4, eta=8.0, kernel=kernel)
    data = rng.standard_normal(nib)
    o = Setup(spec.dim, spec.n, spec.L, spec.origin, spec.markers.X, spec.markers.nrm, spec.markers.ds, spec.pde,
              spec.kappa, spec.mu, spec.bc, spec.eta, spec.kernel, spec.disc)
    psi = rng.standard_normal(o.grid.shape)
    gX, gd = ADJ.gradients(o, data, None, psi)
    with make_problem(spec, "fp64") as pr:
        q, u, info = pr.solve(data, None, tol=1e-13, maxit=200)
        dX, dd, ainfo = pr.backward(q, u, torch.as_tensor(psi), tol=1e-13, maxit=200)
        assert relerr(to_np(dd), gd) < 1e-9
        assert relerr(to_np(dX), gX) < 1e-8
