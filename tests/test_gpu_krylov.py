"""GMRES at the vector lengths where the Arnoldi step changes form (one workgroup up to 256 and 1,024
entries, three launches beyond; batches of up to 1,024, 2,048, 4,096 and more unknowns) and at step
counts beyond the sixteen basis vectors a thread holds and the 64 columns the finish stages, against
the oracle's GMRES: solutions 1e-10 (well-conditioned) or residuals 1e-12 at a tolerance of 1e-13."""
import numpy as np
import pytest
import torch

from oracle.gmres import gmres
from workloads import geometry as geo
from workloads import problems as P

from _helpers import make_oracle, make_problem, relerr, to_np

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs an MI355X")]


def _circle(n_ib, N=64):
    mk = geo.circle((0.5, 0.5), 0.27, n_ib)
    t = np.arctan2(mk.X[:, 1] - 0.5, mk.X[:, 0] - 0.5)
    return P.ProblemSpec("circle", 2, (N, N), (1.0, 1.0), (0.0, 0.0), "screened", 1.0, 1.0, "dirichlet", 0.0, "peskin4",
                         "fd2", mk, np.sin(2 * t) + 0.3 * np.cos(5 * t), None)


@pytest.mark.parametrize("n_ib", [3, 64, 65, 255, 256, 257, 1023, 1024, 1025, 2049])
def test_vector_lengths(n_ib):
    spec = _circle(n_ib)
    o = make_oracle(spec)
    want, k, _ = gmres(o.apply, o.rhs(spec.data, None), 1e-13, 100)
    with make_problem(spec) as pr:
        q, _, info = pr.solve(spec.data, None, tol=1e-13, maxit=100)
        print(f"# {n_ib} markers: {info.iters} iterations (oracle {k})", flush=True)
        assert relerr(to_np(q), want) < 1e-10
        assert abs(info.iters - k) <= 1 and info.true_relres_fp64 < 1e-11


@pytest.mark.parametrize("markers", [400, 600])
def test_many_steps(markers):
    """A cylinder array close to touching with a large completion constant: 802 and 1,202 unknowns,
    about 70 steps; the residual of the solution under the oracle's operator."""
    spec = P.cylinder_array(128, 0.74, eta=1000.0)
    spec.markers = geo.PolarCurve((0.0, 0.0), spec.meta["r"]).markers(markers).flipped()
    spec.data = np.zeros((markers, 2))
    o = make_oracle(spec)
    b = o.rhs(spec.data, spec.g)
    _, k, _ = gmres(o.apply, b, 1e-13, 200)
    with make_problem(spec) as pr:
        q, _, info = pr.solve(spec.data, spec.g, tol=1e-13, maxit=200)
        res = np.linalg.norm(b - o.apply(to_np(q))) / np.linalg.norm(b)
        print(f"# {pr.n_aug} unknowns: {info.iters} iterations (oracle {k}), residual {res:.2e}", flush=True)
        assert k > 64 and abs(info.iters - k) <= 2
        assert res < 1e-12


@pytest.mark.parametrize("largest", [1024, 1025, 2049, 4097])
def test_batch_vector_lengths(largest):
    import paper_2210_07403_amd as ibdl
    specs = [_circle(n) for n in (3, 300, largest)]
    b = ibdl.Batch([dict(dim=2, n=s.n, L=s.L, origin=s.origin, X=s.markers.X, nrm=s.markers.nrm, ds=s.markers.ds,
                         pde="screened", kappa=1.0) for s in specs], precision="fp64")
    qs, _, infos = b.solve([s.data for s in specs], tol=1e-13)
    for s, q, info in zip(specs, qs, infos):
        o = make_oracle(s)
        want, k, _ = gmres(o.apply, o.rhs(s.data, None), 1e-13, 100)
        print(f"# {s.n_ib} of {largest}: {info.iters} iterations (oracle {k})", flush=True)
        assert relerr(to_np(q), want) < 1e-10 and abs(info.iters - k) <= 1
    b.close()
