"""When GMRES replays a captured operator apply: by default on grids of up to 2^14 points from the second
solve with the same markers, and again after anything that replaces what was captured (new markers, grid
arrays that a gradient makes larger).  Replayed and direct launches run the same kernels in the same order,
so every result has to have the bits of a handle that never replays."""
import numpy as np
import pytest
import torch

from workloads import problems as P

from _helpers import make_problem, to_np

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs an MI355X")]

SPECS = {
    # one field for the operator, two and three for the gradient
    "fd": lambda: P.helmholtz_circle(64, 0.75),
    "fd_completed": lambda: P.completed_poisson_exterior(32, 2.0, 10.0, "trig"),
    # the arrays already hold what the gradient needs
    "stokes": lambda: P.stokes_exterior_circle(32, 10.0),
    # beyond 2^14 points: direct launches throughout
    "fd_256": lambda: P.helmholtz_circle(256, 0.75),
}


def _calls(pr, spec):
    """Two solves, both gradients, two more solves and gradients, moved markers, moved back: every result."""
    out = []
    t = lambda v: torch.as_tensor(v, device="cuda")
    m = spec.markers
    psi = None

    def solve():
        q, u, info = pr.solve(spec.data, spec.g, tol=1e-9, maxit=200)
        out.extend([to_np(q), to_np(u), np.array([info.iters, info.status])])
        return q, u

    def gradients(q, u):
        nonlocal psi
        if psi is None:
            psi = t(np.random.default_rng(2).standard_normal(tuple(u.shape))).to(u.dtype)
        dX, dd, info = pr.backward(q, u, psi, tol=1e-9, maxit=200)
        out.extend([to_np(dX), to_np(dd), np.array([info.iters, info.status])])

    solve()
    gradients(*solve())        # the gradient makes the grid arrays larger behind a captured apply
    for _ in range(2):         # replays of a new capture, with direct applies between them
        q, u = solve()
        out.append(to_np(pr.apply(q)))
        gradients(q, u)
    h = spec.L[0] / spec.n[0]
    pr.set_markers(t(m.X + 0.3 * h), t(m.nrm), t(m.ds))
    for _ in range(3):         # direct, then captured, then replayed
        solve()
    pr.set_markers(t(m.X), t(m.nrm), t(m.ds))
    for _ in range(2):
        gradients(*solve())
    return out


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("name", sorted(SPECS))
def test_default_and_forced_replays_match_direct_launches(name, precision):
    spec = SPECS[name]()
    with make_problem(spec, precision) as pr:
        pr.set_graph(False)
        want = _calls(pr, spec)
    for mode in ("default", "forced"):
        with make_problem(spec, precision) as pr:
            if mode == "forced":
                pr.set_graph(True)
            got = _calls(pr, spec)
        assert len(got) == len(want)
        for k, (a, b) in enumerate(zip(got, want)):
            assert np.array_equal(a, b), (mode, k, np.max(np.abs(a - b)))
