"""GMRES where the Krylov space is invariant after one step.  With a screening constant of 1e12 the potential
of the density is below the last place of every entry, so A q is q / 2 exactly and the first step's w is
parallel to V_0: its projection is rounding, and so is what a second projection leaves.

In binary arithmetic that rounding is known.  With |V_0|^2 summed to 1 + j eps (|j| up to 7, by the same sums
throughout) the first pass leaves w = c V_0, c = -j eps / 2, and the second c j eps V_0, to one more rounding of
c V_0 where j is no power of two: |w| is at most (j^2 + |j|) eps^2 / 2, its residual estimate twice that and at
most 64 eps^2 = 3.2e-30, and only j = 0 is a breakdown (w = 0, solved).  A norm formed as sqrt(|c|^2 - h2^2)
would instead be 0, reported as solved, or of the order of eps^1.5 = 3e-24.  The vectors' lengths take every form of the step (one workgroup up to 256 and
1,024 entries, three launches beyond)."""
import numpy as np
import pytest
import torch

from workloads import geometry as geo
from workloads import problems as P

from _helpers import make_problem, to_np

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs an MI355X")]

SEEDS = 8


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("n_ib", [200, 256, 1000, 1025, 2049, 5000])
def test_norm_of_a_vector_at_rounding_level(n_ib, graph):
    mk = geo.circle((0.5, 0.5), 0.27, n_ib)
    spec = P.ProblemSpec("circle", 2, (64, 64), (1.0, 1.0), (0.0, 0.0), "screened", 1e12, 1.0, "dirichlet", 0.0,
                         "peskin4", "fd2", mk, np.zeros(n_ib), None)
    exact = 0
    with make_problem(spec) as pr:
        pr.set_graph(graph)
        for seed in range(SEEDS):
            rng = np.random.default_rng(seed)
            data = rng.uniform(1.0, 2.0, n_ib) * rng.choice([-1.0, 1.0], n_ib)
            q, _, info = pr.solve(data, None, tol=0.0, maxit=1)
            print(f"# {n_ib}: status {info.status} residual {info.krylov_relres:.3e}", flush=True)
            assert info.iters == 1 and np.max(np.abs(to_np(q) / (2.0 * data) - 1.0)) < 1e-14
            if info.status == 0:
                assert info.krylov_relres == 0.0
                exact += 1
            else:
                assert 0.0 < info.krylov_relres <= 3.2e-30
        # |V_0|^2 is 1 to the last place now and then, not as a rule
        assert exact < SEEDS - 1


@pytest.mark.parametrize("n_ib", [1000, 1025, 5000])
def test_zero_data(n_ib):
    mk = geo.circle((0.5, 0.5), 0.27, n_ib)
    spec = P.ProblemSpec("circle", 2, (64, 64), (1.0, 1.0), (0.0, 0.0), "screened", 2.0, 1.0, "dirichlet", 0.0, "peskin4",
                         "fd2", mk, np.zeros(n_ib), None)
    with make_problem(spec) as pr:
        q, u, info = pr.solve(spec.data, None, tol=1e-10, maxit=20)
        assert info.status == 0 and info.iters == 0 and info.krylov_relres == 0.0
        assert not to_np(q).any() and not to_np(u).any()
