"""Dense 2-D grid solves where the x passes' blocks get fewer rows so that every CU has one: from a single row
per block (long rows, few of them) to the full default, in both precisions, one field and two, against the
oracle.  1e-12 in FP64, 2e-5 on float grids as the other grid solves."""
import numpy as np
import pytest
import torch

from workloads import geometry as geo
from workloads import problems as P

from _helpers import make_oracle, make_problem, relerr, to_np

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs an MI355X")]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("pde", ["screened", "stokes"])
@pytest.mark.parametrize("n", [(16, 16), (64, 64), (64, 2048), (512, 128), (512, 512), (1024, 256), (2048, 256), (2048, 1024),
                               (4096, 16), (4096, 512), (8192, 64)])
def test_grid_solve(n, pde, precision):
    h = 1.0 / 64.0
    L = tuple(v * h for v in n)
    mk = geo.Markers(np.array([[0.3, 0.4], [0.5, 0.2]]) * np.array(L), np.array([[1.0, 0.0], [0.0, 1.0]]), np.full(2, h),
                     2 * h)
    spec = P.ProblemSpec("rows", 2, n, L, (0.0, 0.0), pde, 1.5, 1.0, "dirichlet", 0.0, "peskin4",
                         "spectral" if pde == "stokes" else "fd2", mk, np.zeros((2, 2) if pde == "stokes" else 2), None)
    o = make_oracle(spec)
    nc = 2 if pde == "stokes" else 1
    rhs = np.random.default_rng(n[0] + n[1]).standard_normal((nc, n[1], n[0]))
    if precision == "mixed":
        rhs = rhs.astype(np.float32).astype(np.float64)
    want = o._g_response(rhs if nc == 2 else rhs[0]).reshape(rhs.shape)
    with make_problem(spec, precision) as pr:
        got = to_np(pr.grid_solve(torch.as_tensor(rhs, device="cuda"))).reshape(rhs.shape)
    assert relerr(got, want) < (1e-12 if precision == "fp64" else 2e-5)
