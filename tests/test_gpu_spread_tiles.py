"""Problem.spread_tiles is a plain question: answered without a wait, also while a stream is captured, and
right behind new markers.  The counts are recounted on the host from the markers' windows; rows of one and of
several 64-bit words of segments, markers in one corner and across the seams."""
import numpy as np
import pytest
import torch

from test_gpu_parity import _spec_like, _tiles_reference

from _helpers import make_problem

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs an MI355X")]


def _spec(n, kind, seed):
    dim = len(n)
    rng = np.random.default_rng(seed)
    L = np.array(n) / 64.0
    X = rng.uniform(0.0, 1.0, (1 if kind == "one" else 300, dim))
    if kind == "corner":
        X *= 0.1
    nrm = rng.standard_normal(X.shape)
    nrm /= np.linalg.norm(nrm, axis=1, keepdims=True)
    return _spec_like(dim, n, tuple(L), (0.0,) * dim, X * L, nrm, np.full(len(X), 1e-3))


@pytest.mark.parametrize("kind", ["one", "corner", "all"])
@pytest.mark.parametrize("n", [(16, 16), (1024, 64), (2048, 32), (8192, 16), (16, 16, 16), (64, 16, 32), (1024, 16, 16)])
def test_counts_behind_new_markers(n, kind):
    a, b = _spec(n, "all", 1), _spec(n, kind, 2)
    m = b.markers
    if len(a.markers.X) != len(m.X):
        a = _spec(n, kind, 3)
    t = lambda v: torch.as_tensor(v, device="cuda")
    with make_problem(a, "fp64") as pr:
        for spec in (a, b, a):
            s = spec.markers
            pr.set_markers(t(s.X), t(s.nrm), t(s.ds))
            nbusy, nact, nseg, tile, _ = _tiles_reference(spec)
            assert (pr.spread_tiles()[:2], pr.active_rows()[0]) == ((nbusy, nseg), nact)
            assert pr.spread_tiles()[2][:len(n)] == tile


def test_during_a_capture():
    spec = _spec((64, 64), "all", 4)
    nbusy, _, nseg, _, _ = _tiles_reference(spec)
    x = torch.zeros(256, device="cuda")
    with make_problem(spec, "fp64") as pr:
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            y = x + 1.0
            got = pr.spread_tiles()
        assert got[:2] == (nbusy, nseg)
        for k in range(3):
            x.fill_(k)
            g.replay()
            torch.cuda.synchronize()
            assert torch.all(y == k + 1.0)
