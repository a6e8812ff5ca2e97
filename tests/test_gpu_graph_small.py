"""Greedy refinement and objective on the smallest graphs (one group of
sixteen vertices, mostly empty): path, triangle and star with vertices that no
edge touches, one edge, and no edge at all.  Bar: bit-exact with the oracle."""
import numpy as np
import pytest

from oracle import graph as og
from test_gpu_graph import _device_graph, _edges, lrqo_mod  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

GRAPHS = {"edge": (2, [(0, 1)]), "path": (3, [(0, 1), (1, 2)]), "triangle and a vertex": (4, [(0, 1), (0, 2), (1, 2)]),
          "star and two vertices": (7, [(0, 1), (0, 3), (0, 4), (0, 6)]), "two vertices apart": (5, [(1, 4)])}


@pytest.mark.parametrize("name", sorted(GRAPHS))
@pytest.mark.parametrize("K", [2, 3, 4])
@pytest.mark.parametrize("weighted", [False, True])
def test_smallest_graphs(lrqo_mod, name, K, weighted):  # noqa: F811
    n, pairs = GRAPHS[name]
    i, j = np.array(pairs, dtype=np.int64).T
    w = np.arange(1, len(pairs) + 1, dtype=np.float64) if weighted else None
    rp, col, wd = _device_graph(n, i, j, w)
    for start in range(4):
        z0 = np.random.default_rng(start).integers(0, K, n) if start else np.zeros(n, dtype=np.int64)
        zd = torch.from_numpy(z0.astype(np.uint8)).cuda()
        res = lrqo_mod.refine_greedy(rp, col, wd, K, zd)
        zo, rounds, moves = og.greedy(n, _edges(i, j, w), K, z0)
        assert np.array_equal(zd.cpu().numpy(), zo)
        assert (res.rounds, res.moves, res.converged) == (rounds, moves, 1)


@pytest.mark.parametrize("n", [1, 4, 16, 17])
@pytest.mark.parametrize("K", [3, 6])
def test_no_edges(lrqo_mod, n, K):  # noqa: F811
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    col = torch.zeros(0, dtype=torch.int32, device="cuda")
    z = torch.from_numpy(np.random.default_rng(n).integers(0, K, n).astype(np.uint8)).cuda()
    before = z.clone()
    try:
        res = lrqo_mod.refine_greedy(rp, col, None, K, z)
    except lrqo_mod.LrqoError as e:
        pytest.fail(str(e))
    assert torch.equal(z, before)
    assert (res.rounds, res.moves, res.converged) == (0, 0, 1)
    assert (res.quad_before, res.quad_after, res.cut_before, res.cut_after) == (0.0, 0.0, 0.0, 0.0)
