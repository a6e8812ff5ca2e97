"""Greedy refinement at the edges of its row groups: rows shorter and longer
than the sixteen lanes of a group (several trips), vertices without entries,
vertex counts around a wave's sixteen and a block's 128 vertices, and moves
that go on over several batches of rounds.  Bar: bit-exact with the oracle's
rounds (unit and small whole weights, K <= 4: whole numbers in FP64)."""
import numpy as np
import pytest

from oracle import graph as og
from test_gpu_graph import _device_graph, _edges, lrqo_mod  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _hub_edges(n, seed):
    """A sparse graph with a few hubs joined to a third of all vertices, and
    its last vertices isolated."""
    rng = np.random.default_rng(seed)
    m = max(1, n - 3)
    pairs = {(min(a, b), max(a, b)) for a, b in rng.integers(0, m, (2 * n, 2)).tolist() if a != b}
    for hub in range(min(3, m)):
        pairs |= {(min(hub, v), max(hub, v)) for v in rng.choice(m, m // 3, replace=False).tolist() if v != hub}
    i, j = np.array(sorted(pairs), dtype=np.int64).reshape(-1, 2).T
    return i, j


@pytest.mark.parametrize("n", [4, 15, 17, 127, 129, 700])
@pytest.mark.parametrize("K", [2, 3, 4])
@pytest.mark.parametrize("weighted", [False, True])
def test_rows_of_every_length(lrqo_mod, n, K, weighted):  # noqa: F811
    i, j = _hub_edges(n, 11 * n + K)
    if i.size == 0:
        pytest.skip("no edges")
    w = np.random.default_rng(n).integers(1, 4, i.size).astype(np.float64) if weighted else None
    rp, col, wd = _device_graph(n, i, j, w)
    z0 = np.random.default_rng(n + K).integers(0, K, n)
    for every in (1, 0):
        zd = torch.from_numpy(z0.astype(np.uint8)).cuda()
        res = lrqo_mod.refine_greedy(rp, col, wd, K, zd, check_every=every)
        zo, rounds, moves = og.greedy(n, _edges(i, j, w), K, z0)
        assert np.array_equal(zd.cpu().numpy(), zo)
        assert (res.rounds, res.moves, res.converged) == (rounds, moves, 1)
