"""The rank-1 sweep on finite vectors whose sums overflow FP64: no cell's value
is a number, so the first cell is returned, with its labels k_0."""
import numpy as np
import pytest

from test_gpu_rank1 import lrqo_mod  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,K", [(64, 3), (1000, 2), (30_000, 5)])
def test_sums_that_overflow(lrqo_mod, n, K):  # noqa: F811
    # every term's parts are of one size and either sign, so a sum of two of
    # them overflows and a sum of two infinities is not a number
    rng = np.random.default_rng(n)
    theta = rng.uniform(0.0, 2.0 * np.pi, n)
    q = 1.2e308 * (np.cos(theta) + 1j * np.sin(theta))
    z, res = lrqo_mod.solve_rank1(torch.from_numpy(q).cuda(), K)
    assert not res.sweep_obj < np.inf                   # an infinity or not a number
    assert res.best_cell == 0
    t = np.arctan2(q.imag, q.real)
    x = K * t / (2.0 * np.pi)
    clear = np.abs(x - np.rint(x)) > 1e-9
    assert np.array_equal(z.cpu().numpy()[clear], np.mod(np.floor(x), K).astype(np.uint8)[clear])
