"""Loss and gradient of a training step at the edges of the row kernels'
tiles: 32-row tiles of the backward pass, 64-row halves and 256-row items of
the forward pass, several instances in one wave's run of tiles, and more tiles
than waves.  Bar: that of test_gpu_proposal (FP32 kernels against the FP64
derivatives: loss 1e-5, gradient 1e-4 relative; every parameter block 1e-3)."""
import numpy as np
import pytest

from oracle import proposal as P
from paper_2602_20376_amd import inputs
from test_gpu_proposal import K, _cpu_loss_grad, _fp32, lrqo_mod  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("sizes", [[4], [31, 32, 33], [64, 65, 5, 255, 256, 257], [40] * 70, [70_001]])
def test_gradient_at_tile_edges(lrqo_mod, sizes):  # noqa: F811
    from paper_2602_20376_amd import proposal as drv

    Vs = [_fp32(inputs.phase_sync_factor(n, 3, 900 + t)) for t, n in enumerate(sizes)]
    rng = np.random.default_rng(len(sizes))
    cs = inputs.complex_gaussian(rng, (len(sizes), 3))
    cs /= np.linalg.norm(cs, axis=1, keepdims=True)
    theta = inputs.proposal_init(7)
    prop = lrqo_mod.Proposal(theta, K)
    cat, offs, ns = drv.pack_factors(Vs)
    L, g = prop.train_step(torch.from_numpy(cat).cuda(), offs, ns, drv.targets_real(cs), 0.0, update=False,
                           want_grad=True)
    L0, g0 = _cpu_loss_grad(theta.astype(np.float32).astype(np.float64), Vs, cs)
    assert abs(L - L0) <= 1e-5 * abs(L0), (L, L0)
    assert np.linalg.norm(g - g0) <= 1e-4 * np.linalg.norm(g0)
    o = 0
    for name, shp in P.PARAM_SHAPES:
        k = int(np.prod(shp))
        assert np.linalg.norm(g[o:o + k] - g0[o:o + k]) <= 1e-3 * np.linalg.norm(g0[o:o + k]) + 1e-7, name
        o += k
