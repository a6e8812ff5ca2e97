"""GPU parity of the matrix-core scorer on factors whose rows differ in size by
many powers of two (a few hub rows over small ones, sizes that change along the
rows, columns of different size), against the FP64 oracle.

Bar.  In a tile of 256 rows column j of V enters in fixed point: with e the
exponent of its largest entry there, an entry is off by at most 2^(e - 26), so
a component of s by at most d_j = sqrt(2) 2^-26 sum_i 2^e(tile of i, j); s is
rounded to FP32 once per slice and once per addition of slices (P of them), f
adds 2r products, and no part of a root is off by more than u:
|f32 - f| <= 2 ||s|| d + d^2 + (4 P + 4 r + 4) u f with
d = sqrt(2) ||(d_j + u sum_i |V_ij|)_j||, for every labelling that differs from
the FP64 rule's within the reach only."""
import numpy as np
import pytest

import oracle
import parity_helpers as PH
from paper_2602_20376_amd import inputs
from test_gpu_sampled import lrqo_mod, solve_checked  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu
pytest.importorskip("torch")

TILE = 256


def _factor(kind, n, r, real, seed):
    rng = np.random.default_rng(seed)
    V = inputs.random_V(n, r, seed, real=real)
    if kind == "hub":              # one row of order 1, the others of one sign near 1e-9
        V = 1e-9 * (1.0 + rng.random((n, r))) * (1.0 if real else np.exp(0.3j))
        V[n // 3] = 3.9 * np.array([1.0, 0.5, -0.25, 0.125])[:r]
    elif kind == "hubs":           # row sizes with a heavy tail
        V = V * np.minimum(rng.random((n, 1)) ** -3.0, 1e9)
    elif kind == "steps":          # sizes that fall and rise along the rows, zero tiles among them
        V = V * 10.0 ** -np.abs(12.0 * np.sin(np.arange(n) / 1500.0))[:, None]
        V[3 * TILE:5 * TILE] = 0.0
    elif kind == "columns":        # columns that turn zero, and far smaller than the first
        V = V * 10.0 ** (-5.0 * np.arange(r))
        V[n // 2:, r - 1] = 0.0
    return PH.fp32_exact(V)


def _bar(V, f, slices):
    n, r = V.shape
    size = np.maximum(np.abs(V.real), np.abs(V.imag))
    tile = np.maximum.reduceat(size, np.arange(0, n, TILE), axis=0)
    unit = np.where(tile > 0.0, 2.0 ** np.floor(np.log2(np.where(tile > 0.0, tile, 1.0))), 0.0)
    d = np.sqrt(2.0) * 2.0 ** -26 * np.sum(np.repeat(unit, TILE, axis=0)[:n], axis=0) + PH.U32 * np.sum(np.abs(V), axis=0)
    d = np.sqrt(2.0) * np.linalg.norm(d)
    return 2.0 * np.sqrt(f) * d + d * d + (4 * slices + 4 * r + 4) * PH.U32 * f


@pytest.mark.parametrize("kind,n,r,K,real", [
    ("hub", 300_000, 2, 3, True),
    ("hub", 300_000, 3, 16, True),
    ("hub", 300_001, 2, 4, False),
    ("hubs", 20_000, 3, 3, True),
    ("hubs", 20_011, 4, 4, False),
    ("hubs", 9_000, 3, 2, False),
    ("steps", 30_000, 4, 3, True),
    ("steps", 30_100, 3, 8, False),
    ("steps", 12_345, 2, 16, False),
    ("columns", 5_000, 4, 3, False),
    ("columns", 5_100, 3, 16, True),
])
def test_scores_of_uneven_factors(lrqo_mod, kind, n, r, K, real):  # noqa: F811
    V = _factor(kind, n, r, real, 900 + n)
    out, f32, dirs, probe, labels = solve_checked(lrqo_mod, V, K, 96, 17, real=real, n_random_probes=2)
    ref = oracle.score_dirs(V, K, dirs, reach=PH.REACH_PRECISION)
    tol = _bar(V, ref["f"], out.slices)
    off = np.maximum(ref["lo"] - f32, f32 - ref["hi"]) / tol
    assert np.max(off) <= 1.0, float(np.max(off))
    for t, pos in enumerate(probe):
        PH.check_labels(V, K, dirs[pos], labels[t], PH.REACH_PRECISION)
    assert out.obj >= np.max(ref["f"]) * (1.0 - 1e-5)


def test_pieces_of_a_range_score_as_the_whole(lrqo_mod):  # noqa: F811
    """The scores of 2^22 directions, in one call and in two (one row slice
    each), bit for bit: the choice of the scorer does not depend on the length
    of the range."""
    torch = pytest.importorskip("torch")
    n, r, K, S = 2100, 2, 3, 1 << 22
    V = torch.from_numpy(inputs.random_V(n, r, 5).astype(np.complex64)).cuda()
    f = torch.empty(S, dtype=torch.float32, device="cuda")
    g = torch.empty(S, dtype=torch.float32, device="cuda")
    whole = lrqo_mod.solve_sampled(V, K, S, 3, f_out=f)
    parts = [lrqo_mod.solve_sampled(V, K, S // 2, 3, first_index=q * (S // 2), f_out=g[q * (S // 2):(q + 1) * (S // 2)])
             for q in range(2)]
    assert whole.slices == 1 and all(p.slices == 1 for p in parts)
    assert torch.equal(f, g)
    assert max(p.obj for p in parts) == whole.obj
