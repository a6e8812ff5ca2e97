"""GPU parity of the matrix-core scorer from split FP32 values (K = 2, 3, 4, 8,
16, 2 <= r <= 4, n >= 2,048) against the FP64 oracle, at the edges of its tiles
(32-row blocks, 256-row tiles, 256-candidate blocks, row slices), over both
layouts of V and factors of uneven scale.

Bars.  Labels: w is a sum of at most 48 exact F16 products, charged one FP32
ulp (2u) per addition, plus at most 3u for the parts left out, and a quantiser
test's error over the distance to its line is at most 1.42, so a label can
differ from the FP64 rule's only within 1.42 (2 * 48 + 3) u < REACH_PRECISION.
Scores: s is summed exactly from V rounded to 2^-30 of its largest entry, so
an entry is off by at most 2^-31 vmax; a component of s is rounded to FP32
once per slice and once per addition of slices (P of them), f adds 2r
products, and the magnitudes of the K = 16 roots are rounded to 2^-23 (at most
2^-23.9 off: 1.1 u on each part of z, below 1.6 u sum_i |V_ij| on a component).
|f32 - f| <= 2 ||s|| dq + dq^2 + (4 P + 4 r + 4) u f with
dq = n 2^-30 vmax sqrt(2 r) (+ 1.6 u ||(sum_i |V_ij|)_j|| for K = 16), where no
row lies within the reach."""
import numpy as np
import pytest

import parity_helpers as PH
from paper_2602_20376_amd import inputs
from test_gpu_sampled import check_result, lrqo_mod, solve_checked  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = [
    # n, r, K, S, real, scale of the rows
    (2048, 2, 3, 1, False, "even"),
    (2049, 3, 3, 257, True, "even"),
    (2079, 4, 4, 255, True, "even"),
    (2335, 2, 4, 300, False, "even"),
    (4113, 3, 2, 513, False, "even"),
    (9001, 4, 3, 700, False, "even"),
    (5151, 3, 4, 256, False, "even"),
    (50021, 2, 3, 300, True, "even"),
    (2048, 3, 8, 256, False, "even"),
    (2081, 2, 8, 257, True, "even"),
    (7000, 4, 8, 300, False, "even"),
    (2050, 4, 16, 255, True, "even"),
    (2303, 3, 16, 513, False, "even"),
    (9000, 4, 16, 300, False, "uneven"),
    (2200, 2, 16, 300, False, "even"),
    (3000, 3, 3, 400, True, "uneven"),
    (3001, 4, 2, 400, False, "huge"),
    (3002, 3, 4, 400, True, "tiny"),
]


def _factor(n, r, real, scale, seed):
    V = inputs.random_V(n, r, seed, real=real)
    if scale == "uneven":      # rows over six decades, exact zeros among them
        V = V * 10.0 ** np.random.default_rng(seed).uniform(-6.0, 0.0, (n, 1))
        V[::17] = 0.0
    if scale == "huge":
        V = V * 2.0 ** 45
    if scale == "tiny":
        V = V * 2.0 ** -50
    return PH.fp32_exact(V)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,r,K,S,real,scale", CASES)
def test_split_parity(lrqo_mod, n, r, K, S, real, scale, precision):  # noqa: F811
    seed = 5100 + n + r + K
    V = _factor(n, r, real, scale, seed)
    out, f32, dirs, probe, labels = solve_checked(lrqo_mod, V, K, S, seed, real=real, precision=precision)
    check_result(V, K, S, seed, out, real=real, f32=f32, dirs=dirs, probe=probe, labels=labels,
                 reach=PH.REACH_PRECISION)
    ref = PH.check_scores(V, K, dirs, f32, reach=PH.REACH_PRECISION)
    f, clean = ref["f"], ref["nambig"] == 0
    dq = n * 2.0 ** -30 * max(np.abs(V.real).max(), np.abs(V.imag).max()) * np.sqrt(2.0 * r)
    if K == 16:
        dq += 1.6 * PH.U32 * np.linalg.norm(np.sum(np.abs(V), axis=0))
    tol = 2.0 * np.sqrt(f) * dq + dq * dq + (4 * out.slices + 4 * r + 4) * PH.U32 * f
    assert np.all(np.abs(f32 - f)[clean] <= tol[clean]), float(np.max(np.abs(f32 - f)[clean] / tol[clean]))


def test_split_ranges_lists_and_strides(lrqo_mod):  # noqa: F811
    """Index ranges merge to the whole, an explicit list of the stream's own
    directions scores bit for bit as the stream (scaled by a power of two as
    well: labels do not depend on the length of c), a transposed V as a copy of
    it, and the allocation-free entry point as the plain one."""
    n, r, K, S = 2600, 3, 3, 1300
    V = torch.from_numpy(inputs.random_V(n, r, 77).astype(np.complex64)).cuda()
    f = torch.empty(S, dtype=torch.float32, device="cuda")
    d = torch.empty((S, 2 * r), dtype=torch.float32, device="cuda")
    whole = lrqo_mod.solve_sampled(V, K, S, 9, f_out=f, dirs_out=d)
    parts = [lrqo_mod.solve_sampled(V, K, 325, 9, first_index=325 * q) for q in range(4)]
    best = max(parts, key=lambda o: (o.obj, -o.best_index))
    assert (best.best_index, best.obj) == (whole.best_index, whole.obj)
    for kw in ({"directions": d}, {"directions": d * 4096.0}, {"noalloc": True}, {"strided": True}):
        Vs = V.T.contiguous().T if kw.pop("strided", False) else V
        g = torch.empty(S, dtype=torch.float32, device="cuda")
        out = lrqo_mod.solve_sampled(Vs, K, S, 9, f_out=g, **kw)
        assert torch.equal(f, g) and torch.equal(out.z, whole.z) and out.best_index == whole.best_index


def test_split_k16_fold(lrqo_mod):  # noqa: F811
    """One slice of more rows than the K = 16 planes may sum before they are
    folded (65,536): the scores of 64 candidates against the oracle."""
    n, r, K, S = 70_001, 2, 16, 64_000
    V = _factor(n, r, False, "even", 11)
    f = torch.empty(S, dtype=torch.float32, device="cuda")
    d = torch.empty((S, 2 * r), dtype=torch.float32, device="cuda")
    out = lrqo_mod.solve_sampled(torch.from_numpy(V.astype(np.complex64)).cuda(), K, S, 3, f_out=f, dirs_out=d)
    assert out.slices == 1
    pick = np.r_[0:32, S - 32:S]
    dirs = PH.dirs_complex(d.cpu().numpy()[pick], r)
    ref = PH.check_scores(V, K, dirs, f.cpu().numpy()[pick], reach=PH.REACH_PRECISION)
    assert ref["max_ratio"] < 1.0
