"""Lists of directions beyond the range of the matrix-core scorer's F16 parts
(axes, components far apart in size, directions that round whole columns to a
tie, zero, NaN): such a list is scored in FP32, to the FP32 bars of
parity_helpers; a list of ordinary directions is scored as the stream is."""
import numpy as np
import pytest

import parity_helpers as PH
from paper_2602_20376_amd import inputs
from test_gpu_sampled import lrqo_mod  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _solve(lrqo_mod, V, K, c, real, **kw):
    S, r = c.shape
    d = torch.from_numpy(np.ascontiguousarray(np.stack([c.real, c.imag], axis=2).reshape(S, 2 * r).astype(np.float32))).cuda()
    Vd = torch.from_numpy(np.ascontiguousarray(V.astype(np.complex64))).cuda()
    Vd = Vd.real.contiguous() if real else Vd
    f = torch.empty(S, dtype=torch.float32, device="cuda")
    out = lrqo_mod.solve_sampled(Vd, K, S, 0, real=real, directions=d, f_out=f, **kw)
    return out, f.cpu().numpy(), PH.dirs_complex(d.cpu().numpy(), r)


def _directions(r, small, rng, S=40):
    c = rng.standard_normal((S, r)) + 1j * rng.standard_normal((S, r))
    c /= np.linalg.norm(c, axis=1, keepdims=True)
    c[1::2, 0] *= small                       # every other one nearly or wholly without column 0
    return c


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,r,K,real,small", [(2048, 2, 3, True, 0.0), (3000, 2, 16, False, 0.0), (2500, 3, 4, False, 1e-9),
                                              (70_000, 2, 4, True, 0.0), (2304, 4, 8, True, 1e-6), (4000, 3, 2, False, 0.0)])
def test_axis_lists(lrqo_mod, n, r, K, real, small, precision):  # noqa: F811
    """Rows that lie on column 0 but for entries near 1e-13: at a direction
    without column 0 their labels come from those entries alone."""
    rng = np.random.default_rng(n + K)
    V = inputs.random_V(n, r, n, real=real)
    V[: n // 2, 1:] *= 1e-13
    V = PH.fp32_exact(V)
    out, f, c = _solve(lrqo_mod, V, K, _directions(r, small, rng), real, precision=precision)
    ref = PH.check_scores(V, K, c, f)
    assert out.obj >= np.max(ref["f"]) * (1.0 - 1e-5)


@pytest.mark.parametrize("K,real", [(3, True), (4, False)])
def test_list_with_nan_and_zero(lrqo_mod, K, real):  # noqa: F811
    n, r = 2100, 3
    V = PH.fp32_exact(inputs.random_V(n, r, 3, real=real))
    c = _directions(r, 1.0, np.random.default_rng(8))
    c[3] = np.nan
    c[5] = 0.0
    c[7] = np.inf
    out, f, c = _solve(lrqo_mod, V, K, c, real)
    good = np.setdiff1d(np.arange(len(c)), [3, 5, 7])
    assert np.all(np.isfinite(f[good]))
    zero_f = float(np.sum(np.abs(np.sum(V, axis=0)) ** 2))          # every label 0
    assert abs(f[5] - zero_f) <= PH.accumulation_allowance(V, zero_f)
    if not np.isfinite(out.obj) or out.best_index in (3, 7):
        pytest.fail(f"a direction that is not finite was picked: {out.best_index}")
    PH.check_scores(V, K, c[good], f[good])


@pytest.mark.parametrize("K,angle", [(3, 0.0), (3, np.pi), (2, np.pi / 2), (4, np.pi / 4), (4, -np.pi / 4)])
def test_list_on_a_boundary(lrqo_mod, K, angle):  # noqa: F811
    """Real V and directions of one phase, so that rows of one sign lie exactly
    on a boundary: the same labels as the FP32 scorer gives the same rows where
    n is too small for the matrix core."""
    n, r = 2304, 2
    V = PH.fp32_exact(inputs.random_V(n, r, 4, real=True))
    u = np.exp(1j * angle)
    u = complex(np.float32(u.real) * (abs(u.real) > 1e-9), np.float32(u.imag) * (abs(u.imag) > 1e-9))
    if K == 4:
        u = complex(np.copysign(np.float32(0.70710677), u.real), np.copysign(np.float32(0.70710677), u.imag))
    c = np.random.default_rng(1).uniform(0.3, 1.0, (8, r)) * u
    c = c / np.linalg.norm(c, axis=1, keepdims=True)
    c = c.real.astype(np.float32) + 1j * c.imag.astype(np.float32)
    if K == 4:
        c = np.abs(c.real) * complex(np.sign(u.real), np.sign(u.imag))
    c = np.concatenate([c, _directions(r, 1.0, np.random.default_rng(2), 4)])

    def labels(rows):
        S = len(c)
        d = torch.from_numpy(np.ascontiguousarray(np.stack([c.real, c.imag], axis=2).reshape(S, 2 * r).astype(np.float32))).cuda()
        lab = torch.empty((S, len(rows)), dtype=torch.uint16, device="cuda")
        # complex storage: K = 2 takes the matrix core there
        lrqo_mod.solve_sampled(torch.from_numpy(np.ascontiguousarray(rows.astype(np.complex64))).cuda(), K, S, 0,
                               directions=d, probe=list(range(S)), probe_labels=lab)
        return lab.cpu().numpy()

    assert np.array_equal(labels(V), np.concatenate([labels(V[:1152]), labels(V[1152:])], axis=1))
