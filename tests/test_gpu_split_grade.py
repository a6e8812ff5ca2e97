"""Grade of w in the matrix-core scorer, on rows set beside a decision boundary
of one candidate each.

At a distance of about u sum_j |V_ij||c_j| (u = 2^-24) its labels differ from the
FP64 rule's no more often than those of a chain of FP32 FMAs over the same FP32
V and c, which is emulated here (for K = 3 with Re w from c scaled by sqrt(3)
and rounded, and its test |Im w| <= sqrt(3) Re w).  Bar: the wrong labels of the
two forms are counts of independent rows, so the difference has a standard
deviation of at most sqrt(a + b); four of them.

From 64 u sum_j |V_ij||c_j| on (parity_helpers.REACH) they are the FP64 rule's:
the matrix core cuts the eight products with V1 c1 among them off at u of the
largest (8 u), rounds after every sixteen (3 u), the parts left out are below
2 u, and a quantiser's error over the distance to its line is at most 1.42
(sqrt(2) from parts to moduli): 1.42^2 13 u."""
import numpy as np
import pytest

from paper_2602_20376_amd import inputs
from test_gpu_sampled import lrqo_mod  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N, S = 1 << 18, 64
SQRT3 = np.float32(1.7320508075688772)


def _chain(terms):
    """FP32 FMA chain over FP64-exact products (FP64 addition, then rounded)."""
    acc = np.zeros(N, np.float32)
    for t in terms:
        acc = (acc.astype(np.float64) + t).astype(np.float32)
    return acc


def _labels(w, K):
    x = K * np.angle(w) / (2.0 * np.pi)
    return np.mod(np.floor(x + 0.5), K).astype(np.int64)


CASES = [(2, 3, True), (2, 8, True), (2, 16, True), (3, 3, True), (3, 4, True),
                                      (3, 8, True), (3, 16, True), (4, 3, True), (4, 4, True),
                                      (2, 2, False), (2, 3, False), (2, 4, False), (3, 2, False), (3, 3, False),
                                      (3, 4, False), (3, 8, False), (3, 16, False), (4, 2, False), (4, 3, False),
                                      (4, 16, False)]


def _beside(lrqo_mod, r, K, real, seed, steps):
    """Rows at about `steps` u sum_j |V_ij||c_j| from a boundary of candidate
    i mod S, those candidates, and which rows are usable."""
    rng = np.random.default_rng(seed)
    d = torch.empty((S, 2 * r), dtype=torch.float32, device="cuda")
    V0 = torch.from_numpy(inputs.random_V(2048, r, 1, real=real).astype(np.complex64)).cuda()
    lrqo_mod.solve_sampled(V0.real.contiguous() if real else V0, K, S, seed, real=real, dirs_out=d)
    d = d.cpu().numpy().astype(np.float64)
    c = (d[:, 0::2] + 1j * d[:, 1::2])[np.arange(N) % S]
    V = rng.standard_normal((N, r)) + (0.0 if real else 1j * rng.standard_normal((N, r)))
    V = V.astype(np.complex64).astype(np.complex128)
    turn = np.exp(-1j * np.pi * (2 * rng.integers(0, K, N) + 1) / K)   # a boundary to the positive real axis
    rest = np.imag(np.sum(V[:, 1:] * c[:, 1:], axis=1) * turn)
    fixed = rest if real else rest + V[:, 0].imag * np.imag(1j * c[:, 0] * turn)
    fixed = fixed + steps * 2.0 ** -24 * rng.choice([-1.0, 1.0], N) * np.sum(np.abs(V) * np.abs(c), axis=1)
    with np.errstate(divide="ignore", invalid="ignore"):
        x = (-fixed / np.imag(c[:, 0] * turn)).astype(np.float32).astype(np.float64)
    V[:, 0] = x + (0.0 if real else 1j * V[:, 0].imag)
    w = np.sum(V * c, axis=1)
    V[np.real(w * turn) < 0.0] *= -1.0
    use = np.abs(x) < 4.0
    V[~use] = 1.0
    return V, c, use


def _scorer_labels(lrqo_mod, V, K, real, seed, **kw):
    lab = torch.empty((S, N), dtype=torch.uint16, device="cuda")
    Vd = torch.from_numpy(np.ascontiguousarray(V.astype(np.complex64))).cuda()
    lrqo_mod.solve_sampled(Vd.real.contiguous() if real else Vd, K, S, seed, real=real, probe=list(range(S)),
                           probe_labels=lab, **kw)
    return lab.cpu().numpy()[np.arange(N) % S, np.arange(N)].astype(np.int64)


@pytest.mark.parametrize("r,K,real", CASES)
def test_labels_beside_a_boundary(lrqo_mod, r, K, real):  # noqa: F811
    seed = 70 + 10 * r + K
    V, c, use = _beside(lrqo_mod, r, K, real, seed, 0.0)
    w = np.sum(V * c, axis=1)
    got = _scorer_labels(lrqo_mod, V, K, real, seed)

    cr = [np.float32(SQRT3 * c[:, j].real.astype(np.float32)).astype(np.float64) if K == 3 else c[:, j].real for j in range(r)]
    ci = [np.float32(SQRT3 * c[:, j].imag.astype(np.float32)).astype(np.float64) if K == 3 else c[:, j].imag for j in range(r)]
    if real:
        wr = _chain([V[:, j].real * cr[j] for j in range(r)])
        wi = _chain([V[:, j].real * c[:, j].imag for j in range(r)])
    else:
        wr = _chain([t for j in range(r) for t in (-V[:, j].imag * ci[j], V[:, j].real * cr[j])])
        wi = _chain([t for j in range(r) for t in (V[:, j].imag * c[:, j].real, V[:, j].real * c[:, j].imag)])
    if K == 3:
        fp32 = np.where(np.abs(wi) <= wr, 0, np.where(np.signbit(wi), 2, 1))
    else:
        fp32 = _labels(wr.astype(np.float64) + 1j * wi.astype(np.float64), K)
    ref = _labels(w, K)
    a, b = int(np.sum((got != ref) & use)), int(np.sum((fp32 != ref) & use))
    print(f"r={r} K={K} real={real}: wrong of {int(use.sum())}: scorer {a}, FP32 chain {b}", flush=True)
    assert b > 1000
    assert a - b <= 4.0 * np.sqrt(a + b), (a, b)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("r,K,real", CASES)
def test_labels_outside_the_reach(lrqo_mod, r, K, real, precision):  # noqa: F811
    seed = 170 + 10 * r + K
    V, c, use = _beside(lrqo_mod, r, K, real, seed, 100.0)
    w = np.sum(V * c, axis=1)
    x = K * np.angle(w) / (2.0 * np.pi) - 0.5                       # distance to the nearest boundary ray
    dist = np.abs(w) * np.sin(np.minimum(np.abs(x - np.rint(x)) * 2.0 * np.pi / K, np.pi / 2.0))
    far = use & (dist >= 64.0 * 2.0 ** -24 * np.sum(np.abs(V) * np.abs(c), axis=1))
    got = _scorer_labels(lrqo_mod, V, K, real, seed, precision=precision)
    assert np.sum(far) > N // 2
    assert np.array_equal(got[far], _labels(w, K)[far]), int(np.sum((got != _labels(w, K)) & far))
