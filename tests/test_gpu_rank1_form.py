"""The form in which the rank-1 sweep ends: buckets at the edges of its plan,
the general sort for each way of leaving them (a bucket over its capacity, a
run of more than 16 equal images with distinct keys, n beyond 2^24), with the
results checked against the FP64 reference in both."""
import numpy as np
import pytest

from paper_2602_20376_amd import inputs
from test_gpu_rank1 import _check, _clustered, lrqo_mod  # noqa: F401 (fixture)
from test_gpu_rank1_buckets import SIZES, _phases

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,K", [(1, 3), (2, 2)] + SIZES)
def test_spread_points_stay_in_buckets(lrqo_mod, n, K):  # noqa: F811
    _check(lrqo_mod, inputs.random_V(n, 1, 900 + n % 97 + K)[:, 0], K)
    assert lrqo_mod.rank1_form() == 1


def _long_distinct_run(q, K):
    """Whether a run of more than 16 equal 32-bit images holds distinct FP64
    points, with the device's atan2 (its last bit differs from the host's)."""
    d = torch.from_numpy(q).cuda()
    x = K * torch.atan2(d.imag, d.real) / (2.0 * np.pi)
    phi = ((2.0 * np.pi / K) * ((0.5 + torch.floor(x)) - x)).cpu().numpy()
    image = np.floor((phi * K / (2.0 * np.pi) + 0.5) * 2.0 ** 32)
    values, counts = np.unique(image, return_counts=True)
    return any(np.unique(phi[image == v]).size > 1 for v in values[counts > 16])


@pytest.mark.parametrize("kind,n,fits", [("one point", 300, True), ("one point", 8192, True), ("one point", 8193, False),
                                         ("one point", 20_000, False), ("few points", 300, True),
                                         ("few points", 20_000, True), ("narrow", 300, True), ("narrow", 20_000, False),
                                         ("equal run", 300, True), ("equal run", 20_000, True)])
def test_form_of_uneven_points(lrqo_mod, kind, n, fits):  # noqa: F811
    rng = np.random.default_rng(len(kind) + n)
    q = rng.permutation(rng.uniform(0.5, 2.0, n) * np.exp(1j * _phases(kind, n, rng)))
    _check(lrqo_mod, q, 3)
    assert lrqo_mod.rank1_form() == int(fits and not _long_distinct_run(q, 3))


@pytest.mark.parametrize("size,form", [(16, 1), (17, 0)])
def test_form_of_close_runs(lrqo_mod, size, form):  # noqa: F811
    q = np.concatenate([_clustered(40, size, 5 + size, 3), inputs.random_V(70_000, 1, 9)[:, 0]])
    _check(lrqo_mod, q, 3)
    assert lrqo_mod.rank1_form() == form


def test_form_beyond_the_buckets(lrqo_mod):  # noqa: F811
    q = torch.ones(2 ** 24 + 1, dtype=torch.complex128, device="cuda")
    lrqo_mod.solve_rank1(q, 3)
    assert lrqo_mod.rank1_form() == 0
