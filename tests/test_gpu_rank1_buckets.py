"""The rank-1 sweep's bucket form at the edges of its plan, and the inputs
that leave it for the general form, against the FP64 reference (the bars are
those of test_gpu_rank1: the cell and the labels are the reference's wherever
its best cell is separated by more than the summation bound)."""
import numpy as np
import pytest

from paper_2602_20376_amd import inputs
from test_gpu_rank1 import _check, _clustered, lrqo_mod  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# one tile and bucket to two (512 points), the least n with 256 buckets, the
# most tiles, buckets of 512 to 2,048 points, more than 256 buckets
SIZES = [(511, 3), (512, 2), (513, 3), (1025, 8), (65_537, 3), (130_561, 3), (262_145, 4), (300_001, 255),
         (524_289, 3), (1_048_577, 2)]


@pytest.mark.parametrize("n,K", SIZES)
def test_plan_edges(lrqo_mod, n, K):  # noqa: F811
    res = _check(lrqo_mod, inputs.random_V(n, 1, 900 + n % 97 + K)[:, 0], K)
    assert res.sort_passes == 4


def _phases(kind, n, rng):
    if kind == "one point":                     # every point the same: one bucket, one bin, coordinate order
        return np.zeros(n)
    if kind == "few points":
        return rng.integers(0, 5, n) * 0.37
    if kind == "narrow":                        # one bucket beyond its capacity (n = 20,000) or a bin beyond its own
        return rng.uniform(0.2, 0.2 + 1e-4, n)
    return np.concatenate([rng.uniform(-np.pi, np.pi, n - 40), np.full(40, 0.3)])   # a run of 40 equal points


@pytest.mark.parametrize("kind", ["one point", "few points", "narrow", "equal run"])
@pytest.mark.parametrize("n", [300, 20_000])
def test_uneven_points(lrqo_mod, kind, n):  # noqa: F811
    rng = np.random.default_rng(len(kind) + n)
    q = rng.uniform(0.5, 2.0, n) * np.exp(1j * _phases(kind, n, rng))
    res = _check(lrqo_mod, rng.permutation(q), 3)
    assert res.sort_passes >= 4


@pytest.mark.parametrize("size,exact_sort", [(16, False), (17, True)])
def test_run_limit_among_many(lrqo_mod, size, exact_sort):  # noqa: F811
    q = np.concatenate([_clustered(40, size, 5 + size, 3), inputs.random_V(70_000, 1, 9)[:, 0]])
    assert (_check(lrqo_mod, q, 3).sort_passes > 4) == exact_sort


def test_beyond_the_bucket_form(lrqo_mod):  # noqa: F811
    n = 2 ** 24 + 1
    rng = np.random.default_rng(24)
    _check(lrqo_mod, rng.standard_normal(n) + 1j * rng.standard_normal(n), 3)


def test_nonfinite_among_many(lrqo_mod):  # noqa: F811
    q = torch.ones(70_000, dtype=torch.complex128, device="cuda")
    q[69_999] = complex(0.0, float("nan"))
    with pytest.raises(lrqo_mod.LrqoError, match="ENOTFINITE"):
        lrqo_mod.solve_rank1(q, 3)
