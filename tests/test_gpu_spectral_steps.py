"""Lanczos driver at the edges of its step loop: spaces that end early
(complete graphs, tiny graphs), the last permitted step, checks at every step
or seldom, several column groups and partial counts in the Gram-Schmidt
kernels, partial column stripes of W, and scratch too small for the finer
split of its tiles.  Bars: those of test_gpu_spectral; runs that differ only
in when they check agree to 1e-9 (one converged earlier than the other, both
at tol 1e-12)."""
import numpy as np
import pytest

from oracle import spectral
from paper_2602_20376_amd import inputs
from test_gpu_spectral import _dev_graph, lrqo_mod  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,r", [(5, 1), (6, 2), (64, 2), (300, 1)])
def test_space_that_ends_early(lrqo_mod, n, r):  # noqa: F811
    """L of the complete graph has the eigenvalues 0 and n: the Krylov space
    ends after two steps."""
    i, j = np.triu_indices(n, 1)
    V, res = lrqo_mod.laplacian_factor(*_dev_graph(n, i, j, None), r)
    assert res.converged == 1 and res.iterations <= 3
    assert abs(res.eigenvalues[0] - n) <= 1e-10 * n
    if r == 2:
        assert abs(res.eigenvalues[1]) <= 1e-9 * n
    Vg = V.cpu().numpy()
    assert abs(np.linalg.norm(Vg[:, 0]) - np.sqrt(n)) <= 1e-9 * np.sqrt(n)


@pytest.mark.parametrize("n,m,r", [(7, 12, 3), (257, 900, 4), (1025, 5000, 2)])
def test_check_interval_does_not_change_the_pairs(lrqo_mod, n, m, r):  # noqa: F811
    i, j = inputs.random_edges(n, m, 7 + n)
    g = _dev_graph(n, i, j, None)
    lam, _ = spectral.top_factor(spectral.laplacian_dense(n, (i, j, np.ones(m))), r)
    got = [lrqo_mod.laplacian_factor(*g, r, tol=1e-12, max_iter=min(n, 400), check_every=e) for e in (1, 7, 400)]
    for V, res in got:
        assert res.converged == 1
        assert np.allclose(np.array(res.eigenvalues[:r]), lam, rtol=1e-10, atol=1e-10 * lam[0])
    steps = [res.iterations for _, res in got]
    assert steps[0] <= steps[1] <= steps[2]


def test_last_step_without_convergence(lrqo_mod):  # noqa: F811
    i, j = inputs.random_edges(2000, 9000, 3)
    g = _dev_graph(2000, i, j, None)
    _, res = lrqo_mod.laplacian_factor(*g, 2, tol=1e-13, max_iter=11, check_every=4)
    assert (res.iterations, res.converged) == (11, 0)


@pytest.mark.parametrize("n", [1, 2, 255, 257, 600])
def test_phase_sync_partial_stripes(lrqo_mod, n):  # noqa: F811
    rng = np.random.default_rng(n)
    U = np.exp(1j * rng.uniform(0.0, 2.0 * np.pi, (n, 2)))
    sigma, r = 0.5 * np.sqrt(n), min(2, n)
    V, res = lrqo_mod.phase_sync_factor(torch.from_numpy(U).cuda(), sigma, 91, r, tol=1e-10, max_iter=200)
    Q = spectral.phase_sync_matrix(U, sigma, 91)
    lam = np.sort(np.linalg.eigvalsh(Q))[::-1][:r]
    assert np.allclose(np.array(res.eigenvalues[:r]), lam, rtol=1e-5, atol=1e-5 * max(abs(lam[0]), 1.0))


def test_phase_sync_at_the_scratch_limit(lrqo_mod, monkeypatch):  # noqa: F811
    """The smallest scratch that is accepted serves the coarse split of the
    tiles, with the same factor up to summation order."""
    n = 1500
    U = torch.from_numpy(np.exp(1j * np.random.default_rng(4).uniform(0.0, 2.0 * np.pi, (n, 3)))).cuda()
    run = lambda: lrqo_mod.phase_sync_factor(U, 0.5 * np.sqrt(n), 5, 3, tol=1e-9, max_iter=60)[0]  # noqa: E731
    free = run()
    lo, hi = 1 << 16, 1 << 26
    while hi - lo > 256:
        mid = (lo + hi) // 2
        monkeypatch.setenv("LRQO_ARENA_LIMIT", str(mid))
        try:
            last = run()
            hi = mid
        except lrqo_mod.LrqoError as e:
            assert "LRQO_ENOMEM" in str(e)
            lo = mid
    assert torch.max(torch.abs(last - free)) <= 1e-9 * torch.max(torch.abs(free))
