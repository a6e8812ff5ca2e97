"""The enumeration's block-relative unranking and nested label combinations at
the edges: as few rows as a set needs, chunks that end inside a block, ranks
where a higher row of the set moves on, sets with a double group beside sets
without.  Every chunking scores the same sets, so the objective, labels and
counts are the same numbers; small sizes are also held to the brute force."""
import numpy as np
import pytest

from oracle import brute
from paper_2602_20376_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,r,K,real", [(3, 2, 2, False), (4, 2, 2, False), (5, 3, 2, False), (2, 1, 2, False),
                                        (5, 2, 3, True), (7, 2, 4, False), (6, 3, 3, False), (7, 4, 2, False),
                                        (24, 2, 3, True), (24, 2, 5, False)])
def test_every_chunking_agrees(n, r, K, real, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_20376_amd import lrqo

    V = inputs.random_V(n, r, 40 * n + r + K, real=real)
    Vt = torch.from_numpy(np.ascontiguousarray(V, dtype=np.complex128)).cuda()
    monkeypatch.setenv("LRQO_EXACT_FORM", "fused")
    seen = None
    for chunk in ("", "1" if n < 8 else "63", "255", "257"):
        if chunk:
            monkeypatch.setenv("LRQO_EXACT_CHUNK", chunk)
        z, res = lrqo.solve_exact(Vt, K)
        now = (res.obj, res.index_sets, res.rank_deficient, res.candidates, z.cpu().numpy().tolist())
        assert seen is None or now == seen, chunk
        seen = now
    if n < 8:
        opt, _, _ = brute.brute_force(V, K)
        assert abs(seen[0] - opt) <= 1e-12 * opt
