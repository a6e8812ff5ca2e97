"""The one-block end of small sampled solves (selection, FP64 values, pick and
labels together) at the edges of its range, and just beyond it: against the
same steps in FP64 from the scores and directions the call reports.

The kept candidates are the FP32 scores' top T (descending, lower index first),
exactly; the objective is FP64 over at most 257 rows, so 1e-12 relative bounds
its rounding, and the pick may differ only among candidates within it."""
import numpy as np
import pytest

import oracle
from paper_2602_20376_amd import inputs
from parity_helpers import dirs_complex

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# rows around a wave, the block of one row a thread and one more; scores
# around a tile, a tile per wave, and the end of the range
CASES = [(1, 1, 3, 1, False, 64), (63, 2, 4, 5, False, 64), (64, 2, 4, 1024, False, 64), (65, 3, 8, 1025, False, 7),
         (255, 4, 16, 8192, False, 64), (256, 4, 3, 8191, True, 64), (257, 2, 3, 8192, True, 64),
         (256, 3, 5, 8193, False, 1), (200, 1, 2, 64, True, 64), (130, 4, 7, 65, True, 33),
         (64, 2, 255, 4096, False, 64), (64, 4, 5, 300, True, 64), (65, 4, 5, 300, True, 64), (256, 1, 16, 1023, True, 64)]


@pytest.mark.parametrize("n,r,K,S,real,topk", CASES)
def test_small_solve(n, r, K, S, real, topk):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_20376_amd import lrqo

    V = inputs.random_V(n, r, 60 + n + r, real=real)
    Vt = torch.from_numpy(V.real.astype(np.float32) if real else V.astype(np.complex64)).cuda()
    V = Vt.cpu().numpy().astype(np.complex128)
    f = torch.empty(S, dtype=torch.float32, device="cuda")
    dirs = torch.empty((S, 2 * r), dtype=torch.float32, device="cuda")
    out = lrqo.solve_sampled(Vt, K, S, 11 * n + S, topk=topk, f_out=f, dirs_out=dirs)
    f32, c = f.cpu().numpy(), dirs_complex(dirs.cpu().numpy(), r)
    kept = np.lexsort((np.arange(S), -f32.astype(np.float64)))[:min(topk, S)]
    vals = np.empty(kept.size)
    near = np.empty(kept.size, dtype=bool)
    for t, i in enumerate(kept):
        z, dist = oracle.labels(V, K, c[i])
        vals[t] = oracle.objective(V, K, z)
        near[t] = np.min(dist) < 1e-9
    assert out.best_index in kept
    at = int(np.nonzero(kept == out.best_index)[0][0])
    if not near.any():
        assert vals[at] >= vals.max() * (1 - 1e-12)
        assert abs(out.obj - vals[at]) <= 1e-12 * vals[at]
        z, _ = oracle.labels(V, K, c[out.best_index])
        assert np.array_equal(out.z.cpu().numpy(), z)
    assert out.fp32_obj == float(f32[out.best_index])


def test_nonfinite_is_reported():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_20376_amd import lrqo

    V = torch.from_numpy(inputs.random_V(64, 2, 3).astype(np.complex64)).cuda()
    V[63, 1] = complex(float("inf"), 0.0)
    with pytest.raises(lrqo.LrqoError, match="ENOTFINITE"):
        lrqo.solve_sampled(V, 4, 1024, 1)
