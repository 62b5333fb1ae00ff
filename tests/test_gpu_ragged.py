"""Ragged heads at the sizes where the split of the work can go wrong: every row-tile height (1, 2, 4, 8 and a
remainder), column counts around the powers of two that set how many k rows a wavefront reads at once, k counts
below, at and just past what the sixteen wavefronts take in one go.  Integer-coded: every sum is exact, so the
result must match bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 8, 9])
@pytest.mark.parametrize("K", [1, 15, 129, 1025])
def test_ragged_edges(oracle, N, K, dtype):
    import paper_2009_13062_amd as nf
    rng = np.random.default_rng(1000 * N + K)
    nout = [1, 2, 3, 31, 32, 33, 64, 65, 129]
    M = len(nout)
    X = rng.integers(-2, 3, (M, N, K)).astype(np.float32)
    Ws = [rng.integers(-1, 2, (K, n)).astype(np.float32) for n in nout]
    bs = [rng.integers(-4, 5, n).astype(np.float32) for n in nout]
    ref = oracle.linear_ragged(X, Ws, bs, out_bf16=dtype == torch.bfloat16)
    dev = lambda a, dt: torch.from_numpy(np.ascontiguousarray(a)).to("cuda", dt)
    Y = nf.linear_ragged(dev(X, dtype), dev(np.concatenate([w.ravel() for w in Ws]), dtype), nout,
                         bias=dev(np.concatenate(bs), torch.float32))
    for m, y in enumerate(nf.ragged_views(Y, N, nout)):
        assert np.array_equal(y.float().cpu().numpy(), ref[m]), (m, nout[m])
