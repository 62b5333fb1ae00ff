"""Ragged heads at the sizes where the split of the work can go wrong: every row-tile height (1, 2, 4, 8 and a
remainder), column counts around the powers of two that set how many k rows a wavefront reads at once, k counts
below, at and just past what the wavefronts take in one go and either side of where there are 16 instead of 4.  Integer-coded: every sum is exact, so the
result must match bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 8, 9])
@pytest.mark.parametrize("K", [1, 15, 32, 33, 129, 1025])
def test_ragged_edges(oracle, N, K, dtype):
    edges(oracle, [1, 2, 3, 31, 32, 33, 64, 65, 129], N, K, dtype)


@pytest.mark.parametrize("N,K", [(1023, 40), (1024, 40), (1025, 129)])
def test_ragged_many_rows(oracle, N, K):
    edges(oracle, [1, 5, 65], N, K, torch.bfloat16)


def edges(oracle, nout, N, K, dtype):
    import paper_2009_13062_amd as nf
    rng = np.random.default_rng(1000 * N + K)
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


def test_many_rows_of_short_k_are_bound_by_the_output():
    """4096 rows of 8 k and 1000 outputs: six to seven times as long as moving the outputs, not what sixteen wavefronts
    per eight rows take for a k that four can share (22 times)."""
    import paper_2009_13062_amd as nf
    from test_gpu_f32 import us
    M, N, K, n = 4, 4096, 8, 1000
    bf = lambda *s: torch.randn(*s, device="cuda").bfloat16()
    X, W, Y, dst = bf(M, N, K), bf(M * K * n), bf(M * N * n), bf(N, M * n)
    copy = us(lambda: nf.merge_transpose(Y.view(M, N, n), M, True, out=dst))
    head = us(lambda: nf.linear_ragged(X, W, [n] * M, out=Y))
    assert head < 12 * copy, (head, copy)
