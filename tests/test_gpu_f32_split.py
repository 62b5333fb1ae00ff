"""float32 matmul on bf16 matrix instructions: the edges of every tile (64, 48, 32 and 16 wide or high), k remainders
of the 32-element steps and of the four chains, both sides of the rule that chooses the kernel, operands of every size, some that the split
into bf16 parts does not represent, and the same bits whatever tile the number of models or images leads to.

Bounds: a product is off by at most 2^-24.2 (the three of nine products of parts that are left out) and a sum of K of them in any order by
K 2^-24 of sum |x||w|; each 32-k step adds six products of parts.  The measured error, in the 2-norm, is half of a plain float32 sum's."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

rng = np.random.default_rng(77)


@pytest.fixture(scope="module")
def nf():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2009_13062_amd as nf_
    return nf_


def rnd(*shape):
    return rng.standard_normal(shape).astype(np.float32)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


def check(got, ref, absref, K):
    got = got.detach().cpu().numpy().astype(np.float64)
    bound = (K + 10) * 2.0 ** -24 * absref + 1e-30
    assert got.shape == ref.shape and np.isfinite(got).all()
    assert (np.abs(got - ref) <= bound).all(), float((np.abs(got - ref) / bound).max())


@pytest.mark.parametrize("M,N,K,Nout", [
    (1, 1, 64, 1), (2, 15, 68, 31), (2, 17, 92, 33), (1, 16, 256, 64),            # 16-row tiles, k of 32 n + 4 .. 28
    (8, 33, 260, 65), (16, 48, 124, 96), (24, 65, 288, 49), (32, 63, 416, 47),    # 32- and 64-row tiles
    (12, 130, 768, 193), (32, 129, 96, 769), (6, 257, 1028, 95),                  # several tiles per compute unit
    (2, 256, 64, 256), (2, 257, 64, 256), (2, 1030, 64, 255), (2, 1025, 64, 256), (2, 1024, 64, 257),      # either side of the rule at 64 of k
    (2, 1024, 68, 256), (2, 1025, 68, 256),                                       # from 68 of k
    (1, 1449, 128, 1447), (1, 1449, 128, 1449), (1, 40, 60, 40), (3, 21, 66, 20),  # below 256 of k; too few k, k not in fours
], ids=lambda v: str(v))
def test_linear(nf, M, N, K, Nout):
    X, W, b, R = rnd(M, N, K), rnd(M, K, Nout), rnd(M, Nout), rnd(M, N, Nout)
    x, w = X.astype(np.float64), W.astype(np.float64)
    prod = np.matmul(x, w) + b[:, None]
    size = np.matmul(np.abs(x), np.abs(w)) + np.abs(b)[:, None] + np.abs(R)
    check(nf.linear(dev(X), dev(W), bias=dev(b), residual=dev(R), act=nf.ACT_RELU), np.maximum(prod, 0) + R, size, K)
    if M > 1:                                    # nothing of another problem is read, not even times zero
        X[1:], W[1:] = np.nan, np.nan
        check(nf.linear(dev(X), dev(W))[:1], np.matmul(x, w)[:1], size[:1], K)


@pytest.mark.parametrize("N,K,Nout", [(128, 768, 768), (93, 1024, 257), (40, 3072, 130)], ids=lambda v: str(v))
def test_no_further_from_64_bits_than_a_float32_sum(nf, N, K, Nout):
    """The 2-norm of the error against that of the products summed in float32, one rounding each, in four chains of k."""
    X, W = rnd(1, N, K), rnd(1, K, Nout)
    ref = np.matmul(X.astype(np.float64), W.astype(np.float64))
    chains = np.zeros((4, N, Nout), np.float32)
    for k in range(K):
        chains[k // 32 % 4] += X[0, :, k, None] * W[0, k]
    plain = chains[0] + chains[1] + chains[2] + chains[3]
    got = nf.linear(dev(X), dev(W)).cpu().numpy()
    assert np.linalg.norm(got - ref) <= np.linalg.norm(plain - ref)


def test_operands_without_three_parts(nf):
    """Infinities times numbers of one part (whose other parts are 0), NaN, numbers that round up to infinity in 8 bits, products that overflow:
    what float32 gives; rows and columns beside them as they were."""
    N, K, Nout = 40, 96, 70
    X, W = rnd(1, N, K), rnd(1, K, Nout)
    plain = nf.linear(dev(X), dev(W)).cpu().numpy()
    W[0, 5] = np.where(W[0, 5] > 0, 1.0, -1.0)
    clean = nf.linear(dev(X), dev(W)).cpu().numpy()
    bad = X.copy()
    bad[0, 3, 5], bad[0, 7, 5], bad[0, 20, 40], bad[0, 33, 5] = np.inf, -np.inf, np.nan, 3.4e38
    got = nf.linear(dev(bad), dev(W)).cpu().numpy()
    assert np.array_equal(got[0, 3], np.inf * W[0, 5]) and np.array_equal(got[0, 7], -np.inf * W[0, 5])
    assert np.isnan(got[0, 20]).all()
    assert np.allclose(got[0, 33], 3.4e38 * W[0, 5], rtol=1e-6)
    keep = [i for i in range(N) if i not in (3, 7, 20, 33)]
    assert np.array_equal(got[0, keep], clean[0, keep])
    big = nf.linear(dev(X * np.float32(1e30)), dev(W * np.float32(1e30))).cpu().numpy()
    assert not np.isfinite(big).any()
    tiny = nf.linear(dev(X * np.float32(2.0 ** -40)), dev(W * np.float32(2.0 ** 20))).cpu().numpy()
    assert np.array_equal(tiny, clean * np.float32(2.0 ** -20)) and plain.shape == clean.shape


@pytest.mark.parametrize("ex,ew", [(-100, 90), (-112, 100), (-120, 100), (-126, 100), (-140, 100), (100, -120), (-70, -70), (100, 20)])
@pytest.mark.parametrize("N,K,Nout", [(3, 64, 35), (65, 776, 97)], ids=lambda v: str(v))
def test_every_finite_operand(nf, N, K, Nout, ex, ew):
    """Operands down to the smallest float32 numbers beside large ones, so that results are ordinary numbers: the parts hold every bit of them.  The
    bound of a sum at scale 1 holds at every scale, and half a unit of the smallest number for results down there."""
    X = np.ldexp(rng.standard_normal((2, N, K)), ex).astype(np.float32)
    W = np.ldexp(rng.standard_normal((2, K, Nout)), ew).astype(np.float32)
    x, w = X.astype(np.float64), W.astype(np.float64)
    got, ref, size = nf.linear(dev(X), dev(W)).cpu().numpy().astype(np.float64), np.matmul(x, w), np.matmul(np.abs(x), np.abs(w))
    assert (np.abs(got - ref) <= (K + 10) * 2.0 ** -24 * size + 2.0 ** -149).all(), float((np.abs(got - ref) / size).max())
    if -126 < min(ex, ew) and abs(ex + ew) < 60:              # the 2-norm too is what it is at scale 1: 0.5e-7 and 2.0e-7 for these K
        assert np.linalg.norm(got - ref) <= (1e-7 if K == 64 else 3e-7) * np.linalg.norm(ref)


@pytest.mark.parametrize("M,N,K,Nout", [(1, 9, 68, 31), (2, 17, 92, 33), (24, 65, 288, 49), (32, 63, 416, 47), (12, 130, 776, 193), (32, 129, 96, 769),
                                        (1, 40, 3084, 70)], ids=lambda v: str(v))
def test_sums_past_the_range_of_the_parts(nf, M, N, K, Nout):
    """Every second row so large that its sums of parts overflow while float32's do not, beside rows with infinities at either end of k and ordinary ones: in
    every tile float32's results, the ordinary rows with the bits that they have alone."""
    X, W = rnd(M, N, K), rnd(M, K, Nout)
    W[:, 0] = np.where(W[:, 0] > 0, 1.0, -1.0)
    W[:, -1] = np.where(W[:, -1] > 0, 1.0, -1.0)
    clean = nf.linear(dev(X), dev(W)).cpu().numpy()
    bad = X.copy()
    bad[:, ::2] *= np.float32(2.0 ** 110)
    bad[:, 1::4, 0], bad[:, 3::8, -1] = np.inf, -np.inf
    got = nf.linear(dev(bad), dev(W)).cpu().numpy()
    check(torch.from_numpy(got[:, ::2]), np.matmul(bad[:, ::2].astype(np.float64), W.astype(np.float64)),
          np.matmul(np.abs(bad[:, ::2]).astype(np.float64), np.abs(W).astype(np.float64)), K)
    assert np.array_equal(got[:, 1::4], np.broadcast_to(np.inf * W[:, :1], got[:, 1::4].shape))
    assert np.array_equal(got[:, 3::8], np.broadcast_to(-np.inf * W[:, -1:], got[:, 3::8].shape))
    assert np.array_equal(got[:, 7::8], clean[:, 7::8])


def test_infinities_cost_one_more_pass(nf):
    """An infinity in every row, so that no sum is finite: another walk over k (2 to 3 times as long), not one per output (200 times)."""
    X, W, Y = torch.randn(8, 128, 3072, device="cuda"), torch.rand(8, 3072, 768, device="cuda"), torch.empty(8, 128, 768, device="cuda")

    def us():
        best = 1e9
        for _ in range(6):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(8):
                nf.linear(X, W, out=Y)
            end.record()
            end.synchronize()
            best = min(best, start.elapsed_time(end) * 1000 / 8)
        return best
    finite = us()
    X[:, :, 1000] = float("inf")
    assert us() < 10 * finite and bool((Y == float("inf")).all())


@pytest.mark.parametrize("rows,cols,K,taken", [(1, 1, 64, 1), (1, 1, 60, 0), (256, 256, 64, 1), (256, 257, 64, 0), (512, 512, 64, 0), (512, 512, 68, 1),
                                                (512, 513, 68, 0), (2048, 1024, 128, 1),
                                                (2048, 1025, 128, 0), (2048, 1025, 256, 1), (64, 64, 130, 0)])
def test_rule(nf, rows, cols, K, taken):
    assert bool(nf.lib.netfuse_f32_split_takes(rows, cols, K)) == bool(taken)


@pytest.mark.parametrize("N,K,Nout", [(16, 768, 2304), (65, 96, 100), (128, 4096, 1024), (300, 260, 47)], ids=lambda v: str(v))
def test_merged_equals_single(nf, N, K, Nout):
    X, W = torch.randn(32, N, K, device="cuda"), torch.randn(32, K, Nout, device="cuda")
    one = nf.linear(X[31:], W[31:])
    for M in (2, 3, 7, 16, 32):
        assert torch.equal(nf.linear(X[32 - M:], W[32 - M:])[M - 1], one[0]), M
