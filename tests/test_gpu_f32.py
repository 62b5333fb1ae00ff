"""float32 storage on the matrix pipe: sizes at the edges of every tile (64, 48, 32 and 16 wide or high), k remainders
of the 32-element steps and of the split of k over two or four groups, both B paths, kernels of one and of two tap
words; and the same bits for a model whatever tile the number of models or images leads to.  The bound is derived, not fitted: a sum of K products in any order is off by at most
(K + 4) 2^-24 sum |x||w| before the epilogue, whose operations add at most four more roundings of the result's
operands."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

rng = np.random.default_rng(31)


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
    bound = (K + 8) * 2.0 ** -24 * absref + 1e-30
    assert got.shape == ref.shape and np.isfinite(got).all()
    bad = np.abs(got - ref) > bound
    assert not bad.any(), "%d of %d outside the rounding bound, worst %.2f of it" % (
        bad.sum(), bad.size, (np.abs(got - ref) / bound).max())


def us(f):
    """Shortest of five averages over 20 calls."""
    f()
    best = 1e9
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(20):
            f()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 50)
    return best


@pytest.mark.parametrize("M,N,K,Nout", [
    (1, 1, 1, 1), (1, 1, 36, 4),                 # one element; 16 x 64 tile
    (2, 16, 31, 64), (2, 17, 33, 65),            # tile edges, k = 32 -+ 1
    (2, 1, 516, 4), (2, 15, 1025, 63),           # 16 x 64 tile, dense and gathered
    (2, 1, 1540, 4), (2, 15, 1541, 63),          # the same with k in four groups
    (16, 277, 17, 4), (24, 222, 17, 3),          # 32 x 64 tile
    (24, 169, 520, 4), (32, 142, 520, 1),        # 32 x 64 tile
    (24, 169, 1544, 4), (32, 142, 1543, 1),      # the same with k in four groups
    (32, 294, 17, 4),                            # 64 x 48 tile, one column block of four
    (16, 146, 17, 260), (32, 270, 17, 1),        # 64 x 64 tile, k in two groups
    (32, 65, 65, 860), (32, 33, 129, 788 + 1),   # 64 x 64 tile, several per compute unit
    (24, 130, 1545, 516), (24, 130, 1569, 513),  # the same with four chains
    (2, 2047, 32, 3), (2, 2048, 32, 3), (1, 2049, 31, 65), (2, 2050, 33, 7),         # few k, around 2048 rows
], ids=lambda v: str(v))
def test_linear(nf, M, N, K, Nout):
    X, W, b, R = rnd(M, N, K), rnd(M, K, Nout), rnd(M, Nout), rnd(M, N, Nout)
    x, w = X.astype(np.float64), W.astype(np.float64)
    prod = np.matmul(x, w) + b[:, None]
    size = np.matmul(np.abs(x), np.abs(w)) + np.abs(b)[:, None] + np.abs(R)
    check(nf.linear(dev(X), dev(W), bias=dev(b), residual=dev(R), act=nf.ACT_RELU), np.maximum(prod, 0) + R, size, K)
    check(nf.linear(dev(X), dev(W)), np.matmul(x, w), size, K)
    if M > 1:                                    # nothing of another problem is read, not even times zero
        X[1:], W[1:] = np.nan, np.nan
        check(nf.linear(dev(X), dev(W))[:1], np.matmul(x, w)[:1], size[:1], K)


@pytest.mark.parametrize("M,B,Cin,Cout,g,H,W,KH,KW,stride,pad,dil", [
    (1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 0, 1),        # one pixel
    (2, 1, 17, 15, 1, 8, 8, 3, 3, 1, 1, 1),      # 64 positions, k = 153
    (2, 2, 24, 33, 1, 5, 13, 3, 3, 1, 1, 1),     # 65 positions
    (1, 1, 64, 16, 1, 9, 9, 3, 3, 2, 1, 1),      # stride 2, k in four groups
    (3, 1, 8, 20, 2, 11, 7, 5, 5, 1, 2, 1),      # 25 taps
    (2, 1, 6, 20, 1, 12, 12, 6, 5, 1, 3, 1),     # 30 taps, padding wider than half the kernel
    (2, 1, 3, 70, 1, 17, 19, 7, 7, 2, 3, 1),     # 49 taps: two words; k = 147
    (1, 1, 2, 65, 1, 12, 9, 8, 4, 1, 2, 1),      # 32 taps: the first count of the second word
    (2, 1, 5, 9, 1, 10, 10, 3, 3, 1, 2, 2),      # dilation
    (2, 1, 33, 48, 1, 7, 7, 1, 1, 1, 0, 1),      # pointwise, 49 positions: gathered rows
    (2, 1, 33, 48, 1, 6, 6, 1, 1, 1, 0, 1),      # pointwise, 36 positions: dense rows
    (16, 1, 64, 65, 1, 29, 29, 1, 1, 2, 0, 1),   # strided projection, many tiles
], ids=lambda v: str(v))
def test_conv2d(nf, oracle, M, B, Cin, Cout, g, H, W, KH, KW, stride, pad, dil):
    x, w = rnd(B, M * Cin, H, W), rnd(M * Cout, Cin // g, KH, KW)
    Ho, Wo = oracle.conv_out_size(H, KH, stride, pad, dil), oracle.conv_out_size(W, KW, stride, pad, dil)
    R, scale, shift = rnd(B, M * Cout, Ho, Wo), rnd(M * Cout), rnd(M * Cout)
    conv = lambda a, c: torch.nn.functional.conv2d(torch.from_numpy(a).double(), torch.from_numpy(c).double(), stride=stride,
                                                   padding=pad, dilation=dil, groups=M * g).numpy()
    s, t = scale[None, :, None, None].astype(np.float64), shift[None, :, None, None].astype(np.float64)
    size = conv(np.abs(x), np.abs(w)) * np.abs(s) + np.abs(t) + np.abs(R)
    got = nf.conv2d(dev(x), dev(w), M, g=g, scale=dev(scale), shift=dev(shift), residual=dev(R), stride=stride, pad=pad,
                    dil=dil, act=nf.ACT_RELU)
    check(got, np.maximum(conv(x, w) * s + t + R, 0), size, Cin // g * KH * KW)


@pytest.mark.parametrize("M,B,S,heads,d,use_mask", [
    (1, 1, 1, 1, 4, False),                      # one query, one key, a quarter of a feature block
    (3, 1, 7, 2, 20, True), (2, 2, 8, 2, 64, True), (2, 2, 9, 2, 64, True), (1, 2, 9, 1, 4, False),   # 8 tokens and past them
    (2, 1, 63, 2, 16, True), (1, 2, 64, 1, 32, False), (2, 1, 65, 1, 28, True),      # edges of the 64-key stage, d <= 32
    (2, 1, 128, 3, 64, False), (1, 3, 129, 2, 64, True), (2, 1, 17, 1, 60, True),    # d <= 64
    (1, 1, 96, 2, 128, True), (2, 1, 33, 1, 68, False), (1, 1, 100, 1, 80, True),    # d <= 128: 32-key stages
], ids=lambda v: str(v))
def test_attention(nf, oracle, M, B, S, heads, d, use_mask):
    """Against the oracle (double accumulation).  A score carries d products, the weights S of them, and the
    exponential doubles neither: (d + S + 16) 2^-24 times the largest |score| + 4 (the exponent's own rounding is
    absolute in the score), relative to the largest |V| that is averaged."""
    qkv = rnd(M, B * S, 3 * heads * d)
    mask = rnd(M, B, S) if use_mask else None
    ref = oracle.attention_packed(qkv, B, S, heads, mask=mask).astype(np.float64)
    got = nf.attention_packed(dev(qkv), B, S, heads, mask=None if mask is None else dev(mask)).cpu().numpy()
    smax = np.abs(qkv).max() ** 2 * d * d ** -0.5
    assert np.isfinite(got).all()
    assert np.abs(got - ref).max() <= (d + S + 16) * 2.0 ** -24 * (smax + 4) * np.abs(qkv).max()
    if M > 1:                                    # NaN in another model stays there
        dirty = qkv.copy()
        dirty[1:] = np.nan
        alone = nf.attention_packed(dev(dirty), B, S, heads, mask=None if mask is None else dev(mask)).cpu().numpy()
        assert np.array_equal(alone[0], got[0])


@pytest.mark.parametrize("N,K,Nout", [(8, 64, 64), (128, 768, 768), (17, 520, 3), (93, 768, 2304), (128, 1536, 768),
                                      (128, 3072, 768), (256, 1568, 257)], ids=lambda v: str(v))
def test_linear_merged_equals_single(nf, N, K, Nout):
    """One order of the sum for every tile: k below and from 1536 up, dense and gathered columns."""
    X, W = torch.randn(32, N, K, device="cuda"), torch.randn(32, K, Nout, device="cuda")
    one = nf.linear(X[31:], W[31:])
    for M in (2, 5, 8, 12, 32):
        assert torch.equal(nf.linear(X[32 - M:], W[32 - M:])[M - 1], one[0]), M


@pytest.mark.parametrize("Cin,Cout,g,H,KH,stride,pad", [
    (64, 64, 1, 56, 3, 1, 1), (64, 256, 1, 56, 1, 1, 0), (512, 512, 1, 7, 3, 1, 1), (2048, 512, 1, 7, 1, 1, 0),
    (512, 512, 1, 13, 3, 2, 1), (3, 64, 1, 64, 7, 2, 3), (256, 256, 32, 28, 3, 1, 1), (32, 32, 32, 28, 3, 1, 1),
    (128, 128, 32, 21, 3, 1, 1)], ids=lambda v: str(v))
def test_conv2d_merged_equals_single(nf, Cin, Cout, g, H, KH, stride, pad):
    """The same for models and for images of one model, wide and narrow groups."""
    kw = dict(g=g, stride=stride, pad=pad)
    x, w = torch.randn(1, 24 * Cin, H, H, device="cuda"), torch.randn(24 * Cout, Cin // g, KH, KH, device="cuda")
    one = nf.conv2d(x[:, 23 * Cin:].contiguous(), w[23 * Cout:], 1, **kw)[0]
    for M in (2, 5, 8, 24):
        got = nf.conv2d(x[:, (24 - M) * Cin:].contiguous(), w[(24 - M) * Cout:], M, **kw)
        assert torch.equal(got[0, (M - 1) * Cout:], one), M
    xb = torch.cat([torch.randn(7, Cin, H, H, device="cuda"), x[:, 23 * Cin:]])
    for B in (2, 4, 8):
        assert torch.equal(nf.conv2d(xb[8 - B:], w[23 * Cout:], 1, **kw)[B - 1], one), B


@pytest.mark.parametrize("M,B,Cin,Cout,g,H,W,KH,KW,stride,pad,dil", [
    (2, 1, 64, 64, 64, 9, 7, 3, 3, 1, 1, 1), (3, 2, 40, 40, 40, 12, 12, 5, 5, 2, 2, 1),       # depthwise
    (2, 1, 64, 64, 64, 8, 8, 7, 7, 1, 3, 1), (1, 2, 70, 140, 70, 1, 1, 1, 1, 1, 0, 1),
    (2, 1, 128, 128, 32, 11, 13, 3, 3, 1, 1, 2), (2, 2, 64, 256, 16, 10, 8, 3, 3, 1, 1, 1),   # 4 -> 4; 4 -> 16 channels
    (1, 1, 512, 64, 64, 6, 5, 3, 3, 1, 1, 1), (1, 1, 1088, 64, 64, 6, 5, 3, 3, 1, 1, 1),      # 8 -> 1, 17 -> 1, 64 groups
    (2, 1, 64, 8, 8, 6, 4, 3, 3, 1, 1, 1), (2, 1, 72, 8, 8, 6, 4, 3, 3, 1, 1, 1),             # k = 72, 81 with 8 groups
    (2, 1, 64, 32, 8, 8, 4, 1, 1, 1, 0, 1), (2, 1, 64, 72, 8, 8, 4, 1, 1, 1, 0, 1),           # pointwise 8 -> 4, 8 -> 9
], ids=lambda v: str(v))
def test_conv2d_narrow_groups(nf, M, B, Cin, Cout, g, H, W, KH, KW, stride, pad, dil):
    """Either side of the line between the direct and the matrix-pipe kernel."""
    x, w = rnd(B, M * Cin, H, W), rnd(M * Cout, Cin // g, KH, KW)
    scale, shift = rnd(M * Cout), rnd(M * Cout)
    conv = lambda a, b: torch.nn.functional.conv2d(torch.from_numpy(a).double(), torch.from_numpy(b).double(), stride=stride,
                                                   padding=pad, dilation=dil, groups=M * g).numpy()
    s, t = scale[None, :, None, None].astype(np.float64), shift[None, :, None, None].astype(np.float64)
    got = nf.conv2d(dev(x), dev(w), M, g=g, scale=dev(scale), shift=dev(shift), stride=stride, pad=pad, dil=dil)
    check(got, conv(x, w) * s + t, conv(np.abs(x), np.abs(w)) * np.abs(s) + np.abs(t), Cin // g * KH * KW)


def test_depthwise_is_bound_by_memory(nf):
    """Nine products per output: a depthwise 3x3 takes a few times as long as moving its planes (3 times), not as long as
    the 16 x 128 products per output that its smallest matrix tile would spend (57 times)."""
    M, C, H = 8, 256, 28
    x, w = torch.randn(1, M * C, H, H, device="cuda"), torch.randn(M * C, 1, 3, 3, device="cuda")
    y = torch.empty_like(x)
    copy = us(lambda: nf.merge_transpose(x.view(M, C, H * H), M, True, out=y.view(C, M * H * H)))
    conv = us(lambda: nf.conv2d(x, w, M, g=C, pad=1, out=y))
    assert conv < 15 * max(copy, 5.0), (conv, copy)


def test_attention_of_single_tokens_is_bound_by_memory(nf):
    """One token per sequence: about twice as long as moving the operands, not as long as the 64-query tiles of longer
    sequences (15 times)."""
    M, B, heads = 32, 8, 16
    qkv = torch.randn(M, B, 3 * heads * 64, device="cuda")
    out, dst = torch.empty(M, B, heads * 64, device="cuda"), torch.empty(B, M * 3 * heads * 64, device="cuda")
    copy = us(lambda: nf.merge_transpose(qkv, M, True, out=dst))
    att = us(lambda: nf.attention_packed(qkv, B, 1, heads, out=out))
    assert att < 4 * max(copy, 5.0), (att, copy)


def test_few_k_over_many_rows_is_bound_by_memory(nf):
    """65536 rows of 2 k and one output: five times as long as the copy of its 4 MB, which is a launch; the fixed cost of its
    matrix tiles was fifteen."""
    M, N, K = 8, 65536, 2
    X, W, Y = torch.randn(M, N, K, device="cuda"), torch.randn(M, K, 1, device="cuda"), torch.empty(M, N, 1, device="cuda")
    dst = torch.empty(N, M * K, device="cuda")
    copy = us(lambda: nf.merge_transpose(X, M, True, out=dst))
    few = us(lambda: nf.linear(X, W, out=Y))
    assert few < 9 * max(copy, 5.0), (few, copy)
