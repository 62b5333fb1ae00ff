"""Convolutions over planes whose offsets reach the ends of 32 bits: the largest plane a kernel's offsets hold and the next, which
another one takes.  Integer-coded (every sum exact in float32); positions all over the plane are compared with a
float32 product of the pixels they read."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def integers(shape, lo, hi, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.empty(shape, device="cuda", dtype=torch.bfloat16).random_(lo, hi, generator=g)


@pytest.fixture(autouse=True)
def release():
    yield
    torch.cuda.empty_cache()


def check_pointwise(cin, cout, H, W, stride, seed):
    import paper_2009_13062_amd as nf
    x, w = integers((1, cin, H, W), -2, 3, seed), integers((cout, cin, 1, 1), -1, 2, seed + 1)
    y = nf.conv2d(x, w, 1, stride=stride)
    Ho, Wo = y.shape[2:]
    for oy in sorted({0, Ho // 2, Ho - 1}):
        ref = w.view(cout, cin).float() @ x[0, :, oy * stride, ::stride].float()
        assert torch.equal(y[0, :, oy], ref.bfloat16()), oy


# 2^25 positions are the most that 64 planes' byte offsets hold: just below, and beyond.  9 x 9 outputs in 128 x 128
# tiles (160 of them), 7 x 7 in 64 x 64 tiles.
@pytest.mark.parametrize("cin,cout,H,W,out", [(128, 20480, 5791, 5793, 9), (128, 20480, 6001, 6001, 9), (256, 72, 6001, 6001, 7),
                                              (256, 72, 5793, 5791, 7), (128, 128, 6001, 6001, 3001)])
def test_strided_pointwise(cin, cout, H, W, out):
    assert H % 2 and W % 2 and (H * W <= 2 ** 25) == (H < 6000)
    stride = -(-max(H, W) // out)
    check_pointwise(cin, cout, H, W, stride, cin + H)


# Stride 2 over even widths reads pixel pairs, 4, 2 or 1 per load by the output width; 64 planes of fewer than 2^26 positions count
# their pairs in an int (8190 x 8194 is the last such plane, at four positions less).
@pytest.mark.parametrize("W", [8192, 8194, 8196, 8198, 8200])
def test_stride_2_pairs(W):
    H = 8190
    assert (H * W < 2 ** 26) == (W <= 8194)
    check_pointwise(128, 16, H, W, 2, W)


# 3 x 3: 32 planes of up to 2^26 - 1 positions count in an int; groups of 32 k channels, of 16 (2 k + 1) under a wide padding, and
# narrow ones that share a block.
@pytest.mark.parametrize("H", [524287, 700000])
@pytest.mark.parametrize("cin,cout,g,pad", [(32, 40, 1, 1), (48, 8, 1, 3), (32, 32, 4, 1)])
def test_3x3(H, cin, cout, g, pad):
    import paper_2009_13062_amd as nf
    W = 128
    x, w = integers((1, cin, H, W), -2, 3, H), integers((cout, cin // g, 3, 3), -1, 2, cin)
    y = nf.conv2d(x, w, 1, g=g, pad=pad)
    Ho, Wo = y.shape[2:]
    for oy in (0, Ho // 2 + 1, Ho - 1):
        # the image rows that output row oy reads, zeros outside
        rows = torch.zeros(cin, 3, W + 2 * pad, device="cuda")
        for ky in range(3):
            iy = oy - pad + ky
            if 0 <= iy < H:
                rows[:, ky, pad:pad + W] = x[0, :, iy].float()
        taps = torch.stack([rows[:, :, kx:kx + Wo] for kx in range(3)], 2)                     # channel, ky, kx, position
        ref = torch.cat([w[i * cout // g:(i + 1) * cout // g].float().flatten(1) @ taps[i * cin // g:(i + 1) * cin // g].flatten(0, 2)
                         for i in range(g)])
        assert torch.equal(y[0, :, oy], ref.bfloat16()), oy


# The 7 x 7 stem over 3 channels, whose third plane starts beyond 2^30 elements and, in the larger one, whose three end beyond 2^31.
@pytest.mark.parametrize("H", [1050001, 1400003])
def test_stem(H):
    import paper_2009_13062_amd as nf
    W, cout = 512, 8
    x, w = integers((1, 3, H, W), -2, 3, H), integers((cout, 3, 7, 7), -1, 2, 5)
    y = nf.conv2d(x, w, 1, stride=2, pad=3)
    Ho, Wo = y.shape[2:]
    assert 2 * H * W > 2 ** 30 and (3 * H * W > 2 ** 31) == (H > 1.3e6)
    for oy in (0, 1, Ho // 2 + 1, Ho - 1):
        rows = torch.zeros(3, 7, W + 6, device="cuda")
        for ky in range(7):
            iy = 2 * oy - 3 + ky
            if 0 <= iy < H:
                rows[:, ky, 3:3 + W] = x[0, :, iy].float()
        taps = torch.stack([rows[:, :, kx:kx + 2 * Wo:2] for kx in range(7)], 2)
        assert torch.equal(y[0, :, oy], (w.float().flatten(1) @ taps.flatten(0, 2)).bfloat16()), oy
