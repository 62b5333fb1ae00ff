"""3x3 convolutions over planes of any width: rows that start at any 2-byte address, chunks of a row that overlap, planes
narrower than a chunk, several output rows per tile, the last plane of the tensor.  Integer-coded (every sum exact in
float32), so the result must match the oracle bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("H,W", [(1, 1), (3, 2), (4, 3), (5, 5), (7, 7), (6, 9), (13, 13), (15, 15), (9, 19), (25, 25), (29, 29), (50, 50), (5, 131)])
@pytest.mark.parametrize("cig,cog,g", [(32, 40, 1), (64, 128, 1), (8, 8, 4), (4, 4, 8)])
def test_conv_any_width(oracle, H, W, stride, cig, cog, g):
    import paper_2009_13062_amd as nf
    M, B = 2, 2
    rng = np.random.default_rng(100 * W + 10 * stride + cig)
    x = rng.integers(-2, 3, (B, M * g * cig, H, W)).astype(np.float32)
    w = rng.integers(-1, 2, (M * g * cog, cig, 3, 3)).astype(np.float32)
    bias = rng.integers(-4, 5, M * g * cog).astype(np.float32)
    ref = oracle.conv2d(x, w, M, g=g, bias=bias, stride=stride, pad=1, act=nf.ACT_RELU, out_bf16=True)
    dev = lambda a, dt=torch.bfloat16: torch.from_numpy(a).to("cuda", dt)
    got = nf.conv2d(dev(x), dev(w), M, g=g, bias=dev(bias, torch.float32), stride=stride, pad=1, act=nf.ACT_RELU)
    assert np.array_equal(got.float().cpu().numpy(), ref)


@pytest.mark.parametrize("C,W,stride,pad", [(128, 112, 2, 2), (128, 107, 2, 2), (128, 112, 2, 1), (128, 25, 1, 1), (64, 50, 1, 1), (512, 13, 2, 1)])
def test_merged_equals_single(C, W, stride, pad):
    """The row tile follows from the number of models, also where a patch is too large for the tallest one: the same bits."""
    import paper_2009_13062_amd as nf
    M = 10
    x = torch.randn(1, M * C, W, W, device="cuda").bfloat16()
    w = (torch.randn(M * C, C, 3, 3, device="cuda") * 0.05).bfloat16()
    merged = nf.conv2d(x, w, M, stride=stride, pad=pad)
    for m in (0, M - 1):
        one = nf.conv2d(x[:, m * C:(m + 1) * C].contiguous(), w[m * C:(m + 1) * C], 1, stride=stride, pad=pad)
        assert torch.equal(merged[:, m * C:(m + 1) * C], one), m
