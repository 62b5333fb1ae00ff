"""3x3 convolutions over groups of 16 (2 k + 1) channels that conv_wave.h leaves to the patch kernel (conv_patch.h): copies of 8, 4, 2 and
1 pixels, row tiles of 32, 64 and 128 (by the number of tiles), either stride, a padding wider than conv_wave.h takes; and the shapes of
32 k channels and of fused narrow groups whose patches are too tall for conv_tap.h.  Integer-coded (every sum exact in float32):
the oracle's bits."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [   # M, B, channels in and out of a group, groups, H, W, stride, pad
    (2, 1, 48, 33, 1, 20, 24, 1, 1), (2, 2, 48, 40, 1, 15, 20, 1, 1), (1, 1, 80, 72, 1, 12, 18, 1, 1), (2, 1, 48, 64, 1, 14, 17, 1, 0),
    (26, 4, 48, 64, 1, 20, 24, 1, 1), (43, 3, 48, 72, 1, 20, 20, 1, 1), (30, 4, 48, 72, 1, 36, 34, 2, 1), (3, 1, 16, 40, 1, 9, 11, 1, 3),
    (2, 1, 48, 33, 2, 7, 16, 2, 5), (2, 1, 128, 40, 1, 100, 8, 4, 8), (2, 1, 4, 4, 8, 100, 8, 4, 8), (2, 1, 48, 8, 1, 300, 1, 1, 1),
]


@pytest.mark.parametrize("M,B,cig,cog,g,H,W,stride,pad", CASES)
def test_exact(oracle, M, B, cig, cog, g, H, W, stride, pad):
    import paper_2009_13062_amd as nf
    assert nf.lib.netfuse_conv_wave_tile(0, M, B, cig, cog, g, H, W, stride, pad) == 0
    rng = np.random.default_rng(M + cig + H + W)
    Ho, Wo = nf.conv_out_size(H, 3, stride, pad), nf.conv_out_size(W, 3, stride, pad)
    x = rng.integers(-2, 3, (B, M * g * cig, H, W)).astype(np.float32)
    w = rng.integers(-1, 2, (M * g * cog, cig, 3, 3)).astype(np.float32)
    bias = rng.integers(-4, 5, M * g * cog).astype(np.float32)
    res = rng.integers(-8, 9, (B, M * g * cog, Ho, Wo)).astype(np.float32)
    dev = lambda a, dt=torch.bfloat16: torch.from_numpy(a).to("cuda", dt)
    got = nf.conv2d(dev(x), dev(w), M, g=g, bias=dev(bias, torch.float32), residual=dev(res), stride=stride, pad=pad, act=1).float().cpu().numpy()
    sample = sorted({0, M - 1})                                # models the oracle evaluates
    rows = lambda a, c: np.concatenate([a[m * c:(m + 1) * c] for m in sample])
    chan = lambda a, c: np.concatenate([a[:, m * c:(m + 1) * c] for m in sample], axis=1)
    ref = oracle.conv2d(chan(x, g * cig), rows(w, g * cog), len(sample), g=g, bias=rows(bias, g * cog), residual=chan(res, g * cog), stride=stride,
                        pad=pad, act=1, out_bf16=True)
    assert np.array_equal(chan(got, g * cog), ref)
