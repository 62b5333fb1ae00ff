"""3x3 convolutions with wavefront-private pipelines (conv_wave.h): steps that do not divide over four wavefronts, ragged rows, planes
that end inside a 16-byte store, either stride, padding 0 to 2, in tiles of one block of positions (the others, and the rest of the
epilogue: test_gpu_conv_wave_tiles.py); and the same bits for a model whatever tile the number of models leads to.  bf16 is integer-coded (every sum exact in
float32), float32 is held to the rounding bound of a sum of K products in any order: (K + 8) 2^-24 sum |x||w|."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

rng = np.random.default_rng(77)


def dev(a, dt=torch.float32):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).to("cuda", dt)


PLANES = [(7, 7, 1, 1), (7, 7, 2, 1), (14, 14, 1, 1), (13, 13, 2, 1), (2, 2, 1, 1), (1, 3, 1, 1), (9, 5, 1, 0), (5, 9, 2, 2),
          (28, 8, 2, 1), (4, 41, 1, 1), (15, 14, 1, 2)]


@pytest.mark.parametrize("H,W,stride,pad", PLANES)
@pytest.mark.parametrize("cig,cog,g", [(16, 33, 1), (48, 40, 1), (32, 64, 2), (80, 8, 1), (256, 32, 1), (16, 16, 4)])
def test_bf16(oracle, H, W, stride, pad, cig, cog, g):
    import paper_2009_13062_amd as nf
    M, B = 2, 2
    Ho, Wo = nf.conv_out_size(H, 3, stride, pad), nf.conv_out_size(W, 3, stride, pad)
    if Ho < 1 or Wo < 1:
        pytest.skip("no output")
    x = rng.integers(-2, 3, (B, M * g * cig, H, W)).astype(np.float32)
    w = rng.integers(-1, 2, (M * g * cog, cig, 3, 3)).astype(np.float32)
    bias = rng.integers(-4, 5, M * g * cog).astype(np.float32)
    scale = 2.0 ** rng.integers(-1, 2, M * g * cog).astype(np.float32)
    shift = rng.integers(-3, 4, M * g * cog).astype(np.float32)
    res = rng.integers(-9, 10, (B, M * g * cog, Ho, Wo)).astype(np.float32)
    ref = oracle.conv2d(x, w, M, g=g, bias=bias, scale=scale, shift=shift, residual=res, stride=stride, pad=pad, act=nf.ACT_RELU, out_bf16=True)
    b16 = torch.bfloat16
    got = nf.conv2d(dev(x, b16), dev(w, b16), M, g=g, bias=dev(bias), scale=dev(scale), shift=dev(shift), residual=dev(res, b16),
                    stride=stride, pad=pad, act=nf.ACT_RELU)
    assert np.array_equal(got.float().cpu().numpy(), ref)


@pytest.mark.parametrize("H,W,stride,pad", PLANES)
@pytest.mark.parametrize("cig,cog,g", [(8, 33, 1), (24, 32, 1), (16, 16, 4), (64, 40, 1), (96, 7, 1)])
def test_f32(oracle, H, W, stride, pad, cig, cog, g):
    import paper_2009_13062_amd as nf
    M, B = 2, 2
    Ho, Wo = nf.conv_out_size(H, 3, stride, pad), nf.conv_out_size(W, 3, stride, pad)
    if Ho < 1 or Wo < 1:
        pytest.skip("no output")
    x, w = (rng.standard_normal(s).astype(np.float32) for s in ((B, M * g * cig, H, W), (M * g * cog, cig, 3, 3)))
    bias, res = (rng.standard_normal(s).astype(np.float32) for s in ((M * g * cog,), (B, M * g * cog, Ho, Wo)))
    ref = oracle.conv2d(x, w, M, g=g, bias=bias, residual=res, stride=stride, pad=pad).astype(np.float64)
    mag = oracle.conv2d(abs(x), abs(w), M, g=g, bias=abs(bias), residual=abs(res), stride=stride, pad=pad).astype(np.float64)
    got = nf.conv2d(dev(x), dev(w), M, g=g, bias=dev(bias), residual=dev(res), stride=stride, pad=pad).cpu().numpy()
    # the oracle's own result is rounded to float32 once
    assert np.isfinite(got).all() and (np.abs(got - ref) <= (9 * cig + 8 + 1) * 2.0 ** -24 * mag).all()


@pytest.mark.parametrize("dt,C,H,stride", [(torch.bfloat16, 256, 14, 1), (torch.bfloat16, 512, 7, 1), (torch.bfloat16, 128, 50, 2),
                                           (torch.bfloat16, 48, 20, 1), (torch.float32, 64, 28, 1), (torch.float32, 128, 28, 2),
                                           (torch.float32, 8, 40, 1)])
def test_merged_equals_single(dt, C, H, stride):
    """20 models and one take tiles of different sizes: the same bits."""
    import paper_2009_13062_amd as nf
    M = 20
    x = torch.randn(1, M * C, H, H, device="cuda").to(dt)
    w = (torch.randn(M * C, C, 3, 3, device="cuda") * 0.05).to(dt)
    merged = nf.conv2d(x, w, M, stride=stride, pad=1)
    for m in (0, M - 1):
        one = nf.conv2d(x[:, m * C:(m + 1) * C].contiguous(), w[m * C:(m + 1) * C], 1, stride=stride, pad=1)
        assert torch.equal(merged[:, m * C:(m + 1) * C], one), m


@pytest.mark.parametrize("C,g,H,stride", [(8, 32, 28, 1), (8, 8, 56, 1), (8, 16, 56, 2), (16, 8, 40, 1), (16, 4, 72, 2), (16, 32, 14, 1), (16, 32, 28, 2)])
def test_f32_narrow_groups_round_as_two_chains(C, g, H, stride):
    """Groups of 8 and 16 channels, products of one sign: two chains of K / 2 products each (the matrix instruction rounds after
    either of its two).  Adding n terms of one size one after the other leaves a relative error of c sqrt(n / 3 + 1 / 2), c =
    0.425 * 2^-24 the root mean square of one rounding over evenly spread logarithms; two independent chains average theirs and
    add one rounding.  A quarter above that; a single chain is at 1.5 times the bound."""
    import paper_2009_13062_amd as nf
    x = np.abs(rng.standard_normal((2, g * C, H, H))).astype(np.float32)
    w = np.abs(rng.standard_normal((g * C, C, 3, 3))).astype(np.float32)
    ref = torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(w).double(), stride=stride, padding=1, groups=g)
    got = nf.conv2d(dev(x), dev(w), 1, g=g, stride=stride, pad=1).cpu().double()
    n = 9 * C / 2
    bound = 1.25 * 0.425 * 2.0 ** -24 * (((n / 3 + 0.5) / 2) + 1) ** 0.5
    inner = slice(1, -1)                                       # positions that read the whole 3 x 3 window
    err = ((got - ref) / ref)[:, :, inner, inner].pow(2).mean().sqrt().item()
    assert err <= bound, (err, bound)
