"""3x3 convolutions with wavefront-private pipelines (conv_wave.h): every tile that is built, by the number of models and images that
leads to it, with every activation, with and without residual and scale.  test_conv_wave_choice.py checks on the CPU
that the cases run the tiles they name.  bf16 is integer-coded (every sum exact in float32): the oracle's bits without GELU, one
bf16 step with it (its error may move a rounding); float32 is held to the rounding bound of a sum of K products in any order,
(K + 12) 2^-24 sum |x||w| with the epilogue's four roundings.  GELU: slope at most 1.13, 2e-6 for its own error."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

BF16, F32 = torch.bfloat16, torch.float32
CASES = [   # storage, 10 x wavefronts per tile + blocks of positions, M, B, channels in and out of a group, groups, H, W, stride, pad
    (BF16, 11, 5, 1, 16, 40, 1, 11, 11, 1, 2), (BF16, 11, 3, 2, 16, 16, 4, 16, 17, 2, 1),
    (BF16, 12, 48, 1, 16, 40, 1, 15, 17, 1, 2), (BF16, 12, 32, 8, 16, 16, 3, 11, 11, 2, 1),
    (BF16, 14, 48, 1, 16, 40, 2, 25, 27, 1, 1), (BF16, 17, 48, 1, 16, 40, 1, 40, 41, 1, 0),
    (BF16, 41, 2, 1, 128, 40, 2, 5, 30, 2, 1), (BF16, 41, 8, 1, 64, 64, 1, 13, 13, 2, 2),
    (BF16, 42, 24, 1, 128, 40, 2, 11, 11, 1, 0), (BF16, 43, 48, 1, 48, 33, 1, 11, 11, 1, 2), (BF16, 43, 32, 1, 256, 72, 1, 13, 13, 1, 1),
    (BF16, 44, 12, 4, 48, 33, 2, 11, 11, 1, 1), (BF16, 45, 12, 4, 48, 33, 2, 12, 13, 1, 1), (BF16, 45, 48, 1, 256, 72, 1, 12, 40, 2, 2),
    (BF16, 47, 48, 1, 256, 33, 2, 14, 14, 1, 1), (BF16, 47, 12, 4, 512, 33, 2, 11, 11, 1, 2),
    (F32, 11, 5, 1, 8, 33, 2, 7, 7, 1, 2), (F32, 12, 48, 1, 8, 33, 1, 25, 27, 1, 1), (F32, 14, 20, 1, 8, 8, 32, 20, 20, 2, 1),
    (F32, 41, 2, 1, 48, 33, 2, 20, 20, 2, 1), (F32, 42, 24, 1, 24, 72, 1, 20, 20, 1, 0), (F32, 43, 12, 1, 48, 33, 2, 12, 40, 1, 0),
    (F32, 44, 16, 1, 64, 64, 1, 25, 27, 1, 2), (F32, 45, 24, 1, 16, 40, 1, 25, 27, 1, 1), (F32, 47, 24, 1, 32, 64, 1, 33, 31, 1, 1),
]
FORMS = {"plain": (0, False, False), "relu_residual_scale": (1, True, True), "gelu_scale": (2, False, True)}


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("dt,tile,M,B,cig,cog,g,H,W,stride,pad", CASES)
def test_tile(oracle, dt, tile, M, B, cig, cog, g, H, W, stride, pad, form):
    import paper_2009_13062_amd as nf
    act, with_residual, with_scale = FORMS[form]
    rng = np.random.default_rng(tile + cig + H)
    Ho, Wo = nf.conv_out_size(H, 3, stride, pad), nf.conv_out_size(W, 3, stride, pad)
    exact = dt == BF16
    draw = (lambda lo, hi, *s: rng.integers(lo, hi, s).astype(np.float32)) if exact else (lambda lo, hi, *s: rng.standard_normal(s, np.float32))
    x, w = draw(-2, 3, B, M * g * cig, H, W), draw(-1, 2, M * g * cog, cig, 3, 3)
    bias = draw(-4, 5, M * g * cog)
    scale = (2.0 ** rng.integers(-2, 1, M * g * cog)).astype(np.float32) if with_scale else None
    shift = draw(-3, 4, M * g * cog) if with_scale else None
    res = draw(-9, 10, B, M * g * cog, Ho, Wo) if with_residual else None
    dev = lambda a, t=F32: None if a is None else torch.from_numpy(a).to("cuda", t)
    got = nf.conv2d(dev(x, dt), dev(w, dt), M, g=g, bias=dev(bias), scale=dev(scale), shift=dev(shift), residual=dev(res, dt), stride=stride, pad=pad, act=act)
    sample = sorted({0, M - 1})                                # models the oracle evaluates
    rows = lambda a, c: None if a is None else np.concatenate([a[m * c:(m + 1) * c] for m in sample])
    chan = lambda a, c: None if a is None else np.concatenate([a[:, m * c:(m + 1) * c] for m in sample], axis=1)
    ins = (chan(x, g * cig), rows(w, g * cog), rows(bias, g * cog), rows(scale, g * cog), rows(shift, g * cog), chan(res, g * cog))
    run = lambda a, bf, ac: oracle.conv2d(a[0], a[1], len(sample), g=g, bias=a[2], scale=a[3], shift=a[4], residual=a[5], stride=stride, pad=pad,
                                          act=ac, out_bf16=bf).astype(np.float64)
    ref, got = run(ins, exact, act), chan(got.float().cpu().numpy(), g * cog).astype(np.float64)
    if exact and act != 2:
        assert np.array_equal(got, ref)
        return
    if exact:
        bound = 2.0 ** -8 * np.abs(ref) + 2e-6
    else:
        mag = run(tuple(None if a is None else np.abs(a) for a in ins), False, 0)
        bound = (1.13 if act == 2 else 1.0) * (9 * cig + 12) * 2.0 ** -24 * mag + (2e-6 if act == 2 else 0.0)
    assert np.isfinite(got).all() and (np.abs(got - ref) <= bound).all()
