"""Pointwise convolutions over planes of a multiple of 8 positions, at shapes that reach each tile: rows and positions past
the last whole tile, one k-step, several images, the per-channel constants and the residual.  Integer-coded (scales are
powers of two, every sum exact in float32), so the result must match the oracle bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("act", [0, 1])
@pytest.mark.parametrize("M,B,cin,cout,H,W", [
    (2, 1, 64, 40, 3, 8), (2, 3, 128, 72, 8, 8),              # 64 x 64
    (3, 2, 64, 200, 10, 36),
    (8, 2, 192, 136, 28, 28), (9, 2, 256, 200, 16, 30),       # 64 x 128
    (32, 1, 64, 64, 56, 56),                                  # 64 x 256
    (16, 2, 128, 256, 28, 28), (48, 1, 64, 200, 31, 32),      # 128 x 128
    (9, 2, 64, 264, 56, 56),                                  # 128 x 256
    (40, 2, 2048, 136, 2, 4),                                 # the register-staged 64 x 64 tile
])
def test_pointwise_exact(oracle, M, B, cin, cout, H, W, act):
    import paper_2009_13062_amd as nf
    rng = np.random.default_rng(cin + cout + H)
    x = rng.integers(-2, 3, (B, M * cin, H, W)).astype(np.float32)
    w = rng.integers(-1, 2, (M * cout, cin, 1, 1)).astype(np.float32)
    bias = rng.integers(-4, 5, M * cout).astype(np.float32)
    scale = (2.0 ** rng.integers(-1, 2, M * cout)).astype(np.float32)
    shift = rng.integers(-4, 5, M * cout).astype(np.float32)
    res = rng.integers(-8, 9, (B, M * cout, H, W)).astype(np.float32)
    dev = lambda a, dt=torch.bfloat16: torch.from_numpy(a).to("cuda", dt)
    f = torch.float32
    for kw in (dict(bias=bias, scale=scale, shift=shift, residual=res), dict(scale=scale, shift=shift), dict()):
        got = nf.conv2d(dev(x), dev(w), M, act=act, **{k: dev(v, torch.bfloat16 if k == "residual" else f) for k, v in kw.items()})
        sample = [0, M - 1]                                   # models the oracle evaluates
        cut = lambda a, c: np.concatenate([a[m * c:(m + 1) * c] for m in sample])
        chan = lambda a, c: np.concatenate([a[:, m * c:(m + 1) * c] for m in sample], axis=1)
        ref = oracle.conv2d(chan(x, cin), cut(w, cout), len(sample), act=act, out_bf16=True,
                            **{k: chan(v, cout) if k == "residual" else cut(v, cout) for k, v in kw.items()})
        assert np.array_equal(chan(got.float().cpu().numpy(), cout), ref), sorted(kw)


def test_small_planes_do_not_run_in_wide_tiles():
    """32 models of 8 images, 512 -> 2048: 8 x 8 planes, whose weights pass once per image, take 1.8 times as long as the same
    positions in one plane of 512; in 256-column tiles, which they fill to a quarter, it was 3.3 times."""
    import paper_2009_13062_amd as nf
    from test_gpu_f32 import us
    M, B, C, Co = 32, 8, 512, 2048
    w = torch.randn(M * Co, C, 1, 1, device="cuda").bfloat16()
    few, many = torch.randn(1, M * C, 16, 32, device="cuda").bfloat16(), torch.randn(B, M * C, 8, 8, device="cuda").bfloat16()
    wide = us(lambda: nf.conv2d(few, w, M))
    small = us(lambda: nf.conv2d(many, w, M))
    assert small < 2.4 * wide, (small, wide)
