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
    (3, 2, 64, 200, 10, 36),                                  # 64 x 64 and 64 x 128 limits
    (8, 2, 192, 136, 28, 28),                                 # 64 x 128
    (32, 1, 64, 64, 56, 56),                                  # 64 x 256
    (16, 2, 128, 256, 28, 28),                                # 128 x 128
    (9, 2, 64, 264, 56, 56),                                  # 128 x 256
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
