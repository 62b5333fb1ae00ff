"""The 7 x 7 stride-2 convolution over 3 channels: runs of tiles per workgroup (one, several, a shorter last one), output rows that no tile
ends with, 64, fewer and more output channels (blocks of 64 and of 32), images of every class of patch chunks per thread (4, 6, 8, 12), tall and wide ones, a
residual.  Integer-coded, so the oracle's bits."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,B,cout,H,W", [
    (2, 1, 64, 224, 224), (16, 1, 64, 224, 224), (13, 2, 64, 130, 200), (2, 2, 40, 7, 8), (2, 1, 96, 33, 64), (30, 1, 136, 95, 96),
    (2, 1, 64, 30, 512), (1, 2, 64, 20, 736), (3, 1, 64, 300, 16), (2, 1, 64, 1, 288),
    (2, 2, 32, 130, 200), (3, 1, 20, 33, 64), (3, 1, 64, 40, 400), (9, 2, 32, 90, 400), (2, 1, 32, 30, 512), (1, 1, 72, 20, 736),
])
def test_stem_exact(oracle, M, B, cout, H, W):
    import paper_2009_13062_amd as nf
    rng = np.random.default_rng(cout + H + W)
    Ho, Wo = nf.conv_out_size(H, 7, 2, 3), nf.conv_out_size(W, 7, 2, 3)
    x = rng.integers(-2, 3, (B, M * 3, H, W)).astype(np.float32)
    w = rng.integers(-1, 2, (M * cout, 3, 7, 7)).astype(np.float32)
    scale, shift = (2.0 ** rng.integers(-1, 2, M * cout)).astype(np.float32), rng.integers(-4, 5, M * cout).astype(np.float32)
    res = rng.integers(-8, 9, (B, M * cout, Ho, Wo)).astype(np.float32)
    dev = lambda a, dt=torch.bfloat16: torch.from_numpy(a).to("cuda", dt)
    f = torch.float32
    sample = [0, M - 1]                                       # models the oracle evaluates
    cut = lambda a, c: np.concatenate([a[m * c:(m + 1) * c] for m in sample])
    chan = lambda a, c: np.concatenate([a[:, m * c:(m + 1) * c] for m in sample], axis=1)
    for kw in (dict(scale=scale, shift=shift, act=1), dict(residual=res)):
        got = nf.conv2d(dev(x), dev(w), M, stride=2, pad=3, **{k: v if k == "act" else dev(v, torch.bfloat16 if k == "residual" else f) for k, v in kw.items()})
        ref = oracle.conv2d(chan(x, 3), cut(w, cout), len(sample), stride=2, pad=3, out_bf16=True,
                            **{k: v if k == "act" else chan(v, cout) if k == "residual" else cut(v, cout) for k, v in kw.items()})
        assert np.array_equal(chan(got.float().cpu().numpy(), cout), ref), sorted(kw)
