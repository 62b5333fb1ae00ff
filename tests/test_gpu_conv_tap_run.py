"""3 x 3 convolutions with several 128-position tiles per workgroup: a run that divides the tiles and one that does not, a tile whose rows end
inside the image and one that reaches past it, one channel block (its weights stay) and several, one task per thread and two, fused narrow groups, stride 2, pad 0, planes
whose rows hold no whole chunks, a residual.  Integer-coded, so the oracle's bits."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,B,cin,cout,g,H,W,stride,pad", [
    (8, 8, 32, 32, 1, 40, 40, 1, 1), (8, 8, 64, 40, 1, 41, 39, 1, 1), (32, 1, 64, 64, 1, 56, 56, 1, 1), (32, 4, 64, 64, 1, 57, 55, 1, 1),
    (16, 1, 128, 128, 32, 56, 56, 1, 1), (16, 1, 256, 256, 32, 56, 56, 2, 1), (16, 1, 256, 256, 32, 57, 55, 2, 1),
    (16, 2, 64, 64, 4, 33, 47, 1, 0), (8, 8, 32, 64, 1, 75, 81, 2, 1), (7, 9, 32, 32, 1, 130, 17, 1, 1),
    (2, 3, 128, 136, 1, 56, 56, 2, 1), (3, 1, 160, 72, 1, 61, 47, 2, 1), (2, 1, 128, 40, 1, 100, 100, 1, 1), (26, 2, 256, 128, 1, 40, 43, 2, 1),
])
def test_runs_exact(oracle, M, B, cin, cout, g, H, W, stride, pad):
    import paper_2009_13062_amd as nf
    rng = np.random.default_rng(cin + H + W)
    Ho, Wo = nf.conv_out_size(H, 3, stride, pad), nf.conv_out_size(W, 3, stride, pad)
    x = rng.integers(-2, 3, (B, M * cin, H, W)).astype(np.float32)
    w = rng.integers(-1, 2, (M * cout, cin // g, 3, 3)).astype(np.float32)
    scale, shift = (2.0 ** rng.integers(-1, 2, M * cout)).astype(np.float32), rng.integers(-4, 5, M * cout).astype(np.float32)
    res = rng.integers(-8, 9, (B, M * cout, Ho, Wo)).astype(np.float32)
    dev = lambda a, dt=torch.bfloat16: torch.from_numpy(a).to("cuda", dt)
    f = torch.float32
    sample, images = [0, M - 1], [0, B - 1]                   # models and images the oracle evaluates
    cut = lambda a, c: np.concatenate([a[m * c:(m + 1) * c] for m in sample])
    chan = lambda a, c: np.concatenate([a[images][:, m * c:(m + 1) * c] for m in sample], axis=1)
    for kw in (dict(scale=scale, shift=shift, act=1), dict(residual=res)):
        got = nf.conv2d(dev(x), dev(w), M, g=g, stride=stride, pad=pad,
                        **{k: v if k == "act" else dev(v, torch.bfloat16 if k == "residual" else f) for k, v in kw.items()})
        ref = oracle.conv2d(chan(x, cin), cut(w, cout), len(sample), g=g, stride=stride, pad=pad, out_bf16=True,
                            **{k: v if k == "act" else chan(v, cout) if k == "residual" else cut(v, cout) for k, v in kw.items()})
        assert np.array_equal(chan(got.float().cpu().numpy(), cout), ref), sorted(kw)
