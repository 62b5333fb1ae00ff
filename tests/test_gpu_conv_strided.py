"""Strided pointwise convolutions over planes whose width is odd or whose stride is not 2, ragged channels and positions, planes of one
position; and, with an operand off by one element, which conv_plane.h leaves to the register-staged kernels, theirs: the deep pipeline (k a
multiple of its 128 or 256) and the loader that takes any k, in every tile that the number of tiles leads to, pixel pairs over even widths.  Integer-coded (every sum exact in float32): the oracle's bits; and a position of infinities reaches the
outputs that read it only."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [   # M, B, cin, cout, H, W, stride
    (2, 2, 256, 72, 13, 13, 2), (2, 1, 1024, 264, 13, 13, 2),     # 64 x 64 tiles, fewer than 64 positions
    (14, 2, 256, 520, 13, 13, 2), (32, 2, 256, 520, 13, 13, 2),   # 128 x 128 over 49 positions, deep and one k-step in flight
    (3, 2, 256, 136, 25, 25, 2), (14, 2, 256, 264, 25, 25, 2),    # 64 x 64 and 128 x 128, more than 64 positions
    (40, 2, 128, 264, 25, 25, 2), (64, 2, 128, 520, 5, 5, 2), (20, 2, 64, 264, 25, 25, 2),   # 128 x 128, one k-step in flight
    (2, 1, 384, 24, 25, 25, 2), (3, 1, 160, 72, 13, 13, 2),       # up to 32 channels; k of no whole number of pipeline rounds
    (2, 2, 256, 72, 10, 19, 3), (2, 1, 256, 72, 5, 26, 5), (2, 2, 256, 72, 2, 1, 2), (2, 1, 512, 136, 41, 41, 2),
]


PAIRS = [(2, 1, 128, 256, 16, 16, 2), (3, 1, 64, 128, 14, 28, 2), (2, 1, 128, 256, 10, 10, 2), (2, 1, 128, 256, 12, 12, 2), (4, 2, 256, 264, 14, 14, 2)]


@pytest.mark.parametrize("M,B,cin,cout,H,W,stride", CASES)
def test_exact(oracle, M, B, cin, cout, H, W, stride):
    check(oracle, M, B, cin, cout, H, W, stride, "")


@pytest.mark.parametrize("shifted,M,B,cin,cout,H,W,stride", [("x", *c) for c in CASES] + [("w", *c) for c in CASES[1:7] + PAIRS])
def test_exact_in_the_register_staged_kernels(oracle, shifted, M, B, cin, cout, H, W, stride):
    check(oracle, M, B, cin, cout, H, W, stride, shifted)


def check(oracle, M, B, cin, cout, H, W, stride, shifted):
    import paper_2009_13062_amd as nf
    rng = np.random.default_rng(cin + cout + H + stride)
    Ho, Wo = nf.conv_out_size(H, 1, stride, 0), nf.conv_out_size(W, 1, stride, 0)
    x = rng.integers(-2, 3, (B, M * cin, H, W)).astype(np.float32)
    w = rng.integers(-1, 2, (M * cout, cin, 1, 1)).astype(np.float32)
    bias = rng.integers(-4, 5, M * cout).astype(np.float32)
    scale = (2.0 ** rng.integers(-1, 2, M * cout)).astype(np.float32)
    shift = rng.integers(-4, 5, M * cout).astype(np.float32)
    res = rng.integers(-8, 9, (B, M * cout, Ho, Wo)).astype(np.float32)
    dev = lambda a, dt=torch.bfloat16: torch.from_numpy(a).to("cuda", dt)
    f = torch.float32

    def off(a, name):                                         # one element into a buffer of its own
        t = dev(a)
        if name != shifted:
            return t
        t = torch.cat([t.new_zeros(1), t.flatten()])[1:].view(a.shape)
        assert t.data_ptr() % 16 == 2 and t.is_contiguous()
        return t
    got = nf.conv2d(off(x, "x"), off(w, "w"), M, bias=dev(bias, f), scale=dev(scale, f), shift=dev(shift, f), residual=dev(res), stride=stride, act=1)
    sample = [0, M - 1]                                       # models the oracle evaluates
    cut = lambda a, c: np.concatenate([a[m * c:(m + 1) * c] for m in sample])
    chan = lambda a, c: np.concatenate([a[:, m * c:(m + 1) * c] for m in sample], axis=1)
    ref = oracle.conv2d(chan(x, cin), cut(w, cout), 2, bias=cut(bias, cout), scale=cut(scale, cout), shift=cut(shift, cout),
                        residual=chan(res, cout), stride=stride, act=1, out_bf16=True)
    assert np.array_equal(chan(got.float().cpu().numpy(), cout), ref)
    # what the stride passes over is not read, and a position reaches its own output only
    x2 = x.copy()
    skipped = np.ones((H, W), bool)
    skipped[::stride, ::stride] = False
    x2[:, :, skipped] = np.inf
    last = Ho * Wo > 1                                        # a plane of one position has no other output to compare
    if last:
        x2[:, :, stride * (Ho - 1), stride * (Wo - 1)] = np.inf
    got2 = nf.conv2d(off(x2, "x"), off(w, "w"), M, bias=dev(bias, f), scale=dev(scale, f), shift=dev(shift, f), residual=dev(res), stride=stride, act=1)
    same = (got2 == got).reshape(B, M * cout, Ho * Wo)
    same = same[:, :, :-1] if last else same
    assert same.numel() and bool(same.all())
