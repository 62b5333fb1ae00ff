"""Pointwise convolutions over planes that start at any element (conv_plane.h), one group of problems per tile: planes of one position
up to the largest that a tile spans (55 of 56, 196 of 200), rows past the last whole tile, one k-step and fewer than the ring is deep,
several images, several tiles per plane, strides 2, 3 and 5 with output rows that no tile boundary respects; operands that are not 16 bytes
aligned and rows too wide for a tile's chunks, which the register-staged kernels keep.  Integer-coded (scales are powers of two, every
sum exact in float32): the oracle's bits; and a position of infinities reaches the outputs that read it only."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [   # M, B, cin, cout, H, W, stride
    (3, 2, 64, 200, 1, 1, 1), (8, 2, 64, 264, 5, 11, 1), (40, 2, 256, 200, 7, 7, 1), (2, 2, 192, 200, 8, 7, 2),      # 64 x 64, whole planes
    (32, 2, 320, 520, 5, 11, 1), (40, 2, 192, 520, 7, 7, 1), (40, 2, 512, 264, 7, 8, 2),                             # 128 x 64, whole planes
    (32, 1, 64, 264, 4, 47, 1), (40, 1, 256, 520, 28, 7, 1), (32, 2, 128, 72, 10, 18, 1),                            # 64 x 224, whole planes
    (16, 2, 512, 520, 14, 14, 1),                                                                                    # the same, deep
    (16, 1, 320, 520, 18, 18, 1), (40, 1, 128, 40, 4, 51, 1), (8, 2, 320, 264, 14, 14, 1),                           # 64 x 128 of a plane
    (40, 2, 64, 72, 18, 18, 1), (16, 2, 256, 520, 18, 18, 1), (32, 2, 64, 200, 4, 51, 1),                            # 128 x 128 of a plane
    (16, 1, 192, 264, 25, 25, 1), (3, 2, 320, 136, 10, 19, 1), (3, 1, 192, 72, 28, 7, 2), (8, 1, 512, 72, 25, 25, 3),   # 32 x 64
    (2, 1, 256, 72, 5, 26, 5),                                                                                       # the same
    (3, 2, 256, 520, 10, 19, 2), (40, 1, 128, 520, 4, 47, 3), (2, 1, 192, 264, 33, 35, 3),                           # 128 x 64, strided
    (32, 1, 256, 520, 13, 13, 2), (16, 2, 128, 200, 25, 25, 3), (32, 1, 128, 136, 16, 16, 2),                        # the same, k-steps of 32
    (32, 2, 192, 264, 18, 18, 2), (16, 2, 128, 136, 33, 35, 2),                                                      # 128 x 128, strided
    (2, 1, 256, 72, 3, 601, 2), (2, 1, 128, 136, 5, 301, 3),                                                         # rows too wide
]


def _make(M, B, cin, cout, H, W, stride, seed):
    import paper_2009_13062_amd as nf
    rng = np.random.default_rng(seed)
    Ho, Wo = nf.conv_out_size(H, 1, stride, 0), nf.conv_out_size(W, 1, stride, 0)
    return dict(x=rng.integers(-2, 3, (B, M * cin, H, W)).astype(np.float32), w=rng.integers(-1, 2, (M * cout, cin, 1, 1)).astype(np.float32),
                bias=rng.integers(-4, 5, M * cout).astype(np.float32), scale=(2.0 ** rng.integers(-1, 2, M * cout)).astype(np.float32),
                shift=rng.integers(-4, 5, M * cout).astype(np.float32), residual=rng.integers(-8, 9, (B, M * cout, Ho, Wo)).astype(np.float32))


def _check(oracle, M, B, cin, cout, H, W, stride, shifted=False):
    import paper_2009_13062_amd as nf
    a = _make(M, B, cin, cout, H, W, stride, cin + cout + H + stride)
    f32 = ("bias", "scale", "shift")

    def dev(k, v):
        t = torch.from_numpy(v).to("cuda", torch.float32 if k in f32 else torch.bfloat16)
        if shifted and k in ("x", "w", "residual"):           # one element into a buffer of its own
            t = torch.cat([t.new_zeros(1), t.flatten()])[1:].view(v.shape)
            assert t.data_ptr() % 16 == 2 and t.is_contiguous()
        return t
    d = {k: dev(k, v) for k, v in a.items()}
    sample = [0, M - 1]                                       # models the oracle evaluates
    cut = lambda v, c: np.concatenate([v[m * c:(m + 1) * c] for m in sample])
    chan = lambda v, c: np.concatenate([v[:, m * c:(m + 1) * c] for m in sample], axis=1)
    for act, keys in ((1, ("bias", "scale", "shift", "residual")), (0, ("scale", "shift"))):
        got = nf.conv2d(d["x"], d["w"], M, stride=stride, act=act, **{k: d[k] for k in keys})
        ref = oracle.conv2d(chan(a["x"], cin), cut(a["w"], cout), len(sample), stride=stride, act=act, out_bf16=True,
                            **{k: chan(a[k], cout) if k == "residual" else cut(a[k], cout) for k in keys})
        assert np.array_equal(chan(got.float().cpu().numpy(), cout), ref), keys


@pytest.mark.parametrize("M,B,cin,cout,H,W,stride", CASES)
def test_exact(oracle, M, B, cin, cout, H, W, stride):
    _check(oracle, M, B, cin, cout, H, W, stride)


@pytest.mark.parametrize("M,B,cin,cout,H,W,stride", [(40, 2, 256, 200, 7, 7, 1), (8, 2, 320, 264, 14, 14, 1), (32, 1, 256, 520, 13, 13, 2)])
def test_unaligned_operands(oracle, M, B, cin, cout, H, W, stride):
    _check(oracle, M, B, cin, cout, H, W, stride, shifted=True)


@pytest.mark.parametrize("H,W,stride,at", [(7, 7, 1, (6, 6)), (14, 14, 1, (13, 13)), (18, 18, 1, (0, 17)), (13, 13, 2, (12, 12))])
def test_infinities_stay_in_their_position(H, W, stride, at):
    """The last channel's last positions are what the chunks past a stage's end repeat."""
    import paper_2009_13062_amd as nf
    M, B, cin, cout = 16, 2, 256, 264
    a = _make(M, B, cin, cout, H, W, stride, 5)
    x, w = torch.from_numpy(a["x"]).cuda().bfloat16(), torch.from_numpy(a["w"]).cuda().bfloat16()
    clean = nf.conv2d(x, w, M, stride=stride)
    x[1, 3 * cin:4 * cin, at[0], at[1]] = float("inf")
    got = nf.conv2d(x, w, M, stride=stride)
    hit = torch.zeros_like(got, dtype=torch.bool)
    hit[1, 3 * cout:4 * cout, at[0] // stride, at[1] // stride] = True
    assert not torch.isfinite(got[hit]).any()
    assert torch.equal(got[~hit], clean[~hit])
