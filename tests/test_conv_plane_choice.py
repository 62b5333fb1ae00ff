"""Which pointwise convolutions run the kernel of conv_plane.h and in which tile, asked of the library on the CPU."""
import pytest

from test_gpu_conv_plane import CASES

TILES = ("64x64 whole", "128x64 whole", "64x224 whole", "64x224 deep", "64x128", "128x128", "32x64", "128x64 gathered", "128x64 gathered, k 32", "128x128 gathered")


def tile_of(M, B, cin, cout, H, W, stride, residual, g=1):
    import paper_2009_13062_amd as nf
    t = nf.lib.netfuse_conv_plane_tile(M, B, cin // g, cout // g, g, H, W, stride, residual)
    return TILES[t] if t >= 0 else None


@pytest.mark.parametrize("residual", [0, 1])
def test_cases_run_every_tile(residual):
    assert {tile_of(*c, residual) for c in CASES} == set(TILES) | {None}


# Stride 2 over an even width is read as pixel pairs by another kernel, which keeps what is not predicted a sixth slower (24 models 1024 -> 256
# at 25 x 16 took 1.4 times as long here); odd widths have no such kernel.
@pytest.mark.parametrize("M,B,cin,cout,H,W,residual,taken", [
    (24, 1, 1024, 256, 25, 16, 1, False), (32, 1, 1024, 2048, 14, 14, 0, True), (32, 1, 256, 512, 28, 28, 0, False), (3, 4, 512, 1024, 25, 25, 0, True),
    (3, 4, 1024, 2048, 13, 13, 0, True), (16, 1, 1024, 64, 25, 25, 1, True),
])
def test_stride_2(M, B, cin, cout, H, W, residual, taken):
    assert (tile_of(M, B, cin, cout, H, W, 2, residual) is not None) == taken


@pytest.mark.parametrize("M,B,cin,cout,H,W,stride", [(8, 1, 96, 64, 7, 7, 1), (8, 1, 64, 32, 7, 7, 1), (8, 1, 64, 64, 8, 8, 1), (2, 1, 256, 72, 3, 601, 2)])
def test_not_taken(M, B, cin, cout, H, W, stride):
    assert tile_of(M, B, cin, cout, H, W, stride, 0) is None
