"""Which 3x3 convolutions run the kernel of conv_wave.h and in which tile, asked of the library on the CPU."""
import pytest
import torch

from test_gpu_conv_wave_tiles import CASES


def tile_of(f32, *shape):
    import paper_2009_13062_amd as nf
    return nf.lib.netfuse_conv_wave_tile(int(f32), *shape)


def test_cases_run_the_tiles_they_name():
    for dt, tile, *shape in CASES:
        assert tile_of(dt == torch.float32, *shape) == tile, shape
    ran = {(c[0] == torch.float32, c[1]) for c in CASES}
    assert ran == {(f, t) for f in (False, True) for t in (11, 12, 14, 41, 42, 43, 44, 45, 47)} | {(False, 17)}      # every tile that is built


@pytest.mark.parametrize("f32,cig,g,size,stride", [(0, 16, 4, 8, 1), (0, 16, 4, 28, 2), (0, 48, 1, 13, 1), (0, 128, 1, 11, 1), (0, 256, 1, 14, 1), (0, 256, 1, 25, 2),
                                                   (0, 512, 1, 28, 1), (1, 8, 32, 40, 1), (1, 16, 4, 28, 2), (1, 64, 1, 56, 1), (1, 256, 1, 28, 2)])
def test_wavefronts_follow_from_one_group(f32, cig, g, size, stride):
    """The order of a sum, hence the bits, must not depend on how many models or images there are."""
    ran = {tile_of(f32, M, B, cig, cig, g, size, size, stride, 1) // 10 for M in (1, 2, 7, 32) for B in (1, 3, 8)}
    assert len(ran) == 1 and ran != {0}


# Shapes that another kernel runs faster with many images (by 1.1 to 2.3 times), and those next to them that stay.
@pytest.mark.parametrize("f32,cig,g,size,stride,taken", [
    (0, 32, 32, 14, 1, False), (0, 32, 32, 5, 1, True), (0, 64, 1, 14, 1, False), (0, 64, 1, 9, 1, True), (0, 128, 1, 14, 1, False), (0, 128, 1, 56, 2, False),
    (0, 128, 1, 16, 2, True), (0, 256, 1, 17, 1, False), (0, 256, 1, 36, 2, False), (0, 256, 1, 28, 2, False), (0, 512, 1, 36, 2, False), (0, 512, 1, 28, 2, True),
    (0, 16, 6, 10, 1, False), (0, 16, 6, 9, 1, True), (0, 48, 1, 36, 2, False), (0, 48, 4, 14, 1, False), (1, 128, 1, 56, 2, False), (1, 128, 1, 40, 2, True),
    (1, 64, 1, 72, 1, False), (1, 40, 1, 28, 1, False), (1, 16, 1, 111, 2, False),
])
def test_shapes_that_lose_with_many_images_are_left_out(f32, cig, g, size, stride, taken):
    assert (tile_of(f32, 4, 2, cig, cig, g, size, size, stride, 1) != 0) == taken
