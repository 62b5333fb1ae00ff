"""How many 128-position tiles a workgroup of the tap-major 3x3 kernel takes (conv_tap_inst.hip), asked of the library on the CPU."""
import ctypes

import pytest


def run_of(cig, groups, tiles, lds, bm=32):
    import paper_2009_13062_amd as nf
    f = nf.lib.netfuse_conv_tap_run
    f.argtypes, f.restype = [ctypes.c_int, ctypes.c_int, ctypes.c_longlong, ctypes.c_int, ctypes.c_int], ctypes.c_int
    return f(cig, bm, groups, tiles, lds)


# Longer runs of these took up to 1.6 times as long: fewer workgroups, and two on a compute unit do not halve each other's rate.
@pytest.mark.parametrize("cig,groups,tiles,lds,bm", [(256, 288, 4, 66688, 64), (256, 192, 3, 48384, 32), (192, 128, 2, 49664, 32), (64, 64, 9, 46464, 32),
                                                     (64, 1, 98, 89088, 64), (512, 4096, 25, 162176, 128), (256, 48, 32, 68608, 64), (96, 64, 9, 65408, 64), (64, 512, 7, 66048, 64),
                                                     (96, 512, 3, 66688, 64), (64, 256, 2, 136576, 128), (64, 96, 25, 53504, 32)])
def test_several_blocks_take_one_tile(cig, groups, tiles, lds, bm):
    assert run_of(cig, groups, tiles, lds, bm) == 1


# Two and three blocks: runs that measured ahead of one tile, the best ones or within 1 %.
@pytest.mark.parametrize("cig,groups,tiles,lds,bm,run", [
    (64, 18, 76, 83328, 64, 6), (64, 96, 79, 84608, 64, 10), (96, 32, 79, 84608, 64, 10), (64, 32, 13, 96384, 32, 2), (64, 32, 25, 69000, 64, 2),
])
def test_few_blocks_take_the_run_that_evens_out(cig, groups, tiles, lds, bm, run):
    assert run_of(cig, groups, tiles, lds, bm) == run


# One block: the best of every run measured, where another was at least a tenth slower.
@pytest.mark.parametrize("groups,tiles,lds,run", [(128, 5, 49024, 1), (96, 8, 45824, 1), (32, 20, 50944, 1), (384, 7, 47104, 4), (128, 41, 54144, 11), (192, 25, 53504, 7),
                                                  (384, 13, 50304, 7), (768, 2, 50304, 2), (768, 4, 47744, 4), (48, 79, 65664, 8), (256, 5, 49024, 2)])
def test_one_block_takes_the_run_that_fills_the_chip(groups, tiles, lds, run):
    assert run_of(32, groups, tiles, lds) == run


def test_every_run_is_in_range():
    for groups in (1, 7, 255, 256, 257, 5000, 1 << 30):
        for tiles in (1, 2, 3, 63, 64, 65, 524288):
            for lds in (20000, 50000, 54614, 81920, 81921, 163840):
                assert 1 <= run_of(32, groups, tiles, lds) <= tiles


def test_division_is_called_exact_where_it_is():
    """Positions / width as the high half of a product: refused shapes run other kernels, so the bound is the exact one."""
    import paper_2009_13062_amd as nf
    f = nf.lib.netfuse_div_exact
    f.argtypes, f.restype = [ctypes.c_longlong, ctypes.c_int], ctypes.c_int
    for d in list(range(1, 700)) + [1000, 4095, 4097, 65535, 65537]:
        rcp = -(-2 ** 32 // d)
        most = 2 ** 32 - 1 if rcp * d == 2 ** 32 else (2 ** 32 - 1) // (rcp * d - 2 ** 32)       # the largest n that is called exact
        assert f(most, d) and not f(most + 1, d), d
        assert most >= 2 ** 32 // d - 1                        # never less than the bound that holds for every divisor
        for k in (1, 2, most // d // 2, most // d):           # the last value before a step and the step itself
            for n in (k * d - 1, k * d, most):
                if d > 1 and 0 <= n <= most:
                    assert n * rcp >> 32 == n // d, (n, d)
    # tall planes: 128 and 512 columns are powers of two, 650 divides 2^32 + 4
    assert f(524287 * 128, 128) and f(2 ** 26 - 1, 512) and f(2 ** 26 - 1, 650)
