"""The plane kernel's variant and workgroups, on either side of each line (host code only)."""
import ctypes
import os

import pytest


@pytest.fixture(scope="module", autouse=True)
def library():
    from paper_2512_07884_amd import binding
    if not os.path.exists(binding.lib_path()):
        from paper_2512_07884_amd import build
        build.build(verbose=False)


def plane_shape(B, C, H, W, G, dtype, kchunk=0, logits=False):
    """(flat, channels per wave, waves per workgroup, channels on a CU at a time)"""
    from paper_2512_07884_amd import binding
    s = (ctypes.c_int * 4)()
    assert binding.load_library().gspn_plane_shape(B, C, H, W, G, kchunk, int(logits), {"f32": 0, "bf16": 1, "f16": 2}[dtype], s)
    return tuple(s)


# rows of whole chunks: the flat variant where it fills the chip less often than the padded one
@pytest.mark.parametrize("shape,dtype,kchunk,logits,flat", [
    ((1, 4096, 20, 20, 8), "f32", 0, False, 0), ((1, 4160, 20, 20, 8), "f32", 0, False, 1), ((64, 32, 20, 20, 8), "f32", 0, False, 0),
    ((1, 2624, 16, 16, 16), "f16", 0, False, 0), ((4, 1536, 16, 16, 16), "f16", 0, False, 1), ((2, 1536, 8, 8, 192), "bf16", 0, False, 0), ((4, 1536, 8, 8, 192), "bf16", 0, False, 1),
    ((1, 3588, 9, 8, 3588), "f32", 0, False, 0), ((1, 16384, 9, 8, 16384), "f32", 0, False, 1), ((1, 24576, 16, 8, 24576), "bf16", 0, False, 1),
    # a wave that fetches a group's weights by itself; workgroups that wait in place of such as need not
    ((4, 2224, 25, 20, 8), "f32", 5, False, 0), ((1, 4528, 17, 12, 8), "f32", 0, False, 1), ((64, 160, 17, 4, 16), "f32", 0, False, 0),
], ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_flat_where_the_chip_is_filled_less_often(shape, dtype, kchunk, logits, flat):
    assert plane_shape(*shape, dtype, kchunk, logits)[0] == flat


# fp32, shared weights: fewer waves per workgroup only where the chip is then filled less often, and not five in six's place
@pytest.mark.parametrize("shape,logits,waves", [
    ((1, 21120, 3, 3, 8), True, 6), ((1, 49920, 7, 7, 8), False, 4), ((1, 17280, 14, 14, 1), True, 8), ((16, 540, 20, 23, 1), False, 6), ((2, 3600, 12, 63, 8), True, 3), ((1, 25920, 7, 12, 8), False, 3),
    ((32, 192, 28, 28, 8), False, 6), ((96, 192, 28, 28, 8), False, 4), ((1, 1536, 28, 28, 8), False, 8),
], ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_fewer_waves_where_the_chip_is_filled_less_often(shape, logits, waves):
    assert plane_shape(*shape, "f32", 0, logits)[2] == waves
