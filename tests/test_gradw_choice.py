"""Which kernel and tile the weight gradient of the projections takes, and in how many ranges of pixels (host code only)."""
import ctypes
import os

import pytest


@pytest.fixture(scope="module", autouse=True)
def library():
    from paper_2512_07884_amd import binding
    if not os.path.exists(binding.lib_path()):
        from paper_2512_07884_amd import build
        build.build(verbose=False)


def gradw_shape(B, K, M, H, W, apart=True):
    from paper_2512_07884_amd import binding
    s = (ctypes.c_int * 4)()
    binding.load_library().gspn_proxy_gradw_shape(B, K, M, H, W, int(apart), s)
    return tuple(s)


@pytest.mark.parametrize("shape", [(1, 1152, 144, 32, 32), (1, 70, 41, 25, 41), (1, 144, 1152, 33, 32), (1, 40, 33, 45, 29)])
def test_one_image_is_summed_in_halves_only_where_they_have_two_places(shape):
    assert gradw_shape(*shape)[::3] == (2, 2)
    assert gradw_shape(*shape, apart=False)[::3] == (2, 1)
