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
    assert gradw_shape(*shape, apart=False)[3] == 1


# (B, K, M, H, W): the kernel that takes a product (0 rows from memory, 1 16 x 16 tiles, 2 and 3 rows through LDS in stages of 256 and 128
# pixels), on either side of each line
@pytest.mark.parametrize("shape,kernel", [
    ((2, 40, 33, 57, 55), 2), ((2, 40, 33, 55, 55), 1), ((2, 40, 33, 58, 54), 1), ((2, 40, 10, 57, 55), 1), ((2, 40, 10, 73, 71), 2), ((2, 16, 10, 73, 71), 1), ((1, 40, 33, 75, 70), 2), ((1, 40, 33, 60, 70), 1),
    ((16, 1152, 144, 28, 28), 3), ((2, 1152, 144, 48, 56), 2), ((16, 1152, 144, 64, 64), 2), ((16, 1152, 144, 48, 48), 3), ((2, 1152, 144, 50, 54), 2), ((2, 1152, 144, 50, 50), 3), ((2, 144, 1152, 45, 57), 2), ((2, 144, 1152, 45, 55), 3),
    ((4, 96, 96, 20, 20), 0), ((32, 96, 8, 45, 46), 3), ((32, 96, 8, 40, 40), 0), ((32, 96, 24, 40, 40), 2), ((32, 96, 24, 36, 36), 0), ((32, 96, 8, 56, 56), 2),
], ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_kernel_on_either_side_of_the_lines(shape, kernel):
    assert gradw_shape(*shape)[0] == kernel
