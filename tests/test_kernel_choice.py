"""Which kernel a call runs, on either side of the lines between the kernel families and the any-size kernel (host code only)."""
import os

import pytest

from gpu_util import any_size_shape, call_kernel


@pytest.fixture(scope="module", autouse=True)
def library():
    from paper_2512_07884_amd import binding
    if not os.path.exists(binding.lib_path()):
        from paper_2512_07884_amd import build
        build.build(verbose=False)


# (B, C, H, W, G), dtype, call, kchunk, logits: kernel, and without the any-size kernel in the families' place
CALLS = [
    # forward, plane family: 64 to 1024 planes (512 with logits) of more than 196 pixels
    ((3, 21, 14, 16, 7), "bf16", "save", 0, False, "plane", "plane"), ((4, 16, 14, 16, 4), "bf16", "save", 0, False, "any size", "plane"),
    ((4, 16, 14, 14, 4), "f32", "fwd", 0, False, "plane", "plane"), ((8, 128, 14, 16, 8), "f16", "save", 0, False, "any size", "plane"),
    ((5, 205, 14, 16, 5), "bf16", "save", 0, False, "plane", "plane"), ((4, 128, 28, 28, 8), "f32", "save", 0, True, "any size", "plane"),
    ((4, 132, 28, 28, 12), "f32", "save", 0, True, "plane", "plane"), ((2, 48, 56, 56, 4), "bf16", "save", 14, True, "any size", "plane"),
    # ... fp32 rows that are not whole granules, eight channels per group and more: up to 512 planes, up to 128 of up to 330 pixels
    ((4, 128, 20, 34, 16), "f32", "save", 0, False, "any size", "plane"), ((4, 130, 20, 34, 10), "f32", "save", 0, False, "plane", "plane"),
    ((4, 132, 20, 34, 33), "f32", "save", 0, False, "any size", "plane"), ((4, 136, 20, 36, 17), "f32", "save", 0, False, "any size", "plane"),
    ((4, 136, 20, 34, 17), "bf16", "save", 0, False, "any size", "plane"), ((2, 64, 18, 18, 8), "f32", "fwd", 0, False, "any size", "plane"),
    ((2, 72, 18, 18, 9), "f32", "fwd", 0, False, "plane", "plane"), ((2, 72, 15, 22, 9), "f32", "fwd", 0, False, "plane", "plane"),
    ((2, 72, 19, 18, 9), "f32", "fwd", 0, False, "any size", "plane"), ((2, 264, 18, 30, 33), "f32", "bwd", 0, True, "any size", "plane"),
    # forward, tile family: 32 planes and more of up to 20 000 pixels
    ((1, 31, 80, 72, 1), "bf16", "fwd", 0, False, "tile", "tile"), ((1, 32, 80, 72, 1), "bf16", "fwd", 0, False, "any size", "tile"),
    ((1, 32, 80, 64, 4), "f32", "save", 24, False, "any size", "tile"), ((1, 32, 156, 128, 2), "f32", "fwd", 0, False, "any size", "tile"),
    ((1, 32, 240, 96, 2), "f32", "fwd", 0, False, "tile", "tile"), ((64, 96, 56, 56, 8), "f32", "fwd", 0, False, "any size", "tile"),
    # ... 16-bit rows of 224 bytes, up to 64 of them (with logits: more than 512 planes)
    ((1, 64, 64, 112, 8), "f16", "fwd", 0, False, "tile", "tile"), ((1, 64, 66, 112, 8), "f16", "fwd", 0, False, "any size", "tile"),
    ((1, 64, 64, 112, 8), "f32", "fwd", 0, False, "any size", "tile"), ((4, 128, 64, 112, 8), "bf16", "save", 0, True, "any size", "tile"),
    ((4, 129, 64, 112, 3), "bf16", "save", 0, True, "tile", "tile"), ((4, 128, 64, 112, 8), "bf16", "bwd", 0, False, "twopass/tile", "twopass/tile"),
    ((4, 128, 64, 112, 8), "bf16", "bwd", 0, True, "twopass/any size", "twopass/tile"),
    # ... 16-bit rows of 192 and 256 bytes without h_save, more than 512 planes (up to 40 rows: 1024 and more)
    ((4, 128, 104, 96, 16), "bf16", "fwd", 0, False, "any size", "tile"), ((4, 129, 104, 96, 3), "bf16", "fwd", 0, False, "tile", "tile"),
    ((4, 129, 104, 96, 3), "bf16", "save", 0, False, "any size", "tile"), ((4, 129, 104, 96, 3), "f32", "fwd", 0, False, "any size", "tile"),
    ((4, 129, 104, 88, 3), "bf16", "fwd", 0, False, "any size", "tile"), ((4, 129, 104, 64, 3), "bf16", "fwd", 0, False, "any size", "tile"),
    ((4, 255, 40, 128, 15), "f16", "fwd", 0, False, "any size", "tile"), ((4, 256, 40, 128, 16), "f16", "fwd", 0, False, "tile", "tile"),
    ((4, 256, 104, 96, 16), "f16", "bwd", 0, False, "twopass/any size", "twopass/tile"),
    # ... 16-bit rows of 128 bytes, and up to 64 of 112, without h_save and logits, one channel per group, more than 768 planes
    ((1, 768, 104, 64, 768), "f16", "fwd", 0, False, "any size", "tile"), ((1, 769, 104, 64, 769), "f16", "fwd", 0, False, "tile", "tile"),
    ((1, 769, 104, 64, 769), "f16", "save", 0, False, "any size", "tile"), ((1, 769, 104, 64, 769), "f16", "fwd", 0, True, "any size", "tile"),
    ((1, 770, 104, 64, 385), "f16", "fwd", 0, False, "any size", "tile"), ((1, 769, 104, 32, 769), "f32", "fwd", 0, False, "any size", "tile"),
    ((7, 110, 64, 56, 110), "bf16", "fwd", 0, False, "tile", "tile"), ((7, 110, 66, 56, 110), "bf16", "fwd", 0, False, "any size", "tile"),
    ((1, 2560, 100, 64, 2560), "bf16", "fwd", 0, False, "tile", "tile"), ((1, 2561, 100, 64, 2561), "bf16", "fwd", 0, False, "any size", "tile"),
    ((1, 2561, 104, 64, 2561), "bf16", "fwd", 0, False, "tile", "tile"), ((1, 2561, 64, 64, 2561), "bf16", "fwd", 0, False, "tile", "tile"),
    ((1, 769, 104, 64, 769), "f16", "bwd", 0, False, "twopass/any size", "twopass/tile"),
    # ... fp32 rows of 512 bytes of more than 12 800 pixels without h_save, more than 512 planes
    ((4, 128, 102, 128, 16), "f32", "fwd", 0, False, "any size", "tile"), ((4, 129, 102, 128, 3), "f32", "fwd", 0, False, "tile", "tile"),
    ((4, 129, 100, 128, 3), "f32", "fwd", 0, False, "any size", "tile"), ((4, 129, 102, 128, 3), "f32", "save", 0, False, "any size", "tile"),
    ((4, 129, 138, 96, 3), "f32", "fwd", 0, False, "any size", "tile"),
    # backward, plane family: 64 planes and more of more than 256 pixels (one channel per group: up to 2048 planes)
    ((3, 20, 28, 28, 10), "f32", "bwd", 0, False, "plane", "plane"), ((4, 16, 28, 28, 4), "f32", "bwd", 0, False, "any size", "plane"),
    ((4, 16, 16, 16, 4), "f32", "bwd", 0, False, "plane", "plane"), ((32, 192, 28, 28, 192), "f32", "bwd", 0, True, "plane", "plane"),
    ((2, 64, 32, 32, 64), "f16", "bwd", 0, False, "any size", "plane"),
    # ... unless its workgroups fill the CUs: the training stage of the classifier, 256 workgroups of half a weight group each
    ((32, 192, 28, 28, 4), "f32", "bwd", 0, False, "plane", "plane"), ((32, 192, 28, 28, 4), "f32", "bwd", 0, True, "any size", "plane"),
    ((32, 192, 28, 32, 4), "f32", "bwd", 0, False, "any size", "plane"), ((33, 192, 28, 28, 4), "f32", "bwd", 0, False, "any size", "plane"),
    ((32, 192, 24, 24, 4), "f32", "bwd", 0, False, "any size", "plane"), ((64, 192, 28, 28, 8), "f32", "bwd", 0, False, "plane", "plane"),
    ((16, 256, 26, 26, 64), "f32", "bwd", 0, False, "any size", "plane"), ((17, 256, 26, 26, 64), "f32", "bwd", 0, False, "any size", "plane"),
    ((24, 256, 26, 26, 64), "f32", "bwd", 0, False, "plane", "plane"), ((27, 256, 20, 22, 64), "f32", "bwd", 0, False, "plane", "plane"),
    # ... tile family, and the first pass of the two
    ((1, 28, 43, 44, 7), "bf16", "bwd", 0, True, "tile", "tile"), ((1, 32, 43, 44, 8), "bf16", "bwd", 0, True, "any size", "tile"),
    ((2, 24, 56, 56, 2), "f32", "bwd", 0, False, "twopass/any size", "twopass/tile"), ((4, 16, 56, 56, 4), "bf16", "bwd", 0, False, "twopass/any size", "twopass/plane"),
    ((2, 24, 56, 56, 2), "bf16", "bwd", 0, False, "twopass/plane", "twopass/plane"),
    # elsewhere it takes nothing but the plan "generic"
    ((2, 1024, 128, 128, 16), "bf16", "fwd", 0, False, "pair", "pair"), ((2, 1024, 128, 128, 16), "f16", "bwd", 0, False, "twopass/pair", "twopass/pair"),
    ((1, 512, 512, 512, 16), "bf16", "fwd", 0, False, "stream", "stream"), ((1, 512, 512, 512, 16), "bf16", "bwd", 0, False, "twopass/stream", "twopass/stream"),
    ((1, 32, 128, 128, 4), "f32", "fwd", 32, False, "chunk", "chunk"), ((1, 32, 128, 128, 4), "f32", "bwd", 32, False, "twopass/chunk", "twopass/chunk"),
    ((4, 192, 50, 83, 8), "f32", "save", 0, False, "any size", "any size"), ((4, 192, 50, 83, 8), "f32", "bwd", 0, False, "any size", "any size"),
    ((1, 8, 1, 7, 1), "f32", "fwd", 0, False, "line by line", "line by line"), ((1, 2, 1001, 9, 1), "f32", "bwd", 0, False, "line by line", "line by line"),
]


@pytest.mark.parametrize("shape,dtype,call,kchunk,logits,kernel,own", CALLS,
                         ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s).replace(" ", "-"))
def test_either_side_of_the_lines(shape, dtype, call, kchunk, logits, kernel, own, monkeypatch):
    assert call_kernel(*shape, dtype, call, kchunk, logits) == kernel
    monkeypatch.setenv("GSPN_NO_ANY_SIZE", "1")
    assert call_kernel(*shape, dtype, call, kchunk, logits) == own
    monkeypatch.setenv("GSPN_FORCE_GENERIC", "1")
    assert call_kernel(*shape, dtype, call, kchunk, logits) == "line by line"


# Calls that walk no axis both ways (plane family), or the two vertical directions alone (tile family).
@pytest.mark.parametrize("shape,dtype,call,logits,any_size,own", [
    ((4, 64, 26, 28, 16), "bf16", "save", False, (1, 2, 5, 10, 15), ()), ((4, 68, 26, 28, 17), "bf16", "save", True, (3, 12, 7, 14, 15), (1, 8, 5, 9)),
    ((4, 66, 26, 28, 22), "bf16", "fwd", False, (1, 5, 3, 15), ()), ((4, 68, 26, 32, 17), "bf16", "fwd", False, (1, 5, 3, 15), ()),
    ((4, 68, 26, 28, 17), "f32", "fwd", False, (1, 5, 3, 15), ()), ((4, 68, 26, 30, 34), "f32", "fwd", False, (1, 5, 3, 15), ()),
    ((4, 68, 26, 30, 17), "f32", "fwd", False, (3, 12, 7, 15), (2, 4, 6, 10)), ((4, 68, 38, 38, 17), "f32", "save", False, (3, 12), (1, 5)),
    ((4, 68, 40, 38, 17), "f32", "save", False, (1, 5, 3, 12), ()), ((4, 68, 36, 44, 17), "f16", "bwd", False, (1, 5, 3, 15), ()),
    ((4, 68, 34, 44, 17), "f16", "bwd", False, (3, 11, 15), (1, 5)),
    ((4, 128, 72, 80, 8), "bf16", "fwd", False, (1, 3, 4, 12, 5, 15), ()), ((4, 129, 72, 80, 3), "bf16", "fwd", True, (1, 2, 4, 12, 5, 7, 15), (3,)),
    ((8, 128, 20, 112, 16), "f16", "save", False, (1, 4, 12, 5, 14), (3, 7, 15)), ((4, 129, 50, 128, 3), "bf16", "fwd", False, (1, 4, 12, 14), (3, 11, 15)),
    ((4, 256, 50, 96, 8), "bf16", "save", False, (1, 2, 5, 15), (3,)), ((4, 258, 50, 96, 6), "bf16", "save", False, (5, 7, 15), (1, 2, 3)),
    ((7, 110, 64, 56, 110), "bf16", "fwd", False, (1, 2, 12, 7, 11), (3, 15)), ((7, 110, 72, 64, 110), "bf16", "fwd", False, (1, 12, 13, 14), (3, 7, 11, 15)),
    ((4, 129, 72, 80, 3), "f16", "bwd", False, (1, 2, 12, 7, 15), (3,)), ((4, 129, 72, 80, 3), "f32", "bwd", False, (1, 3, 12, 15), ()),
    ((16, 64, 28, 28, 16), "f32", "bwd", False, (1, 5, 3, 15), ()), ((17, 64, 28, 28, 16), "f32", "bwd", False, (5, 10, 3, 15), (1, 8)),
    ((17, 64, 28, 28, 16), "f32", "bwd", True, (1, 8, 5, 3, 15), ()), ((17, 64, 28, 29, 16), "f32", "bwd", False, (1, 8, 5, 3, 15), ())],
    ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_lines_by_direction_mask(shape, dtype, call, logits, any_size, own):
    for mask in any_size + own:
        assert (call_kernel(*shape, dtype, call, logits=logits, mask=mask).split("/")[-1] == "any size") == (mask in any_size), mask


# Narrow maps (the longer side over 128 positions and three times the other) have orders of launch shapes of their own, in which
# short requests with both directions at once come before a merge in global memory; four positions per lane there only for lines of
# up to 256 positions of maps whose shorter side has more than 128.
@pytest.mark.parametrize("shape,dtype,logits,want", [
    ((1, 64, 233, 13, 8), "f32", False, (0, 2, 32, 1, 2, 1, 3)), ((1, 1, 288, 39, 1), "f32", False, (0, 1, 32, 1, 2, 1, 3)),
    ((1, 128, 240, 33, 8), "f32", False, (0, 2, 32, 1, 2, 1, 3)), ((1, 300, 200, 31, 4), "f32", True, (1, 1, 32, 2, 2, 1, 2)),
    ((1, 600, 19, 211, 4), "f32", False, (0, 2, 64, 1, 2, 2, 1)), ((1, 64, 225, 20, 8), "f16", True, (0, 2, 16, 1, 2, 1, 3)),
    ((1, 300, 17, 257, 4), "f16", False, (1, 2, 64, 2, 2, 3, 1)), ((1, 768, 258, 17, 8), "bf16", False, (1, 2, 16, 2, 2, 1, 3)),
    ((1, 16, 129, 43, 8), "bf16", False, (0, 2, 32, 1, 3, 1, 1)), ((1, 16, 129, 44, 8), "f32", False, (0, 2, 64, 1, 3, 1, 1)),
    ((1, 16, 225, 129, 8), "f32", False, (2, 2, 64, 1, 4, 1, 1)), ((1, 16, 225, 128, 8), "f32", False, (2, 2, 64, 1, 2, 1, 3)),
    ((1, 16, 257, 129, 8), "f32", False, (2, 2, 64, 1, 2, 2, 3))],
    ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_launch_shapes_of_narrow_maps(shape, dtype, logits, want):
    assert any_size_shape(*shape, dtype, "save", 0, logits) == any_size_shape(*shape, dtype, "bwd", 0, logits) == want
