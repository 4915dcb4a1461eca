"""Which calls run a wave per line, on either side of each line (host code only)."""
import os

import pytest


@pytest.fixture(scope="module", autouse=True)
def library():
    from paper_2512_07884_amd import binding
    if not os.path.exists(binding.lib_path()):
        from paper_2512_07884_amd import build
        build.build(verbose=False)


# (B, C, H, W, G), dtype, logits: forward, with h_save, backward
CALLS = [
    # in the any-size kernel's place: planes, short and narrow lines, rows of whole granules
    ((1, 512, 44, 44, 16), "bf16", False, (1, 1, 1)), ((1, 1024, 26, 27, 16), "bf16", False, (0, 0, 0)), ((1, 1008, 48, 48, 84), "bf16", False, (1, 1, 0)),
    ((2, 1664, 48, 48, 26), "f32", False, (1, 1, 1)), ((2, 1664, 37, 37, 26), "f32", False, (0, 0, 0)), ((44, 96, 63, 63, 8), "bf16", False, (1, 1, 0)), ((1, 448, 24, 24, 28), "bf16", False, (1, 0, 1)),
    ((1, 768, 21, 21, 32), "bf16", False, (0, 0, 0)), ((1, 512, 21, 21, 32), "bf16", False, (1, 1, 1)),
    ((1, 768, 21, 21, 32), "f32", False, (0, 0, 1)), ((1, 512, 21, 21, 32), "bf16", True, (1, 1, 0)), ((1, 768, 17, 44, 32), "bf16", False, (1, 0, 0)), ((1, 768, 16, 44, 32), "bf16", False, (0, 0, 1)),
    ((1, 768, 34, 34, 32), "f16", False, (1, 1, 1)), ((1, 768, 33, 33, 32), "f16", False, (1, 0, 1)), ((1, 512, 32, 32, 8), "f32", False, (0, 0, 1)), ((1, 512, 33, 32, 8), "f32", False, (1, 0, 1)),
    ((1, 1152, 44, 45, 24), "bf16", False, (1, 1, 1)), ((1, 1152, 44, 45, 32), "bf16", False, (0, 1, 1)), ((1, 760, 31, 17, 40), "bf16", False, (1, 0, 0)), ((1, 800, 31, 17, 40), "bf16", False, (0, 0, 0)), ((1, 1200, 40, 42, 1200), "f32", False, (1, 1, 0)),
    # the plane kernel's: weights of each channel's own, planes, pixels
    ((1, 2648, 64, 48, 2648), "bf16", False, (1, 1, 1)), ((1, 1152, 24, 24, 1152), "f32", True, (0, 0, 0)), ((1, 768, 24, 20, 32), "f32", True, (1, 1, 1)), ((1, 936, 24, 20, 39), "f32", True, (0, 0, 0)),
    ((1, 1008, 24, 20, 42), "f32", True, (0, 0, 0)), ((1, 2048, 18, 28, 2048), "bf16", True, (0, 0, 0)), ((1, 2048, 26, 28, 2048), "bf16", True, (1, 1, 0)), ((2, 1024, 36, 28, 512), "bf16", True, (0, 0, 0)), ((2, 1024, 36, 30, 512), "bf16", True, (1, 1, 0)), ((2, 1152, 64, 64, 16), "bf16", False, (1, 1, 0)),
    # that of calls whose directions would run apart: planes, pixels
    ((1, 66, 30, 40, 2), "bf16", False, (1, 0, 0)), ((1, 66, 30, 40, 2), "f32", False, (0, 0, 0)), ((1, 64, 30, 40, 2), "bf16", False, (0, 0, 0)), ((1, 96, 31, 45, 8), "bf16", False, (0, 0, 0)), ((1, 66, 30, 40, 2), "f32", True, (0, 0, 0)),
    # single-launch backward: planes, lengths, channels of a group
    ((1, 256, 14, 14, 4), "bf16", False, (0, 0, 1)), ((1, 1536, 10, 12, 32), "f32", False, (0, 0, 0)), ((1, 1536, 10, 12, 48), "f32", False, (0, 0, 1)), ((1, 96, 14, 14, 8), "bf16", False, (0, 0, 0)),
    # lines of several waves: rows, narrow maps, planes, types
    ((1, 1024, 160, 160, 16), "bf16", False, (1, 1, 0)), ((1, 1024, 96, 160, 16), "bf16", False, (0, 0, 0)), ((1, 1024, 160, 72, 16), "bf16", False, (0, 0, 0)),
    ((1, 1024, 160, 160, 16), "f32", False, (0, 0, 0)), ((1, 256, 160, 160, 16), "bf16", True, (1, 1, 0)), ((1, 240, 160, 160, 16), "bf16", True, (0, 0, 0)), ((1, 1024, 97, 160, 16), "bf16", False, (1, 0, 0)), ((1, 1024, 97, 128, 16), "bf16", False, (1, 1, 0)), ((1, 1024, 113, 160, 16), "bf16", False, (1, 1, 0)), ((1, 256, 112, 120, 16), "f16", True, (1, 0, 0)), ((1, 512, 160, 160, 16), "f16", True, (1, 1, 0)),
    ((1, 400, 120, 104, 16), "bf16", False, (0, 0, 0)), ((1, 1024, 209, 160, 16), "bf16", False, (0, 0, 0)), ((1, 512, 80, 104, 8), "f32", False, (0, 0, 1)),
]


@pytest.mark.parametrize("shape,dtype,logits,want", CALLS, ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_either_side_of_the_lines(shape, dtype, logits, want, monkeypatch):
    from paper_2512_07884_amd import binding
    code = {"f32": 0, "bf16": 1, "f16": 2}[dtype]
    f = lambda call, kchunk=0, mask=15: int(binding.call_lines(*shape, code, call, kchunk, logits, mask))
    assert tuple(f(c) for c in ("fwd", "save", "bwd")) == want
    # all four directions, the global scan, no testing aid
    assert not any(f(c, mask=m) for c in ("fwd", "save", "bwd") for m in (3, 7, 12))
    assert not any(f(c, kchunk=8) for c in ("fwd", "save", "bwd"))
    for call, w in (("fwd", want[0]), ("save", want[1])):
        if w:                                                # no workspace where it runs
            assert binding.gspn_fwd_workspace_bytes(*shape, binding.GLOBAL_SCAN, logits, 15, code, 0, call == "save") == 0
    before = [binding.call_kernel(*shape, code, c, 0, logits) + str(binding.call_apart(*shape, code, c, 0, logits)) for c in ("fwd", "save", "bwd")]
    for knob in ("GSPN_NO_APART", "GSPN_NO_LINES"):
        monkeypatch.setenv(knob, "1"); binding.gspn_reload_env()
        assert not any(f(c) for c in ("fwd", "save", "bwd"))
        if knob == "GSPN_NO_LINES":                          # nothing else changes with it
            assert before == [binding.call_kernel(*shape, code, c, 0, logits) + str(binding.call_apart(*shape, code, c, 0, logits)) for c in ("fwd", "save", "bwd")]
        monkeypatch.delenv(knob); binding.gspn_reload_env()
