"""Which calls run their directions in workgroups of their own, on either side of each line (host code only): 0 none, 1 given a
workspace, 2 without one, 3 stream kernels that walk half a scan per launch, given a workspace,
4 a wave per direction, without one."""
import os

import pytest


@pytest.fixture(scope="module", autouse=True)
def library():
    from paper_2512_07884_amd import binding
    if not os.path.exists(binding.lib_path()):
        from paper_2512_07884_amd import build
        build.build(verbose=False)


# (B, C, H, W, G), dtype, kchunk, logits: forward, with h_save, backward
CALLS = [
    ((1, 64, 256, 256, 8), "bf16", 0, False, (1, 1, 2)), ((1, 96, 256, 256, 8), "bf16", 0, False, (1, 1, 0)),
    ((1, 104, 256, 256, 8), "bf16", 0, False, (0, 0, 0)), ((1, 128, 256, 256, 8), "f32", 0, False, (1, 2, 2)),
    ((1, 64, 1024, 512, 8), "bf16", 0, False, (3, 3, 0)), ((1, 32, 1024, 512, 8), "bf16", 0, False, (1, 1, 2)), ((1, 128, 1024, 1024, 8), "f32", 0, False, (3, 3, 0)),
    ((1, 130, 1024, 1024, 13), "f32", 0, False, (0, 0, 0)), ((1, 64, 576, 2048, 8), "f16", 0, False, (3, 3, 0)),
    ((1, 144, 128, 128, 8), "bf16", 0, False, (1, 1, 0)), ((1, 152, 128, 128, 4), "f16", 0, False, (0, 0, 0)),
    ((1, 96, 128, 128, 8), "f16", 0, False, (1, 1, 2)), ((1, 32, 128, 128, 4), "f32", 32, False, (1, 2, 2)),
    ((1, 64, 128, 128, 4), "bf16", 32, False, (1, 1, 0)), ((1, 32, 128, 128, 4), "bf16", 32, False, (1, 1, 2)),
    ((1, 144, 50, 83, 9), "bf16", 0, False, (1, 1, 2)), ((1, 160, 50, 83, 10), "bf16", 0, False, (0, 0, 2)),
    ((1, 192, 40, 83, 12), "bf16", 0, False, (1, 1, 2)), ((1, 200, 40, 83, 25), "bf16", 0, False, (0, 0, 2)),
    ((1, 384, 50, 83, 12), "bf16", 0, True, (1, 1, 2)), ((1, 392, 50, 83, 49), "f16", 0, True, (0, 0, 0)),
    ((1, 384, 50, 83, 12), "f32", 0, False, (0, 2, 2)), ((1, 392, 50, 83, 49), "f32", 0, False, (0, 0, 0)),
    ((1, 128, 50, 83, 8), "f16", 16, False, (1, 1, 2)), ((1, 136, 50, 83, 17), "f16", 16, False, (0, 0, 0)),
    ((1, 64, 19, 21, 8), "bf16", 0, False, (4, 4, 0)),
    # small maps: lines of 8, 16, 32; planes; rows of whole granules
    ((1, 384, 14, 14, 8), "bf16", 0, False, (4, 4, 0)), ((2, 8000, 8, 8, 8), "f32", 4, True, (4, 4, 0)), ((2, 8001, 8, 7, 1), "f32", 0, False, (0, 0, 0)),
    ((1, 4096, 14, 14, 8), "f16", 0, False, (4, 4, 0)), ((1, 2056, 14, 14, 8), "f32", 0, False, (0, 0, 0)), ((1, 384, 16, 16, 8), "bf16", 0, False, (0, 0, 0)),
    ((1, 384, 12, 16, 8), "bf16", 7, False, (4, 4, 0)), ((1, 512, 30, 13, 8), "bf16", 0, True, (4, 4, 0)), ((1, 520, 30, 13, 8), "bf16", 0, True, (0, 0, 0)),
    ((1, 64, 26, 8, 8), "f32", 0, False, (0, 0, 0)), ((1, 64, 17, 8, 8), "f32", 0, False, (4, 4, 0)), ((1, 64, 33, 4, 8), "f16", 0, False, (0, 0, 0)), ((1, 64, 20, 20, 8), "bf16", 0, False, (1, 1, 2)),
    ((2, 256, 100, 167, 8), "bf16", 0, True, (0, 0, 0)), ((4, 192, 50, 83, 8), "f32", 0, False, (0, 0, 0)),
    # 16-bit planes whose fp32 tile does not fit, which ran line by line
    ((1, 600, 195, 195, 8), "bf16", 0, False, (1, 1, 0)), ((1, 1100, 400, 90, 11), "bf16", 0, False, (1, 1, 0)),
    ((2, 1024, 195, 195, 16), "bf16", 0, False, (0, 0, 0)),                      # (workspace beyond 1 GiB)
]


@pytest.mark.parametrize("shape,dtype,kchunk,logits,want", CALLS, ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_either_side_of_the_lines(shape, dtype, kchunk, logits, want, monkeypatch):
    from paper_2512_07884_amd import binding
    code = {"f32": 0, "bf16": 1, "f16": 2}[dtype]
    f = lambda call, mask=15: binding.call_apart(*shape, code, call, kchunk, logits, mask)
    assert tuple(f(c) for c in ("fwd", "save", "bwd")) == want
    for save, w in ((False, want[0]), (True, want[1])):
        n = binding.gspn_fwd_workspace_bytes(*shape, kchunk or binding.GLOBAL_SCAN, logits, 15, code, 0, save)
        planes = shape[0] * shape[1]
        assert n == {0: 0, 4: 0, 1: 16 * planes * shape[2] * shape[3], 2: 0, 3: 8 * planes * max(shape[2:4])}[w]
    assert f("fwd", 7) == f("bwd", 12) == 0                                       # all four directions only
    for knob in ("GSPN_NO_APART", "GSPN_FORCE_GENERIC", "GSPN_FWD_NO_PAIR"):
        monkeypatch.setenv(knob, "1")
        assert f("fwd") == f("save") == f("bwd") == 0
        monkeypatch.delenv(knob)


def test_invalid_arguments_ask_for_nothing():
    from paper_2512_07884_amd import binding
    ask = lambda *a, **k: binding.gspn_fwd_workspace_bytes(*a, **k)
    assert ask(1, 8, 50, 50, 3) == ask(0, 8, 50, 50, 1) == ask(1, 8, 50, 50, 1, kchunk=0) == ask(1, 8, 50, 50, 1, dtype=7) == 0
    assert ask(1, 8, 50, 50, 1, flags=8) == ask(1, 8, 50, 5000, 1, logits=True) == 0 < ask(1, 8, 50, 50, 1)


# Calls of as few planes that would run longer so, on either side of each line: (B, C, H, W, G), dtype, kchunk, logits, call, taken
LONGER = [
    # stream kernels: weights of each channel's own, stretches that are no whole granules, beyond 64 planes
    ((1, 64, 256, 256, 64), "bf16", 0, False, "fwd", True), ((1, 72, 256, 256, 72), "bf16", 0, False, "fwd", False), ((1, 72, 256, 256, 24), "bf16", 0, False, "fwd", True),
    ((1, 109, 512, 256, 109), "f32", 0, False, "bwd", False), ((1, 76, 256, 256, 19), "f32", 37, False, "bwd", False), ((1, 76, 256, 256, 19), "f32", 36, False, "bwd", True),
    # per-stretch kernels: many short stretches, high maps, the backward call in 16 bits
    ((1, 12, 128, 128, 2), "bf16", 8, False, "fwd", False), ((1, 12, 128, 128, 2), "bf16", 16, False, "fwd", True), ((1, 91, 256, 64, 13), "f32", 64, False, "fwd", False),
    ((1, 91, 64, 256, 13), "f32", 64, False, "fwd", True), ((1, 16, 128, 128, 8), "bf16", 32, False, "bwd", False), ((1, 16, 128, 128, 2), "bf16", 32, False, "bwd", True),
    ((1, 16, 128, 128, 8), "bf16", 64, False, "bwd", True), ((1, 4, 64, 64, 4), "f32", 8, False, "bwd", False), ((1, 4, 64, 64, 1), "f32", 8, False, "bwd", True),
    # any-size kernel, stretches: begun inside a granule beside many vertical ones, narrow maps, weights of each channel's own, very many
    ((1, 124, 392, 240, 124), "f32", 62, True, "fwd", False), ((1, 32, 392, 240, 32), "f32", 62, True, "fwd", True), ((1, 124, 432, 144, 4), "f16", 72, False, "fwd", True),
    ((1, 124, 432, 144, 4), "f16", 8, False, "fwd", False), ((1, 128, 432, 70, 8), "bf16", 216, False, "save", False), ((1, 128, 420, 72, 8), "bf16", 216, False, "save", True),
    ((1, 100, 100, 90, 100), "bf16", 16, False, "bwd", False), ((1, 100, 100, 90, 25), "bf16", 16, False, "bwd", True),
    # ... long narrow maps: 65 to 128 planes, and beyond
    ((1, 64, 416, 16, 8), "f16", 0, False, "fwd", True), ((1, 76, 282, 42, 1), "f16", 0, False, "fwd", False), ((1, 76, 282, 48, 1), "f16", 0, False, "fwd", True),
    ((1, 76, 250, 30, 1), "bf16", 0, False, "save", False), ((1, 76, 250, 32, 1), "bf16", 0, False, "save", True), ((1, 76, 480, 30, 1), "bf16", 0, False, "fwd", False),
    ((1, 76, 480, 30, 1), "bf16", 0, False, "bwd", True), ((1, 76, 282, 42, 1), "f32", 0, False, "fwd", True), ((1, 76, 282, 34, 1), "f32", 0, False, "fwd", False),
    ((1, 136, 200, 48, 8), "bf16", 0, False, "fwd", False), ((1, 136, 150, 48, 8), "bf16", 0, False, "fwd", True), ((1, 136, 200, 40, 8), "bf16", 0, False, "bwd", True),
    ((1, 190, 416, 16, 2), "f16", 0, False, "bwd", False), ((1, 190, 416, 42, 2), "f16", 0, False, "bwd", True), ((1, 256, 90, 11, 8), "bf16", 0, False, "bwd", False),
    # ... weights of each channel's own; large calls; rows of whole granules
    ((1, 126, 227, 227, 126), "f16", 0, False, "fwd", False), ((1, 126, 227, 227, 42), "f16", 0, False, "fwd", True), ((1, 96, 227, 227, 96), "f16", 0, False, "fwd", True),
    ((1, 144, 60, 60, 144), "bf16", 0, False, "fwd", False), ((1, 144, 60, 50, 144), "bf16", 0, False, "fwd", True), ((1, 144, 128, 125, 9), "bf16", 0, False, "fwd", False),
    ((1, 144, 128, 125, 9), "bf16", 0, True, "fwd", True), ((1, 256, 40, 40, 8), "bf16", 0, True, "fwd", False), ((1, 256, 40, 41, 8), "bf16", 0, True, "fwd", True),
    ((1, 256, 40, 40, 8), "f32", 0, False, "save", True), ((1, 256, 60, 60, 8), "f32", 0, False, "save", False), ((1, 160, 60, 60, 160), "f32", 0, False, "bwd", False),
    ((1, 160, 60, 61, 20), "f32", 0, False, "bwd", True), ((1, 224, 100, 100, 7), "bf16", 0, False, "bwd", False), ((1, 260, 100, 100, 13), "bf16", 0, False, "bwd", True),
    # first of two passes: weights shared by few channels, large calls
    ((1, 136, 64, 64, 17), "bf16", 0, False, "bwd", False), ((1, 136, 64, 64, 8), "bf16", 0, False, "bwd", True), ((1, 252, 104, 104, 4), "bf16", 0, False, "bwd", False),
    ((1, 109, 104, 112, 109), "f16", 0, False, "bwd", False), ((1, 108, 104, 112, 27), "f16", 0, False, "bwd", True),
]


@pytest.mark.parametrize("shape,dtype,kchunk,logits,call,taken", LONGER, ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_calls_that_would_run_longer(shape, dtype, kchunk, logits, call, taken):
    from paper_2512_07884_amd import binding
    assert (binding.call_apart(*shape, {"f32": 0, "bf16": 1, "f16": 2}[dtype], call, kchunk, logits) in (1, 2)) == taken
