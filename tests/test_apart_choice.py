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
    # per-stretch kernels: many short stretches of a small call
    ((1, 16, 128, 128, 8), "bf16", 16, False, "bwd", False), ((1, 16, 128, 128, 8), "bf16", 32, False, "bwd", True), ((1, 16, 128, 128, 2), "bf16", 16, False, "bwd", True),
    ((1, 4, 64, 64, 2), "f32", 8, False, "bwd", False), ((1, 3, 64, 64, 1), "f32", 8, False, "bwd", True), ((1, 4, 64, 64, 2), "f32", 32, False, "bwd", True),
    ((1, 16, 128, 128, 8), "f32", 8, False, "bwd", True), ((1, 7, 128, 128, 1), "f32", 4, False, "fwd", False), ((1, 8, 128, 128, 1), "f32", 4, False, "fwd", True),
    ((1, 7, 128, 128, 1), "f32", 16, False, "fwd", True), ((1, 12, 128, 128, 2), "bf16", 8, False, "fwd", True),
    # stretches begun inside a granule beside many vertical ones, on the any-size and the stream kernel
    ((1, 90, 384, 384, 45), "f32", 37, False, "fwd", False), ((1, 90, 384, 384, 45), "f32", 36, False, "fwd", True), ((1, 90, 384, 384, 18), "f32", 37, False, "fwd", True),
    ((1, 64, 384, 384, 32), "f32", 37, False, "fwd", True), ((1, 90, 384, 384, 45), "f32", 97, False, "fwd", True), ((1, 87, 384, 384, 29), "bf16", 37, False, "bwd", False),
    ((1, 72, 512, 256, 24), "bf16", 37, False, "fwd", False), ((1, 72, 512, 256, 24), "bf16", 40, False, "fwd", True), ((1, 76, 256, 256, 76), "f32", 37, False, "bwd", False),
    # ... others, weights of each channel's own
    ((1, 124, 432, 144, 124), "f16", 16, False, "fwd", False), ((1, 96, 432, 144, 96), "f16", 16, False, "fwd", True), ((1, 124, 432, 144, 62), "f16", 16, False, "fwd", True),
    ((1, 124, 432, 144, 124), "f16", 144, False, "fwd", True), ((1, 100, 100, 90, 100), "bf16", 8, False, "bwd", False), ((1, 100, 100, 90, 50), "bf16", 8, False, "bwd", True),
    # first of two passes, large calls
    ((1, 256, 128, 80, 16), "bf16", 0, False, "bwd", False), ((1, 256, 104, 80, 16), "bf16", 0, False, "bwd", True), ((1, 256, 128, 80, 16), "f32", 0, False, "bwd", True),
    # narrow maps: high ones in 16 bits
    ((1, 136, 192, 40, 8), "bf16", 0, False, "fwd", False), ((1, 128, 192, 40, 8), "bf16", 0, False, "fwd", True), ((1, 136, 168, 46, 8), "bf16", 0, True, "fwd", True),
    ((1, 136, 180, 42, 8), "bf16", 0, False, "fwd", True), ((1, 136, 180, 42, 8), "bf16", 0, True, "fwd", False), ((1, 136, 180, 42, 8), "f32", 0, True, "save", True),
    ((1, 190, 416, 42, 2), "f16", 0, False, "bwd", False), ((1, 190, 416, 46, 2), "f16", 0, False, "bwd", True), ((1, 190, 128, 42, 2), "f16", 0, True, "bwd", True),
    # ... few channels to a weight map
    ((1, 136, 24, 200, 34), "bf16", 0, False, "fwd", False), ((1, 136, 25, 200, 34), "bf16", 0, False, "fwd", True), ((1, 136, 24, 200, 17), "bf16", 0, False, "fwd", True),
    ((1, 136, 24, 200, 34), "bf16", 0, False, "bwd", True), ((1, 136, 16, 200, 34), "f32", 0, False, "save", False), ((1, 136, 20, 200, 34), "f32", 0, False, "save", True),
    ((1, 136, 200, 16, 34), "f32", 0, False, "save", True),
    # ... calls that a limit on large, square or whole-granule maps of few planes once kept off: shorter so
    ((1, 72, 256, 256, 72), "bf16", 0, False, "fwd", True), ((1, 126, 227, 227, 126), "f16", 0, False, "fwd", True), ((2, 144, 64, 64, 18), "bf16", 0, True, "save", True),
    ((1, 256, 40, 40, 8), "bf16", 0, True, "fwd", True), ((1, 160, 60, 60, 160), "f32", 0, False, "bwd", True), ((1, 224, 100, 100, 7), "bf16", 0, False, "bwd", True),
    ((1, 136, 64, 64, 17), "bf16", 0, False, "bwd", True),
]


@pytest.mark.parametrize("shape,dtype,kchunk,logits,call,taken", LONGER, ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_calls_that_would_run_longer(shape, dtype, kchunk, logits, call, taken):
    from paper_2512_07884_amd import binding
    assert (binding.call_apart(*shape, {"f32": 0, "bf16": 1, "f16": 2}[dtype], call, kchunk, logits) in (1, 2)) == taken
