"""The library under HIP graph capture: forward + backward calls recorded once and replayed several times with changed inputs; every
replay must equal the eager result bit for bit.  Each kernel that a call can run is asked for by name: those of calls of few planes (a
workgroup per direction and their merge, half scans, a wave per direction), and, with such calls kept off these, the plane,
two-channel, tile, stream, per-stretch and any-size kernels, the two launches of the two-pass backward, the zero-fill kernel of the
split-group backward and the line-by-line kernels."""
import numpy as np
import pytest

from gpu_util import kernel_of, to_device
from paper_2512_07884_amd import workloads as WL

pytestmark = pytest.mark.gpu


def _captured_step(shape, kchunk=0):
    import torch
    import paper_2512_07884_amd as G
    B, C, H, W, Gr, dtype = shape
    cfg = WL.ScanConfig("graph", B, C, H, W, Gr, dtype, 15, 1.0, 71)
    inp = WL.make_inputs(cfg)
    d = {k: to_device(v, dtype) for k, v in inp.items()}
    outs = {k: torch.empty_like(d[s]) for k, s in (("y", "x"), ("hs", "lam"), ("gx", "x"), ("gw", "w"), ("gl", "lam"), ("gu", "lam"))}
    fwd, bwd, local = (G.gspn_scan_fwd_local, G.gspn_scan_bwd_local, {"kchunk": kchunk}) if kchunk else (G.gspn_scan_fwd, G.gspn_scan_bwd, {})

    def step():
        fwd(d["x"], d["w"], d["lam"], d["u"], outs["y"], outs["hs"], G=Gr, **local)
        bwd(d["gy"], d["x"], d["w"], d["lam"], d["u"], outs["hs"], outs["gx"], outs["gw"], outs["gl"], outs["gu"], G=Gr, **local)

    def snapshot():
        torch.cuda.synchronize()
        return {k: v.clone() for k, v in outs.items()}

    step()                                   # eager warm-up (also sets the kernels' LDS limits)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    gen = torch.Generator(device="cuda"); gen.manual_seed(5)
    bits = torch.int32 if dtype == "f32" else torch.int16
    for rep in range(3):
        # new inputs in place, eager reference, poison, replay, compare
        d["x"].copy_(torch.randn(d["x"].shape, device="cuda", generator=gen).to(d["x"].dtype))
        d["gy"].copy_(torch.randn(d["gy"].shape, device="cuda", generator=gen).to(d["gy"].dtype))
        step()
        ref = snapshot()
        for v in outs.values():
            v.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        got = snapshot()
        for k_ in outs:
            assert torch.equal(got[k_].view(bits), ref[k_].view(bits)), (shape, rep, k_)


@pytest.mark.parametrize("shape", [(2, 96, 28, 28, 2, "f32"), (2, 8, 56, 56, 2, "bf16"), (1, 4, 128, 128, 2, "bf16"),
                                   (1, 2, 256, 256, 1, "bf16")],
                         ids=lambda s: "x".join(map(str, s)))
def test_captured_training_step_replays_like_eager(shape):
    assert kernel_of(shape[:5], shape[5], "save") == kernel_of(shape[:5], shape[5], "bwd") == "apart"
    _captured_step(shape)


# shape, stretch, variable set, kernel of the forward call with h_save, of the backward call
KERNELS = [((1, 96, 14, 14, 8, "bf16"), 0, "", "small", "plane"), ((1, 2, 64, 2048, 1, "f16"), 0, "", "stream halves", "twopass/stream"),
           ((2, 8, 56, 56, 2, "bf16"), 0, "GSPN_NO_APART", "plane", "twopass/plane"), ((1, 4, 128, 128, 2, "bf16"), 0, "GSPN_NO_APART", "pair", "twopass/pair"),
           ((1, 2, 256, 256, 1, "bf16"), 0, "GSPN_NO_APART", "stream", "twopass/stream"), ((1, 8, 40, 72, 2, "f32"), 0, "GSPN_NO_APART", "tile", "twopass/tile"),
           ((1, 4, 43, 44, 1, "bf16"), 0, "GSPN_NO_APART", "any size", "tile"),
           ((1, 4, 128, 128, 2, "f32"), 32, "GSPN_NO_APART", "chunk", "twopass/chunk"), ((2, 6, 50, 83, 2, "f32"), 0, "GSPN_NO_APART", "any size", "any size"),
           ((2, 48, 64, 64, 8, "bf16"), 0, "GSPN_NO_APART", "any size", "twopass/any size"),
           ((2, 96, 28, 28, 2, "f32"), 0, "GSPN_NO_ANY_SIZE", "plane", "plane"), ((1, 3, 33, 35, 1, "bf16"), 0, "GSPN_FORCE_GENERIC", "line by line", "line by line")]


@pytest.mark.parametrize("shape,kchunk,knob,save,bwd", KERNELS, ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s).replace(" ", "-"))
def test_captured_training_step_on_each_kernel(shape, kchunk, knob, save, bwd, monkeypatch):
    if knob:
        monkeypatch.setenv(knob, "1")
    assert (kernel_of(shape[:5], shape[5], "save", kchunk), kernel_of(shape[:5], shape[5], "bwd", kchunk)) == (save, bwd)
    _captured_step(shape, kchunk)
