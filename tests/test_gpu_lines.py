"""A wave per line (gspn_lines*.hip) against the line-by-line kernels: lines of one to four waves and of two positions per lane, on either
side of each limit; sides that end inside a unit, a granule, a chunk, a wave; the last granule of a tensor; weights of each channel's
own, shared ones, one set for all directions.

States, gu and x * e come from the same chain of FMAs as the line-by-line kernels': bit for bit.  The merged outputs are sums of four
products in fp32, here and there in another order, rounded up to four times there."""
import pytest

from test_gpu_apart import close, inputs

pytestmark = pytest.mark.gpu

# (B, C, H, W, G), dtype, logits, forward and backward calls that run on it
CALLS = [
    ((1, 72, 14, 36, 2), "bf16", False, "f"), ((2, 36, 33, 16, 2), "bf16", False, "f"), ((1, 66, 37, 35, 66), "f16", False, "f"), ((1, 66, 20, 37, 66), "bf16", False, "f"),
    ((1, 300, 63, 64, 12), "bf16", False, "fsb"), ((1, 300, 64, 63, 12), "f16", False, "fsb"), ((1, 400, 47, 61, 16), "f32", False, "fs"), ((1, 640, 33, 36, 8), "f32", False, "fb"),
    ((1, 400, 61, 39, 16), "bf16", True, "fsb"), ((2, 304, 49, 53, 8), "f32", True, "fsb"), ((1, 480, 8, 63, 20), "bf16", False, "f"), ((1, 760, 31, 17, 760), "bf16", False, "f"),
    ((1, 800, 37, 35, 800), "bf16", False, "fsb"), ((1, 1100, 26, 28, 1100), "f16", True, "fs"), ((1, 2100, 33, 32, 2100), "f16", True, "fs"), ((1, 256, 16, 16, 4), "bf16", False, "fb"),
    ((1, 1344, 14, 14, 84), "f32", True, "b"), ((1, 150, 9, 15, 10), "f32", False, "b"), ((1, 600, 29, 40, 25), "bf16", False, "fb"), ((1, 600, 35, 40, 25), "bf16", False, "fsb"),
    # lines of several waves
    ((1, 150, 100, 65, 6), "bf16", False, "fs"), ((1, 160, 112, 110, 10), "f16", False, "fs"), ((1, 512, 113, 111, 16), "bf16", False, "fs"),
    ((1, 512, 128, 127, 16), "f16", True, "fs"), ((1, 160, 129, 130, 5), "bf16", False, "fs"), ((1, 150, 160, 161, 6), "f16", False, "fs"),
    ((1, 150, 208, 104, 150), "bf16", False, "fs"), ((1, 160, 144, 201, 4), "bf16", False, "fs"), ((1, 512, 105, 160, 16), "bf16", True, "fs"),
    ((1, 512, 80, 104, 8), "f32", False, "b"), ((1, 512, 112, 120, 8), "bf16", False, "b"), ((1, 288, 112, 68, 18), "f32", True, "b"),
    # ... of the reverse sweep: two positions per lane in fp32, halves of e in 16 bits with the states that two to four waves of a line hand over
    ((1, 400, 128, 128, 5), "f32", False, "b"), ((1, 400, 128, 120, 5), "f32", True, "b"), ((1, 512, 144, 128, 512), "f32", False, "b"), ((1, 256, 80, 112, 8), "bf16", False, "b"),
    ((1, 256, 80, 112, 8), "f16", True, "b"), ((1, 256, 144, 128, 8), "bf16", False, "b"), ((1, 256, 144, 64, 8), "bf16", True, "b"), ((1, 256, 208, 64, 8), "bf16", False, "b"),
]


def gradient_of_weights(inp, dtype, logits, h):
    """gw in 64 bits from the stored states.  Weights that are never read hold NaN and infinities: 0 there, whatever they are."""
    import numpy as np
    from oracle import gspn_oracle as O
    f = lambda t: t.float().cpu().numpy().astype(np.float64)
    w = np.nan_to_num(f(inp["w"]), nan=0.0, posinf=0.0, neginf=0.0)
    lam, u = f(inp["lam"]), f(inp["u"])
    if w.shape[0] == 1:
        w, lam, u = (np.repeat(t, 4, 0) for t in (w, lam, u))
    return (O.scan_bwd_logits if logits else O.scan_bwd)(f(inp["gy"]), f(inp["x"]), w, lam, u, f(h), 15)[1]


def check_gradient_of_weights(got, inp, dtype, logits, h):
    import numpy as np
    from gpu_util import TOL
    want = gradient_of_weights(inp, dtype, logits, h)
    a = got["gw"].float().cpu().numpy().astype(np.float64)
    assert np.isfinite(a).all()
    # e and the sums in fp32, one rounding to storage (with logits the sum of products w gw, again in fp32)
    assert np.max(np.abs(a - want)) <= TOL[dtype] * np.max(np.abs(want))


def run(monkeypatch, knob, call, inp, shape, dtype, logits, h=None, shared=False):
    import torch
    import paper_2512_07884_amd as G
    from paper_2512_07884_amd import binding
    monkeypatch.setenv("GSPN_FORCE_GENERIC", knob); binding.gspn_reload_env()
    x, lam, w = inp["x"], inp["lam"], inp["w"]
    fresh = lambda t: torch.full_like(t, float("nan"))
    kw = {"G": shape[4], **({"flags": binding.GSPN_FLAG_SHARED_PARAMS} if shared else {})}
    if call == "b":
        four = lambda t: torch.full((4, *t.shape[1:]), float("nan"), dtype=t.dtype, device="cuda")
        o = {"gx": fresh(x), "gw": four(w), "glam": four(lam), "gu": four(lam)}
        (G.gspn_scan_bwd_logits if logits else G.gspn_scan_bwd)(inp["gy"], x, w, lam, inp["u"], h, *o.values(), **kw)
    else:
        o = {"y": fresh(x), "h": torch.full((4, *x.shape), float("nan"), dtype=x.dtype, device="cuda") if call == "s" else None}
        (G.gspn_scan_fwd_logits if logits else G.gspn_scan_fwd)(x, w, lam, inp["u"], o["y"], o["h"], **kw)
        if call == "f":
            del o["h"]
    torch.cuda.synchronize()
    return o


@pytest.mark.parametrize("shape,dtype,logits,calls", CALLS, ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_against_line_by_line(shape, dtype, logits, calls, monkeypatch):
    import torch
    from paper_2512_07884_amd import binding
    code = {"f32": 0, "bf16": 1, "f16": 2}[dtype]
    for call in calls:
        assert binding.running_kernel(*shape, code, {"f": "fwd", "s": "save", "b": "bwd"}[call], 0, logits) == "lines", call
    inp = inputs(shape, dtype, logits)
    ref = run(monkeypatch, "1", "s", inp, shape, dtype, logits)
    for call in calls:
        if call == "b":
            want = run(monkeypatch, "1", "b", inp, shape, dtype, logits, ref["h"])
            got = run(monkeypatch, "0", "b", inp, shape, dtype, logits, ref["h"])
            assert torch.equal(got["gu"], want["gu"])
            if dtype == "f32":
                assert torch.equal(got["glam"], want["glam"])
                close(got, want, dtype, ())
            else:
                close({k: got[k] for k in ("gx", "glam")}, want, dtype, ())       # (gw: summed in storage precision line by line)
                check_gradient_of_weights(got, inp, dtype, logits, ref["h"])
            again = run(monkeypatch, "0", "b", inp, shape, dtype, logits, ref["h"])
            assert all(torch.equal(again[n], got[n]) for n in got)
        else:
            got = run(monkeypatch, "0", call, inp, shape, dtype, logits)
            if call == "s":
                assert torch.equal(got["h"], ref["h"])
            close({"y": got["y"]}, ref, dtype, ())
            again = run(monkeypatch, "0", call, inp, shape, dtype, logits)
            assert torch.equal(again["y"], got["y"])


@pytest.mark.parametrize("shape,dtype", [((1, 300, 47, 61, 12), "bf16"), ((1, 160, 101, 105, 5), "f16"), ((1, 256, 80, 112, 8), "f16")],
                         ids=["47x61", "101x105", "80x112"])
def test_one_set_of_parameters(shape, dtype, monkeypatch):
    import torch
    from paper_2512_07884_amd import binding
    assert binding.running_kernel(*shape, {"bf16": 1, "f16": 2}[dtype], "bwd" if shape[2] == 80 else "save") == "lines"
    inp = inputs(shape, dtype, False, slots=1)
    ref = run(monkeypatch, "1", "s", inp, shape, dtype, False, shared=True)
    got = run(monkeypatch, "0", "s", inp, shape, dtype, False, shared=True)
    assert torch.equal(got["h"], ref["h"])
    close({"y": got["y"]}, ref, dtype, ())
    if binding.running_kernel(*shape, {"bf16": 1, "f16": 2}[dtype], "bwd") == "lines":
        want = run(monkeypatch, "1", "b", inp, shape, dtype, False, ref["h"], shared=True)
        got = run(monkeypatch, "0", "b", inp, shape, dtype, False, ref["h"], shared=True)
        assert torch.equal(got["gu"], want["gu"])
        close({k: got[k] for k in ("gx", "glam")}, want, dtype, ())
        check_gradient_of_weights(got, inp, dtype, False, ref["h"])
