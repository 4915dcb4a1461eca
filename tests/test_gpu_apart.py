"""Calls of few planes, a workgroup per (plane, direction, range of lines), against the kernels that hold whole planes
(GSPN_NO_APART=1) and against the line-by-line kernels: lines of one wave at 1, 2 and 4 positions per lane, on either side of each
limit, and of several waves; lines that end inside a lane, a granule, a wave; one chunk of lines and many, ranges of whole stretches
and stretches that are no whole granules; planes that eight divides and such that it does not.

States, gu and x * e come from the same chain of FMAs as the line-by-line kernels': bit for bit.  Merged outputs are summed in fp32 in
another order or rounded up to four times on the other side."""
import ctypes

import pytest

from gpu_util import call_kernel

pytestmark = pytest.mark.gpu

# (B, C, H, W, G), dtype, kchunk, logits
CALLS = [
    ((1, 8, 20, 20, 1), "bf16", 0, False), ((1, 3, 21, 63, 1), "f32", 0, False), ((1, 8, 64, 64, 2), "f16", 0, True),
    ((1, 5, 65, 31, 1), "bf16", 0, True), ((2, 4, 127, 33, 2), "f32", 0, True), ((1, 8, 40, 128, 2), "f16", 0, False),
    ((1, 3, 129, 21, 1), "f32", 0, False), ((1, 8, 100, 167, 2), "bf16", 0, False), ((1, 4, 61, 255, 4), "f32", 0, False),
    ((1, 8, 256, 256, 8), "bf16", 0, False), ((1, 8, 255, 253, 4), "f16", 0, True), ((1, 4, 19, 257, 2), "bf16", 0, False),
    ((1, 2, 257, 30, 1), "f32", 0, True), ((1, 3, 470, 449, 3), "f16", 0, False), ((1, 2, 33, 703, 1), "f32", 0, False),
    ((1, 2, 601, 24, 1), "bf16", 0, True), ((1, 2, 1030, 23, 1), "f16", 0, False), ((1, 2, 21, 1201, 1), "bf16", 0, False),
    ((1, 96, 31, 45, 8), "bf16", 0, False), ((1, 128, 50, 83, 8), "f32", 0, False), ((1, 192, 24, 40, 8), "f32", 0, True),
    # stretches: ranges of one, of several, not of whole granules, the last one short; none (a stretch as long as the map)
    ((1, 8, 128, 128, 2), "f32", 32, False), ((1, 32, 64, 256, 4), "bf16", 8, False), ((1, 8, 70, 90, 1), "f16", 24, True),
    ((1, 4, 77, 50, 2), "bf16", 7, False), ((1, 4, 50, 77, 2), "f32", 6, True), ((1, 6, 45, 300, 2), "f16", 64, False),
    ((1, 4, 40, 40, 1), "bf16", 40, False), ((1, 3, 130, 27, 1), "f32", 1, False),
]


def apart(shape, dtype, call, kchunk, logits):
    from paper_2512_07884_amd import binding
    return binding.call_apart(*shape, {"f32": 0, "bf16": 1, "f16": 2}[dtype], call, kchunk, logits)


def inputs(shape, dtype, logits, slots=4):
    import torch
    B, C, H, W, Gr = shape
    td = {"bf16": torch.bfloat16, "f32": torch.float32, "f16": torch.float16}[dtype]
    g = torch.Generator(device="cuda"); g.manual_seed(H * 1000 + W + C)
    z = torch.randn((4, B, Gr, 3, H, W), generator=g, device="cuda")
    if not logits:
        # what is never read (taps outside the line) must stay out whatever it holds
        z[:2, :, :, 0, :, 0] = -1e30; z[:2, :, :, 2, :, -1] = -1e30; z[2:, :, :, 0, 0, :] = -1e30; z[2:, :, :, 2, -1, :] = -1e30
        z = torch.softmax(z, dim=3)
    z[:2, :, :, 0, :, 0] = float("nan"); z[:2, :, :, 2, :, -1] = float("inf"); z[2:, :, :, 0, 0, :] = float("nan"); z[2:, :, :, 2, -1, :] = float("nan")
    z[0, :, :, :, 0] = float("nan"); z[1, :, :, :, -1] = float("nan"); z[2, :, :, :, :, 0] = float("inf"); z[3, :, :, :, :, -1] = float("nan")
    if slots == 1:
        z = torch.softmax(torch.randn((1, B, Gr, 3, H, W), generator=g, device="cuda"), dim=3)
    r = lambda: torch.rand((slots, B, C, H, W), generator=g, device="cuda").to(td)
    return {"x": torch.randn((B, C, H, W), generator=g, device="cuda").to(td), "w": z.to(td), "lam": r(), "u": r(),
            "gy": torch.randn((B, C, H, W), generator=g, device="cuda").to(td)}


def close(got, ref, dtype, same):
    import torch
    # eight storage roundings of a sum in 16 bits; gw is summed in storage precision by the line-by-line kernels and left out there
    tol = {"bf16": 2e-2, "f16": 2.5e-3, "f32": 2e-5}[dtype]
    for n in got:
        a, b = got[n].float(), ref[n].float()
        assert torch.isfinite(a).all(), n
        if n in same:
            assert bool((got[n] == ref[n]).all()), (n, int((got[n] != ref[n]).sum()))
        e, scale = float((a - b).abs().max()), float(b.abs().max())
        assert e <= tol * scale, (n, e, scale)              # (gw of stretches of one line is 0 throughout)


@pytest.mark.parametrize("shape,dtype,kchunk,logits", CALLS, ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_against_whole_planes_and_line_by_line(shape, dtype, kchunk, logits, monkeypatch):
    import paper_2512_07884_amd as G
    from paper_2512_07884_amd import binding
    from test_gpu_differential import _run
    G.binding = binding
    for call in ("fwd", "save", "bwd"):
        assert apart(shape, dtype, call, kchunk, logits) == (1 if call == "fwd" or (call == "save" and dtype != "f32") else 2), call
    inp = inputs(shape, dtype, logits)
    got = _run(G, inp, shape[4], 15, kchunk, logits)
    # without h_save: the same y, bit for bit
    import torch
    y = torch.full_like(inp["x"], float("nan"))
    G.gspn_scan_fwd_logits(inp["x"], inp["w"], inp["lam"], inp["u"], y, G=shape[4], kchunk=kchunk or binding.GLOBAL_SCAN) if logits else \
        G.gspn_scan_fwd_local(inp["x"], inp["w"], inp["lam"], inp["u"], y, G=shape[4], kchunk=kchunk or binding.GLOBAL_SCAN)
    assert torch.equal(y, got["y"])
    monkeypatch.setenv("GSPN_NO_APART", "1")
    assert not any(apart(shape, dtype, call, kchunk, logits) for call in ("fwd", "save", "bwd"))
    # the kernels of whole planes round e to 16 bits and softmax in other orders where they are not the any-size kernel
    any_size = call_kernel(*shape, dtype, "save", kchunk, logits) == "any size" and call_kernel(*shape, dtype, "bwd", kchunk, logits) == "any size"
    close(got, _run(G, inp, shape[4], 15, kchunk, logits), dtype, ("hs", "gu", "gl", "gw") if any_size else ())
    monkeypatch.setenv("GSPN_FORCE_GENERIC", "1")
    ref = _run(G, inp, shape[4], 15, kchunk, logits)
    ref["gw"] = got["gw"]
    close(got, ref, dtype, ("hs", "gu") + (("gl",) if dtype != "f16" else ()))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_shared_parameters(dtype, monkeypatch):
    import torch
    import paper_2512_07884_amd as G
    from paper_2512_07884_amd.binding import GSPN_FLAG_SHARED_PARAMS as SHARED
    shape = (1, 6, 45, 70, 3)
    inp = inputs(shape, dtype, False, slots=1)
    out = []
    for _ in range(2):
        y, hs = torch.full_like(inp["x"], float("nan")), torch.full((4,) + tuple(inp["x"].shape), float("nan"), device="cuda", dtype=inp["x"].dtype)
        G.gspn_scan_fwd(inp["x"], inp["w"], inp["lam"], inp["u"], y, hs, G=3, flags=SHARED)
        b = {k: torch.full_like(hs, float("nan")) for k in ("gl", "gu")}
        gx, gw = torch.full_like(y, float("nan")), torch.full((4, 1, 3, 3, 45, 70), float("nan"), device="cuda", dtype=y.dtype)
        G.gspn_scan_bwd(inp["gy"], inp["x"], inp["w"], inp["lam"], inp["u"], hs, gx, gw, b["gl"], b["gu"], G=3, flags=SHARED)
        out.append({"y": y, "hs": hs, "gx": gx, "gw": gw, **b})
        monkeypatch.setenv("GSPN_NO_APART", "1")
    close(out[0], out[1], dtype, ("hs", "gu", "gl", "gw"))


def test_workspace_of_the_c_call_and_of_other_streams():
    """The C entry point takes what gspn_fwd_workspace_bytes says and refuses less; without a workspace it runs on whole planes.  The
    Python call on a stream of its own, as an object and as an address, gives the same bits."""
    import torch
    import paper_2512_07884_amd as G
    from paper_2512_07884_amd import binding
    shape = (1, 8, 50, 70, 2)
    B, C, H, W, Gr = shape
    inp = inputs(shape, "bf16", False)
    lib = binding.load_library()
    n = binding.gspn_fwd_workspace_bytes(B, C, H, W, Gr, dtype=1)
    assert n == 16 * B * C * H * W and binding.gspn_fwd_workspace_bytes(B, C, H, W, Gr, dtype=0, has_h_save=True) == 0
    assert binding.gspn_fwd_workspace_bytes(2, 1024, 128, 128, 16, dtype=1) == 0 and binding.gspn_fwd_workspace_bytes(B, C, H, W, Gr, dir_mask=7) == 0
    ys = [torch.full_like(inp["x"], float("nan")) for _ in range(5)]
    ws = torch.empty(n + 16, dtype=torch.uint8, device="cuda")
    p = [inp[k].data_ptr() for k in ("x", "w", "lam", "u")]
    call = lambda y, w, size: lib.gspn_scan_fwd_workspace(*p, y.data_ptr(), None, w, size, B, C, H, W, Gr, 1 << 14, 0, 15, 1, 0,
                                                          ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert call(ys[0], ws.data_ptr(), n) == 0 and call(ys[1], None, 0) == 0
    assert call(ys[2], ws.data_ptr(), n - 1) == 2 and call(ys[2], ws.data_ptr() + 4, n) == 4
    torch.cuda.synchronize()
    assert bool(torch.isnan(ys[2].float()).all())                    # refused calls launch nothing
    side = torch.cuda.Stream()
    G.gspn_scan_fwd(inp["x"], inp["w"], inp["lam"], inp["u"], ys[2], G=Gr, stream=side)
    G.gspn_scan_fwd(inp["x"], inp["w"], inp["lam"], inp["u"], ys[3], G=Gr, stream=side.cuda_stream)
    side.synchronize()
    G.gspn_scan_fwd(inp["x"], inp["w"], inp["lam"], inp["u"], ys[4], G=Gr, stream=0)
    torch.cuda.synchronize()
    for y in ys[2:]:
        assert torch.equal(y, ys[0])
    assert float((ys[1].float() - ys[0].float()).abs().max() / ys[0].float().abs().max()) <= 2e-2


def test_captured_forward_call_keeps_its_workspace():
    """A captured call's workspace lives in the graph: replays between eager work that allocates give the eager result each time."""
    import torch
    import paper_2512_07884_amd as G
    shape = (1, 16, 60, 72, 2)
    inp = inputs(shape, "bf16", False)
    y, ref = torch.empty_like(inp["x"]), torch.empty_like(inp["x"])
    run = lambda out: G.gspn_scan_fwd(inp["x"], inp["w"], inp["lam"], inp["u"], out, G=2)
    run(y)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run(y)
    for i in range(4):
        inp["x"].copy_(torch.randn(inp["x"].shape, device="cuda").to(inp["x"].dtype))
        run(ref)
        junk = [torch.full((1 << 20,), float("nan"), device="cuda") for _ in range(4)]
        y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, ref), i
        del junk
