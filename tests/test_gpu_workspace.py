"""The forward call of few planes in a capture begun by the HIP runtime's own calls: it takes no memory from torch's allocator, so that
replays write nothing but the call's outputs."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


def test_capture_by_the_runtimes_own_calls(monkeypatch):
    import torch
    import paper_2512_07884_amd as G
    from paper_2512_07884_amd import binding
    hip = binding.load_library()                            # (a lookup in the library reaches the runtime it is linked to)
    B, C, H, W, Gr = shape = (1, 16, 60, 72, 2)
    assert binding.call_apart(*shape, 1, "fwd") == 1
    n = binding.gspn_fwd_workspace_bytes(*shape, dtype=1)
    g = torch.Generator(device="cuda"); g.manual_seed(3)
    r = lambda *s: torch.rand(s, generator=g, device="cuda").to(torch.bfloat16)
    x, lam, u = r(B, C, H, W), r(4, B, C, H, W), r(4, B, C, H, W)
    w = torch.softmax(r(4, B, Gr, 3, H, W).float(), dim=3).to(torch.bfloat16)
    y, ref = torch.empty_like(x), torch.empty_like(x)
    run = lambda out, **k: G.gspn_scan_fwd(x, w, lam, u, out, G=Gr, **k)
    run(y)
    monkeypatch.setenv("GSPN_NO_APART", "1")
    run(ref)                                                # what the call gives without a workspace
    monkeypatch.setenv("GSPN_NO_APART", "0")
    torch.cuda.synchronize()

    def ok(status):
        assert status == 0, status
    stream, graph, instance = ctypes.c_void_p(), ctypes.c_void_p(), ctypes.c_void_p()
    ok(hip.hipStreamCreateWithFlags(ctypes.byref(stream), 1))
    ok(hip.hipStreamBeginCapture(stream, 2))
    try:
        before = torch.cuda.memory_allocated()
        run(y, stream=stream.value)
        assert torch.cuda.memory_allocated() == before
    finally:
        ok(hip.hipStreamEndCapture(stream, ctypes.byref(graph)))
    ok(hip.hipGraphInstantiate(ctypes.byref(instance), graph, None, None, ctypes.c_size_t(0)))
    canaries = [torch.full((n,), 0x5a, dtype=torch.uint8, device="cuda") for _ in range(4)]
    for i in range(3):
        y.fill_(float("nan"))
        torch.cuda.synchronize()
        ok(hip.hipGraphLaunch(instance, stream))
        ok(hip.hipStreamSynchronize(stream))
        assert torch.equal(y, ref), i
        assert all(bool((c == 0x5a).all()) for c in canaries), i
    ok(hip.hipGraphExecDestroy(instance)); ok(hip.hipGraphDestroy(graph)); ok(hip.hipStreamDestroy(stream))
