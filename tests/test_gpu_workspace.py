"""The memory of forward calls of few planes: a capture begun by the HIP runtime's own calls takes none from torch's allocator, so that
replays write nothing but the call's outputs; the call with a workspace of the caller's."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


SHAPE = (1, 16, 60, 72, 2)


def tensors():
    import torch
    B, C, H, W, Gr = SHAPE
    g = torch.Generator(device="cuda"); g.manual_seed(3)
    r = lambda *s: torch.rand(s, generator=g, device="cuda").to(torch.bfloat16)
    return r(B, C, H, W), torch.softmax(r(4, B, Gr, 3, H, W).float(), dim=3).to(torch.bfloat16), r(4, B, C, H, W), r(4, B, C, H, W)


def test_capture_by_the_runtimes_own_calls(monkeypatch):
    import torch
    import paper_2512_07884_amd as G
    from paper_2512_07884_amd import binding
    hip = binding.load_library()                            # (a lookup in the library reaches the runtime it is linked to)
    assert binding.call_apart(*SHAPE, 1, "fwd") == 1
    n, Gr = binding.gspn_fwd_workspace_bytes(*SHAPE, dtype=1), SHAPE[4]
    x, w, lam, u = tensors()
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


@pytest.mark.parametrize("logits,kchunk", [(False, 1 << 14), (True, 1 << 14), (False, 24), (True, 24)])
def test_workspace_of_the_callers(logits, kchunk, monkeypatch):
    import torch
    import paper_2512_07884_amd as G
    x, w, lam, u = tensors()
    n = G.gspn_fwd_workspace_bytes(*SHAPE, kchunk, logits, dtype=1)
    ws = torch.full((n,), 0xff, dtype=torch.uint8, device="cuda")
    ref, without, got = (torch.full_like(x, float("nan")) for _ in range(3))
    (G.gspn_scan_fwd_logits if logits else G.gspn_scan_fwd_local)(x, w, lam, u, ref, G=2, kchunk=kchunk)
    call = lambda out, space, **k: G.gspn_scan_fwd_workspace(x, w, lam, u, out, None, space, kchunk=kchunk, logits=logits, G=2, **k)
    before = torch.cuda.memory_allocated()
    call(got, ws)
    call(without, None)
    assert torch.cuda.memory_allocated() == before and torch.equal(got, ref)
    monkeypatch.setenv("GSPN_NO_APART", "1")
    (G.gspn_scan_fwd_logits if logits else G.gspn_scan_fwd_local)(x, w, lam, u, ref, G=2, kchunk=kchunk)
    assert torch.equal(without, ref)
    monkeypatch.setenv("GSPN_NO_APART", "0")
    with pytest.raises(G.GspnError):
        call(got, ws[:n - 1])
    for bad in (torch.empty(n, dtype=torch.uint8), torch.empty((2 * n,), dtype=torch.uint8, device="cuda")[::2]):
        with pytest.raises(ValueError):
            call(got, bad)
