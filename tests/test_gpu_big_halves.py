"""Large maps of few planes, a direction per workgroup and half a scan per launch, against one workgroup per plane (GSPN_NO_APART=1):
each width of the vertical kernel, with and without waves that have no rows, both halves' states handed over, shared parameters.

The states come from the same chain of FMAs: bit for bit.  Per pixel y takes the same four terms, the two of a pass of launches in the other
order in half of the plane: three roundings to the storage type on either side, and fp32 sums."""
import pytest

pytestmark = pytest.mark.gpu

CALLS = [((1, 128, 576, 256, 8), "bf16", 4), ((1, 128, 640, 512, 8), "f16", 1), ((1, 3, 960, 1024, 3), "f32", 4), ((1, 40, 1024, 1024, 4), "bf16", 4),
         ((1, 2, 64, 2048, 1), "f16", 4), ((1, 2, 1024, 2048, 2), "f32", 4), ((1, 2, 832, 2048, 1), "bf16", 1)]


@pytest.mark.parametrize("save", [False, True])
@pytest.mark.parametrize("shape,dtype,slots", CALLS, ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_halves(shape, dtype, slots, save, monkeypatch):
    import torch
    from paper_2512_07884_amd import binding
    B, C, H, W, Gr = shape
    code = {"f32": 0, "bf16": 1, "f16": 2}[dtype]
    assert binding.call_apart(*shape, code, "save" if save else "fwd") == 3
    td = {"bf16": torch.bfloat16, "f32": torch.float32, "f16": torch.float16}[dtype]
    g = torch.Generator(device="cuda"); g.manual_seed(H + W)
    r = lambda *s: torch.rand(s, generator=g, device="cuda").to(td)
    x, lam, u = torch.randn((B, C, H, W), generator=g, device="cuda").to(td), r(slots, B, C, H, W), r(slots, B, C, H, W)
    w = torch.softmax(torch.randn((slots, B, Gr, 3, H, W), generator=g, device="cuda"), dim=3)
    if slots == 4:                                            # what is never read must stay out whatever it holds
        w[:2, :, :, 0, :, 0] = float("nan"); w[:2, :, :, 2, :, -1] = float("inf")
        w[2:, :, :, 0, 0, :] = float("nan"); w[2:, :, :, 2, -1, :] = float("nan")
        w[0, :, :, :, 0] = float("nan"); w[1, :, :, :, -1] = float("nan"); w[2, :, :, :, :, 0] = float("inf"); w[3, :, :, :, :, -1] = float("nan")
    w = w.to(td)
    out = []
    for off in ("1", "0"):
        monkeypatch.setenv("GSPN_NO_APART", off); binding.gspn_reload_env()
        y, hs = torch.full_like(x, float("nan")), torch.full((4,) + tuple(x.shape), float("nan"), device="cuda", dtype=td) if save else None
        binding.gspn_scan_fwd(x, w, lam, u, y, hs, G=Gr, flags=binding.GSPN_FLAG_SHARED_PARAMS if slots == 1 else 0)
        out.append((y, hs))
    monkeypatch.undo(); binding.gspn_reload_env()
    y0, y1 = out[0][0], out[1][0]
    if save: assert torch.equal(out[0][1], out[1][1])
    # three roundings on either side, each by at most eps / 2 of a partial sum of four terms, which may be twice as large as the largest y
    eps = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11, "f32": 2.0 ** -23}[dtype]
    assert (y1.double() - y0.double()).abs().max().item() <= 6 * eps * y0.abs().max().item()
    assert torch.isfinite(y1).all()
