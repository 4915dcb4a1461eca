"""Small maps, a wave per direction, against the line-by-line kernels: lines of each lane group (8, 16, 32) and one short of and beyond it, maps
of one line, planes that do not fill the last workgroup, groups that begin inside one, stretches, logits, shared parameters.

The states are the same chain of FMAs: bit for bit.  y is summed in fp32 and rounded once."""
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [((1, 384, 14, 14, 8), 0), ((1, 13, 7, 8, 1), 0), ((3, 7, 8, 5, 7), 3), ((2, 9, 9, 1, 3), 0), ((1, 5, 1, 16, 5), 0), ((1, 21, 16, 12, 3), 5),
          ((2, 6, 15, 9, 2), 4), ((1, 7, 17, 23, 7), 0), ((5, 3, 4, 32, 1), 8), ((1, 8, 31, 11, 2), 6), ((1, 2, 1, 1, 1), 0), ((1, 1, 32, 3, 1), 0)]


@pytest.mark.parametrize("logits", [False, True])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("shape,kchunk", SHAPES, ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_small(shape, kchunk, dtype, logits, monkeypatch):
    import torch
    from paper_2512_07884_amd import binding
    B, C, H, W, Gr = shape
    code = {"f32": 0, "bf16": 1, "f16": 2}[dtype]
    assert binding.call_apart(*shape, code, "fwd", kchunk, logits) == binding.call_apart(*shape, code, "save", kchunk, logits) == 4
    td = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}[dtype]
    slots = 1 if C == 21 else 4
    g = torch.Generator(device="cuda"); g.manual_seed(H * 100 + W)
    x, lam, u = (torch.randn(s + (C, H, W), generator=g, device="cuda").to(td) for s in ((B,), (slots, B), (slots, B)))
    w = torch.randn((slots, B, Gr, 3, H, W), generator=g, device="cuda")
    if not logits: w = torch.softmax(w, dim=3)
    if slots == 4:                                            # what is never read must stay out whatever it holds
        w[:2, :, :, 0, :, 0] = float("nan"); w[:2, :, :, 2, :, -1] = float("inf")
        w[2:, :, :, 0, 0, :] = float("nan"); w[2:, :, :, 2, -1, :] = float("nan")
        w[0, :, :, :, 0] = float("nan"); w[1, :, :, :, -1] = float("nan"); w[2, :, :, :, :, 0] = float("inf"); w[3, :, :, :, :, -1] = float("nan")
    w = w.to(td)
    scan = binding.gspn_scan_fwd_logits if logits else binding.gspn_scan_fwd_local

    def run(save):
        y, hs = torch.full_like(x, float("nan")), torch.full((4,) + tuple(x.shape), float("nan"), device="cuda", dtype=td) if save else None
        scan(x, w, lam, u, y, hs, G=Gr, kchunk=kchunk or binding.GLOBAL_SCAN, flags=binding.GSPN_FLAG_SHARED_PARAMS if slots == 1 else 0)
        return y, hs
    y, hs = run(True)
    assert torch.equal(run(False)[0], y)
    monkeypatch.setenv("GSPN_FORCE_GENERIC", "1"); binding.gspn_reload_env()
    ry, rhs = run(True)
    monkeypatch.undo(); binding.gspn_reload_env()
    assert torch.equal(hs, rhs)
    # every rounding is by at most eps / 2 of a partial sum of the terms u * h: up to four on either side in fp32, one here and four there
    # in 16 bits (subnormal numbers of fp16: by 2^-25)
    eps = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11, "f32": 2.0 ** -23}[dtype]
    bound = 5 * eps * (u.double() * hs.double()).abs().sum(dim=0) + 2.0 ** -22
    assert bool(((y.double() - ry.double()).abs() <= bound).all())
