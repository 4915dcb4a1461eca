"""Calls on either side of the lines between the plane / tile kernels and the any-size kernel (planes, pixels, row lengths, channels in
flight): forward with h_save and backward against the line-by-line kernels, and each on the kernel that its rule says.  The plans
keep their names on both sides; every line by itself is in test_kernel_choice.py."""
import pytest

from gpu_util import call_kernel

pytestmark = pytest.mark.gpu

# (B, C, H, W, G), dtype, kchunk, logits, forward plan, kernel of the forward call with h_save and of the backward call
CALLS = [((3, 21, 14, 16, 7), "bf16", 0, False, "plane", "plane", "twopass/plane"), ((4, 16, 14, 16, 4), "bf16", 0, False, "plane", "any size", "plane"),
         ((4, 16, 14, 14, 4), "f32", 0, False, "plane", "plane", "plane"), ((8, 128, 14, 16, 8), "f16", 0, False, "plane", "any size", "plane"),
         ((5, 205, 14, 16, 5), "bf16", 0, False, "plane", "plane", "twopass/plane"), ((4, 128, 28, 28, 8), "f32", 0, True, "plane", "any size", "any size"),
         ((4, 132, 28, 28, 12), "f32", 0, True, "plane", "plane", "twopass/plane"), ((2, 48, 56, 56, 4), "bf16", 14, True, "plane", "any size", "twopass/any size"),
         ((2, 64, 32, 32, 64), "f16", 0, False, "plane", "any size", "any size"), ((1, 31, 80, 72, 1), "bf16", 0, False, "tile", "tile", "twopass/tile"),
         ((1, 32, 80, 72, 1), "bf16", 0, False, "tile", "any size", "twopass/any size"), ((1, 32, 80, 64, 4), "f32", 24, False, "tile", "any size", "twopass/any size"),
         ((1, 32, 156, 128, 2), "f32", 0, False, "tile", "any size", "twopass/any size"), ((1, 32, 240, 96, 2), "f32", 0, False, "tile", "tile", "twopass/tile"),
         ((2, 512, 40, 96, 8), "bf16", 0, False, "tile", "any size", "twopass/any size"), ((4, 256, 36, 104, 16), "f16", 0, False, "tile", "any size", "twopass/any size"),
         # fp32 rows that are not whole granules; 16-bit rows of 224 bytes; a plane backward whose workgroups fill the CUs
         ((4, 130, 20, 34, 10), "f32", 0, False, "plane", "plane", "twopass/plane"), ((2, 72, 18, 18, 9), "f32", 12, False, "plane", "plane", "any size"),
         ((1, 48, 34, 112, 6), "bf16", 0, False, "tile", "tile", "twopass/tile"), ((1, 48, 34, 112, 6), "f16", 0, True, "tile", "any size", "twopass/any size"),
         ((18, 256, 26, 26, 64), "f32", 0, False, "plane", "plane", "any size"), ((24, 256, 26, 26, 64), "f32", 0, False, "plane", "plane", "plane")]


@pytest.mark.parametrize("shape,dtype,kchunk,logits,plan,save,bwd", CALLS, ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_either_side_of_the_lines(shape, dtype, kchunk, logits, plan, save, bwd, monkeypatch):
    import torch
    import paper_2512_07884_amd as G
    from paper_2512_07884_amd import binding
    from test_gpu_differential import _rel, _run
    G.binding = binding
    B, C, H, W, Gr = shape
    td, dt = {"bf16": (torch.bfloat16, 1), "f32": (torch.float32, 0), "f16": (torch.float16, 2)}[dtype]
    k = kchunk if kchunk else binding.GLOBAL_SCAN
    assert (G.gspn_fwd_logits_plan if logits else G.gspn_fwd_local_plan)(B, C, H, W, Gr, k, 15, dt, 0, True) == plan
    assert (call_kernel(*shape, dtype, "save", kchunk, logits), call_kernel(*shape, dtype, "bwd", kchunk, logits)) == (save, bwd)
    g = torch.Generator(device="cuda"); g.manual_seed(B * C + H + W)
    z = torch.randn((4, B, Gr, 3, H, W), generator=g, device="cuda")
    if not logits:
        z[:2, :, :, 0, :, 0] = -1e30; z[:2, :, :, 2, :, -1] = -1e30; z[2:, :, :, 0, 0, :] = -1e30; z[2:, :, :, 2, -1, :] = -1e30
        z = torch.softmax(z, dim=3)
    inp = {"x": torch.randn((B, C, H, W), generator=g, device="cuda").to(td), "w": z.to(td),
           "lam": torch.rand((4, B, C, H, W), generator=g, device="cuda").to(td),
           "u": torch.rand((4, B, C, H, W), generator=g, device="cuda").to(td),
           "gy": torch.randn((B, C, H, W), generator=g, device="cuda").to(td)}
    fast = _run(G, inp, Gr, 15, kchunk, logits)
    monkeypatch.setenv("GSPN_FORCE_GENERIC", "1")
    ref = _run(G, inp, Gr, 15, kchunk, logits)
    monkeypatch.delenv("GSPN_FORCE_GENERIC", raising=False)
    for n in fast:
        # the line-by-line kernels sum gw over a group in storage precision, one rounding per channel
        tol = {"bf16": 2e-2, "f16": 2.5e-3, "f32": 2e-5}[dtype] * (max(1.0, C / Gr / 8) if n == "gw" else 1.0)
        e = _rel(fast[n].float(), ref[n].float())
        assert e <= tol, (n, e, tol)
