"""The any-size kernel in each of its launch shapes, which every call is asked for: one chunk of lines in LDS or two, both directions
of an axis at once or one after the other, output merged in LDS or in global memory, one, two and four workgroups per CU, lines of
one wave or of several that meet, one or two granules per thread, one to four chunks in all (a pipeline that is never full, the crossing of the directions in the first, a middle and the
last chunk).  Calls of few planes and four directions run a workgroup per direction here and these launch shapes in
test_gpu_whole_planes.  States, gu and x * e are the line-by-line kernels' bit for bit; merged outputs within the storage roundings of
both (at most one per direction on either side)."""
import pytest

from gpu_util import any_size_shape

pytestmark = pytest.mark.gpu

# (B, C, H, W, G), dtype, kchunk, logits, launch shape (gpu_util.any_size_shape)
CALLS = [
    # LDS tile, both directions at once, two chunks: one to three chunks in all, requests of 64, 32 and 16 bytes
    ((1, 2, 9, 11, 1), "bf16", 0, False, (0, 2, 32, 1, 1, 1, 1)),
    ((1, 2, 33, 41, 2), "f32", 0, False, (0, 2, 64, 1, 1, 1, 1)),
    ((1, 2, 80, 68, 1), "bf16", 0, False, (0, 2, 64, 1, 2, 1, 1)),
    ((1, 4, 100, 167, 2), "bf16", 0, False, (0, 2, 32, 1, 3, 1, 1)),
    ((1, 2, 225, 20, 2), "f16", 0, True, (0, 2, 16, 1, 2, 1, 3)),
    # ... lines of two and three waves
    ((1, 2, 23, 266, 1), "bf16", 0, False, (0, 2, 64, 1, 2, 3, 1)),
    ((1, 2, 233, 13, 1), "f32", 0, False, (0, 2, 32, 1, 2, 1, 3)),
    ((1, 4, 19, 211, 1), "f32", 30, True, (0, 2, 64, 1, 2, 2, 1)),
    # ... one chunk
    ((1, 4, 112, 103, 2), "f16", 0, True, (0, 1, 32, 1, 2, 1, 1)),
    ((1, 1, 160, 144, 1), "bf16", 24, False, (0, 1, 32, 1, 3, 1, 1)),
    ((1, 2, 29, 300, 2), "f16", 0, True, (0, 1, 64, 1, 2, 3, 1)),
    ((1, 2, 262, 31, 1), "f32", 40, False, (0, 1, 32, 1, 2, 1, 3)),
    # LDS tile, one direction after the other: one chunk, and two
    ((1, 2, 144, 192, 1), "bf16", 8, True, (1, 1, 32, 1, 3, 1, 1)),
    ((1, 2, 176, 192, 1), "f16", 0, False, (1, 1, 16, 1, 3, 1, 1)),
    ((1, 6, 172, 102, 2), "bf16", 0, True, (1, 2, 32, 1, 3, 1, 1)),
    # global memory, two chunks: three and four positions per lane, lines of three waves
    ((1, 2, 160, 144, 1), "f32", 0, False, (2, 2, 64, 1, 3, 1, 1)),
    ((1, 2, 135, 181, 2), "f32", 0, True, (2, 2, 64, 1, 3, 1, 1)),
    ((1, 128, 195, 197, 8), "f32", 0, False, (2, 2, 64, 1, 4, 1, 1)),
    ((1, 130, 230, 212, 2), "bf16", 0, False, (2, 2, 64, 1, 4, 1, 1)),
    ((1, 2, 256, 264, 1), "bf16", 0, False, (2, 2, 32, 1, 2, 3, 3)),
    ((1, 4, 100, 225, 2), "f32", 0, False, (2, 2, 64, 1, 2, 3, 1)),
    # ... one chunk
    ((1, 128, 321, 321, 8), "bf16", 0, False, (2, 1, 64, 1, 2, 3, 3)),
    ((1, 130, 257, 513, 2), "bf16", 0, False, (2, 1, 64, 1, 4, 3, 2)),
    ((1, 128, 301, 299, 8), "f16", 0, False, (2, 1, 64, 1, 2, 3, 3)),
    ((1, 128, 321, 323, 8), "f32", 0, False, (2, 1, 64, 1, 2, 3, 3)),
    ((1, 2, 601, 701, 1), "bf16", 50, False, (2, 1, 32, 1, 4, 3, 3)),
    # two workgroups per CU
    ((3, 96, 85, 34, 8), "bf16", 0, False, (0, 1, 64, 2, 2, 1, 1)),
    ((3, 96, 104, 81, 4), "f32", 0, False, (1, 1, 64, 2, 2, 1, 1)),
    ((3, 96, 64, 150, 8), "f16", 0, True, (1, 1, 64, 2, 3, 1, 1)),
    ((1, 288, 17, 257, 4), "f16", 0, False, (1, 2, 64, 2, 2, 3, 1)),
    ((1, 520, 258, 17, 8), "bf16", 0, False, (1, 2, 16, 2, 2, 1, 3)),
    ((1, 520, 200, 31, 8), "f32", 0, False, (1, 2, 32, 2, 2, 1, 2)),
    # four
    ((5, 128, 27, 27, 8), "bf16", 0, False, (0, 1, 64, 4, 1, 1, 1)),
    ((5, 128, 63, 61, 8), "f32", 16, True, (1, 1, 64, 4, 1, 1, 1)),
    ((1, 520, 131, 25, 8), "bf16", 0, False, (1, 2, 16, 4, 3, 1, 1)),
]


@pytest.mark.parametrize("mask", [15, 9])
@pytest.mark.parametrize("shape,dtype,kchunk,logits,launch", CALLS, ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_against_the_line_by_line_kernels(shape, dtype, kchunk, logits, launch, mask, monkeypatch):
    import torch
    import paper_2512_07884_amd as G
    from paper_2512_07884_amd import binding
    from test_gpu_differential import _rel, _run
    G.binding = binding
    B, C, H, W, Gr = shape
    td = {"bf16": torch.bfloat16, "f32": torch.float32, "f16": torch.float16}[dtype]
    g = torch.Generator(device="cuda"); g.manual_seed(H * 1000 + W)
    z = torch.randn((4, B, Gr, 3, H, W), generator=g, device="cuda")
    if not logits:
        z[:2, :, :, 0, :, 0] = -1e30; z[:2, :, :, 2, :, -1] = -1e30; z[2:, :, :, 0, 0, :] = -1e30; z[2:, :, :, 2, -1, :] = -1e30
        z = torch.softmax(z, dim=3)
    inp = {"x": torch.randn((B, C, H, W), generator=g, device="cuda").to(td), "w": z.to(td),
           "lam": torch.rand((4, B, C, H, W), generator=g, device="cuda").to(td),
           "u": torch.rand((4, B, C, H, W), generator=g, device="cuda").to(td),
           "gy": torch.randn((B, C, H, W), generator=g, device="cuda").to(td)}
    assert any_size_shape(*shape, dtype, "save", kchunk, logits, mask) == any_size_shape(*shape, dtype, "bwd", kchunk, logits, mask) == launch
    fast = _run(G, inp, Gr, mask, kchunk, logits)
    monkeypatch.setenv("GSPN_FORCE_GENERIC", "1")
    ref = _run(G, inp, Gr, mask, kchunk, logits)
    monkeypatch.delenv("GSPN_FORCE_GENERIC", raising=False)
    tol = {"bf16": 2e-2, "f16": 2.5e-3, "f32": 2e-5}[dtype]      # eight storage roundings of a sum in 16 bits, as in test_gpu_ragged
    for n in fast:
        a, b = fast[n].float(), ref[n].float()
        nan = torch.isnan(a)
        assert torch.equal(nan, torch.isnan(b)), (n, "slots of unmasked directions differ")
        if n in ("hs", "gu") or (n == "gl" and dtype != "f16"):
            assert bool(((fast[n] == ref[n]) | nan).all()), (n, int((~((fast[n] == ref[n]) | nan)).sum()))
        e = _rel(torch.where(nan, torch.zeros_like(a), a), torch.where(nan, torch.zeros_like(b), b))
        assert e <= tol, (n, e)
