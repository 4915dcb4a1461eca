"""Maps of any size on the kernels that walk them in chunks of lines (the "generic" plan's fast form): forward, forward with
h_save and the backward call against the fp64 oracle, and against the line-by-line kernels over random shapes.  Sizes sit
where the launch shape changes: granules of 8 / 4 elements and their tails, rows narrower than a granule, lines of one wave
(one position per lane up to 64, two up to 128, three up to 192) and of several (two positions per lane from 193, four from
449 up), the longest lines, planes beyond the LDS tile, the last chunk of a scan, the middle of the map where the chunks of
both directions cross, 1024, 512 and 256 threads (from 257 and 513 planes).  Each call is asked which kernel it runs: the plan
name "generic" is also the line-by-line kernels'.  The calls of few planes among them run a workgroup per direction here and the any-size
kernel in test_gpu_whole_planes."""
import ctypes
import os

import numpy as np
import pytest

from gpu_util import kernel_of
from test_gpu_local import check_local
from test_gpu_logits import check_logits

pytestmark = pytest.mark.gpu

SHAPES = [(1, 2, 1, 17, 1), (1, 2, 17, 1, 2), (2, 2, 5, 5, 1), (1, 4, 3, 67, 2), (2, 3, 7, 9, 3), (1, 2, 25, 31, 1),
          (1, 2, 64, 65, 1), (1, 2, 65, 63, 2), (1, 6, 50, 83, 2), (2, 2, 100, 167, 1), (1, 2, 167, 100, 2),
          (1, 1, 30, 193, 1), (1, 1, 193, 30, 1), (1, 1, 385, 21, 1), (1, 1, 20, 391, 1), (1, 1, 450, 12, 1),
          (1, 1, 11, 905, 1), (1, 1, 905, 9, 1), (1, 2, 210, 230, 1), (1, 1, 11, 767, 1), (1, 1, 767, 9, 1), (1, 1, 449, 451, 1),
          (3, 96, 25, 31, 8), (5, 120, 17, 21, 8)]


def threads(shape, dtype, kchunk=0, logits=False, mask=15):
    """Threads per workgroup of the any-size kernel in the forward and the backward call, 0 where another kernel takes it."""
    from paper_2512_07884_amd import binding
    B, C, H, W, Gr = shape
    f = binding.load_library().gspn_any_size_threads
    return tuple(f(B, C, H, W, Gr, kchunk, int(logits), ctypes.c_uint(mask), {"f32": 0, "bf16": 1, "f16": 2}[dtype], b) for b in (0, 1))


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_global_scan(shape, dtype):
    # (fp32 lines beyond 768 positions have no launch shape and run line by line: kept as a test of the hand-over)
    want = 0 if dtype == "f32" and 905 in shape else 1024 if shape[0] * shape[1] <= 256 else 512 if shape[0] * shape[1] <= 512 else 256
    assert threads(shape, dtype) == (want, want)
    check_local(shape + (dtype,), 1 << 14)


@pytest.mark.parametrize("shape,kchunk,mask", [((1, 2, 25, 31, 1), 1, 15), ((1, 4, 50, 83, 2), 3, 15), ((2, 2, 65, 63, 1), 24, 15),
                                               ((1, 2, 100, 167, 2), 8, 5), ((1, 2, 17, 193, 1), 16, 10), ((1, 1, 211, 201, 1), 50, 15)],
                         ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_local_stretches_and_direction_masks(shape, kchunk, mask, dtype):
    assert min(threads(shape, dtype, kchunk, False, mask)) > 0
    check_local(shape + (dtype,), kchunk, mask=mask, poison_starts=dtype != "f16")


@pytest.mark.parametrize("shape,kchunk,mask", [((1, 3, 25, 31, 3), None, 15), ((1, 4, 50, 83, 2), 7, 15), ((1, 2, 100, 167, 1), None, 15),
                                               ((1, 2, 65, 193, 2), 24, 15), ((1, 2, 31, 77, 2), None, 9), ((1, 1, 205, 230, 1), None, 15),
                                               ((1, 2, 21, 501, 1), None, 15), ((1, 2, 501, 21, 2), 24, 15), ((3, 96, 25, 31, 8), None, 15)],
                         ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_weights_as_logits(shape, kchunk, mask, dtype):
    assert min(threads(shape, dtype, kchunk or 0, True, mask)) > 0
    check_logits(shape + (dtype,), kchunk=kchunk, mask=mask, poison=dtype != "f16")


@pytest.mark.parametrize("seed", [31, 32])
def test_against_the_line_by_line_kernels(seed, monkeypatch):
    """Random ragged shapes; both sides hold the state, e and the merged output in fp32 where the plane fits the LDS, so
    they are at most two storage roundings apart (bf16: 2 * 2^-8 of the value; elsewhere one rounding per direction)."""
    import torch
    import paper_2512_07884_amd as G
    from paper_2512_07884_amd import binding
    from test_gpu_differential import _run, _rel
    G.binding = binding
    rng = np.random.default_rng(seed)
    kernels = []
    for it in range(14):
        dtype = ["bf16", "f32", "f16"][int(rng.integers(0, 3))]
        H, W = int(2 ** rng.uniform(1, 8.3)), int(2 ** rng.uniform(1, 8.3)) | 1
        if H * W < 16:
            H = 16
        cpg, Gr, B = int(rng.choice([1, 2, 3, 8])), int(rng.integers(1, 4)), int(rng.integers(1, 3))
        C = cpg * Gr
        mask = int(rng.integers(1, 16)) if rng.random() < 0.3 else 15
        kchunk = int(rng.integers(1, max(H, W))) if rng.random() < 0.35 else 0
        logits = bool(rng.random() < 0.3)
        kernels += [kernel_of((B, C, H, W, Gr), dtype, c, kchunk, logits, mask) for c in ("save", "bwd")]
        td = {"bf16": torch.bfloat16, "f32": torch.float32, "f16": torch.float16}[dtype]
        g = torch.Generator(device="cuda"); g.manual_seed(1000 * seed + it)
        z = torch.randn((4, B, Gr, 3, H, W), generator=g, device="cuda")
        if logits:
            w = z.to(td)
        else:
            z[:2, :, :, 0, :, 0] = -1e30; z[:2, :, :, 2, :, -1] = -1e30; z[2:, :, :, 0, 0, :] = -1e30; z[2:, :, :, 2, -1, :] = -1e30
            w = torch.softmax(z.double(), dim=3).to(td)
        inp = {"x": torch.randn((B, C, H, W), generator=g, device="cuda").to(td), "w": w,
               "lam": torch.rand((4, B, C, H, W), generator=g, device="cuda").to(td),
               "u": torch.rand((4, B, C, H, W), generator=g, device="cuda").to(td),
               "gy": torch.randn((B, C, H, W), generator=g, device="cuda").to(td)}
        monkeypatch.delenv("GSPN_FORCE_GENERIC", raising=False)
        fast = _run(G, inp, Gr, mask, kchunk, logits)
        again = _run(G, inp, Gr, mask, kchunk, logits)
        monkeypatch.setenv("GSPN_FORCE_GENERIC", "1")
        ref = _run(G, inp, Gr, mask, kchunk, logits)
        monkeypatch.delenv("GSPN_FORCE_GENERIC", raising=False)
        tol = {"bf16": 2e-2, "f16": 2.5e-3, "f32": 2e-5}[dtype]
        case = (seed, it, B, C, H, W, Gr, dtype, mask, kchunk, logits)
        for n in fast:
            a, b = fast[n].float(), ref[n].float()
            na, nb = torch.isnan(a), torch.isnan(b)
            assert torch.equal(na, nb), (case, n, "slots of unmasked directions differ")
            e = _rel(torch.where(na, torch.zeros_like(a), a), torch.where(nb, torch.zeros_like(b), b))
            assert e <= tol, (case, n, e)
            assert torch.equal(fast[n].view(torch.uint8), again[n].view(torch.uint8)), (case, n, "not the same twice")
    # most of the calls are to run the kernel under test, or, four directions of so few planes, the one in its place (kept out of
    # test_gpu_whole_planes, which runs this again)
    any_size = sum(k.endswith("any size") for k in kernels)
    assert any_size + sum(k in ("apart", "small") for k in kernels) >= 14, kernels
    assert any_size >= 14 or os.environ.get("GSPN_NO_APART") != "1", kernels


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape,kchunk", [((1, 2, 29, 41, 1), 8), ((1, 2, 100, 167, 2), 24), ((1, 1, 30, 205, 1), 7)],
                         ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_what_is_not_finite_stays_in_its_stretch(shape, kchunk, dtype, monkeypatch):
    """A NaN and an infinity in x and gy: the same elements of every output are finite as on the line-by-line kernels, which
    read nothing across a cut."""
    import torch
    import paper_2512_07884_amd as G
    from paper_2512_07884_amd import binding
    from test_gpu_differential import _run
    G.binding = binding
    B, C, H, W, Gr = shape
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda"); g.manual_seed(5)
    w = torch.softmax(torch.randn((4, B, Gr, 3, H, W), generator=g, device="cuda"), dim=3).to(td)
    inp = {"x": torch.randn((B, C, H, W), generator=g, device="cuda").to(td), "w": w,
           "lam": torch.rand((4, B, C, H, W), generator=g, device="cuda").to(td),
           "u": torch.rand((4, B, C, H, W), generator=g, device="cuda").to(td),
           "gy": torch.randn((B, C, H, W), generator=g, device="cuda").to(td)}
    inp["x"][0, 0, H // 2, W // 2] = float("nan"); inp["x"][0, 0, 0, W - 1] = float("inf")
    inp["gy"][0, C - 1, H - 1, 0] = float("nan"); inp["gy"][0, C - 1, H // 3, W // 3] = float("-inf")
    assert min(threads(shape, dtype, kchunk)) > 0
    fast = _run(G, inp, Gr, 15, kchunk, False)
    monkeypatch.setenv("GSPN_FORCE_GENERIC", "1")
    ref = _run(G, inp, Gr, 15, kchunk, False)
    monkeypatch.delenv("GSPN_FORCE_GENERIC", raising=False)
    for n in fast:
        assert torch.equal(torch.isfinite(fast[n].float()), torch.isfinite(ref[n].float())), n


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("shape,kchunk,mask,logits", [((2, 6, 50, 83, 3), 0, 15, False), ((1, 6, 50, 83, 2), 7, 15, True), ((1, 2, 100, 167, 1), 0, 15, False),
                                                      ((1, 2, 30, 205, 1), 24, 15, False), ((1, 1, 205, 30, 1), 0, 10, True), ((1, 2, 11, 501, 1), 0, 15, False),
                                                      ((1, 1, 501, 13, 1), 50, 15, True), ((5, 120, 25, 31, 8), 0, 15, False), ((9, 128, 21, 17, 16), 0, 15, True)],
                         ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_states_are_those_of_the_line_by_line_kernels(shape, kchunk, mask, logits, dtype, monkeypatch):
    """A scan step adds its terms in the same order on both: h_save, and with it gu, and x * e of the reverse sweep are the
    same numbers.  One, two, three and four positions per lane; lines of one and of several waves; up to 256, 512, 1024 and
    more planes (1024, 512 and 256 threads)."""
    import torch
    import paper_2512_07884_amd as G
    from paper_2512_07884_amd import binding
    from test_gpu_differential import _run
    G.binding = binding
    B, C, H, W, Gr = shape
    td = {"bf16": torch.bfloat16, "f32": torch.float32, "f16": torch.float16}[dtype]
    g = torch.Generator(device="cuda"); g.manual_seed(17)
    z = torch.randn((4, B, Gr, 3, H, W), generator=g, device="cuda")
    inp = {"x": torch.randn((B, C, H, W), generator=g, device="cuda").to(td), "w": (z if logits else torch.softmax(z, dim=3)).to(td),
           "lam": torch.rand((4, B, C, H, W), generator=g, device="cuda").to(td),
           "u": torch.rand((4, B, C, H, W), generator=g, device="cuda").to(td),
           "gy": torch.randn((B, C, H, W), generator=g, device="cuda").to(td)}
    assert min(threads(shape, dtype, kchunk, logits, mask)) > 0
    fast = _run(G, inp, Gr, mask, kchunk, logits)
    monkeypatch.setenv("GSPN_FORCE_GENERIC", "1")
    ref = _run(G, inp, Gr, mask, kchunk, logits)
    monkeypatch.delenv("GSPN_FORCE_GENERIC", raising=False)
    for n in ("hs", "gu", "gl"):
        a, b = fast[n], ref[n]
        same = (a == b) | (torch.isnan(a) & torch.isnan(b))              # (slots of unmasked directions hold NaN)
        if dtype == "f16" and n == "gl":
            # x * e rounded to fp16 at once or by way of fp32, as the compiler chose in either kernel: one spacing at most,
            # 2^-10 of the value (2^-24 in the subnormals), and seldom
            assert float(same.float().mean()) > 0.999
            same |= (a.float() - b.float()).abs() <= torch.clamp(2.0 ** -10 * b.float().abs(), min=2.0 ** -24)
        assert bool(same.all()), (n, int((~same).sum()), a.numel())
