"""Maps whose rows are whole 16-byte chunks, on the plane kernels with two, four and eight channels per wave (lines of up to 32, 16 and
8 lanes, some as long as the lanes of a channel), against the line-by-line kernels: on either side of each line of the choice -- sides, planes
per workgroup, weights of each channel's own, in 16 bits in LDS, maps of up to 4 KB per wave -- with stretches and logits.

y and the states are sums of four products in fp32 in another order than line by line; gw is summed in storage precision there (fp32 alone
compares it)."""
import pytest

from test_gpu_apart import close, inputs
from test_plane_choice import plane_shape

pytestmark = pytest.mark.gpu

# (B, C, H, W, G), dtype, kchunk, logits
CALLS = [
    ((2, 1536, 8, 8, 192), "bf16", 0, False), ((2, 1536, 5, 8, 192), "f16", 3, True), ((4, 1536, 4, 4, 192), "f32", 0, False),
    ((2, 768, 16, 16, 192), "bf16", 0, True), ((2, 768, 9, 16, 192), "f16", 4, False), ((2, 768, 11, 12, 192), "f32", 0, False), ((2, 768, 16, 4, 192), "f32", 5, True),
    ((1, 768, 16, 8, 191 + 1), "f16", 0, False), ((1, 764, 16, 8, 191), "f16", 0, False),
    ((1, 384, 17, 16, 192), "f32", 0, False), ((1, 382, 17, 16, 191), "f32", 0, False), ((1, 384, 22, 20, 192), "f32", 0, True), ((1, 384, 24, 24, 192), "f32", 0, False),
    # 16-bit weights in LDS: one and two channels per wave, one and two pieces of weights per thread, workgroups too small for them (64x64, three
    # channels), lines as long as the lanes of a channel
    ((1, 36, 56, 56, 3), "bf16", 0, False), ((1, 40, 64, 64, 5), "f16", 0, False), ((1, 9, 64, 64, 3), "bf16", 0, False), ((1, 10, 40, 40, 5), "bf16", 0, False),
    ((2, 48, 32, 32, 4), "f16", 0, False), ((1, 24, 19, 24, 2), "bf16", 0, False), ((1, 14, 64, 8, 2), "f16", 0, False), ((1, 12, 2, 64, 2), "bf16", 0, False),
    ((1, 36, 56, 56, 3), "f16", 0, True), ((1, 36, 56, 56, 3), "bf16", 16, False),
    # weights of each channel's own
    ((1, 3072, 12, 12, 3072), "f32", 0, False), ((1, 3072, 12, 16, 3072), "f32", 0, False), ((1, 3072, 16, 16, 3072), "f16", 0, True), ((1, 3068, 16, 16, 3068), "bf16", 0, False),
    ((2, 3072, 7, 8, 3072), "bf16", 2, False), ((1, 6144, 8, 16, 6144), "bf16", 0, False), ((1, 3072, 9, 16, 3072), "bf16", 0, False),
    # ... of one and two channels per wave with up to 4 KB of them, and beyond
    ((1, 510, 28, 28, 510), "f32", 0, True), ((1, 300, 16, 32, 300), "f32", 0, False), ((1, 301, 15, 20, 301), "f32", 6, False), ((1, 300, 32, 32, 300), "f32", 0, False),
    ((1, 300, 33, 32, 300), "f32", 0, False), ((1, 300, 32, 64, 300), "bf16", 0, True), ((1, 300, 33, 64, 300), "f16", 0, False), ((1, 300, 31, 24, 300), "f16", 5, True),
]


# ... and with planes enough that the flat variant fills the chip less often (below, the padded one runs): four and eight channels per wave, lines of
# 17 to 32 positions in fp32, weights of each channel's own
FLAT = [
    ((4, 1536, 8, 8, 192), "bf16", 0, False), ((4, 1536, 5, 8, 192), "f16", 3, True), ((4, 1536, 4, 4, 192), "f32", 0, False), ((8, 1536, 8, 4, 192), "f32", 5, True),
    ((4, 1536, 16, 16, 16), "f16", 0, False), ((4, 1536, 9, 16, 16), "bf16", 4, True), ((4, 1536, 11, 12, 8), "f32", 0, False),
    ((1, 4160, 20, 20, 8), "f32", 0, False), ((1, 4528, 17, 12, 8), "f32", 7, False), ((1, 6144, 20, 12, 8), "f32", 0, True),
    ((1, 24576, 16, 8, 24576), "bf16", 0, False), ((1, 24576, 5, 8, 24576), "f16", 2, True), ((1, 16384, 9, 8, 16384), "f32", 0, False), ((1, 16384, 12, 12, 16384), "f32", 5, False),
]


def run(call, inp, shape, dtype, kchunk, logits, h=None):
    import torch
    import paper_2512_07884_amd as G
    x, w, lam, u = inp["x"], inp["w"], inp["lam"], inp["u"]
    fresh = lambda t: torch.full_like(t, float("nan"))
    kw = {"G": shape[4], **({"kchunk": kchunk} if kchunk else {})}
    kind = "_logits" if logits else "_local" if kchunk else ""
    if call == "bwd":
        o = {"gx": fresh(x), "gw": fresh(w), "glam": fresh(lam), "gu": fresh(lam)}
        getattr(G, "gspn_scan_bwd" + kind)(inp["gy"], x, w, lam, u, h, *o.values(), **kw)
        if dtype != "f32":
            del o["gw"]
    else:
        o = {"y": fresh(x), **({"h": fresh(lam)} if call == "save" else {})}
        getattr(G, "gspn_scan_fwd" + kind)(x, w, lam, u, o["y"], o.get("h"), **kw)
    torch.cuda.synchronize()
    return o


@pytest.mark.parametrize("shape,dtype,kchunk,logits", CALLS, ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_against_line_by_line(shape, dtype, kchunk, logits, monkeypatch):
    from paper_2512_07884_amd import binding
    inp = inputs(shape, dtype, logits)
    monkeypatch.setenv("GSPN_FORCE_GENERIC", "1"); binding.gspn_reload_env()
    ref = run("save", inp, shape, dtype, kchunk, logits)
    ref_bwd = run("bwd", inp, shape, dtype, kchunk, logits, ref["h"])
    monkeypatch.delenv("GSPN_FORCE_GENERIC")
    for knob in ("GSPN_NO_APART", "GSPN_NO_ANY_SIZE", "GSPN_BWD_NO_PLANE"):          # the plane kernels, whatever else would take the call
        monkeypatch.setenv(knob, "1")
    binding.gspn_reload_env()
    code = {"f32": 0, "bf16": 1, "f16": 2}[dtype]
    big = dtype != "f32" and shape[2] * shape[3] * 2 > 6656          # forward calls without h_save: the tile kernel's
    for call, want in (("fwd", "tile" if big else "plane"), ("save", "plane"), ("bwd", "twopass/plane")):
        assert binding.running_kernel(*shape, code, call, kchunk, logits) == want, call
        got = run(call, inp, shape, dtype, kchunk, logits, ref["h"])
        close(got, ref if call != "bwd" else ref_bwd, dtype, ())


@pytest.mark.parametrize("shape,dtype,kchunk,logits", FLAT, ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_flat_variant_against_line_by_line(shape, dtype, kchunk, logits, monkeypatch):
    assert plane_shape(*shape, dtype, kchunk, logits)[0] == 1
    test_against_line_by_line(shape, dtype, kchunk, logits, monkeypatch)
