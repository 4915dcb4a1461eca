"""The work whose speed counts: scan and projection calls as a model that uses this library makes them.

``listed()`` holds the fixed cases, ``draw`` one more case from the same ranges, ``prepare`` what a program has in hand
before the call, ``run`` one pass through the public entry points, ``work`` the bytes and operations of a pass and
``tolerance`` how far two correct results may lie apart.

A case is a dict of plain values:
    op       "fwd": one forward scan.  "step": forward scan that saves its states, then the backward scan (a training
             step of the layer).  "proxy_step": a training step of the whole compressive block: project K channels down
             to C, scan, project back up to K, and the gradients of all of it.
    B, C, H, W, G   batch, scanned channels, map, weight groups;  K: channels outside the projections (0 without them)
    dtype    storage type of every tensor: "f32", "bf16" or "f16"
    kchunk   stretch length of GSPN-local, 0 for the global scan
    logits   the weights are given as raw logits and normalised inside the call
"""
import math

import torch

import paper_2512_07884_amd as G

TORCH_TYPE = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
D = 4                                   # scan directions of every call
MAX_WORK_BYTES = 2.6e9                  # no drawn case moves more than the largest listed one
MAX_STEP_PIXELS_DENSE = 17000           # dense prediction trains at this map size at most (100x167)


def _case(name, op, B, C, H, W, G, dtype, kchunk=0, logits=False, K=0):
    c = {"op": op, "B": B, "C": C, "H": H, "W": W, "G": G, "K": K, "dtype": dtype, "kchunk": kchunk, "logits": logits}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # serving one image: the third stage of the classifier, where launches and the host path are the cost
        _case("infer_14x14_one_image", "fwd", 1, 384, 14, 14, 8, "bf16"),
        # batched classification, first stage (56x56, width 96)
        _case("infer_56x56_batch64", "fwd", 64, 96, 56, 56, 8, "bf16"),
        # training the classifier's second stage, one weight map per channel, weights as the network emits them
        _case("train_28x28_logits_f32", "step", 32, 192, 28, 28, 192, "f32", logits=True),
        # one denoising step of a 1024-px latent, two images (the guided and the free half)
        _case("infer_128x128_latent", "fwd", 2, 1024, 128, 128, 16, "bf16"),
        # the same layer in training, half precision
        _case("train_128x128_f16", "step", 2, 1024, 128, 128, 16, "f16"),
        # a small layer on one latent, propagation confined to stretches: few planes, many stretches
        _case("train_128x128_local_f32", "step", 1, 32, 128, 128, 4, "f32", kchunk=32),
        # dense prediction: an 800x1333 picture at stride 8, an odd width, weights as logits
        _case("infer_100x167_dense", "fwd", 2, 256, 100, 167, 8, "bf16", logits=True),
        # ... and training on it at stride 16
        _case("train_50x83_dense_f32", "step", 4, 192, 50, 83, 8, "f32"),
        # one picture through a narrow layer at a quarter of 1024 px: few planes, long lines
        _case("infer_256x256_few_planes", "fwd", 1, 64, 256, 256, 8, "bf16"),
        # high-resolution scan
        _case("infer_512x512", "fwd", 1, 512, 512, 512, 16, "bf16"),
        # 1024-px feature maps in full precision, a batch of narrow ones (the largest listed case)
        _case("infer_1024x1024_f32", "fwd", 16, 8, 1024, 1024, 1, "f32"),
        # the compressive block of a latent layer as a training step: 1152 channels scanned in 144
        _case("train_64x64_proxy_block", "proxy_step", 2, 144, 64, 64, 18, "bf16", logits=True, K=1152),
    ]


def _spread(rng, lo, hi):
    """An integer between lo and hi, spread over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _fit(rng, case, cap):
    """Halves the batch, then whole weight groups, until the case moves no more than `cap` bytes."""
    cpg = case["C"] // case["G"]
    while work(case)["bytes"] > cap and (case["B"] > 1 or case["G"] > 1):
        if case["B"] > 1:
            case["B"] //= 2
        else:
            case["G"] //= 2
            case["C"] = case["G"] * cpg
    return case


def draw(rng):
    kind = rng.choice(["classifier", "classifier", "latent", "latent", "dense", "dense", "dense", "long", "local", "proxy"])
    dtype = rng.choice(["bf16", "bf16", "f16", "f32"])
    op = rng.choice(["fwd", "step"])
    logits = rng.random() < 0.35
    if kind == "classifier":            # a stage of the classifier at any input resolution and batch
        stage = rng.choice([0, 1, 2, 3])
        res = _spread(rng, 128, 384)
        side = max(4, res // (4 << stage))
        C = 96 << stage
        case = _case("", op, _spread(rng, 1, 64), C, side, side, rng.choice([4, 8, 8, C]), dtype, 0, logits)
    elif kind == "latent":              # latents of a 512- to 1344-px picture in the usual aspect ratios: sides in steps of 8
        H, W = 8 * _spread(rng, 8, 21), 8 * _spread(rng, 8, 21)
        cpg = rng.choice([16, 32, 64])
        case = _case("", op, rng.choice([1, 2, 4]), 16 * cpg, H, W, 16, dtype, 0, logits)
    elif kind == "dense":               # feature maps of pictures of any size: odd sides
        H, W = _spread(rng, 20, 170), _spread(rng, 20, 270)
        if op == "step" and H * W > MAX_STEP_PIXELS_DENSE:
            H, W = H // 2, W // 2
        case = _case("", op, rng.choice([1, 2, 4]), 8 * rng.choice([12, 16, 24, 32]), H, W, 8, dtype, 0, logits)
    elif kind == "long":                # high-resolution maps; in training the crops are multiples of 64
        if op == "step" or rng.random() < 0.5:
            H, W = 64 * _spread(rng, 3, 8 if op == "step" else 16), 64 * _spread(rng, 3, 8 if op == "step" else 16)
        else:
            H, W = _spread(rng, 192, 1024), _spread(rng, 192, 1024)
        cpg = rng.choice([8, 16, 32])
        g = rng.choice([1, 4, 16])
        case = _case("", op, 1, g * cpg, H, W, g, dtype, 0, logits)
    elif kind == "local":               # GSPN-local, stretches that divide the map and such that do not
        H, W = 16 * _spread(rng, 3, 16), 16 * _spread(rng, 3, 16)
        case = _case("", op, rng.choice([1, 1, 2]), 4 * rng.choice([8, 16, 64]), H, W, 4, dtype, rng.choice([8, 16, 24, 32, 64]), logits)
    else:                               # the compressive block
        K = rng.choice([96, 192, 384, 768, 1152])
        C = rng.choice([8, 24, 48, 144])
        H, W = _spread(rng, 14, 128), _spread(rng, 14, 128)
        case = _case("", "proxy_step", _spread(rng, 1, 16), C, H, W, max(1, C // 8), rng.choice(["bf16", "bf16", "f16"]), 0, logits, K)
    return _fit(rng, case, MAX_WORK_BYTES)


def prepare(case, seed):
    """Inputs of the layer on the GPU and the buffers its outputs go to, as a program keeps them."""
    B, C, H, W, g, K = case["B"], case["C"], case["H"], case["W"], case["G"], case["K"]
    td = TORCH_TYPE[case["dtype"]]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def normal(*shape, scale=1.0):
        return torch.randn(shape, generator=gen, device="cuda").mul_(scale).to(td)

    s = {"case": case}
    if K:
        s["inp"] = normal(B, K, H, W)
        s["down"] = normal(C, K, scale=K ** -0.5)
        s["up"] = normal(K, C, scale=C ** -0.5)
        s["gout"] = normal(B, K, H, W)
        s["x"] = torch.empty((B, C, H, W), dtype=td, device="cuda")
    else:
        s["x"] = normal(B, C, H, W)
    s["w"] = torch.empty((D, B, g, 3, H, W), dtype=td, device="cuda")
    s["lam"] = torch.empty((D, B, C, H, W), dtype=td, device="cuda")
    s["u"] = torch.empty((D, B, C, H, W), dtype=td, device="cuda")
    for d in range(D):
        z = torch.randn((B, g, 3, H, W), generator=gen, device="cuda")
        if not case["logits"]:          # row-stochastic over the neighbours that exist
            if d < 2:
                z[:, :, 0, :, 0] = float("-inf")
                z[:, :, 2, :, -1] = float("-inf")
            else:
                z[:, :, 0, 0, :] = float("-inf")
                z[:, :, 2, -1, :] = float("-inf")
            z = torch.softmax(z, dim=2)
        s["w"][d] = z.to(td)
        s["lam"][d] = torch.rand((B, C, H, W), generator=gen, device="cuda").to(td)
        s["u"][d] = torch.rand((B, C, H, W), generator=gen, device="cuda").to(td)
    s["y"] = torch.empty_like(s["x"])
    if case["op"] != "fwd":
        if K:
            s["gy"] = torch.empty_like(s["x"])
            s["out"] = torch.empty_like(s["inp"])
            s["ginp"] = torch.empty_like(s["inp"])
            for name in ("gdown", "gup"):
                s[name] = torch.empty((C, K) if name == "gdown" else (K, C), dtype=torch.float32, device="cuda")
            s["part"] = torch.empty(B * C * K, dtype=torch.float32, device="cuda")
        else:
            s["gy"] = normal(B, C, H, W)
        s["hs"] = torch.empty_like(s["lam"])
        s["gx"] = torch.empty_like(s["x"])
        s["gw"] = torch.empty_like(s["w"])
        s["glam"] = torch.empty_like(s["lam"])
        s["gu"] = torch.empty_like(s["lam"])
    return s


def _scan_fwd(s, hs):
    c = s["case"]
    if c["logits"]:
        kw = {"kchunk": c["kchunk"]} if c["kchunk"] else {}
        G.gspn_scan_fwd_logits(s["x"], s["w"], s["lam"], s["u"], s["y"], hs, G=c["G"], **kw)
    elif c["kchunk"]:
        G.gspn_scan_fwd_local(s["x"], s["w"], s["lam"], s["u"], s["y"], hs, kchunk=c["kchunk"], G=c["G"])
    else:
        G.gspn_scan_fwd(s["x"], s["w"], s["lam"], s["u"], s["y"], hs, G=c["G"])


def _scan_bwd(s):
    c = s["case"]
    args = (s["gy"], s["x"], s["w"], s["lam"], s["u"], s["hs"], s["gx"], s["gw"], s["glam"], s["gu"])
    if c["logits"]:
        kw = {"kchunk": c["kchunk"]} if c["kchunk"] else {}
        G.gspn_scan_bwd_logits(*args, G=c["G"], **kw)
    elif c["kchunk"]:
        G.gspn_scan_bwd_local(*args, kchunk=c["kchunk"], G=c["G"])
    else:
        G.gspn_scan_bwd(*args, G=c["G"])


def run(state):
    s = state
    c = s["case"]
    if c["op"] == "fwd":
        _scan_fwd(s, None)
        return {"y": s["y"]}
    if c["op"] == "step":
        _scan_fwd(s, s["hs"])
        _scan_bwd(s)
        return {k: s[k] for k in ("y", "hs", "gx", "gw", "glam", "gu")}
    B, C, K = c["B"], c["C"], c["K"]
    G.gspn_proxy_project(s["inp"], s["down"], s["x"])
    _scan_fwd(s, s["hs"])
    G.gspn_proxy_project(s["y"], s["up"], s["out"])
    G.gspn_proxy_project_bwd(s["gout"], s["y"], s["up"], s["gy"], s["gup"], s["part"].view(B, K, C))
    _scan_bwd(s)
    G.gspn_proxy_project_bwd(s["gx"], s["inp"], s["down"], s["ginp"], s["gdown"], s["part"].view(B, C, K))
    return {k: s[k] for k in ("out", "hs", "ginp", "gdown", "gup", "gw", "glam", "gu")}


def work(case):
    """Of every call its inputs once and its outputs once: the calls of a step lie either side of the loss, so the
    backward call has to read again what the forward call read.  Operations: a multiply-add is two."""
    B, C, H, W, g, K = case["B"], case["C"], case["H"], case["W"], case["G"], case["K"]
    e = 4 if case["dtype"] == "f32" else 2
    n = B * C * H * W                                           # pixels x channels
    w = D * B * g * 3 * H * W
    elems = 2 * n + 2 * D * n + w                               # x, y; lam, u; w
    flops = 9 * D * n                                           # lam*x, three taps, merge
    if case["op"] != "fwd":
        elems += D * n                                          # h saved
        elems += 3 * n + 5 * D * n + 2 * w                      # gy, x, gx; lam, u, h, glam, gu; w, gw
        flops += 18 * D * n                                     # the sweep, gx, glam, gu, the three sums of gw
    total = e * elems
    if K:
        m = B * K * H * W
        total += e * 5 * (m + n)                                # inp, out, gout, inp, ginp; x, y, y, gy, gx
        total += 4 * C * K * e + 2 * C * K * 4                  # both matrices each way, their gradients in fp32
        flops += 6 * 2 * B * H * W * K * C
    return {"bytes": float(total), "flops": float(flops)}


def tolerance(case):
    """Four times the distance from the same pass in 64 bits on the same stored inputs, over all outputs of the listed
    cases and some seventy drawn ones: at most 2.7e-7 in f32, 4.5e-3 in bf16 and 4.1e-4 in f16 (2-norm over 2-norm);
    the largest single differences were 1.2e-5, 0.11 and 4e-3, all in the gradient of logits with one map per channel,
    where the terms of the softmax gradient cancel (f16 was not drawn there: an eighth of bf16's figure)."""
    return {"f32": {"rel": 1e-6, "max": 5e-5}, "bf16": {"rel": 1.8e-2, "max": 0.45},
            "f16": {"rel": 1.8e-3, "max": 0.055}}[case["dtype"]]
