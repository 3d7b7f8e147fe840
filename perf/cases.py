"""The work a user of this library has it do, as timed cases.

Each case is one layer or block of a diffusion model as a program runs it: the
activations arrive in bf16, the weights were packed when the model was loaded,
and the workspace was allocated with it.  ``run`` quantizes the activations
and calls the layer through the package's tensor helpers, as such a program
does for every denoising step.  The kinds:

  linear    quantize_act + w4a4_linear, per-group scales
  asym      the same with zero points (quantize_act MODE_ASYMMETRIC + w4a4_linear_asym)
  static    the LDM setting (quantize_act_static + w4a4_linear_static)
  mlp       fc1 (GELU, its epilogue quantizes for fc2) + fc2
  conv      3 x 3 convolution of a UNet: quantized feature map + implicit GEMM
  conv_static   the same in the LDM setting
  attention     lzs_attention of all heads
"""
import math

import torch

import paper_2509_26436_amd as q4

GROUP = 64


# ------------------------------------------------------------------- the cases

def listed():
    def lin(name, kind, M, K, N, gs, gelu=False, bias=True, ws=True):
        return {"name": name, "kind": kind, "M": M, "K": K, "N": N, "gs": gs, "gelu": gelu,
                "bias": bias, "ws": ws}

    def conv(name, kind, images, H, W, C, N, gs):
        return {"name": name, "kind": kind, "images": images, "H": H, "W": W, "C": C, "N": N,
                "gs": gs, "gelu": False, "bias": True, "ws": True}

    def attn(name, heads, L, d, gs):
        return {"name": name, "kind": "attention", "heads": heads, "L": L, "d": d, "gs": gs}

    return [
        # a single 1152-wide linear on 256 tokens: the smallest call, launches and latency
        lin("linear_256", "linear", 256, 1152, 1152, 16),
        # a ragged layer (333 text tokens, N no multiple of a tile), fine subgroups, no workspace
        lin("ragged_333", "linear", 333, 2048, 1000, 8, bias=False, ws=False),
        # PixArt-Sigma 1024 px block, qkv: an ordinary mid-size layer
        lin("pixart_qkv", "linear", 4096, 1152, 3456, 16),
        # FLUX.1-schnell joint block: qkv (many tiles) and fc2 (long reduction)
        lin("flux_qkv", "linear", 4608, 3072, 9216, 16),
        lin("flux_fc2", "linear", 4608, 12288, 3072, 16),
        # four images' FLUX MLP as one chain, fc2's input quantized by fc1: the largest call
        {"name": "flux_mlp_batched", "kind": "mlp", "M": 18432, "K": 3072, "H": 12288, "N": 3072,
         "gs": 16, "bias": True, "ws": True},
        # the zero-point mode on the FLUX attention output projection
        lin("flux_out_asym", "asym", 4608, 3072, 3072, 16),
        # the LDM setting on FLUX fc1, with its GELU
        lin("flux_fc1_static", "static", 4608, 3072, 12288, 16, gelu=True),
        # SDXL UNet 3 x 3 convolutions, both settings
        conv("sdxl_conv_640", "conv", 1, 64, 64, 640, 640, 16),
        conv("sdxl_conv_320_static", "conv_static", 1, 128, 128, 320, 320, 16),
        # FLUX joint attention (32 heads of 128, 4096 image + 512 text tokens), and a
        # smaller attention with 64-wide heads and coarse subgroups
        attn("attention_4608", 32, 4608, 128, 16),
        attn("attention_1024_d64", 20, 1024, 64, 32),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


MOST_MACS = 18432 * 3072 * 12288


def draw(rng):
    kind = rng.choice(["linear"] * 5 + ["mlp", "asym", "static", "static", "conv", "conv_static",
                                        "attention", "attention"])
    gs = rng.choice([8, 16, 16, 16, 32, 64])
    if kind == "attention":
        d = rng.choice([64, 128])
        heads = rng.randint(8, 48)
        L = 64 * _log(rng, 4, 72)
        return {"kind": kind, "heads": heads, "L": L, "d": d, "gs": gs}
    if kind in ("conv", "conv_static"):
        while True:
            images, H, W = rng.randint(1, 2), _log(rng, 15, 128), _log(rng, 15, 128)
            C, N = 64 * _log(rng, 2, 20), 8 * _log(rng, 20, 160)
            if images * H * W * 9 * C * N <= MOST_MACS // 4:
                break
        return {"kind": kind, "images": images, "H": H, "W": W, "C": C, "N": N, "gs": gs,
                "gelu": False, "bias": True, "ws": True}
    if kind == "mlp":
        M = _log(rng, 200, 18432)
        K = 64 * _log(rng, 12, 48)
        return {"kind": kind, "M": M, "K": K, "H": 4 * K, "N": K, "gs": gs, "bias": True, "ws": True}
    while True:
        M = _log(rng, 200, 18432)
        K = 64 * _log(rng, 12, 192)
        N = _log(rng, 320, 12288)
        N = N if rng.random() < 0.25 else -(-N // 64) * 64
        if M * N * K <= MOST_MACS:
            break
    return {"kind": kind, "M": M, "K": K, "N": N, "gs": gs, "gelu": rng.random() < 0.3,
            "bias": rng.random() < 0.8, "ws": rng.random() < 0.8}


# ------------------------------------------------------------------- inputs

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 13)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda")


def _outliers(g, x, share, factor):
    K = x.shape[1]
    cols = torch.randperm(K, generator=g, device="cuda")[:max(1, int(round(share * K)))]
    x[:, cols] *= factor
    return x


def _tokens(g, M, K):
    """Transformer activations: Student-t (3 degrees of freedom) with a few
    outlier channels."""
    x = _randn(g, M, K)
    x /= torch.sqrt((_randn(g, M, K) ** 2 + _randn(g, M, K) ** 2 + _randn(g, M, K) ** 2) / 3)
    return _outliers(g, x.mul_(0.05), 0.002, 100.0).to(torch.bfloat16)


def _features(g, M, C):
    """UNet feature map (NHWC rows): SiLU of a Laplace variable, outlier channels."""
    u = torch.rand(M, C, generator=g, device="cuda") - 0.5
    z = -torch.sign(u) * torch.log1p(-2 * u.abs().clamp(max=0.4999999))
    return _outliers(g, torch.nn.functional.silu(z), 0.005, 30.0).to(torch.bfloat16)


def _weight(g, N, K):
    return (_randn(g, N, K) * 0.02).to(torch.bfloat16)


def _static_scale(x):
    return float(x.abs().max()) / 127.0


def _tensors(case, seed):
    """The bf16 tensors of a case, from the seed alone."""
    g = _gen(seed)
    kind = case["kind"]
    if kind == "attention":
        rows = case["heads"] * case["L"]
        t = {n: _outliers(g, _randn(g, rows, case["d"]), 2 / case["d"], 3.0).to(torch.bfloat16)
             for n in ("q", "k", "v")}
        return t
    if kind in ("conv", "conv_static"):
        x = _features(g, case["images"] * case["H"] * case["W"], case["C"])
        K = 9 * case["C"]
    else:
        x = _tokens(g, case["M"], case["K"])
        K = case["K"]
    if kind == "mlp":
        return {"x": x, "w1": _weight(g, case["H"], K), "b1": _randn(g, case["H"]).mul_(0.02).bfloat16(),
                "w2": _weight(g, case["N"], case["H"]), "b2": _randn(g, case["N"]).mul_(0.02).bfloat16()}
    return {"x": x, "w": _weight(g, case["N"], K),
            "bias": _randn(g, case["N"]).mul_(0.02).bfloat16() if case["bias"] else None}


def _workspace(case, M, N, K):
    return q4.gemm_workspace(M, N, K, "cuda") if case["ws"] else None


def prepare(case, seed):
    """Activations, packed weights and workspaces, as a loaded model holds them."""
    t = _tensors(case, seed)
    kind = case["kind"]
    if kind == "attention":
        return {"case": case, **t,
                "ws": q4.attention_workspace(case["heads"], case["L"], case["d"], case["gs"], "cuda")}
    if kind == "mlp":
        M, K, H, N = case["M"], case["K"], case["H"], case["N"]
        return {"case": case, "x": t["x"], "b1": t["b1"], "b2": t["b2"],
                "w1": q4.pack_weight(t["w1"], with_scales=False),
                "w2": q4.pack_weight(t["w2"], with_scales=False),
                "ws1": _workspace(case, M, H, K), "ws2": _workspace(case, M, N, H)}
    s = {"case": case, "x": t["x"], "bias": t["bias"],
         "epi": q4.EPI_GELU_TANH if case["gelu"] else q4.EPI_NONE}
    M, N, K = t["x"].shape[0], case["N"], t["w"].shape[1]
    s["ws"] = _workspace(case, M, N, K)
    if kind in ("static", "conv_static"):
        s["w"] = q4.pack_weight_per_channel(t["w"], with_scales=False)
        s["scale"] = _static_scale(t["x"])
    else:
        s["w"] = q4.pack_weight(t["w"], with_scales=False)
    if kind == "asym":
        s["sums"] = q4.weight_group_sums(s["w"])
    return s


# ------------------------------------------------------------------- one pass

def _act(a):
    return {"codes": a.codes, "flags": a.flags, "scales": a.scales, "zeros": a.zeros}


def run(s):
    c = s["case"]
    kind, gs = c["kind"], c["gs"]
    if kind == "attention":
        return {"o": q4.lzs_attention(s["q"], s["k"], s["v"], c["heads"], gs, workspace=s["ws"])}
    if kind == "mlp":
        a = q4.quantize_act(s["x"], gs)
        h = q4.w4a4_linear_quantize(a, s["w1"], s["b1"], q4.EPI_GELU_TANH, gs, workspace=s["ws1"])
        y = q4.w4a4_linear(h, s["w2"], s["b2"], workspace=s["ws2"])
        return {"y": y, "a": _act(a), "h": _act(h)}
    if kind in ("static", "conv_static"):
        a = q4.quantize_act_static(s["x"], s["scale"], gs)
    elif kind == "asym":
        a = q4.quantize_act(s["x"], gs, mode=q4.MODE_ASYMMETRIC)
    else:
        a = q4.quantize_act(s["x"], gs)
    w, bias, epi, ws = s["w"], s["bias"], s["epi"], s["ws"]
    if kind == "linear":
        y = q4.w4a4_linear(a, w, bias, epi, workspace=ws)
    elif kind == "asym":
        y = q4.w4a4_linear_asym(a, w, s["sums"], bias, epi, workspace=ws)
    elif kind == "static":
        y = q4.w4a4_linear_static(a, w, s["scale"], bias, epi, workspace=ws)
    elif kind == "conv":
        y = q4.w4a4_conv3x3(a, w, c["images"], c["H"], c["W"], bias, epi, workspace=ws)
    else:
        y = q4.w4a4_conv3x3_static(a, w, s["scale"], c["images"], c["H"], c["W"], bias, epi,
                                   workspace=ws)
    return {"y": y, "a": _act(a)}


# ------------------------------------------------------------------- what a pass needs

def _act_bytes(kind, gs, n):
    """Bytes of the quantized form of n activations."""
    per = 0.5 + 1.0 / gs
    if kind not in ("static", "conv_static"):
        per += 2.0 / GROUP
    if kind == "asym":
        per += 1.0 / GROUP
    return per * n


def work(case):
    kind, gs = case["kind"], case["gs"]
    if kind == "attention":
        h, L, d = case["heads"], case["L"], case["d"]
        return {"bytes": 4 * 2.0 * h * L * d, "flops": 4.0 * h * L * L * d}
    if kind == "mlp":
        M, K, H, N = case["M"], case["K"], case["H"], case["N"]
        return {"bytes": 2.0 * M * K + _act_bytes(kind, gs, M * K) + _act_bytes(kind, gs, M * H)
                + 0.53125 * (K * H + H * N) + 2.0 * (H + N) + 2.0 * M * N,
                "flops": 2.0 * M * H * (K + N)}
    if kind in ("conv", "conv_static"):
        M, C, N = case["images"] * case["H"] * case["W"], case["C"], case["N"]
        K = 9 * C
    else:
        M, C, N = case["M"], case["K"], case["N"]
        K = C
    wsums = 2.0 * N * K / GROUP if kind == "asym" else 0.0
    return {"bytes": 2.0 * M * C + _act_bytes(kind, gs, M * C) + 0.53125 * N * K + wsums
            + 2.0 * N * case["bias"] + 2.0 * M * N,
            "flops": 2.0 * M * N * K}


def tolerance(case):
    """bf16 outputs (one rounding, 2^-9 of a value at most); fp32 sums in
    another order move a few of them to the neighbouring bf16 value.  Codes,
    FLAGs and scales of the input are whole numbers and do not move; the ones
    formed from a layer's own output move where its bf16 value does.
    Attention forms codes from fp32 probabilities, and a code that lands on
    the other side of a rounding boundary moves an output by up to a code step."""
    if case["kind"] == "attention":
        return {"rel": 6e-3, "max": 0.2}
    if case["kind"] == "mlp":
        return {"rel": 7e-3, "max": 0.1, "differ": 2e-3}
    return {"rel": 7e-3, "max": 0.05}


# ------------------------------------------------------------------- the same in 64 bits

def _exact_act(x, gs, mode="sym", scale=None):
    """Dequantized activations s (c 2^FLAG - z) as float64 [M, K], from values
    x (bf16, or fp32 probabilities): the definition, one step per line."""
    M, K = x.shape
    v = x.float().reshape(M, K // GROUP, GROUP)
    z = None
    if mode == "static":
        s = torch.full_like(v[..., :1], scale)
    elif mode == "asym":
        lo, hi = v.amin(-1, keepdim=True).clamp(max=0), v.amax(-1, keepdim=True).clamp(min=0)
        s = ((hi - lo) / 254).half().clamp(max=65504).float()
    else:
        s = (v.abs().amax(-1, keepdim=True) / 127).half().clamp(max=65504).float()
    r = torch.where(s == 0, torch.zeros_like(s), 1 / s)
    q = torch.round(v * r)
    if mode == "asym":
        z = (-127 - torch.round(lo * r)).clamp(-127, 127)
        q = q + z
    q = q.clamp(-127, 127).to(torch.int32).reshape(M, K // gs, gs)
    top = q.abs().amax(-1, keepdim=True)
    flag = sum((top >= t).to(torch.int32) for t in (8, 16, 32, 64))
    d = (torch.sign(q) * ((q.abs() >> flag) << flag)).reshape(M, K // GROUP, GROUP)
    d = d.double() if z is None else d.double() - z.double()
    return (d * s.double()).reshape(M, K)


def _exact_weight(w, per_channel=False):
    N, K = w.shape
    v = w.float().reshape(N, 1, K) if per_channel else w.float().reshape(N, K // GROUP, GROUP)
    s = (v.abs().amax(-1, keepdim=True) / 7).half().clamp(max=65504).float()
    r = torch.where(s == 0, torch.zeros_like(s), 1 / s)
    return (torch.round(v * r).clamp(-7, 7).double() * s.double()).reshape(N, K)


def _exact_layer(a, w, bias, gelu):
    y = torch.cat([t @ w.t() for t in a.split(4096)])
    if bias is not None:
        y += bias.double()
    return torch.nn.functional.gelu(y, approximate="tanh") if gelu else y


def exact(case, seed):
    t = _tensors(case, seed)
    kind, gs = case["kind"], case["gs"]
    none = {"codes": None, "flags": None, "scales": None, "zeros": None}
    if kind == "attention":
        h, L, d = case["heads"], case["L"], case["d"]
        qa, ka = _exact_act(t["q"], gs), _exact_act(t["k"], gs)
        o = torch.empty(L, h * d, dtype=torch.float64, device="cuda")
        for i in range(h):
            rows = slice(i * L, (i + 1) * L)
            p = torch.softmax((qa[rows] @ ka[rows].t()) / math.sqrt(d), dim=-1)
            v = _exact_act(t["v"][rows].t().contiguous(), gs)
            o[:, i * d:(i + 1) * d] = _exact_act(p.float(), gs) @ v.t()
        return {"o": o}
    if kind == "mlp":
        y1 = _exact_layer(_exact_act(t["x"], gs), _exact_weight(t["w1"]), t["b1"], True)
        h = y1.float().bfloat16()
        y1 = None
        y = _exact_layer(_exact_act(h, gs), _exact_weight(t["w2"]), t["b2"], False)
        return {"y": y, "a": none, "h": none}
    static = kind in ("static", "conv_static")
    mode = "static" if static else "asym" if kind == "asym" else "sym"
    a = _exact_act(t["x"], gs, mode, _static_scale(t["x"]) if static else None)
    w = _exact_weight(t["w"], static)
    if kind in ("conv", "conv_static"):
        n, H, W, C = case["images"], case["H"], case["W"], case["C"]
        f = torch.nn.functional.pad(a.reshape(n, H, W, C), (0, 0, 1, 1, 1, 1))
        y = torch.zeros(n * H * W, case["N"], dtype=torch.float64, device="cuda")
        for tap in range(9):
            kh, kw = divmod(tap, 3)
            rows = f[:, kh:kh + H, kw:kw + W].reshape(n * H * W, C)
            y += rows @ w[:, tap * C:(tap + 1) * C].t()
        y = y + t["bias"].double()
        return {"y": y, "a": none}
    return {"y": _exact_layer(a, w, t["bias"], case["gelu"]), "a": none}
