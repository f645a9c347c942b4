"""The work that a user of the library has it do, as cases that can be timed and compared.

Shapes are those of Code Llama 7B / 13B / 34B (workloads.MODEL_SHAPES) and generic ones drawn over the
same ranges.  Six kinds of work:
  linear       one call of the quantised linear layer, launched from Python (a program that serves
               single requests, or a prompt chunk); smooth: its activations are divided by the
               smoothing factor first, as in front of a layer whose factor cannot be folded away
  layer        the linears of one decoder layer in a decode step (up to 64 rows), captured once in a
               HIP graph and replayed, as a serving loop does: norm + qkv, smoothing + o,
               norm + fused gate/up + down
  mlp          norm + fused gate/up + down on the rows of a prompt, launched from Python
  weights      offline preparation of one layer's weight in checkpoint orientation: transpose,
               smoothing factor, smoothing, quantise + pack
  mlp_weights  offline preparation of a merged gate/up weight: fold down_proj's factor, interleave,
               smoothing factor, smoothing, quantise + pack, fold the factor into the norm
  search       the search for the smoothing strength of one layer on its calibration rows
"""
import math

import torch

import paper_2312_03788_amd as sqp

EPS = 1e-5
ALPHA = 0.5


def listed():
    return [
        # one token through the smallest square layer: launch latency and host work count most
        {"name": "linear_7b_o_m1", "kind": "linear", "M": 1, "K": 4096, "N": 4096, "group": 128, "smooth": False},
        # single-stream decode of the 7B shapes
        {"name": "layer_7b_m1", "kind": "layer", "M": 1, "H": 4096, "QKV": 12288, "I": 11008, "group": 128},
        # the headline decode batch on the 34B shapes (weights stream from HBM)
        {"name": "layer_34b_m16", "kind": "layer", "M": 16, "H": 8192, "QKV": 10240, "I": 22016, "group": 128},
        # a fuller decode batch, ragged
        {"name": "layer_13b_m48", "kind": "layer", "M": 48, "H": 5120, "QKV": 15360, "I": 13824, "group": 128},
        # finer groups at a decode batch between one and two row tiles
        {"name": "layer_7b_m20_g64", "kind": "layer", "M": 20, "H": 4096, "QKV": 12288, "I": 11008, "group": 64},
        # a short prompt (or a prompt chunk) through the 34B output projection
        {"name": "linear_34b_o_m160", "kind": "linear", "M": 160, "K": 8192, "N": 8192, "group": 128, "smooth": True},
        # a prompt of 512 through the 7B MLP block
        {"name": "mlp_7b_m512", "kind": "mlp", "M": 512, "H": 4096, "I": 11008, "group": 128},
        # the prefill size of the headline metric on the merged 34B qkv projection
        {"name": "linear_34b_qkv_m2048", "kind": "linear", "M": 2048, "K": 8192, "N": 10240, "group": 128, "smooth": False},
        # a long ragged prompt through the largest MLP block
        {"name": "mlp_34b_m3001", "kind": "mlp", "M": 3001, "H": 8192, "I": 22016, "group": 128},
        # one-off preparation of the longest 34B weight from a checkpoint
        {"name": "weights_34b_down", "kind": "weights", "K": 22016, "N": 8192, "T": 512, "group": 128},
        # preparation of the merged 13B gate/up weight with finer groups
        {"name": "mlp_weights_13b_g64", "kind": "mlp_weights", "H": 5120, "I": 13824, "T": 512, "group": 64},
        # the paper's grid of 21 smoothing strengths on a 13B layer
        {"name": "search_13b_o", "kind": "search", "T": 512, "K": 5120, "N": 5120, "group": 128, "n_alpha": 21},
    ]


def _log_int(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(max(int(round(v / step)), -(-lo // step)), hi // step) * step


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "layer", "layer", "mlp", "weights", "mlp_weights", "search"])
    group = rng.choice([128, 128, 128, 64, 32, 256])
    kstep = max(group, 64)
    if kind == "linear":
        while True:
            c = {"kind": kind, "M": _log_int(rng, 1, 4096), "K": _log_int(rng, 1024, 22016, kstep),
                 "N": _log_int(rng, 1024, 44032, 8), "group": group, "smooth": rng.random() < 0.5}
            if c["K"] * c["N"] <= 8192 * 44032:
                return c
    if kind == "layer":
        h = _log_int(rng, 2048, 8192, 256)
        return {"kind": kind, "M": _log_int(rng, 1, 64), "H": h, "QKV": h * rng.choice([5, 6, 12]) // 4,
                "I": int(h * rng.uniform(2.6, 2.8)) // 256 * 256, "group": group}
    if kind == "mlp":
        h = _log_int(rng, 2048, 8192, 256)
        return {"kind": kind, "M": _log_int(rng, 65, 3001), "H": h, "I": int(h * rng.uniform(2.6, 2.68)) // 256 * 256, "group": group}
    if kind == "weights":
        return {"kind": kind, "K": _log_int(rng, 1024, 22016, kstep), "N": _log_int(rng, 1024, 8192, 8),
                "T": _log_int(rng, 128, 512), "group": group}
    if kind == "mlp_weights":
        h = _log_int(rng, 2048, 5120, 256)
        return {"kind": kind, "H": h, "I": int(h * rng.uniform(2.6, 2.7)) // 8 * 8, "T": _log_int(rng, 128, 512), "group": group}
    while True:
        c = {"kind": kind, "T": _log_int(rng, 64, 768), "K": _log_int(rng, 1024, 8192, kstep),
             "N": _log_int(rng, 1024, 8192, 8), "group": group, "n_alpha": rng.choice([6, 11, 21])}
        if c["T"] * c["K"] * c["N"] * c["n_alpha"] <= 21 * 512 * 5120 * 5120:
            return c


# ---------------------------------------------------------------- inputs (from the seed alone)

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)


def _activation(g, M, K):
    """N(0, 1) with 1 % of the channels 50 times larger (a fixed set for all tokens)."""
    x = _randn(g, M, K)
    gain = torch.ones(K, device="cuda")
    gain[torch.randperm(K, generator=g, device="cuda")[: max(1, K // 100)]] = 50.0
    return x.mul_(gain).half()


def _smoothed_activation(g, M, K):
    """Activations after smoothing: outliers drawn in, channels of unequal size."""
    return _randn(g, M, K).mul_(torch.exp(0.4 * _randn(g, K))).half()


def _factor(g, K):
    """Smoothing factors as Eq. 6 gives them at 0.5: most around 7, a few channels around 45."""
    s = 7.0 * torch.exp(0.15 * _randn(g, K))
    s[torch.randperm(K, generator=g, device="cuda")[: max(1, K // 100)]] *= 7.0
    return s


def _quantised(g, K, N, group):
    """A smoothed weight N(0, 0.02) * (unequal channels), quantised as Eq. 1 defines it."""
    packed = torch.empty((K // 8, N), dtype=torch.int32, device="cuda")
    scales = torch.empty((K // group, N), dtype=torch.float16, device="cuda")
    zeros = torch.empty((K // group, N), dtype=torch.uint8, device="cuda")
    row = torch.exp(0.4 * _randn(g, K))
    shift = torch.arange(0, 32, 4, device="cuda", dtype=torch.int32).view(1, 8, 1)
    step = max(group, (1 << 26) // N // group * group)
    for k in range(0, K, step):
        n = min(step, K - k)
        w = (_randn(g, n, N) * (0.02 * row[k:k + n, None])).half().float().view(n // group, group, N)
        lo, hi = w.amin(1).clamp_(max=0), w.amax(1).clamp_(min=0)
        d = ((hi - lo) / 15).half().clamp_(min=2.0 ** -24)
        df = d.float()
        z = torch.round(-lo / df).clamp_(0, 15)
        q = torch.round(w / df[:, None]).add_(z[:, None]).clamp_(0, 15).to(torch.int32).view(n // 8, 8, N)
        packed[k // 8:(k + n) // 8] = (q << shift).sum(1, dtype=torch.int32)
        scales[k // group:(k + n) // group] = d
        zeros[k // group:(k + n) // group] = z.to(torch.uint8)
    return packed, scales, zeros


def _inputs(case, seed):
    g = _gen(seed)
    k = case["kind"]
    s = {"kind": k, "group": case.get("group", 128)}
    if k == "linear":
        M, K, N = case["M"], case["K"], case["N"]
        s["w"] = _quantised(g, K, N, s["group"])
        s["s"] = _factor(g, K) if case["smooth"] else None
        s["x"] = _activation(g, M, K) if case["smooth"] else _smoothed_activation(g, M, K)
    elif k in ("layer", "mlp"):
        M, H, I = case["M"], case["H"], case["I"]
        if k == "layer":
            s["x1"], s["gamma1"] = _activation(g, M, H), (1.0 / _factor(g, H)).half()
            s["w_qkv"] = _quantised(g, H, case["QKV"], s["group"])
            s["attn"], s["s_o"] = _smoothed_activation(g, M, H), _factor(g, H)
            s["w_o"] = _quantised(g, H, H, s["group"])
        s["x2"], s["gamma2"] = _activation(g, M, H), (1.0 / _factor(g, H)).half()
        s["w_gu"] = _quantised(g, H, 2 * I, s["group"])
        s["w_down"] = _quantised(g, I, H, s["group"])
    elif k == "weights":
        s["w_nk"] = (_randn(g, case["N"], case["K"]) * 0.02).half()
        s["x_cal"] = _activation(g, case["T"], case["K"])
    elif k == "mlp_weights":
        s["w_gate"] = (_randn(g, case["H"], case["I"]) * 0.02).half()
        s["w_up"] = (_randn(g, case["H"], case["I"]) * 0.02).half()
        s["s_down"] = _factor(g, case["I"])
        s["gamma"] = (1.0 + 0.1 * _randn(g, 1, case["H"])).half()
        s["x_cal"] = _activation(g, case["T"], case["H"])
    else:
        s["w"] = (_randn(g, case["K"], case["N"]) * 0.02).half()
        s["x_cal"] = _activation(g, case["T"], case["K"])
        s["alphas"] = [i / (case["n_alpha"] - 1) for i in range(case["n_alpha"])]
    return s


def _mlp(s):
    h = sqp.w4a16_gemm_silu_mul(sqp.rmsnorm(s["x2"], s["gamma2"], EPS), *s["w_gu"], s["group"])
    return h, sqp.w4a16_gemm(h, *s["w_down"], s["group"])


def _layer(s):
    qkv = sqp.w4a16_gemm(sqp.rmsnorm(s["x1"], s["gamma1"], EPS), *s["w_qkv"], s["group"])
    o = sqp.w4a16_gemm(sqp.smooth_apply_x(s["attn"], s["s_o"]), *s["w_o"], s["group"])
    return (qkv, o) + _mlp(s)


def prepare(case, seed):
    s = _inputs(case, seed)
    if case["kind"] == "layer":
        _layer(s)  # one eager step: the binding's workspace now covers these shapes
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            s["out"] = _layer(s)
    return s


def run(s):
    k = s["kind"]
    if k == "linear":
        x = s["x"] if s["s"] is None else sqp.smooth_apply_x(s["x"], s["s"])
        return sqp.w4a16_gemm(x, *s["w"], s["group"])
    if k == "layer":
        s["graph"].replay()
        return s["out"]
    if k == "mlp":
        return _mlp(s)
    if k == "weights":
        w = sqp.transpose_nk(s["w_nk"])
        f = sqp.smooth_scales(s["x_cal"], w, ALPHA)
        return (f,) + tuple(sqp.quantize_pack(sqp.smooth_apply_w(w, f), s["group"]))
    if k == "mlp_weights":
        w = sqp.interleave_gate_up(s["w_gate"], sqp.scale_columns(s["w_up"], s["s_down"]))
        f = sqp.smooth_scales(s["x_cal"], w, ALPHA)
        return (f, sqp.smooth_apply_x(s["gamma"], f)) + tuple(sqp.quantize_pack(sqp.smooth_apply_w(w, f), s["group"]))
    best, curve = sqp.alpha_search(s["x_cal"], s["w"], s["group"], s["alphas"])
    return best, [v for _, v in curve]


# ---------------------------------------------------------------- what a pass cannot do without

def _q_bytes(K, N, group):
    return K * N * (0.5 + 3.0 / group)  # codes, one fp16 step and one zero-point byte per group


def work(case):
    k, g = case["kind"], case.get("group", 128)
    if k == "linear":
        M, K, N = case["M"], case["K"], case["N"]
        return {"bytes": _q_bytes(K, N, g) + 2 * M * (K + N) + (4 * K if case["smooth"] else 0), "flops": 2 * M * K * N}
    if k in ("layer", "mlp"):
        M, H, I = case["M"], case["H"], case["I"]
        b = _q_bytes(H, 2 * I, g) + _q_bytes(I, H, g) + 2 * M * (H + I + H) + 2 * H
        f = 2 * M * (2 * H * I + I * H)
        if k == "layer":
            b += _q_bytes(H, case["QKV"], g) + _q_bytes(H, H, g) + 2 * M * (3 * H + case["QKV"]) + 6 * H
            f += 2 * M * H * (case["QKV"] + H)
        return {"bytes": b, "flops": f}
    if k == "weights":
        K, N, T = case["K"], case["N"], case["T"]
        return {"bytes": 2 * K * N + 2 * T * K + 4 * K + _q_bytes(K, N, g), "flops": 0}
    if k == "mlp_weights":
        H, I, T = case["H"], case["I"], case["T"]
        return {"bytes": 4 * H * I + 4 * I + 2 * T * H + 8 * H + _q_bytes(H, 2 * I, g), "flops": 0}
    T, K, N, n = case["T"], case["K"], case["N"], case["n_alpha"]
    # the product with the unsmoothed weight once, the quantised one for each strength
    return {"bytes": 2 * K * N + 2 * T * K + 8 * n, "flops": 2.0 * T * K * N * (n + 1)}


def tolerance(case):
    if case["kind"] in ("weights", "mlp_weights"):
        return "exact"  # every value is defined to the bit
    if case["kind"] == "search":
        return {"rel": 1e-5}  # fp32 sums of products, squared and added in fp64
    # fp16 weights' products or exact ones, fp32 sums, fp16 results; measured against 64 bits:
    # 2.1e-4 to 2.8e-4 for one call, up to 5.4e-4 behind a norm and the fused activation
    return {"rel": 1e-3 if case["kind"] == "linear" else 2e-3, "max": 2e-2}


# ---------------------------------------------------------------- 64-bit values

def _dequantised(q, group):
    packed, scales, zeros = q
    K, N = packed.shape[0] * 8, packed.shape[1]
    shift = torch.arange(0, 32, 4, device="cuda", dtype=torch.int32).view(1, 8, 1)
    codes = ((packed.view(K // 8, 1, N) >> shift) & 15).to(torch.int8).view(K // group, group, N)
    return ((codes - zeros.to(torch.int8)[:, None]).double() * scales.double()[:, None]).view(K, N)


def _linear64(x, q, group):
    return x.double() @ _dequantised(q, group)


def _norm64(x, gamma):
    v = x.double()
    return v / torch.sqrt((v * v).mean(1, keepdim=True) + EPS) * gamma.double()


def _factor64(x_cal, w):
    ax = x_cal.double().abs().amax(0).clamp(min=1e-5)
    aw = w.abs().amax(1).double().clamp(min=1e-5)
    return ax, aw


def _quantise64(w, group):
    """(steps as fp16 in 64 bits, dequantised weight) of a smoothed fp16 weight."""
    K, N = w.shape
    v = w.double().view(K // group, group, N)
    lo, hi = v.amin(1).clamp(max=0), v.amax(1).clamp(min=0)
    d = ((hi - lo) / 15).half().double().clamp(min=2.0 ** -24)
    z = torch.round(-lo / d).clamp(0, 15)
    q = (torch.round(v / d[:, None]) + z[:, None]).clamp(0, 15) - z[:, None]
    return (hi - lo) / 15, (q * d[:, None]).half().double().view(K, N)


def exact(case, seed):
    s = _inputs(case, seed)
    k, g = case["kind"], s["group"]
    if k == "linear":
        x = s["x"] if s["s"] is None else (s["x"].float() / s["s"]).half()
        return _linear64(x, s["w"], g)
    if k in ("layer", "mlp"):
        gu = _linear64(_norm64(s["x2"], s["gamma2"]), s["w_gu"], g)
        gate, up = gu[:, 0::2], gu[:, 1::2]
        h = gate / (1 + torch.exp(-gate)) * up
        out = (h, _linear64(h, s["w_down"], g))
        if k == "mlp":
            return out
        x = _norm64(s["x1"], s["gamma1"])
        o = _linear64((s["attn"].float() / s["s_o"]).half(), s["w_o"], g)
        return (_linear64(x, s["w_qkv"], g), o) + out
    if k == "weights":
        w = s["w_nk"].t()
        ax, aw = _factor64(s["x_cal"], w)
        f = torch.sqrt(ax) / torch.sqrt(aw)
        w_s = (w.float() * f.float()[:, None]).half().contiguous()
        return f, None, _quantise64(w_s, g)[0], None
    if k == "mlp_weights":
        up = (s["w_up"].float() / s["s_down"]).half()
        w = torch.stack([s["w_gate"], up], 2).view(case["H"], 2 * case["I"])
        ax, aw = _factor64(s["x_cal"], w)
        f = torch.sqrt(ax) / torch.sqrt(aw)
        w_s = (w.float() * f.float()[:, None]).half()
        return f, s["gamma"].double() / f, None, _quantise64(w_s, g)[0], None
    ax, aw = _factor64(s["x_cal"], s["w"])
    y = s["x_cal"].double() @ s["w"].double()
    curve = []
    for a in s["alphas"]:
        a = float(torch.tensor(a, dtype=torch.float32))
        f = (ax ** a / aw ** (1.0 - a)).float()
        x_hat = (s["x_cal"].float() / f).half().double()
        w_hat = _quantise64((f[:, None] * s["w"].float()).half(), g)[1]
        curve.append(float(((y - x_hat @ w_hat) ** 2).sum()))
    return s["alphas"][curve.index(min(curve))], curve
