"""The work whose speed matters to a user of this package, as cases that a timer can run.

Three kinds of work:
  layer    one forward pass of an MoE layer through `MoELayer`: routed mode (rollout), replay of a routing log
           (the trainer's second evaluation of the same tokens) and ids-only replay
  linear   a dense FP8 linear layer: activations quantised, then the block-scaled product
  weights  the weight-update path: one layer's expert matrices, bf16 -> e4m3 codes + block scales

`listed()` are the named cases, `draw(rng)` gives others from the same ranges.  Weights, buffers and contexts are what
a program keeps between calls and are made by `prepare`; everything that depends on the batch is done in `run`.
"""
from __future__ import annotations

import math

import torch

import paper_2512_07710_amd as moe

DEV = "cuda:0"
BLOCK = 128
# the largest work a drawn case may have: 6*T*k*d*F of the long-context batch, and its expert weights
MAX_FLOPS = 6 * 32768 * 8 * 7168 * 2048
MAX_WEIGHTS = 3 * 256 * 7168 * 2048


def _layer(name, T, d, E, k, F, mode, load="router", outliers=0.0):
    c = {"kind": "layer", "T": T, "d": d, "E": E, "k": k, "F": F, "mode": mode, "load": load, "outliers": outliers}
    return dict(c, name=name) if name else c


def listed():
    return [
        # one sequence being decoded: every call is a handful of weight rows and a chain of launches
        _layer("decode_1", 1, 4096, 64, 6, 1408, "routed"),
        # a small decode batch on the widest layer: most experts idle, the busy ones hold one or two rows
        _layer("decode_16_wide", 16, 7168, 256, 8, 2048, "routed"),
        # the decode workload of the benchmark: every expert busy with a few rows, bound by the weights
        _layer("decode_256", 256, 4096, 64, 6, 1408, "routed"),
        # a short ragged prefill with odd sizes everywhere, replayed from a log
        _layer("prefill_odd_777", 777, 2176, 60, 5, 896, "replay", "uniform"),
        # rollout with a balancing selection bias: about 256 rows for each expert
        _layer("rollout_4096_balanced", 4096, 5120, 128, 8, 1536, "routed", "balanced"),
        # replay of a skewed log: a few hot experts, many cold ones
        _layer("replay_4096_zipf", 4096, 5120, 128, 8, 1536, "replay", "zipf"),
        # ids-only replay of a micro-batch with few, busy experts
        _layer("replay_ids_6000", 6000, 3072, 16, 2, 2048, "replay_ids", "uniform"),
        # long-context batch with activation outliers: the largest work
        _layer("longctx_32768", 32768, 7168, 256, 8, 2048, "routed", "router", 1e-3),
        # a decode batch through a dense projection, and a prefill batch through a larger one
        {"name": "linear_40", "kind": "linear", "rows": 40, "K": 4096, "NOUT": 6144},
        {"name": "linear_8192", "kind": "linear", "rows": 8192, "K": 7168, "NOUT": 8192},
        # one layer's gate matrices on their way from the trainer to the rollout engine
        {"name": "weights_sync", "kind": "weights", "rows": 128 * 1536, "cols": 5120},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        u = rng.random()
        if u < 0.7:
            T = _log_int(rng, 1, 32768)
            E = _log_int(rng, 8, 256)
            k = rng.randint(1, min(8, E))
            d = BLOCK * rng.randint(8, 56)
            F = BLOCK * rng.randint(4, 16)
            if 6 * T * k * d * F > MAX_FLOPS or 3 * E * d * F > MAX_WEIGHTS:
                continue
            mode = rng.choice(["routed", "routed", "replay", "replay_ids"])
            load = rng.choice(["router", "router", "balanced"]) if mode == "routed" else rng.choice(["uniform", "zipf"])
            return _layer("", T, d, E, k, F, mode, load, rng.choice([0.0, 1e-3]))
        if u < 0.9:
            rows, K, NOUT = _log_int(rng, 1, 16384), BLOCK * rng.randint(8, 56), BLOCK * rng.randint(8, 128)
            if 2 * rows * K * NOUT <= MAX_FLOPS // 8:
                return {"kind": "linear", "rows": rows, "K": K, "NOUT": NOUT}
            continue
        return {"kind": "weights", "rows": BLOCK * _log_int(rng, 8, 2048), "cols": BLOCK * rng.randint(8, 56)}


# ---------------------------------------------------------------------------------------------- inputs
def _gen(seed, tag):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + tag * 7919 + 17) & 0x7FFFFFFFFFFFFFFF)
    return g


def _coded_weights(n, rows, cols, g, std):
    """n matrices [rows, cols] ~ N(0, std^2) as e4m3 codes and one scale per 128 x 128 block."""
    q = torch.empty((n, rows, cols), dtype=torch.uint8, device=DEV)
    s = torch.empty((n, rows // BLOCK, cols // BLOCK), dtype=torch.float32, device=DEV)
    step = max(1, (1 << 28) // (rows * cols))
    for i in range(0, n, step):
        m = min(step, n - i)
        w = torch.randn((m, rows // BLOCK, BLOCK, cols // BLOCK, BLOCK), generator=g, device=DEV).mul_(std)
        sc = torch.maximum(w.amax(dim=(2, 4)), -w.amin(dim=(2, 4))).div_(448.0)
        q[i:i + m] = w.div_(sc[:, :, None, :, None]).to(torch.float8_e4m3fn).view(torch.uint8).view(m, rows, cols)
        s[i:i + m] = sc
    return q, s


def _activations(T, d, outliers, g):
    x = torch.randn((T, d), generator=g, device=DEV)
    if outliers:
        u = torch.rand((T, d), generator=g, device=DEV)
        x = torch.where(u < outliers, torch.where(u < outliers / 2, -20.0, 20.0), x)
    return x.to(torch.bfloat16)


def _log_of(T, E, k, load, g):
    """A routing log: k distinct ids per token (uniform, or p_e ~ (e+1)^-1.2), weights on the simplex."""
    e = torch.arange(1, E + 1, device=DEV, dtype=torch.float32)
    logp = -1.2 * torch.log(e) if load == "zipf" else torch.zeros_like(e)
    u = torch.rand((T, E), generator=g, device=DEV).clamp_(1e-20, 1.0 - 1e-7)
    ids = torch.topk(logp - torch.log(-torch.log(u)), k, dim=1).indices.to(torch.int32).contiguous()
    w = -torch.log(torch.rand((T, k), generator=g, device=DEV).clamp_(1e-20, 1.0))
    return ids, (w / w.sum(dim=1, keepdim=True)).contiguous()


def _balancing_bias(x, W_r, k):
    """A selection bias that evens out the experts' loads (the fixed-point rule of a balanced router)."""
    logits = x.float() @ W_r.T
    T, E = logits.shape
    mean = T * k / E
    b = torch.zeros(E, device=DEV)
    for _ in range(100):
        load = torch.zeros(E, device=DEV)
        sel = torch.topk(logits + b, k, dim=1).indices.flatten()
        load.scatter_add_(0, sel, torch.ones_like(sel, dtype=torch.float32))
        b = b + 0.05 * ((mean - load) / mean).clamp_(-4.0, 4.0)
    return b.contiguous()


def prepare(case, seed):
    if case["kind"] == "weights":
        w = torch.randn((case["rows"], case["cols"]), generator=_gen(seed, 1), device=DEV).mul_(case["cols"] ** -0.5)
        q = torch.empty((case["rows"], case["cols"]), dtype=torch.uint8, device=DEV)
        s = torch.empty((case["rows"] // BLOCK, case["cols"] // BLOCK), dtype=torch.float32, device=DEV)
        # a weight-update pass needs a context for its stream only; its shape is not used
        return {"case": case, "ctx": _Context(0, 128, 1, 1, 128), "w": w.to(torch.bfloat16), "q": q, "s": s}
    if case["kind"] == "linear":
        rows, K, NOUT = case["rows"], case["K"], case["NOUT"]
        wq, ws = _coded_weights(1, NOUT, K, _gen(seed, 1), K ** -0.5)
        return {"case": case, "ctx": _Context(rows, K, 1, 1, NOUT), "x": _activations(rows, K, 1e-3, _gen(seed, 2)),
                "wq": wq[0], "ws": ws[0], "xq": torch.empty((rows, K), dtype=torch.uint8, device=DEV),
                "xs": torch.empty((K // BLOCK, rows), dtype=torch.float32, device=DEV),
                "y": torch.empty((rows, NOUT), dtype=torch.float32, device=DEV)}
    T, d, E, k, F = (case[n] for n in ("T", "d", "E", "k", "F"))
    w = {}
    for tag, (q, s, rows, cols) in enumerate((("W1q", "s1", F, d), ("W3q", "s3", F, d), ("W2q", "s2", d, F))):
        w[q], w[s] = _coded_weights(E, rows, cols, _gen(seed, 10 + tag), d ** -0.5)
    st = {"case": case, "w": w, "x": _activations(T, d, case["outliers"], _gen(seed, 2)), "bias": None,
          "W_r": torch.randn((E, d), generator=_gen(seed, 3), device=DEV).mul_(d ** -0.5)}
    if case["mode"] != "routed":
        st["ids"], st["gates"] = _log_of(T, E, k, case["load"], _gen(seed, 4))
    elif case["load"] == "balanced":
        st["bias"] = _balancing_bias(st["x"], st["W_r"], k)
    st["layer"] = moe.MoELayer(T, d, E, k, F, device=DEV)
    return st


class _Context:
    """A bare library context on torch's current stream, given back with its owner."""

    def __init__(self, T, d, E, k, F):
        self.handle = moe.moe_create(T, d, E, k, F)

    def __del__(self):
        moe.moe_destroy(self.handle)


# ---------------------------------------------------------------------------------------------- one pass
def run(st):
    case = st["case"]
    if case["kind"] == "weights":
        moe.moe_quantize_weights_fp8(st["ctx"].handle, st["w"], case["rows"], case["cols"], st["q"], st["s"])
        return {"q": st["q"], "s": st["s"]}
    if case["kind"] == "linear":
        rows, K = case["rows"], case["K"]
        moe.moe_quantize_fp8(st["ctx"].handle, st["x"], rows, K, BLOCK, None, 1, st["xq"], st["xs"])
        moe.moe_linear_fp8(st["ctx"].handle, st["xq"], st["xs"], rows, K, st["wq"], st["ws"], case["NOUT"], st["y"])
        return st["y"]
    layer, x = st["layer"], st["x"]
    if case["mode"] == "routed":
        y = layer.forward_routed(x, st["W_r"], st["bias"], st["w"])
    elif case["mode"] == "replay":
        y = layer.forward_replay(x, st["ids"], st["gates"], st["w"])
    else:
        layer.route_replay_ids(x, st["W_r"], st["ids"])
        layer.quantize_tokens(x)
        layer.expert_ffn_gather(st["w"])
        layer.combine()
        y = layer.y
    return {"y": y, "topk_idx": layer.topk_idx, "topk_w": layer.topk_w, "offsets": layer.offsets}


# ---------------------------------------------------------------------------------------------- what a pass cannot do without
def _experts_met(T, E, k, load):
    """Expected number of experts that at least one token is sent to."""
    if load == "zipf":                        # drawn one after another with p ~ rank^-1.2: k*p bounds the inclusion probability
        p = [(e + 1) ** -1.2 for e in range(E)]
        total = sum(p)
        return sum(1.0 - (1.0 - min(1.0, k * v / total)) ** T for v in p)
    return E * (1.0 - (1.0 - k / E) ** T)


def work(case):
    if case["kind"] == "weights":
        n = case["rows"] * case["cols"]
        return {"bytes": 3.0 * n + 4.0 * n / BLOCK ** 2, "flops": 0.0}
    if case["kind"] == "linear":
        rows, K, NOUT = case["rows"], case["K"], case["NOUT"]
        return {"bytes": 2.0 * rows * K + NOUT * K * (1.0 + 4.0 / BLOCK ** 2) + 4.0 * rows * NOUT, "flops": 2.0 * rows * K * NOUT}
    T, d, E, k, F = (case[n] for n in ("T", "d", "E", "k", "F"))
    routed = case["mode"] != "replay"
    weights = _experts_met(T, E, k, case["load"]) * 3.0 * d * F * (1.0 + 4.0 / BLOCK ** 2)
    return {"bytes": weights + 4.0 * T * d + (4.0 * E * d if routed else 8.0 * T * k) + 8.0 * T * k,
            "flops": 6.0 * T * k * d * F + (2.0 * T * d * E if routed else 0.0)}


def tolerance(case):
    if case["kind"] == "weights":
        return "exact"
    if case["kind"] == "linear":
        # fp32 sums of FP8 matrix products: 1.4e-5 against a 64-bit evaluation (the matrix pipe's own rounding)
        return {"rel": 6e-5, "max": 1e-3}
    # bf16 output of two FP8 products with e4m3 rounding between them: up to 2.1e-3 against a 64-bit evaluation; expert
    # ids may differ where two scores tie within the rounding of an fp32 sum
    return {"rel": 8e-3, "max": 0.3, "differ": 1e-3}
