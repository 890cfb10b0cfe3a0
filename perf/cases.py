"""The work that is measured: what a program that serves or quantises a model with this library has it do.

A case names a path ("kind"), its sizes and its options; `prepare` makes what such a program holds before the call
(quantised and packed weights, smoothing vectors, hidden states with a few outlier channels, router logits, workspaces),
`run` makes the one call.  Sizes are those of the library's own workloads (OPT-125m linear, OPT-6.7B FFN block, one
Mixtral-8x7B layer) and ragged ones around them.  Everything is drawn on the GPU from the seed.
"""
from __future__ import annotations

import math

import torch

import paper_2508_07329_amd as haq

DEV = "cuda"
POPULARITY = (0.3, 0.2, 0.15, 0.1, 0.1, 0.07, 0.05, 0.03)  # of the experts in the offload workload
CALIBRATION_TOKENS = 256
GRID = tuple(i / 10 for i in range(11))  # exponents tried by the smoothing search


def listed():
    mixtral = {"H": 4096, "I": 14336, "E": 8}
    opt = {"K": 4096, "F": 16384, "N": 4096}
    return [
        # one linear layer of the smallest model on a few tokens: two short kernels, so launches and the host side count
        {"name": "linear_opt125m_16", "kind": "linear", "codes": "sym", "T": 16, "K": 768, "N": 3072, "act": "relu"},
        # a prompt of odd length through one wide linear in asymmetric codes (the method's default), one-sided activations
        {"name": "linear_asym_777", "kind": "linear", "codes": "asym", "T": 777, "K": 2064, "N": 8208, "act": "none"},
        # a dense FFN block while decoding for a few users: its weights are read for eight tokens
        {"name": "ffn_decode_8", "kind": "ffn", **opt, "T": 8},
        # the same block on one prompt of odd length: too few rows to fill the chip with large tiles
        {"name": "ffn_prompt_333", "kind": "ffn", **opt, "T": 333},
        # the same block on a full prefill batch: the headline workload
        {"name": "ffn_prefill_2048", "kind": "ffn", **opt, "T": 2048},
        # routed experts while decoding for one user: the latency of a token
        {"name": "moe_decode_1", "kind": "moe", "codes": "sym", **mixtral, "T": 1, "routing": "gate"},
        # decoding for eight users, from a serving loop without a workspace of its own
        {"name": "moe_decode_8", "kind": "moe_static", "codes": "sym", **mixtral, "T": 8, "routing": "gate"},
        # decoding for 64 users in asymmetric codes: every expert is read, each for a handful of rows
        {"name": "moe_asym_decode_64", "kind": "moe", "codes": "asym", **mixtral, "T": 64, "routing": "gate"},
        # a short prompt or a busy decode batch: some tens of rows per expert, between streaming and prefill
        {"name": "moe_batch_300", "kind": "moe", "codes": "sym", **mixtral, "T": 300, "routing": "gate"},
        # prefill with uneven experts
        {"name": "moe_prefill_4096", "kind": "moe", "codes": "sym", **mixtral, "T": 4096, "routing": "zipf"},
        # half of the experts live in pinned host memory and come over on demand
        {"name": "moe_offload_256", "kind": "offload", "codes": "sym", **mixtral, "T": 256, "routing": "popularity"},
        # offline: smoothing search and Hessian-aware quantisation of one large layer on a calibration batch
        {"name": "quantize_layer_fc1", "kind": "quantize", "T": 2048, "K": 4096, "N": 16384, "use_weight": False},
    ]


def _log_int(rng, lo, hi, step=1):
    """A multiple of `step` in [lo, hi], spread over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))
    return max(lo, min(hi, int(v) // step * step))


def draw(rng):
    kind = rng.choice(("linear", "linear", "ffn", "ffn", "moe", "moe", "moe", "moe_static", "offload", "quantize"))
    codes = rng.choice(("sym", "sym", "asym"))
    if kind == "linear":
        return {"kind": kind, "codes": codes, "T": _log_int(rng, 1, 4096), "K": _log_int(rng, 512, 8192, 16),
                "N": _log_int(rng, 512, 16384, 16), "act": rng.choice(("none", "relu"))}
    if kind == "ffn":
        K = _log_int(rng, 768, 4096, 16)
        return {"kind": kind, "T": _log_int(rng, 1, 2048), "K": K, "F": 4 * K, "N": K}
    if kind == "quantize":
        return {"kind": kind, "T": rng.randrange(256, 2049), "K": _log_int(rng, 512, 4096, 64), "N": _log_int(rng, 512, 16384, 16),
                "use_weight": rng.random() < 0.5}
    E = rng.choice((4, 8, 8, 16))
    H = _log_int(rng, 1024, 4096, rng.choice((64, 256)))
    I = _log_int(rng, 2048, 14336, rng.choice((64, 256)))
    while E * H * I > 8 * 4096 * 14336:
        E //= 2
    if kind == "moe_static":
        return {"kind": kind, "codes": "sym", "H": H, "I": I, "E": E, "T": _log_int(rng, 1, 96), "routing": "gate"}
    if kind == "offload":
        return {"kind": kind, "codes": "sym", "H": H, "I": I, "E": 8, "T": _log_int(rng, 1, 512), "routing": "popularity"}
    T = _log_int(rng, 1, 4096)
    return {"kind": kind, "codes": codes, "H": H, "I": I, "E": E, "T": T, "routing": rng.choice(("gate", "zipf"))}


# ---- what a program holds before the call --------------------------------------------------------------------------
def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((seed * 1000003 + stream) & 0x7FFFFFFFFFFF)
    return g


def _outliers(g, K):
    """Channels whose magnitude is 20 to 80 times the others' (0.5 %), as a multiplier per channel."""
    n = max(1, math.ceil(0.005 * K))
    m = torch.ones(K, device=DEV)
    m[torch.randperm(K, generator=g, device=DEV)[:n]] = 20.0 + 60.0 * torch.rand(n, generator=g, device=DEV)
    return m


def _hidden(g, T, mult):
    return (torch.randn(T, mult.numel(), generator=g, device=DEV) * mult).half()


def _weight(g, K, N):
    return torch.randn(K, N, generator=g, device=DEV) * 0.02


def _dense(x, w):
    """(s, codes, scales) of one linear, calibrated on the activations x."""
    s = haq.haq_smoothing_vector(haq.haq_channel_absmax_f16(x), haq.haq_weight_row_absmax(w))
    wq, sw = haq.haq_quant_weight(w, s)
    return s, wq, sw


def _bytes(n):
    return torch.empty(int(n), dtype=torch.uint8, device=DEV)


class _Context:
    """An offload context that goes with its state."""

    def __init__(self, H, I, n_slots):
        self.handle = haq.haq_ctx_create(H, I, n_slots)

    def __del__(self):
        try:
            torch.cuda.synchronize()
            haq.haq_ctx_destroy(self.handle)
        except Exception:  # the interpreter is going away
            pass


def _prepare_linear(c, seed):
    g = _gen(seed, 1)
    T, K, N = c["T"], c["K"], c["N"]
    x = _hidden(g, T, _outliers(g, K))
    if c["codes"] == "asym":
        x = x.clamp_(min=-0.1)  # what an activation function leaves: nearly one-sided
    s, wq, sw = _dense(x, _weight(g, K, N))
    st = {"x": x, "s": s, "w": haq.haq_pack_weight(wq), "sw": sw, "act": haq.HAQ_ACT_RELU if c["act"] == "relu" else haq.HAQ_ACT_NONE}
    if c["codes"] == "asym":
        st["cs"] = haq.haq_weight_colsum(wq)
        st["ws"] = _bytes(haq.haq_linear_asym_workspace_bytes(T, K, N))
    else:
        st["ws"] = _bytes(haq.haq_linear_workspace_bytes(T, K, N))
    return st


def _prepare_ffn(c, seed):
    g = _gen(seed, 2)
    T, K, F, N = c["T"], c["K"], c["F"], c["N"]
    mult = _outliers(g, K)
    cal = _hidden(g, CALIBRATION_TOKENS, mult)
    s1, w1q, sw1 = _dense(cal, _weight(g, K, F))
    w1 = haq.haq_pack_weight(w1q)
    h = haq.haq_w8a8_linear(cal, s1, w1, sw1, F, haq.HAQ_ACT_RELU)
    s2, w2q, sw2 = _dense(h, _weight(g, F, N))
    return {"x": _hidden(g, T, mult), "s1": s1, "w1": w1, "sw1": sw1, "s2": s2, "w2": haq.haq_pack_weight(w2q), "sw2": sw2,
            "ws": _bytes(haq.haq_ffn_workspace_bytes(T, K, F, N))}


def _logits(c, g, x, mult):
    T, H, E = c["T"], c["H"], c["E"]
    if c["routing"] == "popularity":
        p = torch.tensor(POPULARITY, device=DEV)
        u = torch.rand(T, E, generator=g, device=DEV).clamp_(1e-12, 1.0)
        return (p.log()[None, :] - (-u.log()).log()).half()
    gate = (torch.randn(H, E, generator=g, device=DEV) * 0.02 / mult[:, None]).half()
    base = x.float() @ gate.float()
    if c["routing"] == "zipf":  # a bias that makes the experts' shares follow 1 / rank^1.1
        share = 1.0 / torch.arange(1, E + 1, device=DEV, dtype=torch.float32) ** 1.1
        share /= share.sum()
        b = torch.zeros(E, device=DEV)
        for _ in range(30):
            top = (base + b).topk(2, dim=1).indices
            seen = torch.zeros(E, device=DEV).scatter_add_(0, top.flatten(), torch.ones(2 * T, device=DEV)) / (2 * T)
            b += 0.5 * (share / seen.clamp(min=1e-4)).log()
            b -= b.mean()
        base = base + b
    return base.half()


def _prepare_moe(c, seed):
    g = _gen(seed, 3)
    T, H, I, E = c["T"], c["H"], c["I"], c["E"]
    mult = _outliers(g, H)
    cal = _hidden(g, CALIBRATION_TOKENS, mult)
    cal_logits = torch.randn(CALIBRATION_TOKENS, E, generator=g, device=DEV).half()
    full = [(_weight(g, H, I), _weight(g, H, I)) for _ in range(E)]
    aw = torch.zeros(H, device=DEV)
    for pair in full:
        for w in pair:
            haq.haq_weight_row_absmax(w, aw)
    s_in = haq.haq_smoothing_vector(haq.haq_channel_absmax_f16(cal), aw)
    experts, sums = [], []
    plain = torch.ones(I, device=DEV)
    w2f = [_weight(g, I, H) for _ in range(E)]
    blank = torch.zeros(haq.haq_packed_bytes(I, H), dtype=torch.int8, device=DEV)
    sw_blank = torch.ones(H, device=DEV)
    for e in range(E):
        w1q, sw1 = haq.haq_quant_weight(full[e][0], s_in)
        w3q, sw3 = haq.haq_quant_weight(full[e][1], s_in)
        full[e] = None
        experts.append(haq.ExpertWeights(haq.haq_pack_gate_up(w1q, w3q), blank, sw1, sw3, sw_blank, plain))
        if c["codes"] == "asym":
            sums.append((haq.haq_weight_colsum(w1q), haq.haq_weight_colsum(w3q)))
    # the down projections' smoothing vectors from the intermediate that the calibration tokens leave in each expert
    _, dbg = haq.haq_moe_w8a8_ffn(cal, cal_logits, s_in, experts, I, debug=("mid_fp16", "offsets"))
    off = dbg.offsets.tolist()
    for e in range(E):
        s_mid = plain
        if off[e + 1] > off[e]:
            s_mid = haq.haq_smoothing_vector(haq.haq_channel_absmax_f16(dbg.mid_fp16[off[e]:off[e + 1]]), haq.haq_weight_row_absmax(w2f[e]))
        w2q, sw2 = haq.haq_quant_weight(w2f[e], s_mid)
        w2f[e] = None
        experts[e].w2, experts[e].sw2, experts[e].s_mid = haq.haq_pack_weight(w2q), sw2, s_mid
        if c["codes"] == "asym":
            sums[e] = (*sums[e], haq.haq_weight_colsum(w2q))
    x = _hidden(g, T, mult)
    st = {"x": x, "logits": _logits(c, g, x, mult), "s_in": s_in, "experts": experts, "sums": sums, "I": I}
    if c["kind"] == "moe_static":
        st["out"] = torch.empty(T, H, dtype=torch.float16, device=DEV)
    elif c["codes"] == "asym":
        st["ws"] = _bytes(haq.haq_moe_asym_workspace_bytes(T, H, I, E))
    else:
        st["ws"] = _bytes(haq.haq_moe_workspace_bytes(T, H, I, E))
    if c["kind"] == "offload":  # the four least popular experts move to the host; two slots, so each call streams them
        for e in range(4, E):
            for name in ("w13", "w2"):
                w = getattr(experts[e], name)
                setattr(experts[e], name, torch.empty(w.shape, dtype=w.dtype, pin_memory=True).copy_(w))
            experts[e].location = haq.HAQ_LOC_HOST_PINNED
        st["ctx"] = _Context(H, I, 2)
    return st


def _prepare_quantize(c, seed):
    g = _gen(seed, 4)
    T, K, N = c["T"], c["K"], c["N"]
    # calibration activations whose channels are correlated, as hidden states are
    r = max(4, K // 16)
    x = torch.randn(T, r, generator=g, device=DEV) @ torch.randn(r, K, generator=g, device=DEV) / math.sqrt(r)
    x = ((x + 0.3 * torch.randn(T, K, generator=g, device=DEV)) * _outliers(g, K)).half()
    return {"x": x, "w": _weight(g, K, N), "use_weight": c["use_weight"], "ws": _bytes(haq.haq_quantize_layer_workspace_bytes(T, K, N, len(GRID)))}


def prepare(case, seed):
    make = {"linear": _prepare_linear, "ffn": _prepare_ffn, "quantize": _prepare_quantize}.get(case["kind"], _prepare_moe)
    return {**make(case, seed), "case": case}


# ---- the call ------------------------------------------------------------------------------------------------------
def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "linear":
        if c["codes"] == "asym":
            return haq.haq_w8a8_linear_asym(state["x"], state["s"], state["w"], state["sw"], state["cs"], c["N"], state["act"],
                                            workspace=state["ws"])
        return haq.haq_w8a8_linear(state["x"], state["s"], state["w"], state["sw"], c["N"], state["act"], workspace=state["ws"])
    if kind == "ffn":
        return haq.haq_w8a8_ffn(state["x"], state["s1"], state["w1"], state["sw1"], c["F"], haq.HAQ_ACT_RELU, state["s2"], state["w2"],
                                state["sw2"], c["N"], workspace=state["ws"])
    if kind == "quantize":
        s, wq, sw, losses, best = haq.haq_quantize_layer(state["x"], state["w"], GRID, state["use_weight"], workspace=state["ws"])
        return {"s": s, "wq": wq, "w_scale": sw, "losses": losses, "best": best}
    if kind == "moe_static":
        return haq.haq_moe_w8a8_ffn_static(state["x"], state["logits"], state["s_in"], state["experts"], state["I"], out=state["out"])
    if c["codes"] == "asym":
        return haq.haq_moe_w8a8_ffn_asym(state["x"], state["logits"], state["s_in"], state["experts"], state["sums"], state["I"],
                                         workspace=state["ws"])
    ctx = state["ctx"].handle if kind == "offload" else None
    return haq.haq_moe_w8a8_ffn(state["x"], state["logits"], state["s_in"], state["experts"], state["I"], ctx=ctx, workspace=state["ws"])


# ---- what the path cannot do without -------------------------------------------------------------------------------
def work(case):
    c, kind, T = case, case["kind"], case["T"]
    if kind == "linear":
        K, N = c["K"], c["N"]
        return {"bytes": 2 * T * K + K * N + 8 * N + 4 * K + 2 * T * N, "flops": 2 * T * K * N}
    if kind == "ffn":
        K, F, N = c["K"], c["F"], c["N"]
        return {"bytes": 2 * T * K + K * F + F * N + 2 * T * N, "flops": 2 * T * (K * F + F * N)}
    if kind == "quantize":
        K, N, n = c["K"], c["N"], len(GRID)
        # candidates and full-precision product, Hessian (its lower half), factor and its inverse, compensation
        flops = 2 * T * K * N * (n + 1) + T * K * K + 2 * K ** 3 / 3 + K * K * N
        return {"bytes": 2 * T * K + 4 * K * N + K * N, "flops": flops}
    H, I, E = c["H"], c["I"], c["E"]
    active = E * (1.0 - (1.0 - 2.0 / E) ** T)  # experts that evenly spread tokens activate
    return {"bytes": 4 * T * H + active * 3 * H * I, "flops": 2 * T * 2 * 3 * H * I}


def tolerance(case):
    # Every result is defined to the bit: sums of whole numbers, one rounding for each written binary32 operation, and
    # binary64 sums in a stated order.  Two passes, and another launch shape, show no difference.
    return "exact"
