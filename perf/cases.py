"""The workloads this library is measured on: what a program that uses it has it do, call for call.

Six kinds of work, each through the public entry points:

  forward   one MoE layer over a batch of tokens (moe_forward)
  decode    M = 1 decode of a stack of layers for some steps, with the online statistics (moe_decode)
  finetune  one gate-only router fine-tuning step: both routers, regularisers, their gradient, gate gradient
  trace     the statistics of the routing traces of a batched run: overlap, LRU misses, per-step sums, balance
  cache     the cache simulator under all four replacement policies on the same traces
  reroute   cache-aware rerouting of given routing distributions

Shapes are those of workload/configs.py and of the benchmark programs; hidden states are AR(1)
sequences, weights N(0, 0.02), traces the top-k of AR(1) logits with uneven expert popularity.
"""
import math

import torch

import paper_2605_27081_amd as remoe

DEV = "cuda:0"
CAPS = (16, 32, 64)                       # LRU capacities tracked during decode
LAGS = (1, 2, 4, 8, 16)
WINDOW = 64
COEF = (1.0, 0.1, 0.5, 0.5, 0.2)
EXPERT_BYTES = 3 * 2048 * 768 * 2         # what a miss of the trace statistics fetches


def _layer(hidden, experts, inter, top_k, renorm, shared, shared_gate, dtype):
    return {"hidden": hidden, "experts": experts, "inter": inter, "top_k": top_k, "renorm": renorm,
            "shared": shared, "shared_gate": shared_gate, "dtype": dtype}


TINY = _layer(256, 16, 128, 2, False, 0, False, "f32")
DSV2LITE = _layer(2048, 64, 1408, 6, False, 2816, False, "bf16")
QWEN15 = _layer(2048, 60, 1408, 4, False, 5632, True, "bf16")
QWEN3 = _layer(2048, 128, 768, 8, True, 0, False, "bf16")


def listed():
    return [
        # one decode step of 16 concurrent requests: few rows per expert, the weights dominate
        {"name": "forward_batch16", "kind": "forward", "tokens": 16, "rho": 0.0, **QWEN3},
        # one prompt of ordinary, ragged length
        {"name": "forward_prompt333", "kind": "forward", "tokens": 333, "rho": 0.8, **QWEN3},
        # one sequence of about a thousand tokens, large gated shared expert
        {"name": "forward_seq1021", "kind": "forward", "tokens": 1021, "rho": 0.8, **QWEN15},
        # the DeepSeek-V2-Lite-shaped batch: 8 sequences of 2048 tokens, plain shared expert
        {"name": "forward_batch16k", "kind": "forward", "tokens": 16384, "rho": 0.8, **DSV2LITE},
        # the headline prefill batch, 16 sequences of 4096 tokens, one of its 48 layers
        {"name": "forward_prefill64k", "kind": "forward", "tokens": 65536, "rho": 0.8, **QWEN3},
        # the small fp32 layer: reference precision, launches and latency count
        {"name": "forward_f32_tiny", "kind": "forward", "tokens": 128, "rho": 0.8, **TINY},
        # M = 1 decode through the 48-layer stack in a decoder's dependency order, and overlapped
        {"name": "decode_chained", "kind": "decode", "order": "chained", "layers": 48, "steps": 8, "rho": 0.5, **QWEN3},
        {"name": "decode_overlapped", "kind": "decode", "order": "overlapped", "layers": 48, "steps": 8, "rho": 0.5, **QWEN3},
        # one accumulation step of router fine-tuning: 8 sequences of 2048 tokens
        {"name": "finetune_8x2048", "kind": "finetune", "seqs": 8, "steps": 2048, "rho": 0.8, **DSV2LITE},
        # the traces of the headline prefill: 16 sequences x 48 layers
        {"name": "trace_prefill", "kind": "trace", "layers": 48, "seqs": 16, "steps": 4096, "experts": 128, "top_k": 8,
         "capacity": 32, "rho": 0.8},
        # the cache report over decoded prompts: 128 prompts x 64 tokens x 26 layers, cold cache per prompt
        {"name": "cache_policies", "kind": "cache", "layers": 26, "seqs": 128, "steps": 64, "experts": 64, "top_k": 6,
         "capacity": 12, "rho": 0.8},
        # rerouting of 16 sequences of 4096 tokens with a cache smaller than top-k
        {"name": "reroute_16x4096", "kind": "reroute", "seqs": 16, "steps": 4096, "experts": 128, "top_k": 8, "capacity": 4,
         "factor": 1.5, "renorm": False, "rho": 0.8},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["forward"] * 5 + ["decode", "finetune", "trace", "cache", "reroute"])
    rho = rng.choice([0.0, 0.5, 0.8, 0.9])
    if kind == "forward":
        if rng.random() < 0.2:          # fp32 layers: small, any intermediate size
            h = 32 * rng.randint(2, 32)
            n = rng.randint(4, 64)
            layer = _layer(h, n, rng.randint(33, 512), rng.randint(1, min(n, 8)), rng.random() < 0.5,
                           rng.choice([0, 0, 96, 200]), False, "f32")
            return {"kind": kind, "tokens": _log_int(rng, 1, 2048), "rho": rho, **layer}
        layer = dict(rng.choice([DSV2LITE, QWEN15, QWEN3, None]) or
                     _layer(128 * rng.randint(4, 32), rng.randint(8, 128), 64 * rng.randint(4, 24), rng.randint(1, 8),
                            rng.random() < 0.5, rng.choice([0, 0, 704, 2048]), False, "bf16"))
        top = 65536
        while top > 1024 and work({"kind": kind, "tokens": top, "rho": rho, **layer})["flops"] > 4.9e12:
            top //= 2
        return {"kind": kind, "tokens": _log_int(rng, 1, top), "rho": rho, **layer}
    if kind == "decode":
        layer = rng.choice([QWEN3, _layer(1024, 64, 512, 4, False, 0, False, "bf16"), _layer(2048, 96, 640, 6, True, 0, False, "bf16")])
        return {"kind": kind, "order": rng.choice(["chained", "overlapped"]), "layers": rng.randint(3, 24), "steps": rng.randint(1, 16),
                "rho": rho, **layer}
    if kind == "finetune":
        layer = rng.choice([DSV2LITE, QWEN15, QWEN3])
        return {"kind": kind, "seqs": rng.randint(1, 8), "steps": _log_int(rng, 65, 2048), "rho": rho, **layer}
    experts = rng.choice([60, 64, 128, rng.randint(16, 128)])
    top_k = rng.choice([2, 4, 6, 8])
    if kind == "reroute":
        return {"kind": kind, "seqs": rng.randint(1, 64), "steps": _log_int(rng, 16, 4096), "experts": experts, "top_k": top_k,
                "capacity": _log_int(rng, 4, 64), "factor": rng.choice([1.0, 1.5, 4.0]), "renorm": rng.random() < 0.5, "rho": rho}
    layers, seqs = rng.randint(1, 48), rng.randint(1, 16)
    return {"kind": kind, "layers": layers, "seqs": seqs, "steps": _log_int(rng, 16, 4096), "experts": experts, "top_k": top_k,
            "capacity": _log_int(rng, 4, 64), "rho": rho}


# ---- inputs ------------------------------------------------------------------------------------

def _ar1(gen, n_seq, steps, width, rho):
    """Stationary AR(1) sequences [n_seq, steps, width], N(0, 1) at every step, fp32."""
    x = torch.randn(n_seq, steps, width, generator=gen, device=DEV)
    if rho == 0.0:
        return x
    c, block = math.sqrt(1.0 - rho * rho), 64
    i = torch.arange(block, device=DEV, dtype=torch.float32)
    low = torch.tril(c * rho ** (i[:, None] - i[None, :]).clamp(min=0.0))
    decay = (rho ** (i + 1.0))[None, :, None]
    x[:, 0] /= c                                     # the recurrence then starts from x_0 = eps_0
    prev = torch.zeros(n_seq, 1, width, device=DEV)
    for t in range(0, steps, block):
        n = min(block, steps - t)
        part = low[:n, :n].contiguous().expand(n_seq, n, n).contiguous()
        x[:, t:t + n] = torch.bmm(part, x[:, t:t + n].contiguous()) + decay[:, :n] * prev
        prev = x[:, t + n - 1:t + n].clone()
    return x


def _normal(gen, shape, dtype, std=0.02):
    return torch.empty(shape, dtype=dtype, device=DEV).normal_(0.0, std, generator=gen)


def _desc(case):
    return remoe.LayerDesc(case["hidden"], case["experts"], case["inter"], case["top_k"], int(case["renorm"]), case["shared"],
                           int(case["shared_gate"]), remoe.binding.REMOE_F32 if case["dtype"] == "f32" else remoe.binding.REMOE_BF16)


def _traces(gen, case):
    """Routing traces int32 [layers * seqs, steps, top_k]: top-k of sticky logits, some experts more popular."""
    n, s = case["experts"], case["layers"] * case["seqs"]
    idx = torch.empty(s, case["steps"], case["top_k"], dtype=torch.int32, device=DEV)
    group = max(1, (1 << 28) // (case["steps"] * n))
    for a in range(0, s, group):
        m = min(group, s - a)
        z = _ar1(gen, m, case["steps"], n, case["rho"])
        z += 0.7 * torch.randn(m, 1, n, generator=gen, device=DEV)
        idx[a:a + m] = z.topk(case["top_k"], dim=-1).indices.int()
    return idx


def _prepare_forward(case, gen):
    d = _desc(case)
    t, h, n, i, k, si = case["tokens"], d.hidden, d.n_experts, d.inter, d.top_k, d.shared_inter
    dt = d.torch_dtype
    seq = next(q for q in (4096, 2048, 1024, t) if t % q == 0)
    st = {"desc": d, "x": _ar1(gen, t // seq, seq, h, case["rho"]).to(dt).view(t, h),
          "w_router": _normal(gen, (n, h), torch.float32), "w_gate": _normal(gen, (n, i, h), dt),
          "w_up": _normal(gen, (n, i, h), dt), "w_down": _normal(gen, (n, h, i), dt),
          "ws_gate": None, "ws_up": None, "ws_down": None, "ws_scale": None}
    if si:
        st.update(ws_gate=_normal(gen, (si, h), dt), ws_up=_normal(gen, (si, h), dt), ws_down=_normal(gen, (h, si), dt))
        if d.shared_gate:
            st["ws_scale"] = _normal(gen, (h,), torch.float32)
    st.update(y=torch.empty(t, h, dtype=dt, device=DEV), idx=torch.empty(t, k, dtype=torch.int32, device=DEV),
              w=torch.empty(t, k, dtype=torch.float32, device=DEV),
              ws=torch.empty(remoe.remoe_workspace_bytes(d, t), dtype=torch.uint8, device=DEV))
    return st


def _run_forward(st):
    remoe.moe_forward(st["desc"], st["x"], st["w_router"], st["w_gate"], st["w_up"], st["w_down"], st["ws_gate"], st["ws_up"],
                      st["ws_down"], st["ws_scale"], st["y"], st["idx"], st["w"], st["ws"])
    return {"y": st["y"], "idx": st["idx"], "w": st["w"]}


def _prepare_decode(case, gen):
    d = _desc(case)
    h, n, i, k, layers, steps = d.hidden, d.n_experts, d.inter, d.top_k, case["layers"], case["steps"]
    w = [(_normal(gen, (n, h), torch.float32), _normal(gen, (n, i, h), torch.bfloat16), _normal(gen, (n, i, h), torch.bfloat16),
          _normal(gen, (n, h, i), torch.bfloat16)) for _ in range(layers)]
    counts = torch.zeros(layers * (1 + 2 * len(CAPS)), dtype=torch.int64, device=DEV)
    st = {"desc": d, "order": remoe.REMOE_DECODE_CHAINED if case["order"] == "chained" else remoe.REMOE_DECODE_PIPELINED, "weights": w,
          "table": torch.tensor([[m.data_ptr() for m in lw] for lw in w], dtype=torch.int64, device=DEV),
          "x": _ar1(gen, 1, steps, h, case["rho"]).bfloat16().view(steps, h), "counts": counts,
          "lru": torch.zeros(layers, n, dtype=torch.int32, device=DEV),
          "y": torch.empty(steps, layers, h, dtype=torch.bfloat16, device=DEV),
          "idx": torch.empty(layers, steps, k, dtype=torch.int32, device=DEV), "w": torch.empty(layers, steps, k, device=DEV),
          "overlap": torch.empty(layers, steps, dtype=torch.uint8, device=DEV),
          "miss": torch.empty(len(CAPS), layers, steps, dtype=torch.uint8, device=DEV),
          "ws": torch.empty(remoe.remoe_decode_workspace_bytes(d), dtype=torch.uint8, device=DEV)}
    st["sum_overlap"] = counts[:layers]
    st["total_miss"] = counts[layers:layers * (1 + len(CAPS))].view(len(CAPS), layers)
    st["bytes"] = counts[layers * (1 + len(CAPS)):].view(len(CAPS), layers)
    return st


def _run_decode(st):
    st["counts"].zero_()                     # a new request: empty caches, counters at zero
    st["lru"].zero_()
    d = st["desc"]
    remoe.moe_decode(d, st["table"], st["x"], 0, st["x"].shape[0], st["y"], st["idx"], st["w"], CAPS, 3 * d.hidden * d.inter * 2,
                     st["lru"], st["overlap"], st["miss"], st["sum_overlap"], st["total_miss"], st["bytes"], st["ws"],
                     layer_order=st["order"])
    return {k: st[k] for k in ("y", "idx", "w", "lru", "overlap", "miss", "counts")}


def _prepare_finetune(case, gen):
    d = _desc(case)
    s, t, h, n, k = case["seqs"], case["steps"], d.hidden, d.n_experts, d.top_k
    w = _normal(gen, (n, h), torch.float32)
    return {"desc": d, "seqs": s, "x": _ar1(gen, s, t, h, case["rho"]).bfloat16().view(s * t, h), "w": w,
            "w_ref": w + _normal(gen, (n, h), torch.float32, 0.004),
            "idx": torch.empty(s, t, k, dtype=torch.int32, device=DEV), "gate_w": torch.empty(s, t, k, device=DEV),
            "idx_ref": torch.empty(s, t, k, dtype=torch.int32, device=DEV), "gate_w_ref": torch.empty(s, t, k, device=DEV),
            "probs": torch.empty(s, t, n, device=DEV), "probs_ref": torch.empty(s, t, n, device=DEV),
            "values": torch.empty(s, 6, dtype=torch.float64, device=DEV), "dlogits": torch.empty(s, t, n, device=DEV),
            "dw": torch.empty(n, h, device=DEV),
            "ws_loss": torch.empty(remoe.remoe_loss_workspace_bytes(s), dtype=torch.uint8, device=DEV),
            "ws_grad": torch.empty(remoe.remoe_loss_backward_workspace_bytes(s, t, n, WINDOW), dtype=torch.uint8, device=DEV),
            "ws_gate": torch.empty(remoe.remoe_gate_grad_workspace_bytes(s * t, n, h), dtype=torch.uint8, device=DEV)}


def _run_finetune(st):
    d, x = st["desc"], st["x"]
    remoe.moe_route(d, x, st["w"], st["idx"], st["gate_w"], None, st["probs"])
    remoe.moe_route(d, x, st["w_ref"], st["idx_ref"], st["gate_w_ref"], None, st["probs_ref"])
    remoe.remoe_loss_forward(st["probs"], st["probs_ref"], st["idx"], LAGS, WINDOW, st["values"], st["ws_loss"])
    remoe.remoe_loss_backward(st["probs"], st["probs_ref"], st["idx"], LAGS, WINDOW, COEF, st["values"], st["dlogits"], st["ws_grad"])
    remoe.remoe_gate_grad(st["dlogits"].view(x.shape[0], -1), x, st["dw"], st["ws_gate"])
    return {k: st[k] for k in ("values", "dlogits", "dw", "probs", "probs_ref", "idx", "gate_w")}


def _prepare_trace(case, gen):
    n, s, t = case["experts"], case["layers"] * case["seqs"], case["steps"]

    def per_step():
        return torch.empty(s, t, dtype=torch.uint8, device=DEV)

    def per_trace(dtype=torch.int64):
        return torch.empty(s, dtype=dtype, device=DEV)

    return {"case": case, "idx": _traces(gen, case), "overlap": per_step(), "overlap_sum": per_trace(), "miss": per_step(),
            "miss_total": per_trace(), "bytes": per_trace(), "all": torch.empty(case["seqs"], t, dtype=torch.int16, device=DEV),
            "hist": torch.empty(case["layers"] * case["top_k"] + 1, dtype=torch.int64, device=DEV),
            "pct": torch.empty(3, dtype=torch.int32, device=DEV), "load": torch.empty(s, n, dtype=torch.int32, device=DEV),
            "used": per_trace(torch.int32), "entropy": per_trace(torch.float64), "cv": per_trace(torch.float64)}


def _run_trace(st):
    c, idx = st["case"], st["idx"]
    remoe.trace_reuse(idx, c["experts"], st["overlap"], st["overlap_sum"])
    remoe.lru_simulate(idx, c["experts"], c["capacity"], EXPERT_BYTES, 0, None, st["miss"], st["miss_total"], st["bytes"])
    remoe.step_miss_summary(st["miss"].view(c["layers"], c["seqs"], c["steps"]), st["all"], st["hist"], st["pct"])
    remoe.routing_balance(idx, c["experts"], st["load"], st["used"], st["entropy"], st["cv"])
    return {k: st[k] for k in ("overlap", "overlap_sum", "miss", "miss_total", "bytes", "all", "hist", "pct", "load", "used",
                               "entropy", "cv")}


POLICIES = (remoe.REMOE_CACHE_LRU, remoe.REMOE_CACHE_FIFO, remoe.REMOE_CACHE_LFU, remoe.REMOE_CACHE_BELADY)


def _prepare_cache(case, gen):
    s, t = case["layers"] * case["seqs"], case["steps"]
    out = [{"miss": torch.empty(s, t, dtype=torch.uint8, device=DEV), "uniq": torch.empty(s, t, dtype=torch.uint8, device=DEV),
            "hit": torch.empty(s, t, dtype=torch.uint8, device=DEV), "miss_total": torch.empty(s, dtype=torch.int64, device=DEV),
            "uniq_total": torch.empty(s, dtype=torch.int64, device=DEV), "bytes": torch.empty(s, dtype=torch.int64, device=DEV)}
           for _ in POLICIES]
    ws = torch.empty(remoe.remoe_cache_workspace_bytes(s, t, case["top_k"], remoe.REMOE_CACHE_BELADY), dtype=torch.uint8, device=DEV)
    return {"case": case, "idx": _traces(gen, case), "out": out, "ws": ws}


def _run_cache(st):
    c = st["case"]
    for policy, o in zip(POLICIES, st["out"]):
        remoe.cache_simulate(st["idx"], c["experts"], c["capacity"], policy, EXPERT_BYTES, o["miss"], o["uniq"], o["hit"],
                             o["miss_total"], o["uniq_total"], o["bytes"], st["ws"] if policy == remoe.REMOE_CACHE_BELADY else None)
    return st["out"]


def _prepare_reroute(case, gen):
    s, t, k = case["seqs"], case["steps"], case["top_k"]
    z = _ar1(gen, s, t, case["experts"], case["rho"])
    return {"case": case, "probs": torch.softmax(2.0 * z, -1).contiguous(), "idx": torch.empty(s, t, k, dtype=torch.int32, device=DEV),
            "w": torch.empty(s, t, k, device=DEV), "miss": torch.empty(s, t, dtype=torch.uint8, device=DEV),
            "total": torch.empty(s, dtype=torch.int64, device=DEV)}


def _run_reroute(st):
    c = st["case"]
    remoe.reroute_lru(st["probs"], c["top_k"], c["capacity"], c["factor"], c["renorm"], st["idx"], st["w"], st["miss"], st["total"])
    return {k: st[k] for k in ("idx", "w", "miss", "total")}


_PREPARE = {"forward": _prepare_forward, "decode": _prepare_decode, "finetune": _prepare_finetune, "trace": _prepare_trace,
            "cache": _prepare_cache, "reroute": _prepare_reroute}
_RUN = {"forward": _run_forward, "decode": _run_decode, "finetune": _run_finetune, "trace": _run_trace, "cache": _run_cache,
        "reroute": _run_reroute}


def prepare(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(int(seed) & 0x7FFFFFFF)
    return {"kind": case["kind"], "state": _PREPARE[case["kind"]](case, gen)}


def run(state):
    return _RUN[state["kind"]](state["state"])


# ---- what a pass cannot do without -------------------------------------------------------------

def work(case):
    kind = case["kind"]
    if kind in ("forward", "decode", "finetune"):
        h, n, i, k, si = (case[q] for q in ("hidden", "experts", "inter", "top_k", "shared"))
        es = 4 if case["dtype"] == "f32" else 2
    if kind == "forward":
        t = case["tokens"]
        active = n * (1.0 - (1.0 - k / n) ** t)             # experts that expect at least one token
        return {"bytes": active * 3 * h * i * es + 3 * h * si * es + n * h * 4 + 2 * t * h * es + t * k * 8,
                "flops": t * (2.0 * h * n + 6.0 * k * h * i + 6.0 * h * si + (2.0 * h if case["shared_gate"] else 0.0))}
    if kind == "decode":
        per = n * h * 4 + k * 3 * h * i * 2 + 2 * h * 2
        return {"bytes": case["layers"] * case["steps"] * per,
                "flops": case["layers"] * case["steps"] * (2.0 * h * n + 6.0 * k * h * i)}
    if kind == "finetune":
        t = case["seqs"] * case["steps"]
        return {"bytes": t * (h * 2 + 3 * n * 4 + 2 * k * 8) + 3 * n * h * 4, "flops": 6.0 * t * h * n}
    if kind == "reroute":
        st = case["seqs"] * case["steps"]
        return {"bytes": st * (case["experts"] * 4 + case["top_k"] * 8 + 1) + case["seqs"] * 8, "flops": 0}
    s, t, k = case["layers"] * case["seqs"], case["steps"], case["top_k"]
    if kind == "trace":
        return {"bytes": s * t * (4 * k + 2) + 2 * case["seqs"] * t + s * (4 * case["experts"] + 44), "flops": 0}
    return {"bytes": s * t * (4 * k + 3 * len(POLICIES)) + s * 24 * len(POLICIES), "flops": 0}


def tolerance(case):
    """About four times the distance to the same computation in fp64 (7e-7 and 1e-5 at worst for the fp32
    kinds, 2.9e-3 for bf16 layers); `differ` leaves room for neighbouring ranks that swap at equal logits."""
    kind = case["kind"]
    if kind == "cache":
        return "exact"
    if kind == "trace":
        return {"rel": 1e-12, "differ": 0.0}                # whole numbers, and fp64 sums over at most 128 loads
    if kind == "reroute":
        return {"rel": 1e-6, "differ": 0.0}                 # decided in fp32 on the given values; a sum of K weights
    if kind == "finetune" or case["dtype"] == "f32":
        return {"rel": 3e-6, "max": 4e-5, "differ": 1e-3}
    return {"rel": 1e-2, "max": 0.06, "differ": 1e-3}
