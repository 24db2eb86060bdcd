"""The work that a program built on this library has it do, as cases that can be timed.

An RL step with FP8 rollouts (arXiv 2601.18150) re-quantises the weights, calibrates and fills the FP8 KV cache,
runs prefill and decode forwards through the W8A8 linears (dense and per MoE expert) and the decode attention, and
weighs the sampled tokens by truncated importance sampling.  Each kind below is one of these steps, called through
the Python entry points as such a program calls them; the dense shapes are Qwen3-8B's, the expert shapes
Qwen3-30B-A3B's, tokens and sequences from the smallest calls to the largest the paper's settings reach.

``listed()`` / ``draw(rng)`` give cases, ``prepare`` makes what the program holds before the call, ``run`` is one
pass, ``work`` its unavoidable bytes and operations, ``exact`` the same outputs from plain torch in 64 bits.
"""
import math

import torch

import paper_2601_18150_amd as fp8rl

HIDDEN, INTER, QKV = 4096, 12288, 6144                 # Qwen3-8B
LINEARS = {"qkv": (4096, 6144), "o_proj": (4096, 4096), "gate_up": (4096, 24576), "down": (12288, 4096)}   # (K, N)
MOE_HIDDEN, MOE_INTER, EXPERTS, TOPK, EMPTY = 2048, 768, 128, 8, 8                                         # Qwen3-30B-A3B
DIM, PAGE = 128, 16


def listed():
    return [
        # the smallest call: a tiny linear layer, all launch and host latency
        {"name": "linear_tiny", "kind": "linear", "m": 64, "k": 512, "n": 512, "scales": "fp32", "requant": False},
        # the largest: prefill of 8192 tokens through gate_up right after a weight sync
        {"name": "linear_prefill", "kind": "linear", "m": 8192, "k": 4096, "n": 24576, "scales": "fp32", "requant": True},
        # one decoder layer's linears for a handful of running sequences, captured as serving loops do at small batch
        {"name": "layer_decode_8", "kind": "layer", "m": 8, "graph": True},
        # the same for a full decode batch
        {"name": "layer_decode_256", "kind": "layer", "m": 256, "graph": False},
        # a ragged chunk of prefill tokens mixed with decode tokens through the gated MLP
        {"name": "mlp_chunk", "kind": "mlp", "m": 777},
        # the expert block over a prefill chunk, Zipf routing, some experts empty
        {"name": "moe_prefill", "kind": "moe", "tokens": 4096, "scales": "fp32"},
        # the expert block over a decode batch: a few rows per expert
        {"name": "moe_decode", "kind": "moe", "tokens": 96, "scales": "fp32"},
        # decode attention at the paper's long responses: the cache fills most of the traffic
        {"name": "attn_long", "kind": "attn", "batch": 64, "kv_heads": 8, "q_heads": 32, "min_len": 4096, "max_len": 20480,
         "cache": "fp8"},
        # decode attention early in a rollout: few, short, ragged sequences
        {"name": "attn_short", "kind": "attn", "batch": 20, "kv_heads": 4, "q_heads": 32, "min_len": 37, "max_len": 1500,
         "cache": "fp8"},
        # KV scales calibrated on, and the cache filled from, one layer's keys and values of a few prompts
        {"name": "kv_prefill", "kind": "kv_prefill", "sequences": 6, "kv_heads": 8, "max_len": 3001},
        # the weight sync: every linear of two layers re-quantised in one call
        {"name": "resync", "kind": "resync", "layers": 2},
        # importance weights and mismatch KL of a whole rollout batch (32 prompts x 16 samples x 20480 tokens)
        {"name": "tis", "kind": "tis", "rows": 512, "max_len": 20480},
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["linear", "linear", "layer", "mlp", "moe", "moe", "attn", "attn", "kv_prefill", "resync", "tis"])
    if kind == "linear":
        scales = rng.choice(["fp32", "fp32", "ue8m0"])
        if rng.random() < 0.3:
            k, n = 128 * rng.randint(1, 40), 128 * rng.randint(1, 40)
        else:
            k, n = LINEARS[rng.choice(sorted(LINEARS))]
        return {"kind": kind, "m": _logint(rng, 1, 8192), "k": k, "n": n, "scales": scales, "requant": rng.random() < 0.3}
    if kind == "layer":
        m = _logint(rng, 1, 512)
        return {"kind": kind, "m": m, "graph": m <= 64}
    if kind == "mlp":
        return {"kind": kind, "m": _logint(rng, 16, 4096)}
    if kind == "moe":
        return {"kind": kind, "tokens": _logint(rng, 1, 6000), "scales": rng.choice(["fp32", "fp32", "fp32", "ue8m0"])}
    if kind == "attn":
        kv_heads = rng.choice([4, 8])
        max_len = _logint(rng, 64, 20480)
        cache = rng.choice(["fp8", "fp8", "fp8", "bf16"])
        batch = min(_logint(rng, 1, 256), max(1, 900_000 // max_len // (2 if cache == "bf16" else 1)))
        return {"kind": kind, "batch": batch, "kv_heads": kv_heads, "q_heads": 32,
                "min_len": rng.randint(1, max_len), "max_len": max_len, "cache": cache}
    if kind == "kv_prefill":
        max_len = _logint(rng, 100, 20000)
        return {"kind": kind, "sequences": rng.randint(1, max(1, 40_000 // max_len)), "kv_heads": rng.choice([4, 8]),
                "max_len": max_len}
    if kind == "resync":
        return {"kind": kind, "layers": rng.randint(1, 4)}
    return {"kind": kind, "rows": rng.randint(8, 512), "max_len": _logint(rng, 300, 20480)}


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _gen(seed, salt, device="cuda"):
    g = torch.Generator(device=device)
    g.manual_seed(int(seed) * 1009 + salt)
    return g


def _normal(shape, std, g):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).mul_(std).to(torch.bfloat16)


def _activations(m, k, g):
    """N(0, 1) with one percent of the channels 50 times larger, as transformer activations have them."""
    x = torch.randn((m, k), generator=g, device="cuda", dtype=torch.float32)
    cols = torch.randint(0, k, (max(1, k // 100),), generator=g, device="cuda")
    x[:, cols] *= 50.0
    return x.to(torch.bfloat16)


def _weight(n, k, g):
    """N(0, 0.02) with one weight in a thousand 20 times larger."""
    w = torch.randn((n, k), generator=g, device="cuda", dtype=torch.float32).mul_(0.02)
    w = torch.where(torch.rand((n, k), generator=g, device="cuda") < 0.001, w * 20.0, w)
    return w.to(torch.bfloat16)


def _codes(x, scale):
    """E4M3 codes of fl32(x / scale), the division in 64 bits (its double rounding is that of fp32 division)."""
    q = (x.double() / scale.double()).float().clamp_(-448.0, 448.0)
    return q.to(torch.float8_e4m3fn)


def _scale_of(amax, scales):
    if scales == "ue8m0":
        _, e = torch.frexp(amax.double() / 448.0)                 # amax / 448 = f * 2^e, f in [0.5, 1)
        e = torch.where(amax.double() == 448.0 * torch.exp2((e - 1).double()), e - 1, e)
        s = torch.exp2(e.double().clamp_(min=-127)).float()
    else:
        s = (amax.double() / 448.0).float()
    return torch.where(amax == 0, torch.ones_like(s), s)


def _quant_act(x, scales="fp32"):
    m, k = x.shape
    g = x.view(m, k // 128, 128)
    s = _scale_of(g.abs().amax(2).float(), scales)                                   # [m][k/128]
    return _codes(g, s[:, :, None]).view(m, k).view(torch.uint8), s.t().contiguous()


def _quant_weight(w, scales="fp32"):
    n, k = w.shape
    q = torch.empty((n, k), dtype=torch.uint8, device=w.device)
    s = torch.empty((n // 128, k // 128), dtype=torch.float32, device=w.device)
    for r in range(0, n, 4096):                                                       # bounds the fp64 temporaries
        b = w[r:r + 4096].view(-1, 128, k // 128, 128)
        sb = _scale_of(b.abs().amax((1, 3)).float(), scales)
        s[r // 128:r // 128 + sb.shape[0]] = sb
        q[r:r + 4096] = _codes(b, sb[:, None, :, None]).reshape(-1, k).view(torch.uint8)
    return q, s


def _values(q):
    return q.view(torch.float8_e4m3fn).double()


def _act_values(q, s):
    m, k = q.shape
    return (_values(q).view(m, k // 128, 128) * s[:, :m].t().double()[:, :, None]).view(m, k)


def _weight_values(q, s):
    n, k = q.shape
    return (_values(q).view(n // 128, 128, k // 128, 128) * s.double()[:, None, :, None]).view(n, k)


def _product(qa, sa, qw, sw):
    a, out = _act_values(qa, sa), []
    for r in range(0, qw.shape[0], 8192):
        out.append(a @ _weight_values(qw[r:r + 8192], sw[r // 128:r // 128 + 64]).t())
    return torch.cat(out, 1)


def _silu_mul(gu):
    inter = gu.shape[1] // 2
    g, u = gu[:, :inter].double(), gu[:, inter:].double()
    return (g / (1.0 + torch.exp(-g)) * u).to(torch.bfloat16)


def _routing(tokens, g):
    """Rows grouped by expert: Zipf(1.1) popularity, the last few experts never chosen, eight experts a token."""
    weight = torch.arange(1, EXPERTS + 1, dtype=torch.float64, device="cuda").pow(-1.1)
    weight[-EMPTY:] = 0.0
    perm = torch.randperm(EXPERTS, generator=g, device="cuda")
    logw = torch.empty(EXPERTS, dtype=torch.float64, device="cuda")
    logw[perm] = weight.log()
    u = torch.rand((tokens, EXPERTS), generator=g, device="cuda", dtype=torch.float64).clamp_(1e-300, 1.0 - 1e-12)
    expert = torch.topk(logw - torch.log(-torch.log(u)), TOPK, dim=1).indices.reshape(-1)
    token = torch.arange(tokens, device="cuda").repeat_interleave(TOPK)
    order = torch.argsort(expert * tokens + token)
    offsets = torch.zeros(EXPERTS + 1, dtype=torch.int32, device="cuda")
    offsets[1:] = torch.cumsum(torch.bincount(expert, minlength=EXPERTS), 0).to(torch.int32)
    return token[order].to(torch.int32).contiguous(), offsets


def _prepare_linear(case, seed):
    g = _gen(seed, 1)
    x, w = _activations(case["m"], case["k"], g), _weight(case["n"], case["k"], g)
    if case["requant"]:
        return {"x": x, "w": w, "qw": torch.empty(w.shape, dtype=torch.uint8, device="cuda"),
                "sw": torch.empty((case["n"] // 128, case["k"] // 128), dtype=torch.float32, device="cuda")}
    qw, sw = _quant_weight(w, case["scales"])
    return {"x": x, "qw": qw, "sw": sw}


def _prepare_layer(case, seed):
    g, m = _gen(seed, 2), case["m"]
    s = {"x": _activations(m, HIDDEN, g), "attn": _normal((m, HIDDEN), 1.0, g), "x2": _activations(m, HIDDEN, g)}
    for name, (k, n) in LINEARS.items():
        s["q_" + name], s["s_" + name] = _quant_weight(_weight(n, k, g))
    # the buffers that a decode loop keeps from step to step
    for name in ("x", "attn", "x2"):
        s["qa_" + name] = torch.empty((m, HIDDEN), dtype=torch.uint8, device="cuda")
        s["sa_" + name] = torch.empty((HIDDEN // 128, m), dtype=torch.float32, device="cuda")
    s["qh"] = torch.empty((m, INTER), dtype=torch.uint8, device="cuda")
    s["sh"] = torch.empty((INTER // 128, m), dtype=torch.float32, device="cuda")
    for name in LINEARS:
        s["y_" + name] = torch.empty((m, LINEARS[name][1]), dtype=torch.bfloat16, device="cuda")
    return s


def _prepare_mlp(case, seed):
    g = _gen(seed, 3)
    s = {"x": _activations(case["m"], HIDDEN, g)}
    s["q_gate_up"], s["s_gate_up"] = _quant_weight(_weight(2 * INTER, HIDDEN, g))
    s["q_down"], s["s_down"] = _quant_weight(_weight(HIDDEN, INTER, g))
    return s


def _expert_weights(n, k, scales, g):
    q, s = _quant_weight(_weight(EXPERTS * n, k, g), scales)
    return q.view(EXPERTS, n, k), s.view(EXPERTS, n // 128, k // 128)


def _prepare_moe(case, seed):
    g = _gen(seed, 4)
    s = {"x": _activations(case["tokens"], MOE_HIDDEN, g)}
    s["rows"], s["offsets"] = _routing(case["tokens"], g)
    s["q_gate_up"], s["s_gate_up"] = _expert_weights(2 * MOE_INTER, MOE_HIDDEN, case["scales"], g)
    s["q_down"], s["s_down"] = _expert_weights(MOE_HIDDEN, MOE_INTER, "fp32", g)
    return s


def _pages(lengths, max_len, g):
    """A block table over a paged cache with room for max_len tokens a sequence: physical blocks in random order, as
    after many allocations."""
    need = [(n + PAGE - 1) // PAGE for n in lengths]
    width = (max_len + PAGE - 1) // PAGE
    blocks = len(lengths) * width
    perm = torch.randperm(blocks, generator=g, device="cuda").to(torch.int32)
    table = torch.zeros((len(lengths), width), dtype=torch.int32, device="cuda")
    at = 0
    for b, n in enumerate(need):
        table[b, :n] = perm[at:at + n]
        at += n
    return table, blocks


def _lengths(count, lo, hi, seed):
    g = _gen(seed, 7, "cpu")
    return torch.randint(lo, hi + 1, (count,), generator=g).tolist()


def _prepare_attn(case, seed):
    g, kvh = _gen(seed, 5), case["kv_heads"]
    lengths = _lengths(case["batch"], case["min_len"], case["max_len"], seed)
    table, blocks = _pages(lengths, case["max_len"], g)
    dtype = torch.float8_e4m3fn if case["cache"] == "fp8" else torch.bfloat16
    s = {"q": _normal((case["batch"], case["q_heads"], DIM), 1.0, g), "table": table, "max_len": case["max_len"],
         "lengths": torch.tensor(lengths, dtype=torch.int32, device="cuda"), "sm_scale": 1.0 / math.sqrt(DIM)}
    # cached values N(0, 1): codes of x / scale at the calibrated scale of their largest value
    spread = 448.0 / 5.7 if case["cache"] == "fp8" else 1.0
    for name, shape in (("k_cache", (blocks, kvh, PAGE, DIM)), ("v_cache", (blocks, kvh, PAGE // 4, DIM, 4))):
        x = torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16).mul_(spread).clamp_(-448.0, 448.0)
        s[name] = x.to(dtype) if dtype == torch.bfloat16 else x.to(dtype).view(torch.uint8)
    if case["cache"] == "fp8":
        s["k_scale"], s["v_scale"] = (torch.full((1,), 1.0 / spread, dtype=torch.float32, device="cuda") for _ in range(2))
        # this step's new token of every sequence, and the slot that its page has for it
        s["k_new"], s["v_new"] = (_normal((case["batch"], kvh, DIM), 1.0, g) for _ in range(2))
        last = torch.tensor([n - 1 for n in lengths], device="cuda")
        s["slots"] = table.gather(1, (last // PAGE)[:, None])[:, 0].long() * PAGE + last % PAGE
    s["workspace"] = torch.empty(max(16, fp8rl.fp8rl_attention_decode_workspace_size(
        case["batch"], case["q_heads"], kvh, case["max_len"])), dtype=torch.uint8, device="cuda")
    return s


def _prepare_kv(case, seed):
    g, kvh = _gen(seed, 6), case["kv_heads"]
    lengths = _lengths(case["sequences"], max(1, case["max_len"] // 2), case["max_len"], seed)
    table, blocks = _pages(lengths, case["max_len"], g)
    slots = []
    for b, n in enumerate(lengths):
        t = torch.arange(n, device="cuda")
        slots.append(table[b].long()[t // PAGE] * PAGE + t % PAGE)
    tokens = sum(lengths)
    return {"k": _normal((tokens, kvh, DIM), 1.3, g), "v": _normal((tokens, kvh, DIM), 0.7, g), "slots": torch.cat(slots),
            "k_cache": torch.zeros((blocks, kvh, PAGE, DIM), dtype=torch.uint8, device="cuda"),
            "v_cache": torch.zeros((blocks, kvh, PAGE // 4, DIM, 4), dtype=torch.uint8, device="cuda")}


def _prepare_resync(case, seed):
    g, ws = _gen(seed, 8), []
    for _ in range(case["layers"]):
        for name in LINEARS:
            k, n = LINEARS[name]
            w = _normal((n, k), 0.02, g)
            w[:128, :128] = 0.0                          # a pruned block
            ws.append(w)
    return {"ws": ws, "qs": [torch.empty(w.shape, dtype=torch.uint8, device="cuda") for w in ws],
            "ss": [torch.empty((w.shape[0] // 128, w.shape[1] // 128), dtype=torch.float32, device="cuda") for w in ws]}


def _prepare_tis(case, seed):
    """Confident tokens (-Exp(0.4)), a small policy mismatch, a percent of tokens far off; responses of many lengths."""
    g, rows, width = _gen(seed, 9), case["rows"], case["max_len"]
    lengths = torch.exp(torch.empty(rows, device="cuda").uniform_(math.log(min(256, width)), math.log(width), generator=g))
    mask = (torch.arange(width, device="cuda")[None, :] < lengths.round()[:, None]).to(torch.uint8).reshape(-1)
    n = rows * width
    lr = -torch.empty(n, device="cuda").exponential_(1.0 / 0.4, generator=g)
    d = torch.randn(n, generator=g, device="cuda") * 0.05
    d = torch.where(torch.rand(n, generator=g, device="cuda") < 0.01, torch.randn(n, generator=g, device="cuda"), d)
    return {"train": (lr + d).clamp_(max=0.0), "rollout": lr, "mask": mask,
            "workspace": torch.empty(max(8, fp8rl.fp8rl_tis_workspace_size(n)), dtype=torch.uint8, device="cuda")}


def prepare(case, seed):
    kind = case["kind"]
    s = {"linear": _prepare_linear, "layer": _prepare_layer, "mlp": _prepare_mlp, "moe": _prepare_moe,
         "attn": _prepare_attn, "kv_prefill": _prepare_kv, "resync": _prepare_resync, "tis": _prepare_tis}[kind](case, seed)
    s["case"] = case
    if case.get("graph"):
        # a serving loop captures its decode step once per batch size and replays it
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _layer(s)
        torch.cuda.current_stream().wait_stream(side)
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            s["outputs"] = _layer(s)
    return s


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
def _linear(s):
    case = s["case"]
    pow2 = case["scales"] == "ue8m0"
    if case["requant"]:
        quant = fp8rl.fp8rl_quant_weight_block128_ue8m0 if pow2 else fp8rl.fp8rl_quant_weight_block128
        quant(s["w"], s["qw"], s["sw"])
    if pow2:
        qa, sa = fp8rl.fp8rl_quant_act_token_group128_ue8m0(s["x"])
        y = fp8rl.fp8rl_gemm_w8a8_block_ue8m0(qa, sa, s["qw"], s["sw"])
    else:
        y = fp8rl.linear_w8a8(s["x"], s["qw"], s["sw"])
    return {"y": y, "qw": s["qw"], "sw": s["sw"]} if case["requant"] else {"y": y}


def _layer(s):
    def linear(name, x):
        fp8rl.fp8rl_quant_act_token_group128(s[x], s["qa_" + x], s["sa_" + x])
        return fp8rl.fp8rl_gemm_w8a8_block_noalloc(s["qa_" + x], s["sa_" + x], s["q_" + name], s["s_" + name], s["y_" + name])

    out = {"qkv": linear("qkv", "x"), "o_proj": linear("o_proj", "attn"), "gate_up": linear("gate_up", "x2")}
    fp8rl.fp8rl_silu_mul_quant_group128(out["gate_up"], s["qh"], s["sh"])
    out["down"] = fp8rl.fp8rl_gemm_w8a8_block_noalloc(s["qh"], s["sh"], s["q_down"], s["s_down"], s["y_down"])
    return out


def _mlp(s):
    qa, sa = fp8rl.fp8rl_quant_act_token_group128(s["x"])
    gu = fp8rl.fp8rl_gemm_w8a8_block(qa, sa, s["q_gate_up"], s["s_gate_up"])
    qh, sh, _ = fp8rl.fp8rl_silu_mul_quant_group128(gu)
    return {"gate_up": gu, "down": fp8rl.fp8rl_gemm_w8a8_block(qh, sh, s["q_down"], s["s_down"])}


def _moe(s):
    if s["case"]["scales"] == "ue8m0":
        qa, sa = fp8rl.fp8rl_quant_act_token_group128_ue8m0(s["x"])
        qg, sg = fp8rl.fp8rl_gather_rows_fp8(qa, sa, s["rows"])
        gu = fp8rl.fp8rl_grouped_gemm_w8a8_block_ue8m0(qg, sg, s["q_gate_up"], s["s_gate_up"], s["offsets"])
    else:
        qa, sa = fp8rl.fp8rl_quant_act_token_group128(s["x"])
        gu = fp8rl.fp8rl_grouped_gemm_w8a8_block_gathered(qa, sa, s["rows"], s["q_gate_up"], s["s_gate_up"], s["offsets"])
    qh, sh, _ = fp8rl.fp8rl_silu_mul_quant_group128(gu)
    return {"gate_up": gu, "down": fp8rl.fp8rl_grouped_gemm_w8a8_block(qh, sh, s["q_down"], s["s_down"], s["offsets"])}


def _attn(s):
    if s["case"]["cache"] == "bf16":
        return {"out": fp8rl.fp8rl_attention_decode_bf16kv(s["q"], s["k_cache"], s["v_cache"], s["table"], s["lengths"],
                                                           s["max_len"], s["sm_scale"], workspace=s["workspace"])}
    fp8rl.fp8rl_kv_cache_write_fp8(s["k_new"], s["v_new"], s["slots"], s["k_scale"], s["v_scale"], s["k_cache"], s["v_cache"])
    out = fp8rl.fp8rl_attention_decode_fp8kv(s["q"], s["k_cache"], s["v_cache"], s["table"], s["lengths"], s["max_len"],
                                             s["k_scale"], s["v_scale"], s["sm_scale"], workspace=s["workspace"])
    return {"out": out, "k_cache": s["k_cache"], "v_cache": s["v_cache"]}


def _kv(s):
    ks, vs = fp8rl.fp8rl_kv_calibrate_scale(s["k"]), fp8rl.fp8rl_kv_calibrate_scale(s["v"])
    fp8rl.fp8rl_kv_cache_write_fp8(s["k"], s["v"], s["slots"], ks, vs, s["k_cache"], s["v_cache"])
    return {"k_scale": ks, "v_scale": vs, "k_cache": s["k_cache"], "v_cache": s["v_cache"]}


def _resync(s):
    return [x for pair in fp8rl.fp8rl_quant_weight_block128_batched(s["ws"], s["qs"], s["ss"]) for x in pair]


def _tis(s):
    w, stats = fp8rl.fp8rl_tis_weights_kl(s["train"], s["rollout"], s["mask"], 2.0, workspace=s["workspace"])
    return {"w": w, "stats": stats}


def run(state):
    if "graph" in state:
        state["graph"].replay()
        return state["outputs"]
    return {"linear": _linear, "layer": _layer, "mlp": _mlp, "moe": _moe, "attn": _attn, "kv_prefill": _kv,
            "resync": _resync, "tis": _tis}[state["case"]["kind"]](state)


# --------------------------------------------------------------------------
# unavoidable work, tolerances, 64-bit outputs
# --------------------------------------------------------------------------
def _w(n, k):
    return n * k + 4 * (n // 128) * (k // 128)


def work(case):
    kind = case["kind"]
    if kind == "linear":
        m, k, n = case["m"], case["k"], case["n"]
        weight = 2 * n * k + _w(n, k) if case["requant"] else _w(n, k)
        return {"bytes": weight + 2 * m * k + 2 * m * n, "flops": 2 * m * n * k}
    if kind in ("layer", "mlp"):
        m, names = case["m"], sorted(LINEARS) if kind == "layer" else ["gate_up", "down"]
        inputs = 3 if kind == "layer" else 1
        return {"bytes": 2 * m * HIDDEN * inputs + sum(_w(n, k) + 2 * m * n for k, n in (LINEARS[x] for x in names)),
                "flops": sum(2 * m * k * n for k, n in (LINEARS[x] for x in names))}
    if kind == "moe":
        rows = case["tokens"] * TOPK
        share = [(e + 1) ** -1.1 for e in range(EXPERTS - EMPTY)]
        total = sum(share)
        # experts that at least one token is expected to choose
        active = sum(1.0 - (1.0 - min(1.0, TOPK * p / total)) ** case["tokens"] for p in share)
        per = _w(2 * MOE_INTER, MOE_HIDDEN) + _w(MOE_HIDDEN, MOE_INTER)
        return {"bytes": active * per + 2 * case["tokens"] * MOE_HIDDEN + 4 * rows + 2 * rows * (2 * MOE_INTER + MOE_HIDDEN),
                "flops": 2 * rows * (2 * MOE_INTER * MOE_HIDDEN + MOE_HIDDEN * MOE_INTER)}
    if kind == "attn":
        tokens = case["batch"] * (case["min_len"] + case["max_len"]) / 2
        size = 1 if case["cache"] == "fp8" else 2
        return {"bytes": tokens * case["kv_heads"] * 2 * DIM * size + 4 * case["batch"] * case["q_heads"] * DIM,
                "flops": 4 * tokens * case["q_heads"] * DIM}
    if kind == "kv_prefill":
        tokens = case["sequences"] * 0.75 * case["max_len"]
        return {"bytes": tokens * case["kv_heads"] * DIM * (2 * 2 + 2) + 8 * tokens, "flops": 0}
    if kind == "resync":
        return {"bytes": case["layers"] * sum(2 * n * k + _w(n, k) for k, n in LINEARS.values()), "flops": 0}
    return {"bytes": case["rows"] * case["max_len"] * 13, "flops": 0}


def tolerance(case):
    kind = case["kind"]
    if kind in ("kv_prefill", "resync"):
        return "exact"                       # codes and scales are bit for bit
    if kind == "tis":
        return {"rel": 2e-7, "max": 1e-6}    # one rounding to fp32; the sums are fp64
    if kind in ("linear", "attn"):
        return {"rel": 7e-3, "max": 3e-2}    # one rounding to bf16 of fp32 sums: 1.7e-3 from the 64-bit result
    # the second product's input codes flip where the first one's rounding does: 3.3e-3 from the 64-bit result
    return {"rel": 1.2e-2, "max": 6e-2}


def _exact_mlp(qa, sa, s):
    gu = _product(qa, sa, s["q_gate_up"], s["s_gate_up"])
    qh, sh = _quant_act(_silu_mul(gu.to(torch.bfloat16)))
    return gu, _product(qh, sh, s["q_down"], s["s_down"])


def _exact_moe(case, s):
    qa, sa = _quant_act(s["x"], case["scales"])
    rows, off = s["rows"].long(), s["offsets"].tolist()
    gu = torch.empty((rows.numel(), 2 * MOE_INTER), dtype=torch.float64, device="cuda")
    y = torch.empty((rows.numel(), MOE_HIDDEN), dtype=torch.float64, device="cuda")
    for e in range(EXPERTS):
        r = slice(off[e], off[e + 1])
        if off[e] == off[e + 1]:
            continue
        t = rows[r]
        sub = {n: s[n][e] for n in ("q_gate_up", "s_gate_up", "q_down", "s_down")}
        gu[r], y[r] = _exact_mlp(qa[t], sa[:, t].contiguous(), sub)
    return {"gate_up": gu, "down": y}


def _exact_attn(case, s):
    kvh, group = case["kv_heads"], case["q_heads"] // case["kv_heads"]
    fp8 = case["cache"] == "fp8"
    k_cache, v_cache = s["k_cache"], s["v_cache"]
    if fp8:                                                          # the new tokens land in the cache first
        blk, off = s["slots"] // PAGE, s["slots"] % PAGE
        k_cache[blk, :, off] = _codes(s["k_new"], s["k_scale"]).view(torch.uint8)
        v_cache[blk, :, off // 4, :, off % 4] = _codes(s["v_new"], s["v_scale"]).view(torch.uint8)
    value = (lambda c, sc: _values(c) * sc.double()) if fp8 else (lambda c, sc: c.double())
    out = torch.empty((case["batch"], case["q_heads"], DIM), dtype=torch.float64, device="cuda")
    for b, n in enumerate(s["lengths"].tolist()):
        blocks = s["table"][b, :(n + PAGE - 1) // PAGE].long()
        k = value(k_cache[blocks], s.get("k_scale")).permute(1, 0, 2, 3).reshape(kvh, -1, DIM)[:, :n]
        v = value(v_cache[blocks], s.get("v_scale")).permute(1, 0, 2, 4, 3).reshape(kvh, -1, DIM)[:, :n]
        q = s["q"][b].double().view(kvh, group, DIM)
        p = torch.softmax(torch.matmul(q, k.transpose(1, 2).contiguous()) * s["sm_scale"], dim=2)
        out[b] = torch.matmul(p, v.contiguous()).reshape(case["q_heads"], DIM)
    return {"out": out, "k_cache": None, "v_cache": None} if fp8 else {"out": out}


def exact(case, seed):
    kind = case["kind"]
    s = prepare({k: v for k, v in case.items() if k != "graph"}, seed)
    if kind == "linear":
        qw, sw = _quant_weight(s["w"], case["scales"]) if case["requant"] else (s["qw"], s["sw"])
        qa, sa = _quant_act(s["x"], case["scales"])
        y = {"y": _product(qa, sa, qw, sw)}
        return dict(y, qw=None, sw=sw.double()) if case["requant"] else y
    if kind == "layer":
        out = {n: _product(*_quant_act(s[x]), s["q_" + n], s["s_" + n]) for n, x in (("qkv", "x"), ("o_proj", "attn"))}
        out["gate_up"], out["down"] = _exact_mlp(*_quant_act(s["x2"]), s)
        return out
    if kind == "mlp":
        return dict(zip(("gate_up", "down"), _exact_mlp(*_quant_act(s["x"]), s)))
    if kind == "moe":
        return _exact_moe(case, s)
    if kind == "attn":
        return _exact_attn(case, s)
    if kind == "kv_prefill":
        scales = [_scale_of(s[n].abs().amax().float().reshape(1), "fp32").double() for n in ("k", "v")]
        return {"k_scale": scales[0], "v_scale": scales[1], "k_cache": None, "v_cache": None}
    if kind == "resync":
        return [x for w in s["ws"] for x in (None, _quant_weight(w)[1].double())]
    d = s["train"].double() - s["rollout"].double()
    on = s["mask"] != 0
    w = torch.exp(d)
    stats = torch.stack([-d[on].sum(), (torch.expm1(d[on]) - d[on]).sum(), on.sum().double(), (w[on] > 2.0).sum().double()])
    return {"w": torch.where(on, w.clamp(max=2.0), torch.zeros_like(w)), "stats": stats}
