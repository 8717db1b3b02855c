"""The work that users of this framework have it do, as timed cases.

A case is either the prefill of one batch through a stack of decoder layers (submit, run to the
end, read the residual stream and the keys and values that a decode instance is handed) or one
projection through the single-operator entry point.  The sizes are those of this repository's
configurations (paper_2602_16603_amd/inputs.py) and of the traffic they stand for: requests of
16 to 32768 tokens alone, packed into batches of up to 4096 tokens, or as chunks of a longer
prompt; dense 8B- and 32B-shaped layers, the 30B-A3B mixture of experts, and the tiny shapes of
the parity workloads; bf16 for serving, fp32 for debugging.  Layers are alike, so one or two of
them stand for a stack.
"""
from __future__ import annotations

import math

import torch

from paper_2602_16603_amd import binding as B, inputs as I, runner as R

SHAPES = {"tiny": I.TINY, "8b": I.LLAMA3_8B, "32b": I.QWEN25_32B, "tiny_moe": I.TINY_MOE, "30b_a3b": I.QWEN3_30B_A3B}
DTYPES = {"bf16": (B.FP_DTYPE_BF16, torch.bfloat16), "fp32": (B.FP_DTYPE_F32, torch.float32)}
BLOCK = 16                       # tokens per KV-cache block
TOKEN_BUDGET = 4096              # tokens of a batch of packed requests
SHORT = 1024                     # requests up to this run without a launch-ahead bound


def _prefill(name, shape, layers, dtype, lengths, cached=0):
    """One batch of prompts (`lengths`: tokens, separated by commas) through `layers` layers; each
    prompt's first `cached` positions are in the paged cache already."""
    return {"name": name, "kind": "prefill", "shape": shape, "layers": layers, "dtype": dtype,
            "lengths": ",".join(str(n) for n in lengths), "cached": cached}


def _projection(name, m, n, k, residual):
    return {"name": name, "kind": "projection", "m": m, "n": n, "k": k, "residual": residual}


def listed():
    return [
        # The smallest call: the tiny stack on one short prompt (the parity workload, and what a
        # program runs to see that everything is in place).  Launches and host work.
        _prefill("tiny_prompt", "tiny", 2, "bf16", [200]),
        # A layer of the real shape in fp32, the debug path: a prompt of a few hundred tokens.
        _prefill("debug_fp32", "8b", 1, "fp32", [300]),
        # The short interactive request that preempts a long prompt.
        _prefill("request_256", "8b", 2, "bf16", [256]),
        # A few words: a request far below one tile of rows.
        _prefill("request_50", "8b", 1, "bf16", [50]),
        # The mean text request of the traffic, an odd length.
        _prefill("request_777", "8b", 1, "bf16", [777]),
        # Requests packed to the scheduler's token budget, blocks scattered over the pool.
        _prefill("packed_batch", "8b", 1, "bf16", [1213, 64, 590, 2002, 227]),
        # Chunked prefill: the last 512-token chunk of a 16384-token prompt.
        _prefill("chunk_512_of_16384", "8b", 1, "bf16", [512], 15872),
        # The benchmark's prompt.
        _prefill("prompt_8192", "8b", 1, "bf16", [8192]),
        # The longest prompt: the one that short requests preempt.
        _prefill("prompt_32768", "8b", 1, "bf16", [32768]),
        # A search request on the larger dense shape.
        _prefill("prompt_3001_32b", "32b", 1, "bf16", [3001]),
        # Mixture of experts: the long prompt, and the mean text request.
        _prefill("moe_8192", "30b_a3b", 1, "bf16", [8192]),
        _prefill("moe_590", "30b_a3b", 1, "bf16", [590]),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["alone", "alone", "alone", "packed", "chunk", "moe", "moe", "32b", "tiny", "fp32", "projection"])
    if kind == "alone":
        return _prefill("", "8b", rng.choice([1, 1, 2]), "bf16", [_log_int(rng, 16, 16384)])
    if kind == "packed":
        left, lengths = TOKEN_BUDGET, []
        for _ in range(rng.randint(2, 12)):
            n = min(left, _log_int(rng, 16, 2048))
            if n >= 16:
                lengths.append(n)
                left -= n
        return _prefill("", "8b", 1, "bf16", lengths)
    if kind == "chunk":
        return _prefill("", "8b", 1, "bf16", [_log_int(rng, 128, 2048)], BLOCK * _log_int(rng, 64, 1536))
    if kind == "moe":
        return _prefill("", "30b_a3b", 1, "bf16", [_log_int(rng, 16, 16384)])
    if kind == "32b":
        return _prefill("", "32b", 1, "bf16", [_log_int(rng, 64, 12000)])
    if kind == "tiny":
        return _prefill("", rng.choice(["tiny", "tiny", "tiny_moe"]), 2, "bf16", [_log_int(rng, 16, 1024)])
    if kind == "fp32":
        if rng.random() < 0.5:
            return _prefill("", "tiny", 2, "fp32", [_log_int(rng, 16, 1024)])
        return _prefill("", "8b", 1, "fp32", [_log_int(rng, 32, 512)])
    # One projection of a shape of the caller's own: any multiple of eight for N and K.
    return _projection("", _log_int(rng, 16, 8192), 8 * _log_int(rng, 32, 1024), 8 * _log_int(rng, 32, 1024),
                       rng.random() < 0.5)


def _lengths(case):
    return [int(n) for n in case["lengths"].split(",")]


def _spec(case):
    return SHAPES[case["shape"]].with_layers(case["layers"])


def _weights(case, seed):
    weights = I.make_weights(_spec(case), seed, DTYPES[case["dtype"]][1], "cuda")
    I.randomize_gains(weights, seed)
    return weights


def _hidden(case, seed):
    """The batch's input rows, each prompt's cached positions in front of its new ones."""
    n = sum(_lengths(case)) + case["cached"] * len(_lengths(case))
    return I.make_hidden(n, _spec(case).hidden, seed, DTYPES[case["dtype"]][1], "cuda")


def _operands(case, seed):
    a = I.normal_tensor((case["m"], case["k"]), 1.0, seed, torch.bfloat16, "cuda")
    w = I.normal_tensor((case["n"], case["k"]), 0.02, seed + 1, torch.bfloat16, "cuda")
    x = I.normal_tensor((case["m"], case["n"]), 1.0, seed + 2, torch.float32, "cuda") if case["residual"] else None
    return a, w, x


def prepare(case, seed):
    if case["kind"] == "projection":
        a, w, x = _operands(case, seed)
        ws_bytes = B.fp_op_gemm_workspace_bytes(B.FP_DTYPE_BF16, case["m"], case["n"], case["k"])
        ws = torch.empty(max(ws_bytes, 256), dtype=torch.uint8, device="cuda")
        out = None if case["residual"] else torch.empty(case["m"], case["n"], dtype=torch.bfloat16, device="cuda")
        return {"case": case, "a": a, "w": w, "x": x, "out": out, "ws": ws, "ws_bytes": ws_bytes}
    lengths, cached = _lengths(case), case["cached"]
    spec = _spec(case)
    total = sum(lengths) + cached * len(lengths)
    past = [cached] * len(lengths)
    pool = total // BLOCK + 2 * len(lengths) + 32
    model = R.PrefillModel(spec, _weights(case, seed), DTYPES[case["dtype"]][0], 2 * pool, max(lengths) + cached)
    # Blocks of a pool that has been in use lie scattered over it.
    table, _ = I.permuted_block_tables(lengths, past, BLOCK, pool, seed)
    hidden = _hidden(case, seed)
    state = {"case": case, "model": model, "lengths": lengths, "past": past, "table": table, "hidden": hidden}
    if cached:
        rows = list(hidden.split([v for n in lengths for v in (cached, n)]))
        state["hidden"] = torch.cat(rows[1::2]).contiguous()
        first = model.begin(torch.cat(rows[0::2]).contiguous(), past, [0] * len(lengths), table)
        first.run_to_completion()
        first.end()
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "projection":
        # The residual is updated in a copy: the same state can be run again.
        out = state["x"].clone() if case["residual"] else state["out"]
        B.fp_op_gemm_ws(B.FP_DTYPE_BF16, state["a"].data_ptr(), state["w"].data_ptr(), out.data_ptr(), case["m"],
                        case["n"], case["k"], case["residual"], state["ws"].data_ptr(), state["ws_bytes"],
                        torch.cuda.current_stream().cuda_stream)
        return out
    task = state["model"].begin(state["hidden"], state["lengths"], state["past"], state["table"])
    if sum(state["lengths"]) <= SHORT:
        B.fp_prefill_set_launch_ahead(task.handle, 0)
    task.run_to_completion()
    hidden = task.hidden()
    kv = [task.kv(layer, s) for layer in range(case["layers"]) for s in range(len(state["lengths"]))]
    task.end()
    return {"hidden": hidden, "kv": kv}


def work(case):
    if case["kind"] == "projection":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": 2 * (m * k + n * k) + m * n * (8 if case["residual"] else 2), "flops": 2 * m * n * k}
    spec, lengths, cached = _spec(case), _lengths(case), case["cached"]
    e = 4 if case["dtype"] == "fp32" else 2
    t, d = sum(lengths), spec.hidden
    qd = spec.n_q_heads * spec.head_dim
    pairs = sum(n * cached + n * (n + 1) // 2 for n in lengths)
    active = spec.params_per_layer()
    touched = active
    if spec.n_experts:
        expert = 3 * d * spec.ffn
        active += expert * (spec.top_k - spec.n_experts)
        # Experts that t tokens with top_k choices each reach, spread evenly.
        reached = spec.n_experts * (1 - (1 - spec.top_k / spec.n_experts) ** t)
        touched += int(expert * (reached - spec.n_experts))
    flops = case["layers"] * (2 * t * active + 4 * spec.n_q_heads * spec.head_dim * pairs)
    kv = 2 * spec.n_kv_heads * spec.head_dim * e
    # Weights, the cached positions' keys and values in; hidden states in; residual out; keys and
    # values into the cache and, contiguous, out of it.
    moved = case["layers"] * (touched * e + kv * (3 * t + 2 * cached * len(lengths))) + t * d * (e + 4)
    return {"bytes": int(moved), "flops": int(flops)}


def tolerance(case):
    """Four times the error measured against exact() at these sizes: 2.3e-3 for a bf16 output of one
    projection, up to 5.6e-3 for the residual behind one layer (its intermediates are bf16) and 7.6e-3
    behind two, 3e-6 for a layer in fp32."""
    if case["kind"] == "projection":
        return {"rel": 1e-2}
    if case["dtype"] == "fp32":
        return {"rel": 1.2e-5}
    return {"rel": 2e-2 if case["layers"] == 1 else 2.9e-2}


# ---- the same in 64 bits ----

def _rope(x, pos, theta):
    half = x.shape[-1] // 2
    freq = theta ** (-torch.arange(half, dtype=torch.float64, device=x.device) * 2.0 / x.shape[-1])
    angle = pos.double()[:, None] * freq[None, :]
    c, s = angle.cos()[:, None, :], angle.sin()[:, None, :]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], dim=-1)


def _norm(x, gain, eps):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * gain


def _attend(q, k, v, scale):
    """Causal attention of the last len(q) positions over all of them, a stretch of queries at a time."""
    out = torch.empty_like(q)
    n, total = q.shape[0], k.shape[0]
    group = q.shape[1] // k.shape[1]
    key = torch.arange(total, device=q.device)
    step = max(1, (1 << 27) // total)
    for h in range(q.shape[1]):
        kh, vh = k[:, h // group], v[:, h // group]
        for lo in range(0, n, step):
            hi = min(n, lo + step)
            seen = total - n + hi
            s = (q[lo:hi, h] @ kh[:seen].T) * scale
            s.masked_fill_(key[None, :seen] > (total - n + torch.arange(lo, hi, device=q.device))[:, None], -math.inf)
            out[lo:hi, h] = torch.softmax(s, dim=-1) @ vh[:seen]
    return out


def _ffn(h, w, spec):
    def glu(rows, gate_up, down):
        g, u = (rows @ gate_up.T).split(spec.ffn, dim=-1)
        return (torch.nn.functional.silu(g) * u) @ down.T
    if not spec.n_experts:
        return torch.cat([glu(r, w["w_gate_up"].double(), w["w_down"].double()) for r in h.split(8192)])
    p, chosen = torch.softmax(h @ w["w_router"].double().T, dim=-1).topk(spec.top_k, dim=-1)
    p = p / p.sum(-1, keepdim=True)
    out = torch.zeros_like(h)
    for e in range(spec.n_experts):
        token, slot = (chosen == e).nonzero(as_tuple=True)
        if token.numel():
            out.index_add_(0, token, p[token, slot, None] * glu(h[token], w["w_gate_up"][e].double(), w["w_down"][e].double()))
    return out


def exact(case, seed):
    if case["kind"] == "projection":
        a, w, x = _operands(case, seed)
        y = a.double() @ w.double().T
        return y if x is None else y + x.double()
    spec, lengths, cached = _spec(case), _lengths(case), case["cached"]
    x = _hidden(case, seed).double()
    full = [n + cached for n in lengths]
    pos = torch.cat([torch.arange(n, device="cuda") for n in full])
    hq, hk, dim = spec.n_q_heads, spec.n_kv_heads, spec.head_dim
    kv = []
    for w in _weights(case, seed):
        h = _norm(x, w["attn_norm"].double(), spec.rms_eps)
        qkv = (h @ w["w_qkv"].double().T).view(-1, hq + 2 * hk, dim)
        q, k, v = qkv.split([hq, hk, hk], dim=1)
        q, k = _rope(q, pos, spec.rope_theta), _rope(k, pos, spec.rope_theta)
        parts = list(zip(q.split(full), k.split(full), v.split(full)))
        kv += [(ks, vs) for _, ks, vs in parts]
        o = torch.cat([_attend(qs, ks, vs, dim ** -0.5) for qs, ks, vs in parts]).reshape(-1, hq * dim)
        x = x + o @ w["w_o"].double().T
        x = x + _ffn(_norm(x, w["mlp_norm"].double(), spec.rms_eps), w, spec)
    return {"hidden": torch.cat([xs[cached:] for xs in x.split(full)]), "kv": kv}
