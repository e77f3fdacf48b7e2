"""Performance cases: the work that a serving program has this library do, through its public entry points.

Three kinds of case:

  "step"   one layer step over the pool as the serving engine issues it when the base projections live elsewhere:
           LoRA q,k,v in one call, KV append and paged prefix attention in one call, LoRA o, and for the workload
           with adapters on the MLP gate,up (one call) and down.
  "layer"  one whole decoder layer (`fllayer.Layer.forward`): norms, dense projections with their LoRA branches,
           rotary embedding, append, attention, gated MLP.
  "moves"  blocks between the pinned host tier and the device tier: a fetch, a write-back, or both at once through
           the asynchronous planner, with a compute stream that waits for them.

A case's sizes (sequence lengths, adapters, ranks) are drawn from its "shape_seed", so every preparation of a case
asks for the same amount of work; `prepare`'s seed decides the contents and where in the pool the blocks lie.
"""
import math

import numpy as np
import torch

from paper_2505_03756_amd import fllayer, flpool, flsched
from paper_2505_03756_amd import workload as wl

TORCH_DTYPE = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
BYTES = {"f32": 4, "f16": 2, "bf16": 2}

# model shapes of the repository's workloads: hidden, query heads, kv heads, head_dim, MLP width
MODELS = {
    "tiny": (256, 4, 4, 64, 704),
    "7b": (4096, 32, 32, 128, 11008),
    "13b": (5120, 40, 40, 128, 13824),
    "34b": (8192, 64, 8, 128, 22016),
}


def _case(name, kind, model, dtype, n_seqs, prefix, new, decode_frac, n_adapters, ranks, dist, projections,
          block_tokens=16, shape_seed=1):
    return {"name": name, "kind": kind, "model": model, "dtype": dtype, "n_seqs": n_seqs, "prefix_lo": prefix[0],
            "prefix_hi": prefix[1], "new_lo": new[0], "new_hi": new[1], "decode_frac": decode_frac,
            "n_adapters": n_adapters, "rank_lo": ranks[0], "rank_hi": ranks[1], "adapter_dist": dist,
            "projections": projections, "block_tokens": block_tokens, "shape_seed": shape_seed}


def _moves(name, model, dtype, n_in, n_out, block_tokens=16):
    return {"name": name, "kind": "moves", "model": model, "dtype": dtype, "n_in": n_in, "n_out": n_out,
            "block_tokens": block_tokens}


def listed():
    return [
        # the smallest step: the fp32 workload, where launches and host work are everything
        _case("step_tiny_f32", "step", "tiny", "f32", 8, (0, 64), (1, 32), 0.0, 4, (8, 8), "uniform", "q,v"),
        # the decode workload: 256 running queries, one token each, adapters of mixed rank
        _case("step_7b_decode_bf16", "step", "7b", "bf16", 256, (512, 4096), (1, 1), 1.0, 100, (8, 64), "uniform", "q,k,v,o"),
        # the prefill workload: a batch of queries with reused prefixes
        _case("step_7b_prefill_f16", "step", "7b", "f16", 64, (0, 2048), (128, 512), 0.0, 32, (16, 16), "zipf", "q,k,v,o"),
        # adapters on all seven projections, the largest amount of LoRA work
        _case("step_13b_prefill_f16", "step", "13b", "f16", 128, (0, 4096), (128, 512), 0.0, 200, (32, 32), "zipf",
              "q,k,v,o,gate,up,down"),
        # prefill and decode mixed under grouped-query attention, contexts up to 16 k: the largest case
        _case("step_34b_mixed_bf16", "step", "34b", "bf16", 512, (0, 16384), (128, 512), 0.75, 500, (64, 64), "zipf", "q,k,v,o"),
        # a handful of long conversations being decoded (a lightly loaded server)
        _case("step_34b_longctx_bf16", "step", "34b", "bf16", 6, (8192, 16384), (1, 1), 1.0, 500, (64, 64), "uniform", "q,k,v,o"),
        # whole layer, a few queries being decoded: the weights are the traffic
        _case("layer_7b_decode8_bf16", "layer", "7b", "bf16", 8, (256, 2048), (1, 1), 1.0, 32, (16, 16), "uniform", "q,k,v,o"),
        # whole layer, a full decode batch
        _case("layer_7b_decode200_bf16", "layer", "7b", "bf16", 200, (256, 2048), (1, 1), 1.0, 100, (8, 64), "uniform", "q,k,v,o"),
        # whole layer, one query's prompt (what the time to first token of an idle server consists of)
        _case("layer_7b_prompt_f16", "layer", "7b", "f16", 1, (700, 700), (499, 499), 0.0, 32, (16, 16), "uniform", "q,k,v,o"),
        # whole layer, a batch of prompts, adapters on every projection
        _case("layer_13b_prefill_f16", "layer", "13b", "f16", 32, (0, 2048), (128, 512), 0.0, 200, (32, 32), "zipf",
              "q,k,v,o,gate,up,down"),
        # the fetch of a prefill batch's missing blocks (40 % of what it needs)
        _moves("fetch_7b_f16", "7b", "f16", 1400, 0),
        # one query joins, one leaves: a few blocks each way through the planner
        _moves("exchange_34b_bf16", "34b", "bf16", 150, 150),
    ]


def draw(rng):
    def log_int(lo, hi):
        return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))

    while True:
        c = _draw(rng, log_int)
        if c["kind"] == "moves":
            if (c["n_in"] + c["n_out"]) * block_bytes(c) <= 420e6:
                return c
            continue
        w = work(c)
        # no dearer than the largest listed cases: bytes, products and the size of the pool
        if w["bytes"] <= 16e9 and w["flops"] <= (9e12 if c["kind"] == "layer" else 11e12) and _pool_bytes(c) <= 17e9:
            return c


def _draw(rng, log_int):
    bt = 32 if rng.random() < 0.15 else 16
    kind = rng.choices(("step", "layer", "moves"), (9, 9, 3))[0]
    model = rng.choices(("tiny", "7b", "13b", "34b"), (1, 4, 2, 4))[0] if kind != "moves" else rng.choice(("7b", "13b", "34b"))
    dtype = rng.choice(("f16", "bf16"))
    if kind == "moves":
        way = rng.choice(("in", "out", "both"))
        n = log_int(1, 4000)
        m = log_int(1, 4000)
        c = _moves("", model, dtype, n if way != "out" else 0, m if way != "in" else 0, bt)
        del c["name"]
        return c
    if model == "tiny":
        dtype = "f32"
        n_seqs, hi, nlo, nhi, dec = log_int(1, 24), log_int(1, 512), 1, log_int(1, 64), rng.choice((0.0, 0.5, 1.0))
    else:
        phase = rng.choice(("decode", "prefill", "mixed"))
        if phase == "decode":
            n_seqs, hi, nlo, nhi, dec = log_int(1, 300), log_int(64, 16384), 1, 1, 1.0
        else:
            n_seqs, hi, nhi = log_int(1, 200), log_int(1, 8192), log_int(16, 1024)
            nlo = rng.randint(max(1, nhi // 4), nhi)
            dec = 0.0 if phase == "prefill" else rng.choice((0.5, 0.75))
    lo = rng.randint(0, hi)
    rank = rng.choice((8, 16, 32, 64))
    ranks = (8, rank) if rng.random() < 0.3 else (rank, rank)
    projections = "q,k,v,o,gate,up,down" if model != "34b" and rng.random() < 0.3 else ("q,v" if rng.random() < 0.1 else "q,k,v,o")
    c = _case("", kind, model, dtype, n_seqs, (lo, hi), (nlo, nhi), dec, log_int(4, 500), ranks,
              rng.choice(("uniform", "zipf")), projections, bt, rng.randrange(1 << 30))
    del c["name"]
    return c


# ------------------------------------------------------------------------------------------ shapes
def block_bytes(c):
    _, _, n_kv, d, _ = MODELS[c["model"]]
    return 2 * c["block_tokens"] * n_kv * d * BYTES[c["dtype"]]


def _config(c):
    hidden, n_q, n_kv, d, mlp = MODELS[c["model"]]
    ranks = tuple(r for r in (8, 16, 32, 64) if c["rank_lo"] <= r <= c["rank_hi"])
    return wl.LayerConfig(c["model"], c["dtype"], hidden, n_q, n_kv, d, 1, 1, c["n_adapters"], ranks,
                          tuple(c["projections"].split(",")), c["n_seqs"], (c["prefix_lo"], c["prefix_hi"]),
                          (c["new_lo"], c["new_hi"]), decode_frac=c["decode_frac"], adapter_dist=c["adapter_dist"],
                          block_tokens=c["block_tokens"], mlp_dim=mlp)


def _shape(c):
    """The step's sizes, adapters and tables; block ids 0, 1, 2, ... in the order they are asked for."""
    used = [0]

    def alloc(n):
        ids = np.arange(used[0], used[0] + n, dtype=np.int32)
        used[0] += n
        return ids

    st = wl.make_step(_config(c), seed=c["shape_seed"], alloc_dev=alloc, alloc_host=alloc, with_acts=False, fill_content=False)
    return st, used[0]


def _pool_bytes(c):
    return _shape(c)[1] * block_bytes(c)


def work(c):
    if c["kind"] == "moves":
        return {"bytes": 2.0 * (c["n_in"] + c["n_out"]) * block_bytes(c), "flops": 0.0}
    st, _ = _shape(c)
    cfg, e = st.cfg, BYTES[c["dtype"]]
    T, P, N = st.n_tokens, st.prefix_len.astype(np.float64), st.new_len.astype(np.float64)
    qd, kd = cfg.n_q_heads * cfg.head_dim, cfg.n_kv_heads * cfg.head_dim
    # attention: K and V of the prefixes once, the new K and V in and into the pool, q in and the result out
    by = (2 * P.sum() * kd + 4 * T * kd + 2 * T * qd) * e
    fl = 4.0 * qd * float((N * (P + (N + 1) / 2)).sum())
    rank_of_token = st.rank[st.token_adapter].astype(np.float64).sum()
    rank_sum = float(st.rank[np.unique(st.seq_adapter)].sum())
    for p in cfg.projections:                           # LoRA: the adapters' pages, two thin products
        d_in, d_out = cfg.proj_dims(p)
        by += rank_sum * (d_in + d_out) * e
        fl += 2.0 * rank_of_token * (d_in + d_out)
    if c["kind"] == "step":                             # x once for each call that shares it, every y in and out
        for group in (("q", "k", "v"), ("o",), ("gate", "up"), ("down",)):
            have = [p for p in group if p in cfg.projections]
            if have:
                by += T * cfg.proj_dims(have[0])[0] * e
            by += sum(2 * T * cfg.proj_dims(p)[1] * e for p in have)
    else:                                               # the dense weights, the residual stream in and out
        for p in ("q", "k", "v", "o", "gate", "up", "down"):
            d_in, d_out = cfg.proj_dims(p)
            by += d_in * d_out * e
            fl += 2.0 * T * d_in * d_out
        by += 2 * T * cfg.hidden * e
        by -= (4 * T * kd + 2 * T * qd) * e - 2 * T * kd * e    # q, k, v and the result need not leave the layer; K, V go to the pool
    return {"bytes": float(by), "flops": float(fl)}


def tolerance(c):
    if c["kind"] == "moves":
        return "exact"
    return {"rel": {"f32": 1e-5, "f16": 2e-3, "bf16": 1e-2}[c["dtype"]]}


# ------------------------------------------------------------------------------------------ inputs
def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return (_prepare_moves if case["kind"] == "moves" else _prepare_compute)(case, seed, g)


def _normal(shape, dtype, g, std=1.0):
    return torch.empty(shape, dtype=TORCH_DTYPE[dtype], device="cuda").normal_(0.0, std, generator=g)


def _prepare_compute(c, seed, g):
    st, n_blocks = _shape(c)
    cfg, dt = st.cfg, c["dtype"]
    hidden, n_q, n_kv, d, mlp = MODELS[c["model"]]
    T = st.n_tokens
    place = np.random.default_rng(seed).permutation(n_blocks).astype(np.int32)     # a shuffled free list
    kv_tables = np.where(st.kv_tables >= 0, place[np.maximum(st.kv_tables, 0)], -1).astype(np.int32)
    lora_tables = place[st.lora_tables].astype(np.int32)
    dev = _normal((n_blocks, cfg.block_elems), dt, g)
    for lo in range(0, len(lora_tables), 4096):
        ids = torch.from_numpy(lora_tables[lo:lo + 4096].astype(np.int64)).cuda()
        dev[ids] = _normal((len(ids), cfg.block_elems), dt, g, cfg.lora_std)
    pool = flpool.Pool(dt, n_kv, d, n_blocks, 0, block_tokens=cfg.block_tokens, dev=dev)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    s = {"kind": c["kind"], "pool": pool, "dev": dev, "dtype": dt, "T": T, "cu_new": st.cu_new, "prefix_len": st.prefix_len,
         "kv_tables": up(kv_tables), "lora_tables": up(lora_tables), "token_adapter": up(st.token_adapter),
         "rank": up(st.rank), "scale": up(st.scale), "n_adapters": len(st.rank), "max_rank": int(st.rank.max()),
         "n_q": n_q, "hidden": hidden, "mlp": mlp}
    places = {p: {k: up(getattr(pr, k)) for k in ("a_tab_off", "a_row_base", "b_tab_off", "b_row_base")}
              for p, pr in st.proj.items()}
    if c["kind"] == "step":
        s["x"] = _normal((T, hidden), dt, g)
        s["q"], s["k"], s["v"] = (_normal((T, n * d), dt, g) for n in (n_q, n_kv, n_kv))
        s["attn"] = torch.empty_like(s["q"])
        s["y"] = {p: _normal((T, pr.d_out), dt, g) for p, pr in st.proj.items()}
        s["act"] = _normal((T, mlp), dt, g) if "down" in st.proj else None
        s["calls"] = []
        for group, src, d_in in ((("q", "k", "v"), "x", hidden), (("o",), "attn", n_q * d), (("gate", "up"), "x", hidden),
                                 (("down",), "act", mlp)):
            projs = [dict(y=s["y"][p], d_out=st.proj[p].d_out, **places[p]) for p in group if p in st.proj]
            s["calls"].append((projs, src, d_in))
        return s
    dims = {p: cfg.proj_dims(p) for p in ("q", "k", "v", "o", "gate", "up", "down")}
    w = {p: _normal((o, i), dt, g, (0.25 if p in ("o", "down") else 1.0) / math.sqrt(i)) for p, (i, o) in dims.items()}
    w["in_norm"], w["post_norm"] = (1 + _normal((hidden,), dt, g, 0.05) for _ in range(2))
    s["layer"] = fllayer.Layer(pool, hidden, n_q, mlp, w)
    positions = np.concatenate([np.arange(p, p + n) for p, n in zip(st.prefix_len, st.new_len)]).astype(np.int32)
    s["batch"] = fllayer.Batch(st.cu_new, st.prefix_len, up(positions), s["kv_tables"], s["token_adapter"], s["rank"],
                               s["scale"], s["lora_tables"], places, s["n_adapters"], s["max_rank"], kv_tables.shape[1])
    s["h"] = _normal((T, hidden), dt, g)
    s["scratch_bytes"] = s["layer"].scratch_bytes(T)
    s["scratch"] = torch.empty(s["scratch_bytes"], dtype=torch.uint8, device="cuda")
    return s


def _prepare_moves(c, seed, g):
    _, _, n_kv, d, _ = MODELS[c["model"]]
    n = c["n_in"] + c["n_out"]
    elems = block_bytes(c) // BYTES[c["dtype"]]
    dev = _normal((n, elems), c["dtype"], g)
    host = torch.empty((n, elems), dtype=TORCH_DTYPE[c["dtype"]], pin_memory=True)
    host.copy_(_normal((n, elems), c["dtype"], g))
    pool = flpool.Pool(c["dtype"], n_kv, d, n, n, block_tokens=c["block_tokens"], dev=dev, host=host)
    rng = np.random.default_rng(seed)
    pd, ph = rng.permutation(n).astype(np.int32), rng.permutation(n).astype(np.int32)
    k = c["n_in"]
    return {"kind": "moves", "pool": pool, "dev": dev, "host": host, "in_dev": pd[:k], "in_host": ph[:k],
            "out_dev": pd[k:], "out_host": ph[k:], "planner": flsched.Planner(pool) if k and k < n else None, "request": 0}


# ------------------------------------------------------------------------------------------ one pass
def run(s):
    if s["kind"] == "moves":
        return _run_moves(s)
    if s["kind"] == "layer":
        s["layer"].forward(s["batch"], s["h"], s["scratch"], s["scratch_bytes"])
        return {"h": s["h"], "pool": s["dev"]}

    def lora(call):
        projs, src, d_in = call
        if projs:
            s["pool"].lora_apply_paged(s[src], s["token_adapter"], s["rank"], s["scale"], s["lora_tables"], projs,
                                       n_tokens=s["T"], d_in=d_in, n_adapters=s["n_adapters"], max_rank=s["max_rank"])

    qkv, o, gate_up, down = s["calls"]
    lora(qkv)
    s["pool"].paged_prefix_attention(s["q"], s["attn"], s["cu_new"], s["prefix_len"], s["kv_tables"], s["n_q"],
                                     k_new=s["k"], v_new=s["v"])
    lora(o)
    lora(gate_up)
    lora(down)
    # the pool's words as integers: appended K and V are copies, so they are the same bit for bit
    return {"attn": s["attn"], "y": s["y"], "pool": s["dev"].view(torch.int32 if s["dtype"] == "f32" else torch.int16)}


def _run_moves(s):
    pool = s["pool"]
    if s["planner"] is None:
        if len(s["in_dev"]):
            pool.swap_in(s["in_host"], s["in_dev"])
        else:
            pool.swap_out(s["out_dev"], s["out_host"])
    else:
        stream = torch.cuda.current_stream()
        s["request"] += 1
        s["planner"].compute_enqueued(stream)
        s["planner"].submit(s["request"], host_ids=s["in_host"], dev_ids=s["in_dev"], out_dev_ids=s["out_dev"],
                            out_host_ids=s["out_host"])
        s["planner"].stream_wait(s["request"], stream)
    return {"dev": s["dev"].view(torch.int16), "host": s["host"].view(torch.int16)}
