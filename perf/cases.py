"""The work whose speed is measured: what a user of the blended decoder-layer step has it do.

A case is a dict of plain values.  `path` names the entry point, `shape` the layer, the rest the batch:

  step       Layer.blend_step, one forward step of one layer (the call a serving loop makes per layer)
  layers     Layer.blend_layers, one descriptor through several layers with weights and pools of their own
  attention  Layer.attention, the paged attention alone over an appended pool
  pool       engine.make_scheduler + engine.serve + Layer.blend_step: a request pool served to completion

Batches are either one of the named configurations of `workloads` (`config`) or laid out from numbers:
`segments` prefill chunks of about `rows` rows behind about `cached` tokens of their own, and `decode`
sequences in `groups` prefix groups (`prefix` shared tokens; `children` sub-groups of `child_prefix` further
tokens) with private tails of about `tail` tokens.  `ragged` spreads all lengths, `layout` seeds them.
Lengths follow from the case alone; physical pages, weights, activations and cached keys and values
follow from the seed (N(0, 0.02^2) weights, N(0, 1) activations and cache, gains around 1).
"""
import ctypes
import math

import numpy as np
import torch

import paper_2411_16102_amd as pkg
from paper_2411_16102_amd import binding, engine, workloads as W

SHAPES = {
    "tiny": W.TINY,
    "head64": W.LayerShape(2048, 32, 8, 64, 8192),   # a small layer with 64-wide heads
    "8b": W.LLAMA3_8B,
    "70b": W.LLAMA3_70B,
}
PAGE = W.PAGE
MAX_CONTEXT = 16384   # positions of a layer context created with its defaults


def listed():
    blank = dict(config="", segments=0, rows=0, cached=0, decode=0, groups=0, prefix=0, children=0, child_prefix=0, tail=0,
                 ragged=True, layout=0, layers=1, flags=0)

    def case(name, path, shape, **kw):
        return dict(blank, name=name, path=path, shape=shape, **kw)

    return [
        # the smallest whole step: launches and host work are all there is to it
        case("tiny_blended", "step", "tiny", config="tiny"),
        # the end of a pool: a handful of long outputs still decoding; every weight is read for seven rows
        case("decode_few_8b", "step", "8b", decode=7, tail=2000, layout=1),
        # an odd number of decode rows, part of them behind shared system prompts
        case("decode_shared_8b", "step", "8b", decode=77, groups=3, prefix=1024, tail=500, layout=2),
        # the memory-bound configuration: 256 sequences of context 1024
        case("decode_8b", "step", "8b", config="decode_8b"),
        # the compute-bound configuration: 8 segments of 1024 rows
        case("prefill_8b", "step", "8b", config="prefill_8b"),
        # chunked prefill of two long prompts: attention over many cached tokens
        case("prefill_long_8b", "step", "8b", segments=2, rows=1024, cached=9000, layout=3),
        # an ordinary step of a pool run: ragged chunks, some behind cached tokens, and grouped decode rows
        case("step_odd_8b", "step", "8b", segments=5, rows=187, cached=300, decode=487, groups=20, prefix=700, tail=600, layout=4),
        # the blended configuration of the benchmark, with co-scheduling allowed
        case("blended_8b", "step", "8b", config="blended_8b", flags=1),
        # the large blended configuration
        case("blended_70b", "step", "70b", config="blended_70b", flags=1),
        # layers back to back behind one descriptor, as an engine runs them; 64-wide heads
        case("layers_head64", "layers", "head64", segments=2, rows=150, cached=100, decode=129, groups=8, prefix=256, tail=400,
             layout=5, layers=4, flags=1),
        # attention alone under a two-level prefix tree
        case("attention_tree_70b", "attention", "70b", decode=640, groups=8, prefix=2048, children=5, child_prefix=512, tail=400,
             layout=6),
        # a small pool from its first step to its last: scheduler, descriptors and steps of every size
        case("pool_8b", "pool", "8b", layout=7, groups=3, decode=4, segments=8, tail=40, rows=1024),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        c = dict(path=rng.choices(["step", "layers", "attention"], [8, 1, 2])[0], shape=rng.choices(list(SHAPES), [1, 2, 6, 1])[0],
                 config="", segments=0, rows=0, cached=0, decode=0, groups=0, prefix=0, children=0, child_prefix=0, tail=0,
                 ragged=rng.random() < 0.8, layout=rng.randrange(1 << 20), layers=1, flags=rng.choice([0, 1]))
        kind = rng.choice(["decode", "decode", "prefill", "blended", "blended"])
        if kind != "decode":
            total = _log_int(rng, 16, 8192 if kind == "prefill" else 4096)
            c["segments"] = rng.randint(1, min(8, max(1, total // 16)))
            c["rows"] = max(1, total // c["segments"])
            c["cached"] = rng.choice([0, _log_int(rng, 16, 9000)])
        if kind != "prefill":
            c["decode"] = _log_int(rng, 1, 1024)
            c["tail"] = _log_int(rng, 16, 4096)
            if c["decode"] >= 4 and rng.random() < 0.6:
                c["groups"] = rng.randint(1, max(1, min(32, c["decode"] // 4)))
                c["prefix"] = PAGE * _log_int(rng, 1, 128)
                if rng.random() < 0.3:
                    c["children"], c["child_prefix"] = rng.randint(2, 6), PAGE * _log_int(rng, 1, 32)
        if c["path"] == "layers":
            c["layers"] = rng.randint(2, 4)
        w = work(c)
        if w["flops"] <= 8.0e12 and w["bytes"] <= 4.0e9 and (c["path"] != "attention" or w["bytes"] > 1e6):
            return c


# ---- batches -----------------------------------------------------------------
def _spread(rng, n, mean, ragged):
    """n lengths around `mean`, at least 1."""
    f = np.exp(0.5 * rng.standard_normal(n)) if ragged else np.ones(n)
    return np.maximum(1, np.rint(mean * f)).astype(np.int64)


def _batch(case, seed):
    """The step's descriptor: lengths from the case, physical pages from the seed."""
    if case["config"]:
        b = W.CONFIGS[case["config"]][1](seed=0)
        perm = np.random.default_rng([seed, 11]).permutation(b.n_pages)
        b.page_ids = np.ascontiguousarray(perm[b.page_ids], dtype=np.int32)
        b.node_page_ids = np.ascontiguousarray(perm[b.node_page_ids], dtype=np.int32)
        return b
    rng = np.random.default_rng([case["layout"], 3])
    rows = np.minimum(_spread(rng, case["segments"], case["rows"], case["ragged"]), MAX_CONTEXT // 2)
    held = _spread(rng, case["segments"], case["cached"], case["ragged"]) if case["cached"] else np.zeros(case["segments"], dtype=np.int64)
    seqs = [(int(q), int(q + min(h, MAX_CONTEXT - q)), -1) for q, h in zip(rows, held)]
    nodes, leaves = [], []
    for _ in range(case["groups"]):
        root = len(nodes)
        nodes.append((-1, case["prefix"] // PAGE))
        for _ in range(case["children"]):
            nodes.append((root, case["child_prefix"] // PAGE))
        leaves += list(range(root + 1, len(nodes))) if case["children"] else [root]
    tails = _spread(rng, case["decode"], case["tail"], case["ragged"])
    shared = case["prefix"] + (case["child_prefix"] if case["children"] else 0) if case["groups"] else 0
    # members of a leaf are neighbours; about a tenth of the sequences of a ragged batch stand outside the groups
    member = case["decode"] - (case["decode"] // 10 if case["ragged"] else 0) if leaves else 0
    for i, t in enumerate(tails):
        leaf = leaves[i * len(leaves) // member] if i < member else -1
        above = shared if leaf >= 0 else 0
        seqs.append((1, int(min(above + t, MAX_CONTEXT)), leaf))
    return W.assemble_batch(PAGE, seqs, case["segments"], nodes, np.random.default_rng([seed, 11]))


# ---- the request pool ----------------------------------------------------------
POOL_TOKENS, POOL_PAGES = 60_000, 8192


def _pool_requests(case):
    reqs = W.synthetic_pool(case["layout"], n_groups=case["groups"], per_group=case["decode"], n_fresh=case["segments"])
    for r in reqs:                # outputs short enough that a pass stays well under a second
        r.d_true, r.d_est = min(r.d_true, case["tail"]), min(r.d_est, case["tail"])
    return reqs


def _pool_scheduler(case, reqs):
    shape = SHAPES[case["shape"]]
    hw = dict(p_model=8_030_000_000, kv_bytes=shape.kv_bytes_per_token * 32, compute=2.5e15, bandwidth=8.0e12)
    return engine.make_scheduler(pkg.load(), reqs, hw, POOL_TOKENS, case["rows"], POOL_PAGES, split_t=4096,
                                 split_budget=int(0.01 * sum(len(r.tokens) for r in reqs)))


def _pool_batch(d):
    return W.Batch(page_size=PAGE, **{k: v for k, v in d.items() if k != "seq_request"})


# ---- inputs ----------------------------------------------------------------------
def _normal(gen, shape, std=1.0, mean=0.0):
    out = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    flat = out.view(-1)
    for lo in range(0, flat.numel(), 1 << 28):
        part = flat[lo:lo + (1 << 28)]
        part.normal_(mean, std, generator=gen)
    return out


def _weights(gen, shape):
    d, f, hd = shape.d_model, shape.d_ffn, shape.n_q_heads * shape.head_dim
    keep = [_normal(gen, (shape.n_qkv, d), 0.02), _normal(gen, (d, hd), 0.02), _normal(gen, (2 * f, d), 0.02),
            _normal(gen, (d, f), 0.02), _normal(gen, (d,), 0.1, 1.0), _normal(gen, (d,), 0.1, 1.0)]
    return binding.Weights(*[ctypes.c_void_p(k.data_ptr()) for k in keep]), keep


def prepare(case, seed):
    api = pkg.load()
    shape = SHAPES[case["shape"]]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    layer = api.Layer(shape, device=0)
    page_elems = layer.page_bytes() // 2
    if case["path"] == "pool":
        reqs = _pool_requests(case)
        _, sched, _ = _pool_scheduler(case, reqs)
        total = int(engine.serve(sched, lambda d: None)["rows"])
        w, keep = _weights(gen, shape)
        x = _normal(gen, (total, shape.d_model))
        pool = torch.zeros(POOL_PAGES * page_elems, dtype=torch.bfloat16, device="cuda")
        return dict(case=case, layer=layer, api=api, reqs=reqs, w=w, keep=keep, x=x, y=torch.empty_like(x), pool=pool)
    batch = _batch(case, seed)
    if case["path"] == "attention":
        q = _normal(gen, (batch.n_rows, shape.n_q_heads * shape.head_dim))
        pool = _normal(gen, (batch.n_pages * page_elems,))
        return dict(case=case, layer=layer, batch=batch, q=q, pool=pool)
    devs = []
    x = _normal(gen, (batch.n_rows, shape.d_model))
    for _ in range(case["layers"]):
        w, keep = _weights(gen, shape)
        devs.append(api.binding_device_state(w, keep, x, _normal(gen, (batch.n_pages * page_elems,)), batch.n_pages))
    return dict(case=case, layer=layer, batch=batch, devs=devs, y=torch.empty_like(x))


def run(state):
    case, layer = state["case"], state["layer"]
    if case["path"] == "step":
        dev = state["devs"][0]
        layer.blend_step(dev, state["batch"], flags=case["flags"], y=state["y"])
        return {"y": state["y"], "kv_pool": dev.kv_pool}
    if case["path"] == "layers":
        layer.blend_layers(state["devs"], state["batch"], flags=case["flags"], y=state["y"])
        return {"y": state["y"], "kv_pools": [d.kv_pool for d in state["devs"]]}
    if case["path"] == "attention":
        return layer.attention(state["batch"], state["q"], state["pool"], state["batch"].n_pages)
    _, sched, _ = _pool_scheduler(case, state["reqs"])
    at = [0]

    def step(d):
        lo, hi = at[0], at[0] + d["n_rows"]
        at[0] = hi
        dev = state["api"].binding_device_state(state["w"], state["keep"], state["x"][lo:hi], state["pool"], POOL_PAGES)
        layer.blend_step(dev, _pool_batch(d), flags=case["flags"], y=state["y"][lo:hi])

    engine.serve(sched, step)
    return {"y": state["y"], "kv_pool": state["pool"]}


def work(case):
    shape = SHAPES[case["shape"]]
    if case["path"] == "pool":
        steps = []
        _, sched, _ = _pool_scheduler(case, _pool_requests(case))
        engine.serve(sched, lambda d: steps.append(W.work_of(shape, _pool_batch(d))))
        return {"bytes": sum(w["bytes_once"] for w in steps), "flops": sum(w["flops"] for w in steps)}
    batch = _batch(case, 0)
    w = W.work_of(shape, batch)
    if case["path"] == "attention":
        io = 2 * 2.0 * batch.n_rows * shape.n_q_heads * shape.head_dim
        return {"bytes": w["kv_tokens_once"] * shape.kv_bytes_per_token + io, "flops": w["flops"] - w["gemm_flops"]}
    return {"bytes": w["bytes_once"] * case["layers"], "flops": w["flops"] * case["layers"]}


def tolerance(case):
    # bfloat16 storage between operators, float32 sums.  The same path with its sums in another order (other GEMM
    # tiles, other chunks of the attention) differs by up to 3.0e-3 (relative) and 2.4e-2 (single values).
    return {"rel": 1.2e-2, "max": 0.1}
