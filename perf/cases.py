"""The calls whose speed is watched: tree-attention decode as a serving program makes it.

Every case is one tree, one head layout and one way of planning, and a pass is the attention call of one layer
through the binding (`deft_tree_attn_decode`), or, for the "iteration" cases, what one decode iteration costs: the
plan of the grown tree made from the plan before it, its upload, and the call of every layer.  Trees are the
shapes the benchmark and the tests use: few-shot, speculative, reasoning, long context, a single sequence, a
forest of sequences that share nothing.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2404_00242_amd import binding, workloads

PRECISE_PATH = 1024  # groups with a shorter path than this keep their softmax weights in two terms

# Fields of a case:
#   tree     shape of the tree, see _lens_parents_queries
#   a,b,lo,hi  its sizes (prefix or root tokens; width, tree nodes or depth; branch lengths from lo..hi)
#   Hq,Hkv,d heads and head dimension
#   split    "flatten" (the paper's, the default of deft_plan) or "balanced" (the benchmark's default)
#   chunk    tokens per chunk; 0: the library's default, -1: deft_suggest_chunk_size, as the README does
#   page     0: contiguous cache; P: a pool of P-token pages handed out in random order
#   f32      float32 output instead of bf16
#   layers   0: one layer-call on a plan that is kept; L: a decode iteration, re-planned, with L layer-calls


def _case(name, tree, a, b, lo, hi, Hq, Hkv, d=128, split="balanced", chunk=-1, page=0, f32=False, layers=0):
    c = dict(tree=tree, a=a, b=b, lo=lo, hi=hi, Hq=Hq, Hkv=Hkv, d=d, split=split, chunk=chunk, page=page, f32=f32,
             layers=layers)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest tree of the benchmark: launch latency and the host path are all there is
        _case("tiny", "fewshot", 256, 4, 32, 32, 4, 4, d=64),
        # few-shot prompting, one query per generation, multi-head attention: the benchmark's second workload
        _case("fewshot_mha", "fewshot", 4000, 20, 256, 256, 32, 32),
        # the same prompt with grouped-query heads over 16-token pages, as a serving engine stores it
        _case("fewshot_gqa_paged", "fewshot", 4000, 20, 256, 256, 32, 8, page=16),
        # a wide ragged few-shot tree planned with nothing but defaults (128-token chunks, equal-token split)
        _case("fewshot_defaults", "fewshot", 2977, 50, 1, 400, 32, 8, split="flatten", chunk=0),
        # speculative decoding: 64 one-token tree nodes over a committed prefix: the benchmark's third workload
        _case("speculative_mha", "speculative", 4000, 64, 1, 1, 32, 32),
        # a small draft tree over a longer grouped-query prefix, the README's way of planning, float32 out
        _case("speculative_gqa_f32", "speculative", 12345, 26, 1, 1, 32, 8, split="flatten", f32=True),
        # multi-step reasoning, 256 leaves: the benchmark's fourth workload
        _case("reasoning_gqa", "reasoning", 1000, 4, 128, 512, 32, 8),
        # a reasoning tree early on: every path is short, so softmax weights are kept in two terms; d = 64 heads
        _case("reasoning_short_d64", "reasoning", 200, 3, 32, 190, 32, 8, d=64),
        # a very long shared prefix with ragged branches: the benchmark's fifth workload and the largest call
        _case("longcontext_gqa", "longcontext", 32768, 64, 64, 2048, 32, 8),
        # one sequence, one query: where every tree begins, and what a step without branches costs
        _case("single_gqa", "single", 8191, 1, 0, 0, 32, 8, split="flatten"),
        # sixteen sequences of a batch that share nothing, some of them short
        _case("forest_gqa", "forest", 0, 16, 200, 4000, 32, 8),
        # one decode iteration of a model: every leaf has grown by a token, the plan follows, eight layers run
        _case("iteration_paged", "fewshot", 4000, 20, 1, 300, 32, 8, page=16, layers=8),
    ]


def draw(rng):
    """A case of the same ranges: the trees, heads and options above in other combinations and sizes."""
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    most = work(_case(None, "longcontext", 32768, 64, 64, 2048, 32, 8))
    while True:
        tree = rng.choice(["fewshot", "fewshot", "speculative", "speculative", "reasoning", "reasoning", "longcontext",
                           "single", "forest"])
        Hq, Hkv = rng.choice([(32, 32), (32, 8), (32, 8), (32, 8), (64, 8), (28, 4), (16, 16), (12, 2), (8, 8), (5, 5), (4, 4)])
        d = rng.choice([128, 128, 128, 64])
        split = rng.choice(["balanced", "balanced", "flatten"])
        chunk = rng.choice([-1, -1, 0, 256])
        page = rng.choice([0, 0, 0, 16, 64, 1])
        lo, hi, b = 0, 0, 1
        if tree == "fewshot":
            a, b, lo = log(200, 8000), log(2, 50), log(1, 256)
            hi = rng.randint(lo, 2 * lo + 16)
        elif tree == "speculative":
            a, b, lo, hi = log(500, 16000), log(4, 64), 1, 1
        elif tree == "reasoning":
            a, b, lo = log(100, 2000), rng.randint(2, 4), log(16, 128)
            hi = rng.randint(lo, 4 * lo)
        elif tree == "longcontext":
            a, b, lo = log(8192, 32768), log(4, 64), log(16, 64)
            hi = rng.randint(256, 2048)
        elif tree == "single":
            a = log(384, 32768)
        else:
            a, b, lo = 0, log(2, 32), log(64, 512)
            hi = rng.randint(lo, 4000)
        c = _case(None, tree, a, b, lo, hi, Hq, Hkv, d, split, chunk, page, rng.random() < 0.2)
        if page == 1 and a > 5000:
            continue
        if rng.random() < 0.15:
            c["layers"] = 4
        w = work(c)
        if w["bytes"] <= most["bytes"] and w["flops"] <= most["flops"]:
            return c


def _lens_parents_queries(case):
    """Node lengths, parents and query nodes of a case's tree; ragged lengths depend on its sizes alone."""
    tree, a, b, lo, hi = (case[k] for k in ("tree", "a", "b", "lo", "hi"))
    rng = np.random.default_rng([a, b, lo, hi])
    if tree == "fewshot":
        lens, parents = [a] + [int(x) for x in rng.integers(lo, hi + 1, b)], [-1] + [0] * b
        return lens, parents, list(range(1, b + 1))
    if tree == "speculative":
        t = workloads.config3_speculative(prefix=a, keep=b)
    elif tree == "reasoning":
        t = workloads.config4_reasoning(root=a, depth=b, lo=lo, hi=hi)
    elif tree == "longcontext":
        subs = min(8, b // 8)
        t = workloads.config5_longcontext(root=a, branches=b, lo=lo, hi=hi, sub_parents=subs)
    elif tree == "single":
        return [a], [-1], [0]
    else:
        return [int(x) for x in rng.integers(lo, hi + 1, b)], [-1] * b, list(range(b))
    return [int(x) for x in t.node_tok_len], [int(x) for x in t.node_parent], [int(x) for x in t.query_node]


def _storage(case, lens, spare):
    """(node_page_ptr, page_ids, pool pages) of a paged cache in which every node has room for `spare` more tokens,
    pages in random order; for a contiguous cache (node_tok_begin, None, rows)."""
    if not case["page"]:
        begins = np.concatenate([[0], np.cumsum(lens)[:-1]])
        return begins, None, int(sum(lens))
    need = [-(-(n + spare) // case["page"]) for n in lens]
    ptr = np.concatenate([[0], np.cumsum(need)])
    order = np.random.default_rng([case["a"], case["b"], case["page"]]).permutation(int(ptr[-1]) + 3)
    return ptr, order[: int(ptr[-1])], int(ptr[-1]) + 3


def _rows(case, store, lens, u):
    """Cache rows of node u's tokens, in order."""
    where, pages, _ = store
    t = np.arange(lens[u])
    if pages is None:
        return where[u] + t
    P = case["page"]
    return pages[where[u] + t // P] * P + t % P


def _plan(case, store, lens, parents, queries, prev=None):
    where, pages, room = store
    flags = binding.SPLIT_MODES[case["split"]]
    if case["split"] == "balanced":
        flags |= binding.rows_per_query(case["Hq"] // case["Hkv"])
    chunk = case["chunk"]
    if chunk < 0:
        chunk = binding.deft_suggest_chunk_size(lens, parents, queries, case["Hq"], case["Hkv"], flags)
    if pages is None:
        return binding.deft_plan(where, lens, parents, queries, room, chunk, flags, prev=prev)
    return binding.deft_plan_paged(where, pages, case["page"], room, lens, parents, queries, chunk, flags, prev=prev)


def prepare(case, seed):
    """What a serving loop holds: tables of the tree as it is now, the plan (of the tree one token ago, for an
    iteration), each layer's query and its K/V pools.  Values are N(0, 1) rounded to bf16, as in the benchmark."""
    dev = torch.device("cuda", torch.cuda.current_device())
    lens, parents, queries = (np.asarray(x, dtype=np.int32) for x in _lens_parents_queries(case))
    growing = case["layers"] > 0
    tips = np.zeros_like(lens)
    if growing:
        tips[queries] = 1
    before = lens - tips  # one iteration ago: the node of every query was a token shorter
    store = _storage(case, lens, 0)
    s = {"case": case, "lens": lens, "parents": parents, "queries": queries, "store": store}
    s["plan"] = _plan(case, store, before, parents, queries)
    if not growing:
        s["plan"].image(case["Hq"], case["Hkv"], dev)
    rows = store[2] * case["page"] if case["page"] else store[2]
    g = torch.Generator(device=dev).manual_seed(int(seed))
    s["q"], s["k"], s["v"] = [], [], []
    for _ in range(max(1, case["layers"])):
        q = torch.empty((len(queries), case["Hq"], case["d"]), dtype=torch.bfloat16, device=dev)
        k, v = binding.alloc_kv_cache(rows, case["Hkv"], case["d"], dev)
        for into, x in (("q", q), ("k", k), ("v", v)):
            s[into].append(x.normal_(generator=g))
    return s


def run(s):
    case = s["case"]
    dtype = torch.float32 if case["f32"] else torch.bfloat16
    plan = s["plan"]
    if case["layers"]:
        plan = _plan(case, s["store"], s["lens"], s["parents"], s["queries"], prev=plan)
    return [binding.deft_tree_attn_decode(plan, q, k, v, out_dtype=dtype) for q, k, v in zip(s["q"], s["k"], s["v"])]


def _path(parents, u):
    up = []
    while u >= 0:
        up.append(int(u))
        u = parents[u]
    return up[::-1]


def work(case):
    """K and V of every token some query sees, once per KV head, each query read and each result written; two products
    of 2 * d operations per (query head, token of its path)."""
    lens, parents, queries = _lens_parents_queries(case)
    seen = [False] * len(lens)
    path_tokens = 0
    for j in queries:
        path = _path(parents, j)
        path_tokens += sum(lens[u] for u in path)
        for u in path:
            seen[u] = True
    total = sum(n for n, on in zip(lens, seen) if on)
    L, Hq, Hkv, d = max(1, case["layers"]), case["Hq"], case["Hkv"], case["d"]
    rows = len(queries) * Hq
    return {"bytes": float(L * (total * Hkv * d * 4 + rows * d * (2 + (4 if case["f32"] else 2)))),
            "flops": float(L * 4 * path_tokens * Hq * d)}


def tolerance(case):
    """Against 64 bits a bf16 result is 2.3e-3 off (2-norm; 1.6e-3 of it the rounding of the output itself, the rest the
    bf16 softmax weights of long paths), a float32 result of long paths 1.6e-3; four times that.  Where every path is
    short the weights are held in two terms and a float32 result is good to 2.4e-6."""
    if not case["f32"]:
        return {"rel": 9e-3, "max": 6e-2}
    lens, parents, queries = _lens_parents_queries(case)
    if max(sum(lens[u] for u in _path(parents, j)) for j in queries) < PRECISE_PATH:
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 6.4e-3, "max": 4e-2}


def exact(case, seed):
    s = prepare(case, seed)
    lens, parents, queries, store = s["lens"], s["parents"], s["queries"], s["store"]
    Hq, Hkv, d = case["Hq"], case["Hkv"], case["d"]
    G, scale = Hq // Hkv, 1.0 / math.sqrt(d)
    outs = []
    for q, k, v in zip(s["q"], s["k"], s["v"]):
        k64, v64 = (x.double().transpose(0, 1).contiguous() for x in (k, v))  # [Hkv, rows, d]
        o = torch.zeros((len(queries), Hq, d), dtype=torch.float64, device=q.device)
        for j, u in enumerate(queries):
            at = torch.from_numpy(np.concatenate([_rows(case, store, lens, w) for w in _path(parents, u)])).to(q.device)
            kj, vj = k64[:, at], v64[:, at]
            p = torch.softmax(torch.matmul(q[j].double().view(Hkv, G, d), kj.transpose(1, 2).contiguous()) * scale, dim=-1)
            o[j] = torch.matmul(p, vj).reshape(Hq, d)
        outs.append(o)
    return outs
