"""The work that a user of this library has it do, as cases to be measured: attention of one layer
over batches of reasoning DAGs, called through `paper_2602_07529_amd.binding`.

Five kinds of pass:
  prefill   the node table becomes meta tables, Q and K are rotated in place, attention (inference)
  train     attention forward with log-sum-exp, then its backward (the meta belongs to the batch and
            is shared by all layers of a model, so it is built once)
  decode    one step of every live branch: K/V append, then cascade attention over the shared
            context of its sibling group and its own pages
  frontier  the same over contexts given as lists of KV segments (root | mid nodes | live leaves)
  paged     new tokens of many nodes: K/V append, then prefill against the cached pages
`listed()` takes the benchmark's configurations where there is one and generic sizes otherwise; the
rest of a case's fields are what `draw()` varies.
"""
import math
import random

import numpy as np
import torch

from paper_2602_07529_amd import binding as B

PAGE = 16
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
LAYER = dict(hq=32, hkv=8, d=128)


def listed():
    return [
        # one small request in the accuracy path's data type: launches and latency
        dict(name="tiny_prefill_f32", kind="prefill", dtype="f32", dag="fork", batch=1, prefix=128, branches=4,
             branch=64, join=64, jitter=0, hq=4, hkv=4, d=64, theta=10000.0, dag_seed=0),
        # one short interactive request with uneven branches: launches and latency in bf16
        dict(name="short_prefill_bf16", kind="prefill", dtype="bf16", dag="fork", batch=1, prefix=301, branches=3,
             branch=90, join=77, jitter=20, theta=500000.0, dag_seed=1, **LAYER),
        # a batch of prompts with eight plans each: the benchmark's prefill
        dict(name="layer_prefill_bf16", kind="prefill", dtype="bf16", dag="fork", batch=4, prefix=2048, branches=8,
             branch=256, join=512, jitter=0, theta=500000.0, dag_seed=2, **LAYER),
        # multi-level DAGs with joins and node lengths that are no multiple of a tile: half the tiles are masked
        dict(name="random_prefill_bf16", kind="prefill", dtype="bf16", dag="random", batch=8, nodes=64, depth=6,
             len_lo=32, len_hi=256, theta=500000.0, dag_seed=3, **LAYER),
        # the longest contexts, five query heads for each KV head
        dict(name="long_prefill_bf16", kind="prefill", dtype="bf16", dag="fork", batch=2, prefix=32768, branches=32,
             branch=512, join=1024, jitter=0, hq=40, hkv=8, d=128, theta=1000000.0, dag_seed=4),
        # fine-tuning through the mask on the benchmark's prompts
        dict(name="layer_train_bf16", kind="train", dtype="bf16", dag="fork", batch=4, prefix=2048, branches=8,
             branch=256, join=512, jitter=0, dag_seed=5, **LAYER),
        # fine-tuning a model with small heads on multi-level DAGs
        dict(name="random_train_d64_bf16", kind="train", dtype="bf16", dag="random", batch=4, nodes=64, depth=6,
             len_lo=32, len_hi=256, hq=16, hkv=8, d=64, dag_seed=6),
        # a single request that decodes four branches: latency
        dict(name="single_decode_bf16", kind="decode", groups=1, branches=4, shared=1500, own=200, jitter=50,
             theta=500000.0, dag_seed=7, **LAYER),
        # a full serving batch: the benchmark's decode
        dict(name="branch_decode_bf16", kind="decode", groups=16, branches=8, shared=8192, own=1024, jitter=0,
             theta=500000.0, dag_seed=8, **LAYER),
        # few requests with many siblings over a very long shared context
        dict(name="wide_decode_bf16", kind="decode", groups=2, branches=32, shared=32768, own=640, jitter=0,
             hq=40, hkv=8, d=128, theta=1000000.0, dag_seed=9),
        # live leaves under two levels of shared nodes, partly filled pages
        dict(name="frontier_decode_bf16", kind="frontier", groups=16, mids=2, leaves=4, reads=1, root=4096, mid=2048,
             own=1031, jitter=31, theta=500000.0, dag_seed=10, **LAYER),
        # step headers and join prompts of many nodes prefilled against their cached predecessors
        dict(name="paged_prefill_bf16", kind="paged", groups=16, nodes=8, shared=8192, own=1024, new=256, jitter=0,
             theta=500000.0, dag_seed=11, **LAYER),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        case = _draw(rng)
        flops, most = work(case)["flops"], 4.0e13
        if case.get("dtype") == "f32":
            most = 1.0e11
        elif case["kind"] == "train":
            most = 8.0e12
        elif case["kind"] == "paged":
            most = 2.0e13
        if flops <= most and _pool_tokens(case) <= 600000:
            return case


def _draw(rng):
    kind = rng.choice(["prefill", "prefill", "train", "decode", "decode", "frontier", "paged"])
    case = dict(kind=kind, dag_seed=rng.randrange(1 << 30), hkv=rng.choice([1, 2, 4, 8]), d=rng.choice([64, 128, 128]),
                theta=rng.choice([10000.0, 500000.0, 1000000.0]))
    case["hq"] = case["hkv"] * rng.choice([1, 2, 4, 4, 5, 6, 8])
    if kind in ("prefill", "train"):
        case["dtype"] = rng.choice(["bf16", "bf16", "bf16", "f32"]) if kind == "prefill" else "bf16"
        case["dag"] = rng.choice(["fork", "random"])
        case["batch"] = _log_int(rng, 1, 8)
        if case["dag"] == "fork":
            case.update(prefix=_log_int(rng, 64, 32768), branches=_log_int(rng, 2, 32), branch=_log_int(rng, 32, 512),
                        join=_log_int(rng, 32, 1024), jitter=rng.choice([0, 7, 30]))
        else:
            case.update(depth=rng.randint(3, 6), len_lo=_log_int(rng, 8, 40), len_hi=_log_int(rng, 64, 400))
            case["nodes"] = rng.randint(2 * case["depth"], 100)
    elif kind == "decode":
        case.update(groups=_log_int(rng, 1, 16), branches=_log_int(rng, 1, 32), shared=_log_int(rng, 100, 32768),
                    own=_log_int(rng, 40, 1500), jitter=rng.choice([0, 13, 39]))
    elif kind == "frontier":
        case.update(groups=_log_int(rng, 1, 16), mids=rng.randint(1, 4), leaves=rng.randint(1, 6), root=_log_int(rng, 64, 8192),
                    mid=_log_int(rng, 40, 3000), own=_log_int(rng, 40, 1500), jitter=rng.choice([0, 13, 39]))
        case["reads"] = rng.randint(1, case["mids"])
    else:
        case.update(groups=_log_int(rng, 1, 16), nodes=_log_int(rng, 1, 12), shared=_log_int(rng, 100, 12000),
                    own=_log_int(rng, 16, 1500), new=_log_int(rng, 20, 700), jitter=rng.choice([0, 11]))
    return case


# --------------------------------------------------------------------------- DAGs and contexts
def _dags(case):
    """[(node lengths, parents of every node)] of the batch."""
    rng = random.Random(case["dag_seed"])
    out = []
    for _ in range(case["batch"]):
        if case["dag"] == "fork":
            vary = lambda n: n + rng.randint(-case["jitter"], case["jitter"])  # noqa: E731
            lens = [vary(case["prefix"])] + [vary(case["branch"]) for _ in range(case["branches"])] + [vary(case["join"])]
            parents = [[]] + [[0]] * case["branches"] + [list(range(1, case["branches"] + 1))]
        else:
            n, depth = case["nodes"], case["depth"]
            cuts = [0, 1] + sorted(rng.sample(range(2, n), depth - 2)) + [n]  # first node of every level
            parents = [[]]
            for lv in range(1, depth):
                before = range(cuts[lv - 1], cuts[lv])
                for _ in range(cuts[lv], cuts[lv + 1]):
                    joins = rng.randint(2, 3) if lv >= 2 and rng.random() < 0.3 else 1
                    parents.append(rng.sample(before, min(joins, len(before))))
            lens = [rng.randint(case["len_lo"], case["len_hi"]) for _ in range(n)]
        out.append((lens, parents))
    return out


def _ancestors(parents):
    anc = []
    for ps in parents:
        anc.append(set(ps).union(*[anc[p] for p in ps]))
    return anc


def _pairs(case):
    """(tokens, visible query-key pairs) of the batch."""
    tokens = pairs = 0
    for lens, parents in _dags(case):
        for n, anc in zip(lens, _ancestors(parents)):
            tokens += n
            pairs += n * sum(lens[u] for u in anc) + n * (n + 1) // 2
    return tokens, pairs


def _lengths(case):
    """Context lengths of the paged kinds, one entry for each live branch / node: (tokens in its own
    pages, how many of them are new); and [(tokens, readers)] of every shared stretch of context."""
    rng = random.Random(case["dag_seed"])
    vary = lambda n: n + rng.randint(-case["jitter"], case["jitter"])  # noqa: E731
    live, shared = [], []
    for g in range(case["groups"]):
        if case["kind"] == "frontier":
            first = len(live)
            live += [(vary(case["own"]), 1) for _ in range(case["mids"] * case["leaves"])]
            shared.append((vary(case["root"]), list(range(first, len(live)))))
            for m in range(case["mids"]):
                shared.append((vary(case["mid"]), [r for r in range(first, len(live))
                                                   if (m - (r - first) // case["leaves"]) % case["mids"] < case["reads"]]))
        else:
            n = case["branches"] if case["kind"] == "decode" else case["nodes"]
            shared.append((case["shared"], list(range(len(live), len(live) + n))))
            new = case["new"] if case["kind"] == "paged" else 0
            for _ in range(n):
                mine = max(1, vary(new)) if new else 1
                live.append((mine + vary(case["own"]), mine) if new else (vary(case["own"]), 1))
    return live, shared


def _pool_tokens(case):
    if case["kind"] in ("prefill", "train"):
        return 0
    live, shared = _lengths(case)
    return sum(n for n, _ in live) + sum(n for n, _ in shared)


def work(case):
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    if case["kind"] in ("prefill", "train"):
        tokens, pairs = _pairs(case)
        size = DTYPES[case["dtype"]].itemsize
        flops = 4 * d * hq * pairs
        if case["kind"] == "prefill":  # q, k read and rotated in place, v read, out written
            return {"bytes": tokens * d * size * (3 * hq + 3 * hkv), "flops": flops}
        # q, k, v, dout read; out, dq, dk, dv and the log-sum-exp written; five products backward
        return {"bytes": tokens * (d * size * (4 * hq + 4 * hkv) + 4 * hq), "flops": 3.5 * flops}
    live, shared = _lengths(case)
    rows = sum(new for _, new in live)
    pairs = sum(n * sum(live[r][1] for r in readers) for n, readers in shared)
    pairs += sum(new * (n - new) + new * (new + 1) // 2 for n, new in live)
    # K/V of every cached stretch once, the new K/V read and stored, q read, out written
    return {"bytes": 2 * d * (2 * hkv * _pool_tokens(case) + 4 * hkv * rows + 2 * hq * rows), "flops": 4 * d * hq * pairs}


def tolerance(case):
    """About four times what the same path in 64 bits differs by (largest seen over listed and drawn
    shapes: rel 2.4e-7 in 32 bits; in bf16 rel 3.3e-3, and of single elements 0.09 of the result's
    root mean square in packed prefill, 0.02 in the paged kinds and 0.7 in dQ, whose elements differ
    by orders of magnitude between rows)."""
    if case.get("dtype") == "f32":
        return {"rel": 3e-6, "max": 1e-4}
    return {"rel": 1.2e-2, "max": {"prefill": 0.36, "train": 0.9}.get(case["kind"], 0.08)}


# --------------------------------------------------------------------------- states
def _normal(gen, shape, scale, dtype):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, scale, generator=gen)


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if case["kind"] in ("prefill", "train"):
        return _prepare_packed(case, gen)
    return _prepare_paged(case, gen, np.random.default_rng(seed))


def _prepare_packed(case, gen):
    hq, hkv, d, dtype = case["hq"], case["hkv"], case["d"], DTYPES[case["dtype"]]
    dags = _dags(case)
    words = max(-(-len(lens) // 64) for lens, _ in dags)
    lens = [n for ls, _ in dags for n in ls]
    bits = np.zeros((len(lens), words), dtype=np.uint64)
    v = 0
    for _, parents in dags:
        for anc in _ancestors(parents):
            for u in anc:
                bits[v, u >> 6] |= np.uint64(1 << (u & 63))
            v += 1
    offsets = np.cumsum([0] + [len(ls) for ls, _ in dags])
    code = B.DAG_F32 if dtype == torch.float32 else B.DAG_BF16
    desc = B.DagDesc(offsets, lens, bits, words, *B.dag_prefill_tile_shape(hq, hkv, d, code))
    meta = B.DagMeta(desc, B.dag_meta_sizes(desc), "cuda")
    tokens = int(sum(lens))
    s = dict(case=case, desc=desc, meta=meta)
    for name, heads in (("q", hq), ("k", hkv), ("v", hkv)):
        s[name] = _normal(gen, (tokens, heads, d), 0.5 if dtype == torch.bfloat16 else 1.0, dtype)
    s["out"] = torch.empty_like(s["q"])
    s["ws"] = torch.empty(max(256, B.dag_prefill_workspace_bytes(meta, hkv, d, code)), dtype=torch.uint8, device="cuda")
    if case["kind"] == "train":
        B.dag_build_meta(desc, meta)
        s["dout"] = _normal(gen, (tokens, hq, d), 0.5, dtype)
        s["lse"] = torch.empty((tokens, hq), dtype=torch.float32, device="cuda")
        s["dq"], s["dk"], s["dv"] = torch.empty_like(s["q"]), torch.empty_like(s["k"]), torch.empty_like(s["v"])
        s["bws"] = torch.empty(B.dag_prefill_bwd_workspace_bytes(meta, hq, hkv, d), dtype=torch.uint8, device="cuda")
    return s


def _prepare_paged(case, gen, rng):
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    live, shared = _lengths(case)
    stretches = [n for n, _ in shared] + [n for n, _ in live]
    counts = [-(-n // PAGE) for n in stretches]
    n_pages = sum(counts)
    perm = rng.permutation(n_pages).astype(np.int32)
    ends = np.cumsum([0] + counts)
    pages = [perm[ends[i]:ends[i + 1]] for i in range(len(stretches))]
    own = pages[len(shared):]
    rows = sum(new for _, new in live)
    s = dict(case=case,
             k_pool=_normal(gen, (n_pages, hkv, d // 8, PAGE, 8), 1.0, torch.bfloat16),
             v_pool=_normal(gen, (n_pages, hkv, d, PAGE), 1.0, torch.bfloat16),
             q=_normal(gen, (rows, hq, d), 1.0, torch.bfloat16),
             k_new=_normal(gen, (rows, hkv, d), 1.0, torch.bfloat16),
             v_new=_normal(gen, (rows, hkv, d), 1.0, torch.bfloat16))
    s["out"] = torch.empty_like(s["q"])
    before = [sum(n for n, readers in shared if r in readers) for r in range(len(live))]
    none = np.zeros(1, dtype=np.int32)
    if case["kind"] == "decode":
        branches = case["branches"]
        s["desc"] = B.DecodeDesc(dict(
            n_groups=case["groups"], n_live=rows, page_size=PAGE,
            group_branch_off=np.arange(0, rows + 1, branches), shared_page_off=ends[:len(shared) + 1],
            shared_pages=perm[:ends[len(shared)]], shared_len=[n for n, _ in shared],
            branch_page_off=ends[len(shared):] - ends[len(shared)], branch_pages=perm[ends[len(shared)]:],
            branch_len=[n for n, _ in live], branch_pos=[b + n - 1 for b, (n, _) in zip(before, live)]), "cuda")
        s["append"] = s["desc"]
        need = B.dag_decode_workspace_bytes(s["desc"], hq, hkv, d)
    else:
        # every new token is an entry of its own: the page it goes to and its place there
        place = [(own[r], n - new + i, before[r]) for r, (n, new) in enumerate(live) for i in range(new)]
        s["append"] = B.DecodeDesc(dict(
            n_groups=0, n_live=rows, page_size=PAGE, group_branch_off=none, shared_page_off=none, shared_pages=none,
            shared_len=none, branch_page_off=np.arange(rows + 1), branch_pages=[p[t // PAGE] for p, t, _ in place],
            branch_len=[t % PAGE + 1 for _, t, _ in place], branch_pos=[b + t for _, t, b in place]), "cuda")
    if case["kind"] == "frontier":
        readers = [r for _, r in shared] + [[r] for r in range(len(live))]
        entries = [[] for _ in live]
        for e, r in enumerate(r for seg in readers for r in seg):
            entries[r].append(e)
        s["desc"] = B.SegDecodeDesc(dict(
            n_live=rows, n_segments=len(stretches), page_size=PAGE, seg_page_off=ends, seg_pages=perm, seg_len=stretches,
            seg_reader_off=np.cumsum([0] + [len(r) for r in readers]), seg_readers=[r for seg in readers for r in seg],
            branch_entry_off=np.cumsum([0] + [len(e) for e in entries]), branch_entries=[e for b in entries for e in b]), "cuda")
        need = B.dag_decode_segments_workspace_bytes(s["desc"], hq, hkv, d)
    elif case["kind"] == "paged":
        ctx = [[i for i, (_, readers) in enumerate(shared) if r in readers] + [len(shared) + r] for r in range(len(live))]
        s["desc"] = B.PagedPrefillDesc(dict(
            page_size=PAGE, q_off=np.cumsum([0] + [new for _, new in live]),
            ctx_page_off=np.cumsum([0] + [sum(counts[i] for i in c) for c in ctx]),
            ctx_pages=np.concatenate([pages[i] for c in ctx for i in c]),
            ctx_page_len=[min(PAGE, stretches[i] - PAGE * j) for c in ctx for i in c for j in range(counts[i])],
            own_page=[sum(counts[i] for i in c[:-1]) for c in ctx], own_len=[n for n, _ in live]), "cuda")
        need = B.dag_prefill_paged_workspace_bytes(s["desc"])
    s["ws"] = torch.empty(max(256, need), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "prefill":
        B.dag_build_meta(s["desc"], s["meta"])
        B.dag_rope_qk(s["meta"].t["pos_ids"], s["q"], s["k"], case["theta"])
        B.dag_attn_prefill(s["meta"], s["q"], s["k"], s["v"], s["out"], workspace=s["ws"])
        return {"q": s["q"], "k": s["k"], "out": s["out"]}
    if kind == "train":
        B.dag_attn_prefill(s["meta"], s["q"], s["k"], s["v"], s["out"], lse=s["lse"], workspace=s["ws"])
        B.dag_attn_prefill_bwd(s["meta"], s["q"], s["k"], s["v"], s["out"], s["dout"], s["lse"], s["dq"], s["dk"], s["dv"],
                               workspace=s["bws"])
        return {n: s[n] for n in ("out", "lse", "dq", "dk", "dv")}
    B.dag_kv_append_rope(s["append"], s["k_new"], s["v_new"], s["k_pool"], s["v_pool"], case["theta"])
    attend = {"decode": B.dag_attn_decode, "frontier": B.dag_attn_decode_segments, "paged": B.dag_attn_prefill_paged}[kind]
    attend(s["desc"], s["q"], s["k_pool"], s["v_pool"], s["out"], s["ws"])
    return {"out": s["out"], "k_pool": s["k_pool"], "v_pool": s["v_pool"]}
