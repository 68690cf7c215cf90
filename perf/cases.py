"""The work that a user of this library has it do, as measurable cases.

A case is one pass through the public entry points: a whole verification step (tree attention of
every layer, per-node arg-max, acceptance, compaction of the cache), the sampling form of the
acceptance, the draft's tree growth, the fused output head, or the visual token compressors.
Sizes are those of the five workload configurations and of the compressors' and the head's own
measurements, or generic ones between them; all inputs are synthetic and made on the GPU.
"""
import math

import numpy as np
import torch

import paper_2509_11815_amd as sv

DEV = "cuda:0"
TYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
TOPK = 10                     # children per expanded node, nodes expanded per level


def listed():
    return [
        # the smallest call: one fp32 layer, a tree of 8 nodes, the four calls of a step on their own
        {"name": "fp32_small", "kind": "step", "dtype": "f32", "layers": 1, "q_heads": 4, "kv_heads": 4, "head_dim": 64,
         "nodes": 8, "depth": 3, "prefix": "64", "vocab": 1000, "paged": False, "replay": False},
        # 7B-shaped target, one image of 576 visual tokens, early in an answer; calls made eagerly from Python
        {"name": "step_576_visual", "kind": "step", "dtype": "bf16", "layers": 32, "q_heads": 32, "kv_heads": 32, "head_dim": 128,
         "nodes": 60, "depth": 6, "prefix": "768", "vocab": 32000, "paged": False, "replay": False},
        # 7B-shaped target, 2880 visual tokens, the step captured once as a HIP graph and replayed every round
        {"name": "step_2880_visual", "kind": "step", "dtype": "bf16", "layers": 32, "q_heads": 32, "kv_heads": 32, "head_dim": 128,
         "nodes": 60, "depth": 6, "prefix": "3264", "vocab": 32000, "paged": False, "replay": True},
        # eight requests whose visual prefixes were compressed differently: one cache, very different lengths
        {"name": "step_ragged_batch", "kind": "step", "dtype": "bf16", "layers": 32, "q_heads": 32, "kv_heads": 32, "head_dim": 128,
         "nodes": 60, "depth": 6, "prefix": "170,390,253,339,350,906,365,287", "vocab": 32000, "paged": False, "replay": True},
        # 13B-shaped target, four requests of 8 frames each in a paged cache (8 of the layers)
        {"name": "step_paged_batch", "kind": "step", "dtype": "bf16", "layers": 8, "q_heads": 40, "kv_heads": 40, "head_dim": 128,
         "nodes": 60, "depth": 7, "prefix": "4864,4864,4864,4864", "vocab": 32000, "paged": True, "replay": False},
        # a target whose query heads share KV heads, with a large vocabulary, four requests (8 of the layers)
        {"name": "step_grouped_heads", "kind": "step", "dtype": "bf16", "layers": 8, "q_heads": 32, "kv_heads": 8, "head_dim": 128,
         "nodes": 64, "depth": 7, "prefix": "2048,1311,3000,777", "vocab": 152064, "paged": False, "replay": False},
        # temperature 1: the sampling form of the acceptance for four requests
        {"name": "accept_sampled", "kind": "sample", "dtype": "bf16", "batch": 4, "nodes": 60, "depth": 7, "vocab": 32000,
         "temperature": 1.0},
        # the draft's side of a round: six levels of Top-K, then the tree
        {"name": "grow_tree", "kind": "grow", "dtype": "bf16", "batch": 1, "nodes": 60, "depth": 6, "vocab": 32000},
        # output head and greedy choice in one call: one request, 7B-shaped; eight requests, 13B-shaped
        {"name": "head_one_request", "kind": "head", "batch": 1, "nodes": 60, "hidden": 4096, "vocab": 32000},
        {"name": "head_eight_requests", "kind": "head", "batch": 8, "nodes": 60, "hidden": 5120, "vocab": 32000},
        # the draft's compressed visual prefix, once per request: one small image; a batch of large ones
        {"name": "compress_one_image", "kind": "compress", "dtype": "bf16", "batch": 1, "tokens": 576, "features": 4096, "ratio": 4,
         "ragged": False},
        {"name": "compress_batch", "kind": "compress", "dtype": "bf16", "batch": 8, "tokens": 2880, "features": 4096, "ratio": 20,
         "ragged": False},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "step", "sample", "grow", "head", "head", "compress"])
    if kind == "step":
        dtype = "f32" if rng.random() < 0.1 else "bf16"
        kv_heads = rng.choice([4, 8, 16, 32, 40])
        group = rng.choice([g for g in (1, 1, 1, 2, 4, 8) if kv_heads * g <= 40])
        head_dim = rng.choice([64, 128, 128])
        batch = _log_int(rng, 1, 8)
        nodes = rng.choice([60, 64, rng.randint(8, 64)])
        # the requests of a batch are of one length or of very different ones
        longest = _log_int(rng, 64, 5000)
        spread = rng.random() < 0.5
        prefix = [_log_int(rng, min(64, longest), longest) if spread else longest for _ in range(batch)]
        layers = rng.choice([4, 8, 16, 32])
        if dtype == "f32":                               # the small checking path, not a serving one
            layers, kv_heads, group = 1, min(kv_heads, 8), 1
            prefix = [min(p, 512) for p in prefix]
        keys = sum(p + nodes for p in prefix)
        while layers > 1 and layers * keys * kv_heads * head_dim * 4 > 2.0e9:
            layers //= 2
        while layers > 1 and layers * keys * kv_heads * group * head_dim > 6.0e8:
            layers //= 2
        return {"kind": kind, "dtype": dtype, "layers": layers, "q_heads": kv_heads * group, "kv_heads": kv_heads,
                "head_dim": head_dim, "nodes": nodes, "depth": rng.randint(3, 7), "prefix": ",".join(str(p) for p in prefix),
                "vocab": _log_int(rng, 1000, 152064) if batch <= 4 else _log_int(rng, 1000, 50000),
                "paged": rng.random() < 0.35, "replay": rng.random() < 0.5}
    if kind == "sample":
        return {"kind": kind, "dtype": rng.choice(["bf16", "bf16", "f32"]), "batch": _log_int(rng, 1, 16),
                "nodes": rng.randint(16, 64), "depth": rng.randint(3, 7), "vocab": _log_int(rng, 4000, 152064),
                "temperature": round(rng.uniform(0.5, 1.5), 2)}
    if kind == "grow":
        return {"kind": kind, "dtype": rng.choice(["bf16", "bf16", "f32"]), "batch": _log_int(rng, 1, 8),
                "nodes": rng.randint(16, 64), "depth": rng.randint(3, 7), "vocab": _log_int(rng, 4000, 152064)}
    if kind == "head":
        hidden = rng.choice([2048, 3584, 4096, 5120])
        batch = _log_int(rng, 1, 8)
        most = min(152064, int(1.3e9 // (hidden * batch)))
        return {"kind": kind, "batch": batch, "nodes": rng.choice([60, rng.randint(8, 64)]), "hidden": hidden,
                "vocab": _log_int(rng, 8000, most)}
    return {"kind": kind, "dtype": rng.choice(["bf16", "bf16", "f32"]), "batch": _log_int(rng, 1, 8),
            "tokens": _log_int(rng, 64, 4608), "features": rng.choice([1024, 4096, 5120]), "ratio": _log_int(rng, 2, 30),
            "ragged": rng.random() < 0.3}


# ---- inputs ------------------------------------------------------------------------------------------
def _tree(rng, nodes, depth):
    """Parents of a draft tree in level order: one chain down to `depth` and likely nodes around it, as
    the best candidates of level-by-level Top-K growth."""
    chain = min(depth, nodes - 1)
    par, dep, weight, kids = [-1], [0], [1.0], [0]
    for d in range(chain):
        par.append(len(par) - 1)
        dep.append(d + 1)
        weight.append(weight[-1] * 0.6)
        kids[-1] += 1
        kids.append(0)
    while len(par) < nodes:
        w = np.array([weight[i] / (1 + kids[i]) if dep[i] < depth and kids[i] < TOPK else 0.0 for i in range(len(par))])
        p = int(rng.choice(len(par), p=w / w.sum()))
        par.append(p)
        dep.append(dep[p] + 1)
        weight.append(weight[p] * 0.5 / (1 + kids[p]))
        kids[p] += 1
        kids.append(0)
    order = sorted(range(nodes), key=lambda i: (dep[i], i))
    place = {old: new for new, old in enumerate(order)}
    return [-1 if par[i] < 0 else place[par[i]] for i in order]


def _trees(rng, gen, batch, nodes, depth, vocab, dtype):
    """Trees, target logits ~ N(0, 2) and draft tokens: siblings differ, and with probability 0.75 the
    first child of a node carries the target's own token."""
    parent = np.array([_tree(rng, nodes, depth) for _ in range(batch)], dtype=np.int32)
    logits = torch.empty((batch, nodes, vocab), dtype=dtype, device=DEV).normal_(0.0, 2.0, generator=gen)
    top = logits.float().argmax(dim=2).cpu().numpy()
    tok = np.zeros((batch, nodes), dtype=np.int32)
    for b in range(batch):
        tok[b] = rng.choice(vocab, size=nodes, replace=False)
        seen = set()
        for i in range(1, nodes):
            p = int(parent[b, i])
            if p not in seen:
                seen.add(p)
                if rng.random() < 0.75:
                    tok[b, i] = top[b, p]
    return torch.from_numpy(parent).to(DEV), torch.from_numpy(tok).to(DEV), logits


def _i32(*shape):
    return torch.zeros(shape, dtype=torch.int32, device=DEV)


def _accept_outputs(batch, cap):
    return _i32(batch), _i32(batch, cap), _i32(batch), _i32(batch, cap)


def _lengths(case):
    return [int(x) for x in case["prefix"].split(",")]


def _prepare_step(case, rng, gen):
    dtype, L, N, D = TYPES[case["dtype"]], case["layers"], case["nodes"], case["head_dim"]
    P = _lengths(case)
    B, longest = len(P), max(P) + N
    s = {"case": case, "P": torch.tensor(P, dtype=torch.int32, device=DEV)}
    if case["paged"]:
        per = (longest + 15) // 16
        pool = B * per + max(1, B * per // 10)
        table = rng.permutation(pool)[: B * per].reshape(B, per).astype(np.int32)
        s["table"] = torch.from_numpy(table).to(DEV)
        shape = (L, pool, case["kv_heads"], 16, D)
    else:
        s["table"] = None
        shape = (L, B, case["kv_heads"], (longest + 15) // 16 * 16, D)
    s["k"], s["v"] = (torch.empty(shape, dtype=dtype, device=DEV).normal_(generator=gen) for _ in range(2))
    s["q"] = torch.empty((L, B, N, case["q_heads"], D), dtype=dtype, device=DEV).normal_(generator=gen)
    s["o"] = torch.zeros_like(s["q"])
    s["parent"], s["tok"], s["logits"] = _trees(rng, gen, B, N, case["depth"], case["vocab"], dtype)
    cap = case["depth"] + 1
    s["desc"] = sv.binding.make_attn_desc(s["q"][0], s["k"][0], s["o"][0], block_table=s["table"])
    need = sv.specvlm_tree_verify_attn_workspace_bytes(s["desc"])
    s["ws"] = torch.zeros(max(need, 256), dtype=torch.uint8, device=DEV)
    s["counters"], s["amax"], s["err"], s["new_P"] = _i32(B * sv.binding.COUNTER_STRIDE), _i32(B, N), _i32(1), _i32(B)
    s["out"] = _accept_outputs(B, cap)
    # a program keeps views of its layers, not the stacked tensor alone
    s["layers"] = [tuple(s[x][i] for x in ("q", "k", "v", "o")) for i in range(L)]
    s["graph"] = None
    if case["replay"]:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _step(s)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            _step(s)
    return s


def _step(s):
    for q, k, v, o in s["layers"]:
        sv.specvlm_tree_verify_attn(q, k, v, s["P"], s["parent"], block_table=s["table"], out=o, workspace=s["ws"],
                                    err_flag=s["err"], desc=s["desc"])
    if s["case"]["dtype"] == "f32":
        sv.specvlm_node_argmax(s["logits"], out=s["amax"])
        sv.specvlm_tree_accept(s["parent"], s["tok"], s["amax"], err_flag=s["err"], out=s["out"])
    else:
        sv.specvlm_node_argmax_accept(s["logits"], s["parent"], s["tok"], counters=s["counters"], amax=s["amax"],
                                      err_flag=s["err"], out=s["out"])
    # the prefix lengths are not advanced, so that every pass is the same step
    sv.specvlm_kv_compact(s["k"], s["v"], s["P"], s["out"][1], s["out"][0], block_table=s["table"],
                          new_prefix_len=s["new_P"], err_flag=s["err"])


def _run_step(s):
    if s["graph"] is not None:
        s["graph"].replay()
    else:
        _step(s)
    return {"o": s["o"], "amax": s["amax"], "accept": s["out"], "new_P": s["new_P"], "k": s["k"], "v": s["v"], "err": s["err"]}


def _prepare_sample(case, rng, gen):
    B, N = case["batch"], case["nodes"]
    parent, tok, logits = _trees(rng, gen, B, N, case["depth"], case["vocab"], TYPES[case["dtype"]])
    return {"case": case, "parent": parent, "tok": tok, "logits": logits, "err": _i32(1),
            "u_accept": torch.rand((B, N), device=DEV, generator=gen), "u_bonus": torch.rand(B, device=DEV, generator=gen)}


def _run_sample(s):
    got = sv.specvlm_tree_accept_sample(s["parent"], s["tok"], s["logits"], s["u_accept"], s["u_bonus"],
                                        temperature=s["case"]["temperature"], path_cap=s["case"]["depth"] + 1,
                                        err_flag=s["err"])
    return {"accept": got, "err": s["err"]}


def _prepare_grow(case, rng, gen):
    B, V, depth = case["batch"], case["vocab"], case["depth"]
    rows = [1 if d == 0 else TOPK for d in range(depth)]
    C = sum(r * TOPK for r in rows)
    s = {"case": case, "rows": rows, "root": torch.randint(0, V, (B,), dtype=torch.int32, device=DEV, generator=gen),
         "logits": [torch.empty((B, r, V), dtype=TYPES[case["dtype"]], device=DEV).normal_(0.0, 2.0, generator=gen) for r in rows],
         "score": torch.zeros((B, C), dtype=torch.float32, device=DEV), "token": _i32(B, C), "par": _i32(B, C) - 1,
         "sel": [(_i32(B, TOPK), torch.zeros((B, TOPK), dtype=torch.float32, device=DEV), _i32(B)) for _ in range(depth)],
         "counters": _i32(B * sv.binding.COUNTER_STRIDE), "err": _i32(1),
         "out": (_i32(B, case["nodes"]), _i32(B, case["nodes"]), _i32(B, case["nodes"]), _i32(B))}
    return s


def _run_grow(s):
    base = 0
    for d, rows in enumerate(s["rows"]):
        end = base + rows * TOPK
        to = {"score_out": s["score"][:, base:end], "token_out": s["token"][:, base:end], "parent_out": s["par"][:, base:end]}
        if d:
            to.update(cum=s["sel"][d][1], parent_idx=s["sel"][d][0])
        if d + 1 < len(s["rows"]):
            nxt = s["sel"][d + 1]
            sv.specvlm_draft_topk_select(s["logits"][d], TOPK, TOPK, index_base=base, sel_out=nxt[0], sel_score_out=nxt[1],
                                         count_out=nxt[2], counters=s["counters"], **to)
        else:
            sv.specvlm_draft_topk(s["logits"][d], TOPK, **to)
        base = end
    sv.specvlm_draft_finalize(s["score"], s["par"], s["token"], s["root"], s["case"]["nodes"], err_flag=s["err"], out=s["out"])
    return {"score": s["score"], "token": s["token"], "par": s["par"], "tree": s["out"], "err": s["err"]}


def _prepare_head(case, rng, gen):
    B, N, E, V = case["batch"], case["nodes"], case["hidden"], case["vocab"]
    return {"hidden": torch.empty((B, N, E), dtype=torch.bfloat16, device=DEV).normal_(generator=gen),
            "weight": torch.empty((V, E), dtype=torch.bfloat16, device=DEV).normal_(0.0, 2.0 / E ** 0.5, generator=gen),
            "ws": torch.zeros(sv.specvlm_head_argmax_workspace_bytes(B, N, V), dtype=torch.uint8, device=DEV),
            "out": _i32(B, N), "logit": torch.zeros((B, N), dtype=torch.float32, device=DEV)}


def _run_head(s):
    sv.specvlm_head_argmax(s["hidden"], s["weight"], out=s["out"], max_logit=s["logit"], workspace=s["ws"])
    return {"token": s["out"], "logit": s["logit"]}


def _kept(case):
    return -(-case["tokens"] // case["ratio"])


def _token_counts(case):
    """How many of `tokens` each request has."""
    T, B = case["tokens"], case["batch"]
    return [max(1, T - b * T // (B + 1)) for b in range(B)] if case["ragged"] else [T] * B


def _prepare_compress(case, rng, gen):
    B, T, E = case["batch"], case["tokens"], case["features"]
    keep = np.full((B, _kept(case)), -1, dtype=np.int32)
    for b, n in enumerate(_token_counts(case)):
        m = -(-n // case["ratio"])
        keep[b, :m] = np.sort(rng.choice(n, size=m, replace=False))
    return {"case": case, "x": torch.empty((B, T, E), dtype=TYPES[case["dtype"]], device=DEV).normal_(generator=gen),
            "keep": torch.from_numpy(keep).to(DEV), "err": _i32(1),
            "count": torch.tensor(_token_counts(case), dtype=torch.int32, device=DEV) if case["ragged"] else None}


def _run_compress(s):
    pooled, n = sv.specvlm_visual_pool(s["x"], s["case"]["ratio"], num_tokens=s["count"], err_flag=s["err"])
    pruned = sv.specvlm_visual_prune(s["x"], s["keep"], err_flag=s["err"])
    return {"pooled": pooled, "n": n, "pruned": pruned, "err": s["err"]}


_PREPARE = {"step": _prepare_step, "sample": _prepare_sample, "grow": _prepare_grow, "head": _prepare_head,
            "compress": _prepare_compress}
_RUN = {"step": _run_step, "sample": _run_sample, "grow": _run_grow, "head": _run_head, "compress": _run_compress}


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    return {"run": _RUN[case["kind"]], "state": _PREPARE[case["kind"]](case, np.random.default_rng(seed), gen)}


def run(state):
    return state["run"](state["state"])


# ---- what a pass cannot do without -------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    esize = 4 if case.get("dtype") == "f32" else 2
    if kind == "step":
        # K and V of every layer once, queries and outputs once, the logits once (the compaction moves a few rows)
        P, N, L, D, Hq = _lengths(case), case["nodes"], case["layers"], case["head_dim"], case["q_heads"]
        kv = L * sum(p + N for p in P) * case["kv_heads"] * D * 2 * esize
        qo = 2 * L * len(P) * N * Hq * D * esize
        return {"bytes": kv + qo + len(P) * N * case["vocab"] * esize, "flops": 4 * L * Hq * D * N * sum(P)}
    if kind == "sample":
        # the rows the walk visits depend on the draws: the root's row and the bonus token's at least
        return {"bytes": case["batch"] * 2 * case["vocab"] * esize, "flops": 6 * case["batch"] * case["vocab"]}
    if kind == "grow":
        rows = 1 + (case["depth"] - 1) * TOPK
        n = case["batch"] * rows * case["vocab"]
        return {"bytes": n * esize + case["batch"] * rows * TOPK * 12, "flops": 3 * n}
    if kind == "head":
        M = case["batch"] * case["nodes"]
        return {"bytes": (case["vocab"] + M) * case["hidden"] * 2 + M * 8, "flops": 2 * M * case["hidden"] * case["vocab"]}
    # every token's features are read once for the pooling; the pruned rows are read among them and written
    rows = sum(_token_counts(case))
    return {"bytes": (rows + 2 * case["batch"] * _kept(case)) * case["features"] * esize, "flops": rows * case["features"]}


def tolerance(case):
    if case["kind"] == "sample":
        return "exact"                                   # tokens and node numbers
    if case["kind"] == "head":
        return {"rel": 1e-5, "differ": 0.005}            # fp32 sums; two logits of a row closer than their rounding
    if case["kind"] == "grow":
        return {"rel": 1e-5, "max": 1e-4}                # fp32 log-sum-exp
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 1e-5}
