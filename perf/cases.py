"""Cases for measuring the verify path the way a serving loop calls it.

Every case prepares device-resident inputs, outputs and workspace once (as a
serving program keeps them) and runs one pass through the public functions of
``paper_2606_04446_amd.d2sd``. The kinds:

  step     tree_build -> cascade_verify_attention -> accept_path: one greedy
           verify step of a canonical tree, host node offsets known
  general  tree_from_parents -> cascade_verify_attention -> accept_path: the
           same step on third-level cascade trees (parent arrays)
  attn     cascade_verify_attention alone: what every further layer of the
           target pass runs after the tree of the step is built
  draw     sample_targets -> accept_path: verification from logits, a draw per
           node (T > 0) or the argmax (T = 0)
  plan     select_reanchor -> tree_indptr -> tree_build: drafter confidences
           to candidate trees with no host round trip
  commit   commit_accepted_kv: accepted path appended to the paged cache

Shapes follow the workloads of ``workload.py`` (block 16, K = 2..8 branches,
32/8 and 64/8 heads of 128, pages of 16, contexts of 512 to 32,768 tokens, 1
to 64 requests), with odd and ragged sizes between them in ``draw``.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2606_04446_amd import d2sd
from paper_2606_04446_amd import workload as wl

DEV = "cuda"
D = 128


def listed():
    return [
        # One interactive request with a short prompt, in the exact-precision build.
        dict(name="step-f32-b1-ctx512", kind="step", dtype="f32", batch=1, lo=512, hi=512, hq=32, hkv=8, B=16, K=2, host=True),
        # One interactive request: the latency of a single verify step.
        dict(name="step-bf16-b1-ctx4096", kind="step", dtype="bf16", batch=1, lo=4096, hi=4096, hq=32, hkv=8, B=16, K=4, host=True),
        # A small server: eight requests at different points of their generations.
        dict(name="step-bf16-b8-ctx1k-8k", kind="step", dtype="bf16", batch=8, lo=1024, hi=8192, hq=32, hkv=8, B=16, K=4, host=True),
        # One request over a long document.
        dict(name="attn-bf16-b1-ctx32k", kind="attn", dtype="bf16", batch=1, lo=32768, hi=32768, hq=32, hkv=8, B=16, K=4, host=True),
        # A layer of a loaded server at 16k contexts.
        dict(name="attn-bf16-b32-ctx16k", kind="attn", dtype="bf16", batch=32, lo=16384, hi=16384, hq=32, hkv=8, B=16, K=8, host=True),
        # The largest: a layer of a full batch at 32k contexts, 64 query heads.
        dict(name="attn-bf16-b64-ctx32k-hq64", kind="attn", dtype="bf16", batch=64, lo=32768, hi=32768, hq=64, hkv=8, B=16, K=8, host=True),
        # Ragged contexts and third-level trees, node offsets known to the device only.
        dict(name="general-bf16-b16-ctx0-8k", kind="general", dtype="bf16", batch=16, lo=37, hi=8191, hq=32, hkv=8, B=16, K=4, host=False),
        # Exact-precision attention on a ragged batch.
        dict(name="attn-f32-b4-ctx300-3k", kind="attn", dtype="f32", batch=4, lo=300, hi=3001, hq=32, hkv=8, B=16, K=4, host=True),
        # Sampling verification of a full batch at T = 1.
        dict(name="draw-bf16-b64-T1", kind="draw", dtype="bf16", batch=64, B=16, K=8, vocab=32000, T=1.0),
        # Greedy verification straight from float32 logits, a small batch.
        dict(name="draw-f32-b8-T0", kind="draw", dtype="f32", batch=8, B=16, K=4, vocab=32000, T=0.0),
        # Candidate trees from drafter confidences, a full batch.
        dict(name="plan-b64", kind="plan", batch=64, B=16, K=8),
        # The accepted paths of a batch into the cache.
        dict(name="commit-bf16-b32-ctx2k", kind="commit", dtype="bf16", batch=32, lo=2048, hi=2048, hq=32, hkv=8, B=16, K=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _attn_flops(c):
    return 4.0 * D * c["hq"] * c["batch"] * _mean_nodes(c) * (c["lo"] + c["hi"]) / 2


def draw(rng):
    kind = rng.choice(["step", "step", "attn", "attn", "general", "draw", "draw", "plan", "commit"])
    B = rng.choice([8, 16, 16, 16, 24, 32])
    K = rng.randint(0, 8) if B > 8 else rng.randint(0, 6)
    if kind == "plan":
        return dict(kind=kind, batch=_log_int(rng, 1, 512), B=B, K=max(K, 1))
    if kind == "draw":
        c = dict(kind=kind, dtype=rng.choice(["bf16", "bf16", "f32"]), batch=_log_int(rng, 1, 64), B=B, K=K,
                 vocab=rng.choice([32000, 32000, _log_int(rng, 1000, 150000), _log_int(rng, 1000, 150000) // 8 * 8]),
                 T=rng.choice([0.0, 0.6, 1.0, 1.0]))
        while c["batch"] > 1 and c["batch"] * _mean_nodes(c) * c["vocab"] > 4e8:
            c["batch"] = c["batch"] // 2
        return c
    hq, hkv = rng.choice([(32, 8), (32, 8), (64, 8), (16, 8), (8, 2), (40, 8)])
    c = dict(kind=kind, dtype="bf16", batch=_log_int(rng, 1, 64), lo=0, hi=0, hq=hq, hkv=hkv, B=B, K=K)
    if kind == "commit":
        # one context length: the commit of a repeated pass then writes the same slots
        c["lo"] = c["hi"] = _log_int(rng, 64, 4096)
        c["dtype"] = rng.choice(["bf16", "bf16", "f32"])
        return c
    c["hi"] = _log_int(rng, 64, 32768)
    c["lo"] = c["hi"] if rng.random() < 0.3 else max(1, int(c["hi"] * rng.uniform(0.05, 1.0)))
    c["host"] = rng.random() < 0.7
    most = 3e12
    if rng.random() < 0.2:
        c["dtype"] = "f32"
        most = 6e10
    while c["batch"] > 1 and _attn_flops(c) > most:
        c["batch"] = c["batch"] // 2
    while _attn_flops(c) > most:
        c["hi"] = c["hi"] // 2
        c["lo"] = min(c["lo"], c["hi"])
    return c


# ---- trees (host side, for the inputs and for the 64-bit results) ----

def _mean_nodes(c):
    n = c["B"] + c["K"] * c["B"] / 2.0
    if c.get("kind") == "general":
        n += c["K"] * c["B"] / 4.0
    return n


def _parents(B, p_row, q_row=None):
    """Parent array of a canonical tree: the block chain, then a branch per
    re-anchor position p (ascending) under chain node p - 1; with q_row, then
    a sub-branch per branch under its node at position q - 1."""
    par = [-1] + list(range(B - 1))
    order = sorted(range(len(p_row)), key=lambda k: p_row[k])
    first = {}
    for k in order:
        first[k] = len(par)
        for pos in range(int(p_row[k]), B):
            par.append(int(p_row[k]) - 1 if pos == p_row[k] else len(par) - 1)
    if q_row is not None:
        for k in order:
            q = int(q_row[k])
            for pos in range(q, B if q > 0 else q):
                par.append(first[k] + q - 1 - int(p_row[k]) if pos == q else len(par) - 1)
    return np.asarray(par, np.int32)


def _visible(par):
    """Ancestor-or-self matrix [N, N] of a parent array."""
    n = len(par)
    vis = np.eye(n, dtype=bool)
    for i in range(n):
        if par[i] >= 0:
            vis[i] |= vis[par[i]]
    return vis


def _layout(case, seed):
    """Layout and parent arrays. The batch's set of trees and context lengths
    belongs to the case, so that every seed asks for the same amount of work;
    which request has which, the pages and all values come from the seed."""
    lo, hi = case.get("lo", 16), case.get("hi", 16)
    spec = wl.Spec("case", case.get("dtype", "bf16"), case["batch"], (lo, hi), case.get("hq", 32), case.get("hkv", 8),
                   B=case["B"], K=case["K"])
    lay = wl.draw_layout(spec, 1)
    q = wl.draw_sub_branch_positions(lay) if case["kind"] == "general" else None
    rng = np.random.default_rng([seed, 7])
    tree_of, ctx_of = rng.permutation(lay.batch), rng.permutation(lay.batch)
    lay.seed, lay.K, lay.p, lay.ctx_len = seed, lay.K[tree_of], lay.p[tree_of], lay.ctx_len[ctx_of]
    lay.page_table, lay.num_pages = wl.pages_for(lay.ctx_len, 16, True, rng)
    par = [_parents(case["B"], lay.p[b, :lay.K[b]], None if q is None else q[tree_of[b], :lay.K[b]])
           for b in range(lay.batch)]
    return lay, par


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


# ---- inputs ----

def prepare(case, seed):
    lay, par = _layout(case, seed)
    B, kind = case["B"], case["kind"]
    s = {"kind": kind, "B": B, "lay": lay, "par": par}
    if kind == "plan":
        s["conf"] = _dev(wl.draw_confidences(lay))
        s["K"] = _dev(lay.K)
        s["kmax"] = case["K"]
        ip, s["W"] = d2sd.tree_plan(B, lay.K, lay.p[:, :case["K"]])
        # Node counts depend on the confidences: room for the largest trees.
        s["total"] = case["batch"] * (B + sum(range(B - case["K"], B)))
        s["p"] = torch.empty((case["batch"], case["K"]), dtype=torch.int32, device=DEV)
        s["ip"] = torch.empty(case["batch"] + 1, dtype=torch.int32, device=DEV)
        s["tree"] = d2sd.tree_build(B, s["K"], _dev(lay.p[:, :case["K"]]), _dev(ip), s["total"], s["W"])
        for t in s["tree"].values():
            t.zero_()
        return s
    nodes = np.asarray([len(x) for x in par])
    ip = np.concatenate([[0], np.cumsum(nodes)]).astype(np.int32)
    s.update(ip_host=ip, total=int(ip[-1]), max_nodes=int(nodes.max()), ip=_dev(ip))
    parents = np.concatenate(par)
    draft, argmax = wl.draw_tokens(lay, ip, parents)
    s["draft"], s["argmax"], s["parent"] = _dev(draft), _dev(argmax), _dev(parents)
    s["tree"] = d2sd.tree_from_parents(s["ip"], s["total"], s["max_nodes"], s["parent"], (s["max_nodes"] + 31) // 32)
    s["tree"]["parent"] = s["parent"]
    if kind == "draw":
        V = case["vocab"]
        s["logits"] = wl.draw_logits(lay, argmax % V, vocab=V, device=DEV, dtype=case["dtype"])
        s["draft"] = _dev((draft % V).astype(np.int32))
        s["T"] = case["T"]
        s["u"] = _dev(wl.draw_uniforms(lay, s["total"])) if case["T"] > 0 else None
        s["tokens"] = torch.empty(s["total"], dtype=torch.int32, device=DEV)
        s["acc"] = _accept(s, s["argmax"], None)
        return s
    if kind == "step":
        s["W"] = d2sd.mask_words(B)
        s["K"], s["p"] = _dev(lay.K), _dev(lay.p)
        s["tree"] = d2sd.tree_build(B, s["K"], s["p"], s["ip"], s["total"], s["W"])
    s["ctx"], s["max_ctx"] = _dev(lay.ctx_len), int(lay.ctx_len.max())
    if kind == "commit":
        s["acc"] = _accept(s, s["argmax"], None)
        # the caller reserves pages up to the context length plus a block
        pages = (s["max_ctx"] + B + 15) // 16
        table = np.random.default_rng([seed, 9]).permutation(case["batch"] * pages).reshape(case["batch"], pages)
        s["pt"] = _dev(table.astype(np.int32))
        shape = (case["batch"] * pages, case["hkv"], 16, D)
        dt = wl.torch_dtype(case["dtype"])
        gen = torch.Generator(device=DEV)
        gen.manual_seed(seed)
        s["k_cache"] = torch.randn(shape, generator=gen, device=DEV).to(dt)
        s["v_cache"] = torch.randn(shape, generator=gen, device=DEV).to(dt)
        s["k_tree"] = torch.randn((s["total"], case["hkv"], D), generator=gen, device=DEV).to(dt)
        s["v_tree"] = torch.randn((s["total"], case["hkv"], D), generator=gen, device=DEV).to(dt)
        return s
    s["x"] = wl.draw_tensors(lay, s["total"], device=DEV)
    s["pt"] = _dev(lay.page_table)
    s["host"] = ip if case["host"] else None
    s["out"] = torch.empty_like(s["x"]["q"])
    s["lse"] = torch.empty(s["x"]["q"].shape[:2], dtype=torch.float32, device=DEV)
    x = s["x"]
    a = d2sd.attn_args(x["q"], x["k_cache"], x["v_cache"], s["pt"], s["ctx"], x["k_tree"], x["v_tree"], s["ip"],
                       s["tree"]["anc_mask"], s["out"], s["lse"], total_nodes=s["total"], max_nodes=s["max_nodes"],
                       max_ctx_len=s["max_ctx"], node_indptr_host=s["host"])
    need = d2sd.cascade_workspace_size(a)
    s["ws"] = torch.empty(need, dtype=torch.uint8, device=DEV) if need > 0 else None
    s["acc"] = _accept(s, s["argmax"], None) if kind != "attn" else None
    return s


# ---- one pass ----

def _accept(s, targets, out):
    t = s["tree"]
    return d2sd.accept_path(s["B"], s["ip"], s["total"], t["parent"], t["depth"], t["path_id"], s["draft"], targets, out=out)


def _attention(s):
    x = s["x"]
    d2sd.cascade_verify_attention(
        x["q"], x["k_cache"], x["v_cache"], s["pt"], s["ctx"], x["k_tree"], x["v_tree"], s["ip"],
        s["tree"]["anc_mask"], total_nodes=s["total"], max_nodes=s["max_nodes"], max_ctx_len=s["max_ctx"],
        out=s["out"], lse=s["lse"], workspace=s["ws"], node_indptr_host=s["host"])


def run(s):
    kind = s["kind"]
    if kind == "attn":
        _attention(s)
        return {"out": s["out"], "lse": s["lse"]}
    if kind == "step":
        tree = d2sd.tree_build(s["B"], s["K"], s["p"], s["ip"], s["total"], s["W"], out=s["tree"])
        _attention(s)
        return {"out": s["out"], "lse": s["lse"], "tree": tree, "acc": _accept(s, s["argmax"], s["acc"])}
    if kind == "general":
        t = s["tree"]
        d2sd.tree_from_parents(s["ip"], s["total"], s["max_nodes"], s["parent"], t["anc_mask"].shape[1], out=t)
        _attention(s)
        return {"out": s["out"], "lse": s["lse"], "tree": t, "acc": _accept(s, s["argmax"], s["acc"])}
    if kind == "draw":
        d2sd.sample_targets(s["ip"], s["total"], s["max_nodes"], s["parent"], s["draft"], s["logits"], s["T"],
                            uniform=s["u"], out=s["tokens"])
        return {"tokens": s["tokens"], "acc": _accept(s, s["tokens"], s["acc"])}
    if kind == "plan":
        p, _ = d2sd.select_reanchor(s["B"], s["conf"], s["K"], s["kmax"], p_out=s["p"])
        ip = d2sd.tree_indptr(s["B"], s["K"], p, out=s["ip"])
        tree = d2sd.tree_build(s["B"], s["K"], p, ip, s["total"], s["W"], out=s["tree"])
        return {"p": p, "ip": ip, "tree": tree}
    # commit: contexts of one length, so the clamp at max_ctx makes a repeated
    # pass write the same slots
    d2sd.commit_accepted_kv(s["B"], s["ip"], s["total"], s["acc"]["path_nodes"], s["acc"]["accept_len"], s["k_tree"],
                            s["v_tree"], s["pt"], s["ctx"], s["k_cache"], s["v_cache"], s["max_ctx"])
    return {"k_cache": s["k_cache"], "v_cache": s["v_cache"], "ctx": s["ctx"]}


# ---- what a pass cannot do without ----

def work(case):
    kind, b, n = case["kind"], case["batch"], _mean_nodes(case)
    tree = b * n * 4 * (3 + (n + 31) // 32)          # parent, depth, path id, mask
    accept = b * n * 4 * 5 + b * case["B"] * 8
    if kind == "plan":
        return {"bytes": b * case["B"] * 4 + tree, "flops": b * case["B"] ** 2}
    e = 2 if case["dtype"] == "bf16" else 4
    if kind == "draw":
        return {"bytes": b * n * (case["vocab"] * e + 8) + accept, "flops": b * n * case["vocab"] * (3.0 if case["T"] > 0 else 1.0)}
    if kind == "commit":
        # about three tokens a request are committed at 0.7 agreement and K = 4
        return {"bytes": b * 4 * case["hkv"] * D * e * 2 * 2, "flops": 0.0}
    ctx = (case["lo"] + case["hi"]) / 2
    kv = b * (ctx + n) * case["hkv"] * D * e * 2
    qo = b * n * case["hq"] * (D * e * 2 + 4)
    return {"bytes": kv + qo + (tree + accept if kind != "attn" else 0), "flops": 4.0 * D * case["hq"] * b * n * (ctx + case["B"] / 2)}


def tolerance(case):
    if case["kind"] in ("plan", "commit"):
        return "exact"
    if case["kind"] == "draw":
        # a draw whose uniform lies within the rounding of the float32 running
        # sums of a cumulative boundary may take the neighbouring token
        return "exact" if case["T"] == 0 else {"rel": 0.0, "differ": 0.005}
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-2, "max": 0.1}


# ---- the same in 64 bits ----

def exact(case, seed):
    """Attention outputs by definition: every node attends to the whole
    context and to its ancestors-or-self, one softmax, float64."""
    if case["kind"] not in ("step", "attn", "general"):
        return None
    s = prepare(case, seed)
    lay, x = s["lay"], s["x"]
    G = case["hq"] // case["hkv"]
    scale = 1.0 / math.sqrt(D)
    out = torch.zeros(s["x"]["q"].shape, dtype=torch.float64, device=DEV)
    lse = torch.zeros(s["lse"].shape, dtype=torch.float64, device=DEV)
    for b in range(lay.batch):
        i0, i1, C = int(s["ip_host"][b]), int(s["ip_host"][b + 1]), int(lay.ctx_len[b])
        N = i1 - i0
        vis = _dev(_visible(s["par"][b])).repeat_interleave(G, 0)                     # [N G, N]
        pages = s["pt"][b, :(C + 15) // 16].long()
        for h in range(case["hkv"]):
            rows = lambda cache, tree: torch.cat(
                [cache[pages, h].reshape(-1, D)[:C], tree[i0:i1, h]]).double()        # [C + N, D]
            q = x["q"][i0:i1, h * G:(h + 1) * G].reshape(N * G, D).double()
            sc = (q @ rows(x["k_cache"], x["k_tree"]).t().contiguous()) * scale
            sc[:, C:].masked_fill_(~vis, float("-inf"))
            m = sc.amax(1, keepdim=True)
            p = torch.exp_(sc.sub_(m))
            l = p.sum(1, keepdim=True)
            out[i0:i1, h * G:(h + 1) * G] = ((p @ rows(x["v_cache"], x["v_tree"])) / l).reshape(N, G, D)
            lse[i0:i1, h * G:(h + 1) * G] = (m + l.log()).reshape(N, G)
    # by path: tokens and tree arrays have no 64-bit value
    return {"out": out, "lse": lse}
