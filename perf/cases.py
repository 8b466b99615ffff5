"""The work a user of this library has it do, as cases to be timed.

A decoding step is: the draft's tokens (input projection, QKV, window attention; for a tree also
top-k and expansion), verification attention in every layer of the target, acceptance, commit.  The
cases are those phases through the public entry points, over one-sequence and batched serving,
chains and trees, greedy and sampled acceptance, both storage types, both head sizes, both K/V
layouts, and model widths besides the one the benchmark is quoted on.

A case is a dict of plain values; "kind" says which phase it is:
  step    draft window attention, verification attention of `layers` layers, greedy acceptance
          (graph = 1: captured once in a HIP graph and replayed, as bench.py does)
  draft   the draft's new token of each of B sequences: Eq. 1 projection, QKV step with the cache
          append, window attention
  tree    the dynamic draft tree "total - depth - width": top-k of every level's rows, expansion,
          final selection
  verify  verification attention of `layers` layers
  accept  greedy acceptance
  finish  acceptance at temperature 1 and the commit of the accepted rows in `layers` layers
"""
import math
import random

import numpy as np
import torch

import paper_2602_15318_amd as sp

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
ESIZE = {"f32": 4, "bf16": 2}

# heads, head size, width and vocabulary of the benchmark's model
BASE = {"dtype": "bf16", "Hq": 28, "Hkv": 4, "d": 128, "hidden": 3584, "vocab": 152064}


def listed():
    return [
        # the smallest call: the tiny fp32 configuration, one whole step; launches and host time
        {"name": "step_tiny_f32", "kind": "step", "dtype": "f32", "Hq": 4, "Hkv": 1, "d": 64, "hidden": 256,
         "vocab": 1024, "B": 1, "ctx": 512, "ragged": 0, "window": 32, "n_q": 4, "tree": "chain", "layers": 1,
         "layout": "token", "graph": 0, "shape": 1},
        # one request drafting a chain on a long video: one new token
        {"name": "draft_one_token_26k", "kind": "draft", **BASE, "B": 1, "ctx": 26112, "ragged": 0, "window": 512,
         "shape": 2},
        # a decode batch drafting one token each on a model of another width and head size
        {"name": "draft_batch6_width2560", "kind": "draft", "dtype": "bf16", "Hq": 40, "Hkv": 8, "d": 64,
         "hidden": 2560, "vocab": 32000, "B": 6, "ctx": 5000, "ragged": 1, "window": 256, "shape": 3},
        # the dynamic tree 30-4-8 of one request over the full vocabulary
        {"name": "draft_tree_30_4_8", "kind": "tree", **BASE, "total": 30, "depth": 4, "width": 8, "shape": 4},
        # a short video, chain of 5, every layer of the target, launched call by call
        {"name": "verify_8k_chain5", "kind": "verify", **BASE, "B": 1, "ctx": 8192, "ragged": 0, "n_q": 5,
         "tree": "chain", "layers": 28, "layout": "token", "lse": 0, "shape": 5},
        # a long video verified with a 60-node tree
        {"name": "verify_26k_tree60", "kind": "verify", **BASE, "B": 1, "ctx": 26112, "ragged": 0, "n_q": 60,
         "tree": "shared", "layers": 8, "layout": "pair", "lse": 0, "shape": 6},
        # a ragged decode batch, chains of 6
        {"name": "verify_ragged8_chain6", "kind": "verify", **BASE, "B": 8, "ctx": 10240, "ragged": 1, "n_q": 6,
         "tree": "chain", "layers": 4, "layout": "head", "lse": 0, "shape": 7},
        # a batch in which every request grew a 30-node tree of its own, other head grouping
        {"name": "verify_batch12_trees30", "kind": "verify", **BASE, "Hq": 32, "Hkv": 8, "B": 12, "ctx": 4099,
         "ragged": 1, "n_q": 30, "tree": "own", "layers": 4, "layout": "token", "lse": 1, "shape": 8},
        # a smaller target with heads of 64, a batch of four
        {"name": "verify_batch4_d64_chain8", "kind": "verify", "dtype": "bf16", "Hq": 16, "Hkv": 4, "d": 64,
         "hidden": 1024, "vocab": 32000, "B": 4, "ctx": 6001, "ragged": 1, "n_q": 8, "tree": "chain", "layers": 6,
         "layout": "head", "lse": 0, "shape": 9},
        # the benchmark's step: 28 layers at 26,112 context, chain of 8, replayed from a HIP graph
        {"name": "step_26k_chain8_graph", "kind": "step", **BASE, "B": 1, "ctx": 26112, "ragged": 0, "window": 512,
         "n_q": 8, "tree": "chain", "layers": 28, "layout": "pair", "graph": 1, "shape": 10},
        # greedy acceptance of a batch of 30-node trees: 248 rows against the whole vocabulary
        {"name": "accept_batch8_trees30", "kind": "accept", **BASE, "B": 8, "n_q": 30, "tree": "own", "shape": 11},
        # a small batch at temperature 1 against a sampled draft, then the commit; another width
        {"name": "finish_batch4_t1_width2048", "kind": "finish", "dtype": "bf16", "Hq": 16, "Hkv": 4, "d": 128,
         "hidden": 2048, "vocab": 64003, "B": 4, "ctx": 1500, "ragged": 1, "n_q": 8, "tree": "chain", "layers": 24,
         "layout": "pair", "sampled": 1, "shape": 12},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _fits(case):
    w = work(case)
    if case["dtype"] == "f32":            # fp32 work runs at a fraction of the bf16 rate
        return w["bytes"] <= 1.5e9 and w["flops"] <= 4e10
    return w["bytes"] <= 2.5e9 and w["flops"] <= 2.5e11


def draw(rng):
    """One more case of the same ranges: every phase, 1 to 16 sequences, 200 to 32,000 tokens of
    context, 1 to 64 draft rows, widths 256 to 5120, vocabularies 1,000 to 152,064."""
    while True:
        c = _draw(rng)
        if _fits(c):
            return c


def _draw(rng):
    kind = rng.choice(["step", "draft", "tree", "verify", "verify", "verify", "accept", "finish"])
    c = {"kind": kind, "dtype": "f32" if rng.random() < 0.15 else "bf16"}
    if rng.random() < 0.4:                # the benchmark's model ...
        c.update({k: v for k, v in BASE.items() if k != "dtype"})
    else:                                 # ... or another one
        c["Hkv"] = rng.choice([1, 2, 4, 8])
        c["Hq"] = c["Hkv"] * rng.choice([1, 2, 3, 4, 5, 6, 7, 8])
        c["d"] = rng.choice([64, 128, 128])
        c["hidden"] = 8 * _log_int(rng, 32, 640)
        if rng.random() < 0.75:           # widths are multiples of 128 as a rule
            c["hidden"] = max(256, c["hidden"] // 128 * 128)
        c["vocab"] = _log_int(rng, 1000, 152064)
    c["shape"] = rng.randrange(1 << 20)
    if kind == "tree":
        c["width"] = rng.randint(2, 16)
        c["depth"] = rng.randint(1, 8)
        c["total"] = rng.randint(2, min(64, c["width"] * c["depth"] + 1))
        return c
    c["B"] = _log_int(rng, 1, 16)
    c["ctx"] = _log_int(rng, 200, 32000)
    c["ragged"] = int(c["B"] > 1 and rng.random() < 0.7)
    if kind in ("step", "draft"):
        c["window"] = _log_int(rng, 16, 1024)
    if kind == "draft":
        return c
    c["n_q"] = _log_int(rng, 1, 64)
    if kind in ("accept", "finish"):
        c["n_q"] = min(c["n_q"], 512 // c["B"] - 1)
    if kind == "step":
        c["n_q"] = min(c["n_q"], 512 // c["B"] - 1)
        c["graph"] = rng.randrange(2)
    c["tree"] = "chain" if c["n_q"] <= 12 else rng.choice(["shared", "own"])
    if kind == "accept":
        return c
    c["layers"] = rng.randint(1, 32)
    c["layout"] = rng.choice(["token", "head", "pair"])
    if kind == "verify":
        c["lse"] = rng.randrange(2)
    if kind == "finish":
        c["sampled"] = rng.randrange(2)
    return c


# ------------------------------------------------------------------ shapes of a case
def lengths(case):
    """Context length of every sequence: equal, or spread between 0.4 and 1.6 of the mean."""
    rng = random.Random(case["shape"])
    return [max(16, int(case["ctx"] * rng.uniform(0.4, 1.6))) if case["ragged"] else case["ctx"]
            for _ in range(case["B"])]


def _cu(lens):
    return np.concatenate(([0], np.cumsum(lens))).astype(np.int32)


def work(case):
    c, e = case, ESIZE[case["dtype"]]
    if c["kind"] == "tree":
        rows = 1 + (c["depth"] - 1) * c["width"]
        return {"bytes": c["depth"] * c["vocab"] * c["hidden"] * e + rows * c["hidden"] * e,
                "flops": 2 * rows * c["vocab"] * c["hidden"]}
    b = f = 0
    B, H, Hq, Hkv, d = c["B"], c["hidden"], c["Hq"], c["Hkv"], c["d"]
    if c["kind"] == "draft":
        feats = (Hq + 2 * Hkv) * d
        b += (2 * H * H + feats * H) * e + B * (3 * H + feats) * e
        f += 2 * B * (2 * H * H + feats * H)
    if c["kind"] in ("draft", "step"):
        n = sum(min(c["window"], _n_text(L)) for L in lengths(c))
        b += 2 * n * Hkv * d * e + 2 * B * Hq * d * e
        f += 4 * n * Hq * d
    if c["kind"] in ("verify", "step"):
        n = sum(lengths(c)) + B * c["n_q"]
        b += c["layers"] * (2 * n * Hkv * d + 2 * B * c["n_q"] * Hq * d) * e
        f += c["layers"] * 4 * c["n_q"] * Hq * d * n
    if c["kind"] in ("accept", "step", "finish"):
        M = B * (c["n_q"] + 1)
        b += (c["vocab"] + M) * H * e
        f += 2 * M * c["vocab"] * H
    if c["kind"] == "finish":
        b += 4 * c["layers"] * B * Hkv * d * e          # one row or more of K and of V moved per sequence
        if c["sampled"]:
            b += B * c["vocab"] * 4                     # the draft distribution of one row per sequence
    return {"bytes": b, "flops": f}


def tolerance(case):
    """bf16 results carry one rounding of the output (2^-9) and one of the probabilities; fp32
    results the order of their sums.  Rows whose best tokens tie within that are a rare exception
    at these vocabularies, so token ids and paths agree."""
    if case["kind"] == "accept":
        return "exact"
    if case["dtype"] == "f32" or case["kind"] == "tree":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-2, "max": 0.1}


# ------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(g, shape, dtype, std=1.0):
    # in slices, so that the fp32 draw of a large tensor does not double its memory
    out = torch.empty(shape, dtype=dtype, device="cuda")
    flat = out.view(-1)
    step = 1 << 27
    for i in range(0, flat.numel(), step):
        n = min(step, flat.numel() - i)
        flat[i:i + n] = torch.randn(n, generator=g, device="cuda") * std
    return out


def _n_text(L):
    """Text positions of a context: a video's visual tokens are all but a few percent of it."""
    return max(8, min(L, 64 + L // 28))


def _text_index(L, rng):
    """Ascending text positions: a prompt in front, now and then a run in the middle, the rest at
    the end (the query's own position is the last one)."""
    n = _n_text(L)
    head = rng.randint(0, n // 2)
    mid = rng.randint(0, (n - head) // 2)
    tail = n - head - mid
    at = rng.randint(head, max(head, L - tail - mid))
    return np.concatenate([np.arange(head), np.arange(at, at + mid), np.arange(L - tail, L)]).astype(np.int32)


def _kv(g, case, rows, n):
    """n layers of K/V in one allocation and the [rows, Hkv, d] views the library takes."""
    Hkv, d, dt = case["Hkv"], case["d"], DTYPES[case["dtype"]]
    if case.get("layout", "token") == "pair":          # a token's K row followed by its V row, head by head
        t = _normal(g, (n, Hkv, rows, 2, d), dt)
        return t, [(t[i, :, :, 0].permute(1, 0, 2), t[i, :, :, 1].permute(1, 0, 2)) for i in range(n)]
    if case.get("layout", "token") == "head":
        t = _normal(g, (n, 2, Hkv, rows, d), dt)
        return t, [(t[i, 0].permute(1, 0, 2), t[i, 1].permute(1, 0, 2)) for i in range(n)]
    t = _normal(g, (n, 2, rows, Hkv, d), dt)
    return t, [(t[i, 0], t[i, 1]) for i in range(n)]


def _tree(rng, n_q):
    """A draft tree of the dynamic kind: nodes level by level, up to 8 levels, parents among the
    better half of the level before."""
    parent, level = [], [-1]
    depth = min(8, max(2, n_q // 6))
    for lv in range(depth):
        want = n_q // depth + (1 if lv < n_q % depth else 0)
        first = len(parent)
        for i in range(want):
            parent.append(level[min(rng.randrange(max(1, (len(level) + 1) // 2)) if lv else 0, len(level) - 1)])
        parent[first:] = sorted(parent[first:])
        level = list(range(first, len(parent))) or level
    return np.array(parent, dtype=np.int32)


def _parents(case, seed):
    """(host [B, n_q] parents, what the library is given: None, [n_q] or [B, n_q])."""
    B, n_q = case["B"], case["n_q"]
    rng = random.Random(seed)
    if case["tree"] == "chain":
        return np.tile(np.arange(-1, n_q - 1, dtype=np.int32), (B, 1)), None
    if case["tree"] == "shared":
        t = _tree(rng, n_q)
        return np.tile(t, (B, 1)), torch.from_numpy(t).cuda()
    t = np.stack([_tree(rng, n_q) for _ in range(B)])
    return t, torch.from_numpy(t).cuda()


def _head(g, case, rows):
    """lm_head weights at the initialiser's scale and hidden rows as a trained model has them: six
    tokens share nearly all of a row's probability, the first of them two thirds."""
    H, V, dt = case["hidden"], case["vocab"], DTYPES[case["dtype"]]
    W = _normal(g, (V, H), dt, 0.02)
    ids = torch.randint(0, V, (rows, 6), generator=g, device="cuda")
    logit = math.log(V) + 6.0 - torch.tensor([0.0, 1.5, 2.0, 3.0, 4.0, 5.0], device="cuda")
    coef = logit / (4e-4 * H)             # |W[v]|^2 is about 4e-4 H
    hid = 0.3 * torch.randn(rows, H, generator=g, device="cuda")
    for j in range(6):
        hid += W[ids[:, j]].float() * coef[j]
    return W, ids[:, 0], hid.to(dt)


def _greedy_drafts(case, seed, parents, ids):
    """Draft tokens: the first child of a node is the target's token four times in five."""
    B, n_q, V = case["B"], case["n_q"], case["vocab"]
    rng = random.Random(seed + 1)
    t = ids.cpu().numpy().reshape(B, n_q + 1)
    d = np.zeros((B, n_q), dtype=np.int32)
    for b in range(B):
        seen = set()
        for i in range(n_q):
            p = int(parents[b, i])
            d[b, i] = t[b, p + 1] if p not in seen and rng.random() < 0.8 else rng.randrange(V)
            seen.add(p)
    return torch.from_numpy(d.reshape(-1)).cuda()


def _sampled_drafts(case, g, parents, hid, W):
    """The draft's distribution of every row (close to the target's, not equal) and tokens drawn
    from it, node by node from its parent's row."""
    B, n_q = case["B"], case["n_q"]
    noisy = (hid.float() + 0.5 * torch.randn(hid.shape, generator=g, device="cuda")).to(hid.dtype)
    q = torch.softmax((noisy @ W.t()).float(), dim=1).contiguous()
    row = torch.from_numpy((parents + 1 + np.arange(B)[:, None] * (n_q + 1)).reshape(-1)).long().cuda()
    tok = torch.cat([torch.multinomial(q[r], 1, generator=g) for r in row.split(64)])
    return q, tok.view(-1).to(torch.int32)


def _ws(nbytes):
    return torch.empty(max(int(nbytes), 1), dtype=torch.uint8, device="cuda")


def _prepare_draft_attn(s, case, g, seed, append):
    lens = lengths(case)
    rng = random.Random(seed + 2)
    tidx = [_text_index(L, rng) for L in lens]
    s["draft_cu"], s["cu_text"] = _cu(lens), _cu([len(t) for t in tidx])
    s["text_idx"] = torch.from_numpy(np.concatenate(tidx)).cuda()
    s["draft_kv"], ((s["dk"], s["dv"]),) = _kv(g, {**case, "layout": "token"}, sum(lens), 1)
    if not append:
        s["dq"] = _normal(g, (case["B"], case["Hq"], case["d"]), DTYPES[case["dtype"]])


def _prepare_verify(s, case, g):
    lens = [L + case["n_q"] for L in lengths(case)]
    s["cu"] = _cu(lens)
    dt = DTYPES[case["dtype"]]
    s["kv"], s["layers"] = _kv(g, case, sum(lens), case["layers"])
    s["q"] = [_normal(g, (case["B"] * case["n_q"], case["Hq"], case["d"]), dt) for _ in range(case["layers"])]
    s["out"] = [torch.empty_like(q) for q in s["q"]]
    s["lse"] = [torch.empty(q.shape[:2], dtype=torch.float32, device="cuda") if case.get("lse") else None for q in s["q"]]
    k, v = s["layers"][0]
    s["ws_v"] = _ws(sp.verify_attn_workspace_bytes(s["q"][0], k, v, case["B"], case["n_q"], int(s["cu"][-1])))


def prepare(case, seed):
    g = _gen(seed)
    dt, B, H = DTYPES[case["dtype"]], case.get("B", 1), case["hidden"]
    code = {"f32": 0, "bf16": 1}[case["dtype"]]    # sparrow_dtype
    s = {"case": case}
    kind = case["kind"]
    if kind == "draft":
        _prepare_draft_attn(s, case, g, seed, append=True)
        d, feats = case["d"], (case["Hq"] + 2 * case["Hkv"]) * case["d"]
        s["embed"] = _normal(g, (case["vocab"], H), dt, 0.02)
        s["tok"] = torch.randint(0, case["vocab"], (B,), generator=g, device="cuda", dtype=torch.int32)
        s["h_prev"] = _normal(g, (B, H), dt)
        s["w_fc"], s["b_fc"] = _normal(g, (H, 2 * H), dt, 0.02), _normal(g, (H,), dt, 0.02)
        s["norm"] = (1.0 + 0.1 * torch.randn(H, generator=g, device="cuda")).to(dt)
        s["w_qkv"], s["b_qkv"] = _normal(g, (feats, H), dt, 0.02), _normal(g, (feats,), dt, 0.5)
        pos = torch.tensor([L - 1 for L in lengths(case)], device="cuda", dtype=torch.float64)
        ang = pos[:, None] * (1e6 ** (-2.0 * torch.arange(d // 2, device="cuda", dtype=torch.float64) / d))[None, :]
        s["cos"], s["sin"] = ang.cos().float(), ang.sin().float()
        s["kv_rows"] = s["draft_cu"][1:] - 1
    if kind == "step":
        _prepare_draft_attn(s, case, g, seed, append=False)
    if kind in ("step", "verify"):
        _prepare_verify(s, case, g)
    if kind == "finish":
        lens = [L + case["n_q"] for L in lengths(case)]
        s["cu"] = _cu(lens)
        s["kv"], s["layers"] = _kv(g, case, sum(lens), case["layers"])
    if kind in ("step", "verify", "accept", "finish"):
        parents, s["parent"] = _parents(case, seed)
    if kind in ("step", "accept", "finish"):
        s["W"], ids, s["hid"] = _head(g, case, B * (case["n_q"] + 1))
        s["drafts"] = _greedy_drafts(case, seed, parents, ids)
    if kind in ("step", "accept"):
        s["ws_a"] = _ws(sp.accept_workspace_bytes(code, B, case["n_q"], H, case["vocab"]))
    if kind == "finish":
        s["probs"] = None
        if case["sampled"]:
            s["probs"], s["drafts"] = _sampled_drafts(case, g, parents, s["hid"], s["W"])
        s["u_accept"] = torch.rand(B, case["n_q"], generator=g, device="cuda")
        s["u_bonus"] = torch.rand(B, generator=g, device="cuda")
        s["ws_a"] = _ws(sp.accept_sample_workspace_bytes(code, B, case["n_q"], H, case["vocab"]))
    if kind == "tree":
        s["W"], _, s["rows"] = _head(g, case, 1 + case["width"] * (case["depth"] - 1))
    if case.get("graph"):
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _step(s)                      # once outside the capture: set-up of the first call
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            s["result"] = _step(s)
    return s


# ------------------------------------------------------------------ one pass
def _draft_attn(s, q):
    return sp.draft_window_attn(q, s["dk"], s["dv"], s["draft_cu"], s["text_idx"], s["cu_text"],
                                s["case"]["window"])


def _verify(s):
    c = s["case"]
    for i, (k, v) in enumerate(s["layers"]):
        sp.verify_attn(s["q"][i], k, v, s["cu"], s["parent"], c["n_q"], out=s["out"][i], lse=s["lse"][i],
                       want_lse=bool(c.get("lse")), workspace=s["ws_v"])
    return s["out"], [x for x in s["lse"] if x is not None]


def _accept(s):
    c = s["case"]
    return sp.accept(s["hid"], s["W"], s["drafts"], s["parent"], c["B"], c["n_q"], workspace=s["ws_a"])


def _step(s):
    return _draft_attn(s, s["dq"]), _verify(s), _accept(s)


def _draft(s):
    c = s["case"]
    z = sp.hsr_fc(s["embed"], s["tok"], s["h_prev"], s["w_fc"], s["b_fc"])
    q = sp.draft_qkv_append(z, s["norm"], 1e-6, s["w_qkv"], s["b_qkv"], s["cos"], s["sin"], s["kv_rows"], c["Hq"],
                            s["dk"], s["dv"])
    return z, q, s["draft_kv"], _draft_attn(s, q)


def _draft_tree(s):
    c = s["case"]
    w = c["width"]
    pool = sp.TreePool(w, c["depth"])
    tops = []
    for level in range(c["depth"]):
        rows = s["rows"][:1] if level == 0 else s["rows"][1 + (level - 1) * w:1 + level * w]
        ids, logp = sp.draft_topk(rows, s["W"], w)
        pool.expand(ids, logp)
        tops.append((ids, logp))
    return tops, pool.select(c["total"])


def _finish(s):
    c = s["case"]
    if s["probs"] is None:
        r = sp.accept_sample(s["hid"], s["W"], s["drafts"], s["parent"], c["B"], c["n_q"], 1.0, s["u_accept"],
                             s["u_bonus"], workspace=s["ws_a"])
    else:
        r = sp.accept_sample_q(s["hid"], s["W"], s["drafts"], s["parent"], c["B"], c["n_q"], 1.0,
                               draft_probs=s["probs"], u_accept=s["u_accept"], u_bonus=s["u_bonus"],
                               workspace=s["ws_a"])
    nxt = sp.kv_commit([k for k, _ in s["layers"]], [v for _, v in s["layers"]], s["cu"], c["n_q"], r["accept_path"],
                       r["accept_len"], hidden_rows=s["hid"])
    return r, nxt, s["kv"]


def run(state):
    if "graph" in state:
        state["graph"].replay()
        return state["result"]
    return {"step": _step, "draft": _draft, "tree": _draft_tree, "verify": _verify, "accept": _accept,
            "finish": _finish}[state["case"]["kind"]](state)


# ------------------------------------------------------------------ the same results in 64 bits
def _attend(q, k, v, keep=None):
    """q [rows, Hq, d], k and v [n, Hkv, d] in 64 bits, keep [rows, n] or None: (out, lse)."""
    rows, Hq, d = q.shape
    n, Hkv = k.shape[0], k.shape[1]
    g = Hq // Hkv
    out, lse = torch.empty_like(q), torch.empty((rows, Hq), dtype=q.dtype, device=q.device)
    for c in range(Hkv):
        qc = q[:, c * g:(c + 1) * g].reshape(rows * g, d)
        sc = (qc @ k[:, c].t().contiguous()).view(rows, g, n) / math.sqrt(d)
        if keep is not None:
            sc.masked_fill_(~keep[:, None, :], -math.inf)
        lse[:, c * g:(c + 1) * g] = torch.logsumexp(sc, dim=2)
        p = torch.softmax(sc, dim=2).view(rows * g, n)
        out[:, c * g:(c + 1) * g] = (p @ v[:, c].contiguous()).view(rows, g, d)
    return out, lse


def _exact_draft_attn(s, q, k, v):
    cu, ct, w = s["draft_cu"], s["cu_text"], s["case"]["window"]
    outs, lses = [], []
    for b in range(s["case"]["B"]):
        at = s["text_idx"][int(ct[b]):int(ct[b + 1])][-w:].long() + int(cu[b])
        o, l = _attend(q[b:b + 1], k[at].double(), v[at].double())
        outs.append(o)
        lses.append(l)
    return torch.cat(outs), torch.cat(lses)


def _exact_verify(s, parents):
    c = s["case"]
    n_q = c["n_q"]
    outs, lses = [], []
    sees = []                             # draft rows that a draft row may attend: itself and its ancestors
    for b in range(c["B"]):
        m = torch.zeros((n_q, n_q), dtype=torch.bool)
        for i in range(n_q):
            a = i
            while a >= 0:
                m[i, a] = True
                a = int(parents[b, a])
        sees.append(m.cuda())
    for (k, v), q in zip(s["layers"], s["q"]):
        o, l = torch.empty(q.shape, dtype=torch.float64, device="cuda"), torch.empty(q.shape[:2], dtype=torch.float64, device="cuda")
        for b in range(c["B"]):
            t0, t1 = int(s["cu"][b]), int(s["cu"][b + 1])
            keep = torch.ones((n_q, t1 - t0), dtype=torch.bool, device="cuda")
            keep[:, t1 - t0 - n_q:] = sees[b]
            r = slice(b * n_q, (b + 1) * n_q)
            o[r], l[r] = _attend(q[r].double(), k[t0:t1].double(), v[t0:t1].double(), keep)
        outs.append(o)
        lses.append(l)
    return outs, [l for l, x in zip(lses, s["lse"]) if x is not None]


def _exact_draft(s):
    c = s["case"]
    Hq, Hkv, d, M = c["Hq"], c["Hkv"], c["d"], c["B"]
    z = torch.cat([s["embed"][s["tok"].long()], s["h_prev"]], dim=1).double() @ s["w_fc"].double().t() + s["b_fc"].double()
    x = z * torch.rsqrt((z * z).mean(dim=1, keepdim=True) + 1e-6) * s["norm"].double()
    f = (x @ s["w_qkv"].double().t() + s["b_qkv"].double()).view(M, Hq + 2 * Hkv, d)
    cos, sin = s["cos"].double()[:, None], s["sin"].double()[:, None]
    lo, hi = f[..., :d // 2], f[..., d // 2:]
    turned = torch.cat([lo * cos - hi * sin, hi * cos + lo * sin], dim=2)
    kv = s["draft_kv"].double()
    rows = torch.from_numpy(s["kv_rows"].astype(np.int64)).cuda()
    kv[0, 0, rows] = turned[:, Hq:Hq + Hkv]
    kv[0, 1, rows] = f[:, Hq + Hkv:]
    q = turned[:, :Hq].contiguous()
    return z, q, kv, _exact_draft_attn(s, q, kv[0, 0], kv[0, 1])


def _exact_tree(s):
    c = s["case"]
    w, tops = c["width"], []
    W = s["W"].double()
    for level in range(c["depth"]):
        rows = s["rows"][:1] if level == 0 else s["rows"][1 + (level - 1) * w:1 + level * w]
        logp = torch.log_softmax(rows.double() @ W.t(), dim=1)
        tops.append((None, torch.topk(logp, w, dim=1).values))
    return tops, None


def exact(case, seed):
    """What run() returns, where that is a computed number, in 64 bits; token ids, paths, parents
    and moved rows are none."""
    kind = case["kind"]
    if kind in ("accept", "finish"):
        return None
    s = prepare({**case, "graph": 0}, seed)
    if kind == "draft":
        return _exact_draft(s)
    if kind == "tree":
        return _exact_tree(s)
    verified = _exact_verify(s, _parents(case, seed)[0])
    if kind == "verify":
        return verified
    return _exact_draft_attn(s, s["dq"].double(), s["dk"], s["dv"]), verified, None
