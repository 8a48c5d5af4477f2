"""The work a user has this package do, as cases that can be timed and compared.

Each case goes through the public entry points (`paper_2609_29029_amd`): the
calls of one scene-query on their own (Stage-1 scoring, selection and
compaction, the contextual merge, the decoder prefill, a decode step), at the
sizes of this repository's workloads, and whole scene-queries (`SceneQuery`).
Shapes: 336 x 336 px tiles of 576 tokens, an 8 x 8 and a 20 x 20 scene, token
budgets 576/288/144/64 by score rank, 35 system and 32 question rows, a
LLaMA-7B-shaped decoder; a small float32 scene and a 20-head decoder with
64-dimensional heads are the small ends.  `draw` gives more of the same calls,
with sizes over the whole range between them.

Inputs are made on the GPU from the seed: N(0, 1) tokens with a query-aligned
component planted on a few tiles, unit query and background vectors, N(0, 0.02)
weights, gains around 1, key/value caches with the spread the projections give.
"""
import math

import numpy as np
import torch

import paper_2609_29029_amd as R
from paper_2609_29029_amd.pipeline import PrefillShape, SceneQuery

TIERS = (1, 3, 4)          # sixteenths of the kept tiles at the first three levels
UTILITY = dict(levels=[576, 432, 288, 144, 72], alpha_pos=[0.92, 0.90, 0.85, 0.74, 0.58],
               alpha_neg=[0.95, 0.95, 0.94, 0.93, 0.91], energy=[1.0, 0.75, 0.5, 0.25, 0.125], lam=0.1)
WEIGHTS = ("wq", "wk", "wv", "wo", "w_gate", "w_up", "w_down")


# ------------------------------------------------------------------ the cases
def _score(name, n_tiles, n_v, d, dt="bf16", n_bg=15, knn=0, keep=None, sims=True):
    c = dict(kind="score", dt=dt, n_tiles=n_tiles, n_v=n_v, d=d, n_bg=n_bg, knn=knn, sims=sims,
             keep=max(1, n_tiles // 4) if keep is None else keep)
    return dict(name=name, **c) if name else c


def _pack(name, n_tiles, n_v, d, n_keep, levels, n_sys, n_qry, shared, dt="bf16"):
    c = dict(kind="pack", dt=dt, n_tiles=n_tiles, n_v=n_v, d=d, n_keep=n_keep, levels=levels, n_sys=n_sys,
             n_qry=n_qry, shared=shared)
    return dict(name=name, **c) if name else c


def _merge(name, n_tiles, n_v, d, n_keep, levels, dt="bf16"):
    c = dict(kind="merge", dt=dt, n_tiles=n_tiles, n_v=n_v, d=d, n_keep=n_keep, levels=levels, num=10, den=64)
    return dict(name=name, **c) if name else c


def _prefill(name, n_keep, levels, n_sys, n_qry, shared, d, heads, ffn, layers, kv, dt="bf16"):
    c = dict(kind="prefill", dt=dt, n_keep=n_keep, levels=levels, n_sys=n_sys, n_qry=n_qry, shared=shared, d=d,
             heads=heads, ffn=ffn, layers=layers, kv=kv)
    return dict(name=name, **c) if name else c


def _decode(name, n_keep, levels, n_sys, n_qry, shared, d, heads, ffn, layers, step):
    c = dict(kind="decode", dt="bf16", n_keep=n_keep, levels=levels, n_sys=n_sys, n_qry=n_qry, shared=shared, d=d,
             heads=heads, ffn=ffn, layers=layers, step=step, max_new=8)
    return dict(name=name, **c) if name else c


def _query(name, n_tiles, n_v, d, keep, levels, n_sys, n_qry, shared, heads, ffn, layers, dt="bf16", knn=0,
           merge=False, utility=False, tau=0.37, n_bg=15):
    c = dict(kind="query", dt=dt, n_tiles=n_tiles, n_v=n_v, d=d, n_bg=n_bg, knn=knn, keep=keep, levels=levels,
             n_sys=n_sys, n_qry=n_qry, shared=shared, heads=heads, ffn=ffn, layers=layers, merge=merge,
             utility=utility, tau=tau)
    return dict(name=name, **c) if name else c


def listed():
    full = "576,288,144,64"
    return [
        # the smallest whole query: 4 tiles, a float32 model of width 256, 2 kept; launches and latency count
        _query("query_small_f32", 4, 576, 256, 2, "64", 8, 16, False, 4, 688, 1, dt="f32"),
        # Stage 1 on the 8 x 8 walkthrough scene and on the 20 x 20 scene of about 6700 x 6700 px
        _score("score_64_tiles", 64, 576, 4096, keep=16),
        _score("score_400_tiles", 400, 576, 4096, keep=100),
        # the same with each score averaged over its six most similar tiles
        _score("score_400_tiles_knn6", 400, 576, 4096, knn=6, keep=100),
        # selection under the elastic budgets and packing of the 100 kept prompts
        _pack("pack_400_tiles", 400, 576, 4096, 100, full, 35, 32, True),
        # the remainder of the 100 kept tiles merged into contextual tokens
        _merge("merge_400_tiles", 400, 576, 4096, 100, full),
        # one tile at full budget, 643 rows: a single question about one image
        _prefill("prefill_one_tile", 1, "576", 35, 32, False, 4096, 32, 11008, 1, True),
        # the 16 kept prompts of the 8 x 8 scene, system rows shared
        _prefill("prefill_64_tiles", 16, full, 35, 32, True, 4096, 32, 11008, 1, False),
        # a small decoder with 64-dimensional heads, few ragged prompts, odd sizes
        _prefill("prefill_small_ragged", 9, "557,331,101,23", 13, 7, False, 1280, 20, 3456, 2, True),
        # one generated token for each of 100 prompts, and for a single one
        _decode("decode_100_prompts", 100, full, 35, 32, True, 4096, 32, 11008, 4, 3),
        _decode("decode_one_prompt", 1, "576", 35, 32, False, 4096, 32, 11008, 4, 3),
        # the whole query on the 20 x 20 scene through the 32-layer decoder
        _query("query_400_tiles_l32", 400, 576, 4096, 100, full, 35, 32, True, 32, 11008, 32),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _levels(rng, n_v, lo=1):
    lo = max(lo, n_v // 24)
    four = set()
    while len(four) < min(4, n_v - lo + 1):
        four.add(_log(rng, lo, n_v))
    return ",".join(str(x) for x in sorted(four, reverse=True)) if len(four) == 4 else str(max(four))


def _model(rng, dt, largest):
    """d, heads, ffn of a decoder no larger than `largest` wide."""
    if dt == "f32":
        hd = rng.choice([64, 128])
        d = hd * rng.randint(1, 1024 // hd)
        return d, d // hd, 16 * rng.randint(d // 16, 3 * d // 16)
    hd = rng.choice([64, 128, 128])
    d = 256 * rng.choice([x for x in (1, 2, 3, 4, 5, 6, 8, 10, 12, 16) if 256 * x <= largest])
    return d, d // hd, 128 * rng.randint(2 * d // 128, 3 * d // 128)


def draw(rng):
    kind = rng.choice(["score", "score", "pack", "merge", "prefill", "prefill", "prefill", "decode", "decode", "query"])
    dt = "f32" if rng.random() < 0.2 else "bf16"
    if kind == "score":
        n_tiles, n_v = _log(rng, 1, 400), _log(rng, 16, 1024)
        d = 32 * _log(rng, 2, 128)
        while n_tiles * n_v * d * (2 if dt == "f32" else 1) > 400 * 576 * 4096:
            n_tiles = max(1, n_tiles // 2)
        knn = rng.randint(1, 8) if rng.random() < 0.3 else 0
        keep = rng.choice([0, max(1, n_tiles // 4)])
        return _score(None, n_tiles, n_v, d, dt, rng.randint(0, 15), knn, keep, rng.random() < 0.8)
    if kind == "pack":
        n_tiles, n_v = _log(rng, 1, 400), _log(rng, 24, 1024)
        d = 32 * _log(rng, 2, 128)
        while n_tiles * n_v * d * (2 if dt == "f32" else 1) > 400 * 576 * 4096:
            n_tiles = max(1, n_tiles // 2)
        n_keep = rng.randint(1, n_tiles)
        return _pack(None, n_tiles, n_v, d, n_keep, _levels(rng, n_v), rng.randint(1, 48), rng.randint(1, 48),
                     rng.random() < 0.5, dt)
    if kind == "merge":
        n_keep, n_v = _log(rng, 1, 100), _log(rng, 24, 1024 if dt == "bf16" else 576)
        d = 32 * _log(rng, 2, 128 if dt == "bf16" else 32)
        return _merge(None, n_keep + rng.randint(0, 8), n_v, d, n_keep, _levels(rng, n_v, 8), dt)
    if kind == "prefill":
        d, heads, ffn = _model(rng, dt, 4096)
        n_keep = _log(rng, 1, 64) if dt == "bf16" else _log(rng, 1, 8)
        levels = _levels(rng, rng.randint(24, 640) if dt == "bf16" else rng.randint(24, 160))
        return _prefill(None, n_keep, levels, rng.randint(1, 48), rng.randint(1, 48), rng.random() < 0.5, d, heads, ffn,
                        rng.randint(1, 2), rng.random() < 0.5, dt)
    if kind == "decode":
        d, heads, ffn = _model(rng, "bf16", 4096)
        return _decode(None, _log(rng, 1, 160), _levels(rng, rng.randint(24, 640)), rng.randint(1, 48),
                       rng.randint(1, 48), rng.random() < 0.5, d, heads, ffn, rng.randint(1, 4), rng.randint(0, 7))
    d, heads, ffn = _model(rng, dt, 2048)
    n_tiles, n_v = _log(rng, 2, 64), _log(rng, 32, 576 if dt == "bf16" else 144)
    how = rng.choice(["top", "threshold", "utility"])
    if how == "utility":
        n_v = 576
        n_tiles = min(n_tiles, 64 if dt == "bf16" else 6)
    keep = 0 if how == "threshold" else max(1, n_tiles // 4)
    return _query(None, n_tiles, n_v, d, keep, _levels(rng, n_v), rng.randint(1, 40), rng.randint(1, 40),
                  rng.random() < 0.5, heads, ffn, rng.randint(1, 2), dt, rng.choice([0, 0, 6]),
                  how == "top" and rng.random() < 0.4, how == "utility", 0.6, rng.randint(1, 15))


# ------------------------------------------------------------------ inputs
def _dt(case):
    return torch.float32 if case["dt"] == "f32" else torch.bfloat16


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(g, dt, *shape, std=1.0, mean=0.0):
    x = torch.empty(*shape, dtype=dt, device="cuda")
    x.normal_(mean, std, generator=g)
    return x


def _levels_of(case):
    return [int(x) for x in case["levels"].split(",")]


def _budgets(case, n_keep):
    lv = _levels_of(case)
    tiers = TIERS if len(lv) == 4 else ()
    out = []
    for num, b in zip(tiers, lv):
        out += [b] * (n_keep * num // 16)
    return out + [lv[-1]] * (n_keep - len(out))


def _bank(g, case):
    """Query row and background rows, unit norm, in the storage type."""
    q = torch.randn(1 + case["n_bg"], case["d"], generator=g, device="cuda")
    return (q / q.norm(dim=1, keepdim=True)).to(_dt(case))


def _scene(g, case, bank):
    """N(0, 1) tokens; one tile in twenty (at least one) carries the query on a fifth of its tokens."""
    n_tiles, n_v, d = case["n_tiles"], case["n_v"], case["d"]
    x = _normal(g, _dt(case), n_tiles, n_v, d)
    planted = torch.randperm(n_tiles, generator=g, device="cuda")[:max(1, n_tiles // 20)]
    alpha = 0.5 * math.sqrt(d / 256)
    for t in planted.tolist():
        x[t, ::5] += (alpha * bank[0].float()).to(x.dtype)
    return x


def _layers(g, case):
    d, f, dt = case["d"], case["ffn"], _dt(case)
    shape = dict(wq=(d, d), wk=(d, d), wv=(d, d), wo=(d, d), w_gate=(f, d), w_up=(f, d), w_down=(d, f))
    out = []
    for _ in range(case["layers"]):
        w = {n: _normal(g, dt, *shape[n], std=0.02) for n in WEIGHTS}
        w["g_attn"] = _normal(g, dt, d, std=0.05, mean=1.0)
        w["g_ffn"] = _normal(g, dt, d, std=0.05, mean=1.0)
        out.append(w)
    return out


def _cfg(case):
    return R.model_cfg(case["d"], case["heads"], case["d"] // case["heads"], case["ffn"], case["layers"], 1e-6,
                       10000.0, R.RIFT_F32 if case["dt"] == "f32" else R.RIFT_BF16)


def _sequences(case):
    """Prefix rows, and the prompts' own lengths after them."""
    pre = case["n_sys"] if case["shared"] else 0
    own = case["n_qry"] + (0 if case["shared"] else case["n_sys"])
    return pre, [own + b for b in _budgets(case, case["n_keep"])]


def _cu_pos(case):
    pre, lens = _sequences(case)
    seqs = ([pre] if pre else []) + lens
    cu = np.concatenate([[0], np.cumsum(seqs)]).astype(np.int32)
    pos = np.concatenate(([np.arange(pre)] if pre else []) + [pre + np.arange(n) for n in lens]).astype(np.int32)
    return pre, seqs, cu, pos


def _bytes(n):
    return torch.empty(max(256, n), dtype=torch.uint8, device="cuda")


def _i32(*shape):
    return torch.empty(*shape, dtype=torch.int32, device="cuda")


def _selection(g, case, budgets):
    """Distinct ascending token indices of each kept tile, as selection leaves them, and their offsets."""
    keys = torch.rand(case["n_keep"], case["n_v"], generator=g, device="cuda")
    rank = keys.argsort(dim=1).argsort(dim=1)
    b = torch.tensor(budgets, device="cuda")
    sel = (rank < b[:, None]).nonzero()[:, 1].to(torch.int32)
    offs = torch.zeros(case["n_keep"] + 1, dtype=torch.int32, device="cuda")
    offs[1:] = b.cumsum(0)
    return sel, offs


def prepare(case, seed):
    g, kind, dt = _gen(seed), case["kind"], _dt(case)
    s = {"case": case}
    if kind in ("score", "query"):
        s["bank"] = _bank(g, case)
        s["tokens"] = _scene(g, case, s["bank"])
    if kind == "score":
        n, nt = case["n_tiles"] * case["n_v"], case["n_tiles"]
        s["key"] = torch.empty(n, dtype=torch.float64, device="cuda")
        s["sim"] = torch.empty(n, 1 + case["n_bg"], dtype=torch.float32, device="cuda") if case["sims"] else None
        s["score"] = torch.empty(nt, dtype=torch.float64, device="cuda")
        s["u"] = torch.empty(nt, dtype=torch.float32, device="cuda")
        s["order"], s["n_keep"] = _i32(nt), _i32(1)
        s["ws"] = _bytes(R.rift_score_workspace_size(nt, case["n_v"], case["d"], case["knn"]))
    elif kind == "pack":
        budgets = _budgets(case, case["n_keep"])
        pre, seqs, cu, _ = _cu_pos(case)
        total = int(cu[-1])
        s["tokens"] = _normal(g, dt, case["n_tiles"], case["n_v"], case["d"])
        s["sys"], s["qry"] = _normal(g, dt, case["n_sys"], case["d"]), _normal(g, dt, case["n_qry"], case["d"])
        s["key"] = torch.randn(case["n_tiles"] * case["n_v"], dtype=torch.float64, device="cuda", generator=g)
        s["kept"] = torch.randperm(case["n_tiles"], generator=g, device="cuda")[:case["n_keep"]].to(torch.int32)
        s["budgets"] = torch.tensor(budgets, dtype=torch.int32, device="cuda")
        s["offs"], s["sel"], s["cu"] = _i32(case["n_keep"] + 1), _i32(sum(budgets)), _i32(len(cu))
        s["packed"], s["pos"] = torch.empty(total, case["d"], dtype=dt, device="cuda"), _i32(total)
        s["st1"], s["st2"] = _i32(1), _i32(1)
    elif kind == "merge":
        dom, ctx = R.rift_split_budgets(_budgets(case, case["n_keep"]), case["n_v"], case["num"], case["den"])
        s["tokens"] = _normal(g, dt, case["n_tiles"], case["n_v"], case["d"])
        s["kept"] = torch.randperm(case["n_tiles"], generator=g, device="cuda")[:case["n_keep"]].to(torch.int32)
        s["sel"], s["offs"] = _selection(g, case, dom.tolist())
        s["coffs"] = torch.from_numpy(np.concatenate([[0], np.cumsum(ctx)]).astype(np.int32)).cuda()
        s["rows"] = torch.empty(int(ctx.sum()), case["d"], dtype=dt, device="cuda")
        s["status"], s["ws"] = _i32(1), _bytes(R.rift_merge_workspace_size(case["n_keep"], case["n_v"]))
    elif kind == "prefill":
        pre, seqs, cu, pos = _cu_pos(case)
        total, longest = int(cu[-1]), pre + max(seqs[1:] if pre else seqs)
        s["cfg"], s["layers"], s["x"] = _cfg(case), _layers(g, case), _normal(g, dt, total, case["d"])
        s["cu"], s["pos"] = torch.from_numpy(cu).cuda(), torch.from_numpy(pos).cuda()
        s["n_seq"], s["longest"], s["pre"] = len(seqs), longest, pre
        s["hidden"] = torch.empty(total, case["d"], dtype=torch.float32, device="cuda")
        s["kv"] = torch.empty(case["layers"], 2, total, case["d"], dtype=dt, device="cuda") if case["kv"] else None
        s["ws"] = _bytes(R.rift_prefill_workspace_size(s["cfg"], total, longest))
    elif kind == "decode":
        pre, seqs, cu, _ = _cu_pos(case)
        total, longest = int(cu[-1]), pre + max(seqs[1:] if pre else seqs)
        n, d, spread = case["n_keep"], case["d"], 0.02 * math.sqrt(case["d"])
        s["cfg"], s["layers"], s["x"] = _cfg(case), _layers(g, case), _normal(g, dt, n, d)
        s["cu"], s["total"], s["longest"], s["pre"] = torch.from_numpy(cu).cuda(), total, longest, pre
        s["kv"] = _normal(g, dt, case["layers"], 2, total, d, std=spread)
        s["kv_new"] = _normal(g, dt, case["layers"], 2, n, case["max_new"], d, std=spread)
        s["hidden"] = torch.empty(n, d, dtype=torch.float32, device="cuda")
        s["ws"] = _bytes(R.rift_decode_workspace_size(s["cfg"], n, longest, case["max_new"]))
    elif kind == "query":
        lv = _levels_of(case)
        s["sys"], s["qry"] = _normal(g, dt, case["n_sys"], case["d"]), _normal(g, dt, case["n_qry"], case["d"])
        s["layers"] = _layers(g, case)
        shape = PrefillShape(case["d"], case["heads"], case["d"] // case["heads"], case["ffn"], case["layers"])
        s["query"] = SceneQuery(s["tokens"], s["bank"], s["sys"], s["qry"], s["layers"], shape, case["keep"], case["tau"],
                                lv, list(TIERS) if len(lv) == 4 else [], 16, knn_m=case["knn"],
                                utility=UTILITY if case["utility"] else None,
                                merge=(10, 64) if case["merge"] else None, shared_prefix=case["shared"])
    return s


# ------------------------------------------------------------------ one pass
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "score":
        R.rift_score_tiles(s["tokens"], s["bank"], case["keep"], 0.6, s["key"], s["sim"], s["score"], s["u"], s["order"],
                           s["n_keep"], s["ws"], knn_m=case["knn"])
        return {"key": s["key"], "sim": s["sim"], "score": s["score"], "u": s["u"], "order": s["order"],
                "n_keep": s["n_keep"]}
    if kind == "pack":
        R.rift_select_tokens(s["key"], case["n_tiles"], case["n_v"], s["kept"], s["budgets"], case["n_keep"], s["offs"],
                             s["sel"], s["st1"])
        R.rift_compact(s["tokens"], s["kept"], s["offs"], s["sel"], case["n_keep"], s["sys"], s["qry"], s["packed"],
                       s["cu"], s["pos"], s["st2"], shared_prefix=case["shared"])
        return {k: s[k] for k in ("offs", "sel", "packed", "cu", "pos", "st1", "st2")}
    if kind == "merge":
        R.rift_merge_context(s["tokens"], s["kept"], s["offs"], s["sel"], s["coffs"], case["n_keep"], s["rows"],
                             s["status"], s["ws"])
        return {"rows": s["rows"], "status": s["status"]}
    if kind == "prefill":
        R.rift_prefill(s["cfg"], s["layers"], s["x"], s["cu"], s["pos"], s["n_seq"], s["longest"], s["hidden"], s["ws"],
                       kv_cache=s["kv"], n_prefix=s["pre"])
        return {"hidden": s["hidden"], "kv": s["kv"]}
    if kind == "decode":
        R.rift_decode_step(s["cfg"], s["layers"], s["x"], s["cu"], s["total"], s["longest"], s["kv"], s["kv_new"],
                           case["step"], s["hidden"], s["ws"], n_prefix=s["pre"])
        return {"hidden": s["hidden"], "kv_new": s["kv_new"]}
    q = s["query"]
    q.run()
    return {"hidden": q.hidden, "key": q.token_key, "order": q.tile_order, "offs": q.sel_offsets,
            "sel": q.sel_idx[:q.n_dominant], "cu": q.cu_seqlens, "pos": q.position_ids}


# ------------------------------------------------------------------ what a pass cannot do without
def _element(case):
    return 4 if case["dt"] == "f32" else 2


def _score_work(case):
    n, d, nq = case["n_tiles"] * case["n_v"], case["d"], 1 + case["n_bg"]
    by = n * d * _element(case) + nq * d * _element(case) + 8 * n + (4 * n * nq if case.get("sims", True) else 0)
    fl = 4 * n * d + (2 * n * d * nq if case.get("sims", True) else 0)
    if case["knn"]:
        fl += 2 * n * d + case["n_tiles"] ** 2 * d
    return by, fl


def _pack_work(case, n_keep):
    pre, lens = _sequences(dict(case, n_keep=n_keep))
    rows = pre + sum(lens)
    vision = sum(_budgets(case, n_keep))
    row = case["d"] * _element(case)
    return 8 * n_keep * case["n_v"] + (vision + case["n_sys"] + case["n_qry"] + rows) * row + 8 * rows + 4 * vision


def _merge_work(case, n_keep):
    by = fl = 0
    row = case["d"] * _element(case)
    for b in _budgets(case, n_keep):
        k = min(b * 10 // 64, case["n_v"] - b)
        r = case["n_v"] - (b - k)
        if k:
            by += (r + k) * row
            fl += 2 * (r - k) * k * case["d"] * (k > 1) + r * case["d"]
    return max(by, 1), fl


def _prefill_work(case, pre, lens):
    rows, d, f, e = pre + sum(lens), case["d"], case["ffn"], _element(case)
    keys = pre * (pre + 1) // 2 + sum(n * pre + n * (n + 1) // 2 for n in lens)
    fl = case["layers"] * (2 * rows * (4 * d * d + 3 * d * f) + 4 * d * keys)
    by = case["layers"] * ((4 * d * d + 3 * d * f + 2 * d) * e + (2 * rows * d * e if case.get("kv") else 0))
    return by + rows * d * (e + 4), fl


def work(case):
    kind, d = case["kind"], case["d"]
    if kind == "score":
        by, fl = _score_work(case)
    elif kind == "pack":
        by, fl = _pack_work(case, case["n_keep"]), 0
    elif kind == "merge":
        by, fl = _merge_work(case, case["n_keep"])
    elif kind == "prefill":
        by, fl = _prefill_work(case, *_sequences(case))
    elif kind == "decode":
        pre, lens = _sequences(case)
        n, f = case["n_keep"], case["ffn"]
        keys = sum(pre + x + case["step"] + 1 for x in lens)
        stored = pre + sum(lens) + n * (case["step"] + 1)      # each cached row once, the shared ones too
        by = case["layers"] * ((4 * d * d + 3 * d * f) * 2 + stored * d * 4) + n * d * 6
        fl = case["layers"] * (2 * n * (4 * d * d + 3 * d * f) + 4 * d * keys)
    else:
        keep = case["keep"] or max(1, case["n_tiles"] // 4)    # threshold mode keeps what passes: taken as a quarter
        c = dict(case, n_keep=keep)
        if case["utility"]:
            c["levels"] = "288"
        by, fl = _score_work(case)
        by += _pack_work(c, keep)
        if case["merge"]:
            m = _merge_work(c, keep)
            by, fl = by + m[0], fl + m[1]
        p = _prefill_work(c, *_sequences(c))
        by, fl = by + p[0], fl + p[1]
    return {"bytes": by, "flops": fl}


# ------------------------------------------------------------------ how far another correct implementation may be
def tolerance(case):
    kind = case["kind"]
    if kind in ("pack", "merge"):
        return "exact"     # indices and copied rows; contextual rows are defined bit for bit
    if kind == "score":
        return {"rel": 2e-6, "max": 1e-4, "differ": 0.0}    # float32 cosines; the keys and ranks are exact
    if case["dt"] == "f32":
        return {"rel": 1e-6, "max": 1e-4, "differ": 0.0}
    if kind == "query" and case["layers"] > 4:
        return {"rel": 2.5e-2, "max": 0.5, "differ": 0.0}
    return {"rel": 1e-2, "max": 0.1, "differ": 0.0}


# ------------------------------------------------------------------ the same in 64 bits
def _exact_score(tokens, bank, knn):
    n_tiles, n_v, d = tokens.shape
    q = bank.double()
    w = q[0] - q[1:].mean(dim=0) if q.shape[0] > 1 else q[0]
    w = w.float().double()
    key, sim = [], []
    emb = torch.empty(n_tiles, d, dtype=torch.float64, device=tokens.device)
    for t in range(n_tiles):
        x = tokens[t].double()
        nrm = x.norm(dim=1)
        key.append((x @ w) / nrm)
        sim.append((x @ q.t().contiguous()) / nrm[:, None])
        emb[t] = (x / nrm[:, None]).sum(dim=0)
    key = torch.stack(key)
    s = key.mean(dim=1)
    if knn:
        e = emb.float().double()
        e = e / e.norm(dim=1, keepdim=True)
        c = e @ e.t().contiguous()
        c.fill_diagonal_(-2.0)
        m = min(knn, n_tiles - 1)
        if m > 0:
            s = (s + s[c.topk(m, dim=1).indices].sum(dim=1)) / (1 + m)
    u = (s - s.min()) / (s.max() - s.min()) if n_tiles > 1 else torch.ones_like(s)
    return key, torch.cat(sim), s, u


def _rms(x, g):
    return x * torch.rsqrt(x.square().mean(dim=1, keepdim=True) + 1e-6) * g.double()


def _rope(x, pos):
    half = x.shape[-1] // 2
    theta = 10000.0 ** (-torch.arange(half, dtype=torch.float64, device=x.device) / half)
    a = pos.double()[:, None] * theta
    c, s = a.cos()[:, None], a.sin()[:, None]
    x1, x2 = x[..., :half], x[..., half:]
    return torch.cat([x1 * c - x2 * s, x2 * c + x1 * s], dim=-1)


def _attend(q, k, v, first):
    """q [n, H, hd] at positions first.. against keys and values [m, H, hd]."""
    qh, kh, vh = (t.transpose(0, 1).contiguous() for t in (q, k, v))
    sc = torch.matmul(qh, kh.transpose(1, 2).contiguous()) / math.sqrt(q.shape[-1])
    i = first + torch.arange(q.shape[0], device=q.device)
    sc.masked_fill_(torch.arange(k.shape[0], device=q.device)[None, :] > i[:, None], -math.inf)
    return torch.matmul(sc.softmax(dim=-1), vh).transpose(0, 1).reshape(q.shape[0], -1)


def _mlp(x, w):
    h = _rms(x, w["g_ffn"])
    a = torch.nn.functional.silu(h @ w["w_gate"].double().t()) * (h @ w["w_up"].double().t())
    return x + a @ w["w_down"].double().t()


def _exact_prefill(x, layers, heads, pre, cu, pos):
    x = x.double()
    kv = []
    for w in layers:
        h = _rms(x, w["g_attn"])
        q, k, v = ((h @ w[n].double().t()).reshape(x.shape[0], heads, -1) for n in ("wq", "wk", "wv"))
        q, k = _rope(q, pos), _rope(k, pos)
        kv.append(torch.stack([k.reshape(x.shape), v.reshape(x.shape)]))
        o = torch.empty_like(x)
        for i in range(len(cu) - 1):
            a, b = int(cu[i]), int(cu[i + 1])
            p = pre if i else 0
            kk, vv = (torch.cat([t[:p], t[a:b]]) for t in (k, v))
            o[a:b] = _attend(q[a:b], kk, vv, p)
        x = _mlp(x + o @ w["wo"].double().t(), w)
    return x, torch.stack(kv)


def _exact_decode(s):
    case = s["case"]
    x, kv_new, pre, step = s["x"].double(), s["kv_new"].double(), s["pre"], case["step"]
    cu = s["cu"].tolist()[1 if pre else 0:]
    pos = torch.tensor([pre + cu[i + 1] - cu[i] + step for i in range(len(cu) - 1)], device="cuda")
    for l, w in enumerate(s["layers"]):
        h = _rms(x, w["g_attn"])
        q, k, v = ((h @ w[n].double().t()).reshape(x.shape[0], case["heads"], -1) for n in ("wq", "wk", "wv"))
        q, k = _rope(q, pos), _rope(k, pos)
        kv_new[l, 0, :, step], kv_new[l, 1, :, step] = k.reshape(x.shape), v.reshape(x.shape)
        o = torch.empty_like(x)
        for i in range(x.shape[0]):
            a, b = cu[i], cu[i + 1]
            kk, vv = (torch.cat([s["kv"][l, j, :pre].double(), s["kv"][l, j, a:b].double(), kv_new[l, j, i, :step + 1]])
                      .reshape(-1, case["heads"], case["d"] // case["heads"]) for j in range(2))
            o[i:i + 1] = _attend(q[i:i + 1], kk, vv, kk.shape[0] - 1)
        x = _mlp(x + o @ w["wo"].double().t(), w)
    return {"hidden": x, "kv_new": kv_new}


def _exact_merge(s):
    case, out = s["case"], []
    offs, coffs, kept = s["offs"].tolist(), s["coffs"].tolist(), s["kept"].tolist()
    for i, tile in enumerate(kept):
        k = coffs[i + 1] - coffs[i]
        if not k:
            continue
        left = torch.ones(case["n_v"], dtype=torch.bool, device="cuda")
        left[s["sel"][offs[i]:offs[i + 1]].long()] = False
        x = s["tokens"][tile][left].double()
        t = torch.arange(k, device="cuda") * x.shape[0] // k
        y = x[t] / x[t].norm(dim=1, keepdim=True)
        to = (x @ y.t().contiguous()).argmax(dim=1)
        to[t] = torch.arange(k, device="cuda")
        acc = torch.zeros(k, case["d"], dtype=torch.float64, device="cuda").index_add_(0, to, x)
        out.append(acc / torch.bincount(to, minlength=k)[:, None])
    return {"rows": torch.cat(out) if out else s["rows"].double(), "status": None}


def exact(case, seed):
    kind = case["kind"]
    if kind == "pack" or (kind == "query" and (case["layers"] > 4 or case["merge"] or case["utility"] or not case["keep"])):
        return None
    s = prepare(case, seed)
    if kind == "score":
        key, sim, score, u = _exact_score(s["tokens"], s["bank"], case["knn"])
        return {"key": key.reshape(-1), "sim": sim if case["sims"] else None, "score": score, "u": u, "order": None,
                "n_keep": None}
    if kind == "merge":
        return _exact_merge(s)
    if kind == "decode":
        return _exact_decode(s)
    if kind == "prefill":
        hidden, kv = _exact_prefill(s["x"], s["layers"], case["heads"], s["pre"], s["cu"].tolist(), s["pos"])
        return {"hidden": hidden, "kv": kv if case["kv"] else None}
    key, _, score, _ = _exact_score(s["tokens"], s["bank"], case["knn"])
    kept = score.argsort(descending=True)[:case["keep"]].tolist()
    rows, pre = [], case["n_sys"] if case["shared"] else 0
    if pre:
        rows.append(s["sys"])
    for tile, b in zip(kept, _budgets(case, len(kept))):
        best = key[tile].topk(b).indices.sort().values
        rows += ([] if pre else [s["sys"]]) + [s["tokens"][tile][best], s["qry"]]
    _, _, cu, pos = _cu_pos(dict(case, n_keep=len(kept)))
    hidden, _ = _exact_prefill(torch.cat(rows), s["layers"], case["heads"], pre, cu.tolist(),
                               torch.from_numpy(pos).cuda())
    return {"hidden": hidden, "key": key.reshape(-1), "order": None, "offs": None, "sel": None, "cu": None, "pos": None}
