"""Workloads by which the speed of this library is judged: what a decoder that drafts trees calls, over the range of
sizes it meets.

A case is a dict of plain values.  Every kind of case goes through the public entry points only (the Step class of
paper_2601_12212_amd.step and the dt_* functions of the package):

  step       one speculative step: build the draft tree, attend the tree tokens, accept (Step.run, or the same three
             calls captured once in a HIP graph and replayed, as a serving loop does)
  turn       a whole decoding turn whose tree limits the policy chooses on the device: dt_policy_step, the three calls
             of the step, dt_commit over all layers, dt_reward_step.  The host never learns the limits, so the buffers
             and launches are sized for the widest action.
  levels     the tree built level by level, as when the draft model runs in between: dt_expand_level, dt_finish_tree
  attention  the target's verification pass: dt_tree_attention once per layer, each layer with its own K/V cache
  rows       row top-k and log-sum-exp on its own: dt_topk_rows

Per-sequence sizes (tree limits, prefix lengths) are drawn from the case's ranges with its "mix" number, so they belong
to the case; prepare()'s seed only makes values.  Logits are N(0, 3) in the case's type, a node's target row is the draft
row it owns plus N(0, 1) (acceptance is then partial, as in use), Q/K/V are N(0, 1).
"""
import math
import random

import torch

import paper_2601_12212_amd as dt
from paper_2601_12212_amd.step import Step

MODES = {"greedy": dt.DT_ACCEPT_GREEDY, "stochastic": dt.DT_ACCEPT_STOCHASTIC, "sampled": dt.DT_ACCEPT_SAMPLED}
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
DEV = "cuda"

POLICY_F, POLICY_H, POLICY_INTERVAL = 3 * 4096, 128, 30   # three hidden-state vectors, the cache interval at inference


def _step(name, B, Hq, Hkv, D, V, tt, d, k, L, dtype="bf16", mode="greedy", call="step", head_major=False,
          early_stop=False, mix=0):
    c = dict(kind="step", call=call, dtype=dtype, B=B, Hq=Hq, Hkv=Hkv, D=D, V=V, tt_lo=tt[0], tt_hi=tt[1], d_lo=d[0],
             d_hi=d[1], k_lo=k[0], k_hi=k[1], L_lo=L[0], L_hi=L[1], mode=mode, head_major=head_major,
             early_stop=early_stop, mix=mix)
    return dict(name=name, **c) if name else c


def _attention(name, layers, B, Hq, Hkv, D, tt, d, k, L, head_major=False, mix=0):
    c = dict(kind="attention", dtype="bf16", layers=layers, B=B, Hq=Hq, Hkv=Hkv, D=D, tt_lo=tt[0], tt_hi=tt[1],
             d_lo=d[0], d_hi=d[1], k_lo=k[0], k_hi=k[1], L_lo=L[0], L_hi=L[1], head_major=head_major, mix=mix)
    return dict(name=name, **c) if name else c


def _levels(name, B, V, tt, d, k, mix=0):
    c = dict(kind="levels", dtype="bf16", B=B, V=V, tt_lo=tt[0], tt_hi=tt[1], d_lo=d[0], d_hi=d[1], k_lo=k[0],
             k_hi=k[1], L_lo=512, L_hi=2048, mix=mix)
    return dict(name=name, **c) if name else c


def _turn(name, layers, B, Hq, Hkv, D, V, L, mode, mix=0):
    c = dict(kind="turn", dtype="bf16", layers=layers, B=B, Hq=Hq, Hkv=Hkv, D=D, V=V, L_lo=L[0], L_hi=L[1], mode=mode,
             mix=mix)
    return dict(name=name, **c) if name else c


def _rows(name, n, V, k, dtype):
    c = dict(kind="rows", dtype=dtype, n=n, V=V, k=k)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest step there is here: one short sequence of a toy model in fp32, called eagerly
        _step("tiny_fp32", 1, 4, 4, 64, 1024, (8, 8), (3, 3), (2, 2), (128, 128), dtype="f32"),
        # the headline configuration: one sequence of the 8B shape, its step captured once and replayed
        _step("8b_b1_graph", 1, 32, 8, 128, 128256, (60, 60), (6, 6), (10, 10), (1024, 1024), call="graph"),
        # one sequence of the 13B shape (no grouped heads, small vocabulary), called eagerly
        _step("13b_b1", 1, 40, 40, 128, 32000, (64, 64), (7, 7), (8, 8), (2048, 2048)),
        # a small serving batch, every sequence with limits and a context of its own
        _step("8b_b16_ragged", 16, 32, 8, 128, 128256, (32, 96), (4, 8), (4, 12), (256, 4096), mix=4),
        # the 70B shape with long contexts, sampling with the printed acceptance rule
        _step("70b_b4_stochastic", 4, 64, 8, 128, 128256, (96, 96), (8, 8), (12, 12), (8192, 8192), mode="stochastic"),
        # a large serving batch over the whole action space
        _step("8b_b64_wide", 64, 32, 8, 128, 128256, (32, 128), (3, 8), (8, 32), (256, 4096), mix=64),
        # a few sequences of a model with 64-wide heads, seven query heads to a kv head and an odd vocabulary (rows
        # that start at any 2-byte address), verified with the distribution-preserving rule
        _step("odd_vocab_head64_sampled", 3, 14, 2, 64, 50001, (33, 64), (4, 6), (6, 12), (37, 1500), mode="sampled", mix=3),
        # a turn of two interactive users whose limits the policy sets on the device
        _turn("8b_turn_b2", 32, 2, 32, 8, 128, 128256, (300, 1100), "greedy", mix=2),
        # the headline tree, the draft model running between its levels
        _levels("8b_levels_b1", 1, 128256, (60, 60), (6, 6), (10, 10)),
        # the verification pass of one sequence through all layers
        _attention("8b_attention_b1_layers", 32, 1, 32, 8, 128, (60, 60), (6, 6), (10, 10), (1024, 1024)),
        # long contexts in a small batch, caches laid out by head
        _attention("8b_attention_b8_long", 4, 8, 32, 8, 128, (48, 96), (5, 8), (8, 16), (4096, 16384), head_major=True, mix=8),
        # row top-k of logits that were kept in fp32, odd vocabulary
        _rows("rows_f32_odd", 61, 50001, 20, "f32"),
    ]


# -------------------------------------------------------------------------------------------------- drawn cases

def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _vocab(rng):
    v = _logint(rng, 1000, 131072)
    return v if rng.random() < 0.4 else max(1024, v // 64 * 64)      # any size, or a multiple of 64 as most models have


def _span(rng, lo, hi, ragged):
    a, b = sorted((rng.randint(lo, hi), rng.randint(lo, hi)))
    return (a, b) if ragged else (b, b)


def _draw_one(rng):
    kind = rng.choices(["step", "attention", "levels", "rows", "turn"], [46, 20, 10, 14, 10])[0]
    mix = rng.randrange(1 << 20)
    if kind == "rows":
        dtype = rng.choice(["bf16", "bf16", "f32"])
        V = _vocab(rng)
        return _rows(None, _logint(rng, 1, 2000), V, rng.randint(1, 32), dtype)
    B = _logint(rng, 1, 64)
    ragged = B > 1
    tt, d, k = _span(rng, 16, 128, ragged), _span(rng, 2, 8, ragged), _span(rng, 3, 32, ragged)
    if kind == "levels":
        return _levels(None, min(B, 16), _vocab(rng), tt, d, k, mix)
    Hkv, G = rng.choice([(8, 4), (8, 8), (8, 4), (4, 7), (2, 7), (40, 1), (32, 1), (4, 4)])
    l = _logint(rng, 16, 8192)
    L = (max(1, l // rng.choice([1, 4, 16])), l) if ragged else (l, l)
    if kind == "turn":
        Hkv = min(Hkv, 8)
        return _turn(None, rng.choice([16, 32, 40]), min(B, 4), Hkv * G, Hkv, 128, _vocab(rng), (min(L[0], 1100), min(L[1], 1100)),
                     rng.choice(list(MODES)), mix)
    D = 64 if rng.random() < 0.15 else 128
    head_major = rng.random() < 0.3
    if kind == "attention":
        return _attention(None, rng.choice([1, 4, 32]), B, Hkv * G, Hkv, D, tt, d, k, L, head_major, mix)
    if rng.random() < 0.1:                                            # small steps in fp32
        return _step(None, min(B, 2), 4, 4, rng.choice([64, 128]), _logint(rng, 1000, 32000), (8, 32), (2, 5), (2, 6),
                     (16, min(L[1], 600)), dtype="f32", mode=rng.choice(list(MODES)), mix=mix)
    return _step(None, B, Hkv * G, Hkv, D, _vocab(rng), tt, d, k, L, mode=rng.choice(list(MODES)),
                 call=rng.choice(["step", "step", "graph"]), head_major=head_major, early_stop=rng.random() < 0.15, mix=mix)


def draw(rng):
    """One more case of these ranges that costs no more than the largest listed one."""
    top = work(next(c for c in listed() if c["name"] == "8b_b64_wide"))
    while True:
        c = _draw_one(rng)
        w = work(c)
        # heads that are not 128 wide, and fp32, are meant for small problems
        small = c.get("D", 128) == 128 and (c["kind"] == "rows" or c["dtype"] == "bf16")
        if w["bytes"] <= 0.8 * top["bytes"] and w["flops"] <= (0.8 * top["flops"] if small else 2e9):
            return c


# ------------------------------------------------------------------------------------------------ sizes and work

def _sizes(case):
    """Per-sequence (TT, d, k) and prefix lengths."""
    r = random.Random(case["mix"])
    params, plen = [], []
    for _ in range(case["B"]):
        if case["kind"] == "turn":
            params.append((dt.DT_TT_MAX, dt.DT_D_MAX, dt.DT_K_MAX))
        else:
            params.append((r.randint(case["tt_lo"], case["tt_hi"]), r.randint(case["d_lo"], case["d_hi"]),
                           r.randint(case["k_lo"], case["k_hi"])))
        plen.append(r.randint(case["L_lo"], case["L_hi"]))
    return params, plen


def _nodes(p):
    TT, d, k = p
    return min(TT, 1 + k + (d - 1) * k * k)


def _mean_action():
    t = dt.dt_action_table()
    return sum(a[0] for a in t) / len(t), sum(1 + (a[1] - 1) * a[2] for a in t) / len(t)


def work(case):
    e = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "rows":
        n, V, k = case["n"], case["V"], case["k"]
        return {"bytes": float(e * n * V + 8 * n * k + 4 * n), "flops": 3.0 * n * V}
    params, plen = _sizes(case)
    nbytes = flops = 0.0
    mean_tt, mean_rows = _mean_action() if case["kind"] == "turn" else (0, 0)
    for p, L in zip(params, plen):
        N, R = (mean_tt, mean_rows) if case["kind"] == "turn" else (_nodes(p), 1 + (p[1] - 1) * p[2])
        if case["kind"] in ("step", "turn", "levels"):
            nbytes += e * case["V"] * R + 44.0 * N
            flops += 3.0 * case["V"] * R
        if case["kind"] in ("step", "turn"):
            nbytes += e * case["V"] * N
            flops += (1.0 if case["mode"] == "greedy" else 3.0) * case["V"] * N
        if case["kind"] in ("step", "turn", "attention"):
            layers = case["layers"] if case["kind"] == "attention" else 1
            nbytes += layers * e * (2 * case["Hkv"] * case["D"] * (L + N) + 2 * N * case["Hq"] * case["D"])
            flops += layers * 4.0 * N * case["Hq"] * (L + N) * case["D"]
        if case["kind"] == "turn":   # two rows of every layer's K and V, moved; the policy runs once per interval
            nbytes += case["layers"] * 2 * 2 * 2 * e * case["Hkv"] * case["D"]
    if case["kind"] == "turn":
        nbytes += POLICY_F * POLICY_H * 4.0 / POLICY_INTERVAL
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Scores, log-probabilities and log-sum-exps are 32-bit sums; attention outputs in bf16 are one rounding of sums over
    # probabilities that were themselves rounded to bf16.  Which of two candidates from different rows is kept can turn
    # on the last bit of a log-sum-exp: a tie.
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.0 if case["kind"] == "rows" else 0.01}
    if case["kind"] in ("rows", "levels"):
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.0 if case["kind"] == "rows" else 0.01}
    return {"rel": 1e-2, "max": 0.1, "differ": 0.0 if case["kind"] == "attention" else 0.01}


# ------------------------------------------------------------------------------------------------------ prepare

def _normal(shape, gen, dtype, std=1.0, out=None):
    """N(0, std) in `dtype`; large tensors are filled in pieces."""
    t = torch.empty(shape, dtype=dtype, device=DEV) if out is None else out
    flat = t.view(-1)
    for i in range(0, flat.numel(), 1 << 27):
        n = min(1 << 27, flat.numel() - i)
        x = torch.randn(n, generator=gen, device=DEV)
        flat[i:i + n].copy_(x if std == 1.0 else x.mul_(std))
    return t


def _fill_targets(st, gen):
    """Target rows of the tree that the draft logits give: the node's draft row + N(0, 1), a fresh row where it owns none."""
    st.build_tree()
    for b in range(st.Bsz):
        src = st.src_row[b].long()
        rows = st.draft_logits[int(st.host_row_off[b]) + src.clamp(min=0)].float()
        fresh = torch.randn(rows.shape, generator=gen, device=DEV).mul_(3.0)
        rows = torch.where((src >= 0)[:, None], rows, fresh)
        rows += torch.randn(rows.shape, generator=gen, device=DEV)
        st.target_logits[b].copy_(rows)


def _make_step(case, gen, params, plen, TT_cap=None):
    st = Step(params, plen, case["Hq"], case["Hkv"], case["D"], case["V"], dtype=DTYPES[case["dtype"]],
              mode=MODES[case.get("mode", "greedy")], TT_cap=TT_cap, philox_seed=0x5EED,
              tree_flags=dt.DT_TREE_EARLY_STOP if case.get("early_stop") else 0, kv_head_major=case.get("head_major", False))
    _normal(None, gen, None, 3.0, out=st.draft_logits)
    st.root_token.copy_(torch.randint(0, case["V"], (st.Bsz,), generator=gen, device=DEV))
    for t in [st.q, st.k_tree, st.v_tree] + st.k_prefix + st.v_prefix:
        _normal(None, gen, None, out=t)
    return st


def _prepare_step(case, gen):
    params, plen = _sizes(case)
    st = _make_step(case, gen, params, plen)
    _fill_targets(st, gen)
    s = {"kind": "step", "st": st, "graph": None}
    if case["call"] == "graph":
        st.prepare()
        st.run_prepared(torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            st.run_prepared(torch.cuda.current_stream().cuda_stream)
    return s


def _prepare_turn(case, gen):
    params, plen = _sizes(case)
    B, nl = case["B"], case["layers"]
    table = torch.tensor(dt.dt_action_table(), dtype=torch.int32, device=DEV)
    A = table.shape[0]
    weights = [_normal((POLICY_F, POLICY_H), gen, torch.float32, POLICY_F ** -0.5), _normal((POLICY_H,), gen, torch.float32, 0.1),
               _normal((POLICY_H, POLICY_H), gen, torch.float32, POLICY_H ** -0.5), _normal((POLICY_H,), gen, torch.float32, 0.1),
               _normal((POLICY_H, A), gen, torch.float32, POLICY_H ** -0.5), _normal((A,), gen, torch.float32, 0.1)]
    feat = _normal((B, POLICY_F), gen, torch.bfloat16)
    i32 = dict(dtype=torch.int32, device=DEV)
    st = _make_step(case, gen, params, plen, dt.DT_TT_MAX)
    wsp = torch.empty(dt.dt_policy_workspace_bytes(B, POLICY_F, POLICY_H), dtype=torch.uint8, device=DEV)
    s = {"kind": "turn", "st": st, "weights": weights, "feat": feat, "table": table, "wsp": wsp,
         "cache_step": torch.zeros(B, **i32), "cached_action": torch.full((B,), -1, **i32), "action": torch.zeros(B, **i32)}
    # the limits that the target rows follow are those the policy will choose
    scratch = [torch.zeros(B, **i32), torch.full((B,), -1, **i32)]
    dt.dt_policy_step(feat, *weights, table, 1, 0, 0, 0, scratch[0], scratch[1], st.params, None, None, None, wsp)
    _fill_targets(st, gen)
    # all layers' caches with room for the accepted path; the attended layer's is the step's own
    cap = max(plen) + dt.DT_D_MAX + 1
    s["caches"] = torch.zeros((2, nl, B, cap, case["Hkv"], case["D"]), dtype=torch.bfloat16, device=DEV)
    trees = _normal((2, nl, B, st.TT_cap, case["Hkv"], case["D"]), gen, torch.bfloat16)
    ptrs = lambda ts: torch.tensor([t.data_ptr() for t in ts], dtype=torch.int64, device=DEV)
    s["trees"] = trees
    s["ktree"], s["vtree"] = ptrs(trees[0]), ptrs(trees[1])
    s["kpre"], s["vpre"] = (ptrs([s["caches"][i, l, b] for l in range(nl) for b in range(B)]).view(nl, B) for i in (0, 1))
    s["cap"] = torch.full((B,), cap, **i32)
    s["new_len"], s["next_root"] = torch.zeros(B, **i32), torch.zeros(B, **i32)
    s["reward_sum"], s["reward_avg"] = torch.zeros(B, device=DEV), torch.zeros(B, device=DEV)
    s["reward_steps"], s["interval_done"] = torch.zeros(B, **i32), torch.zeros(B, **i32)
    return s


def _prepare_levels(case, gen):
    params, plen = _sizes(case)
    B, V = case["B"], case["V"]
    d, R, TT_cap = max(p[1] for p in params), max(p[2] for p in params), max(p[0] for p in params)
    i32 = dict(dtype=torch.int32, device=DEV)
    tree = lambda dtype=torch.int32: torch.zeros((B, TT_cap), dtype=dtype, device=DEV)
    return {"kind": "levels", "d": d, "R": R, "V": V, "TT_cap": TT_cap,
            "params": torch.tensor(params, **i32), "plen": torch.tensor(plen, **i32),
            "root": torch.randint(0, V, (B,), generator=gen, device=DEV, dtype=torch.int32),
            "logits": [_normal((B * (1 if l == 0 else R), V), gen, torch.bfloat16, 3.0) for l in range(d)],
            "state": torch.zeros(dt.dt_level_state_bytes(B), dtype=torch.uint8, device=DEV),
            "ws": torch.empty(dt.dt_workspace_bytes(B, B * R, V, TT_cap, 1, 1), dtype=torch.uint8, device=DEV),
            "n_exp": torch.zeros((d, B), **i32), "exp": [torch.zeros((d, B, dt.DT_K_MAX), **i32) for _ in range(4)],
            "exp_mask": torch.zeros((d, B, dt.DT_K_MAX, 4), dtype=torch.int64, device=DEV),
            "out": [torch.zeros(B, **i32), tree(), tree(), tree(), tree(torch.float32), tree(torch.float32), tree(),
                    torch.zeros((B, TT_cap, dt.DT_MASK_WORDS), dtype=torch.int64, device=DEV)]}


def _prepare_attention(case, gen):
    params, plen = _sizes(case)
    B, Hq, Hkv, D, nl = case["B"], case["Hq"], case["Hkv"], case["D"], case["layers"]
    # the masks are those of a drafted tree; its vocabulary does not matter here
    tr = Step(params, [1] * B, 1, 1, D, 2048)
    _normal(None, gen, None, 3.0, out=tr.draft_logits)
    tr.build_tree()
    cap = max(plen)
    if case["head_major"]:
        shapes, stok, shead = [(Hkv, cap, D)] * B, D, cap * D
    else:
        shapes, stok, shead = [(L, Hkv, D) for L in plen], Hkv * D, D
    layers = []
    for _ in range(nl):
        kp = [_normal(s, gen, torch.bfloat16) for s in shapes]
        vp = [_normal(s, gen, torch.bfloat16) for s in shapes]
        ptrs = [torch.tensor([t.data_ptr() for t in ts], dtype=torch.int64, device=DEV) for ts in (kp, vp)]
        layers.append((_normal((B, tr.TT_cap, Hq, D), gen, torch.bfloat16), _normal((B, tr.TT_cap, Hkv, D), gen, torch.bfloat16),
                       _normal((B, tr.TT_cap, Hkv, D), gen, torch.bfloat16), ptrs[0], ptrs[1], kp, vp))
    return {"kind": "attention", "tr": tr, "layers": layers, "stok": stok, "shead": shead, "maxlen": cap,
            "plen": torch.tensor(plen, dtype=torch.int32, device=DEV), "scale": D ** -0.5,
            "out": torch.zeros((nl, B, tr.TT_cap, Hq, D), dtype=torch.bfloat16, device=DEV),
            "ws": torch.empty(dt.dt_workspace_bytes(B, B, 2048, tr.TT_cap, Hq, D), dtype=torch.uint8, device=DEV)}


def _prepare_rows(case, gen):
    n, V, k = case["n"], case["V"], case["k"]
    return {"kind": "rows", "k": k, "x": _normal((n, V), gen, DTYPES[case["dtype"]], 3.0),
            "val": torch.empty((n, k), dtype=torch.float32, device=DEV), "id": torch.empty((n, k), dtype=torch.int32, device=DEV),
            "lse": torch.empty(n, dtype=torch.float32, device=DEV),
            "ws": torch.empty(dt.dt_workspace_bytes(1, n, V, 8, 1, 64), dtype=torch.uint8, device=DEV)}


def prepare(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    return {"step": _prepare_step, "turn": _prepare_turn, "levels": _prepare_levels, "attention": _prepare_attention,
            "rows": _prepare_rows}[case["kind"]](case, gen)


# ---------------------------------------------------------------------------------------------------------- run

def _step_outputs(st):
    return {"n_nodes": st.n_nodes, "tokens": st.tokens, "parents": st.parents, "depth": st.depth, "score": st.score,
            "logp": st.logp, "src_row": st.src_row, "anc_mask": st.anc_mask, "out": st.out, "accept_len": st.accept_len,
            "best_node": st.best_node, "path_nodes": st.path_nodes, "out_tokens": st.out_tokens, "node_argmax": st.node_argmax}


def _run_step(s):
    if s["graph"] is not None:
        s["graph"].replay()
    else:
        s["st"].run()
    return _step_outputs(s["st"])


def _run_turn(s):
    st = s["st"]
    dt.dt_policy_step(s["feat"], *s["weights"], s["table"], POLICY_INTERVAL, 0, 0, 0, s["cache_step"], s["cached_action"],
                      st.params, s["action"], None, None, s["wsp"])
    st.run()
    dt.dt_commit(st.q, st.Hkv, st.D, s["ktree"], s["vtree"], s["kpre"], s["vpre"], st.prefix_len, s["cap"],
                 st.Hkv * st.D, st.D, st.n_nodes, st.path_nodes, st.accept_len, st.out_tokens, st.TT_cap, s["new_len"],
                 s["next_root"])
    dt.dt_reward_step(st.accept_len, 1, 0.02, s["cache_step"], s["reward_sum"], s["reward_steps"], s["reward_avg"],
                      s["interval_done"])
    out = _step_outputs(st)
    out.update({n: s[n] for n in ("action", "caches", "new_len", "next_root", "cache_step", "cached_action", "reward_sum",
                                  "reward_steps", "reward_avg", "interval_done")})
    return out


def _run_levels(s):
    for l in range(1, s["d"] + 1):
        dt.dt_expand_level(l, s["params"], s["logits"][l - 1], s["R"], s["plen"], s["TT_cap"], s["state"], s["n_exp"][l - 1],
                           *[e[l - 1] for e in s["exp"]], s["exp_mask"][l - 1], s["ws"])
    dt.dt_finish_tree(s["params"], s["V"], s["root"], s["TT_cap"], s["state"], *s["out"])
    return {"n_exp": s["n_exp"], "exp": s["exp"], "exp_mask": s["exp_mask"], "tree": s["out"]}


def _run_attention(s):
    tr = s["tr"]
    for i, (q, kt, vt, kp, vp, _, _) in enumerate(s["layers"]):
        dt.dt_tree_attention(q, kt, vt, tr.n_nodes, kp, vp, s["plen"], s["maxlen"], s["stok"], s["shead"], tr.anc_mask,
                             s["scale"], s["out"][i], s["ws"])
    return s["out"]


def _run_rows(s):
    dt.dt_topk_rows(s["x"], s["k"], s["val"], s["id"], s["lse"], s["ws"])
    return {"val": s["val"], "id": s["id"], "lse": s["lse"]}


def run(state):
    return {"step": _run_step, "turn": _run_turn, "levels": _run_levels, "attention": _run_attention,
            "rows": _run_rows}[state["kind"]](state)
