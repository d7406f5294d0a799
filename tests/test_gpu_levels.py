"""GPU parity of the level-at-a-time build (dt_expand_level / dt_finish_tree) against the oracle.

A toy draft model (a seeded function from a token string to a logit row) sits between the levels, as a real
one would: each call's rows are computed from the strings of the nodes the previous call reported."""
import numpy as np
import pytest

import dt_synth
from oracle import ref
from tests._brute import toy_logits
from tests._cases import TREE_MARGIN, assert_tree_equal

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def toy_logits_3(seed, string, V):
    return toy_logits(seed, string, V, sigma=3.0)


def few_viable(seed, string, V):
    """A row of the toy model with few viable tokens: enough for every k near the root; below, none or one on every other level, and three to eight
    on those between (which levels, by the seed)."""
    x = toy_logits(seed, string, V, sigma=3.0)
    r = np.random.default_rng([seed, 7, len(string)] + [t + 1 for t in string])
    n = 32 if len(string) < 2 else int(r.integers(0, 2)) if (len(string) + seed) % 2 else int(r.integers(3, 9))
    keep = r.permutation(V)[:n]
    row = np.full(V, -np.inf, np.float32)
    row[keep] = x[keep]
    return row


def drive(params, prefix_len, V, bf16, seed, flags=0, twice=False, rows=toy_logits_3, again={}, state=None, other=False, last=0):
    """again: levels; behind each one's call the calls from that many levels back on are made again, with the same logits.  other: and that level's
    first call has other logits.  last: that level's call is made again before the tree is finished.  Returns the numbers of
    nodes of every level, sequence by sequence."""
    import paper_2601_12212_amd as dt
    B = len(params)
    KR = max(p[2] for p in params)
    TT_cap = max(p[0] for p in params)
    max_d = max(p[1] for p in params)
    i32 = dict(dtype=torch.int32, device="cuda")
    d_params = torch.tensor(params, **i32)
    d_plen = torch.tensor(prefix_len, **i32)
    if state is None:
        state = torch.full((dt.dt_level_state_bytes(B),), 0xEE, dtype=torch.uint8, device="cuda")   # never cleared
    ws = torch.empty(dt.dt_workspace_bytes(B, B * KR, V, TT_cap, 1, 1), dtype=torch.uint8, device="cuda")
    n_exp = torch.full((B,), -5, **i32)
    e_tok = torch.full((B, 32), -5, **i32); e_par = torch.full((B, 32), -5, **i32)
    e_row = torch.full((B, 32), -5, **i32); e_pos = torch.full((B, 32), -5, **i32)
    e_mask = torch.zeros((B, 32, 4), dtype=torch.int64, device="cuda")

    def fn(b, s):
        x = rows(seed * 100 + b, s, V)
        return dt_synth.bf16_bits_to_f32(dt_synth.f32_to_bf16_bits(x)) if bf16 else x

    rows_all = [np.zeros((1 + (d - 1) * k, V), np.float32) for (TT, d, k) in params]
    strings = [{0: [()]} for _ in range(B)]
    got_levels = [dict() for _ in range(B)]
    given = {}
    rng = np.random.default_rng(seed)
    for level in range(1, max_d + 1):
        R = 1 if level == 1 else KR
        logits = (rng.standard_normal((B * R, V)) * 50).astype(np.float32)      # rows nobody may look at
        for b, (TT, d, k) in enumerate(params):
            for s, st in enumerate(strings[b].get(level - 1, [])):
                row = fn(b, st)
                logits[b * R + s] = row
                if level <= d:
                    rows_all[b][0 if level == 1 else 1 + (level - 2) * k + s] = row
        dev = torch.from_numpy(logits).cuda()
        if bf16:
            dev = dev.to(torch.bfloat16)
        given[level] = dev
        calls = [(level, dev.flip(-1)), (level, dev)] if twice and level < min(p[1] for p in params) else [(level, dev)]
        if level in again:
            calls[0] = (level, dev.flip(-1) if other else dev)
            calls += [(l, given[l]) for l in range(max(1, level - again[level]), level + 1)]
        for l, x in calls:
            dt.dt_expand_level(l, d_params, x.contiguous(), KR, d_plen, TT_cap, state, n_exp, e_tok, e_par, e_row, e_pos, e_mask,
                               ws, flags=flags)
        torch.cuda.synchronize()
        for b in range(B):
            n = int(n_exp[b])
            tok, par = e_tok[b, :n].cpu().numpy(), e_par[b, :n].cpu().numpy()
            prev = strings[b].get(level - 1, [])
            strings[b][level] = [(prev[par[s]] if par[s] >= 0 else ()) + (int(tok[s]),) for s in range(n)]
            got_levels[b][level] = dict(tokens=tok, parent_slot=par, rows=e_row[b, :n].cpu().numpy(),
                                        pos=e_pos[b, :n].cpu().numpy(),
                                        mask=e_mask[b, :n].cpu().numpy().view(np.uint64))
    # finish
    if last:
        dt.dt_expand_level(last, d_params, given[last].contiguous(), KR, d_plen, TT_cap, state, n_exp, e_tok, e_par, e_row, e_pos, e_mask, ws, flags=flags)
    n_nodes = torch.zeros(B, **i32)
    mk = lambda dtype: torch.zeros((B, TT_cap), dtype=dtype, device="cuda")
    tokens, parents, depth, src_row = mk(torch.int32), mk(torch.int32), mk(torch.int32), mk(torch.int32)
    score, logp = mk(torch.float32), mk(torch.float32)
    anc = torch.zeros((B, TT_cap, 2), dtype=torch.int64, device="cuda")
    roots = torch.tensor([100 + b for b in range(B)], **i32)
    dt.dt_finish_tree(d_params, V, roots, TT_cap, state, n_nodes, tokens, parents, depth, score, logp, src_row, anc,
                      flags=flags)
    torch.cuda.synchronize()
    for b, (TT, d, k) in enumerate(params):
        host = dt_synth.f32_to_bf16_bits(rows_all[b]) if bf16 else rows_all[b]
        want = ref.build_tree(host, TT, d, k, 100 + b, with_levels=True, early_stop=bool(flags))
        assert want["min_margin"] >= TREE_MARGIN, ("pick another seed", b, want["min_margin"])
        N = int(n_nodes[b])
        got = dict(n_nodes=N, tokens=tokens[b, :N].cpu().numpy(), parents=parents[b, :N].cpu().numpy(),
                   depth=depth[b, :N].cpu().numpy(), src_row=src_row[b, :N].cpu().numpy(),
                   score=score[b, :N].cpu().numpy(), logp=logp[b, :N].cpu().numpy(),
                   anc_mask=anc[b, :N].cpu().numpy().view(np.uint64))
        assert_tree_equal(got, want, "seq %d" % b)
        for level in range(1, max_d + 1):
            g = got_levels[b][level]
            if level >= d or TT == 1:
                assert len(g["tokens"]) == 0, (b, level)
                continue
            w = want["levels"][level]
            assert np.array_equal(g["tokens"], w["tokens"]), (b, level)
            assert np.array_equal(g["parent_slot"], w["parent_slot"]), (b, level)
            assert np.array_equal(g["rows"], w["rows"]), (b, level)
            assert np.array_equal(g["mask"], w["mask"]), (b, level)
            assert (g["pos"] == prefix_len[b] + level).all()
    return [[len(got_levels[b][level]["tokens"]) for level in range(1, max_d + 1)] for b in range(B)]


def test_level_by_level_fp32_ragged_batch():
    drive([(30, 4, 3), (60, 6, 4), (1, 3, 2), (12, 1, 5), (128, 8, 2), (20, 3, 8)], [5, 0, 9, 1000, 77, 3], V=300,
          bf16=False, seed=1)


def test_level_by_level_with_the_token_count_exit():
    # the draft model's loop ends early: levels past the exit report no node, the rows handed in for them are
    # ignored, and the finished tree is the one-shot tree under the same flag
    import paper_2601_12212_amd as dt
    drive([(5, 3, 8), (12, 5, 4), (30, 4, 3), (60, 6, 10), (128, 3, 3), (1, 4, 4), (40, 8, 2)], [3, 0, 9, 100, 77, 5, 6],
          V=300, bf16=False, seed=4, flags=dt.DT_TREE_EARLY_STOP)


def test_level_by_level_bf16_wide_levels():
    drive([(96, 4, 16), (64, 3, 32), (40, 5, 6)], [11, 12, 13], V=4099, bf16=True, seed=2)


@pytest.mark.parametrize("k", [2, 16, 17, 22, 23, 32])
def test_level_by_level_to_the_deepest_level(k):
    # each level starts from what the one before handed on, the last ones where the state's rows just leave room for it; and from the
    # row results alone where a level is asked for a second time, with other logits
    for d in (3, 4, 8):
        drive([(100, d, k), (37, 8, max(2, k - 3))], [5, 0], V=300, bf16=False, seed=1)
        drive([(100, d, k), (37, d, max(2, k - 3))], [5, 0], V=300, bf16=False, seed=1, twice=True)


FEW = [(100, 8), (60, 8), (90, 7)]


@pytest.mark.parametrize("back", [0, 1, 3, 7])
@pytest.mark.parametrize("k,seed", [(4, 1), (12, 2), (20, 1), (32, 1)])
def test_levels_asked_for_again(k, seed, back):
    # levels of fewer nodes than k, more or fewer than the level before: a level asked for again starts from the nodes of the one before it, however
    # many a later call has chosen
    for level in range(2, 9):
        counts = drive([(TT, d, k) for TT, d in FEW], [5, 0, 9], V=300, bf16=False, seed=seed, rows=few_viable, again={level: back})
        assert any(c[6] > c[5] > 0 for c in counts) and any(0 < c[6] < c[5] for c in counts), counts


@pytest.mark.parametrize("k", [8, 20])
def test_a_state_that_an_earlier_step_has_left(k):
    # trees that the token count ends at their first or second level, on what trees of three and more levels have handed on
    import paper_2601_12212_amd as dt
    state = torch.full((dt.dt_level_state_bytes(2),), 0xEE, dtype=torch.uint8, device="cuda")
    for d in (3, 4, 8):
        drive([(100, d, k), (90, d, 3)], [5, 0], V=300, bf16=False, seed=1, state=state)
        drive([(5, 8, k), (12, 8, 3)], [5, 0], V=300, bf16=False, seed=4, state=state, flags=dt.DT_TREE_EARLY_STOP)
        drive([(100, d, k), (90, d, 3)], [5, 0], V=300, bf16=False, seed=1, state=state)
        drive([(90, 8, k), (90, 8, 3)], [5, 0], V=300, bf16=False, seed=3, state=state, rows=few_viable)


@pytest.mark.parametrize("back", [0, 1, 3, 7])
@pytest.mark.parametrize("k,seed", [(4, 1), (12, 2), (20, 1), (32, 1)])
def test_levels_asked_for_again_with_other_logits(k, seed, back):
    # the call that counts finds every node's row, also where a call between has chosen fewer nodes than the level before, the last level's among them
    for level in range(2, 9):
        drive([(TT, d, k) for TT, d in FEW], [5, 0, 9], V=300, bf16=False, seed=seed, rows=few_viable, again={level: back}, other=True)


@pytest.mark.parametrize("last", [1, 2, 5, 7, 8])
@pytest.mark.parametrize("k,seed,few", [(3, 1, False), (16, 1, False), (17, 1, False), (4, 1, True), (12, 2, True), (20, 1, True)])
def test_a_tree_finished_behind_a_level_asked_for_again(k, seed, few, last):
    # what later levels have left does not follow from that one any more; the last one's does
    if few:
        drive([(TT, d, k) for TT, d in FEW], [5, 0, 9], V=300, bf16=False, seed=seed, rows=few_viable, last=min(last, 7))
    else:
        drive([(100, 8, k), (37, 8, max(2, k - 3)), (9, 2, 4), (5, 1, 2)], [5, 0, 9, 1], V=300, bf16=False, seed=seed, last=last)


# vocabularies of both row paths: held by 1,024 threads with the log-sum-exps apart, two passes of one chunk to a workgroup;
# sequences that end before the others leave rows of nodes that do not exist
@pytest.mark.parametrize("V,bf16", [(20000, True), (50001, True), (50001, False), (128256, True)])
def test_level_by_level_of_large_vocabularies(V, bf16):
    drive([(40, 3, 12), (1, 2, 2), (30, 4, 5), (9, 1, 4), (25, 2, 12), (33, 5, 3)], [5, 0, 9, 1000, 77, 3], V=V, bf16=bf16, seed=1)


# a level's nodes chosen in the launch of its rows: every kernel of rows that does it, at the ends of its vocabularies; one and four candidates to a lane, and the
# first width that has a launch of its own (17)
@pytest.mark.parametrize("V,bf16", [(2048, True), (8192, True), (8193, False), (16384, True), (16385, False), (32769, True)])
@pytest.mark.parametrize("k", [1, 8, 9, 16, 17])
def test_levels_chosen_beside_their_rows(V, bf16, k):
    drive([(60, 4, k), (1, 2, 2), (33, 3, max(1, k - 7)), (20, 1, k), (9, 2, 1)], [5, 0, 9, 1000, 77], V=V, bf16=bf16, seed=1)


def test_a_level_whose_waiting_workgroups_find_no_room_in_the_grid():
    # 16 million rows of 256 threads are within 2^32 threads, with a workgroup more to each of a million sequences they are not: the level's nodes are then
    # chosen by a launch of their own.  All but three of the sequences draft nothing.
    import paper_2601_12212_amd as dt
    if torch.cuda.mem_get_info()[0] < 95e9:
        pytest.skip("needs 80 GB of device memory")
    B, V, R, live = 1000000, 8, 16, [0, 77777, 999999]
    gen = torch.Generator("cuda").manual_seed(3)
    logits = [torch.randn((B * r, V), generator=gen, device="cuda") for r in (1, R)]
    limits = torch.ones((B, 3), dtype=torch.int32, device="cuda")
    limits[live] = torch.tensor([30, 3, 4], dtype=torch.int32, device="cuda")

    def levels(limits, logits):
        n = len(limits)
        state = torch.empty(dt.dt_level_state_bytes(n), dtype=torch.uint8, device="cuda")
        ws = torch.empty(dt.dt_workspace_bytes(n, n * R, V, 30, 1, 1), dtype=torch.uint8, device="cuda")
        out = []
        for l, x in enumerate(logits):
            n_exp = torch.zeros(n, dtype=torch.int32, device="cuda")
            exp = [torch.zeros((n, 32), dtype=torch.int32, device="cuda") for _ in range(4)] + [torch.zeros((n, 32, 4), dtype=torch.int64, device="cuda")]
            dt.dt_expand_level(l + 1, limits, x, R, None, 30, state, n_exp, *exp, ws)
            out += [n_exp] + exp
        return out

    few = levels(limits[live], [x.view(B, -1, V)[live].reshape(-1, V) for x in logits])
    many = levels(limits, logits)
    assert few[0].tolist() == few[6].tolist() == [4, 4, 4] and int(many[6].sum()) == 12
    for a, b in zip(few, many):
        assert torch.equal(a, b[live])
    del many, logits
    torch.cuda.empty_cache()


def test_level_by_level_of_launches_that_take_two_chunks_to_a_workgroup():
    # 33 sequences of 32 rows of 16 chunks, 16,896 in all, most of them of nodes that do not exist
    drive([(30, 3, 4)] * 7 + [(70, 3, 32)] + [(5, 2, 2)] * 25, list(range(33)), V=61441, bf16=True, seed=1)


def test_the_level_loop_can_be_captured_and_replayed():
    # The d-level loop with the finish call as one HIP graph (the draft model's passes would be nodes in
    # between; here each level's logits sit in their own buffer).  Replayed several times with the outputs
    # wiped and eager work in between; every replay must reproduce the eager result.
    import paper_2601_12212_amd as dt
    params, V, KR, TT_cap, d = [(40, 4, 5), (25, 3, 4)], 1000, 5, 40, 4
    B = len(params)
    i32 = dict(dtype=torch.int32, device="cuda")
    rng = np.random.default_rng(3)
    d_params = torch.tensor(params, **i32)
    level_logits = [torch.from_numpy((rng.standard_normal((B * (1 if l == 1 else KR), V)) * 3).astype(np.float32)).cuda()
                    for l in range(1, d + 1)]
    state = torch.zeros(dt.dt_level_state_bytes(B), dtype=torch.uint8, device="cuda")
    ws = torch.empty(dt.dt_workspace_bytes(B, B * KR, V, TT_cap, 1, 1), dtype=torch.uint8, device="cuda")
    n_exp = torch.zeros(B, **i32)
    ex = [torch.zeros((B, 32), **i32) for _ in range(4)]
    e_mask = torch.zeros((B, 32, 4), dtype=torch.int64, device="cuda")
    roots = torch.tensor([1, 2], **i32)
    outs = [torch.zeros(B, **i32)] + [torch.zeros((B, TT_cap), **i32) for _ in range(3)] + \
           [torch.zeros((B, TT_cap), dtype=torch.float32, device="cuda") for _ in range(2)] + \
           [torch.zeros((B, TT_cap), **i32), torch.zeros((B, TT_cap, 2), dtype=torch.int64, device="cuda")]

    def run():
        for l in range(1, d + 1):
            dt.dt_expand_level(l, d_params, level_logits[l - 1], KR, None, TT_cap, state, n_exp, *ex, e_mask, ws)
        dt.dt_finish_tree(d_params, V, roots, TT_cap, state, *outs)

    run()
    torch.cuda.synchronize()
    eager = [o.clone() for o in outs]
    assert int(eager[0].min()) > 1
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        run()                                      # first touches on the capture stream
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            run()
    for rep in range(3):
        for o in outs:
            o.fill_(-3)
        state.fill_(rep)                           # the state carries nothing from one step to the next
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        N = eager[0]
        for o, e in zip(outs, eager):
            if o.dim() == 1:
                assert torch.equal(o, e), rep
            else:
                for b in range(B):
                    assert torch.equal(o[b, :int(N[b])], e[b, :int(N[b])]), (rep, b)
        (torch.ones(1000, device="cuda") * 2).sum().item()    # eager work between replays
