"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on the same seeded inputs.

Bars: token ids, parents, depth, src_row, ancestor masks, arg maxes, accepted paths and output tokens are
bit-exact; scores/log-probs within a few fp32 ulp per level; attention within max-abs 2e-2 (bf16) or
1e-5 (fp32).
"""
import numpy as np
import pytest

import dt_synth
from oracle import ref
from tests._cases import assert_accept_equal, assert_tree_equal, make_step, oracle_case

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev_logits(a):
    if a.dtype == np.uint16:
        return torch.from_numpy(a.view(np.int16)).cuda().view(torch.bfloat16)
    return torch.from_numpy(a).cuda()


def run_topk(x, k):
    import paper_2601_12212_amd as dt
    R, V = x.shape
    xd = dev_logits(x)
    val = torch.empty((R, k), dtype=torch.float32, device="cuda")
    idx = torch.empty((R, k), dtype=torch.int32, device="cuda")
    lse = torch.empty(R, dtype=torch.float32, device="cuda")
    ws = torch.zeros(dt.dt_workspace_bytes(1, R, V, 8, 1, 64), dtype=torch.uint8, device="cuda")
    dt.dt_topk_rows(xd, k, val, idx, lse, ws)
    torch.cuda.synchronize()
    return val.cpu().numpy(), idx.cpu().numpy(), lse.cpu().numpy()


def check_topk(x, k):
    val, idx, lse = run_topk(x, k)
    wval, widx, wlse = ref.topk_rows(x, k)
    assert np.array_equal(idx, widx)
    assert np.array_equal(val, wval)
    fin = np.isfinite(wlse)
    assert np.array_equal(np.isneginf(lse), np.isneginf(wlse))
    assert (np.abs(lse[fin] - wlse[fin]) <= 4e-6 * np.maximum(1.0, np.abs(wlse[fin]))).all()


# ------------------------------------------------------------------------------------ A1 row kernels

@pytest.mark.parametrize("V,k,bf16", [(1024, 2, False), (1000, 10, True), (4097, 32, True), (32000, 8, True),
                                       (128256, 10, True), (128256, 16, True), (128256, 20, True), (128256, 32, True), (50001, 12, False),
                                       (33, 32, True), (8192 * 3 + 5, 1, True),
                                       (5, 3, True), (7, 7, False), (8, 8, True), (15, 4, True), (16, 16, False)])
def test_topk_rows_random(V, k, bf16):
    rng = np.random.default_rng(V + k)
    x = (rng.standard_normal((7, V)) * 3).astype(np.float32)
    check_topk(dt_synth.f32_to_bf16_bits(x) if bf16 else x, k)


def test_topk_rows_ties_constant_rows_and_minus_inf():
    V = 20000
    rng = np.random.default_rng(1)
    x = np.zeros((6, V), np.float32)                          # row 0: all equal -> ids 0..k-1
    x[1] = rng.integers(-2, 3, V)                             # heavy ties
    x[2] = -np.inf; x[2, [7, 19999, 4096]] = [1.0, 1.0, 2.0]  # three viable entries
    x[3] = -np.inf                                            # nothing viable
    x[4] = np.arange(V)                                       # ascending: the top sits in the last chunk
    x[5] = -np.arange(V)                                      # descending: the top sits in the first chunk
    for k in (1, 5, 32):
        check_topk(x, k)
        check_topk(dt_synth.f32_to_bf16_bits(x), k)           # bf16 rounding makes rows 4/5 tie in runs


def test_topk_rows_unaligned_row_stride_takes_the_scalar_path():
    import paper_2601_12212_amd as dt
    rng = np.random.default_rng(2)
    V, stride, R, k = 5003, 5005, 4, 6
    buf = dt_synth.f32_to_bf16_bits((rng.standard_normal((R, stride)) * 3).astype(np.float32))
    xd = dev_logits(buf)[:, :V]
    val = torch.empty((R, k), dtype=torch.float32, device="cuda")
    idx = torch.empty((R, k), dtype=torch.int32, device="cuda")
    lse = torch.empty(R, dtype=torch.float32, device="cuda")
    ws = torch.zeros(dt.dt_workspace_bytes(1, R, V, 8, 1, 64), dtype=torch.uint8, device="cuda")
    dt.dt_topk_rows(xd, k, val, idx, lse, ws)
    torch.cuda.synchronize()
    wval, widx, wlse = ref.topk_rows(np.ascontiguousarray(buf[:, :V]), k)
    assert np.array_equal(idx.cpu().numpy(), widx) and np.array_equal(val.cpu().numpy(), wval)


# ------------------------------------------------------------------------- whole step on the configs

# Attention bars.  The target's bar: max-abs 2e-2 (bf16) / 1e-5 (fp32).  Our own, tighter one for bf16: both
# sides round their result to bf16 once (half an ulp each, an ulp being at most 2^-7 |O|), and the unrounded
# values differ by e: the probabilities are rounded to bf16 before the second product (relative 2^-9 each,
# partly averaging out over the keys, so e grows with |O| too) and sums are fp32.  Bound:
# |out - want| <= OWN_ABS + 2^-6 |want|.  On the five configurations |O| <= 0.4 and the observed max-abs error
# is 4.9e-4 .. 2.0e-3 (5e-4 beyond the two ulps); trees without a prefix (a handful of keys per node) reach
# |O| ~ 4, 1.6e-2 max-abs and 2.0e-3 beyond the two ulps, the largest seen: OWN_ABS is twice that.
# Every test prints what it observed (pytest -rP shows it).
NORTH_STAR_TOL = {"f32": 1e-5, "bf16": 2e-2}
OWN_ABS = {"f32": 2e-6, "bf16": 4e-3}
OWN_REL = {"f32": 0.0, "bf16": 2.0 ** -6}

_CASES, _ATTN = {}, {}


def cached_case(ci):
    """The oracle side of benchmark configuration ci, computed once per test session."""
    if ci not in _CASES:
        _CASES[ci] = oracle_case(ci)
    return _CASES[ci]


def oracle_attention(case, b, scale, key=None):
    """Every attention output of sequence b from the oracle (cached when the case is a cached one)."""
    c = case.cfg
    q, kt, vt, kp, vp = dt_synth.qkv(c, b)
    N = case.trees[b]["n_nodes"]
    if key is not None and (key, b) in _ATTN:
        return _ATTN[(key, b)]
    want = ref.tree_attention(q[:N], kt[:N], vt[:N], kp, vp, case.trees[b]["anc_mask"], scale)
    if key is not None:
        _ATTN[(key, b)] = want
    return want


def assert_attention(out, want, dtype, tag, own_abs=None):
    """Every output element against the oracle; NaN or inf anywhere fails."""
    assert out.shape == want.shape, tag
    assert np.isfinite(out).all(), (tag, "non-finite attention output")
    diff = np.abs(out - want)
    err = float(diff.max())
    own = float((diff - OWN_REL[dtype] * np.abs(want)).max())      # what is left after two ulps of the result
    assert err <= NORTH_STAR_TOL[dtype], (tag, "attention max-abs", err)
    assert own <= (OWN_ABS[dtype] if own_abs is None else own_abs), (tag, "attention error above our own bound", own, err)
    return err, own


def check_case(case, key=None, kv_head_major=False):
    c = case.cfg
    st = make_step(case, kv_head_major=kv_head_major)
    st.run(philox_step=0)
    torch.cuda.synchronize()
    worst, worst_own = 0.0, -1.0
    for b in range(c.B):
        tag = "%s seq %d" % (c.name, b)
        got = st.tree(b)
        assert_tree_equal(got, case.trees[b], tag)
        assert_accept_equal(st.accepted(b), case.accepts[b], tag)
        e, o = assert_attention(st.attention_out(b), oracle_attention(case, b, st.scale, key), c.dtype, tag)
        worst, worst_own = max(worst, e), max(worst_own, o)
    print("attention error %s: max-abs %.3e, beyond two ulps of the result %.3e (all %d outputs compared)"
          % (c.name, worst, worst_own, sum(t["n_nodes"] for t in case.trees) * c.Hq * c.D))
    return st


def test_config1_tiny_fp32():
    check_case(cached_case(1), key=1)


def test_config2_llama3_8b_tt60():
    case = cached_case(2)
    assert case.trees[0]["n_nodes"] == 60
    assert 0 < sum(a["accept_len"] for a in case.accepts)          # acceptance is partial, not trivial
    check_case(case, key=2)


def test_config3_vicuna_13b_tt64():
    check_case(cached_case(3), key=3)


def test_config4_batch16_ragged():
    case = cached_case(4)
    assert len({p for p in case.cfg.params}) > 8                   # really ragged
    check_case(case, key=4)


def test_config5_llama3_70b_stochastic():
    case = cached_case(5)
    lens = [a["accept_len"] for a in case.accepts]
    assert max(lens) > 0
    check_case(case, key=5)


# ------------------------------------------------------------------------------------------ edge cases

def small_cfg(params, prefix_len, V=4099, dtype="bf16", Hq=8, Hkv=2, D=128, seed=0, mode=dt_synth.GREEDY):
    return dt_synth.StepConfig("edge", dtype, Hq, Hkv, D, V, params, prefix_len, seed=seed, mode=mode)


@pytest.mark.parametrize("params", [[(1, 3, 4)], [(2, 1, 1)], [(128, 8, 3)], [(5, 1, 9), (128, 3, 32), (17, 8, 1)],
                                    [(64, 2, 32)], [(100, 4, 4)]])
def test_degenerate_tree_shapes(params):
    # TT=1 (root only), d=1 (star), k=1 (chain), pool smaller than TT (clamp), the largest k
    cfg = small_cfg(params, [70 + 13 * i for i in range(len(params))])
    check_case(oracle_case(0, cfg=cfg))


def test_token_count_exit_of_the_expansion_loop():
    # DT_TREE_EARLY_STOP: expansion ends once the root and the proposed candidates number TT.  No expansion
    # at all (1 + k >= TT), a stop after one, two and three levels, a budget that never binds, wide levels
    # that go through the bucket selection, TT = 1; the draft rows of the unexpanded levels are still there.
    params = [(5, 3, 8), (12, 5, 4), (30, 4, 3), (60, 6, 10), (128, 3, 3), (96, 8, 20), (1, 4, 4), (40, 8, 2)]
    cfg = small_cfg(params, [40 + 7 * i for i in range(len(params))])
    case = oracle_case(0, cfg=cfg, early_stop=True)
    depths = [int(t["depth"].max()) for t in case.trees]
    assert depths[0] == 1 and depths[1] == 2 and depths[3] == 2 and depths[4] == 3 and depths[5] == 2, depths
    plain = oracle_case(0, cfg=small_cfg(params, [40 + 7 * i for i in range(len(params))]))
    assert any(p["n_nodes"] != e["n_nodes"] or not np.array_equal(p["tokens"], e["tokens"])
               for p, e in zip(plain.trees, case.trees))            # the flag does change trees here
    check_case(case)


def test_config2_shape_with_the_token_count_exit():
    # the Llama-3-8B configuration (TT=60, d=6, k=10) under DT_TREE_EARLY_STOP: 1 + 10 + 100 >= 60 ends the
    # expansion after level 1's nodes have been expanded, so the tree has depth 2 and 41 of its 51 rows go unused
    case = oracle_case(2, early_stop=True)
    assert int(case.trees[0]["depth"].max()) == 2 and case.trees[0]["n_nodes"] == 60
    check_case(case)


def test_large_pool_uses_the_workgroup_wide_cut():
    cfg = small_cfg([(128, 8, 16)], [40], V=2000)                # pool 16 + 7*256 = 1808 > 1024
    check_case(oracle_case(0, cfg=cfg))
    cfg = small_cfg([(96, 8, 32)], [33], V=1500)                 # the largest pool: 7200
    check_case(oracle_case(0, cfg=cfg))


def test_empty_prefix_and_tt1_decode_and_fp32_heads():
    check_case(oracle_case(0, cfg=small_cfg([(24, 4, 3)], [0])))                     # no prefix at all
    check_case(oracle_case(0, cfg=small_cfg([(1, 1, 1)], [300])))                    # TT=1: ordinary decode
    check_case(oracle_case(0, cfg=small_cfg([(30, 4, 3)], [65], dtype="f32", D=64, Hq=4, Hkv=4)))
    check_case(oracle_case(0, cfg=small_cfg([(30, 4, 3)], [65], dtype="f32", D=128, Hq=6, Hkv=2)))
    check_case(oracle_case(0, cfg=small_cfg([(30, 4, 3)], [65], dtype="bf16", D=64, Hq=4, Hkv=1)))  # simple path


def test_attention_key_splits_and_long_prefix():
    # few (sequence, kv head) pairs and a long prefix: the small-batch kernel splits the keys over
    # several workgroups, whose partials meet in the same launch
    check_case(oracle_case(0, cfg=small_cfg([(30, 4, 3)], [2000], Hq=8, Hkv=2)))
    check_case(oracle_case(0, cfg=small_cfg([(128, 6, 6), (7, 2, 3)], [4097, 640], Hq=4, Hkv=4)))


def test_prefix_caches_laid_out_head_major():
    # [kv head, token, D] caches with one common token capacity instead of [token, kv head, D]: the two
    # strides of the call are all that changes; every attention kernel is visited
    check_case(cached_case(1), key=1, kv_head_major=True)                                            # plain ALU path
    check_case(oracle_case(0, cfg=small_cfg([(30, 4, 3)], [300], Hq=8, Hkv=2)), kv_head_major=True)   # one workgroup per unit
    check_case(oracle_case(0, cfg=small_cfg([(128, 6, 6), (7, 2, 3)], [4097, 640], Hq=4, Hkv=4)), kv_head_major=True)  # key splits
    rng = np.random.default_rng(78)
    params = [(int(rng.choice([1, 33, 64, 96])), int(rng.integers(1, 6)), int(rng.integers(1, 7))) for _ in range(24)]
    plen = [int(rng.choice([0, 1, 63, 65, 300, 2500])) for _ in range(24)]
    check_case(oracle_case(0, cfg=small_cfg(params, plen, V=2053, Hq=32, Hkv=8)), kv_head_major=True)  # balanced schedule
    params = [(int(rng.choice([5, 40])), 3, 3) for _ in range(70)]
    check_case(oracle_case(0, cfg=small_cfg(params, [int(rng.integers(0, 200)) for _ in range(70)], V=1031,
                                            Hq=8, Hkv=2)), kv_head_major=True)                       # one workgroup per item


def test_attention_balanced_schedule_on_ragged_batches():
    # enough (sequence, kv head, row tile) items for the large-batch kernel, too few to fill the chip:
    # every kv head's workgroup slots share out the key blocks of all sequences evenly, so one slot
    # walks through several short sequences (written directly) and parts of long ones (partials that
    # a second kernel merges).  Row-tile counts 1..3, empty and one-block prefixes, TT = 1.
    rng = np.random.default_rng(77)
    params, plen = [], []
    for i in range(24):
        TT = int(rng.choice([1, 7, 32, 33, 64, 65, 96]))
        params.append((TT, int(rng.integers(1, 6)), int(rng.integers(1, 7))))
        plen.append(int(rng.choice([0, 1, 63, 64, 65, 300, 900, 2500])))
    plen[3], plen[4] = 6000, 0
    check_case(oracle_case(0, cfg=small_cfg(params, plen, V=2053, Hq=32, Hkv=8)))
    # one class only, sequences much longer than a slot's share: every sequence is cut several times
    check_case(oracle_case(0, cfg=small_cfg([(96, 4, 6)] * 3, [5000, 4100, 37], V=2053, Hq=64, Hkv=8)))
    # more whole items than slots would need splitting: plain one-workgroup-per-item launch (batch > 64)
    params = [(int(rng.choice([5, 40])), 3, 3) for _ in range(70)]
    check_case(oracle_case(0, cfg=small_cfg(params, [int(rng.integers(0, 200)) for _ in range(70)], V=1031,
                                            Hq=8, Hkv=2)))


@pytest.mark.parametrize("V,dtype,mode", [(7, "bf16", dt_synth.GREEDY), (7, "f32", dt_synth.STOCHASTIC),
                                          (13, "bf16", dt_synth.STOCHASTIC), (13, "bf16", dt_synth.SAMPLED),
                                          (8, "bf16", dt_synth.SAMPLED)])
def test_whole_step_on_vocabularies_around_eight_entries(V, dtype, mode):
    # below eight entries no 16-byte group fits a row (element loads only), just above it the last group of
    # a row straddles its end: row streams, arg-max rows and the sampler's chunk re-read all take that path
    cfg = small_cfg([(6, 3, 2), (12, 2, 5), (1, 1, 1)], [9, 70, 3], V=V, dtype=dtype, mode=mode,
                    D=128 if dtype == "bf16" else 64, Hq=4, Hkv=2)
    check_case(oracle_case(0, cfg=cfg, max_bumps=200))


@pytest.mark.parametrize("seed", [11, 12, 13, 14])
def test_random_batches_of_random_shapes(seed):
    # a sweep nobody chose by hand: per sequence random (TT, d, k) over the whole range of the limits, random
    # prefix lengths, a vocabulary that is not a multiple of anything; greedy and stochastic in turn
    rng = np.random.default_rng(seed)
    B = 20
    params, plen = [], []
    for _ in range(B):
        k = int(rng.choice([1, 2, 3, 5, 8, 11, 12, 16, 20, 32]))
        d = int(rng.integers(1, 9))
        params.append((int(rng.integers(1, 129)), d, k))
        plen.append(int(rng.choice([0, 1, 31, 32, 33, 64, 200, 777])))
    mode = dt_synth.GREEDY if seed % 2 else dt_synth.STOCHASTIC
    cfg = small_cfg(params, plen, V=int(rng.choice([611, 1000, 4099])), Hq=8, Hkv=2, seed=seed, mode=mode)
    check_case(oracle_case(0, seed=seed, cfg=cfg, max_bumps=60))


def test_stochastic_small_and_many_steps():
    cfg = small_cfg([(40, 5, 4), (64, 6, 6)], [100, 31], V=3001, mode=dt_synth.STOCHASTIC)
    case = oracle_case(0, cfg=cfg)
    st = check_case(case)
    # more Philox steps on the same tree: every step must agree (margin-guarded per step)
    agree = 0
    for step in range(1, 40):
        st.accept(philox_step=step)
        torch.cuda.synchronize()
        for b in range(cfg.B):
            t = case.trees[b]
            want = ref.accept(cfg.mode, case.targets[b], t["tokens"], t["parents"], t["depth"], logp=t["logp"],
                              temperature=cfg.temperature, seed=cfg.philox_seed, step=step, seq=b)
            if want["min_margin"] < 1e-5:
                continue
            assert_accept_equal(st.accepted(b), want, "step %d seq %d" % (step, b))
            agree += 1
    assert agree > 60


def test_target_sampled_verification_small_and_llama_vocabulary():
    # distribution-preserving mode: every node draws the target's own token; tokens, path and node samples exact
    cfg = small_cfg([(40, 5, 4), (64, 6, 6), (1, 1, 1)], [100, 31, 7], V=3001, mode=dt_synth.SAMPLED)
    cfg.temperature = 0.8
    case = oracle_case(0, cfg=cfg)
    st = check_case(case)
    agree = 0
    for step in range(1, 25):
        st.accept(philox_step=step)
        torch.cuda.synchronize()
        for b in range(cfg.B):
            t = case.trees[b]
            want = ref.accept(cfg.mode, case.targets[b], t["tokens"], t["parents"], t["depth"],
                              temperature=cfg.temperature, seed=cfg.philox_seed, step=step, seq=b)
            if want["min_margin"] < 1e-5:
                continue
            got = st.accepted(b)
            assert_accept_equal(got, want, "step %d seq %d" % (step, b))
            agree += 1
    assert agree > 50
    big = small_cfg([(60, 6, 10), (33, 4, 8)], [64, 5], V=128256, Hq=8, Hkv=2, mode=dt_synth.SAMPLED)
    check_case(oracle_case(0, cfg=big))


def test_all_layers_attention_under_one_graph():
    # verification touches every layer: the attention calls of several layers (own Q/K/V/prefix per layer,
    # shared tree masks and lengths) captured as one HIP graph, replayed with the outputs wiped and eager
    # work in between; every replay must reproduce every layer's oracle result.
    import paper_2601_12212_amd as dt
    cfg = small_cfg([(30, 4, 3), (64, 5, 5)], [300, 45], Hq=8, Hkv=2)
    case = oracle_case(0, cfg=cfg)
    st = make_step(case)
    st.build_tree()
    torch.cuda.synchronize()
    n_layers, B, TC = 3, cfg.B, st.TT_cap
    rng = np.random.default_rng(8)
    bf = lambda sh: dt_synth.f32_to_bf16_bits(rng.standard_normal(sh).astype(np.float32))
    dev = lambda a: torch.from_numpy(a.view(np.int16)).cuda().view(torch.bfloat16)
    layers = []
    for l in range(n_layers):
        h = dict(q=bf((B, TC, cfg.Hq, cfg.D)), kt=bf((B, TC, cfg.Hkv, cfg.D)), vt=bf((B, TC, cfg.Hkv, cfg.D)),
                 kp=[bf((max(L, 1), cfg.Hkv, cfg.D)) for L in cfg.prefix_len],
                 vp=[bf((max(L, 1), cfg.Hkv, cfg.D)) for L in cfg.prefix_len])
        d = dict(q=dev(h["q"]), kt=dev(h["kt"]), vt=dev(h["vt"]), kp=[dev(a) for a in h["kp"]], vp=[dev(a) for a in h["vp"]],
                 out=torch.zeros((B, TC, cfg.Hq, cfg.D), dtype=torch.bfloat16, device="cuda"))
        d["kpp"] = torch.tensor([t.data_ptr() for t in d["kp"]], dtype=torch.int64, device="cuda")
        d["vpp"] = torch.tensor([t.data_ptr() for t in d["vp"]], dtype=torch.int64, device="cuda")
        layers.append((h, d))

    def run():
        for h, d in layers:
            dt.dt_tree_attention(d["q"], d["kt"], d["vt"], st.n_nodes, d["kpp"], d["vpp"], st.prefix_len,
                                 max(cfg.prefix_len), cfg.Hkv * cfg.D, cfg.D, st.anc_mask, st.scale, d["out"], st.ws)

    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        run()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            run()
    for rep in range(3):
        for h, d in layers:
            d["out"].fill_(7.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for l, (h, d) in enumerate(layers):
            for b in range(B):
                N, L = case.trees[b]["n_nodes"], cfg.prefix_len[b]
                want = ref.tree_attention(h["q"][b, :N], h["kt"][b, :N], h["vt"][b, :N], h["kp"][b][:L], h["vp"][b][:L],
                                          case.trees[b]["anc_mask"], st.scale)
                got = d["out"][b, :N].float().cpu().numpy()
                assert_attention(got, want, "bf16", (rep, l, b))
        (torch.ones(1000, device="cuda") * 3).sum().item()


@pytest.mark.parametrize("ci", [2, 4])
def test_whole_step_replayed_from_a_graph_matches_the_oracle(ci):
    # the launch configuration bench.py times: the three calls of the step captured once as a HIP graph and
    # replayed, at the full size of the configuration; every replay (outputs wiped before it, eager work
    # after it) must give the oracle's tree, acceptance and every attention output
    case = cached_case(ci)
    c = case.cfg
    st = make_step(case).prepare()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        st.run_prepared(side.cuda_stream)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            st.run_prepared(side.cuda_stream)
    for rep in range(3):
        for t in (st.n_nodes, st.tokens, st.parents, st.depth, st.src_row, st.accept_len, st.best_node, st.path_nodes,
                  st.out_tokens):
            t.fill_(-7)
        st.out.fill_(3.0)
        st.anc_mask.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for b in range(c.B):
            tag = "%s seq %d replay %d" % (c.name, b, rep)
            got = st.tree(b)
            assert_tree_equal(got, case.trees[b], tag)
            assert_accept_equal(st.accepted(b), case.accepts[b], tag)
            assert_attention(st.attention_out(b), oracle_attention(case, b, st.scale, ci), c.dtype, tag)
        (torch.ones(1000, device="cuda") * 3).sum().item()


def test_exact_score_ties_across_rows_go_to_the_lowest_pool_index():
    # identical draft rows: every candidate of a level has exactly the same score on both sides, so the
    # level cuts and the rerank are decided by the tie-break alone (the margin guard would reject these
    # inputs, so the oracle is called directly)
    from paper_2601_12212_amd.step import Step
    for V, TT, d, k, bf16 in [(8, 6, 3, 2, False), (8, 9, 3, 2, False), (1000, 60, 4, 10, True), (2048, 128, 8, 32, True),
                              (700, 100, 5, 12, False)]:
        rows = np.zeros((1 + (d - 1) * k, V), np.float32)
        rows[:, V // 3] = 1.0                                # one clear winner per row, the rest tie
        want = ref.build_tree(dt_synth.f32_to_bf16_bits(rows) if bf16 else rows, TT, d, k, 3)
        assert want["min_margin"] == 0.0
        st = Step([(TT, d, k)], [1], 4, 4, 64, V, dtype=torch.bfloat16 if bf16 else torch.float32, TT_cap=128)
        st.set_draft(0, dt_synth.f32_to_bf16_bits(rows) if bf16 else rows)
        st.set_root_token(0, 3)
        st.build_tree()
        torch.cuda.synchronize()
        assert_tree_equal(st.tree(0), want, "ties V=%d TT=%d d=%d k=%d" % (V, TT, d, k))


@pytest.mark.parametrize("V,sigma,TT,d,k", [(2000, 0.02, 100, 4, 12),      # 144 level-2 scores inside one bucket
                                             (128256, 0.02, 40, 8, 3),     # the cut among 54 scores below -32
                                             (128256, 0.02, 60, 8, 4),     # 96 scores below -32
                                             (3000, 0.3, 128, 8, 16)])     # pool of 1808, crowded deep levels
def test_nearly_flat_rows_crowd_the_score_buckets(V, sigma, TT, d, k):
    """Draft rows that are almost flat give every candidate of a level nearly the same score: the rerank then
    finds its cut inside one crowded score bucket (or among the scores below the bucket range) and has to
    order distinct, close keys exactly."""
    from paper_2601_12212_amd.step import Step
    R = 1 + (d - 1) * k
    for seed in range(20):
        rows = (np.random.default_rng(seed).standard_normal((R, V)) * sigma).astype(np.float32)
        want = ref.build_tree(rows, TT, d, k, 7)
        if want["min_margin"] >= 1e-4:
            break
    else:
        pytest.fail("margin guard: no acceptable seed")
    st = Step([(TT, d, k)], [1], 4, 4, 64, V, dtype=torch.float32, TT_cap=128)
    st.set_draft(0, rows)
    st.set_root_token(0, 7)
    st.build_tree()
    torch.cuda.synchronize()
    assert_tree_equal(st.tree(0), want, "flat rows V=%d TT=%d d=%d k=%d seed=%d" % (V, TT, d, k, seed))


def test_masked_vocabulary_rows():
    """-inf logits (tokens that may never be proposed) and rows with fewer than k viable tokens."""
    cfg = small_cfg([(20, 3, 4)], [50], V=3000)
    drafts = dt_synth.draft_rows(cfg, 0).copy()
    ninf = dt_synth.f32_to_bf16_bits(np.array([-np.inf], np.float32))[0]
    drafts[:, 100:] = ninf            # only 100 tokens viable
    drafts[2, 2:] = ninf              # this row has 2 viable tokens (k = 4)
    drafts[3, :] = ninf               # this row has none
    case = oracle_case(0, cfg=cfg)
    case.drafts = [drafts]
    t = ref.build_tree(drafts, 20, 3, 4, dt_synth.root_token(cfg, 0))
    assert t["min_margin"] >= 1e-4
    case.trees = [t]
    case.targets = [dt_synth.target_rows(cfg, 0, t["src_row"], drafts)]
    case.accepts = [ref.accept(cfg.mode, case.targets[0], t["tokens"], t["parents"], t["depth"])]
    check_case(case)


@pytest.mark.parametrize("ci,repeats", [(2, 100), (4, 25), (5, 10)])
def test_determinism_same_inputs_same_bits(ci, repeats):
    # config 2: small-batch attention with key splits and its merge; config 4: the balanced large-batch
    # schedule with partials and their combine; config 5: the same with Philox draws in the acceptance
    case = cached_case(ci)
    st = make_step(case)
    st.out.fill_(5.0)
    st.run()
    torch.cuda.synchronize()
    outs = lambda: [st.n_nodes, st.tokens, st.parents, st.anc_mask, st.out, st.accept_len, st.out_tokens, st.score,
                    st.node_argmax]
    first = [t.clone() for t in outs()]
    for r in range(repeats):
        st.out.fill_(5.0)
        st.run()
        if r % 10 == 9 or r == repeats - 1:
            torch.cuda.synchronize()
            for i, (a, b) in enumerate(zip(first, outs())):
                assert torch.equal(a, b), (ci, r, i)


def test_driving_the_build_level_by_level_matches_the_oracle():
    """The call pattern of a real draft model: rows become known one level at a time."""
    from paper_2601_12212_amd.step import Step
    from tests._brute import toy_logits
    from tests._drive import rows_from_fn
    V, d, k, TT = 64, 4, 3, 30

    def gpu_build(rows, TT_, d_, k_, root):
        st = Step([(TT_, d_, k_)], [1], 4, 4, 64, V, dtype=torch.float32, TT_cap=128)
        full = np.zeros((1 + (d_ - 1) * k_, V), np.float32)
        full[:] = rows[: full.shape[0]]
        st.set_draft(0, full)
        st.set_root_token(0, root)
        st.build_tree()
        torch.cuda.synchronize()
        return st.tree(0)

    fn = lambda s: toy_logits(3, s, V)
    rows_gpu = rows_from_fn(gpu_build, fn, V, d, k)
    rows_ref = rows_from_fn(ref.build_tree, fn, V, d, k)
    assert np.array_equal(rows_gpu, rows_ref)
    assert_tree_equal(gpu_build(rows_gpu, TT, d, k, 7), ref.build_tree(rows_ref, TT, d, k, 7))


# ------------------------------------------------------------------ the tree mask on the device

def _attention_shapes():
    rng = np.random.default_rng(31)
    tile_params = [(int(rng.choice([5, 40])), 3, 3) for _ in range(70)]
    return {
        # one workgroup per (sequence, kv head, 32 rows), 144 of them: no key splits
        "wave": small_cfg([(60, 6, 10)], [300], V=1500, Hq=72, Hkv=18),
        # the same kernel with the keys dealt over several workgroups
        "wave_split": small_cfg([(60, 6, 10), (33, 4, 8)], [2000, 1700], V=1500, Hq=8, Hkv=2),
        # balanced large-batch schedule (partials, merged by a workgroup of the launch)
        "gang": small_cfg([(64, 5, 6)] * 12 + [(96, 4, 6)] * 4, [300 + 211 * i for i in range(16)], V=1031, Hq=32, Hkv=8),
        # one workgroup per (sequence, kv head, 128-row tile): more than 64 sequences
        "tile": small_cfg(tile_params, [int(rng.integers(0, 200)) for _ in range(70)], V=1031, Hq=8, Hkv=2),
    }


@pytest.mark.parametrize("shape", ["wave", "wave_split", "gang", "tile"])
def test_keys_outside_a_nodes_ancestor_set_do_not_reach_its_output(shape):
    """Overwrite K and V of one tree token per sequence: the outputs of the nodes that do not have it among
    their ancestors must not change by a single bit, those of the token itself and its descendants must."""
    cfg = _attention_shapes()[shape]
    case = oracle_case(0, cfg=cfg)
    st = make_step(case)
    st.build_tree()
    st.tree_attention()
    torch.cuda.synchronize()
    before = st.out.clone()
    rng = np.random.default_rng(5)
    hit = []
    for b in range(cfg.B):
        N = case.trees[b]["n_nodes"]
        if N < 3:
            hit.append(None)
            continue
        j = int(rng.integers(1, N))                      # never the root: every node sees the root
        hit.append(j)
        noise = torch.from_numpy(rng.standard_normal((2, cfg.Hkv, cfg.D)).astype(np.float32) * 40.0).cuda()
        st.k_tree[b, j] = noise[0].to(st.k_tree.dtype)
        st.v_tree[b, j] = noise[1].to(st.v_tree.dtype)
    st.tree_attention()
    torch.cuda.synchronize()
    after = st.out
    unchanged = changed = 0
    for b in range(cfg.B):
        j = hit[b]
        if j is None:
            continue
        mask = case.trees[b]["anc_mask"]
        for i in range(case.trees[b]["n_nodes"]):
            sees = (int(mask[i, j // 64]) >> (j % 64)) & 1
            same = torch.equal(before[b, i].view(torch.int16), after[b, i].view(torch.int16))
            if sees:
                assert not same, (shape, b, i, j, "a visible key was ignored")
                changed += 1
            else:
                assert same, (shape, b, i, j, "a hidden key reached the output")
                unchanged += 1
    assert changed > 0 and unchanged > changed


@pytest.mark.parametrize("shape", ["wave", "wave_split", "gang", "tile"])
def test_scores_that_grow_along_the_keys_move_the_softmax_reference_late(shape):
    """The kernels move their softmax reference lazily and rescale the output accumulators only then.  Keys
    whose length grows with their position (prefix and tree) make the scores of every query climb by many
    powers of two along the key axis, so the reference moves several times while the accumulators are far
    from zero; every output is still compared with the oracle."""
    cfg = _attention_shapes()[shape]
    case = oracle_case(0, cfg=cfg)
    st = make_step(case)
    st.build_tree()
    worst = 0.0
    want_all = []
    for b in range(cfg.B):
        q, kt, vt, kp, vp = (dt_synth.as_f32(x).copy() for x in dt_synth.qkv(cfg, b))
        N, L = case.trees[b]["n_nodes"], kp.shape[0]
        q[:] = np.abs(q)                                      # q . k then grows with |k| instead of cancelling
        ramp = np.linspace(0.05, 6.0, L + N, dtype=np.float32)
        kp[:] = np.abs(kp) * ramp[:L, None, None]
        kt[:N] = np.abs(kt[:N]) * ramp[L:, None, None]
        rnd = lambda x: dt_synth.f32_to_bf16_bits(x)
        qb, ktb, vtb, kpb, vpb = rnd(q), rnd(kt), rnd(vt), rnd(kp), rnd(vp)
        st.set_qkv(b, qb, ktb, vtb, kpb, vpb)
        want_all.append(ref.tree_attention(qb[:N], ktb[:N], vtb[:N], kpb, vpb, case.trees[b]["anc_mask"], st.scale))
    st.tree_attention()
    torch.cuda.synchronize()
    for b in range(cfg.B):
        # A softmax this peaked puts nearly all weight on one or two keys with |v| up to 4: the bf16 rounding of
        # the probabilities (2^-9 relative) alone is then worth 8e-3, twice the bound derived for N(0,1) scores.
        e, _ = assert_attention(st.attention_out(b), want_all[b], cfg.dtype, "%s seq %d" % (shape, b), own_abs=1e-2)
        worst = max(worst, e)
    print("growing scores, %s: max-abs %.3e" % (shape, worst))


def test_more_rows_than_a_grid_dimension_holds():
    # 70,000 rows in one call: rows ride in the x dimension of the launch grid
    rng = np.random.default_rng(3)
    x = dt_synth.f32_to_bf16_bits((rng.standard_normal((70000, 96)) * 3).astype(np.float32))
    check_topk(x, 5)


def test_a_sequence_that_owns_fewer_rows_than_its_tree_needs():
    """row_off hands sequence 0 only 4 of the 1 + (d-1) k = 10 rows its parameters ask for: the missing
    rows count as rows without a viable token, whatever the workspace held before."""
    from paper_2601_12212_amd.step import Step
    V, TT, d, k = 3000, 40, 4, 3
    cfg = small_cfg([(TT, d, k), (TT, d, k)], [10, 10], V=V)
    rows = [dt_synth.draft_rows(cfg, b) for b in range(2)]
    st = Step(cfg.params, cfg.prefix_len, cfg.Hq, cfg.Hkv, cfg.D, V)
    owned = 4
    packed = np.concatenate([rows[0][:owned], rows[1]])            # sequence 1 keeps all of its rows
    st.draft_logits[:packed.shape[0]].copy_(torch.from_numpy(packed.view(np.int16)).cuda().view(torch.bfloat16))
    st.row_off.copy_(torch.tensor([0, owned, owned + rows[1].shape[0]], dtype=torch.int64))
    st.total_rows = owned + rows[1].shape[0]
    st.ws.fill_(0x7F)                                              # stale scratch: huge positive floats
    st.build_tree()
    torch.cuda.synchronize()
    short = rows[0].copy()
    short[owned:] = dt_synth.f32_to_bf16_bits(np.array([-np.inf], np.float32))[0]
    want0 = ref.build_tree(short, TT, d, k, 0)
    want1 = ref.build_tree(rows[1], TT, d, k, 0)
    assert want0["min_margin"] >= 1e-4 and want1["min_margin"] >= 1e-4
    assert want0["n_nodes"] < want1["n_nodes"]
    assert_tree_equal(st.tree(0), want0, "short span")
    assert_tree_equal(st.tree(1), want1, "full span")


def test_first_library_call_of_a_process_inside_a_graph_capture():
    """The one-time set-up (LDS opt-in, compute-unit count) happens in the first launching call; here that call
    is recorded into a HIP graph in a fresh process, and the replayed step must equal an eager run."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    child = r"""
import sys
sys.path.insert(0, %r)
import numpy as np, torch
import dt_synth
from paper_2601_12212_amd.step import Step
cfg = dt_synth.StepConfig("cap", "bf16", 8, 2, 128, 5003, [(40, 5, 4), (64, 6, 6)], [700, 90], seed=3)
st = Step(cfg.params, cfg.prefix_len, cfg.Hq, cfg.Hkv, cfg.D, cfg.V)
dt_synth.fill_draft_and_qkv(st, cfg)
st.target_logits.copy_(torch.randn(st.target_logits.shape, device="cuda").to(torch.bfloat16) * 3)
torch.cuda.synchronize()
side = torch.cuda.Stream()
g = torch.cuda.CUDAGraph()
with torch.cuda.stream(side):
    with torch.cuda.graph(g, stream=side):
        st.run(philox_step=0)              # the library's first call in this process
torch.cuda.synchronize()
names = ("n_nodes", "tokens", "parents", "anc_mask", "out", "accept_len", "out_tokens")
for rep in range(3):
    for n in names:
        getattr(st, n).fill_(3)
    g.replay()
    torch.cuda.synchronize()
    got = [getattr(st, n).clone() for n in names]
    for n in names:
        getattr(st, n).fill_(3)
    st.run(philox_step=0)
    torch.cuda.synchronize()
    for n, a in zip(names, got):
        assert torch.equal(a, getattr(st, n)), (rep, n)
    assert int(st.n_nodes[0]) == 40 and int(st.n_nodes[1]) == 64
print("FIRST-CALL-CAPTURE-OK")
""" % root
    r = subprocess.run([sys.executable, "-c", child], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "FIRST-CALL-CAPTURE-OK" in r.stdout, (r.returncode, r.stdout[-2000:], r.stderr[-2000:])
