"""GPU parity of row top-k at the sizes where it changes its path: rows held by one workgroup (256, 512 and 1024 threads, 8 to
32 entries each), the two-pass path beyond, one chunk more than the selection keeps in registers, odd strides, and rows whose
clusters or equal values defeat the first bound."""
import numpy as np
import pytest

import dt_synth
from oracle import ref
from paper_2601_12212_amd import dt_topk_rows, dt_workspace_bytes
from tests._cases import TREE_MARGIN, assert_tree_equal, oracle_case
from tests.test_gpu_parity import check_case, check_topk, dev_logits

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("V", [7, 8, 9, 300, 2047, 2048, 2049, 4096, 4097, 8191, 8193, 16384, 16385, 32768, 32769, 65537, 131072, 131081])
@pytest.mark.parametrize("bf16", [False, True])
def test_topk_rows_around_the_edges_of_its_paths(V, bf16):
    rng = np.random.default_rng(V)
    x = (rng.standard_normal((6, V)) * 3).astype(np.float32)
    x[1] = 40.0 + rng.integers(0, 3, V)                       # three values: ties everywhere
    x[2, V // 3:V // 3 + 200] += 50.0                         # a cluster of neighbours
    x[3] = -np.inf
    x[3, rng.integers(0, V, 5)] = 1.5                         # at most five viable entries
    x[4, -1] = x[4, 0] = 30.0                                 # the ends of the row
    for k in sorted({1, min(V, 20), min(V, 32)}):
        check_topk(dt_synth.f32_to_bf16_bits(x) if bf16 else x, k)


@pytest.mark.parametrize("V,n", [(20000, 256), (20000, 257), (1000, 700)])
def test_topk_rows_of_many_rows(V, n):
    x = (np.random.default_rng(n).standard_normal((n, V)) * 3).astype(np.float32)
    check_topk(dt_synth.f32_to_bf16_bits(x), 9)


@pytest.mark.parametrize("V,n,bf16", [(32769, 1821, True), (65537, 1821, True), (131072, 1025, True), (131081, 1000, True),
                                      (16385, 1821, False), (65536, 1025, False), (16385, 1821, True), (20000, 1640, True),
                                      (31001, 1025, True), (32768, 1025, True), (65001, 129, True)])
def test_topk_rows_of_launches_of_many_chunks(V, n, bf16):
    """More than 16,384 chunks: odd and even numbers of them to a row, a last one of one element, nine elements and whole, one
    and two to a workgroup.  2,064 chunks: a workgroup more to a row than there are chunks."""
    check_repeated_rows(V, n, bf16)


@pytest.mark.parametrize("V,n", [(9, 2049), (10, 2100), (40, 2049), (511, 2049), (513, 2100), (2047, 2049), (2048, 2049), (2049, 1025), (2560, 4097),
                                 (4096, 4200), (4097, 2600), (4104, 513), (8192, 2100), (9411, 257), (16384, 1025), (16385, 129), (20481, 700),
                                 (32760, 600), (32768, 129), (32768, 1024), (32767, 513), (32769, 410), (40961, 342), (65535, 257), (65536, 257)])
@pytest.mark.parametrize("gap", [0, 1, 2])
def test_topk_rows_of_large_launches(V, n, gap):
    # one to sixteen waves to a row of 32 or 64 entries a lane, the last group of a wave whole, begun, of one entry and empty; and
    # chunks of 8,192 entries, five to eight to a row
    check_repeated_rows(V, n, True, gap)


# where the bisection over the registers can go wrong: one to eight waves of 32 or 64 entries a lane, the last group of a wave whole, begun, of one entry
# and empty, an entry before the row
@pytest.mark.parametrize("V,n", [(300, 2100), (2048, 2049), (2049, 1030), (4103, 2600), (8192, 2100), (9411, 260), (16384, 1025), (16385, 140), (32767, 520), (32768, 1024)])
def test_ties_of_large_launches(V, n):
    import paper_2601_12212_amd as dt
    rng = np.random.default_rng(V)
    k = 32
    x = np.zeros((9, V), np.float32)
    x[1] = np.where(rng.random(V) < 0.5, 0.0, -0.0)           # equal under two signs
    x[2] = np.where(rng.random(V) < 0.5, 0.0, -0.0)
    x[2, rng.permutation(V)[:k // 2]] = 2.0 ** -130           # a denormal number
    x[3] = -1.0
    x[3, rng.permutation(V)[:k]] = -0.0                       # as many as are asked for
    x[4] = -np.inf
    x[4, V - 290:] = -3.0e38                                  # equal at the end, nothing else viable
    x[5] = 1.0 + np.arange(V) % 2                             # two values, every other entry
    x[6] = np.floor(np.arange(V) / (V / 64))                  # runs
    x[7] = -x[6]
    x[8] = rng.integers(-3, 1, V)
    rows = dt_synth.f32_to_bf16_bits(x)
    wval, widx, _ = ref.topk_rows(rows, k)
    which = torch.arange(n, device="cuda") % 9
    val, idx = torch.empty((n, k), device="cuda"), torch.empty((n, k), dtype=torch.int32, device="cuda")
    lse = torch.empty(n, device="cuda")
    ws = torch.full((dt.dt_workspace_bytes(1, n, V, 8, 1, 64),), 0x7f, dtype=torch.uint8, device="cuda")
    dt.dt_topk_rows(dev_logits(rows)[which], k, val, idx, lse, ws)
    torch.cuda.synchronize()
    which = which.cpu().numpy()
    assert np.array_equal(idx.cpu().numpy(), widx[which])
    assert np.array_equal(val.cpu().numpy(), wval[which])


@pytest.mark.parametrize("V,n,gap", [(65536, 129, 1), (65536, 129, 2), (131072, 129, 3), (32768, 1025, 1)])
def test_topk_rows_of_whole_chunks_at_odd_addresses(V, n, gap):
    """Sixteen whole chunks to a row: a workgroup more where the rows' stride is odd, none where it is even."""
    check_repeated_rows(V, n, True, gap)


@pytest.mark.parametrize("V,bf16", [(32769, True), (61441, True), (65537, True), (119331, True), (131072, True), (131081, True),
                                    (16385, False), (65536, False)])
def test_draft_rows_of_launches_that_take_two_chunks_to_a_workgroup(V, bf16):
    """More than 16,384 chunks of rows that are looked up: 9, 16, 9, 15, 16, 17, 9 and 16 to a row, a last one of one element, nine
    elements, part of one and whole; a sequence in the middle without live rows."""
    from paper_2601_12212_amd.step import Step
    TT, d, k = 70, 4, 16
    R = 1 + (d - 1) * k
    nl = next(n for n in (1, 2, 4) if V <= 16 * 2048 * n or n == 4)
    B = 16384 // (R * -(-V // (2048 * nl))) + 2
    for seed in range(20):
        rows = (np.random.default_rng(seed).standard_normal((R, V)) * 3).astype(np.float32)
        rows[1, V - 1] = rows[2, 0] = 20.0
        if bf16:
            rows = dt_synth.f32_to_bf16_bits(rows)
        want = ref.build_tree(rows, TT, d, k, 3)
        if want["min_margin"] >= TREE_MARGIN:
            break
    assert want["min_margin"] >= TREE_MARGIN
    params = [(TT, d, k)] * B
    params[B // 2] = (1, d, k)
    st = Step(params, [1] * B, 1, 1, 64, V, dtype=torch.bfloat16 if bf16 else torch.float32)
    for b in range(B):
        st.set_root_token(b, 3)
        if b != B // 2:
            st.set_draft(b, rows)
    st.build_tree()
    torch.cuda.synchronize()
    for b in range(B):
        if b != B // 2:
            assert_tree_equal(st.tree(b), want, "sequence %d" % b)
    assert st.tree(B // 2)["n_nodes"] == 1


# the most rows whose exponentials workgroups of their own sum, and one more; the most 256-thread rows whose waves all find
# the bound, and one more; 512 threads
@pytest.mark.parametrize("V,n,bf16", [(32768, 128, True), (32768, 129, True), (8193, 128, False), (8193, 129, False),
                                      (4096, 512, True), (4096, 513, True), (9, 513, False), (8192, 513, True)])
def test_topk_rows_that_a_workgroup_holds(V, n, bf16):
    check_repeated_rows(V, n, bf16)


def check_repeated_rows(V, n, bf16, gap=0):
    import paper_2601_12212_amd as dt
    k, R = min(20, V), 7
    x = (np.random.default_rng(V + n).standard_normal((R, V)) * 3).astype(np.float32)
    x[1] = 40.0 + np.random.default_rng(V).integers(0, 3, V)   # three values: ties everywhere
    x[2, V // 3:V // 3 + 200] += 50.0                          # a cluster of neighbours
    x[3, -1] = x[3, 0] = 30.0                                  # the ends of the row
    x[4] = -np.inf
    x[4, [0, 8, V // 2, V - 2, V - 1]] = 1.5                   # five viable entries
    rows = dt_synth.f32_to_bf16_bits(x) if bf16 else x
    wval, widx, wlse = ref.topk_rows(rows, k)
    which = torch.arange(n, device="cuda") % R
    logits = torch.nn.functional.pad(dev_logits(rows)[which], (0, gap), value=1e9)[:, :V]   # row stride V + gap
    val = torch.empty((n, k), dtype=torch.float32, device="cuda")
    idx = torch.empty((n, k), dtype=torch.int32, device="cuda")
    lse = torch.empty(n, dtype=torch.float32, device="cuda")
    ws = torch.full((dt.dt_workspace_bytes(1, n, V, 8, 1, 64),), 0x7f, dtype=torch.uint8, device="cuda")
    dt.dt_topk_rows(logits, k, val, idx, lse, ws)
    torch.cuda.synchronize()
    which = which.cpu().numpy()
    assert np.array_equal(idx.cpu().numpy(), widx[which]) and np.array_equal(val.cpu().numpy(), wval[which])
    # as for smaller launches: fp32 partial sums against double ones
    assert np.all(np.abs(lse.cpu().numpy() - wlse[which]) <= 4e-6 * np.maximum(1.0, np.abs(wlse[which])))


# Both passes in one launch and the first sizes beyond: 13 * 2^19 bf16 entries, 2,048 workgroups of which each row has one more than chunks; one row, rows that do not
# fill the last eight; then the same bits whatever the workspace held before, and from a replayed graph whose launch keeps its number.
@pytest.mark.parametrize("V,n,bf16", [(128256, 53, True), (128256, 54, True), (32769, 200, True), (65537, 1, True), (16385, 200, False), (16385, 201, False),
                                      (131072, 120, False), (131072, 121, False), (131073, 9, False)])
def test_topk_rows_in_one_launch_of_both_passes(V, n, bf16):
    check_repeated_rows(V, n, bf16, 1)
    k = 13
    x = torch.randn((n, V), device="cuda", generator=torch.Generator("cuda").manual_seed(V)).mul_(3).to(torch.bfloat16 if bf16 else torch.float32)
    ws = torch.empty(dt_workspace_bytes(1, n, V, 8, 1, 64), dtype=torch.uint8, device="cuda")
    out = [torch.empty((n, k), device="cuda"), torch.empty((n, k), dtype=torch.int32, device="cuda"), torch.empty(n, device="cuda")]
    want = None
    for fill in (0x00, 0xff, 0x3f):
        ws.fill_(fill)
        dt_topk_rows(x, k, *out, ws)
        got = [o.clone() for o in out]
        assert want is None or all(torch.equal(a, b) for a, b in zip(got, want)), fill
        want = got
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        g = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(g, stream=side):
            dt_topk_rows(x, k, *out, ws)
            dt_topk_rows(x, k, *out, ws)
    for rep, fill in enumerate((None, None, 0x5a, None)):
        if fill is not None:
            ws.fill_(fill)
        for o in out:
            o.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, want)), rep


@pytest.mark.parametrize("V", [18433, 34817, 36865, 67585, 74365, 126977])   # 10, 9, 10, 9, 10 and 16 chunks, the last one begun
@pytest.mark.parametrize("bf16", [False, True])
def test_topk_rows_whose_lanes_hold_unequal_shares(V, bf16):
    x = (np.random.default_rng(V).standard_normal((6, V)) * 3).astype(np.float32)
    x[1, V // 2:V // 2 + 16] += 30.0                          # neighbours in one lane or two
    x[2, :V // 4] += 20.0                                     # one wave has all that is read again
    x[3, 5::V // 40] += 25.0                                  # about one to each of its groups
    x[4] = -np.inf
    x[4, 3 * V // 4::V // 100] = np.arange(len(x[4, 3 * V // 4::V // 100]))   # viable entries in fewer groups than k
    x[5, V - 9:] += 30.0                                      # the overlapping last group of eight
    for k in (1, 13, 32):
        check_topk(dt_synth.f32_to_bf16_bits(x) if bf16 else x, k)


@pytest.mark.parametrize("V", [1001, 8190, 16381, 40001])
def test_topk_rows_at_any_two_byte_address(V):
    import paper_2601_12212_amd as dt
    rng = np.random.default_rng(V)
    R, k = 5, 12
    buf = dt_synth.f32_to_bf16_bits((rng.standard_normal((R, V + 3)) * 3).astype(np.float32))
    val = torch.empty((R, k), dtype=torch.float32, device="cuda")
    idx = torch.empty((R, k), dtype=torch.int32, device="cuda")
    lse = torch.empty(R, dtype=torch.float32, device="cuda")
    ws = torch.zeros(dt.dt_workspace_bytes(1, R, V, 8, 1, 64), dtype=torch.uint8, device="cuda")
    dt.dt_topk_rows(dev_logits(buf)[:, 1:V + 1], k, val, idx, lse, ws)
    torch.cuda.synchronize()
    wval, widx, _ = ref.topk_rows(np.ascontiguousarray(buf[:, 1:V + 1]), k)
    assert np.array_equal(idx.cpu().numpy(), widx) and np.array_equal(val.cpu().numpy(), wval)


@pytest.mark.parametrize("V", [7, 9, 301, 2047, 8193, 16383, 20001, 40001, 128257])
@pytest.mark.parametrize("gap", [0, 2])
def test_topk_rows_of_odd_vocabularies(V, gap):
    # every other row begins at an odd two-byte address and is read from the entry before it on (with a gap a large one)
    check_repeated_rows(V, 14, True, gap) if V > 8 else check_topk(dt_synth.f32_to_bf16_bits(np.random.default_rng(V).standard_normal((14, V)).astype(np.float32)), 3)


@pytest.mark.parametrize("V", [7, 9, 301, 2049, 8193, 16383, 20001, 128257])
@pytest.mark.parametrize("mode", [dt_synth.GREEDY, dt_synth.STOCHASTIC, dt_synth.SAMPLED])
def test_target_rows_at_odd_addresses(V, mode):
    # the same rows at even and at odd two-byte addresses behind a large entry: the best first, last, everywhere, nowhere
    from paper_2601_12212_amd.step import Step
    B, TT = 3, 24
    st = Step([(TT, 4, 5)] * B, [1] * B, 1, 1, 64, V, mode=mode, temperature=0.7)
    gen = torch.Generator("cuda").manual_seed(V)
    st.draft_logits.copy_(torch.randn(st.draft_logits.shape, generator=gen, device="cuda") * 2)
    st.build_tree()
    x = (torch.randn((B, TT, V), generator=gen, device="cuda") * 2).bfloat16()
    x[:, 1, 0] = 30.0
    x[:, 2, V - 1] = 30.0
    x[:, 3] = 1.0
    if mode == dt_synth.GREEDY:
        x[:, 4] = -float("inf")
    got = []
    for gap in (7, 2):  # V is odd: rows at even and at odd addresses
        st.target_logits = torch.nn.functional.pad(x, (0, gap), value=100.0)[:, :, :V]
        st.accept()
        torch.cuda.synchronize()
        got.append([t.clone() for t in (st.accept_len, st.best_node, st.path_nodes, st.out_tokens, st.node_argmax)])
    for even, odd in zip(*got):
        assert torch.equal(even, odd)
    if mode != dt_synth.SAMPLED:
        n = st.n_nodes.tolist()
        for b in range(B):
            # the first of equal entries
            assert torch.equal(got[1][4][b, :n[b]].long().cpu(), torch.from_numpy(np.argmax(x[b, :n[b]].float().cpu().numpy(), axis=1)))


# Target rows that the acceptance reduces itself: up to 16 nodes and 2,048 entries, a wave to a row of up to four groups of 512; one more of either.  Against the oracle,
# and rows whose best is first, last, everywhere and nowhere against numpy.
@pytest.mark.parametrize("V", [8, 9, 511, 513, 1024, 2047, 2048, 2049])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("mode", [dt_synth.GREEDY, dt_synth.STOCHASTIC])
def test_target_rows_that_the_acceptance_reduces(V, bf16, mode):
    from paper_2601_12212_amd.step import Step
    for TT in (1, 15, 16, 17):
        cfg = dt_synth.StepConfig("rows", "bf16" if bf16 else "f32", 2, 1, 64, V, [(TT, 3, 4), (min(TT, 5), 2, 3)], [3, 9], mode=mode, seed=3)
        check_case(oracle_case(0, cfg=cfg))
    TT = 16
    st = Step([(TT, 4, min(5, V - 1))], [1], 1, 1, 64, V, dtype=torch.bfloat16 if bf16 else torch.float32, mode=mode, temperature=0.7)
    gen = torch.Generator("cuda").manual_seed(V)
    st.draft_logits.copy_(torch.randn(st.draft_logits.shape, generator=gen, device="cuda") * 2)
    st.build_tree()
    x = torch.randn((1, TT, V), generator=gen, device="cuda") * 2
    x[:, 1, 0] = x[:, 2, V - 1] = 30.0
    x[:, 3] = 1.0
    x[:, 4, V // 2:] = 3.0e4
    if mode == dt_synth.GREEDY:
        x[:, 5] = -float("inf")
    for gap in (0, 1):
        st.target_logits = torch.nn.functional.pad(x.to(st.draft_logits.dtype), (0, gap), value=1e9)[:, :, :V]
        st.accept()
        n = int(st.n_nodes[0])
        want = np.argmax(st.target_logits[0, :n].float().cpu().numpy(), axis=1)   # the first of equal entries
        assert torch.equal(st.node_argmax[0, :n].long().cpu(), torch.from_numpy(want))


# The most sequences whose rows the acceptance reduces itself, and one more, of up to 120 KB of rows and of more; room for a node more has a launch of rows.
@pytest.mark.parametrize("B,V", [(256, 1001), (257, 1001), (16, 2048), (17, 2048)])
def test_target_rows_of_many_sequences(B, V):
    got = [[t.clone() for t in (st.accept_len, st.best_node, st.out_tokens, st.node_argmax[:, :5])] for st in accepted(B, V, dt_synth.GREEDY)]
    assert all(torch.equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("mode", [dt_synth.GREEDY, dt_synth.STOCHASTIC])
def test_target_rows_of_many_sequences_do_not_come_in_turns(mode):
    """Equal times; with the rows of 320 sequences reduced by the acceptance, one and a half times as long as by a launch of rows."""
    sides = accepted(320, 2048, mode)
    times = [[], []]
    for _ in range(15):
        for st, of in zip(sides, times):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            a.record()
            st.graph.replay()
            b.record()
            torch.cuda.synchronize()
            of.append(a.elapsed_time(b))
    took = [sorted(of)[7] for of in times]
    assert took[0] <= 1.25 * took[1], took


def accepted(B, V, mode):
    """Steps whose trees, three to five nodes of fp32 rows, have been accepted, once in room for 16 nodes and once for 17; and graphs of 20 acceptances."""
    from paper_2601_12212_amd.step import Step
    sides = []
    for cap in (16, 17):
        gen = torch.Generator("cuda").manual_seed(V)
        st = Step([(3 + b % 3, 4, 5) for b in range(B)], [1] * B, 1, 1, 64, V, dtype=torch.float32, mode=mode, temperature=0.7, TT_cap=cap)
        st.draft_logits.copy_(torch.randn(st.draft_logits.shape, generator=gen, device="cuda") * 3)
        st.build_tree()
        st.target_logits[:, :5].copy_(torch.randn((B, 5, V), generator=gen, device="cuda") * 3)
        for i in range(1, 5):   # most nodes are their parents' best
            par = st.parents[:, i].clamp(min=0).long()
            at = torch.arange(B, device="cuda")
            st.target_logits[at, par, st.tokens[:, i].clamp(min=0).long()] += 30.0 * (at % 4 != i % 4) * (st.parents[:, i] >= 0)
        st.node_argmax.fill_(-3)
        st.accept()
        torch.cuda.synchronize()
        st.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(st.graph):
            for _ in range(20):
                st.accept()
        sides.append(st)
    return sides


# Draft rows that the tree kernel reduces itself, a wave to a row: up to eight rows of 2,048 entries.  Against the general path, which a ninth row that belongs to no tree
# selects; log-sum-exps of sums in another order differ by two ulp of 10 at most.  Rows whose best are more neighbours than a list holds, equal, few and none.
@pytest.mark.parametrize("V", [8, 9, 63, 511, 513, 1024, 2047, 2048])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("params", [[(16, 3, 3)], [(16, 2, 7)], [(30, 3, 3), (1, 2, 2)], [(20, 2, 32)]])
def test_draft_rows_that_the_tree_kernel_reduces(V, bf16, params):
    from paper_2601_12212_amd.step import Step
    B, R = len(params), min(8, 1 + (params[0][1] - 1) * params[0][2])       # of 33 rows all but eight do not exist
    total = R + B - 1
    gen = torch.Generator("cuda").manual_seed(V + R)
    x = torch.randn((total + 9, V), generator=gen, device="cuda") * 3
    x[1, :min(V, 100)] += 20.0
    x[2] = x[2].round()
    x[3] = 1.0
    x[4, 3:] = -float("inf")
    x[5] = -float("inf")
    got = []
    for gap in (0, 1):
        for n in (total, total + 9):
            st = Step(params, [1] * B, 1, 1, 64, V, dtype=torch.bfloat16 if bf16 else torch.float32)
            st.draft_logits, st.total_rows = torch.nn.functional.pad(x[:n].to(st.draft_logits.dtype), (0, gap), value=1e9)[:, :V], n
            st.ws = torch.empty(dt_workspace_bytes(B, n, V, st.TT_cap, 1, 64), dtype=torch.uint8, device="cuda")
            st.row_off.copy_(torch.tensor([0, R, total][:B + 1]))
            st.root_token.fill_(1)
            st.build_tree()
            N = st.n_nodes.tolist()
            got.append([st.n_nodes.clone()] + [t[b, :N[b]].clone() for b in range(B) for t in (st.tokens, st.parents, st.depth, st.src_row, st.anc_mask, st.score, st.logp)])
    for other in got[1:]:
        for u, v in zip(got[0], other):
            if u.dtype == torch.float32:
                assert torch.allclose(u, v, rtol=2e-6, atol=2e-6)
            else:
                assert torch.equal(u, v)


# The most sequences whose rows the tree kernel reduces itself, and one more.
@pytest.mark.parametrize("B", [256, 257])
def test_draft_rows_of_many_sequences(B):
    from paper_2601_12212_amd.step import Step
    got, V = [], 1001
    for more in (0, 9):   # nine rows that belong to no tree: a launch of rows
        st = Step([(8, 1, 5)] * (B - 1) + [(16, 2, 7)], [1] * B, 1, 1, 64, V)
        gen = torch.Generator("cuda").manual_seed(B)
        st.total_rows += more
        st.draft_logits = torch.randn((st.total_rows, V), generator=gen, device="cuda").mul_(3).bfloat16()
        st.ws = torch.empty(dt_workspace_bytes(B, st.total_rows, V, st.TT_cap, 1, 64), dtype=torch.uint8, device="cuda")
        st.build_tree()
        got.append([t.clone() for t in (st.n_nodes, st.tokens, st.parents, st.depth, st.src_row, st.anc_mask, st.score, st.logp)])
    assert got[0][0].tolist() == [6] * (B - 1) + [16]
    for a, b in zip(*got):
        assert torch.allclose(a, b, rtol=2e-6, atol=2e-6) if a.dtype == torch.float32 else torch.equal(a, b)


def test_a_launch_of_more_threads_than_one_grid_dimension_takes():
    # 2^22 rows, each held by a workgroup of 1,024 threads; all but the tree's own rows belong to no tree (and are not read)
    from paper_2601_12212_amd.step import Step
    n, V, TT, d, k = 1 << 22, 8193, 30, 4, 5
    if torch.cuda.mem_get_info()[0] < 110e9:
        pytest.skip("needs 92 GB of device memory")
    rows = dt_synth.f32_to_bf16_bits((np.random.default_rng(8).standard_normal((1 + (d - 1) * k, V)) * 3).astype(np.float32))
    want = ref.build_tree(rows, TT, d, k, 3)
    assert want["min_margin"] >= TREE_MARGIN
    st = Step([(TT, d, k)], [1], 4, 4, 64, V)
    st.draft_logits, st.total_rows = torch.empty((n, V), dtype=torch.bfloat16, device="cuda"), n
    st.ws = torch.empty(dt_workspace_bytes(1, n, V, TT, 4, 64), dtype=torch.uint8, device="cuda")
    st.set_draft(0, rows)
    st.set_root_token(0, 3)
    st.build_tree()
    assert_tree_equal(st.tree(0), want)
    del st
    torch.cuda.empty_cache()


def times_in_turn(xs, k, n=20):
    """Of calls on each of xs: medians over replays of graphs of n calls, one after the other so that they share the machine's state."""
    import paper_2601_12212_amd as dt
    graphs = []
    for x in xs:
        R, V = x.shape
        out = (torch.empty((R, k), dtype=torch.float32, device="cuda"), torch.empty((R, k), dtype=torch.int32, device="cuda"),
               torch.empty(R, dtype=torch.float32, device="cuda"),
               torch.zeros(dt.dt_workspace_bytes(1, R, V, 8, 1, 64), dtype=torch.uint8, device="cuda"))
        dt.dt_topk_rows(x, k, *out)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(n):
                dt.dt_topk_rows(x, k, *out)
        graphs.append((graph, out))
    times = [[] for _ in xs]
    for _ in range(20):
        for (graph, _out), of in zip(graphs, times):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            graph.replay()
            b.record()
            torch.cuda.synchronize()
            of.append(a.elapsed_time(b))
    return [sorted(of)[10] / n for of in times]


# Neighbours, and how many times as long as rows without them a call may take.  1.04 and 2.2 where they are spread over the slots of the
# bound and where they fall into few of them; 1.12 and 1.65 with the hits of a lane written in a row and in a loop; 2.9 and 250 with
# one pass over them and k over the row where fewer pairs of lanes than k hold them; 1.18 and 1.8 with room for 256 and 128 of them.
@pytest.mark.parametrize("n,V,k,M,times", [(51, 128256, 10, 512, 1.6), (51, 128256, 10, 1024, 1.6), (28, 115042, 28, 32, 1.45), (51, 128256, 28, 256, 6), (51, 128256, 28, 100, 1.55)])
def test_neighbours_among_the_best_do_not_slow_top_k_rows_down(n, V, k, M, times):
    x = torch.randn((n, V), generator=torch.Generator("cuda").manual_seed(M), device="cuda") * 3
    plain = x.bfloat16()
    x[:, 1000:1000 + M] += 20
    took = times_in_turn([x.bfloat16(), plain], k)
    assert took[0] <= times * took[1], took


@pytest.mark.parametrize("n,V", [(2000, 8000), (2600, 2048), (300, 16384), (200, 30000)])
def test_ties_of_large_launches_are_not_looked_up_in_memory(n, V):
    """5 to 7 times as long as rows of differing values; 35 to 75 with every step of the search over the row in memory."""
    x = torch.randn((n, V), generator=torch.Generator("cuda").manual_seed(5), device="cuda").bfloat16()
    took = times_in_turn([torch.ones_like(x), x], 24, 5)
    assert took[0] <= 12 * took[1], took


def test_large_calls_of_short_chunks_are_not_one_chunk_to_a_workgroup():
    """1,990 rows 1.25 times as long as 1,100, which take one; 1.55 if they did so too."""
    x = torch.randn((1990, 26944), generator=torch.Generator("cuda").manual_seed(5), device="cuda").bfloat16()
    took = times_in_turn([x, x[:1100]], 12)
    assert took[0] <= 1.4 * took[1], took


def test_top_k_rows_whose_best_are_in_one_part_take_no_longer():
    """0.99 times as long as rows whose best are anywhere; 1.4 with a quarter of the row to a wave."""
    x = torch.randn((51, 128256), generator=torch.Generator("cuda").manual_seed(5), device="cuda") * 3
    falling = x - torch.linspace(0, 12, 128256, device="cuda")
    took = times_in_turn([falling.bfloat16(), x.bfloat16()], 28)
    assert took[0] <= 1.2 * took[1], took


# How many neighbours hold all of the best: fewer pairs of lanes than k (the first two bounds do not cut), as many as the list of
# candidates has places and one more, and more.
@pytest.mark.parametrize("M", [40, 127, 128, 129, 200, 255, 256, 257, 500, 3000])
@pytest.mark.parametrize("V,bf16", [(20000, False), (40001, True), (128256, True), (131081, False)])
def test_topk_rows_whose_best_are_neighbours(V, M, bf16):
    rng = np.random.default_rng(M)
    x = (rng.standard_normal((7, V)) * 3).astype(np.float32)
    at = V // 3
    x[0, at:at + M] += 20.0
    x[1, at:at + M] = 20.0                                    # equal: the smallest ids
    x[2, at:at + M] = 20.0 + rng.integers(0, 2, M)            # two values
    # Many octaves.  (Not past 2^25: the log-sum-exp's exponents are x log2e rounded once, off by 2^-24 |x|, and no longer those of the
    # maximum, 0, and the others, some 100 below, from 2^30 on.)
    x[3, at:at + M] = np.exp2(rng.uniform(5, 25, M))
    x[4] = -np.inf
    x[4, at:at + M] = rng.standard_normal(M)                  # the only viable entries
    x[5] = -x[0]                                              # the worst
    x[6] = 1.0 + 2.0 ** -20 * rng.integers(0, 300, V)         # one leading half of the key (bf16: equal everywhere)
    for k in (1, 13, 32):
        check_topk(dt_synth.f32_to_bf16_bits(x) if bf16 else x, k)
