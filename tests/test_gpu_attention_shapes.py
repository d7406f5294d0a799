"""GPU parity of the attention kernels that serve 64-wide heads (matrix cores) and every other head size (plain ALU), at
the edges of their tiles: row counts around 32, key counts around a block, key splits, and head sizes around the widths
that decide how a row is loaded; and of the large-batch schedule where it cuts sequences into key ranges."""
import numpy as np
import pytest

import dt_synth
from oracle import ref
from tests._cases import oracle_case
from tests.test_gpu_parity import assert_attention, check_case, make_step

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _cfg(dtype, D, params, prefix_len, Hq, Hkv):
    return dt_synth.StepConfig("shape", dtype, Hq, Hkv, D, 1031, params, prefix_len, seed=5)


@pytest.mark.parametrize("Hq,Hkv", [(4, 4), (14, 2), (8, 1)])
@pytest.mark.parametrize("prefix_len", [[0, 1, 31], [32, 33, 64], [700, 1500, 5]])
def test_heads_of_64(Hq, Hkv, prefix_len):
    # 1, 32 and 65 nodes: with 1, 7 or 8 query heads per kv head the 32-row blocks are full, ragged and nearly empty; the
    # long prefixes split their keys over several workgroups, the short ones do not
    check_case(oracle_case(0, cfg=_cfg("bf16", 64, [(1, 1, 1), (32, 5, 6), (65, 4, 6)], prefix_len, Hq, Hkv)))


def test_heads_of_64_large_batch_and_head_major():
    rng = np.random.default_rng(6)
    params = [(int(rng.choice([1, 17, 40, 96])), 4, 5) for _ in range(40)]
    plen = [int(rng.choice([0, 63, 130, 400])) for _ in range(40)]
    case = oracle_case(0, cfg=_cfg("bf16", 64, params, plen, 16, 4))
    check_case(case)
    check_case(case, kv_head_major=True)


@pytest.mark.parametrize("dtype,D", [("f32", D) for D in (1, 3, 4, 20, 63, 64, 65, 68, 127, 128)] +
                         [("bf16", D) for D in (7, 8, 20, 72, 80, 96, 112)])
def test_plain_kernel_head_sizes(dtype, D):
    # rows shorter than one 16-byte load, a multiple of it or not, one and two columns per lane; key counts below, at and
    # past one block, and enough for every wave to have several
    check_case(oracle_case(0, cfg=_cfg(dtype, D, [(1, 1, 1), (20, 4, 3), (70, 4, 6)], [0, 44, 600], 4, 2)))


@pytest.mark.parametrize("plen", [[5000] + [0, 1, 63, 64, 65] * 4, [300 + 97 * (i % 23) for i in range(64)]],
                         ids=["one_long", "batch_64"])
def test_balanced_schedule_cut_sequences(plen):
    # one sequence cut into many key ranges among short ones, and the largest batch that the schedule takes; the partials are
    # merged by whichever workgroup comes last, with the same bits each time and whatever the workspace held before
    params = [(1 if i % 7 == 3 else 30 + 3 * (i % 5), 4, 6) for i in range(len(plen))]
    case = oracle_case(0, cfg=_cfg("bf16", 128, params, plen, 8, 8))
    check_case(case)
    st = make_step(case)
    st.build_tree()
    st.tree_attention()
    first = st.out.clone()
    for fill in (0x00, 0xff, 0x3f):
        st.ws.fill_(fill)
        st.out.fill_(7.0)
        st.tree_attention()
        for b in range(len(plen)):
            n = case.trees[b]["n_nodes"]
            assert torch.equal(st.out[b, :n].view(torch.int16), first[b, :n].view(torch.int16)), (b, fill)


@pytest.mark.parametrize("Hq,Hkv", [(4, 4), (14, 2)])
@pytest.mark.parametrize("prefix_len", [[0, 1, 31], [700, 1500, 5], [4000, 300, 64]])
def test_heads_of_64_keep_their_probabilities_in_32_bits(Hq, Hkv, prefix_len):
    # against 64-bit arithmetic: one rounding of the result to bf16 (half an ulp, at most 2^-8 of it), and 32-bit scores,
    # exponentials and sums, whose relative errors (some 2^-21 where scores reach 8 binary orders) weigh sum_j p_j |v_j|.
    # Probabilities rounded to bf16 would be off by up to 2^-9 of that sum.
    cfg = _cfg("bf16", 64, [(1, 1, 1), (32, 5, 6), (65, 4, 6)], prefix_len, Hq, Hkv)
    case = oracle_case(0, cfg=cfg)
    st = make_step(case)
    st.build_tree()
    st.tree_attention()
    for b in range(cfg.B):
        n = case.trees[b]["n_nodes"]
        q, kt, vt, kp, vp = (torch.from_numpy(dt_synth.as_f32(x).copy()).double() for x in dt_synth.qkv(cfg, b))
        k, v = torch.cat([kp, kt[:n]]), torch.cat([vp, vt[:n]])
        words = case.trees[b]["anc_mask"]
        tree = torch.tensor([[int(words[i, j // 64]) >> (j % 64) & 1 for j in range(n)] for i in range(n)], dtype=torch.bool)
        sees = torch.cat([torch.ones(n, kp.shape[0], dtype=torch.bool), tree], 1)
        got = st.out[b, :n].double().cpu()
        for h in range(Hq):
            g = h // (Hq // Hkv)
            s = (q[:n, h] @ k[:, g].t() * st.scale).masked_fill(~sees, -np.inf)
            p = torch.softmax(s, 1)
            want, weight = p @ v[:, g], p @ v[:, g].abs()
            over = (got[:, h] - want).abs() - want.abs() * 2.0 ** -8 - weight * 2.0 ** -19
            assert float(over.max()) <= 0, (b, h, float(over.max()))


@pytest.mark.parametrize("Hq,Hkv", [(4, 4), (14, 2)])
@pytest.mark.parametrize("L", [0, 45, 1410])
def test_heads_of_64_do_not_multiply_the_values_of_hidden_keys(Hq, Hkv, L):
    # infinities and a NaN in V of one tree token (one in the middle, and the last, which also pads the last block): the nodes
    # that see it get them, the others what they get without them, up to the order of 32-bit sums.  Visible everywhere when
    # they stand in the prefix.
    cfg = _cfg("bf16", 64, [(65, 4, 6)], [L], Hq, Hkv)
    case = oracle_case(0, cfg=cfg)
    st = make_step(case)
    st.build_tree()
    st.tree_attention()
    n = case.trees[0]["n_nodes"]
    clean = st.out[0, :n].float()
    words = case.trees[0]["anc_mask"]
    odd = torch.tensor([float("inf"), float("-inf"), float("nan")], device="cuda")

    def check(sees, what):
        st.tree_attention()
        got = st.out[0, :n].float()
        seen = got[sees][:, :, 10:13]
        assert bool((torch.isposinf(seen[..., 0]) & torch.isneginf(seen[..., 1]) & torch.isnan(seen[..., 2])).all()), what
        got[:, :, 10:13] = torch.where(sees[:, None, None], clean[:, :, 10:13], got[:, :, 10:13])
        # one bf16 ulp of the result: both sides are one rounding of 32-bit sums
        assert bool(((got - clean).abs() <= clean.abs() * 2.0 ** -7 + 1e-6).all()), what

    for j in (n // 2, n - 1):
        keep = st.v_tree[0, j].clone()
        st.v_tree[0, j, :, 10:13] = odd.to(st.v_tree.dtype)
        sees = torch.tensor([bool(int(words[i, j // 64]) >> (j % 64) & 1) for i in range(n)], device="cuda")
        assert 0 < int(sees.sum()) < n
        check(sees, j)
        st.v_tree[0, j] = keep
    for t in {0, L // 2, L - 1} if L else ():
        keep = st.v_prefix[0][t].clone()
        st.v_prefix[0][t, :, 10:13] = odd.to(st.v_prefix[0].dtype)
        check(torch.ones(n, dtype=torch.bool, device="cuda"), "prefix %d" % t)
        st.v_prefix[0][t] = keep


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("L", [330, 700, 1060, 1410, 1760, 2110, 2460, 2810])
def test_an_infinite_value_in_any_key_split(D, L):
    # one short sequence: its keys are dealt over 1 to 8 workgroups (the more, the longer it is) and the partials merged;
    # an infinite V element of a visible prefix key makes that column infinite, whichever split holds the key
    cfg = _cfg("bf16", D, [(32, 5, 6)], [L], 4, 4)
    case = oracle_case(0, cfg=cfg)
    st = make_step(case)
    st.build_tree()
    st.tree_attention()
    n = case.trees[0]["n_nodes"]
    clean = st.out[0, :n].clone()
    keep = st.v_prefix[0].clone()
    for block in range(0, L // 32, 3):
        st.v_prefix[0].copy_(keep)
        st.v_prefix[0][32 * block + block % 32, :, 5] = float("inf")
        st.tree_attention()
        got = st.out[0, :n]
        assert bool(torch.isposinf(got[:, :, 5]).all()), block
        a, b = (x[:, :, [c for c in range(D) if c != 5]].float() for x in (got, clean))
        # 64-wide heads take the second product of that block in another order: one bf16 ulp of the result
        over = (a - b).abs() - (b.abs() * 2.0 ** -7 + 1e-6 if D == 64 else 0.0)
        w = int(over.argmax())
        assert float(over.max()) <= 0, (block, w, float(a.flatten()[w]), float(b.flatten()[w]))


@pytest.mark.parametrize("B,Hq,Hkv,TT,long", [(16, 14, 2, 64, 6000), (64, 2, 2, 40, 5000), (16, 32, 8, 96, 7000)])
def test_balanced_schedule_merges_of_many_parts(B, Hq, Hkv, TT, long):
    # one long sequence among short ones, cut into 50, 80 and 18 key ranges of one sequence: the merge is shared by the
    # workgroups that are there.  Against the oracle; then the same bits whatever the workspace held before, and from a replayed
    # graph whose launch keeps its number while lengths (so what is cut where) and workspace change between the replays.
    params = [(TT if b % 5 < 4 else 9, 5, 6) for b in range(B)]
    case = oracle_case(0, cfg=_cfg("bf16", 128, params, [long] + [7 + 40 * (b % 5) for b in range(1, B)], Hq, Hkv))
    st = check_case(case)
    lengths = [st.prefix_len.clone()]
    for cut in (2, 64):
        lengths.append(torch.clamp(lengths[0] // cut, min=1))

    def run():
        st.tree_attention()
        return [st.out[b, :case.trees[b]["n_nodes"]].view(torch.int16).clone() for b in range(B)]

    want = []
    for plen in lengths:
        st.prefix_len.copy_(plen)
        want.append(run())
        for fill in (0x00, 0xff, 0x3f):
            st.ws.fill_(fill)
            st.out.fill_(7.0)
            assert all(torch.equal(x, y) for x, y in zip(run(), want[-1])), fill
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        g = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(g, stream=side):
            st.tree_attention()
    for rep, (which, fill) in enumerate([(0, None), (0, None), (1, None), (2, 0x5a), (1, None), (0, 0xff), (0, None)]):
        st.prefix_len.copy_(lengths[which])
        if fill is not None:
            st.ws.fill_(fill)
        st.out.fill_(7.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        got = [st.out[b, :case.trees[b]["n_nodes"]].view(torch.int16) for b in range(B)]
        assert all(torch.equal(x, y) for x, y in zip(got, want[which])), rep


def test_shared_merge_at_its_edges():
    # one block to a part: a sequence of n blocks has n parts.  The most that one workgroup merges and one more, the parts that
    # are in flight together, the marks that a wave looks at together
    B, TT = 64, 40
    cfg = _cfg("bf16", 128, [(TT, 5, 6)] * B, [64 * 80 - TT] + [7 + 40 * (b % 3) for b in range(1, B)], 2, 2)
    case = oracle_case(0, cfg=cfg)
    st = make_step(case)
    st.build_tree()
    n = case.trees[0]["n_nodes"]
    assert n == TT
    q, kt, vt, kp, vp = dt_synth.qkv(cfg, 0)
    for blocks in (8, 9, 16, 17, 32, 33, 64, 65, 80):
        L = 64 * blocks - TT
        st.prefix_len[0] = L
        st.tree_attention()
        want = ref.tree_attention(q[:n], kt[:n], vt[:n], kp[:L], vp[:L], case.trees[0]["anc_mask"], st.scale)
        assert_attention(st.attention_out(0), want, "bf16", "%d parts" % blocks)


# four units (a kv head's 32 rows each) in two to eight splits; 72 and 100 of them, with room for three and two
@pytest.mark.parametrize("D,Hkv,L", [(128, 4, L) for L in (224, 225, 352, 353, 480, 608, 736, 864, 992)] +
                         [(128, 72, L) for L in (288, 289, 353, 481)] + [(128, 100, L) for L in (352, 353, 481)] +
                         [(64, 4, L) for L in (864, 865, 993, 1121, 1500, 1800)] + [(64, 72, 865), (64, 100, 1856), (64, 100, 1857)])
def test_numbers_of_key_splits(D, Hkv, L):
    check_case(oracle_case(0, cfg=_cfg("bf16", D, [(32, 5, 6)], [L], Hkv, Hkv)))


# Both sides of the lines where splits begin, and of those where two become three, three four and two (or three) one again: blocks of 32 keys, the last of one
# key, whole, or one less; with room for eight, three and two.  And 129 units, which have room for one.
@pytest.mark.parametrize("D,Hkv,blocks", [(128, 4, n) for n in (5, 6, 8, 9, 12, 13, 16, 17)] + [(128, 72, n) for n in (12, 13, 16, 17)] + [(128, 100, n) for n in (5, 6, 8, 9, 12, 13)] +
                         [(64, 4, n) for n in (12, 13, 16, 17)] + [(64, 72, n) for n in (16, 17)] + [(64, 100, n) for n in (28, 29, 32, 33, 36, 37)] + [(128, 129, 20), (64, 129, 40)])
def test_lines_where_key_splits_begin(D, Hkv, blocks):
    for L in (32 * (blocks - 1), 32 * (blocks - 1) - 31, 32 * (blocks - 1) - 1):   # and 32 nodes
        check_case(oracle_case(0, cfg=_cfg("bf16", D, [(32, 5, 6)], [L], Hkv, Hkv)))


# Splits of a row block that meet in one XCD, in two to eight; and, 84 row blocks in three splits, the last four of them spread over the XCDs, where
# partials go by the memory side.  Rows and keys that end early (one sequence of one node), the same bits whatever the workspace
# held before and from a replayed graph whose launch keeps its number, lengths and workspace changing between the replays.
@pytest.mark.parametrize("D,Hkv,B,L", [(128, 4, 1, 700), (128, 4, 1, 330), (64, 4, 1, 1300), (128, 20, 1, 1000), (64, 28, 3, 1100), (128, 28, 3, 460)])
def test_key_splits_meet(D, Hkv, B, L):
    params = [(32, 5, 6) if b != 1 else (1, 1, 1) for b in range(B)]
    case = oracle_case(0, cfg=_cfg("bf16", D, params, [L - 7 * b for b in range(B)], Hkv, Hkv))
    st = check_case(case)
    lengths = [st.prefix_len.clone(), torch.clamp(st.prefix_len // 3, min=1)]

    def run():
        st.tree_attention()
        return [st.out[b, :case.trees[b]["n_nodes"]].view(torch.int16).clone() for b in range(B)]

    want = []
    for plen in lengths:
        st.prefix_len.copy_(plen)
        want.append(run())
        for fill in (0x00, 0xff, 0x3f):
            st.ws.fill_(fill)
            st.out.fill_(7.0)
            assert all(torch.equal(x, y) for x, y in zip(run(), want[-1])), fill
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        g = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(g, stream=side):
            st.tree_attention()
            st.tree_attention()
    for rep, (which, fill) in enumerate([(0, None), (0, None), (1, None), (0, 0x5a), (1, 0xff), (0, None)]):
        st.prefix_len.copy_(lengths[which])
        if fill is not None:
            st.ws.fill_(fill)
        st.out.fill_(7.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        got = [st.out[b, :case.trees[b]["n_nodes"]].view(torch.int16) for b in range(B)]
        assert all(torch.equal(x, y) for x, y in zip(got, want[which])), rep


# one sequence far longer than the others, in every kernel: the balanced schedule (320 and 512 row blocks, four to a kv head), the small-batch kernel with key
# splits (256, two and one to a kv head) and whole tiles (320, two to a kv head; 260, one, more tiles than compute units).  (The lines between the kernels lie
# elsewhere: test_lines_between_the_three_kernels and the two before it.)
@pytest.mark.parametrize("B,Hq,Hkv,L", [(B, Hq, Hkv, L + i) for B, Hq, Hkv, L in ((40, 8, 2, 6816), (64, 8, 2, 1824), (32, 8, 4, 4768), (40, 8, 4, 608),
                                                                                 (64, 4, 4, 6368)) for i in (0, 1)] +
                         [(52, 5, 5, 150)])
def test_lines_between_the_two_kernels(B, Hq, Hkv, L):
    check_case(oracle_case(0, cfg=_cfg("bf16", 128, [(32, 5, 6)] * B, [L] + [7 + 40 * (b % 3) for b in range(1, B)], Hq, Hkv)))


# Plans of the balanced schedule: sequences whole, cut because that is cheaper, and cut because there are fewer slots than tiles.  Four sequences of three
# tiles: whole, in two parts, of differing lengths; with two tiles each, 32 sequences have exactly the slots there are, 33 two too few.
@pytest.mark.parametrize("Hq,Hkv,plen", [(64, 8, [1300] * 4), (64, 8, [1700] * 4), (64, 8, [2600, 1300, 70, 300]), (32, 8, [1300] + [130, 60] * 15 + [1]),
                                         (32, 8, [1300] + [130, 60] * 16)])
def test_plans_of_the_balanced_schedule(Hq, Hkv, plen):
    check_case(oracle_case(0, cfg=_cfg("bf16", 128, [(40, 4, 6)] * len(plen), plen, Hq, Hkv)))


def test_short_sequences_under_a_long_bound():
    # the bound that the caller gives may be far above the lengths, which the plan then finds: against the oracle, and against the same call with a bound
    # that sends it to the kernel of whole tiles
    B, TT, long = 8, 64, 6000
    cfg = _cfg("bf16", 128, [(TT, 5, 6)] * B, [long] * B, 32, 8)
    case = oracle_case(0, cfg=cfg)
    st = make_step(case)
    st.build_tree()
    n = case.trees[0]["n_nodes"]
    for lengths in ([1, 40, 64 * 4 - n, 64 * 4 - n + 1, 300, 700, 0, 1000], [1100] * B):
        for b, L in enumerate(lengths):
            st.prefix_len[b] = L
        st.tree_attention()
        for b in (0, 2, 3, 7):
            q, kt, vt, kp, vp = dt_synth.qkv(cfg, b)
            want = ref.tree_attention(q[:n], kt[:n], vt[:n], kp[:lengths[b]], vp[:lengths[b]], case.trees[b]["anc_mask"], st.scale)
            assert_attention(st.attention_out(b), want, "bf16", "%d keys" % lengths[b])


def test_shared_merge_of_a_dozen_to_thirty_parts():
    # one sequence of 90 to 210 blocks among 63 of 22, six or seven blocks to a part: the counts around those that are read together
    B, TT = 64, 40
    cfg = _cfg("bf16", 128, [(TT, 5, 6)] * B, [64 * 210 - TT] + [1368] * (B - 1), 2, 2)
    case = oracle_case(0, cfg=cfg)
    st = make_step(case)
    st.build_tree()
    n = case.trees[0]["n_nodes"]
    assert n == TT
    q, kt, vt, kp, vp = dt_synth.qkv(cfg, 0)
    for blocks in range(90, 211, 8):
        L = 64 * blocks - TT
        st.prefix_len[0] = L
        st.tree_attention()
        want = ref.tree_attention(q[:n], kt[:n], vt[:n], kp[:L], vp[:L], case.trees[0]["anc_mask"], st.scale)
        assert_attention(st.attention_out(0), want, "bf16", "%d blocks" % blocks)


@pytest.mark.parametrize("B", [32, 33])
def test_whole_tiles_of_every_length(B):
    # 256 tiles, one to a compute unit, four K and V tiles in LDS, and 264, two: ranges of one to a dozen 64-key blocks, ragged and not
    TT = 40
    lens = [0, 1, 23, 24, 25, 80, 88, 89] + [64 * n - TT + (n % 3 - 1) * (n % 2) for n in range(3, 27)] + [500]
    check_case(oracle_case(0, cfg=_cfg("bf16", 128, [(TT, 5, 6)] * B, lens[:B], 8, 8)))


# 152 tiles, a compute unit to each, are whole up to 56 blocks of 32 keys
@pytest.mark.parametrize("L", [1752, 1753])
def test_line_of_a_tile_to_each_compute_unit(L):
    check_case(oracle_case(0, cfg=_cfg("bf16", 128, [(40, 5, 6)] * 19, [L] + [7 + 90 * b for b in range(1, 19)], 8, 8)))


# few tiles: up to 144 the small-batch kernel keeps 320 row blocks, and 400 from 33 blocks of 32 keys on (152 tiles of 304 row blocks; 120 of 400 at 32 and
# 33 blocks, of 440; 144 of 288 at 56 and 57)
@pytest.mark.parametrize("Hq,B,TT,L", [(8, 19, 40, 300), (8, 18, 40, 300), (32, 5, 80, 944), (32, 5, 80, 945), (32, 5, 81, 1000), (8, 18, 40, 1752), (8, 18, 40, 1753)])
def test_lines_of_few_tiles(Hq, B, TT, L):
    check_case(oracle_case(0, cfg=_cfg("bf16", 128, [(TT, 5, 6)] * B, [L] + [7 + 40 * (b % 5) for b in range(1, B)], Hq, 8)))


# 256 (sequence, kv head, 32-row block)s, which the small-batch kernel takes, and 264, which the kernel of whole tiles takes up to 40 blocks of 32 keys and the
# balanced schedule from 41 on
@pytest.mark.parametrize("B,L", [(32, 1248), (33, 100), (33, 1248), (33, 1249)])
def test_lines_between_the_three_kernels(B, L):
    check_case(oracle_case(0, cfg=_cfg("bf16", 128, [(32, 5, 6)] * B, [L] + [7 + 40 * (b % 3) for b in range(1, B)], 8, 8)))


# Shapes of the kernel of whole tiles, and of the balanced schedule with sequences whole and cut.
FAR = {"whole tiles": (8, 8, [60, 300, 700] + [10] * 30), "whole tiles, a compute unit each": (8, 8, [60, 300, 1100] + [10] * 16), "schedule, whole": (8, 8, [1250, 300, 700] + [10] * 30),
       "schedule, cut": (64, 8, [1700, 1700, 1500, 1600])}


@pytest.mark.parametrize("top", [12.0, 60.0])
@pytest.mark.parametrize("shape", list(FAR))
def test_scores_far_above_those_of_the_first_block(shape, top):
    # The softmax reference is that of a range's first block; ranges whose sums come near the end of the exponents are gone through again with a
    # reference that moves.  Scores that climb by some 100 and 600 powers of two along the keys, of one sequence only in the even heads
    Hq, Hkv, plen = FAR[shape]
    cfg = _cfg("bf16", 128, [(40, 4, 6)] * len(plen), plen, Hq, Hkv)
    case = oracle_case(0, cfg=cfg)
    st = make_step(case)
    st.build_tree()
    for b in range(4):
        q, kt, vt, kp, vp = (dt_synth.as_f32(x).copy() for x in dt_synth.qkv(cfg, b))
        N, L = case.trees[b]["n_nodes"], kp.shape[0]
        q[:] = np.abs(q)
        ramp = np.linspace(0.05, top, L + N, dtype=np.float32)[:, None, None]
        heads = slice(0, None, 2) if b == 1 else slice(None)
        kp[:, heads] = np.abs(kp[:, heads]) * ramp[:L]
        kt[:N, heads] = np.abs(kt[:N, heads]) * ramp[L:]
        ops = [dt_synth.f32_to_bf16_bits(x) for x in (q, kt, vt, kp, vp)]
        st.set_qkv(b, *ops)
        st.tree_attention()
        want = ref.tree_attention(ops[0][:N], ops[1][:N], ops[2][:N], ops[3], ops[4], case.trees[b]["anc_mask"], st.scale)
        # nearly all weight on one or two keys with |v| up to 4.5: the rounding of the probabilities, 2^-9, alone is worth 9e-3
        assert_attention(st.attention_out(b), want, "bf16", "%s seq %d" % (shape, b), own_abs=1e-2)


@pytest.mark.parametrize("shape", list(FAR))
def test_values_near_the_end_of_the_exponents(shape):
    # finite values of 1e35 under probabilities that leave their sums finite stay finite, an infinity shows in its column and nowhere else
    Hq, Hkv, plen = FAR[shape]
    cfg = _cfg("bf16", 128, [(40, 4, 6)] * len(plen), plen, Hq, Hkv)
    case = oracle_case(0, cfg=cfg)
    st = make_step(case)
    st.build_tree()
    st.tree_attention()
    n = case.trees[0]["n_nodes"]
    clean = st.out[0, :n].float()
    L = plen[0]
    for value, t in ((1e35, 0), (1e35, L - 1), (float("inf"), 0), (float("inf"), L - 1), (float("nan"), L // 2)):
        keep = st.v_prefix[0][t].clone()
        st.v_prefix[0][t, :, 5] = value
        st.tree_attention()
        got = st.out[0, :n].float()
        column = got[:, :, 5]
        if value == 1e35:
            assert bool((torch.isfinite(column) & (column > 0)).all()), (value, t)
        else:
            assert bool((torch.isposinf(column) if value == float("inf") else torch.isnan(column)).all()), (value, t)
        others = [c for c in range(128) if c != 5]
        # one bf16 ulp of the result: a range gone through again has another reference
        assert bool(((got - clean)[:, :, others].abs() <= clean[:, :, others].abs() * 2.0 ** -7 + 1e-6).all()), (value, t)
        st.v_prefix[0][t] = keep


def low_scores(cfg, st, b, n, L, mask=None, samples=None):
    """Sequence b with its first n nodes and L prefix keys: scores around -80, -89, -100 and -200 in turn from kv head to kv head, the tree's keys
    some natural units above the prefix's, so that both have weight.  Against the oracle."""
    q, kt, vt, kp, vp = (dt_synth.as_f32(x).copy() for x in dt_synth.qkv(cfg, b))
    q, kt, vt, kp, vp = q[:n], kt[:n], vt[:n], kp[:L], vp[:L]
    q[:] = 1.0
    level = np.array([-80.0, -89.0, -100.0, -200.0], np.float32)[np.arange(cfg.Hkv) % 4]
    per_unit = np.float32(1.0 / (st.scale * cfg.D))
    for k, above in ((kp, 0.0), (kt, np.log(max(L, 1)) - 1.0)):
        k *= 0.3
        k += ((level + np.float32(above)) * per_unit)[None, :, None]
    ops = [dt_synth.f32_to_bf16_bits(x) for x in (q, kt, vt, kp, vp)]
    st.set_qkv(b, *ops)
    st.prefix_len[b] = L
    words = np.zeros((n, 2), np.uint64)
    for i in range(n):
        for j in mask(i):
            words[i, j // 64] |= np.uint64(1) << np.uint64(j % 64)
    st.anc_mask[b, :n] = torch.from_numpy(words.view(np.int64)).cuda()
    st.n_nodes[b] = n
    st.tree_attention()
    got = st.out[b, :n].float().cpu().numpy()
    want = ref.tree_attention(*ops, words, st.scale, samples=samples)
    if samples is not None:
        got = got[samples[:, 0], samples[:, 1]]
    # a few keys with nearly all the weight: the bound of scores that climb, above
    assert_attention(got, want, "bf16", "%d keys" % L, own_abs=1e-2)


def test_key_ranges_that_begin_behind_what_a_query_sees():
    # Trees of 128 nodes over 64 n + 20 prefix keys have three blocks of tree keys, and some of these plans cut in front of the second.  A node of the third whose
    # ancestors are in the first then finds nothing in its range's first block, and scores far below 0 behind it.
    plen = [2900, 1900, 2300]
    cfg = _cfg("bf16", 128, [(128, 8, 20)] * 3, plen, 64, 8)
    case = oracle_case(0, cfg=cfg)
    st = make_step(case)
    st.build_tree()
    samples = np.array([(i, 8 * h + i % 8) for i in (0, 43, 44, 107, 108, 113, 120, 127) for h in range(8)], np.int32)
    for L in range(1428, 2900, 64):
        low_scores(cfg, st, 0, 128, L, mask=lambda i: {0, i // 8, i}, samples=samples)


@pytest.mark.parametrize("Hq,Hkv,B,bound", [(8, 8, 33, 100), (8, 8, 19, 100), (64, 8, 4, 2600)], ids=["whole tiles", "whole tiles, a compute unit each", "schedule"])
def test_masks_that_hide_the_first_block(Hq, Hkv, B, bound):
    # no prefix, or a few keys of one, and nodes that see themselves and one more behind the first 64 keys
    cfg = _cfg("bf16", 128, [(128, 8, 20)] + [(40, 4, 6)] * (B - 1), [bound] * B, Hq, Hkv)
    case = oracle_case(0, cfg=cfg)
    st = make_step(case)
    st.build_tree()
    for L, n in ((0, 128), (0, 66), (1, 128), (40, 120)):
        low_scores(cfg, st, 0, n, L, mask=lambda i: {i, max(i - 3, 0)} if i >= 64 else {i})


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,TT", [(65535, 1, 3), (65534, 2, 8), (65535, 3, 16), (12000, 2, 16)])
def test_thousands_of_query_heads_to_a_kv_head(Hq, Hkv, TT, D):
    # rows are told apart by a multiplication with the reciprocal of their number to a node: rounded to 32 bits behind the point, it would find the last rows of a
    # node one too large from about 2^32 / (Hq / Hkv)^2 nodes on (not in the last shape)
    from paper_2601_12212_amd.step import Step
    G, L = Hq // Hkv, 37
    st = Step([(TT, 4, 6)], [L], Hq, Hkv, D, 1031)
    gen = torch.Generator("cuda").manual_seed(TT)
    for t in (st.draft_logits, st.q, st.k_tree, st.v_tree, st.k_prefix[0], st.v_prefix[0]):
        t.copy_(torch.randn(t.shape, generator=gen, device="cuda") * (3.0 if t is st.draft_logits else 1.0))
    st.build_tree()
    st.out.fill_(7.0)
    st.tree_attention()
    assert st.tree(0)["n_nodes"] == TT
    bits = st.anc_mask[0, :, 0, None] >> torch.arange(TT, device="cuda") & 1
    sees = torch.cat([torch.ones((TT, L), dtype=torch.bool, device="cuda"), bits.bool()], 1)
    for h in range(Hkv):
        k, v = (torch.cat([p[0][:, h], t[0, :, h]]).float() for p, t in ((st.k_prefix, st.k_tree), (st.v_prefix, st.v_tree)))
        for i in range(TT):
            q, got = (t[0, i, h * G:(h + 1) * G].float() for t in (st.q, st.out))
            want = torch.softmax((q @ k.t() * st.scale).masked_fill(~sees[i], -float("inf")), 1) @ v
            # one ulp for each side's rounding, and the rounded probabilities of some forty keys
            over = ((got - want).abs() - 2.0 ** -6 * want.abs()).max()
            assert float(over) <= 4e-3, (h, i, float(over))
