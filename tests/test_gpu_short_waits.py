"""The ways out of the hand-overs' waits (csrc/hands.hpp) that a chip of its own hardly ever takes: offers withdrawn, also at the moment when they are
taken, a waiting workgroup that goes, and the last of the others to come doing its work.  A second build of the library, whose waits end after 0
to 1.2 us by the clock, takes all of them, at random, through the tests of the launches that hand over, and through replayed graphs (whose launches keep
their numbers) with other inputs each time, which have to give the bits of the build that waits."""
import contextlib
import importlib.util

import pytest

import paper_2601_12212_amd as dt
from paper_2601_12212_amd import binding
from paper_2601_12212_amd.build import PYCALL_SHORT
from paper_2601_12212_amd.step import Step
from tests import test_gpu_attention_shapes as attention
from tests import test_gpu_levels as levels
from tests import test_gpu_rows_shapes as rows

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

_short = None


@contextlib.contextmanager
def short_waits():
    global _short
    if _short is None:
        spec = importlib.util.spec_from_file_location("_dtcall", PYCALL_SHORT)
        _short = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(_short)
        _short.setup(torch.float32, torch.bfloat16, torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream)
        _short.set_reader(binding._tensor_reader(torch.__version__))
    usual = binding._native()
    binding._call = _short
    try:
        yield
    finally:
        binding._call = usual


CASES = [(rows.test_topk_rows_in_one_launch_of_both_passes, a) for a in
         ((128256, 53, True), (32769, 200, True), (65537, 1, True), (16385, 200, False), (131072, 120, False), (131073, 9, False))] + \
        [(levels.test_levels_chosen_beside_their_rows, a) for a in ((2048, True, 8), (8193, False, 16), (16384, True, 9), (16385, False, 8), (32769, True, 16))] + \
        [(levels.test_level_by_level_of_large_vocabularies, a) for a in ((20000, True), (50001, False), (128256, True))] + \
        [(levels.test_the_level_loop_can_be_captured_and_replayed, ())] + \
        [(attention.test_key_splits_meet, a) for a in ((128, 4, 1, 700), (128, 4, 1, 330), (64, 4, 1, 1300), (128, 20, 1, 1000), (64, 28, 3, 1100), (128, 28, 3, 460))] + \
        [(attention.test_balanced_schedule_merges_of_many_parts, a) for a in ((16, 14, 2, 64, 6000), (16, 32, 8, 96, 7000))]


@pytest.mark.parametrize("test,args", CASES, ids=["%s-%s" % (t.__name__, "-".join(map(str, a))) for t, a in CASES])
def test_waits_that_end_early(test, args):
    with short_waits():
        test(*args)


def replays(run, inputs, outs, wipe, n=40):
    """`run` on other inputs, called with the usual waits and replayed with short ones: outputs `outs`, wiped in between."""
    sets = [[torch.randn(x.shape, device="cuda", generator=torch.Generator("cuda").manual_seed(i)).mul_(3).to(x.dtype) for x in inputs] for i in range(4)]

    def load(i):
        for x, v in zip(inputs, sets[i]):
            x.copy_(v)
        for o in outs:
            o.fill_(wipe)

    want = []
    for i in range(len(sets)):
        load(i)
        run()
        want.append([o.clone() for o in outs])
    assert not all(torch.equal(a, b) for a, b in zip(want[0], want[1]))
    side = torch.cuda.Stream()
    with short_waits(), torch.cuda.stream(side):
        g = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(g, stream=side):
            run()
    for rep in range(n):
        load(rep % len(sets))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(outs, want[rep % len(sets)])), rep


@pytest.mark.parametrize("V,dtype,params", [(128256, torch.bfloat16, [(60, 6, 10)]), (50001, torch.float32, [(40, 4, 8), (33, 3, 16)]),
                                            (2048, torch.float32, [(60, 6, 10), (40, 5, 4)]), (30000, torch.bfloat16, [(96, 5, 12)] * 3)])
def test_levels_replayed(V, dtype, params):
    # two passes, a workgroup to a row, and log-sum-exps of their own
    B, d, R, TT_cap = len(params), max(p[1] for p in params), max(p[2] for p in params), max(p[0] for p in params)
    i32 = dict(dtype=torch.int32, device="cuda")
    limits, roots = torch.tensor(params, **i32), torch.zeros(B, **i32)
    logits = [torch.empty((B * (1 if l == 0 else R), V), dtype=dtype, device="cuda") for l in range(d)]
    state = torch.zeros(dt.dt_level_state_bytes(B), dtype=torch.uint8, device="cuda")
    ws = torch.empty(dt.dt_workspace_bytes(B, B * R, V, TT_cap, 1, 1), dtype=torch.uint8, device="cuda")
    n_exp = [torch.zeros(B, **i32) for _ in range(d)]
    exp = [[torch.zeros((B, 32), **i32) for _ in range(4)] + [torch.zeros((B, 32, 4), dtype=torch.int64, device="cuda")] for _ in range(d)]
    tree = [torch.zeros(B, **i32)] + [torch.zeros((B, TT_cap), **i32) for _ in range(3)] + [torch.zeros((B, TT_cap), device="cuda") for _ in range(2)] + \
           [torch.zeros((B, TT_cap), **i32), torch.zeros((B, TT_cap, 2), dtype=torch.int64, device="cuda")]

    def run():
        for l in range(d):
            dt.dt_expand_level(l + 1, limits, logits[l], R, None, TT_cap, state, n_exp[l], *exp[l], ws)
        dt.dt_finish_tree(limits, V, roots, TT_cap, state, *tree)

    replays(run, logits, n_exp + sum(exp, []) + tree, -3)


@pytest.mark.parametrize("V,n,dtype", [(128256, 28, torch.bfloat16), (50001, 61, torch.float32)])
def test_rows_replayed(V, n, dtype):
    x, k = torch.empty((n, V), dtype=dtype, device="cuda"), 13
    outs = [torch.empty((n, k), device="cuda"), torch.empty((n, k), dtype=torch.int32, device="cuda"), torch.empty(n, device="cuda")]
    ws = torch.empty(dt.dt_workspace_bytes(1, n, V, 8, 1, 64), dtype=torch.uint8, device="cuda")
    replays(lambda: dt.dt_topk_rows(x, k, *outs, ws), [x], outs, -3)


# three, eight and four splits that meet in an XCD, and three whose last units lie apart
@pytest.mark.parametrize("D,Hq,Hkv,B,L", [(128, 32, 8, 1, 1024), (128, 4, 4, 1, 2000), (64, 14, 2, 2, 1500), (64, 28, 28, 3, 1100)])
def test_key_splits_replayed(D, Hq, Hkv, B, L):
    st = Step([(32, 5, 6)] * B, [L - 9 * b for b in range(B)], Hq, Hkv, D, 1031)
    st.draft_logits.normal_(generator=torch.Generator("cuda").manual_seed(1)).mul_(3)
    st.build_tree()
    assert st.n_nodes.tolist() == [32] * B
    replays(st.tree_attention, [st.q, st.k_tree, st.v_tree] + st.k_prefix + st.v_prefix, [st.out], 7.0)
