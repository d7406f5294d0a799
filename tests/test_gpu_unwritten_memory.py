"""The tree does not depend on memory that nothing wrote for it: local memory as an earlier kernel left it, the rows of a
build state that belong to no node, and logit rows that belong to no node hold infinities and NaN here."""
import numpy as np
import pytest

from oracle import ref
from tests._brute import toy_logits
from tests._cases import TREE_MARGIN, assert_tree_equal

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

V, D = 300, 5


def _rows(k, viable, seed):
    """Draft rows as a draft model would hand them over, and which of them belong to a node.  viable: tokens with a finite
    logit in every row (fewer than k: the first levels expand fewer than k nodes)."""
    rows = np.zeros((1 + (D - 1) * k, V), np.float32)
    live = np.zeros(len(rows), bool)
    strings = [()]
    for level in range(1, D + 1):
        for s, string in enumerate(strings):
            r = 0 if level == 1 else 1 + (level - 2) * k + s
            rows[r] = toy_logits(seed, string, V, sigma=3.0)
            if viable:
                rows[r, np.argsort(rows[r])[viable:]] = -np.inf
            live[r] = True
        if level < D:
            lv = ref.build_tree(rows, 128, D, k, 7, with_levels=True)["levels"][level]
            strings = [(strings[p] if p >= 0 else ()) + (int(t),) for t, p in zip(lv["tokens"], lv["parent_slot"])]
    return rows, live


def _case(k, viable, TT=100):
    for seed in range(50):
        rows, live = _rows(k, viable, seed)
        want = ref.build_tree(rows, TT, D, k, 7, with_levels=True)
        if want["min_margin"] >= TREE_MARGIN:
            return rows, live, want
    raise RuntimeError("no seed with a margin")


class Litter:
    """Leaves the local memory of every compute unit full of pairs of bf16 infinities (as a float: a NaN): 512 workgroups of
    the large-batch attention kernel, 64 KB each, whose K and V tiles are infinite."""

    def __init__(self):
        B, H, L, N = 32, 8, 512, 128
        inf = lambda *shape: torch.full(shape, float("inf"), dtype=torch.bfloat16, device="cuda")
        self.q, self.tree, self.prefix, self.out = inf(B, N, H, 128), inf(B, N, H, 128), inf(L, H, 128), inf(B, N, H, 128)
        i32 = dict(dtype=torch.int32, device="cuda")
        self.n, self.plen = torch.full((B,), N, **i32), torch.full((B,), L, **i32)
        self.ptrs = torch.full((B,), self.prefix.data_ptr(), dtype=torch.int64, device="cuda")
        self.mask = torch.full((B, N, 2), -1, dtype=torch.int64, device="cuda")
        import paper_2601_12212_amd as dt
        self.ws = torch.zeros(dt.dt_workspace_bytes(B, B, V, N, H, 128), dtype=torch.uint8, device="cuda")

    def __call__(self):
        import paper_2601_12212_amd as dt
        dt.dt_tree_attention(self.q, self.tree, self.tree, self.n, self.ptrs, self.ptrs, self.plen, 512, 8 * 128, 128, self.mask,
                             0.1, self.out, self.ws)


CASES = [(k, 0) for k in (2, 3, 4, 5, 9, 10, 12, 15, 20)] + [(5, 2), (8, 3), (10, 2), (12, 7), (16, 2), (20, 2), (32, 3)]


@pytest.mark.parametrize("k,viable", CASES)
def test_level_by_level(k, viable):
    import paper_2601_12212_amd as dt
    rows, live, want = _case(k, viable)
    TT = 100
    litter = Litter()
    i32 = dict(dtype=torch.int32, device="cuda")
    params = torch.tensor([(TT, D, k)], **i32)
    state = torch.empty(dt.dt_level_state_bytes(1), dtype=torch.uint8, device="cuda")
    state.view(torch.float32).fill_(float("inf"))
    ws = torch.empty(dt.dt_workspace_bytes(1, k, V, TT, 1, 1), dtype=torch.uint8, device="cuda")
    n_exp = torch.full((1,), -5, **i32)
    ex = [torch.full((1, 32), -5, **i32) for _ in range(4)]
    mask = torch.zeros((1, 32, 4), dtype=torch.int64, device="cuda")
    for level in range(1, D + 1):
        r0, R = (0, 1) if level == 1 else (1 + (level - 2) * k, k)
        logits = np.where(live[r0:r0 + R, None], rows[r0:r0 + R], np.float32(np.inf))
        dev = torch.from_numpy(logits).cuda()
        litter()
        dt.dt_expand_level(level, params, dev, k, None, TT, state, n_exp, *ex, mask, ws)
        n = int(n_exp[0])
        if level == D:
            assert n == 0
            continue
        lv = want["levels"][level]
        assert n == len(lv["tokens"]), level
        assert np.array_equal(ex[0][0, :n].cpu().numpy(), lv["tokens"]), level
        assert np.array_equal(ex[1][0, :n].cpu().numpy(), lv["parent_slot"]), level
        assert np.array_equal(mask[0, :n].cpu().numpy().view(np.uint64), lv["mask"]), level
    mk = lambda dtype: torch.zeros((1, TT), dtype=dtype, device="cuda")
    out = dict(n_nodes=torch.zeros(1, **i32), tokens=mk(torch.int32), parents=mk(torch.int32), depth=mk(torch.int32),
               score=mk(torch.float32), logp=mk(torch.float32), src_row=mk(torch.int32),
               anc_mask=torch.zeros((1, TT, 2), dtype=torch.int64, device="cuda"))
    litter()
    dt.dt_finish_tree(params, V, torch.tensor([7], **i32), TT, state, *out.values())
    N = int(out["n_nodes"][0])
    got = {name: t[0, :N].cpu().numpy() for name, t in out.items() if name != "n_nodes"}
    got["anc_mask"] = got["anc_mask"].view(np.uint64)
    assert_tree_equal(dict(n_nodes=N, **got), want, "k=%d viable=%d" % (k, viable))


@pytest.mark.parametrize("k,viable", CASES)
def test_one_shot(k, viable):
    from paper_2601_12212_amd.step import Step
    rows, live, want = _case(k, viable)
    st = Step([(100, D, k)], [1], 4, 4, 64, V, dtype=torch.float32)
    st.set_draft(0, np.where(live[:, None], rows, np.float32(np.inf)))
    st.set_root_token(0, 7)
    st.ws.view(torch.int32).fill_(0x7F807F80)
    Litter()()
    st.build_tree()
    assert_tree_equal(st.tree(0), want, "k=%d viable=%d" % (k, viable))
