"""GPU parity of the tree kernel at the edges of its paths: level sizes around the registers of one wave and around the
change to all waves, pools around one and two candidates per thread, and equal scores that straddle every cut."""
import numpy as np
import pytest

import dt_synth
from oracle import ref
from tests.test_gpu_parity import assert_tree_equal

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(40, 3, 8), (128, 8, 8), (60, 4, 9), (127, 5, 11), (100, 4, 12), (64, 8, 12), (33, 2, 16), (128, 4, 16), (70, 8, 16),
          (65, 3, 17), (128, 4, 17), (20, 4, 22), (128, 3, 22), (66, 2, 23), (50, 8, 32), (128, 2, 32), (128, 8, 31)]


def _build(rows, bf16, TT, d, k):
    from paper_2601_12212_amd.step import Step
    st = Step([(TT, d, k)], [1], 4, 4, 64, rows.shape[1], dtype=torch.bfloat16 if bf16 else torch.float32, TT_cap=128)
    st.set_draft(0, dt_synth.f32_to_bf16_bits(rows) if bf16 else rows)
    st.set_root_token(0, 3)
    st.build_tree()
    torch.cuda.synchronize()
    return st.tree(0)


@pytest.mark.parametrize("TT,d,k", SHAPES)
def test_paths_of_the_expansion_and_of_the_rerank(TT, d, k):
    tag = "TT=%d d=%d k=%d" % (TT, d, k)
    checked = 0
    for seed in range(40):
        rows = np.random.default_rng(seed).standard_normal((1 + (d - 1) * k, 1500)).astype(np.float32) * (1.0 + seed % 4)
        want = ref.build_tree(rows, TT, d, k, 3)
        if want["min_margin"] >= 2e-5:
            assert_tree_equal(_build(rows, False, TT, d, k), want, tag)
            checked += 1
        if checked == 2:
            break
    assert checked
    # identical rows with one winner: all other candidates of a level tie, and the lowest pool indices have to win
    rows = np.zeros((1 + (d - 1) * k, 900), np.float32)
    rows[:, 300] = 1.0
    assert_tree_equal(_build(rows, True, TT, d, k), ref.build_tree(dt_synth.f32_to_bf16_bits(rows), TT, d, k, 3), "ties " + tag)


# three and four candidates per lane, one and two per thread, pools whose threads hold up to 5, 9 and 15
@pytest.mark.parametrize("TT,d,k", [(90, 5, 13), (90, 5, 14), (90, 6, 22), (90, 6, 23), (90, 5, 32), (90, 6, 32)])
def test_paths_sized_by_k_and_by_the_pool(TT, d, k):
    test_paths_of_the_expansion_and_of_the_rerank(TT, d, k)
