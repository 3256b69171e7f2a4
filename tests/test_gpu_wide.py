"""GPU parity of the many-row LM-head kernel's row shapes (32*RB rows per workgroup, RB = 4 ..
9, chosen from the rows and the vocabulary): the smallest problem that takes it, one and
several row tiles, last tiles of one row and full ones, and K tails in either head."""
import numpy as np
import pytest

from paper_2608_12913_amd import synth
from tests.test_gpu_parity import _check_greedy, _check_sample, _gpu, _greedy_tokens, _sampled_tree_setup  # noqa: F401

pytestmark = pytest.mark.gpu
V3 = synth.VOCAB_LLAMA3


# rows -> row blocks per wave at this vocabulary: 129 -> 5 (the first problem above 128
# rows), 192 -> 6 (exactly one tile), 211 -> 7, 250 -> 8, 287 -> 9, 289 -> 5 (two row tiles),
# 513 -> 9 (two row tiles)
@pytest.mark.parametrize("rows", [129, 192, 211, 250, 287, 289, 513])
@pytest.mark.parametrize("theta", [0.1, 0.0])
def test_row_shapes(rows, theta):
    case = synth.make_case("b8_tree64", 50, B=1, N=rows, tree="chain", V=V3, dp=64, dq=64, theta=theta)
    _check_greedy(case, _greedy_tokens(case), f"{rows} rows, theta {theta}")


# a small vocabulary takes the smallest row shape (128 rows) and several row tiles, the last
# of one row; one K chunk shorter than 128 bytes, K tails, and whole chunks
@pytest.mark.parametrize("rows,V,dp,dq", [(129, 257, 8, 40), (257, 1000, 72, 64), (385, 600, 192, 136),
                                          (129, 2500, 448, 448)])
@pytest.mark.parametrize("theta", [0.1, 0.0])
def test_small_row_shape(rows, V, dp, dq, theta):
    case = synth.make_case("b8_tree64", 51, B=1, N=rows, tree="chain", V=V, dp=dp, dq=dq, theta=theta)
    _check_greedy(case, _greedy_tokens(case), f"{rows} rows, V={V}, theta {theta}")


@pytest.mark.parametrize("theta", [0.1, 0.0])
def test_sampled_trees(theta):
    # 5 trees of 31 nodes = 155 rows, sampled: the dense y rows at theta = 0
    case = synth.make_case("s8_chain16x8", 52, B=5, N=31, tree="tree", depth=6, max_children=4,
                           V=2500, dp=256, dq=136, theta=theta)
    probs, tokens = _sampled_tree_setup(case)
    g, _ = _check_sample(case, probs, tokens, f"sampled trees, 155 rows, theta {theta}")
    assert np.all(g["status"] == 0)
