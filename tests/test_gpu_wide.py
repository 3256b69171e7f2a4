"""GPU parity of the many-row LM-head kernel's row shapes (32*RB rows per workgroup, RB = 4 ..
9, chosen from the rows and the vocabulary): the smallest problem that takes it, one and
several row tiles, last tiles of one row and full ones, and K tails in either head."""
import numpy as np
import pytest

import oracle
from paper_2608_12913_amd import synth
from tests import parity
from tests.routes import route_of
from tests.test_gpu_parity import _check_greedy, _check_sample, _gpu, _greedy_tokens, _sampled_tree_setup  # noqa: F401

pytestmark = pytest.mark.gpu
V3 = synth.VOCAB_LLAMA3


# the route of every case is checked, so that another choice of the shape shows here
def _takes(case, rb):
    assert route_of(case) == ("wide", rb)


# 501 tiles, one K chunk: rows -> row blocks per wave: 129 -> 5 (the first problem above 128
# rows), 192 -> 6 (exactly one tile), 211 -> 7, 250 -> 8, 287 -> 9, 289 -> 5 (two row tiles),
# 513 -> 9 (two row tiles)
@pytest.mark.parametrize("rows,rb", [(129, 5), (192, 6), (211, 7), (250, 8), (287, 9), (289, 5), (513, 9)])
@pytest.mark.parametrize("theta", [0.1, 0.0])
def test_row_shapes(rows, rb, theta):
    case = synth.make_case("b8_tree64", 50, B=1, N=rows, tree="chain", V=V3, dp=64, dq=64, theta=theta)
    _takes(case, rb)
    _check_greedy(case, _greedy_tokens(case), f"{rows} rows, theta {theta}")


# every shape with one row tile (non-temporal weights, K walks that start at another chunk per
# vocabulary tile) and with several, over enough K chunks that both LDS rings turn (3 or 4 weight
# stages of a chunk, 3 or 4 hidden-state stages of half a chunk): 6 and 8 chunks that end in a
# tail of 16 bytes, or 7 and 5 whole ones.  Last row tiles of one row, last tiles of one token and of 7
MULTI = [(129, 13313, 4), (257, 21767, 5), (321, 21767, 6), (385, 21767, 7), (449, 21767, 8), (513, 21767, 9)]
ONE = [(129, 32769, 5), (161, 32769, 6), (194, 32769, 7), (225, 32769, 8), (257, 32769, 9)]


@pytest.mark.parametrize("rows,V,rb", ONE + MULTI)
@pytest.mark.parametrize("theta", [0.1, 0.0])
def test_rings_turn(rows, V, rb, theta):
    tail = (rb % 2 == 0) == (theta > 0)
    dp, dq = (328, 456) if tail else (448, 320)
    case = synth.make_case("b8_tree64", 53, B=1, N=rows, tree="chain", V=V, dp=dp, dq=dq, theta=theta)
    _takes(case, rb)
    _check_greedy(case, _greedy_tokens(case), f"{rows} rows, V={V}, {dp}/{dq}, theta {theta}")


# a small vocabulary takes the smallest row shape (128 rows) and several row tiles, the last
# of one row; one K chunk shorter than 128 bytes, K tails, and whole chunks
@pytest.mark.parametrize("rows,V,dp,dq", [(129, 13057, 8, 40), (257, 7425, 72, 64), (385, 4866, 192, 136),
                                          (129, 13313, 448, 448)])
@pytest.mark.parametrize("theta", [0.1, 0.0])
def test_small_row_shape(rows, V, dp, dq, theta):
    case = synth.make_case("b8_tree64", 51, B=1, N=rows, tree="chain", V=V, dp=dp, dq=dq, theta=theta)
    _takes(case, 4)
    _check_greedy(case, _greedy_tokens(case), f"{rows} rows, V={V}, theta {theta}")


# trees of 31 nodes, sampled: the dense y rows at theta = 0, from expert logits kept in
# registers (4 row blocks) and parked in those rows (more), in one and in several row tiles
@pytest.mark.parametrize("B,V,rb", [(5, 13313, 4), (5, 32769, 5), (13, 21767, 7)])
@pytest.mark.parametrize("theta", [0.1, 0.0])
def test_sampled_trees(B, V, rb, theta):
    case = synth.make_case("s8_chain16x8", 52, B=B, N=31, tree="tree", depth=6, max_children=4,
                           V=V, dp=256, dq=136, theta=theta)
    _takes(case, rb)
    probs, tokens = _sampled_tree_setup(case)
    g, _ = _check_sample(case, probs, tokens, f"sampled trees, {case.R} rows, theta {theta}")
    assert np.all(g["status"] == 0)


def test_wide_mask_on_either_side_of_256_rows():
    """More than 256 rows take 4 tiles per lane in the finish kernel and not 8, so above 65,536
    tokens the mask members are listed in two rounds and log Z is added in another order.  A flat
    target with some hundred members per row: both within the parity tolerance of the oracle, and
    within 1e-5 of each other where no token lies at the cutoff (fp32 sums of 1e3 terms in [0, 1] in
    another order).  So many members put a token within the boundary gate of 1e-4 in some of the
    rows: their share is checked, not their bits."""
    def run(rows):
        case = synth.make_case("b8_tree64", 54, B=257, N=1, tree="chain", V=70001, dp=64, dq=64, theta=0.002,
                               h_scale=0.5)
        case.B, case.parents = rows, case.parents[:rows]
        case.hp, case.hq = case.hp[:rows], case.hq[:rows]
        case.u_acc, case.u_res = case.u_acc[:rows], case.u_res[:rows]
        return _check_greedy(case, np.zeros((rows, 1), np.int32), f"{rows} rows, wide mask",
                             gates=dict(max_ambiguous=0.15 * rows, max_gated=0.15 * rows))[:2]
    g, o = run(257)
    h, _ = run(200)
    assert g["row_stats"][:, oracle.RS_COUNT].min() > 100
    clear = np.flatnonzero(o["row_gap"][:200] > parity.BOUNDARY_GATE)
    assert len(clear) >= 170
    np.testing.assert_allclose(h["row_stats"][clear, oracle.RS_LOGZ], g["row_stats"][clear, oracle.RS_LOGZ],
                               rtol=0, atol=1e-5)
