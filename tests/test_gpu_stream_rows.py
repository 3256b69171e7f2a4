"""GPU parity of the streaming LM-head kernel's row shapes (16, 32, 48, 64 and 128 rows per
workgroup, chosen from the rows, the vocabulary and the type): one row, full and nearly empty
last row blocks, several row blocks, ragged vocabularies and K tails; and the many-row
kernel's smallest shape on vocabularies just large enough for it."""
import pytest

from paper_2608_12913_amd import synth
from tests.routes import route
from tests.test_gpu_parity import _check_greedy, _check_sample, _gpu, _greedy_tokens, _sampled_tree_setup  # noqa: F401

pytestmark = pytest.mark.gpu
V3 = synth.VOCAB_LLAMA3


# (type, rows, V, dp, dq), rows per workgroup masked and untruncated ("wide": the many-row kernel)
CASES = [
    ("bf16", 1, 257, 72, 8, 16, 16),
    ("bf16", 17, 1000, 64, 40, 16, 16),          # the last block of one row
    ("bf16", 130, 8000, 136, 64, 32, 32),        # 16 rows would make two rounds
    ("bf16", 20, 32999, 64, 72, 32, 32),         # one block
    ("bf16", 20, 65793, 520, 512, 32, 32),       # one block, more tiles than CUs
    ("bf16", 81, 32003, 64, 72, 48, 48),         # two blocks
    ("bf16", 40, 32999, 72, 64, 48, 48),         # one block
    ("bf16", 40, 65793, 520, 512, 48, 48),       # one block, more tiles than CUs
    ("bf16", 128, 32003, 64, 64, 64, 64),        # two full blocks
    ("bf16", 6, V3, 64, 64, 64, 16),             # one block
    ("bf16", 33, V3, 64, 64, 64, 48),            # one block
    ("bf16", 6, 65793, 520, 512, 32, 16),        # one block
    ("bf16", 65, V3, 64, 64, 128, 128),
    ("bf16", 129, 13057, 8, 40, "wide", "wide"),  # 128 rows, last tiles of one row and one token
    ("bf16", 257, 7425, 72, 64, "wide", "wide"),  # the same, three row tiles
    ("f32", 1, 257, 36, 4, 16, 16),
    ("f32", 33, 1000, 64, 100, 16, 16),          # the last block of one row
    ("f32", 64, 32003, 32, 36, 32, 16),          # two and four blocks
    ("f32", 128, 32003, 32, 64, 32, 16),
    ("f32", 20, V3, 100, 64, 32, 32),            # one block
    ("f32", 40, V3, 32, 32, 48, 16),
    ("f32", 34, 64257, 328, 456, 48, 48),        # one block
    ("f32", 419, 12545, 512, 256, 48, 48),       # nine blocks
    ("f32", 64, V3, 32, 32, 64, 16),
    ("f32", 50, V3, 100, 64, 64, 64),            # one block
    ("f32", 434, 12545, 328, 456, 64, 64),       # seven blocks
    ("f32", 304, V3, 32, 32, 64, 16),
    ("f32", 100, V3, 1004, 500, 128, 128),       # one block
    ("f32", 450, 28929, 1004, 500, 128, 128),    # four blocks
]


@pytest.mark.parametrize("dtype,rows,V,dp,dq,masked,full", CASES)
@pytest.mark.parametrize("theta", [0.1, 0.0])
def test_row_shapes(dtype, rows, V, dp, dq, masked, full, theta):
    kind, shape = route(rows, V, dp, dq, dtype, theta)
    want = masked if theta else full
    assert (kind if kind == "wide" else shape) == want
    case = synth.make_case("b8_tree64" if dtype == "bf16" else "tiny_chain8", 60, B=1, N=rows, tree="chain", V=V,
                           dp=dp, dq=dq, dtype=dtype, theta=theta)
    _check_greedy(case, _greedy_tokens(case), f"{dtype}, {rows} rows, V={V}, theta {theta}")


# sampled: the dense y rows at theta = 0
@pytest.mark.parametrize("dtype,N,V", [("bf16", 11, 1000), ("bf16", 40, 32003), ("f32", 20, 1000)])
@pytest.mark.parametrize("theta", [0.1, 0.0])
def test_sampled(dtype, N, V, theta):
    case = synth.make_case("s8_chain16x8", 61, B=2, N=N, tree="tree", depth=6, max_children=4, V=V, dp=64, dq=40,
                           dtype=dtype, theta=theta)
    probs, tokens = _sampled_tree_setup(case)
    _check_sample(case, probs, tokens, f"sampled, {dtype}, 2 x {N}, V={V}, theta {theta}")
