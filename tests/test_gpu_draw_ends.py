"""Untruncated draws at the end of the distribution, where no token's running sum exceeds the
target (a uniform of 1): the token is the last one of positive weight, in the spread walk (up to
64 sequences), in the walk of one workgroup per sequence and in the proposals.  The hidden
states are zero, so the target is the bias' 1 / (v + 1): the last weight is above 1e-5 of the
total, the sums' rounding below 1e-12.  The draft's proposals have no mass there, so that token
is the last of the vocabulary after a rejection too."""
import numpy as np
import pytest

from paper_2608_12913_amd import synth
from tests.test_gpu_parity import _gpu  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,V", [(1, 300), (3, 5001), (33, 1025), (65, 1025)])
def test_last_positive_token(B, V):
    from paper_2608_12913_amd.runner import DeviceProblem
    N = 4
    case = synth.make_case("s8_chain16x8", 80, B=B, N=N, V=V, dp=64, dq=32, theta=0.0, T=1.0)
    case.hp, case.hq = np.zeros_like(case.hp), np.zeros_like(case.hq)
    q = np.zeros((case.R, V), np.float32)
    q[:, :100] = 0.01
    case.u_acc, case.u_res = np.full(case.R, 0.5, np.float32), np.ones(case.R, np.float32)
    case.u_acc[1::2 * N] = 1e-30  # the first draft token of every other chain is accepted
    dev = DeviceProblem.from_case(case, np.full((B, N), 90, np.int32), draft_probs=q)
    first = None
    for _ in range(5):
        g = dev.run("sample")
        assert np.all(g["status"] == 0)
        assert np.all(g["accept_len"][::2] >= 1)
        assert np.array_equal(g["next_token"], np.full(B, V - 1)), g["next_token"]
        first = first or g
        assert np.array_equal(g["accept_len"], first["accept_len"])
    assert np.array_equal(dev.propose(case.u_res)["tokens"], np.full(case.R, V - 1))
