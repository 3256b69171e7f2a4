"""GPU parity of untruncated proposals at the edges of the slices the vocabulary is cut into
(2,048 tokens): one slice, exactly one, one token more, and more slices than a workgroup has
threads; draws at both ends of the distribution; and the outputs wanted alone."""
import numpy as np
import pytest

from paper_2608_12913_amd import synth
from tests.test_gpu_propose import _check, _gpu  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,rows,dtype", [(1, 3, "bf16"), (2047, 5, "f32"), (2048, 5, "bf16"), (2049, 7, "bf16"),
                                          (6150, 300, "bf16"), (530001, 2, "bf16")])
def test_slices(V, rows, dtype):
    name = "s8_chain16x8" if dtype == "bf16" else "tiny_chain8"
    case = synth.make_case(name, 70, B=1, N=rows, V=V, dp=16, dq=8, theta=0.0, T=0.9, mode="greedy")
    u = np.random.default_rng(70).random(case.R).astype(np.float32)
    if rows >= 64:  # (draws at either end lie within the draw's gate of a breakpoint: 2 of these rows)
        u[0], u[-1] = 0.0, np.nextafter(np.float32(1), np.float32(0))
    g, _ = _check(case, u, f"slices of {V} tokens")
    assert np.all((g["tokens"] >= 0) & (g["tokens"] < V))


def test_outputs_alone():
    from paper_2608_12913_amd import dcd
    from paper_2608_12913_amd.runner import DeviceProblem
    case = synth.make_case("s8_chain16x8", 71, B=2, N=9, V=4100, dp=64, dq=32, theta=0.0, mode="greedy")
    u = np.random.default_rng(71).random(case.R).astype(np.float32)
    dev = DeviceProblem.from_case(case, np.zeros((case.B, case.N), np.int32), row_outputs=False)
    both = dev.propose(u)
    assert np.array_equal(dev.propose(u, want_probs=False)["tokens"], both["tokens"])
    probs = torch.empty(case.R, case.V, dtype=torch.float32, device=dev.device)
    dcd.propose(dev.problem, dev.inputs, None, None, probs, None, dev.workspace, dev.ws_bytes,
                torch.cuda.current_stream(dev.device))
    assert np.array_equal(probs.cpu().numpy(), both["probs"])


def test_more_tokens_than_slices_of_the_grid():
    """2^27 + 5 tokens: more than 65,536 slices (the grid's limit in y) of 2,048, so a slice
    holds two of those.  The states and weights are zero, so the logits are the bias: three
    tokens share all but 134e6 exp(-30) = 2e-5 of the total alike."""
    from paper_2608_12913_amd import dcd
    V, d, dev = (1 << 27) + 5, 8, "cuda:0"
    picks = [5, (1 << 26) + 2047, V - 1]
    bf16 = dict(dtype=torch.bfloat16, device=dev)
    bias = torch.full((V,), -30.0, device=dev)
    bias[picks] = 0.0
    u = torch.tensor([0.1, 0.5, 0.9], device=dev)
    h, w = torch.zeros(3, d, **bf16), torch.zeros(V, d, **bf16)
    prob = dcd.make_problem(1, 3, V, d, d, "bf16", 0.0, 0.5, 1.0)
    n = dcd.workspace_bytes(prob)
    ws = torch.zeros(n, dtype=torch.uint8, device=dev)
    inputs = dcd.make_inputs(h, h, w, w, bias, bias, None, None)
    tokens, argmax = (torch.full((3,), -7, dtype=torch.int32, device=dev) for _ in range(2))
    stream = torch.cuda.current_stream()
    dcd.propose(prob, inputs, u, tokens, None, argmax, ws, n, stream)
    assert tokens.tolist() == picks and argmax.tolist() == [5, 5, 5]
    probs = torch.empty(3, V, device=dev)
    tokens.fill_(-7)
    dcd.propose(prob, inputs, u, tokens, probs, None, ws, n, stream)
    assert tokens.tolist() == picks
    p = probs[:, picks].cpu().numpy()
    np.testing.assert_allclose(p, 1 / 3, rtol=1e-4)
    assert float((probs > 1e-3).sum()) == 9 and float(probs.min()) > 0
