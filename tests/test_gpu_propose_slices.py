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
