"""GPU tests of the plan for the narrow top of circuits with long rows (TopPlan): circuits it takes whole and in part, whose
layers of the circuit plan itself end in a narrow top too (B0 < L) or not, batches on both sides of every rule, the three
semirings, free literals, both entry points of a forward pass, and a backward pass called twice."""
import numpy as np
import pytest

from klay_synth import as_inputs, leaf_probs
from klay_synth.circuits import layered_random
from tests.gpu_util import assert_grad_close, gpu_eval, oracle_eval
from tests.test_gpu_parity import build, check_both, check_max, klay  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu
REAL, LOG = 0, 1


def _circuit(which):
    return {"whole": lambda: layered_random(3, num_vars=40, depth=10, num_gates=3000, fanin=("zipf", 1.5, 600), groups=1, num_roots=9),
            "part": lambda: layered_random(4, num_vars=48, depth=12, num_gates=30000, fanin=("zipf", 1.6, 900), groups=2, num_roots=64),
            "leaves": lambda: layered_random(5, num_vars=7000, depth=20, num_gates=9000, fanin=("zipf", 1.5, 400), groups=1, num_roots=5)}[which]()


@pytest.mark.parametrize("which,cap", [("whole", 0), ("whole", 400), ("part", 0), ("part", 900), ("leaves", 0)])
@pytest.mark.parametrize("B", [1, 17, 40, 130, 300])
def test_top_plan_matches_the_oracle(klay, which, cap, B):  # noqa: F811
    c = _circuit(which)
    V = c.num_vars
    p = leaf_probs(B, B, V, ("beta", 0.5, 0.5))
    k = build(klay, c, tail_rows_cap=cap)
    k.set_profiling(True)
    gpu_eval(k, as_inputs(p, True), LOG, np.ones((B, c.roots.shape[0]), np.float32))
    prof = k.get_profile()
    assert prof["tail_fwd"]["launches"] == 1 and prof["tail_bwd"]["launches"] == 1, "a persistent kernel ran"
    assert k.persistent_layers(B, LOG)[1] == 2, "of the top plan"
    k.close()
    check_both(klay, c, p, semirings=(LOG,), what="top %s cap %d B=%d" % (which, cap, B), tail_rows_cap=cap)
    check_max(klay, c, p, what="top %s max B=%d" % (which, B))


@pytest.mark.parametrize("which", ["whole", "part"])
def test_top_plan_in_the_real_semiring_with_zeros_and_ones(klay, which):  # noqa: F811
    """forward in the plan, reverse sweep by the launches from the values that are put back into rows"""
    c = layered_random(6, num_vars=30, depth=8, num_gates=1200 if which == "whole" else 26000, fanin=("zipf", 1.8 if which == "whole" else 2.2, 120),
                       groups=1, num_roots=7)
    p = leaf_probs(3, 33, c.num_vars, ("uniform", 0.2, 0.8))
    p[:, 3] = 0.0
    p[1::3, 5] = 1.0
    k = build(klay, c)
    assert k.persistent_layers(33, REAL)[1] == 2
    k.close()
    check_both(klay, c, p, semirings=(REAL,), what="top real %s" % which)


@pytest.mark.parametrize("which", ["whole", "part"])
def test_top_plan_twice_backward_static_and_replayed(klay, which):  # noqa: F811
    """the second backward pass after one forward pass, the entry point that allocates nothing, and replays of a captured
    step give what the first eager one gave"""
    import torch
    c, B = _circuit(which), 70
    k = build(klay, c)
    w = torch.from_numpy(as_inputs(leaf_probs(1, B, c.num_vars, ("beta", 0.5, 0.5)), True)).cuda()
    dout = torch.rand((B, k.num_roots), device="cuda") - 0.3
    out = k.forward(w, LOG)
    g = [k.backward(dout) for _ in range(2)]
    torch.cuda.synchronize()
    assert torch.equal(g[0], g[1])
    if k.workspace_bytes(B, False) < klay.binding.KLAY_STATIC_WORKSPACE_BYTES:
        assert torch.equal(k.forward_static(w, LOG), out)
    k.forward(w, LOG)
    eager = k.backward(dout).clone()
    graph_out, graph_g = torch.empty_like(out), torch.empty_like(eager)
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            k.forward(w, LOG, out=graph_out, stream=side)
            k.backward(dout, dleaf=graph_g, stream=side)
    torch.cuda.synchronize()
    for _ in range(3):
        graph_out.zero_()
        graph_g.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(graph_out, out) and torch.equal(graph_g, eager)
        torch.rand(1000, device="cuda").sum().item()
    _, rd = oracle_eval(c, w.cpu().numpy(), LOG, dout.cpu().numpy(), or_levels=k.num_layers // 2)
    assert_grad_close(eager.cpu().numpy(), rd, "top %s" % which)
    k.close()
