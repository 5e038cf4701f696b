"""What a pass needs of device memory where a TopPlan takes the narrow layers of a circuit with long rows: klay_workspace_bytes, the limit of
the entry point with the fixed array, and caller workspaces of every size that suffices for one of the ways to run a pass."""
import numpy as np
import pytest

from klay_synth import as_inputs, leaf_probs
from klay_synth.circuits import layered_random
from tests.gpu_util import assert_grad_close, assert_log_close, oracle_eval

LOG = 1


def circuit(which):
    """layers that the circuit plan itself leaves to the launches (alias_top_layer = num_layers), taken whole and in part"""
    if which == "whole":
        return layered_random(3, num_vars=40, depth=10, num_gates=4000, fanin=("zipf", 1.4, 700), groups=1, num_roots=19)
    return layered_random(4, num_vars=48, depth=12, num_gates=40000, fanin=("zipf", 1.6, 900), groups=2, num_roots=64)


@pytest.mark.parametrize("which", ["whole", "part"])
@pytest.mark.parametrize("batch", [1, 16, 17, 64, 200, 1000])
def test_a_pass_that_keeps_nothing_needs_what_the_launches_need(which, batch):
    from paper_2410_11415_amd import Circuit
    c = circuit(which)
    k = Circuit(*c.arrays(), device=-1, no_fusion=True)
    launches = Circuit(*c.arrays(), device=-1, no_fusion=True, no_tail=True)
    assert k.info()["alias_top_layer"] == k.info()["num_layers"]
    assert k.workspace_bytes(batch, False) == launches.workspace_bytes(batch, False)
    assert k.workspace_bytes(batch, True) >= launches.workspace_bytes(batch, True)
    k.close()
    launches.close()


@pytest.mark.gpu
@pytest.mark.parametrize("which", ["whole", "part"])
def test_the_fixed_array_takes_what_klay_workspace_bytes_says(which):
    import torch
    import paper_2410_11415_amd as klay
    c = circuit(which)
    k = klay.Circuit(*c.arrays(), device=0)
    limit = klay.binding.KLAY_STATIC_WORKSPACE_BYTES
    most = max(b for b in range(1, 20000) if k.workspace_bytes(b, False) <= limit)
    over = next(b for b in range(most + 1, 20000) if k.workspace_bytes(b, False) > limit)
    for batch in (most, 16, 17, 70):
        w = torch.from_numpy(as_inputs(leaf_probs(1, batch, c.num_vars, ("beta", 0.5, 0.5)), True)).cuda()
        assert torch.equal(k.forward_static(w, LOG), k.forward(w, LOG))
    w = torch.zeros((over, c.num_vars), device="cuda")
    with pytest.raises(klay.KlayError) as err:
        k.forward_static(w, LOG)
    assert err.value.status == 3 and str(k.workspace_bytes(over, False)) in str(err.value)
    k.close()


@pytest.mark.gpu
@pytest.mark.parametrize("which", ["whole", "part"])
@pytest.mark.parametrize("batch", [16, 17, 130])
def test_caller_workspaces(which, batch):
    import torch
    import paper_2410_11415_amd as klay
    c = circuit(which)
    k = klay.Circuit(*c.arrays(), device=0, no_fusion=True)
    launches = klay.Circuit(*c.arrays(), device=-1, no_fusion=True, no_tail=True)
    k.set_profiling(True)
    p = leaf_probs(batch, batch, c.num_vars, ("uniform", 0.2, 0.8))
    w = torch.from_numpy(as_inputs(p, True)).cuda()
    dout = torch.rand((batch, k.num_roots), device="cuda") + 0.5
    ref, rgrad = oracle_eval(c, w.cpu().numpy(), LOG, dout.cpu().numpy(), or_levels=k.num_layers // 2)
    out = k.forward(w, LOG)
    grad = k.backward(dout)
    assert k.get_profile()["tail_bwd"]["launches"] == 1
    sizes = (k.workspace_bytes(batch, True), launches.workspace_bytes(batch, True), k.workspace_bytes(batch, False))
    for size, kernels in zip(sizes, (1, 0, 1)):
        # guards at the end: nothing is written past the size that was given
        buf = torch.full((size // 4 + 4096,), 7.0, device="cuda")
        k.set_workspace(buf[:size // 4])
        got = k.forward(w, LOG)
        assert_log_close(got.cpu().numpy(), ref, "%s B=%d in %d bytes" % (which, batch, size))
        assert k.get_profile()["tail_fwd"]["launches"] == kernels
        if size == sizes[2]:
            assert torch.equal(got, out)
            with pytest.raises(klay.KlayError) as err:
                k.backward(dout)
            assert err.value.status == 3
        else:
            g = k.backward(dout)
            assert_grad_close(g.cpu().numpy(), rgrad, "%s B=%d in %d bytes" % (which, batch, size))
            if kernels:
                assert torch.equal(got, out) and torch.equal(g, grad)
        assert (buf[size // 4:] == 7.0).all()
        k.set_workspace(None)
    small = torch.empty(sizes[2] // 4 - 64, device="cuda")
    k.set_workspace(small)
    with pytest.raises(klay.KlayError) as err:
        k.forward(w, LOG)
    assert err.value.status == 3
    k.close()
    launches.close()
