"""Fused AND rows (klay_options.no_fusion) of circuits whose narrow layers a TopPlan can take: they are there for the batches that
do not use the plan, and no kernel reads a row that a pass left out where it is used."""
import numpy as np
import pytest

from klay_synth import as_inputs, leaf_probs
from klay_synth.circuits import layered_random
from tests.gpu_util import assert_grad_close, assert_log_close, assert_real_close, gpu_eval, oracle_eval

REAL, LOG, MAXLOG = 0, 1, 2
SHAPES = {"whole": dict(), "part": dict(tail_rows_cap=3000), "small_part": dict(tail_rows_cap=700)}


def circuit():
    return layered_random(111, num_vars=60, depth=10, num_gates=60000, fanin=("zipf", 2.2, 300), groups=1, num_roots=40)


@pytest.mark.parametrize("shape", SHAPES)
def test_wide_layers_keep_their_fused_rows(shape):
    from paper_2410_11415_amd import Circuit
    c = circuit()
    k, launches = Circuit(*c.arrays(), device=-1, **SHAPES[shape]), Circuit(*c.arrays(), device=-1, no_tail=True)
    plain = Circuit(*c.arrays(), device=-1, no_tail=True, no_fusion=True)
    # (two of its layers are wide enough where the plan may take them, kTopFusedRows)
    assert k.info()["alias_top_layer"] == launches.info()["alias_top_layer"] == k.info()["num_layers"]
    assert launches.info()["num_fused_rows"] > 1000 and plain.info()["num_fused_rows"] == 0
    assert k.info()["num_fused_rows"] > 0.6 * launches.info()["num_fused_rows"]
    for h in (k, launches, plain):
        h.close()


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("batch", [65, 130, 300, 1100])
def test_no_kernel_reads_a_row_that_was_left_out(shape, batch):
    """in a workspace of NaN, so that a row that nothing wrote shows"""
    import torch
    import paper_2410_11415_amd as klay
    c = circuit()
    k = klay.Circuit(*c.arrays(), device=0, **SHAPES[shape])
    k.set_profiling(True)
    p = leaf_probs(batch, batch, c.num_vars, ("uniform", 0.3, 0.7))
    dout = np.ones((batch, c.roots.shape[0]), np.float32)
    for semiring in (LOG, REAL, MAXLOG):
        w = as_inputs(p, semiring != REAL)
        train = semiring != MAXLOG
        ref, rgrad = oracle_eval(c, w, semiring, dout if train else None, or_levels=k.num_layers // 2)
        # forward alone first, then followed by a reverse sweep that evaluates the rows itself, then as in a training loop
        for backward in (False, train, train):
            k.set_workspace(torch.full((k.workspace_bytes(batch, True) // 4,), float("nan"), device="cuda"))
            out, grad = gpu_eval(k, w, semiring, dout if backward else None)
            (assert_real_close if semiring == REAL else assert_log_close)(out, ref, "%s B=%d semiring %d" % (shape, batch, semiring))
            if backward:
                assert_grad_close(grad, rgrad, "%s B=%d semiring %d" % (shape, batch, semiring), real=semiring == REAL)
        if train:
            gpu_eval(k, w, semiring)               # (a pass that no reverse sweep follows, for the next semiring)
    out, _ = gpu_eval(k, as_inputs(p, True), LOG)
    prof = k.get_profile()
    if batch == 1100 and shape != "whole":
        assert prof["fwd_or_fused"]["launches"] > 0
    k.close()
