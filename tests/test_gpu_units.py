"""Narrow layers in the persistent kernels (GPU) against the oracle: rows of 1 to 384 children at the edges of lanes, layers at the
edges of units and at the limit above which a layer is none, roots read by one wave and by all, one, two and four columns, every
semiring, both directions.  (tests/host_unit_check.cpp executes the units on the host.)"""
import numpy as np
import pytest

from klay_synth import as_inputs
from tests.gpu_util import assert_grad_close, assert_log_close, assert_real_close, gpu_eval, oracle_eval
from tests.test_gpu_cols import stack

pytestmark = pytest.mark.gpu
REAL, LOG, MAXLOG = 0, 1, 2
EDGE_FANS = (1, 2, 3, 4, 6, 7, 12, 13, 24, 25, 47, 48, 49, 60)


def check(c, batch, seed, zeros, top=False):
    import paper_2410_11415_amd as klay
    rng = np.random.default_rng(seed)
    k = klay.Circuit(*c.arrays(), device=0, no_merge=True)
    assert k.persistent_layers(batch)[0] == 1
    p = rng.uniform(0.5, 0.9, size=(batch, c.num_vars))
    u = rng.random(p.shape)
    p[u < zeros], p[u > 1 - zeros / 2] = 0.0, 1.0
    dout = rng.normal(size=(batch, c.roots.shape[0])).astype(np.float32)
    for semiring in (LOG, MAXLOG) if top else (LOG, REAL, MAXLOG):
        with np.errstate(divide="ignore"):
            w = as_inputs(p, semiring != REAL)
        d = None if semiring == MAXLOG else dout
        out, grad = gpu_eval(k, w, semiring, d)
        ref, rgrad = oracle_eval(c, w, semiring, d, or_levels=k.num_layers // 2)
        (assert_real_close if semiring == REAL else assert_log_close)(out, ref, "values")
        if d is not None:
            assert_grad_close(grad, rgrad, "gradients", real=semiring == REAL)
    k.close()


@pytest.mark.parametrize("widths,batch", [
    ((64, 64, 64, 1), 1), ((65, 63, 66, 33, 64, 65), 3), ((960, 961, 959, 256), 2), ((1921, 1920, 500, 257), 5), ((3840, 3841, 700, 300), 2),
    ((400, 300, 200, 100, 50, 25), 300), ((400, 300, 200, 100, 50, 25), 601), ((90, 31) * 35, 2)])
@pytest.mark.parametrize("fan", ["short", "edges"])
def test_layers_at_the_edges_of_units(widths, batch, fan):
    rng = np.random.default_rng(widths[0])
    if len(widths) > 64:
        pick = lambda r: int(r.random() < 0.03)              # (mostly one child: values stay small over 70 layers)
    else:
        pick = (lambda r: 1 + int(r.integers(3))) if fan == "short" else (lambda r: EDGE_FANS[int(r.integers(len(EDGE_FANS)))] if r.random() < 0.2 else 1)
    check(stack(rng, 30, widths, pick, 0.3), batch, 1, 0.004)


@pytest.mark.parametrize("batch", [1, 70, 260])
def test_long_rows_of_a_top_plan(batch):
    """rows of more than 64 children: 65, 96, 97, 192, 193, 384 lanes' worth, and one of 385 (a layer that is none)"""
    rng = np.random.default_rng(3)
    fans = [65, 95, 96, 97, 191, 192, 193, 383, 384, 385]
    check(stack(rng, 200, (700, 500, 600, 40, 20, 8), lambda r: fans[int(r.integers(len(fans)))] if r.random() < 0.02 else 1, 0.2), batch, 2, 0.0, top=True)
