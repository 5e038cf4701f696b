"""The streaming kernel (GPU) against the oracle with tasks of every length around its chunks of four: layers of 1 to 40 rows (one or two
tasks, the last one short), of rows of 1 to 30 entries, two and four columns per lane with lanes past the batch, split rows, every
semiring, both directions."""
import numpy as np
import pytest

from klay_synth import as_inputs
from tests.gpu_util import assert_grad_close, assert_log_close, assert_real_close, gpu_eval, oracle_eval
from tests.test_gpu_cols import stack

pytestmark = pytest.mark.gpu
REAL, LOG, MAXLOG = 0, 1, 2


@pytest.mark.parametrize("batch", [90, 128, 129, 255, 260])
@pytest.mark.parametrize("widths,fan,options", [
    ((1, 2, 3, 4), 4, {}), ((5, 7, 9, 8), 3, {}), ((17, 33, 18, 15), 1, {}), ((40, 21, 39, 6), 6, {}), ((13, 26, 11, 3), 30, dict(heavy_fan=5, min_segment=3)),
    ((600, 500, 300, 40), 2, dict(heavy_fan=3, min_segment=2))])
def test_tasks_around_the_chunks(batch, widths, fan, options):
    import paper_2410_11415_amd as klay
    rng = np.random.default_rng(sum(widths))
    c = stack(rng, 20, widths, lambda r: int(r.integers(fan + 1)), 0.2)
    k = klay.Circuit(*c.arrays(), device=0, no_tail=True, no_merge=True, **options)
    p = rng.uniform(0.4, 0.9, size=(batch, 20))
    # (no probability of 1: its negated literal has an infinite derivative in the log domain, which says nothing about the kernel)
    p[0, 0], p[1, 1], p[-1, 2] = 0.0, 0.0, 0.0
    dout = rng.normal(size=(batch, c.roots.shape[0])).astype(np.float32)
    for semiring in (LOG, REAL, MAXLOG):
        with np.errstate(divide="ignore"):
            w = as_inputs(p, semiring != REAL)
        d = None if semiring == MAXLOG else dout
        out, grad = gpu_eval(k, w, semiring, d)
        ref, rgrad = oracle_eval(c, w, semiring, d, or_levels=k.num_layers // 2)
        (assert_real_close if semiring == REAL else assert_log_close)(out, ref, "values")
        if d is not None:
            assert_grad_close(grad, rgrad, "gradients", real=semiring == REAL)
    k.close()
