"""The generic row kernels (GPU) over their shapes: every number of lanes per row and columns per lane (batches that are no
multiple of four, launches of few and of many rows), rows of 1 to hundreds of children, segments and combine rows of split
rows; fp32 in the three semirings with gradients, and the double-precision kernels; against the oracle."""
import numpy as np
import pytest

from klay_synth import as_inputs
from klay_synth.circuits import layered_random
from tests.gpu_util import assert_grad_close, assert_log_close, assert_real_close, gpu_eval, oracle_eval

pytestmark = pytest.mark.gpu
REAL, LOG, MAXLOG = 0, 1, 2


def check(c, batch, **options):
    import torch
    import paper_2410_11415_amd as klay
    rng = np.random.default_rng(batch)
    k = klay.Circuit(*c.arrays(), device=0, no_tail=True, **options)
    p = rng.uniform(0.02, 0.98, size=(batch, c.num_vars))
    p[0, 0], p[-1, 1] = 0.0, 1.0
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
        w64 = torch.from_numpy(np.asarray(w, np.float64)).cuda()
        out64 = k.forward_f64(w64, semiring).cpu().numpy()
        fin = np.isfinite(ref)
        np.testing.assert_array_equal(out64[~fin], ref[~fin])
        # the order of the sums differs: a few roundoffs of 2^-53 per level on values of up to a few hundred
        np.testing.assert_allclose(out64[fin], ref[fin], rtol=1e-12, atol=1e-12)
        if d is not None:
            g64 = k.backward_f64(torch.from_numpy(dout.astype(np.float64)).cuda()).cpu().numpy()
            gf = np.isfinite(rgrad)
            np.testing.assert_allclose(g64[gf], np.asarray(rgrad)[gf], rtol=1e-9, atol=1e-9 * max(1.0, float(np.abs(np.asarray(rgrad)[gf]).max())))
    k.close()


@pytest.mark.parametrize("batch", [1, 2, 3, 4, 5, 7, 9, 16, 21, 31, 33, 50, 64, 67, 129])
def test_few_rows_with_split_rows(batch):
    check(layered_random(3, 60, 8, 3000, fanin=("zipf", 1.6, 400), groups=1), batch, heavy_fan=20, min_segment=7)


@pytest.mark.parametrize("batch", [1, 3, 5, 32])
def test_split_rows_of_few_segments(batch):
    """(at most 8 partial rows: a lane group per split row instead of four waves)"""
    check(layered_random(5, 60, 8, 3000, fanin=("geom", 2.2), groups=1), batch, heavy_fan=6, min_segment=5)


@pytest.mark.parametrize("batch", [6, 10, 30, 61])
def test_many_rows(batch):
    check(layered_random(4, 128, 6, 150_000, fanin=("geom", 2.0), groups=2), batch)
