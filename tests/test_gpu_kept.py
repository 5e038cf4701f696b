"""Forward passes (GPU) that leave fused AND rows out, against the oracle: the kept rows by the generic kernel (up to 84 columns), by the
streaming kernel with two and four columns per lane, with split rows among them, in the three semirings."""
import numpy as np
import pytest

from klay_synth import as_inputs, make_config
from tests.gpu_util import assert_log_close, assert_real_close, gpu_eval, oracle_eval

pytestmark = pytest.mark.gpu
REAL, LOG, MAXLOG = 0, 1, 2


@pytest.mark.parametrize("batch,options", [(65, {}), (70, dict(heavy_fan=3, min_segment=2)), (97, {}), (128, dict(heavy_fan=3, min_segment=2)),
                                           (131, dict(heavy_fan=2, min_segment=1)), (260, {})])
def test_kept_rows(batch, options):
    import paper_2410_11415_amd as klay
    c, p, _ = make_config("layered_100k", seed=6, scale=0.3, batch=batch)
    k = klay.Circuit(*c.arrays(), device=0, tail_rows_cap=900, **options)
    info = k.info()
    assert 0 < info["num_fused_rows"] and info["alias_top_layer"] > 2
    for semiring in (LOG, MAXLOG, REAL):
        w = as_inputs(p, semiring != REAL)
        out, _ = gpu_eval(k, w, semiring)
        ref, _ = oracle_eval(c, w, semiring)
        (assert_real_close if semiring == REAL else assert_log_close)(out, ref, "B=%d" % batch)
    k.close()
