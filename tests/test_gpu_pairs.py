"""Batches of 65 to 128 columns (GPU): the rule that takes a pass to the generic or to the streaming kernel, on both sides of its
column limit, in circuits of short rows and of mostly split ones; three semirings with gradients, against the oracle.
test_both_kernels has layers of fewer than 2000 rows, which the generic kernel takes one or two columns per lane; the two tests after it
have the layers of four columns per lane, three rows (65 to 84 columns) or two in a wave."""
import numpy as np
import pytest

from klay_synth.circuits import Circuit, layered_random
from paper_2410_11415_amd import Circuit as Handle
from tests.test_gpu_rows import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [65, 83, 84, 85, 100, 127, 128])
@pytest.mark.parametrize("fanin,options", [(("geom", 2.0), {}), (("zipf", 1.5, 400), {"heavy_fan": 20, "min_segment": 7}), (("zipf", 1.5, 400), {"unary_chains": True})])
def test_both_kernels(batch, fanin, options):
    check(layered_random(6, 60, 8, 3000, fanin=fanin, groups=1), batch, **options)


FILL = 64 * 2048           # lanes of a launch from which on a lane takes more than one column


def lanes(batch):
    return (batch + 3) // 4


@pytest.mark.parametrize("batch", [65, 66, 83, 84, 85])
def test_many_rows_of_four_columns_per_lane(batch):
    c = layered_random(4, 128, 6, 150_000, fanin=("geom", 2.0), groups=2)
    k = Handle(*c.arrays(), device=-1, no_tail=True)
    rows = k.layer_sizes()[0]
    assert (rows[1:4] * lanes(batch) >= FILL).all() and 64 // lanes(84) == 3 and 64 // lanes(85) == 2
    k.close()
    check(c, batch, no_fusion=True)


@pytest.mark.parametrize("batch", [84, 85, 100, 127, 128])
def test_many_segments_of_split_rows(batch):
    """300 OR gates of 1500 children among 9000 AND gates: both directions are rows of 48 children or more, cut into segments"""
    rng = np.random.default_rng(3)
    ands = [sorted(int(v) + (64 if rng.random() < 0.5 else 0) for v in rng.permutation(64)[:2]) for _ in range(9000)]
    ors = [sorted(128 + int(x) for x in rng.permutation(9000)[:1500]) for _ in range(300)]
    kids = [[]] * 128 + ands + ors
    ptr = np.concatenate([[0], np.cumsum([len(x) for x in kids])]).astype(np.int64)
    lit = np.array(list(range(1, 65)) + list(range(-1, -65, -1)) + [0] * 9300, np.int32)
    c = Circuit(64, np.array([0] * 128 + [1] * 9000 + [2] * 300, np.uint8), lit, ptr, np.array([x for k in kids for x in k], np.int32),
                np.arange(9128, 9428, dtype=np.int32))
    k = Handle(*c.arrays(), device=-1, no_tail=True, no_merge=True)
    info = k.info()
    # the OR rows and all rows by child are split, into segments of at most 24 entries
    assert info["num_split_rows"] == 300 + 9000 + 128 and 450_000 / 24 * lanes(batch) >= FILL
    k.close()
    check(c, batch, no_merge=True)
