"""Batches of 65 to 128 columns (GPU): the rule that takes a pass to the generic or to the streaming kernel, on both sides of its
column limit, in circuits of short rows and of mostly split ones; three semirings with gradients, against the oracle."""
import pytest

from klay_synth.circuits import layered_random
from tests.test_gpu_rows import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [65, 83, 84, 85, 100, 127, 128])
@pytest.mark.parametrize("fanin,options", [(("geom", 2.0), {}), (("zipf", 1.5, 400), {"heavy_fan": 20, "min_segment": 7}), (("zipf", 1.5, 400), {"unary_chains": True})])
def test_both_kernels(batch, fanin, options):
    check(layered_random(6, 60, 8, 3000, fanin=fanin, groups=1), batch, **options)
