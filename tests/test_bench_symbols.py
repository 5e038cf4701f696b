"""bench.py finds the traffic table's entry for a kernel also where the table has two forms of it, with no GPU: a table of a loop with
backward passes holds the launches of its first step, which leaves fused rows out, as kernels of their own."""
import pytest

import bench


@pytest.mark.parametrize("cls,op", [("fwd_sum", 0), ("bwd_sum", 0), ("fwd_prod", 1)])
@pytest.mark.parametrize("batch,vec", [(256, 4), (100, 2)])
def test_both_forms_in_the_table(cls, op, batch, vec):
    table = {"klay::stream_kernel<%d, %d, false>" % (op, vec): "all rows", "klay::stream_kernel<%d, %d, true>" % (op, vec): "kept rows"}
    assert bench.measured_kernel(table, bench.kernel_symbol(cls, batch, backward=True)) == "all rows"


@pytest.mark.parametrize("form", ["false", "true"])
def test_one_form_in_the_table(form):
    table = {"klay::stream_kernel<0, 4, %s>" % form: "it", "klay::stream_kernel<2, 4, false>": "another"}
    assert bench.measured_kernel(table, bench.kernel_symbol("fwd_sum", 256)) == "it"
