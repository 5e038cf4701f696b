"""Real-semiring reverse sweep (GPU), one quotient per row: rows whose own value is zero in some columns, parents with one and
with several zero children, plain and shared entries in one row, split rows; against the oracle.  Values at the ends of the
fp32 range, where a sum of the parents' P rows is out of range though the quotients are not; against sums in double."""
import numpy as np
import pytest

from klay_synth.circuits import AND, OR, CircuitBuilder, layered_random
from oracle import oracle
from tests.gpu_util import assert_grad_close, assert_real_close, gpu_eval, oracle_eval

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("options", [{}, {"unary_chains": True}, {"heavy_fan": 6, "min_segment": 5}, {"small_batch_edges": True}])
@pytest.mark.parametrize("batch", [1, 7, 32, 33, 66, 131])
def test_zero_values_in_wide_product_layers(batch, options):
    import paper_2410_11415_amd as klay
    c = layered_random(11, 48, 8, 3000, fanin=("geom", 2.2), groups=1)
    rng = np.random.default_rng(batch)
    p = rng.uniform(0.05, 0.95, size=(batch, c.num_vars)).astype(np.float32)
    p[rng.random(p.shape) < 0.08] = 0.0
    p[rng.random(p.shape) < 0.08] = 1.0
    dout = rng.normal(size=(batch, c.roots.shape[0])).astype(np.float32)
    k = klay.Circuit(*c.arrays(), device=0, no_tail=True, **options)
    out, grad = gpu_eval(k, p, klay.KLAY_REAL, dout)
    ref, rgrad = oracle_eval(c, p, klay.KLAY_REAL, dout, or_levels=k.num_layers // 2)
    vals = oracle.forward(*c.arrays(), p.astype(np.float64), klay.KLAY_REAL, nthreads=8, return_node_values=True)[1]
    zeros = np.array([(vals[:, c.children(n)] == 0.0).sum(axis=1) for n in np.flatnonzero(c.node_type == AND)])
    assert all((zeros == z).any() for z in (0, 1, 2)) and (vals[:, c.node_type == OR] == 0.0).any()
    assert_real_close(out, ref, "values")
    assert_grad_close(grad, rgrad, "gradients", real=True)
    k.close()


def products(parents, unary):
    """For each n of `parents` a variable with n parents AND(variable, a variable of its own); roots: those, or an OR gate over each"""
    b = CircuitBuilder(len(parents) + sum(parents))
    gates, hub, other = [], [], len(parents)
    for h, n in enumerate(parents):
        for _ in range(n):
            gates.append(b.and_(b.lit(h), b.lit(other)))
            hub.append(h)
            other += 1
    return b.finish([b.or_(g) for g in gates] if unary else gates), np.array(hub)


@pytest.mark.parametrize("options", [{"no_tail": True}, {"no_tail": True, "heavy_fan": 6, "min_segment": 5},
                                     {"no_tail": True, "small_batch_edges": True}])
@pytest.mark.parametrize("unary", [False, True])
@pytest.mark.parametrize("batch", [3, 7, 31, 50, 70, 100, 131, 300])
def test_values_at_the_ends_of_the_range(batch, unary, options):
    """values of 1e20 and 3e38 with parents whose products are near 2e38, tiny and subnormal values, zero"""
    import paper_2410_11415_amd as klay
    c, hub = products([2, 3, 20, 200], unary)
    rng = np.random.default_rng(batch)
    own = np.array([1e20, 0.0, 1.0, 3e38, 1e-30, 5e-39, 2e37])[(np.arange(batch) + rng.integers(7)) % 7]
    size = np.where(own >= 1e20, 2e38 / np.maximum(own, 1e20), np.where((own > 0) & (own < 1), 1e-10 / np.maximum(own, 5e-39), 1.0))
    size = np.minimum(size, 1e20)
    p = np.empty((batch, c.num_vars), np.float32)
    p[:, :4] = own[:, None] * rng.choice([1.0, -1.0], size=(batch, 4))
    p[:, 4:] = size[:, None] * rng.uniform(0.5, 1.0, size=(batch, c.num_vars - 4))
    dout = rng.uniform(0.5, 1.0, size=(batch, hub.size)).astype(np.float32)
    k = klay.Circuit(*c.arrays(), device=0, no_merge=True, **options)
    out, grad = gpu_eval(k, p, klay.KLAY_REAL, dout)
    k.close()
    x, d = p.astype(np.float64), dout.astype(np.float64)
    ref = np.concatenate([np.stack([(d * x[:, 4:])[:, hub == h].sum(axis=1) for h in range(4)], axis=1), d * x[:, hub]], axis=1)
    assert np.isfinite(ref.astype(np.float32)).all()
    # roundings: product, adjoint times value, lowest bit cleared (an ulp), the sum of n terms of one sign, the quotient; scaled subnormal
    # terms half of 2^-149, doubled by the quotient, and its own rounding
    n = np.concatenate([np.array([2, 3, 20, 200]), np.ones(hub.size)])
    bound = (0.5 * n + 4) * 2.0 ** -23 * np.abs(ref) + (n + 1) * 2.0 ** -149
    np.testing.assert_array_less(np.abs(grad - ref) - bound, 1e-300)


@pytest.mark.parametrize("options", [{"no_tail": True}, {"no_tail": True, "heavy_fan": 6, "min_segment": 5},
                                     {"no_tail": True, "small_batch_edges": True}])
@pytest.mark.parametrize("every_column", [False, True])
@pytest.mark.parametrize("batch", [3, 31, 50, 100, 300])
def test_an_infinite_adjoint_beside_a_sum_out_of_range(batch, every_column, options):
    """P rows of 2e38 each over a value of 1e20, and one of -inf: -inf, as the sum of the quotients, not inf - inf"""
    import paper_2410_11415_amd as klay
    c, hub = products([4, 20, 40, 200], False)
    p = np.full((batch, c.num_vars), 2e18, np.float32)
    p[:, :4] = 1e20
    dout = np.ones((batch, hub.size), np.float32)
    down = (np.arange(batch) % 3 > 0) | every_column       # the other columns stay finite
    for h in range(4):
        gate = np.flatnonzero(hub == h)[[-1, len(hub[hub == h]) // 2]]
        dout[np.ix_(down, gate[:1 + h % 2])] = -np.inf
    k = klay.Circuit(*c.arrays(), device=0, no_merge=True, **options)
    out, grad = gpu_eval(k, p, klay.KLAY_REAL, dout)
    k.close()
    assert (grad[down, :4] == -np.inf).all()
    n = np.array([4, 20, 40, 200])
    # (roundings: product, adjoint times value, an ulp, the sum, the quotient)
    assert (np.abs(grad[~down, :4] / (2e18 * n) - 1.0) < (0.5 * n + 4) * 2.0 ** -23).all()


@pytest.mark.parametrize("options", [{"no_tail": True}, {"no_tail": True, "heavy_fan": 6, "min_segment": 5},
                                     {"no_tail": True, "small_batch_edges": True}, {}])
@pytest.mark.parametrize("batch", [7, 32, 33, 66, 131, 257])
def test_each_number_of_zero_children_beside_plain_entries(batch, options):
    """rows with parents AND(x, a, b) and an OR gate above: x, a and b zero or not in every combination, against the product rule"""
    import paper_2410_11415_amd as klay
    parents = [1, 2, 4, 12, 60]
    b = CircuitBuilder(len(parents) + 2 * sum(parents))
    gates, plain, hub, other = [], [], [], len(parents)
    for h, n in enumerate(parents):
        for _ in range(n):
            gates.append(b.and_(b.lit(h), b.lit(other), b.lit(other + 1)))
            hub.append(h)
            other += 2
        plain.append(b.or_(b.lit(h), gates[-1]))
    c, hub = b.finish(gates + plain), np.array(hub)
    rng = np.random.default_rng(batch)
    p = rng.uniform(0.2, 2.0, size=(batch, c.num_vars)).astype(np.float32)
    p[rng.random(p.shape) < 0.3] = 0.0
    # columns in which every entry of a row concerns it, and none does
    p[0, :len(parents)], p[0, len(parents):] = 0.0, 1.5
    p[1, :len(parents)], p[1, len(parents):] = 1.5, 0.0
    dout = rng.uniform(0.5, 1.0, size=(batch, c.roots.shape[0])).astype(np.float32)
    x, d = p.astype(np.float64), dout.astype(np.float64)
    own, a, e = x[:, hub], x[:, len(parents)::2], x[:, len(parents) + 1::2]
    zeros = (own == 0).astype(int) + (a == 0) + (e == 0)
    assert all(((zeros == z) & (own == 0)).any() for z in (1, 2, 3)) and all(((zeros == z) & (own != 0)).any() for z in (0, 1, 2))
    g = d[:, :len(gates)].copy()
    for h in range(len(parents)):
        g[:, np.flatnonzero(hub == h)[-1]] += d[:, len(gates) + h]
    ref = np.empty(x.shape)
    for h in range(len(parents)):
        ref[:, h] = (g * a * e)[:, hub == h].sum(axis=1) + d[:, len(gates) + h]
    ref[:, len(parents)::2], ref[:, len(parents) + 1::2] = g * own * e, g * own * a
    k = klay.Circuit(*c.arrays(), device=0, no_merge=True, **options)
    out, grad = gpu_eval(k, p, klay.KLAY_REAL, dout)
    k.close()
    np.testing.assert_allclose(out[:, :len(gates)], own * a * e, rtol=2.0 ** -22, atol=0)
    # a sum of positive terms: product and adjoint (two roundings each and an ulp), up to 62 terms, the quotient
    np.testing.assert_allclose(grad, ref, rtol=(62 / 2 + 5) * 2.0 ** -23, atol=0)
