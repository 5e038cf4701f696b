"""Real-semiring reverse sweep (GPU), one quotient per row: rows whose own value is zero in some columns, parents with one and
with several zero children, plain and shared entries in one row, split rows; against the oracle.  Values at the ends of the
fp32 range, where a sum of the parents' P rows is out of range though the quotients are not; against sums in double."""
import numpy as np
import pytest

from klay_synth.circuits import CircuitBuilder, layered_random
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
    assert (np.asarray(ref) == 0.0).any() or (p == 0.0).any()
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
