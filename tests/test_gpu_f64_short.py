"""Rows of 1 to 13 entries in the double-precision generic kernel (GPU), a wave to a row (33 to 64 columns, one per lane, and 65 to 128, two) and
several rows to a wave, alone (seven entries a row on average) and among many of two, where a wave with one row takes no exponential past its
end; with NaN, infinite and extreme weights, against numpy: a NaN passes on, except from a row whose other children are all impossible."""
import numpy as np
import pytest

from klay_synth.circuits import CircuitBuilder

pytestmark = pytest.mark.gpu
VARS = 40


@pytest.mark.parametrize("batch", [20, 33, 50, 64, 67, 128])
@pytest.mark.parametrize("pairs", [0, 4000])
def test_short_rows(batch, pairs):
    import torch
    import paper_2410_11415_amd as klay
    rng = np.random.default_rng(batch)
    kids = [rng.choice(VARS, size=n, replace=False) for n in range(1, 14) for _ in range(30)]
    kids += [rng.choice(VARS, size=2, replace=False) for _ in range(pairs)]
    kids += [np.array([0, 1]), np.array([1, 0]), np.array([2, 0]), np.array([0, 2])]
    b = CircuitBuilder(VARS)
    lits = [b.lit(v) for v in range(VARS)]
    c = b.finish([b.or_(*[lits[v] for v in row]) for row in kids])
    w = -rng.exponential(3.0, size=(batch, VARS))
    special = np.array([-np.inf, -np.inf, np.inf, np.nan, np.finfo(np.float64).min, -1e300, 0.0])
    w[4:] = np.where(rng.random((batch - 4, VARS)) < 0.3, rng.choice(special, size=(batch - 4, VARS)), w[4:])
    w[2], w[3, 1:] = -np.inf, -np.inf
    w[1] = np.log(0.5)                                    # equal terms
    k = klay.Circuit(*c.arrays(), device=0, no_tail=True)
    got = k.forward_f64(torch.from_numpy(w).cuda(), klay.KLAY_LOG).cpu().numpy()
    k.close()
    ref = np.empty_like(got)
    with np.errstate(all="ignore"):
        for r, row in enumerate(kids):
            x = w[:, row]
            m = np.where(np.isnan(x), -np.inf, x).max(axis=1)
            s = m + np.log(np.exp(x - np.clip(m, -1.7e308, 1.7e308)[:, None]).sum(axis=1))
            # (the lowest value is taken for an impossible child where nothing is above it)
            ref[:, r] = np.where((m == -np.inf) | (m == np.finfo(np.float64).min), -np.inf, s)
    np.testing.assert_array_equal(np.isnan(got), np.isnan(ref))
    inf = np.isinf(ref)
    np.testing.assert_array_equal(got[inf], ref[inf])
    fin = np.isfinite(ref)
    # exponentials and the logarithm within an ulp or two, up to thirteen terms
    np.testing.assert_allclose(got[fin], ref[fin], rtol=1e-14, atol=1e-14)
