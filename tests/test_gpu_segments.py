"""Segments of split logsumexp rows in a launch of their own (GPU): 33 to 64 columns, two and four per lane, segments shorter and longer than
the eight entries a step takes, against numpy in double, over ordinary weights and over those at the ends of the range."""
import numpy as np
import pytest

from klay_synth.circuits import CircuitBuilder

pytestmark = pytest.mark.gpu
VARS, ROWS = 512, 1200


def circuit(rng):
    """1200 OR gates of 201 to 219 literals each (more than 10^5 entries: not a small launch), and some of two"""
    b = CircuitBuilder(VARS)
    kids = [rng.choice(VARS, size=int(rng.integers(201, 220)), replace=False) for _ in range(ROWS)]
    kids += [rng.choice(VARS, size=2, replace=False) for _ in range(20)]
    lits = [b.lit(v) for v in range(VARS)]
    return b.finish([b.or_(*[lits[v] for v in row]) for row in kids]), kids


def reference(w, kids):
    out = np.empty((w.shape[0], len(kids)))
    with np.errstate(all="ignore"):
        for r, row in enumerate(kids):
            x = np.where(np.isnan(w[:, row]), -np.inf, w[:, row])
            m = x.max(axis=1)
            out[:, r] = np.where(np.isinf(m), m, m + np.log(np.exp(x - np.where(np.isinf(m), 0.0, m)[:, None]).sum(axis=1)))
    return out


@pytest.mark.parametrize("batch", [33, 34, 47, 50, 61, 64])
@pytest.mark.parametrize("segment", [24, 9, 5])
def test_segments(batch, segment):
    import torch
    import paper_2410_11415_amd as klay
    rng = np.random.default_rng(batch + segment)
    c, kids = circuit(rng)
    k = klay.Circuit(*c.arrays(), device=0, no_tail=True, heavy_fan=40, min_segment=segment)
    assert k.info()["num_split_rows"] >= ROWS
    w = -rng.exponential(10.0, size=(batch, VARS)).astype(np.float32)
    w[1] *= 1e4                                            # one term outweighs the others, of any size
    w[2] = -7e4 - rng.random(VARS)                         # large values close together: the sum counts
    w[3] = 1e6 + rng.random(VARS)
    w[4] = -2e8 * (1.0 + rng.random(VARS))                 # above 2^27: the maximum alone
    w[5] = np.where(rng.random(VARS) < 0.97, np.finfo(np.float32).min, w[5])     # masks of the lowest value
    w[6] = np.finfo(np.float32).min
    w[7] = -np.inf
    u = rng.random((batch - 8, VARS))
    w[8:][u < 0.3] = -np.inf
    w[8:][(u >= 0.3) & (u < 0.4)] = np.nan
    w[8, 5] = np.inf
    ref = reference(w.astype(np.float64), kids)
    got = k.forward(torch.from_numpy(w).cuda(), klay.KLAY_LOG).cpu().numpy().astype(np.float64)
    k.close()
    inf = np.isinf(ref)
    np.testing.assert_array_equal(got[inf], ref[inf])
    # Two stages, each with an ulp of the value; and in the logarithm of the sum: the exponent of a term that counts (up to 2^5) rounded
    # to 2^-24 of itself, and fewer than 32 sums and products in a row of half an ulp each
    np.testing.assert_allclose(got[~inf], ref[~inf], rtol=4 * 2.0 ** -24, atol=64 * 2.0 ** -24)


def test_segments_of_thousands():
    """Beyond 2^27, where an ulp is 16, the logarithm of 2980 equal terms does not round away any more."""
    import torch
    import paper_2410_11415_amd as klay
    from klay_synth.circuits import LIT, OR
    variables, rows, segment = 6200, 2060, 3000            # two segments a row, enough of them for two columns per lane
    fan = np.array([2 * segment] * rows + [2])             # (and a row that is not split)
    child = np.concatenate([(np.arange(k) * 7 + r) % variables for r, k in enumerate(fan)]).astype(np.int32)
    n = variables + len(fan)
    node_type = np.array([LIT] * variables + [OR] * len(fan), dtype=np.uint8)
    lit = np.concatenate([np.arange(1, variables + 1), np.zeros(len(fan))]).astype(np.int32)
    ptr = np.concatenate([np.zeros(variables + 1), np.cumsum(fan)]).astype(np.int64)
    k = klay.Circuit(variables, node_type, lit, ptr, child, np.arange(variables, n, dtype=np.int32), device=0, no_tail=True, min_segment=segment)
    assert k.info()["num_split_rows"] >= rows
    x = np.float32(1.03 * 2 ** 27)
    got = k.forward(torch.full((64, variables), float(x), device="cuda"), klay.KLAY_LOG).cpu().numpy()
    k.close()
    assert (got[:, :rows] == x + np.float32(16)).all()     # 8.7 more, of an ulp of 16
    assert (got[:, rows] == x).all()
