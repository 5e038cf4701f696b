"""Segments of split logsumexp rows in a launch of their own (GPU): 33 to 64 columns, two and four per lane, segments shorter and longer than
the eight entries a step takes and of whole steps, against numpy in double, over ordinary weights and over those at the ends of the range."""
import numpy as np
import pytest

from klay_synth.circuits import CircuitBuilder

pytestmark = pytest.mark.gpu
VARS = 512
FILL = 64 * 2048             # lanes from which on a lane takes more columns
SMALL = 100000               # entries up to which segments and main rows go together

# fan-in of the split rows, shortest segment asked for, the entries of a whole segment that come of it
SHAPES = [((43, 49), 5, 7), ((50, 64), 5, 8), ((65, 81), 5, 9), ((197, 225), 5, 15), ((226, 256), 5, 16), ((257, 289), 5, 17), ((201, 219), 24, 24), ((201, 219), 32, 32)]


def cases():
    for batch in (33, 34, 47, 50, 61, 64):
        for columns in (2, 4):
            for fans, least, length in SHAPES:
                per_row = -(-sum(fans) // 2 // length)
                segments = int(1.04 * max(FILL / -(-batch // columns), SMALL * per_row / (sum(fans) / 2))) + 40
                if columns == 4 or segments * -(-batch // 4) < FILL:
                    yield pytest.param(batch, columns, fans, least, length, segments, id="%d-%d-%d" % (batch, columns, length))


def circuit(rng, fans, length, segments):
    """OR gates of as many literals, so many segments in all, and some of two literals"""
    b = CircuitBuilder(VARS)
    kids, count = [], 0
    while count < segments:
        kids.append(rng.choice(VARS, size=int(rng.integers(fans[0], fans[1] + 1)), replace=False))
        count += -(-len(kids[-1]) // length)
    entries = sum(len(row) for row in kids)
    kids += [rng.choice(VARS, size=2, replace=False) for _ in range(20)]
    lits = [b.lit(v) for v in range(VARS)]
    return b.finish([b.or_(*[lits[v] for v in row]) for row in kids]), kids, count, entries


def reference(w, kids):
    out = np.empty((w.shape[0], len(kids)))
    with np.errstate(all="ignore"):
        for r, row in enumerate(kids):
            x = np.where(np.isnan(w[:, row]), -np.inf, w[:, row])
            m = x.max(axis=1)
            out[:, r] = np.where(np.isinf(m), m, m + np.log(np.exp(x - np.where(np.isinf(m), 0.0, m)[:, None]).sum(axis=1)))
    return out


@pytest.mark.parametrize("batch,columns,fans,least,length,segments", cases())
def test_segments(batch, columns, fans, least, length, segments):
    import torch
    import paper_2410_11415_amd as klay
    rng = np.random.default_rng(batch + length)
    c, kids, count, entries = circuit(rng, fans, length, segments)
    k = klay.Circuit(*c.arrays(), device=0, no_tail=True, heavy_fan=40, min_segment=least)
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
    k.set_profiling(True)
    got = k.forward(torch.from_numpy(w).cuda(), klay.KLAY_LOG).cpu().numpy().astype(np.float64)
    split = k.get_profile()["split"]
    k.close()
    # a launch of segments, as many and as long as meant, with as many columns per lane
    assert split["launches"] == 1 and split["alg_bytes"] == 4 * (batch + 1) * (entries + count)
    assert count * -(-batch // columns) >= FILL and (columns == 4 or count * -(-batch // 4) < FILL)
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
