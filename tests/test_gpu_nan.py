"""NaN and infinite weights in the log domain (GPU).  A child that is NaN (a NaN weight, or the negated literal of a weight above 0)
is an impossible child of an OR gate and makes an AND gate NaN; a child at +inf makes its OR gate +inf.  The fp32 kernels agree on
that whichever of them a batch and an option select; compared with those rules applied gate by gate in double.  The
double-precision kernel passes a NaN on, except from a gate whose other children are all impossible."""
import numpy as np
import pytest

from klay_synth.circuits import AND, FALSE, LIT, OR, CircuitBuilder, layered_random
from tests.gpu_util import LOG_ATOL

pytestmark = pytest.mark.gpu
LOG, MAXLOG = 1, 2


def evaluate(c, w, semiring):
    """[B, R]: the gates in order, a NaN child of an OR gate left out"""
    vals = [None] * c.num_nodes
    with np.errstate(all="ignore"):
        for n in range(c.num_nodes):
            t, kids = c.node_type[n], c.child_idx[c.child_ptr[n]:c.child_ptr[n + 1]]
            if t == LIT:
                x = w[:, abs(c.node_lit[n]) - 1]
                vals[n] = x if c.node_lit[n] > 0 else np.log(-np.expm1(x))
            elif t == AND:
                vals[n] = np.sum([vals[i] for i in kids], axis=0)
            elif t == OR:
                e = np.array([np.where(np.isnan(vals[i]), -np.inf, vals[i]) for i in kids])
                m = e.max(axis=0)
                s = np.where(np.isinf(m), m, m + np.log(np.exp(e - np.where(np.isinf(m), 0.0, m)).sum(axis=0)))
                vals[n] = m if semiring == MAXLOG else s
            else:
                vals[n] = np.full(w.shape[0], -np.inf if t == FALSE else 0.0)
    return np.stack([vals[r] for r in c.roots], axis=1)


def weights(rng, batch, num_vars):
    w = np.log(rng.uniform(0.05, 0.95, size=(batch, num_vars)))
    u = rng.random(w.shape)
    w[u < 0.06] = np.nan
    w[(u >= 0.06) & (u < 0.1)] = 1e-3                     # above 0: the negated literal is NaN
    w[(u >= 0.1) & (u < 0.13)] = -np.inf
    w[(u >= 0.13) & (u < 0.135)] = np.inf
    return w.astype(np.float32)


NARROW = layered_random(11, 40, 8, 1500, fanin=("geom", 2.0), groups=1, num_roots=16, shuffle_ids=False)
SPLIT = layered_random(12, 60, 8, 3000, fanin=("zipf", 1.6, 400), groups=1, num_roots=16, shuffle_ids=False)


@pytest.mark.parametrize("c,batch,options", [
    (NARROW, 3, {}), (NARROW, 260, {}), (NARROW, 600, {}),                            # persistent kernels, one, two and four columns
    (NARROW, 1, dict(no_tail=True)), (NARROW, 10, dict(no_tail=True)),               # generic row kernel
    (SPLIT, 5, dict(heavy_fan=20, min_segment=7)), (SPLIT, 31, dict(heavy_fan=20, min_segment=7)),      # and combine rows
    (SPLIT, 6, dict(heavy_fan=20, min_segment=7, no_tail=True, small_batch_edges=True)),
    (SPLIT, 40, dict(heavy_fan=20, min_segment=7, no_tail=True)),                     # one column per lane
    (SPLIT, 130, dict(heavy_fan=20, min_segment=7, no_tail=True)),                    # streams, fused rows
    (SPLIT, 300, dict(heavy_fan=20, min_segment=7, no_tail=True, no_fusion=True)),
])
def test_nan_and_infinite_weights(c, batch, options):
    import torch
    import paper_2410_11415_amd as klay
    assert np.all(c.child_idx < np.repeat(np.arange(c.num_nodes), np.diff(c.child_ptr)))       # children come first
    assert np.all(c.node_type[c.roots] == OR)
    w = weights(np.random.default_rng(batch), batch, c.num_vars)
    k = klay.Circuit(*c.arrays(), device=0, **options)
    for semiring in (LOG, MAXLOG):
        ref = evaluate(c, w.astype(np.float64), semiring)
        got = k.forward(torch.from_numpy(w).cuda(), semiring).cpu().numpy()
        assert np.isfinite(ref).any() and not np.isnan(ref).any()
        np.testing.assert_array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
        assert np.abs(got[np.isfinite(ref)] - ref[np.isfinite(ref)]).max() <= LOG_ATOL
    k.close()


@pytest.mark.parametrize("children,batch", [(1, 2), (2, 70), (4, 3), (7, 5), (33, 4)])
def test_rows_of_nothing_but_nan_and_impossible_children(children, batch):
    """every fp32 kernel answers -inf, the double-precision one too; one possible child more, and fp32 answers that child and
    double NaN"""
    import torch
    import paper_2410_11415_amd as klay
    b = CircuitBuilder(40)
    lits = [b.lit(v) for v in range(children)]
    c = b.finish([b.or_(*lits), b.or_(*lits, b.lit(children))])
    w = np.full((batch, 40), -1.0, np.float32)
    w[:, 0], w[:, 1:children] = np.nan, -np.inf
    for options in ({}, dict(no_tail=True), dict(no_tail=True, small_batch_edges=True)):
        k = klay.Circuit(*c.arrays(), device=0, **options)
        for semiring in (LOG, MAXLOG):
            got = k.forward(torch.from_numpy(w).cuda(), semiring).cpu().numpy()
            np.testing.assert_array_equal(got, np.tile(np.float32([-np.inf, -1.0]), (batch, 1)))
        f64 = k.forward_f64(torch.from_numpy(w.astype(np.float64)).cuda(), LOG).cpu().numpy()
        assert np.all(np.isneginf(f64[:, 0])) and np.all(np.isnan(f64[:, 1]))
        k.close()
