"""The persistent kernels (GPU) against the oracle, in the three semirings, with gradients: runs of every kind at the edges of
their chunks, quarters and blocks (EDGES; tests/test_host_cols.py checks on the host that these circuits have such runs),
circuits that merge to a few hundred gates, rows of 1 to 60 children, literals with thousands of parents, one, two and four columns
per workgroup, impossible and certain literals."""
import numpy as np
import pytest

from klay_synth import as_inputs
from klay_synth.circuits import Circuit
from tests.gpu_util import assert_grad_close, assert_log_close, assert_real_close, gpu_eval, oracle_eval

pytestmark = pytest.mark.gpu
REAL, LOG, MAXLOG = 0, 1, 2


def stack(rng, num_vars, widths, fan, hub):
    """Alternating AND / OR layers of the given widths; every gate draws fan(rng) distinct children of the layer below
    (and, with probability `hub`, one of the first four literals in an AND gate, which then have many parents)."""
    types, lits, kids = [0] * (2 * num_vars), [s * (v + 1) for v in range(num_vars) for s in (1, -1)], [[] for _ in range(2 * num_vars)]
    below = list(range(2 * num_vars))
    for depth, n in enumerate(widths):
        here = []
        for i in range(n):
            # every node below gets a parent where the layer is wide enough
            c = {below[i % len(below)]} | {int(x) for x in rng.choice(below, size=min(len(below), fan(rng)), replace=False)}
            if depth % 2 == 0 and rng.random() < hub:
                c.add(int(rng.integers(4)))
            here.append(len(types))
            types.append(1 if depth % 2 == 0 else 2)
            lits.append(0)
            kids.append(sorted(c))
        below = here
    ptr = np.concatenate([[0], np.cumsum([len(k) for k in kids])]).astype(np.int64)
    idx = np.array([x for k in kids for x in k], dtype=np.int32)
    return Circuit(num_vars, np.array(types, np.uint8), np.array(lits, np.int32), ptr, idx, np.array(below, np.int32))


FANS = {"one": lambda r: 1, "two": lambda r: 1 + int(r.integers(2)), "few": lambda r: 1 + int(r.integers(4)),
        "eight": lambda r: 1 + int(r.integers(8)), "long": lambda r: 1 + int(r.integers(60)) if r.random() < 0.1 else 1}


# (number of variables, layers from the bottom up: gates, times every node below is a child, gates with further random children and
# how many of those)
EDGES = {
    "wide": (8224, [(16385, 1, 0, 0), (4161, 1, 0, 0), (8321, 2, 0, 0), (8321, 2, 0, 0), (8321, 2, 0, 0), (8256, 2, 0, 0)]),
    "wide_odd": (8192, [(16383, 1, 0, 0), (16383, 1, 0, 0), (4223, 1, 0, 0), (8255, 2, 0, 0), (4161, 2, 0, 0), (4223, 3, 0, 0),
                        (4161, 3, 0, 0), (4223, 3, 0, 0)]),
    "long": (100, [(1999, 10, 1500, 40), (1983, 1, 1900, 50), (1951, 1, 0, 0), (129, 1, 0, 0)]),
    "two_columns": (2500, [(10239, 3, 0, 0), (8193, 1, 0, 0), (8193, 2, 0, 0), (8193, 2, 0, 0), (9025, 2, 1500, 20), (7743, 1, 1400, 18),
                           (4161, 1, 0, 0), (4097, 3, 0, 0)]),
    "four_columns": (1200, [(4031, 3, 0, 0), (2111, 1, 0, 0), (2047, 2, 0, 0), (2049, 2, 0, 0), (3009, 3, 500, 20), (2431, 1, 450, 18),
                            (1087, 1, 0, 0), (961, 3, 0, 0)]),
}


def edge_circuit(name):
    """Alternating AND / OR layers of exactly these sizes (build with no_merge)"""
    rng = np.random.default_rng(1)
    num_vars, layers = EDGES[name]
    types, lits, kids = [0] * (2 * num_vars), [s * (v + 1) for v in range(num_vars) for s in (1, -1)], [[] for _ in range(2 * num_vars)]
    first, m = 0, 2 * num_vars
    for depth, (n, times, long_gates, more) in enumerate(layers):
        at = len(types)
        shares = np.array_split(np.concatenate([rng.permutation(m) for _ in range(times)]), n)
        for i in range(n):
            c = {int(x) for x in shares[i]}
            if i < long_gates:
                c |= {int(x) for x in rng.permutation(m)[:more]}
            types.append(1 if depth % 2 == 0 else 2)
            lits.append(0)
            kids.append(sorted(first + x for x in c))
        first, m = at, n
    ptr = np.concatenate([[0], np.cumsum([len(k) for k in kids])]).astype(np.int64)
    idx = np.array([x for k in kids for x in k], dtype=np.int32)
    return Circuit(num_vars, np.array(types, np.uint8), np.array(lits, np.int32), ptr, idx, np.arange(first, first + m, dtype=np.int32))


@pytest.mark.parametrize("name,batch,zeros,cap,first", [
    ("wide", 2, 0.02, 0, 1), ("wide_odd", 1, 0.02, 0, 1), ("long", 3, 0.004, 0, 1), ("long", 258, 0.004, 0, 1), ("two_columns", 2, 0.01, 0, 1),
    ("two_columns", 257, 0.01, 0, 1), ("long", 514, 0.004, 0, 1), ("long", 1025, 0.004, 1990, 3), ("four_columns", 515, 0.01, 0, 1),
    ("four_columns", 1027, 0.01, 3100, 3), ("four_columns", 300, 0.01, 0, 1), ("four_columns", 2, 0.01, 0, 1), ("two_columns", 3, 0.01, 9100, 3), ("two_columns", 300, 0.01, 9100, 3), ("long", 5, 0.004, 1990, 3),
    ("wide_odd", 2, 0.02, 8300, 4)])
def test_runs_at_their_edges(name, batch, zeros, cap, first):
    import paper_2410_11415_amd as klay
    rng = np.random.default_rng(batch)
    c = edge_circuit(name)
    k = klay.Circuit(*c.arrays(), device=0, no_merge=True, tail_rows_cap=cap)
    assert k.info()["num_nodes"] == c.num_nodes and k.info()["tail_first_layer"] == first
    p = rng.uniform(0.5, 0.9, size=(batch, c.num_vars))
    u = rng.random(p.shape)
    p[u < zeros], p[u > 1 - zeros / 2] = 0.0, 1.0          # products with no, one and several zero children
    dout = rng.normal(size=(batch, c.roots.shape[0])).astype(np.float32)
    for semiring in (LOG, REAL, MAXLOG):
        with np.errstate(divide="ignore"):
            w = as_inputs(p, semiring != REAL)
        d = None if semiring == MAXLOG else dout
        out, grad = gpu_eval(k, w, semiring, d)
        ref, rgrad = oracle_eval(c, w, semiring, d, or_levels=k.num_layers // 2)
        (assert_real_close if semiring == REAL else assert_log_close)(out, ref, "values")
        if d is not None:
            assert_grad_close(grad, rgrad, "gradients", real=semiring == REAL)
    k.close()


@pytest.mark.parametrize("widths,fan,batch", [
    ((1, 1), "two", 1), ((63, 64, 65, 3), "two", 3), ((64, 128, 129, 127), "few", 2), ((255, 256, 257, 5), "eight", 257),
    ((1023, 1024, 1025, 40), "one", 5), ((1025, 511, 513, 9), "two", 2), ((2049, 2047, 300, 2), "few", 3), ((5000, 3000, 700, 64), "long", 2),
])
def test_layers_around_chunk_and_block_sizes(widths, fan, batch):
    """(gates that name the same children merge and gates without a parent go: a few hundred rows in the widest layer at most)"""
    import torch
    import paper_2410_11415_amd as klay
    rng = np.random.default_rng(len(widths) * 1000 + widths[0])
    c = stack(rng, 24, widths, FANS[fan], 0.6)
    k = klay.Circuit(*c.arrays(), device=0)
    assert k.info()["tail_first_layer"] == 1
    p = rng.uniform(0.05, 0.95, size=(batch, 24))
    p[0, 0], p[-1, 1] = 0.0, 1.0
    dout = rng.normal(size=(batch, c.roots.shape[0])).astype(np.float32)
    for semiring in (LOG, REAL, MAXLOG):
        with np.errstate(divide="ignore"):
            w = as_inputs(p, semiring != REAL)
        d = None if semiring == MAXLOG else dout
        out, grad = gpu_eval(k, w, semiring, d)
        ref, rgrad = oracle_eval(c, w, semiring, d, or_levels=k.num_layers // 2)
        (assert_real_close if semiring == REAL else assert_log_close)(out, ref, "values")
        if d is not None:
            assert_grad_close(grad, rgrad, "gradients", real=semiring == REAL)
    # a second reverse sweep of the same pass, and the entry point with no buffer for values
    w = torch.from_numpy(as_inputs(np.clip(p, 1e-6, 1 - 1e-6), True)).cuda()
    out = k.forward(w, LOG)
    g = [k.backward(torch.from_numpy(dout).cuda()) for _ in range(2)]
    assert torch.equal(g[0], g[1]) and torch.equal(out, k.forward_static(w, LOG))
    k.close()


@pytest.mark.parametrize("widths,batch,cap", [((40, 30, 20, 10), 3, 0), ((300, 500, 200, 90, 40), 5, 0), ((700, 400, 260, 130, 60, 20), 4, 200),
                                              ((700, 400, 260, 130, 60, 20), 4, 300), ((90, 70, 33), 259, 0), ((2000, 900, 500, 30), 1, 1000)])
def test_real_gradients_with_zeros_everywhere(widths, batch, cap):
    """products with no, one and several zero children in every layer the persistent reverse kernel takes, tops of both
    kinds, boundaries at odd and even layers"""
    import paper_2410_11415_amd as klay
    rng = np.random.default_rng(sum(widths))
    c = stack(rng, 10, widths, FANS["two"], 0.3)
    k = klay.Circuit(*c.arrays(), device=0, tail_rows_cap=cap)
    p = rng.uniform(0.2, 0.9, size=(batch, 10))
    p[rng.random(p.shape) < 0.3] = 0.0
    p[rng.random(p.shape) < 0.2] = 1.0
    w = as_inputs(p, False)
    dout = rng.normal(size=(batch, c.roots.shape[0])).astype(np.float32)
    for _ in range(2):
        out, grad = gpu_eval(k, w, REAL, dout)
    ref, rgrad = oracle_eval(c, w, REAL, dout, or_levels=k.num_layers // 2)
    assert (ref == 0).any() or (rgrad == 0).any()
    assert_real_close(out, ref, "values")
    assert_grad_close(grad, rgrad, "gradients", real=True)
    k.close()


def test_literal_with_hundreds_of_thousands_of_parents():
    """a leaf row of 287300 entries in the reverse kernel (281 blocks of one unit): every AND gate counts 20 leaf nodes of one
    literal next to two literals of its own"""
    import paper_2410_11415_amd as klay
    n = 170
    types, lits, kids = [0] * (n + 19), [v + 1 for v in range(n)] + [1] * 19, [[] for _ in range(n + 19)]
    ones = [0] + list(range(n, n + 19))
    gates = [(i, j) for i in range(1, n) for j in range(1, i)]
    gates += [(0, j) for j in range(1, n)]
    for i, j in gates:
        types.append(1)
        lits.append(0)
        kids.append(sorted(set(ones + [i, j])))
    first = n + 19
    roots = []
    for a in range(0, len(gates), 64):
        roots.append(len(types))
        types.append(2)
        lits.append(0)
        kids.append(list(range(first + a, first + min(a + 64, len(gates)))))
    ptr = np.concatenate([[0], np.cumsum([len(k) for k in kids])]).astype(np.int64)
    c = Circuit(n, np.array(types, np.uint8), np.array(lits, np.int32), ptr, np.array([x for k in kids for x in k], np.int32), np.array(roots, np.int32))
    k = klay.Circuit(*c.arrays(), device=0)
    info = k.info()
    assert info["tail_first_layer"] == 1 and info["max_fan_out"] > 255 * 1024
    rng = np.random.default_rng(5)
    p = rng.uniform(0.8, 0.99, size=(2, n))
    dout = rng.uniform(0.5, 1.5, size=(2, len(roots))).astype(np.float32)
    for semiring in (LOG, REAL):
        w = as_inputs(p, semiring != REAL)
        out, grad = gpu_eval(k, w, semiring, dout)
        ref, rgrad = oracle_eval(c, w, semiring, dout, or_levels=1)
        (assert_real_close if semiring == REAL else assert_log_close)(out, ref, "values")
        assert_grad_close(grad, rgrad, "gradients", real=semiring == REAL)
    k.close()


def covered_stack(rng, num_vars, widths, and_extra=0.02, or_fan=2):
    """Alternating AND / OR layers of exactly the given widths (build with no_merge): gate i of n has the nodes i, i + n, ..
    of the layer below, so every node has a parent; an AND gate has one more with probability `and_extra`, an OR gate
    or_fan - 1 more."""
    types, lits, kids = [0] * (2 * num_vars), [s * (v + 1) for v in range(num_vars) for s in (1, -1)], [[] for _ in range(2 * num_vars)]
    first, m = 0, 2 * num_vars
    for depth, n in enumerate(widths):
        at = len(types)
        for i in range(n):
            more = int(rng.random() < and_extra) if depth % 2 == 0 else or_fan - 1
            c = set(range(i % m, m, n)) | {int(x) for x in rng.integers(m, size=more)}
            types.append(1 if depth % 2 == 0 else 2)
            lits.append(0)
            kids.append(sorted(first + x for x in c))
        first, m = at, n
    ptr = np.concatenate([[0], np.cumsum([len(k) for k in kids])]).astype(np.int64)
    idx = np.array([x for k in kids for x in k], dtype=np.int32)
    return Circuit(num_vars, np.array(types, np.uint8), np.array(lits, np.int32), ptr, idx, np.arange(first, first + m, dtype=np.int32))


@pytest.mark.parametrize("widths,batch", [
    ([900] * 24, 3),                                   # own values of every step behind the two arrays
    ([900] * 24, 258),                                 # the same with two columns per workgroup
    ([2500] * 20 + [1300, 700], 2),                    # of some steps only: the rest a step ahead
    ([5000, 5000] + [600] * 10, 2),                    # in the part of an array that only the wide layers need
    ([6000, 6000] + [2999] * 7 + [60, 60, 20], 259),
    ([900] * 24, 514), ([2999] * 9 + [60, 60, 20], 517),                 # four columns
])
def test_own_values_wherever_the_reverse_kernel_keeps_them(widths, batch):
    import paper_2410_11415_amd as klay
    rng = np.random.default_rng(sum(widths) + batch)
    c = covered_stack(rng, 300, widths)
    k = klay.Circuit(*c.arrays(), device=0, no_merge=True)
    assert k.info()["num_nodes"] == 600 + sum(widths) and k.info()["tail_first_layer"] == 1
    p = rng.uniform(0.3, 0.7, size=(batch, 300))
    dout = rng.normal(size=(batch, widths[-1])).astype(np.float32)
    for semiring in (LOG, REAL):
        w = as_inputs(p, semiring != REAL)
        out, grad = gpu_eval(k, w, semiring, dout)
        ref, rgrad = oracle_eval(c, w, semiring, dout, or_levels=len(widths) // 2)
        (assert_real_close if semiring == REAL else assert_log_close)(out, ref, "values")
        assert_grad_close(grad, rgrad, "gradients", real=semiring == REAL)
    k.close()


def test_sums_of_long_rows_are_balanced():
    """A literal with 15000 parents whose adjoints are 2^27 once and 1 otherwise: an addition with the large number in it is
    off by at most 8.  With the 8 entries of a line summed as pairs, and the two lines of a block (16 ones, exact) before they
    join, the seven ones of its line are lost, and up to 8 in its block, in the partial last block and in each of the 6
    steps over the lanes: 71.  Adding a line's entries or pairs one after another loses all 8 of every line: up to 234."""
    import torch
    import paper_2410_11415_amd as klay
    n = 15000
    types = [0] * (n + 1) + [1] * n + [2] * n
    lits = [v + 1 for v in range(n + 1)] + [0] * (2 * n)
    ptr = np.concatenate([np.zeros(n + 1), 2 * np.arange(n + 1), 2 * n + 1 + np.arange(n)]).astype(np.int64)
    pairs = np.stack([np.zeros(n, np.int32), 1 + np.arange(n, dtype=np.int32)], axis=1).ravel()
    idx = np.concatenate([pairs, n + 1 + np.arange(n)]).astype(np.int32)
    c = Circuit(n + 1, np.array(types, np.uint8), np.array(lits, np.int32), ptr, idx, 2 * n + 1 + np.arange(n, dtype=np.int32))
    k = klay.Circuit(*c.arrays(), device=0)
    assert k.info()["tail_first_layer"] == 1 and k.info()["max_fan_out"] == n
    batch = 16
    dout = np.ones((batch, n), np.float32)
    for b in range(batch):
        dout[b, n * b // batch] = 2.0 ** 27
    k.forward(torch.full((batch, n + 1), -0.5, device="cuda"), LOG)
    got = k.backward(torch.from_numpy(dout).cuda()).cpu().numpy().astype(np.float64)
    np.testing.assert_array_equal(got[:, 1:], dout)
    assert np.abs(got[:, 0] - (2.0 ** 27 + n - 1)).max() <= 71, got[:, 0] - 2.0 ** 27
    k.close()
