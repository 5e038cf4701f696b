"""The double-precision persistent kernels (GPU) against the oracle, in the three semirings, with gradients where there are any: runs of
every kind at the edges of their chunks, quarters and blocks (the circuits of test_gpu_cols.py), layers on both sides of what the
LDS holds, circuits with long rows that a TopPlan takes whole and in part, impossible and certain literals, batches of one turn and
of two, and a backward pass called twice."""
import numpy as np
import pytest

from klay_synth import leaf_probs
from klay_synth.circuits import layered_random
from tests.test_gpu_cols import edge_circuit, stack
from tests.test_gpu_parity import _f64_case, build, klay  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu
REAL, LOG, MAXLOG = 0, 1, 2


def first_layers(c, batch, **options):
    """(first layer, plan) that the double-precision kernels take in the three passes of _f64_case; the second follows a backward pass"""
    from paper_2410_11415_amd import Circuit
    k = Circuit(*c.arrays(), device=-1, **options)
    out = [k.persistent_layers(batch, LOG, True), k.persistent_layers(batch, REAL, True, training=True), k.persistent_layers(batch, MAXLOG, True, training=True)]
    k.close()
    return out


@pytest.mark.parametrize("name,batch", [("long", 1), ("long", 258), ("four_columns", 5), ("two_columns", 2), ("wide_odd", 2)])
def test_edges_of_runs(klay, name, batch):  # noqa: F811
    c = edge_circuit(name)
    first = {("long", 1): 3, ("long", 258): 1, ("four_columns", 5): 1, ("two_columns", 2): 7, ("wide_odd", 2): 5}[name, batch]
    # (two layers of a wide circuit do not pay for the rows of the real semiring's sweep)
    assert first_layers(c, batch, no_merge=True) == [(first, 1), (0, 0) if name == "two_columns" else (first, 1), (first, 1)]
    _f64_case(klay, c, leaf_probs(batch, batch, c.num_vars, ("uniform", 0.3, 0.7)), name, no_merge=True)


@pytest.mark.parametrize("widths", [[1, 1], [3, 2, 1], [64, 63, 65, 1], [5119, 5100, 40, 7], [10232, 5112, 10232, 5112, 9], [10240, 5112, 10300, 5200, 33, 2]])
def test_layers_around_what_the_lds_holds(klay, widths):  # noqa: F811
    rng = np.random.default_rng(len(widths))
    c = stack(rng, 60, widths, lambda r: 1 + int(r.integers(3)), 0.05)
    assert first_layers(c, 2, no_merge=True) == [(1, 1)] * 3
    p = leaf_probs(2, 7, 60, ("uniform", 0.3, 0.7))
    _f64_case(klay, c, p, str(widths), no_merge=True)
    p[1:, ::9] = 0.0
    p[::2, 4::11] = 1.0
    _f64_case(klay, c, p, "zeros %s" % widths, no_merge=True, backward=False)


@pytest.mark.parametrize("which", ["whole", "part", "capped"])
@pytest.mark.parametrize("batch", [3, 70, 257])
def test_long_rows(klay, which, batch):  # noqa: F811
    gates = {"whole": 3000, "part": 30000, "capped": 3000}[which]
    c = layered_random(3, num_vars=40, depth=10, num_gates=gates, fanin=("zipf", 1.6, 600), groups=1, num_roots=9)
    options = dict(tail_rows_cap=400) if which == "capped" else {}
    # (in part only up to 256 columns, in the real semiring where the rows it leaves to the launches are few)
    want = {"whole": [(1, 2)] * 3, "part": [(3, 2)] * 3 if batch == 3 else [(1, 2)] * 3, "capped": [(7, 2)] * 3 if batch < 257 else [(0, 0)] * 3}[which]
    if which == "part" and batch == 257:
        want[1] = (0, 0)
    assert first_layers(c, batch, **options) == want
    _f64_case(klay, c, leaf_probs(batch, batch, 40, ("beta", 0.5, 0.5)), which, neg=batch == 3, **options)


def test_backward_twice_after_one_forward(klay):  # noqa: F811
    import torch
    for c, options in ((layered_random(3, num_vars=40, depth=10, num_gates=3000, fanin=("zipf", 1.6, 600), groups=1, num_roots=9), dict(tail_rows_cap=400)),
                       (layered_random(4, num_vars=40, depth=10, num_gates=9000, fanin=("geom", 2.0), groups=1, num_roots=9), dict(tail_rows_cap=700)),
                       (layered_random(4, num_vars=40, depth=10, num_gates=900, fanin=("geom", 2.0), groups=1, num_roots=9), {})):
        k = build(klay, c, **options)
        w = torch.log(torch.rand((21, 40), device="cuda", dtype=torch.float64))
        dout = torch.rand((21, k.num_roots), device="cuda", dtype=torch.float64)
        k.forward_f64(w, LOG)
        a, b = k.backward_f64(dout).clone(), k.backward_f64(dout).clone()
        assert torch.equal(a, b)
        k.close()


@pytest.mark.parametrize("which,batch", [("two_columns", 2), ("wide_odd", 2), ("part", 257), ("long", 258)])
def test_the_real_semiring_in_the_first_step(klay, which, batch):  # noqa: F811
    """the reverse sweep by launches, from values that are put into rows; a later step may leave the layers to the launches"""
    import torch
    from oracle import oracle
    c = (layered_random(3, num_vars=40, depth=10, num_gates=30000, fanin=("zipf", 1.6, 600), groups=1, num_roots=9) if which == "part"
         else edge_circuit(which))
    k = build(klay, c, no_merge=which != "part")
    assert k.persistent_layers(batch, REAL, True)[1] == (2 if which == "part" else 1)
    p = leaf_probs(batch, batch, c.num_vars, ("uniform", 0.3, 0.7)).astype(np.float64)
    p[:, 1] = 0.0
    d = np.random.default_rng(batch).normal(size=(batch, c.roots.shape[0]))
    out = k.forward_f64(torch.from_numpy(p).cuda(), REAL).cpu().numpy()
    grad = k.backward_f64(torch.from_numpy(d).cuda()).cpu().numpy()
    k.close()
    np.testing.assert_allclose(out, oracle.forward(*c.arrays(), p, REAL, nthreads=8), rtol=1e-12, atol=1e-300)
    ref = oracle.backward(*c.arrays(), p, REAL, d, nthreads=8)
    mass = oracle.backward(*c.arrays(), p, REAL, d, nthreads=8, path_mass=True)
    assert np.all(np.abs(grad - ref) <= 1e-10 * np.maximum(1.0, mass))
