"""Circuits with literals of few of their variables (GPU): the persistent kernel's leaf layer by the list of those variables, and without
it, against the same circuit over these variables alone, whose passes do the same sums."""
import numpy as np
import pytest

from klay_synth.circuits import layered_random, tiny_ddnnf

pytestmark = pytest.mark.gpu
REAL, LOG = 0, 1


@pytest.mark.parametrize("batch", [1, 5, 300, 1030])               # one, two and four columns per workgroup
@pytest.mark.parametrize("num_vars,kind", [(40, "tiny"), (1200, "tiny"), (9000, "tiny"), (9000, "layered")])
def test_few_variables(num_vars, kind, batch):
    import torch
    import paper_2410_11415_amd as klay
    c = tiny_ddnnf(3, 12, 30)[0] if kind == "tiny" else layered_random(3, 60, 12, 4000, fanin=("zipf", 1.6, 400), groups=2)
    rng = np.random.default_rng(num_vars + batch)
    at = np.sort(rng.choice(num_vars, size=c.num_vars, replace=False))
    _, node_type, lit, ptr, idx, roots = c.arrays()
    spread = np.where(lit == 0, 0, np.sign(lit) * (at[np.abs(lit) - 1] + 1)).astype(lit.dtype)
    few, alone = klay.Circuit(num_vars, node_type, spread, ptr, idx, roots, device=0), klay.Circuit(*c.arrays(), device=0)
    # (a variable without literals: a value that would show wherever it is used)
    w = torch.full((batch, num_vars), float("nan"), device="cuda")
    w[:, at] = torch.from_numpy(rng.uniform(0.05, 0.95, size=(batch, c.num_vars)).astype(np.float32)).cuda()
    neg = torch.full_like(w, float("nan"))
    neg[:, at] = torch.from_numpy(rng.uniform(0.05, 0.95, size=(batch, c.num_vars)).astype(np.float32)).cuda()
    unused = np.setdiff1d(np.arange(num_vars), at)
    for semiring in (LOG, REAL):
        x, y = (torch.log(w), torch.log(neg)) if semiring == LOG else (w, neg)
        xs, ys = x[:, at].contiguous(), y[:, at].contiguous()
        for explicit in (False, True):
            got = few.forward(x, semiring, neg_weights=y if explicit else None)
            want = alone.forward(xs, semiring, neg_weights=ys if explicit else None)
            assert torch.equal(got, want)
            dout = torch.rand_like(got)
            grads, wants = few.backward(dout), alone.backward(dout)
            for g, h in zip(grads if explicit else (grads,), wants if explicit else (wants,)):
                assert torch.equal(g[:, at], h) and not g[:, unused].any()
        assert torch.equal(few.forward_static(x, semiring), alone.forward_static(xs, semiring))
    few.close()
    alone.close()
