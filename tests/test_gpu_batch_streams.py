"""GPU: the batch's separate band products load the bands of a list that exceeds
the last-level cache non-temporally (7282 tiles of 1024 nodes and more); on either
side of that line a problem gets the bits it gets alone."""
import pytest
import torch

import paper_0904_4152_amd as mg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("levels", [[11], [11, 11, 6], [9] * 28, [9] * 29, [10, 11, 10, 11]])
@pytest.mark.parametrize("nu", [(1, 1), (0, 3)])
def test_each_problem_as_alone(levels, nu):
    ctx = mg.Context(0)
    o = mg.default_opts(precision=1, nu_pre=nu[0], nu_post=nu[1], fixed_cycles=2)
    hs = [mg.Hierarchy(ctx, L, jitter=0.2, seed=20 + i) for i, L in enumerate(levels)]
    bs = [torch.zeros(h.n, dtype=torch.float64, device="cuda") for h in hs]
    for i, h in enumerate(hs):
        h.rhs_uniform(40 + i, bs[i])
    xs = [torch.zeros_like(b) for b in bs]
    mg.solve_batch(hs, bs, xs, o)
    for i in {0, len(levels) // 2, len(levels) - 1}:
        # mg_solve runs these counts as separate launches of its own
        x = torch.zeros_like(bs[i])
        hs[i].solve(bs[i], x, o)
        torch.cuda.synchronize()
        assert torch.equal(x, xs[i]), i
    for h in hs:
        h.close()
    ctx.close()
