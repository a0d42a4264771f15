"""A V(2,2) cycle's post pass merged with the next cycle's pre pass: the chained
cycles of a solve against the same cycles one by one, exact equality (the same
arithmetic per node)."""
import pytest
import torch

import paper_0904_4152_amd as mg

pytestmark = pytest.mark.gpu


def problem(level, sides, coarse=1):
    ctx = mg.Context(0)
    h = mg.Hierarchy(ctx, level, coarse_level=coarse, jitter=0.2, seed=7, dirichlet_sides=sides)
    b = torch.zeros(h.n, dtype=torch.float64, device="cuda")
    h.rhs_uniform(11, b)
    return ctx, h, b


@pytest.mark.parametrize("level,sides,coarse", [(3, 15, 2), (6, 5, 1), (8, 15, 2), (9, 14, 1), (10, 15, 1),
                                                (11, 15, 1), (11, 5, 2), (12, 14, 2)])
@pytest.mark.parametrize("cycles", [1, 2, 5])
def test_fp64_chain_is_its_cycles(level, sides, coarse, cycles):
    ctx, h, b = problem(level, sides, coarse)
    start = torch.randn(h.n, dtype=torch.float64, device="cuda",
                        generator=torch.Generator(device="cuda").manual_seed(4))
    want = start.clone()
    for _ in range(cycles):
        h.vcycle(level, b, want, fused=True)
    for graph in (0, 1):
        got = start.clone()
        h.solve(b, got, mg.default_opts(precision=0, fixed_cycles=cycles, use_graph=graph))
        torch.cuda.synchronize()
        assert torch.equal(got, want)
        # stopped by the tolerance (a hair above the last residual: r <= (r / |b|) |b|
        # may fail by rounding): the chain ends with a merged pass
        again = start.clone()
        st = h.solve(b, again, mg.default_opts(precision=0, max_cycles=cycles, rel_tol=0.0,
                                               use_graph=graph), raise_on_error=False)
        assert st.cycles == cycles and torch.equal(again, want)
        loose = start.clone()
        st = h.solve(b, loose, mg.default_opts(precision=0, rel_tol=st.rel_res * (1 + 1e-9),
                                               use_graph=graph))
        assert st.cycles == cycles and torch.equal(loose, want)
    h.close()
    ctx.close()


@pytest.mark.parametrize("level,sides,coarse", [(6, 15, 1), (8, 5, 2), (9, 15, 1), (10, 14, 2),
                                                (11, 15, 1), (12, 15, 1), (12, 5, 2)])
def test_mixed_chain_is_its_cycles(level, sides, coarse):
    # a first solve queues two inner cycles and then single ones, a second the
    # number the first one took, as one chain
    ctx, h, b = problem(level, sides, coarse)
    o = mg.default_opts(precision=1, inner_reduction=1e-5, inner_max_cycles=12)
    first, second = torch.zeros_like(b), torch.zeros_like(b)
    s1 = h.solve(b, first, o)
    s2 = h.solve(b, second, o)
    assert s1.cycles > 2 * s1.outer_steps
    assert s2.cycles == s1.cycles and s2.rel_res == s1.rel_res
    assert torch.equal(first, second)
    h.close()
    ctx.close()
