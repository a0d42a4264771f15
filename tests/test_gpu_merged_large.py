"""GPU: the merged pass of FP64 solves at the two largest levels, where its
vectors reach (L = 14: pass) 2^31 bytes and unwanted stores and loads must still
fall outside every buffer: solves equal their cycles one by one, bit for bit."""
import pytest
import torch

import paper_0904_4152_amd as mg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("level,sides", [(13, 5), (14, 15)])
def test_fp64_chain_is_its_cycles(level, sides):
    ctx = mg.Context(0)
    h = mg.Hierarchy(ctx, level, jitter=0.2, seed=7, dirichlet_sides=sides)
    b = torch.zeros(h.n, dtype=torch.float64, device="cuda")
    h.rhs_uniform(11, b)
    start = torch.randn(h.n, dtype=torch.float64, device="cuda",
                        generator=torch.Generator(device="cuda").manual_seed(4))
    want, got = start.clone(), torch.empty_like(start)
    for cycles in (1, 2, 3):
        h.vcycle(level, b, want, fused=True)
        got.copy_(start)
        h.solve(b, got, mg.default_opts(precision=0, fixed_cycles=cycles))
        torch.cuda.synchronize()
        assert torch.equal(got, want), cycles
    h.close()
    ctx.close()
