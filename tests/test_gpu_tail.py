"""GPU: the coarse tail (levels of at most 33 x 33 nodes in one launch) and the
one-sweep block passes against the same cycle composed of the library's single
operators, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

import paper_0904_4152_amd as mg  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    c = mg.Context(0)
    yield c
    c.close()


def composed_cycle(h, level, b, x, nu_pre, nu_post):
    if level == h.Lc:
        h.coarse_solve(b, x)
        return
    h.smooth(level, b, x, sweeps=nu_pre)
    d = torch.empty_like(b)
    h.defect(level, b, x, d)
    bc = torch.empty(h.level_size(level - 1), dtype=b.dtype, device=b.device)
    h.restrict(level, d, bc)
    xc = torch.zeros_like(bc)
    composed_cycle(h, level - 1, bc, xc, nu_pre, nu_post)
    h.prolong(level, xc, x)
    h.smooth(level, b, x, sweeps=nu_post)


# every (top, coarse) pair of the tail: top = L - 1 <= 5, below a finest
# level of 6 or less; sides with and without free corners; both coarse solvers
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("L,Lc", [(2, 1), (3, 1), (3, 2), (4, 1), (4, 2), (4, 3), (5, 1), (5, 2),
                                  (5, 3), (5, 4), (6, 1), (6, 2), (6, 3), (6, 4)])
@pytest.mark.parametrize("sides", [15, 1, 12])
def test_tail_equals_single_operators(ctx, L, Lc, sides, dtype):
    for cg in (0, 1):
        h = mg.Hierarchy(ctx, L, coarse_level=Lc, jitter=0.2, seed=31 + L, dirichlet_sides=sides)
        if cg:
            h.set_coarse_solver(mg.MG_COARSE_CG)
        b64 = torch.zeros(h.n, dtype=torch.float64, device="cuda")
        h.rhs_uniform(77, b64)
        b = b64.to(dtype)
        x0 = (0.01 * b64.roll(5) * (b64 != 0)).to(dtype)
        for pre, post in ((2, 2), (1, 1), (3, 0), (0, 2)):
            x = x0.clone()
            h.vcycle(L, b, x, nu_pre=pre, nu_post=post)
            y = x0.clone()
            composed_cycle(h, L, b, y, pre, post)
            torch.cuda.synchronize()
            assert np.array_equal(x.cpu().numpy(), y.cpu().numpy()), (cg, pre, post)
        h.close()


# one-sweep block passes above the tail: FP32 up to L = 11, FP64 up to L = 10;
# one side with a single sweep, the other separate kernels
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("L", [6, 7, 9, 11])
@pytest.mark.parametrize("nu", [(1, 1), (1, 3), (2, 1)])
def test_one_sweep_cycles_equal_single_operators(ctx, L, nu, dtype):
    h = mg.Hierarchy(ctx, L, jitter=0.2, seed=3, dirichlet_sides=13)
    b64 = torch.zeros(h.n, dtype=torch.float64, device="cuda")
    h.rhs_uniform(78, b64)
    b = b64.to(dtype)
    x = (0.01 * b64.roll(5) * (b64 != 0)).to(dtype)
    y = x.clone()
    h.vcycle(L, b, x, nu_pre=nu[0], nu_post=nu[1])
    composed_cycle(h, L, b, y, *nu)
    torch.cuda.synchronize()
    assert np.array_equal(x.cpu().numpy(), y.cpu().numpy())
    h.close()
