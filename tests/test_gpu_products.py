"""GPU: the band products on either side of the line between nine stored bands
(small matrices) and five bands through LDS: SpMV, defect and Jacobi sweep of
one x agree with each other, and the FP32 SpMV with the FP64 one."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

import paper_0904_4152_amd as mg  # noqa: E402


# FP32 reads nine bands up to L = 9, FP64 up to L = 8
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("L", [1, 3, 8, 9, 10, 12])
def test_products_agree(L, dtype):
    ctx = mg.Context(0)
    h = mg.Hierarchy(ctx, L, jitter=0.2, seed=12, dirichlet_sides=9)
    g = torch.Generator(device="cuda")
    g.manual_seed(L)
    x = torch.randn(h.n, generator=g, device="cuda", dtype=torch.float64).to(dtype)
    b = torch.randn(h.n, generator=g, device="cuda", dtype=torch.float64).to(dtype)
    y, d, z = (torch.empty_like(x) for _ in range(3))
    h.spmv(L, x, y)
    h.defect(L, b, x, d)
    h.jacobi(L, b, x, z, omega=0.75)
    torch.cuda.synchronize()
    assert torch.equal(d, b - y)
    diag = torch.from_numpy(h.bands(L)[4]).cuda()
    if dtype == torch.float64:
        assert torch.equal(z, x + (0.75 * (b - y)) / diag)
        # the FP32 bands and x are within u32 of the FP64 ones, and the nine
        # terms and their sum add at most nine roundings more
        x32, y32 = x.float(), torch.empty_like(x, dtype=torch.float32)
        h.spmv(L, x32, y32)
        ab = torch.from_numpy(abs(h.bands(L)).max(0)).cuda() * 9 * x.abs().max()
        assert bool(((y32.double() - y).abs() <= 12 * 2.0 ** -24 * ab + 1e-30).all())
    else:
        # reciprocal within one ulp, one product, one fused add
        step = (0.75 * (b - y)) / diag.float()
        err = (z.double() - (x.double() + step.double())).abs()
        assert bool((err <= 4 * 2.0 ** -24 * (step.abs() + x.abs()).double()).all())
    h.close()
    ctx.close()
