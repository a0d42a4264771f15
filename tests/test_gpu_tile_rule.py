"""GPU: the tile rule of the single-problem fused passes (block tiles up to
513 nodes per side, marching tiles from a cost model above) gives the bits of
plain marching tiles in both types, on either side of the line."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

import paper_0904_4152_amd as mg  # noqa: E402


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("L", [2, 6, 8, 9, 10, 11])
def test_rule_equals_marching_tiles(L, dtype):
    ctx = mg.Context(0)
    h = mg.Hierarchy(ctx, L, jitter=0.2, seed=5, dirichlet_sides=13)
    b64 = torch.zeros(h.n, dtype=torch.float64, device="cuda")
    h.rhs_uniform(9, b64)
    b = b64.to(dtype)
    x = (0.1 * b64.roll(3) * (b64 != 0)).to(dtype)
    xc = torch.randn(h.level_size(L - 1), dtype=torch.float64, device="cuda").to(dtype)

    def passes():
        out = []
        for zero in (False, True):
            x2 = torch.empty_like(b)
            bc = torch.empty_like(xc)
            h.pre_smooth(L, b, x, x2, bc, x_zero=zero)
            out += [x2, bc]
        y = torch.empty_like(b)
        norm = h.post_smooth(L, b, x, xc, y, norm=True)
        z = torch.empty_like(b)
        h.post_smooth(L, b, x, xc, z)
        torch.cuda.synchronize()
        return [t.cpu().numpy() for t in out + [y, z]] + [np.array([norm])]

    mg.batch_clear_tiles()
    try:
        rule = passes()
        mg.batch_set_tiles([{"level": L, "problems": 1, "tile_rows": 8, "row_waves": 2}])
        march = passes()
    finally:
        mg.batch_clear_tiles()
    for a, c in zip(rule, march):
        assert np.array_equal(a, c)
    h.close()
    ctx.close()
