"""Preconditioned CG with p.q taken in the product's pass: the true residual
meets the tolerance on both kinds of product tile and their edges, and neither
the first direction nor b depends on what an earlier solve left behind."""
import pytest
import torch

import paper_0904_4152_amd as mg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("level", [2, 5, 8, 9, 11])
def test_true_residual_and_leftovers(level, precision):
    ctx = mg.Context(0)
    h = mg.Hierarchy(ctx, level, jitter=0.2, seed=7)
    b = torch.zeros(h.n, dtype=torch.float64, device="cuda")
    h.rhs_uniform(11, b)
    o = mg.default_opts(precision=precision, krylov=1, rel_tol=1e-9)
    x = torch.zeros_like(b)
    st = h.solve(b, x, o)
    # the recurrence residual met 1e-9; FP64 rounding of a few steps separates
    # the true one from it by far less than a thousandth of that
    assert st.rel_res <= 1.001e-9
    d = torch.empty_like(b)
    h.defect(level, b, x, d)
    torch.cuda.synchronize()
    assert abs(float(d.norm() / b.norm()) - st.rel_res) <= 1e-3 * st.rel_res + 1e-15
    for krylov in (1, 0):
        bad = torch.full_like(b, float("nan"))
        s2 = h.solve(b, bad, mg.default_opts(precision=precision, krylov=krylov),
                     raise_on_error=False)
        assert s2.status == mg.MG_ERR_NUMERIC
        again = torch.zeros_like(b)
        s3 = h.solve(b, again, o)
        assert s3.cycles == st.cycles and torch.equal(again, x)
    h.close()
    ctx.close()
