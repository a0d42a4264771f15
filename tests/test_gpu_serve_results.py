"""GPU: served solutions held past the pinned result buffers' limit (256 MiB:
seven of L = 11) are the same as those within it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

import paper_0904_4152_amd as mg  # noqa: E402


def test_results_beyond_the_pinned_limit():
    ctx = mg.Context(0)
    srv = mg.Server(ctx, slots=4, budget_bytes=16 << 30, max_level=11)
    n = ((1 << 11) + 1) ** 2
    tickets = [srv.submit(11, 1e-6, 0.1, 5, 6, keep_x=True) for _ in range(9)]
    small = srv.submit(6, 1e-8, 0.1, 7, 8, keep_x=True)
    # nothing is collected until every request has finished
    while srv.info().completed < 10:
        pass
    xs = []
    for t in tickets:
        rc, st, x = srv.poll(t, n)
        assert rc == mg.MG_OK and st.rel_res <= 1e-6
        xs.append(x)
    for x in xs[1:]:
        assert np.array_equal(x, xs[0])
    rc, _, x = srv.poll(small, 65 * 65)
    assert rc == mg.MG_OK and np.any(x)
    srv.close()
    ctx.close()
