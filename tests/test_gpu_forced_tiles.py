"""GPU: MG_FUSED_BT and MG_FUSED_WAVES force the tiles of passes without a tuned
entry, on every level and in the batch, and change no bit."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = """
import hashlib
import torch
import paper_0904_4152_amd as mg
ctx = mg.Context(0)
digest = hashlib.sha256()
us = []
for level in (7, 9):
    h = mg.Hierarchy(ctx, level, jitter=0.2, seed=7)
    b = torch.zeros(h.n, dtype=torch.float64, device="cuda")
    h.rhs_uniform(11, b)
    x, y = torch.zeros_like(b), torch.zeros_like(b)
    h.solve(b, x, mg.default_opts(precision=1, rel_tol=1e-6))
    h.solve(b, y, mg.default_opts(precision=0, rel_tol=1e-6))
    z = torch.zeros_like(b)
    mg.solve_batch([h], [b], [z], mg.default_opts(precision=1, rel_tol=1e-6))
    c = torch.zeros(h.level_size(level - 1), dtype=torch.float64, device="cuda")
    t = torch.zeros_like(b)
    start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    best = 1e9
    for _ in range(5):
        start.record()
        for _ in range(20):
            h.pre_smooth(level, b, x, t, c)
        end.record()
        torch.cuda.synchronize()
        best = min(best, start.elapsed_time(end) * 1e3 / 20)
    us.append(best)
    for v in (x, y, z, t, c):
        digest.update(v.cpu().numpy().tobytes())
    h.close()
print("RESULT", digest.hexdigest(), *us)
"""


def run(**env):
    r = subprocess.run([sys.executable, "-c", PROGRAM], capture_output=True, text=True,
                       timeout=100, cwd=ROOT, env=dict(os.environ, **env))
    assert r.returncode == 0, r.stderr[-2000:]
    line = next(l for l in r.stdout.splitlines() if l.startswith("RESULT")).split()
    return line[1], [float(v) for v in line[2:]]


def test_forced_marching_tiles():
    bits, us = run()
    # marching tiles of 64 rows take a step per row, block tiles a few steps
    # in all: 30 us against 4
    for env in ({"MG_FUSED_WAVES": "1"}, {"MG_FUSED_BT": "256", "MG_FUSED_WAVES": "1"}):
        forced_bits, forced_us = run(**env)
        assert forced_bits == bits
        for f, u in zip(forced_us, us):
            assert f > 2 * u, (env, forced_us, us)
