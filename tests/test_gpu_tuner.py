"""GPU: tiles the single-problem autotuner leaves in force, and those its saved
rows install, are not slower than the rules' in either type."""
import pytest
import torch

import paper_0904_4152_amd as mg

pytestmark = pytest.mark.gpu


def pair_us(h, level, dtype):
    """A pre and a post pass (shortest of eight runs of 30 pairs)."""
    v = [torch.zeros(h.level_size(level), dtype=dtype, device="cuda") for _ in range(3)]
    c = torch.zeros(h.level_size(level - 1), dtype=dtype, device="cuda")
    a, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = 1e9
    for _ in range(8):
        a.record()
        for _ in range(30):
            h.pre_smooth(level, v[0], v[1], v[2], c)
            h.post_smooth(level, v[0], v[2], c, v[1])
        e.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(e) * 1e3 / 30)
    return best


def test_tuned_tiles_are_not_slower(tmp_path):
    ctx = mg.Context(0)
    h = mg.Hierarchy(ctx, 12, jitter=0.2, seed=7)
    # levels whose passes are longer than their launches
    kinds = [(10, torch.float64), (11, torch.float32), (11, torch.float64),
             (12, torch.float32), (12, torch.float64)]
    mg.batch_clear_tiles()
    try:
        rows = h.autotune(reps=5)
        mg.save_tiles(rows, str(tmp_path / "tiles.json"))
        mg.batch_clear_tiles()
        rule = [pair_us(h, *k) for k in kinds]
        h.autotune(reps=5)
        tuned = [pair_us(h, *k) for k in kinds]
        mg.batch_clear_tiles()
        mg.load_tiles(str(tmp_path / "tiles.json"))
        loaded = [pair_us(h, *k) for k in kinds]
    finally:
        mg.batch_clear_tiles()
    print([(k[0], str(k[1])) + t for k, t in zip(kinds, zip(rule, tuned, loaded))], rows)
    # FP32 tiles in FP64 passes: 1.10 at L = 10; a losing row installed from the
    # file: 1.18 in FP32 at L = 11.  Runs of one tile differ by 2 %.
    for k, r, t, l in zip(kinds, rule, tuned, loaded):
        assert t < 1.06 * r and l < 1.06 * r, (k, r, t, l)
    h.close()
    ctx.close()
