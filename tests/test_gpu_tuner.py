"""GPU: the tiles that the single-problem autotuner's saved rows install are not
slower than the rules' in either type."""
import pytest
import torch

import paper_0904_4152_amd as mg

pytestmark = pytest.mark.gpu


def test_tuned_tiles_are_not_slower(tmp_path):
    ctx = mg.Context(0)
    h = mg.Hierarchy(ctx, 12, jitter=0.2, seed=7)
    # levels whose passes are longer than their launches
    kinds = [(10, torch.float64), (11, torch.float32), (11, torch.float64),
             (12, torch.float32), (12, torch.float64)]
    vectors = {}
    for level, dtype in kinds:
        sizes = [h.level_size(level)] * 3 + [h.level_size(level - 1)]
        vectors[level, dtype] = [torch.zeros(n, dtype=dtype, device="cuda") for n in sizes]
    a, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

    def pair_us(kind):
        u, v, w, c = vectors[kind]
        best = 1e9
        for _ in range(4):
            a.record()
            for _ in range(30):
                h.pre_smooth(kind[0], u, v, w, c)
                h.post_smooth(kind[0], u, w, c, v)
            e.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(e) * 1e3 / 30)
        return best

    path = str(tmp_path / "tiles.json")
    rule, tuned = dict.fromkeys(kinds, 1e9), dict.fromkeys(kinds, 1e9)
    try:
        mg.save_tiles(h.autotune(reps=5), path)
        for _ in range(4):  # in turn
            mg.batch_clear_tiles()
            for k in kinds:
                rule[k] = min(rule[k], pair_us(k))
            mg.load_tiles(path)
            for k in kinds:
                tuned[k] = min(tuned[k], pair_us(k))
    finally:
        mg.batch_clear_tiles()
    # FP32's fastest tile in FP64 passes: 1.10 at L = 10; the rule's loser
    # installed from the file: 1.18 in FP32 at L = 11.  Runs of one tile differ by 2 %.
    for k in kinds:
        print(k, rule[k], tuned[k])
        assert tuned[k] < 1.06 * rule[k], (k, rule[k], tuned[k])
    h.close()
    ctx.close()
