"""GPU: the tile rule above its block tiles (FP64 L = 11 and up, FP32 L = 12 and
up: marching tiles from a cost model, non-temporal loads and stores where a
pass exceeds the cache) gives the bits of 8-row marching tiles."""
import pytest
import torch

from test_gpu_tile_rule import test_rule_equals_marching_tiles as rule_equals_marching_tiles

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("L", [12, 13])
def test_rule_equals_marching_tiles_on_large_levels(L, dtype):
    rule_equals_marching_tiles(L, dtype)
