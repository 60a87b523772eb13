"""GPU: short items that a wave takes alone (four in a workgroup), in the persistent and in the tile kernel.

Batches planned for a few compute units, so that the items outnumber the workgroups; private lengths on both sides of a tile
and of the longest such item, counts that leave the last four incomplete, groups of one to sixteen rows, and lists longer
than the persistent kernel's header ring.  Bars as everywhere (gpu_helpers), float32-probability outputs in bf16 included."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

LENS = [1, 0, 16, 31, 32, 33, 64, 65, 250, 256, 257, 500, 512, 513, 17, 3, 129]

# name, (q heads, kv heads, d, block, q, kv), models, prefixes, compute units planned for
CASES = [
    ("g4", (32, 8, 128, 16, "bf16", "bf16"), 4, [700, 33, 0], 4),                 # one row tile
    ("g4_wide", (32, 8, 128, 16, "bf16", "bf16"), 8, [300, 1], 2),                # two row tiles
    ("g7_four_tiles", (28, 4, 128, 32, "bf16", "bf16"), 7, [300, 64], 1),
    ("g8_e4m3", (64, 8, 128, 16, "bf16", "fp8_e4m3"), 3, [520, 16, 40], 3),
    ("g8_two_requests", (64, 8, 128, 64, "bf16", "bf16"), 2, [90, 400, 1], 2),     # eight rows beside one row tile
    ("g1_shared_too", (8, 8, 128, 16, "bf16", "bf16"), 1, [1, 31, 32, 33, 147, 512, 513, 300, 64, 2, 90], 2),
    ("g2_e4m3_lists", (16, 8, 128, 16, "bf16", "fp8_e4m3"), 2, [40] * 30, 1),      # hundreds of items a workgroup
    ("tile_d64", (32, 8, 64, 32, "bf16", "bf16"), 4, [700, 33, 0], 2),
    ("tile_d64_wide", (16, 2, 64, 16, "bf16", "bf16"), 6, [300, 64], 1),           # G = 8, 48 rows per shared item
    ("tile_d256", (16, 4, 256, 16, "bf16", "bf16"), 5, [300, 64], 2),
    ("tile_f32_d128", (32, 8, 128, 16, "f32", "f32"), 3, [300, 64, 17], 2),
    ("tile_f32_d256", (8, 4, 256, 32, "f32", "f32"), 5, [300, 64], 1),
    ("tile_g16", (32, 2, 64, 16, "bf16", "bf16"), 3, [90, 20, 5], 1),              # sixteen rows
    ("tile_e4m3_f32", (16, 4, 64, 16, "f32", "fp8_e4m3"), 5, [90, 20], 1),
]


@pytest.mark.parametrize("spec", CASES, ids=lambda s: s[0])
def test_short_items_a_wave_each(spec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from gpu_helpers import GpuCase, check_against_oracle
    name, geo, models, prefixes, cus = spec
    n = models * len(prefixes)
    w = wl.make_workload(name, wl.Geometry(*geo), models, prefixes, [list(range(models))] * len(prefixes),
                         [LENS[i % len(LENS)] for i in range(n)], pool_factor=1.3, seed=7)
    case = GpuCase(w)
    case.replan(num_cus=cus)
    first = None
    for _ in range(2):
        case.poison_workspace()
        case.batch.decode_attention()
        check_against_oracle(case, label=name, scaled_bar=True)
        assert not torch.isnan(case.batch.workspace_views()[1]).any()          # every partial state was written
        first = case.batch.out.clone() if first is None else first
    assert torch.equal(first.view(torch.uint8), case.batch.out.view(torch.uint8))
    case.close()
