"""General forward: how a row's list of blocks is walked (chunks of 64 ids, stretches of 16-key groups)."""
import pytest

from lcsa_harness import geoms, sample_rows
from paper_2510_12747_amd import workloads as wl
from test_gpu_parity import run_primed

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("d,grid,tile,topk", [
    (32, (21, 35), (4, 4), 64),          # one chunk of ids, exactly
    (64, (21, 35), (4, 4), 65),          # the 65th by itself
    (40, (21, 35), (4, 4), 150),         # three chunks, channels that end inside a 16- and a 32-channel piece
    (96, (21, 35), (2, 17), 70),         # 34 tokens: three groups a block, the last with two rows; stretches straddle chunks
    (200, (21, 35), (3, 5), 67),         # 15 tokens: one group, a row short
    (32, (39, 60), (9, 16), 70),         # 144 tokens: more queries than four wavefronts take at a time, the chunks once more for the rest
])
def test_rows_of_more_than_64_blocks(dtype, d, grid, tile, topk):
    w = wl.with_overrides(wl.WORKLOADS["tiny"], name=f"walk-{dtype}-{d}-{topk}", dtype=dtype, heads=2, head_dim=d, grid_h=grid[0], grid_w=grid[1],
                          tile_h=tile[0], tile_w=tile[1], radius=-1, topk=topk)
    _, og = geoms(w)
    run_primed(w, rows=sample_rows(og, 40), check_lse=True)
