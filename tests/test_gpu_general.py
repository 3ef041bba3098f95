"""General kernels: how a row's list of blocks is walked (chunks of 64 ids, stretches of 16-key groups), appends of many tiles."""
import pytest

from lcsa_harness import geoms, sample_rows
from paper_2510_12747_amd import workloads as wl
from test_gpu_backward import run_backward
from test_gpu_parity import F32_MAX, F32_MEAN, run_primed

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


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("heads,grid", [(3, (32, 32)), (3, (33, 32)), (7, (33, 33))])
def test_appends_of_192_tiles_and_more(dtype, heads, grid):
    """192 tiles a launch: a workgroup each; 216 and 1134: four to a workgroup, the last with two.  Three appends
    fill the cache, a fourth goes round the ring; the step's selection and attention read every tile of it."""
    w = wl.with_overrides(wl.WORKLOADS["tiny"], name=f"append-{dtype}-{heads}x{grid}", dtype=dtype, heads=heads, head_dim=64, grid_h=grid[0], grid_w=grid[1],
                          tile_h=4, tile_w=8 if heads == 3 else 4, radius=-1, topk=9)
    p, r = run_primed(w)
    for _ in range(3):
        q, qd = p.feed()
    p.check_pooled_k()
    tol = dict(max_abs=F32_MAX, mean_abs=F32_MEAN) if dtype == "fp32" else {}
    p.step(q, qd, **tol)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("heads,d,grid,tile,topk", [
    (1, 32, (10, 14), (4, 4), 8),        # two groups a wavefront: one stretch held
    (2, 32, (10, 14), (4, 4), 9),        # three, of which the others have two: two stretches
    (1, 32, (10, 14), (4, 4), 17),       # five: walked twice
    (5, 24, (37, 61), (4, 4), 16),       # held rows, but 1600 of them: walked twice
    (1, 64, (16, 24), (2, 8), 80),       # more than 64 ids, pieces that are whole rows of unclipped tiles
    (2, 64, (17, 23), (5, 7), 11),       # 35 tokens: pieces that are not, every extent
    (1, 96, (16, 24), (4, 8), 33),       # key side: ids searched, not listed
])
def test_backward_rows_and_pieces(dtype, heads, d, grid, tile, topk):
    w = wl.with_overrides(wl.WORKLOADS["tiny"], name=f"bwd-{dtype}-{d}-{topk}", dtype=dtype, heads=heads, head_dim=d, grid_h=grid[0], grid_w=grid[1],
                          tile_h=tile[0], tile_w=tile[1], radius=-1, topk=topk)
    run_backward(w)
