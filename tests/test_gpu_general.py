"""General kernels: how a row's list of blocks is walked (chunks of 64 ids, stretches of 16-key groups), appends of many tiles, weights
and values at the ends of their ranges."""
import math

import pytest
import torch

from lcsa_harness import geoms, sample_rows
from paper_2510_12747_amd import binding as B
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
    (64, (39, 61), (4, 4), 70),          # 640 rows, more than two a unit: keys requested in their turn, in float
    (96, (27, 45), (4, 4), 66),          # 336 rows, more than one a unit: the same
    (128, (21, 35), (4, 8), 66),         # 32-token blocks: a stretch ahead, in bf16 too
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
    (1, 136, (10, 20), (4, 9), 7),       # beyond 128 channels, where rows and columns are loaded in turn: 36 tokens, three pieces
    (2, 200, (9, 17), (4, 8), 5),        # two, all four extents
    (1, 256, (8, 24), (8, 8), 6),        # four, all channels
])
def test_backward_rows_and_pieces(dtype, heads, d, grid, tile, topk):
    w = wl.with_overrides(wl.WORKLOADS["tiny"], name=f"bwd-{dtype}-{d}-{topk}", dtype=dtype, heads=heads, head_dim=d, grid_h=grid[0], grid_w=grid[1],
                          tile_h=tile[0], tile_w=tile[1], radius=-1, topk=topk)
    run_backward(w)


def whole_numbers(*shape, seed):
    return torch.randint(1, 4, shape, generator=torch.Generator().manual_seed(seed)).float()


def backward_in(dtype, d, tile, q, k, v, d_o, lse=None, scale=0.0):
    """Gradients of two frames of 2 x 2 blocks of `tile`, every block kept, in the kernels for tensors of that type."""
    g = B.Geom(1, d, 2 * tile[0], 2 * tile[1], *tile, 2, 2, -1, -1, 8, dtype=B.LCSA_BF16 if dtype == torch.bfloat16 else B.LCSA_F32)
    q, k, v, d_o = (x.to("cuda", dtype) for x in (q, k, v, d_o))
    cache = B.lcsa_cache_init(g)
    B.lcsa_kv_cache_append(cache, k, v, 2)
    _, sel_idx, sel_cnt, _ = B.lcsa_pool_select_blocks(g, q, cache)
    assert (sel_cnt == 8).all()
    if lse is None:
        lse = torch.empty(q.shape[0], 1, device="cuda")
        B.lcsa_sparse_attn_fwd(g, q, cache, sel_idx, sel_cnt, lse=lse, scale=scale)
    return B.lcsa_sparse_attn_bwd(g, q, k, v, 2, sel_idx, sel_cnt, d_o, lse, scale=scale)


def same(got, want, rel, cancels=()):
    """The same infinities and NaN in the same places, and everywhere else within rel of the 2-norm, but where the sums cancel."""
    for name, a, b in zip(("d_q", "d_k", "d_v", "delta"), got, want):
        assert (a.isnan() == b.isnan()).all() and (a.isinf() == b.isinf()).all(), name
        assert (a[a.isinf()] == b[b.isinf()]).all(), name
        if name in cancels:
            continue
        a, b = (torch.where(x.isfinite(), x, 0).double() for x in (a, b))
        assert (a - b).norm() <= rel * b.norm(), (name, float((a - b).norm() / b.norm()))


@pytest.mark.parametrize("d,tile", [(32, (2, 8)), (32, (4, 8)), (64, (4, 8)), (96, (5, 7)), (128, (4, 12)), (32, (9, 16))])      # the last: three rounds over a block
def test_backward_weights_that_bf16_does_not_hold(d, tile):
    """bf16 rows meet float weights in pieces of bf16; weights beyond what those hold give what the float kernels give for the same
    numbers, to the order of float sums of some 2^10 terms (1e-6).  With all keys alike d_q is the sum of a row's u, which is
    zero but for rounding, where it is finite."""
    n = 2 * 2 * tile[0] * 2 * tile[1]
    q, k, v, d_o = (whole_numbers(n, 1, d, seed=s) for s in range(4))
    q[..., 1::2] = -q[..., ::2]
    k[:] = 1                                                 # every score is zero
    large, short = torch.zeros(n, 1, d), torch.full((n, 1), -127.9988 * math.log(2.0), device="cuda")
    large[5, 0, 0] = 2.0 ** 120
    v_large = v.clone()
    v_large[::2, :, 0] = 2.0 ** 7
    normal = [torch.randn(n, 1, d, generator=torch.Generator().manual_seed(7 + s)).bfloat16().float() for s in range(4)]
    cases = [
        ("u = p (t - D) scale is infinite, and d_k with it", [False, True, False], (q, k, v_large, d_o + large, None, 2.0 ** 9)),
        ("p rounds to an infinity in bf16, u is one", [True, True, False], (q, k, v, d_o * 2.0 ** -20, short, 0.0)),
        ("the last bits of u lie among the subnormals", [False] * 3, (*normal[:3], normal[3] * 2.0 ** -112, None, 0.0)),
    ]
    for name, infinite, case in cases:
        got, want = (backward_in(dtype, d, tile, *case) for dtype in (torch.bfloat16, torch.float32))
        assert [bool(x.isinf().any()) for x in want[:3]] == infinite, name
        same(got, want, 1e-6, cancels=() if not any(infinite) else ("d_q",))


@pytest.mark.parametrize("d,tile", [(64, (4, 8)), (32, (4, 4))])
def test_forward_small_weights_of_large_values(d, tile):
    """One key whose weight is 1.23 x 2^-124 has values of about 2^127, the others none: the output is that product, rounded to bf16 once."""
    n = 2 * 2 * tile[0] * 2 * tile[1]
    g = B.Geom(1, d, 2 * tile[0], 2 * tile[1], *tile, 2, 2, -1, -1, 8)
    q, k, v = torch.ones(n, 1, d), torch.ones(n, 1, d), torch.zeros(n, 1, d)
    k[3] = -1
    v[3] = 2.0 ** 126 * (1 + torch.arange(d) / 128.0)
    scale = 123.7 * math.log(2.0) / (2 * d)
    q, k, v = (x.to("cuda", torch.bfloat16) for x in (q, k, v))
    cache = B.lcsa_cache_init(g)
    B.lcsa_kv_cache_append(cache, k, v, 2)
    _, sel_idx, sel_cnt, _ = B.lcsa_pool_select_blocks(g, q, cache)
    o = B.lcsa_sparse_attn_fwd(g, q, cache, sel_idx, sel_cnt, scale=scale).double()
    p = torch.softmax((q.double() * scale).permute(1, 0, 2) @ k.double().permute(1, 2, 0).contiguous(), dim=-1)
    want = (p @ v.double().permute(1, 0, 2).contiguous()).permute(1, 0, 2)
    half_unit = 2.0 ** (want.abs().log2().floor() - 8)       # of bf16; and the exponent's float rounding, 124 x 2^-24 with that of the scale
    assert ((o - want).abs() <= half_unit + 2e-5 * want.abs()).all(), float(((o - want).abs() / half_unit).max())


@pytest.mark.parametrize("d,tile", [(32, (2, 8)), (64, (4, 8)), (96, (5, 7))])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
def test_values_that_are_not_finite(d, tile, value):
    """One of them in an even or an odd channel (either half of a word) of V, dO, K or Q of bf16 tensors: what the float kernels make of
    the same numbers, and where it is V's or dO's, no other channel of o or d_v changes."""
    n = 2 * 2 * tile[0] * 2 * tile[1]
    normal = [torch.randn(n, 1, d, generator=torch.Generator().manual_seed(20 + s)).bfloat16().float() for s in range(4)]
    plain = backward_in(torch.bfloat16, d, tile, *normal)
    for which in (2, 3, 1, 0):                               # of q, k, v, d_o
        for channel in (6, 9):
            inputs = [x.clone() for x in normal]
            inputs[which][17, 0, channel] = value
            got, want = (backward_in(dtype, d, tile, *inputs) for dtype in (torch.bfloat16, torch.float32))
            assert not all(x.isfinite().all() for x in want)
            same(got, want, 2e-6)
            if which == 3:
                others = [c for c in range(d) if c != channel]
                assert torch.equal(got[2][..., others], plain[2][..., others]) and not got[2][..., channel].isfinite().any()


@pytest.mark.parametrize("d,tile", [(32, (4, 4)), (64, (4, 8)), (96, (5, 7)), (128, (8, 8))])
def test_forward_values_that_are_not_finite(d, tile):
    n = 2 * 2 * tile[0] * 2 * tile[1]
    g = B.Geom(1, d, 2 * tile[0], 2 * tile[1], *tile, 2, 2, -1, -1, 8)
    q, k, v = (torch.randn(n, 1, d, generator=torch.Generator().manual_seed(30 + s)).to("cuda", torch.bfloat16) for s in range(3))

    def forward(v):
        cache = B.lcsa_cache_init(g)
        B.lcsa_kv_cache_append(cache, k, v, 2)
        _, sel_idx, sel_cnt, _ = B.lcsa_pool_select_blocks(g, q, cache)
        assert (sel_cnt == 8).all()
        return B.lcsa_sparse_attn_fwd(g, q, cache, sel_idx, sel_cnt)

    plain, planted = forward(v), v.clone()
    values = {6: float("inf"), 9: float("inf"), 10: float("-inf"), 13: float("-inf"), 16: float("nan"), 21: float("nan")}
    for i, (channel, value) in enumerate(values.items()):
        planted[5 + 7 * i, 0, channel] = value
    planted[3, 0, 24], planted[50, 0, 24] = float("inf"), float("-inf")      # of both signs: NaN
    got = forward(planted)
    for channel, value in {**values, 24: float("nan")}.items():
        assert (got[..., channel].isnan() if value != value else got[..., channel] == value).all(), channel
    others = [c for c in range(d) if c not in values and c != 24]
    assert torch.equal(got[..., others], plain[..., others])
