// Block-sparse attention, general path: any head_dim <= 256, any block shape, f32 or bf16 storage, float products on the
// matrix cores (lcsa_fp32_mma.h).  Used where the shape constraints of the bf16 / d = 128 kernel do not hold.
//
// One workgroup per (head, query block), four wavefronts.  A wavefront owns 16 QS query rows (columns of S^T = K Q^T, so
// that a query's statistics live in four lanes and S^T is the operand of O^T += V^T P^T as it stands) and walks the
// 16-key groups of the selected blocks, GI groups at a time.  Blocks with fewer query rows than four wavefronts take
// split the key groups instead: each wavefront keeps a softmax of its own over every (4 / ways)-th stretch of GI groups,
// and the partial results meet in LDS at the end.  No LDS and no barrier otherwise.
//
// What bounds it: latency.  A row is a chain of ids -> keys -> scores -> values, and a wavefront of a short row goes through
// it once or twice, so the kernel spends what it can on having loads in flight: ids are turned into tile addresses 64 at a time,
// one per lane, before the walk, the keys of the next stretch are requested as soon as the scores of this one are formed where that
// pays (launch()), and bf16 weights go through bf16 products (ColGroups), which leaves registers for three wavefronts a SIMD.  8 heads,
// d = 64, bf16, 32-token blocks, k = 16 on a 24 x 44 grid (576 workgroups): 32.1 -> 16.2 us.  36 rows of 20 64-token blocks, float, d = 32
// 49.7 -> 34.8, d = 64 78.4 -> 57.6 us; rows of one stretch, d = 64: 60 of 4 groups, 32-token blocks, 8.3 -> 8.1,
// 560 of 7 groups, 16-token blocks, 10.7 -> 10.0.
#include "lcsa_fp32_mma.h"
#include <type_traits>

namespace lcsa {
namespace {

using namespace fp32mma;

constexpr int kThreads = 256;

// Wavefronts a SIMD, where the operands of GI groups leave room for more than one.
template <typename T, int NT, int QS, int GI> constexpr int kWaves = sizeof(T) == 2 ? (NT * QS <= 12 ? 2 : 1) : (NT * QS == 2 ? 4 : NT < 16 && NT * QS * GI <= 16 ? 2 : 1);

// AHEAD: the keys of the next stretch are requested before the weights of this one are formed, else when their turn comes.
template <typename T, int NT, int QS, int GI, bool AHEAD>
__global__ __launch_bounds__(kThreads, (kWaves<T, NT, QS, GI>)) void attn_generic_kernel(
    KGeom g, KCache c, const T *__restrict__ q, int64_t q_st, int64_t q_sh,
    const int32_t *__restrict__ sel_idx, const int32_t *__restrict__ sel_cnt,
    T *__restrict__ o, int64_t o_st, int64_t o_sh, float *__restrict__ lse, float scale_log2, int per_xcd) {
    __shared__ float part_ml[4][QS][2][16];                  // [wavefront][piece][max, sum][query]
    __shared__ f32x4 part_o[4][QS][NT][64];
    // XCD-aware order: an XCD (workgroup id mod 8) gets a contiguous run of (head, query block) items
    const int n_qb = g.q_groups * g.nb;
    const int item = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (item >= n_qb * g.heads) return;
    const int head = g.by_n_qb(item), qb = item - head * n_qb;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = lane & 15, g4 = lane >> 4;
    const int fq = g.by_nb(qb), tile = qb - fq * g.nb, by = g.by_tx(tile), bx = tile - by * g.tx;
    const BlockTokens qt(g, min(g.th, g.H - by * g.th), min(g.tw, g.W - bx * g.tw));
    const int ways = row_ways(qt.n_valid, 16 * QS), splits = 4 / ways;
    const int qw = wave / splits, ks = wave - qw * splits;

    const int64_t row = (int64_t)head * n_qb + qb;
    const int32_t *sel = sel_idx + row * g.topk;
    const int start = ring_start(c, g);                      // requested together with the count and the first ids
    const int32_t first_id = lane < g.topk ? sel[lane] : 0;
    const int cnt = min(max(sel_cnt[row], 0), g.topk);       // a row holds at most topk ids
    const int per_block = (g.bt + 15) >> 4, total = cnt * per_block;      // 16-key groups
    // f / per_block: exact while f * per_block < 2^32 (8192 blocks of 64 groups reach 2^25)
    const uint32_t m_block = per_block == 1 ? 0 : 0xffffffffu / (uint32_t)per_block + 1u;
    const uint32_t row_bytes = g.d * sizeof(T);
    const char *k_head = (const char *)c.k + (int64_t)head * g.cap * g.nb * g.bt * row_bytes;
    const char *v_head = (const char *)c.v + (int64_t)head * g.cap * g.nb * g.bt * row_bytes;
    const uint32_t k_lane = RowFrag<T, NT>::lane_offset(g4), v_lane = ColGroups<T, NT, GI>::lane_offset(m);

    // Selected blocks of the row, 64 at a time, one per lane: tile index and valid keys.  The divisions take more
    // instructions than the products of a group.
    int chunk = 0, chunk_tile = 0, chunk_keys = 0;
    auto take_chunk = [&](int32_t id) {
        const int kb = min(max(id, 0), c.valid * g.nb - 1);  // ids outside the cache must not become wild addresses
        const int grp = g.by_nb(kb), kt = kb - grp * g.nb, kby = g.by_tx(kt), kbx = kt - kby * g.tx;
        chunk_tile = cache_slot(c, g, start, head, grp) * g.nb + kt;
        chunk_keys = g.tt * min(g.th, g.H - kby * g.th) * min(g.tw, g.W - kbx * g.tw);
    };
    take_chunk(first_id);
    auto block_of = [&](int f) { return per_block == 1 ? f : (int)__umulhi((uint32_t)f, m_block); };

    // more than one round only where four wavefronts do not cover the block, and then splits == 1
    for (int q0 = qw * 16 * QS; q0 < qt.n_valid || splits > 1; q0 += ways * 16 * QS) {
        // Groups i0 .. i0 + GI - 1: values requested beside their keys, or, AHEAD, when these arrive, and then the keys of the next ones as
        // soon as the products with the present ones are issued.
        RowFrag<T, NT> kf[GI];
        ColGroups<T, NT, GI> vf;
        int64_t at[GI];                                      // of the group's first row in the head's tiles
        int left[GI], present[GI];                           // valid keys of the group, rows of it that the tile has; <= 0: none
        auto request_keys = [&](int i0) {
            const int b_last = block_of(min(i0 + GI - 1, total - 1));
            if (b_last >= chunk + 64) {                      // uniform
                chunk = block_of(i0);
                take_chunk(chunk + lane < cnt ? sel[chunk + lane] : 0);
            }
#pragma unroll
            for (int i = 0; i < GI; ++i) {
                const int f = min(i0 + i, total - 1), b = block_of(f), first = (f - b * per_block) * 16;
                at[i] = ((int64_t)__builtin_amdgcn_readlane(chunk_tile, b - chunk) * g.bt + first) * row_bytes;
                left[i] = i0 + i < total ? __builtin_amdgcn_readlane(chunk_keys, b - chunk) - first : 0;
                present[i] = i0 + i < total ? g.bt - first : 0;
                // rows beyond the block's bt (bt not a multiple of 16) repeat its last key, which is masked
                kf[i].load_at(k_head + at[i], min(m * row_bytes, (g.bt - 1 - first) * row_bytes) + k_lane);
            }
        };
        if (chunk != 0) { chunk = 0; take_chunk(sel[min(lane, g.topk - 1)]); }      // left by a round before this one
        int i0 = ks * GI;
        if (AHEAD && i0 < total) request_keys(i0);

        RowFrag<T, NT> qf[QS];
        int token[QS];                                       // ~: a padding row's
#pragma unroll
        for (int s = 0; s < QS; ++s) {
            int ft, r, cc;
            const bool there = qt.at(q0 + 16 * s + m, ft, r, cc);
            if (!there) ft = r = cc = 0;                     // padding rows compute on the block's first token and store nothing
            const int64_t t = raster_token(g, fq, ft, by * g.th + r, bx * g.tw + cc);
            token[s] = there ? (int)t : ~(int)t;
            qf[s].load(q + t * q_st + (int64_t)head * q_sh, g.d, g4);
        }
        f32x4 oacc[QS][NT];
        float mx[QS], l[QS];
#pragma unroll
        for (int s = 0; s < QS; ++s) {
            mx[s] = -__builtin_inff();
            l[s] = 0.f;
#pragma unroll
            for (int t = 0; t < NT; ++t) oacc[s][t] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        for (; i0 < total; i0 += splits * GI) {
            if (!AHEAD) request_keys(i0);
            f32x4 sc[QS][GI];
            int rows[GI];
#pragma unroll
            for (int i = 0; i < GI; ++i) {
                rows[i] = present[i];
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    vf.load_at(i, r, v_head + at[i], min((4 * g4 + r) * row_bytes, max(present[i] - 1, 0) * row_bytes) + v_lane);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < GI; ++i) {
                kf[i].clear_beyond(g.d, g4);
#pragma unroll
                for (int s = 0; s < QS; ++s) {
                    sc[s][i] = RowFrag<T, NT>::mma(kf[i], qf[s], f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
                    for (int r = 0; r < 4; ++r) sc[s][i][r] = 4 * g4 + r < left[i] ? sc[s][i][r] * scale_log2 : -__builtin_inff();
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            if (AHEAD && i0 + splits * GI < total) request_keys(i0 + splits * GI);
#pragma unroll
            for (int s = 0; s < QS; ++s) {
                float mnew = mx[s];
#pragma unroll
                for (int i = 0; i < GI; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) mnew = fmaxf(mnew, sc[s][i][r]);
                mnew = column_max(mnew);
                const float ref = mnew == -__builtin_inff() ? 0.f : mnew;     // nothing but padding so far
                if (__ballot(mnew != mx[s])) {
                    const float alpha = __builtin_amdgcn_exp2f(mx[s] - ref);
                    l[s] *= alpha;
#pragma unroll
                    for (int t = 0; t < NT; ++t) oacc[s][t] *= alpha;
                    mx[s] = mnew;
                }
#pragma unroll
                for (int i = 0; i < GI; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        sc[s][i][r] = __builtin_amdgcn_exp2f(sc[s][i][r] - ref);
                        l[s] += sc[s][i][r];
                    }
            }
#pragma unroll
            for (int i = 0; i < GI; ++i) vf.keep(i, rows[i], g4);
            vf.clear_beyond(g.d, m);
            vf.mma(sc, oacc);
        }
#pragma unroll
        for (int s = 0; s < QS; ++s) l[s] = column_sum(l[s]);

        if (splits > 1) {                                    // uniform over the workgroup
#pragma unroll
            for (int s = 0; s < QS; ++s) {
                if (g4 == 0) { part_ml[wave][s][0][m] = mx[s]; part_ml[wave][s][1][m] = l[s]; }
#pragma unroll
                for (int t = 0; t < NT; ++t) part_o[wave][s][t][lane] = oacc[s][t];
            }
            __syncthreads();
            if (ks != 0) return;
#pragma unroll
            for (int s = 0; s < QS; ++s) {
                float all = mx[s];
                for (int w = 1; w < splits; ++w) all = fmaxf(all, part_ml[wave + w][s][0][m]);
                const float ref = all == -__builtin_inff() ? 0.f : all;
                const float own = __builtin_amdgcn_exp2f(mx[s] - ref);
                l[s] *= own;
#pragma unroll
                for (int t = 0; t < NT; ++t) oacc[s][t] *= own;
                for (int w = 1; w < splits; ++w) {
                    const float theirs = __builtin_amdgcn_exp2f(part_ml[wave + w][s][0][m] - ref);
                    l[s] = fmaf(part_ml[wave + w][s][1][m], theirs, l[s]);
#pragma unroll
                    for (int t = 0; t < NT; ++t) oacc[s][t] += part_o[wave + w][s][t][lane] * theirs;
                }
                mx[s] = all;
            }
        }
#pragma unroll
        for (int s = 0; s < QS; ++s) {
            if (token[s] < 0) continue;
            const float inv = l[s] > 0.f ? 1.f / l[s] : 0.f;
#pragma unroll
            for (int p = 0; p < NT / 2; ++p) {
                float x[8];
                channels_of(oacc[s], p, x);
#pragma unroll
                for (int i = 0; i < 8; ++i) x[i] *= inv;
                store8(o + (int64_t)token[s] * o_st + (int64_t)head * o_sh, 32 * p + 8 * g4, g.d, x);
            }
            if (lse && g4 == 0) lse[(int64_t)token[s] * g.heads + head] = l[s] > 0.f ? (mx[s] + __builtin_amdgcn_logf(l[s])) * kLn2 : -__builtin_inff();
        }
        if (splits > 1) return;
    }
}

// 16-key groups of a full row that a wavefront of rows_per_wave queries walks
int groups_per_wave(const KGeom &g, const KCache &c, int rows_per_wave) {
    const int admissible = max_candidates(g, c.valid), k = g.topk < admissible ? g.topk : admissible, splits = 4 / row_ways(g.bt, rows_per_wave);
    return (k * ((g.bt + 15) >> 4) + splits - 1) / splits;
}

// Whether float rows are walked two groups at a time instead of four.  Four pay where few, long rows at d <= 32 leave a wavefront alone
// with its loads (two / four, 36 rows of 64-token blocks, 40 and 80 groups a wavefront: 36.8 / 35.2, 68.6 / 65.0 us; 110 rows of 16-token
// blocks, 7 groups: 8.12 / 7.95).  Not where there are more workgroups than fit at four groups' registers (`resident` a unit: 1344 rows
// of 7 groups, d = 64, 39.9 / 45.8; 672 in 32-token blocks 40.8 / 56.0), not where the last stretch of four would be half empty (10 groups
// 9.05 / 9.81), and not for the four groups of a short row (264 rows of 4: 7.24 / 7.69).  Over 300 random geometries (in profiles/) the rule
// is the better form at d <= 32 (two 1.009, four 1.101 of it).  At 32 < d <= 64 it is 1.004 where two alone would be 1.001: four still takes
// rows of 128-token blocks (0.98), and rows of 7 groups in 32-token blocks for up to 1.07 of the time (60 rows, d = 64: 17.1 / 18.1).
bool two_groups(const KGeom &g, int per_wave, int resident) {
    return per_wave <= 4 || g.q_groups * g.nb * g.heads > resident * compute_units() || (per_wave - 1) % 4 < 2;
}

template <typename T, int NT, int QS>
void launch(const KGeom &g, const KCache &c, const void *q, int64_t q_st, int64_t q_sh, const int32_t *sel_idx, const int32_t *sel_cnt,
            void *o, int64_t o_st, int64_t o_sh, float *lse, float scale, hipStream_t stream) {
    const int per_xcd = (g.q_groups * g.nb * g.heads + 7) / 8;
    constexpr int GI = sizeof(T) == 2 ? 2 : NT <= 4 ? 4 : NT <= 8 ? 2 : 1;        // groups whose operands are loaded together
    const int per_wave = groups_per_wave(g, c, 16 * QS);
    auto start = [&](auto gi, auto ahead) {
        attn_generic_kernel<T, NT, QS, gi, ahead><<<dim3(per_xcd * 8), kThreads, 0, stream>>>(
            g, c, (const T *)q, q_st, q_sh, sel_idx, sel_cnt, (T *)o, o_st, o_sh, lse, scale * kLog2e, per_xcd);
    };
    // Whether to request keys a stretch ahead.  It costs registers, and a row of one stretch its order of requests; it pays where a wavefront is
    // alone with its loads, rows are long and a stretch's products long enough to cover a request.  In turn / ahead, us (groups a wavefront,
    // 16-token blocks unless stated; all of it in profiles/): float, d = 64, 256 rows of 2 groups 6.1 / 6.6, of 6 9.7 / 9.5, of 16 22.2 / 17.8,
    // 512 rows of 4 12.4 / 11.9, of 7 (by four) 19.3 / 21.6; d = 96, 256 rows of 4 11.6 / 10.7, 512 of them 17.9 / 19.7, but in 32-token blocks
    // 35.2 / 32.4; d = 200 always (256 rows of 4 24.2 / 21.8); d = 32 not (256 rows of 2 4.6 / 5.2), except, for 1.06 of the time, by four in blocks
    // of more than 16 tokens, of which two_groups() counts two workgroups a unit.  bf16: not up to d = 96 (d = 64, 256 rows of 2 4.8 / 5.0, of 4
    // 5.9 / 6.0), beyond in blocks of more than 16 tokens (d = 128, 32-token blocks, 256 rows of 6 15.6 / 14.6).
    auto call = [&](auto gi) {
        constexpr bool ALWAYS = NT == 16 || NT * QS * gi == 16 && NT == 2, SOMETIMES = !ALWAYS && (sizeof(T) == 4 ? NT >= 4 : NT * QS == 16);
        if constexpr (SOMETIMES)
            if (per_wave >= (sizeof(T) == 4 && NT * QS >= 12 ? 3 : 4) &&
                (NT * QS >= 12 || (NT == 8 && per_wave >= 6) || g.q_groups * g.nb * g.heads <= (NT * QS * gi == 8 ? 2 : 1) * compute_units()))
                return start(gi, std::true_type{});
        start(gi, std::bool_constant<ALWAYS>{});
    };
    if constexpr (GI == 4 && sizeof(T) == 4)
        if (two_groups(g, per_wave, NT == 2 ? (QS == 1 ? 4 : 2) : (QS == 1 ? 2 : 1))) return call(std::integral_constant<int, 2>{});
    call(std::integral_constant<int, GI>{});
}

template <typename T>
void launch(const KGeom &g, const KCache &c, const void *q, int64_t q_st, int64_t q_sh, const int32_t *sel_idx, const int32_t *sel_cnt,
            void *o, int64_t o_st, int64_t o_sh, float *lse, float scale, hipStream_t stream) {
#define LCSA_CALL(NT)                                                                                                       \
    {                                                                                                                       \
        constexpr int QS = NT <= 8 ? 2 : 1;      /* 32 query rows per wavefront share each operand fragment */             \
        if (QS == 2 && g.bt > 16) launch<T, NT, QS>(g, c, q, q_st, q_sh, sel_idx, sel_cnt, o, o_st, o_sh, lse, scale, stream); \
        else launch<T, NT, 1>(g, c, q, q_st, q_sh, sel_idx, sel_cnt, o, o_st, o_sh, lse, scale, stream);                    \
    }
    LCSA_FOR_HEAD_DIM(g.d, LCSA_CALL)
#undef LCSA_CALL
}

} // namespace

hipError_t launch_attn_generic(const KGeom &g, const KCache &c, const void *q, int64_t q_st, int64_t q_sh,
                               const int32_t *sel_idx, const int32_t *sel_cnt,
                               void *o, int64_t o_st, int64_t o_sh, float *lse, float scale, hipStream_t stream) {
    if (g.bf16) launch<__bf16>(g, c, q, q_st, q_sh, sel_idx, sel_cnt, o, o_st, o_sh, lse, scale, stream);
    else launch<float>(g, c, q, q_st, q_sh, sel_idx, sel_cnt, o, o_st, o_sh, lse, scale, stream);
    return hipGetLastError();
}

} // namespace lcsa
