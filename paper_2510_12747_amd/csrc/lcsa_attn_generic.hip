// Block-sparse attention, general path: any head_dim <= 256, any block shape, f32 or bf16 storage, float products on the
// matrix cores (lcsa_fp32_mma.h).  Used where the shape constraints of the bf16 / d = 128 kernel do not hold.
//
// One workgroup per (head, query block), four wavefronts.  A wavefront owns 16 QS query rows (columns of S^T = K Q^T, so
// that a query's statistics live in four lanes and S^T is the operand of O^T += V^T P^T as it stands) and walks the
// 16-key groups of the selected blocks, GI groups at a time.  Blocks with fewer query rows than four wavefronts take
// split the key groups instead: each wavefront keeps a softmax of its own over every (4 / ways)-th stretch of GI groups,
// and the partial results meet in LDS at the end.  No LDS and no barrier otherwise.
//
// What bounds it: at 8 heads, d = 64, bf16, 32-token blocks, k = 16 on a 24 x 44 grid 34 us, of which the float P V products
// are 9 us of matrix time and the rest is load latency (two wavefronts per SIMD).  A wavefront per query token with
// lane-per-key dot products in vector FMA took 1429 us there (every query re-read all its keys) and 49 us where this
// takes 7.5 us on the smallest case (1 head, d = 32, f32, 16-token blocks, k = 4).
#include "lcsa_fp32_mma.h"
#include <type_traits>

namespace lcsa {
namespace {

using namespace fp32mma;

constexpr int kThreads = 256;

template <typename T, int NT, int QS, int GI>
__global__ __launch_bounds__(kThreads) void attn_generic_kernel(
    KGeom g, KCache c, const T *__restrict__ q, int64_t q_st, int64_t q_sh,
    const int32_t *__restrict__ sel_idx, const int32_t *__restrict__ sel_cnt,
    T *__restrict__ o, int64_t o_st, int64_t o_sh, float *__restrict__ lse, float scale_log2, int per_xcd) {
    __shared__ float part_ml[4][QS][2][16];                  // [wavefront][piece][max, sum][query]
    __shared__ f32x4 part_o[4][QS][NT][64];
    // XCD-aware order: an XCD (workgroup id mod 8) gets a contiguous run of (head, query block) items
    const int n_qb = g.q_groups * g.nb;
    const int item = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (item >= n_qb * g.heads) return;
    const int head = item / n_qb, qb = item - head * n_qb;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = lane & 15, g4 = lane >> 4;
    const int fq = qb / g.nb, tile = qb - fq * g.nb, by = tile / g.tx, bx = tile - by * g.tx;
    const BlockTokens qt(g, min(g.th, g.H - by * g.th), min(g.tw, g.W - bx * g.tw));
    const int ways = row_ways(qt.n_valid, 16 * QS), splits = 4 / ways;
    const int qw = wave / splits, ks = wave - qw * splits;

    const int64_t row = (int64_t)head * n_qb + qb;
    const int cnt = min(max(sel_cnt[row], 0), g.topk);       // a row holds at most topk ids
    const int32_t *sel = sel_idx + row * g.topk;
    const int start = ring_start(c, g);
    const int per_block = (g.bt + 15) >> 4, total = cnt * per_block;      // 16-key groups
    const T *k_head = (const T *)c.k + (int64_t)head * g.cap * g.nb * g.bt * g.d;
    const T *v_head = (const T *)c.v + (int64_t)head * g.cap * g.nb * g.bt * g.d;

    // more than one round only where four wavefronts do not cover the block, and then splits == 1
    for (int q0 = qw * 16 * QS; q0 < qt.n_valid || splits > 1; q0 += ways * 16 * QS) {
        RowFrag<T, NT> qf[QS];
        int64_t token[QS];
        bool q_valid[QS];
#pragma unroll
        for (int s = 0; s < QS; ++s) {
            int ft, r, cc;
            q_valid[s] = qt.at(q0 + 16 * s + m, ft, r, cc);
            if (!q_valid[s]) ft = r = cc = 0;                // padding rows compute on the block's first token and store nothing
            token[s] = raster_token(g, fq, ft, by * g.th + r, bx * g.tw + cc);
            qf[s].load(q + token[s] * q_st + (int64_t)head * q_sh, g.d, g4);
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
        for (int i0 = ks * GI; i0 < total; i0 += splits * GI) {
            RowFrag<T, NT> kf[GI];
            ColFrag<T, NT> vf[GI];
            int left[GI];                                    // valid keys of the group, <= 0: none
#pragma unroll
            for (int i = 0; i < GI; ++i) {
                const int f = min(i0 + i, total - 1), b = f / per_block, first = (f - b * per_block) * 16;
                const int kb = min(max(sel[b], 0), c.valid * g.nb - 1);   // ids outside the cache must not become wild addresses
                const int grp = kb / g.nb, kt = kb - grp * g.nb, kby = kt / g.tx, kbx = kt - kby * g.tx;
                const int n = g.tt * min(g.th, g.H - kby * g.th) * min(g.tw, g.W - kbx * g.tw);
                left[i] = i0 + i < total ? n - first : 0;
                const int64_t base = ((int64_t)cache_slot(c, g, start, head, grp) * g.nb + kt) * g.bt;
                // rows beyond the block's bt (bt not a multiple of 16) repeat its last key, which is masked, and have no value
                kf[i].load(k_head + (base + min(first + m, g.bt - 1)) * g.d, g.d, g4);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int j = first + 4 * g4 + r;
                    vf[i].load(r, j < g.bt && i0 + i < total ? v_head + (base + j) * g.d : (const T *)zero_row, g.d, m);
                }
            }
#pragma unroll
            for (int s = 0; s < QS; ++s) {
                f32x4 sc[GI];
                float mnew = mx[s];
#pragma unroll
                for (int i = 0; i < GI; ++i) {
                    sc[i] = RowFrag<T, NT>::mma(kf[i], qf[s], f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        sc[i][r] = 4 * g4 + r < left[i] ? sc[i][r] * scale_log2 : -__builtin_inff();
                        mnew = fmaxf(mnew, sc[i][r]);
                    }
                }
                mnew = column_max(mnew);
                const float ref = mnew == -__builtin_inff() ? 0.f : mnew;     // nothing but padding so far
                const float alpha = __builtin_amdgcn_exp2f(mx[s] - ref);
                mx[s] = mnew;
                l[s] *= alpha;
#pragma unroll
                for (int t = 0; t < NT; ++t) oacc[s][t] *= alpha;
#pragma unroll
                for (int i = 0; i < GI; ++i) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        sc[i][r] = __builtin_amdgcn_exp2f(sc[i][r] - ref);
                        l[s] += sc[i][r];
                    }
                    ColFrag<T, NT>::mma(vf[i], sc[i], oacc[s]);
                }
            }
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
            if (!q_valid[s]) continue;
            const float inv = l[s] > 0.f ? 1.f / l[s] : 0.f;
#pragma unroll
            for (int p = 0; p < NT / 2; ++p) {
                float x[8];
                channels_of(oacc[s], p, x);
#pragma unroll
                for (int i = 0; i < 8; ++i) x[i] *= inv;
                store8(o + token[s] * o_st + (int64_t)head * o_sh, 32 * p + 8 * g4, g.d, x);
            }
            if (lse && g4 == 0) lse[token[s] * g.heads + head] = l[s] > 0.f ? (mx[s] + __builtin_amdgcn_logf(l[s])) * kLn2 : -__builtin_inff();
        }
        if (splits > 1) return;
    }
}

// Whether float rows are walked two groups at a time instead of four.  Four have their loads in flight together, which two make
// up for where there are more workgroups than fit at four groups' registers (`resident` a unit: 1344 rows of 20 16-token blocks at
// d = 64 50.7 us with four, 40.2 with two; 384 rows of 20 64-token blocks 157 / 131), or where the last stretch of four would be
// half empty (5 groups a wavefront, 200 rows, 20.6 / 17.4; one group, 8 rows, 7.1 / 5.6; 10 groups 18.5 / 17.3).  Elsewhere two are
// slower (28 groups 18.5 / 19.3, 40 groups 78.6 / 83.0).  bf16 rows take half the registers: 33.1 us with four, 35.0 with two.
bool two_groups(const KGeom &g, const KCache &c, int rows_per_wave, int resident) {
    const int admissible = max_candidates(g, c.valid), k = g.topk < admissible ? g.topk : admissible;
    const int per_wave = (k * ((g.bt + 15) >> 4) + 4 / row_ways(g.bt, rows_per_wave) - 1) / (4 / row_ways(g.bt, rows_per_wave));
    return g.q_groups * g.nb * g.heads > resident * compute_units() || (per_wave - 1) % 4 < 2;
}

template <typename T, int NT, int QS>
void launch(const KGeom &g, const KCache &c, const void *q, int64_t q_st, int64_t q_sh, const int32_t *sel_idx, const int32_t *sel_cnt,
            void *o, int64_t o_st, int64_t o_sh, float *lse, float scale, hipStream_t stream) {
    const int per_xcd = (g.q_groups * g.nb * g.heads + 7) / 8;
    constexpr int GI = NT <= 4 ? 4 : NT <= 8 ? 2 : 1;        // groups whose operands are loaded together
    auto call = [&](auto gi) {
        attn_generic_kernel<T, NT, QS, gi><<<dim3(per_xcd * 8), kThreads, 0, stream>>>(
            g, c, (const T *)q, q_st, q_sh, sel_idx, sel_cnt, (T *)o, o_st, o_sh, lse, scale * kLog2e, per_xcd);
    };
    if constexpr (GI == 4 && sizeof(T) == 4)
        if (two_groups(g, c, 16 * QS, NT == 2 ? (QS == 1 ? 4 : 2) : (QS == 1 ? 2 : 1))) return call(std::integral_constant<int, 2>{});
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
