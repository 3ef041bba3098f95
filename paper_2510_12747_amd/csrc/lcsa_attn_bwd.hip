// Backward of the block-sparse attention (Sec. 3.2 "Stage 2": the model is trained with this attention).
// The discrete top-k choice carries no gradient, so this is the backward of eq. (1) restricted to the kept
// block pairs: with s_ij = scale q_i.k_j, p_ij = exp(s_ij - lse_i), g_i = dL/do_i,
//     t_ij = g_i.v_j,  D_i = sum_j p_ij t_ij (= g_i.o_i),  u_ij = scale p_ij (t_ij - D_i),
//     dq_i = sum_j u_ij k_j,   dk_j = sum_i u_ij q_i,   dv_j = sum_i p_ij g_i.
//
// Two kernels, float products on the matrix cores (lcsa_fp32_mma.h), any shape the general forward covers, no atomics and
// fixed summation orders (results are reproducible bit for bit):
//   bwd_dq_kernel    one workgroup per (head, query block), a wavefront per 16 query tokens: first over the kept keys to
//                    form D_i from the kernel's own p and t (the forward's output, rounded to its element type, would
//                    put an error of ~2^-9 |o| |g| sqrt(d) into D and through it into dq and dk; D_i is also stored for
//                    the second kernel), then again for u and dq.
//   bwd_dkv_kernel   one workgroup per (head, key block), a wavefront per 16 key tokens: lists the query blocks that kept
//                    this block (their id lists are ascending: one binary search per row), walks them in ascending order;
//                    every key token belongs to exactly one block, so dk and dv are written in full.
// Blocks with fewer rows than four wavefronts take share the walk among the wavefronts; the partial sums meet in LDS, in
// wavefront order.  K and V are read from the caller's raster tensors (the frames the cache held at the forward, oldest
// first), token rows straight into registers.
//
// What bounds them: latency (2 heads, d = 32, fp32, 16-token blocks, k = 16 on a 24 x 44 grid: 20 + 19 us, of which
// 2.4 us would be matrix work).  Token-per-wavefront dot products in vector FMA with the key block's accumulators in LDS
// took 541 + 182 us there.
#include "lcsa_fp32_mma.h"

namespace lcsa {
namespace {

using namespace fp32mma;

constexpr int kThreads = 256;
constexpr int kListed = 2048;            // query blocks whose kept flags are turned into a list at a time

struct BlockRef { int group, by, bx, vh, vw, n_valid; };
__device__ inline BlockRef block_ref(const KGeom &g, int block) {
    BlockRef b;
    b.group = block / g.nb;
    const int tile = block - b.group * g.nb;
    b.by = tile / g.tx;
    b.bx = tile - b.by * g.tx;
    b.vh = min(g.th, g.H - b.by * g.th);
    b.vw = min(g.tw, g.W - b.bx * g.tw);
    b.n_valid = g.tt * b.vh * b.vw;
    return b;
}
// raster token of block token i; rows beyond the valid ones repeat the block's first token (their probability is zero; what
// it multiplies is read from zero_row)
__device__ inline int64_t token_of(const KGeom &g, const BlockRef &b, const BlockTokens &bt, int i) {
    int ft, r, c;
    if (!bt.at(i, ft, r, c)) ft = r = c = 0;
    return raster_token(g, b.group, ft, b.by * g.th + r, b.bx * g.tw + c);
}

// dst (+)= the partial sums of the other wavefronts of a piece, in wavefront order; part is [4][N][64]
template <int N> __device__ inline void add_parts(const f32x4 (*part)[N][64], int wave, int splits, int lane, f32x4 (&acc)[N]) {
    for (int w = 1; w < splits; ++w)
#pragma unroll
        for (int t = 0; t < N; ++t) acc[t] += part[wave + w][t][lane];
}

// ---------------------------------------------------------------------------------------------------------------
template <typename T, int NT>
__global__ __launch_bounds__(kThreads) void bwd_dq_kernel(
    KGeom g, int kv_groups, const T *__restrict__ q, int64_t q_st, int64_t q_sh,
    const T *__restrict__ k, const T *__restrict__ v, int64_t kv_st, int64_t kv_sh,
    const int32_t *__restrict__ sel_idx, const int32_t *__restrict__ sel_cnt,
    const T *__restrict__ d_o, int64_t o_st, int64_t o_sh, const float *__restrict__ lse,
    float *__restrict__ d_q, float *__restrict__ delta, float scale) {
    __shared__ float part_d[4][16];
    __shared__ f32x4 part_q[4][NT][64];
    const int qb = blockIdx.x / g.heads, head = blockIdx.x - qb * g.heads;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = lane & 15, g4 = lane >> 4;
    const int n_qb = g.q_groups * g.nb;
    const BlockRef qr = block_ref(g, qb);
    const BlockTokens qt(g, qr.vh, qr.vw);
    const int ways = row_ways(qr.n_valid, 16), splits = 4 / ways;
    const int qw = wave / splits, ks = wave - qw * splits;
    const int64_t row = (int64_t)head * n_qb + qb;
    const int cnt = min(max(sel_cnt[row], 0), g.topk);
    const int32_t *sel = sel_idx + row * g.topk;
    const int per_block = (g.bt + 15) >> 4, total = cnt * per_block;      // 16-key groups
    const float scale_log2 = scale * kLog2e;
    k += (int64_t)head * kv_sh;
    v += (int64_t)head * kv_sh;

    // more than one round only where four wavefronts do not cover the block, and then splits == 1
    for (int q0 = qw * 16; q0 < qr.n_valid || splits > 1; q0 += ways * 16) {
        const bool q_valid = q0 + m < qr.n_valid;
        const int64_t token = token_of(g, qr, qt, q0 + m);
        RowFrag<T, NT> qf, gf;
        qf.load(q + token * q_st + (int64_t)head * q_sh, g.d, g4);
        gf.load(d_o + token * o_st + (int64_t)head * o_sh, g.d, g4);
        const float l2 = lse[token * g.heads + head] * kLog2e;

        // p and t of this lane's query and the four keys 4 g4 + r of group f (p = 0 for keys beyond the valid ones)
        auto key_group = [&](int f, f32x4 &p, f32x4 &t, auto &&also) {
            const int b = f / per_block, first = (f - b * per_block) * 16;
            const BlockRef kr = block_ref(g, min(max(sel[b], 0), kv_groups * g.nb - 1));   // ids outside the visible blocks must not become wild addresses
            const BlockTokens kt(g, kr.vh, kr.vw);
            const int64_t at = token_of(g, kr, kt, first + m) * kv_st;
            RowFrag<T, NT> kf, vf;
            kf.load(k + at, g.d, g4);
            vf.load(first + m < kr.n_valid ? v + at : (const T *)zero_row, g.d, g4);
            also(kr, kt, first);
            p = RowFrag<T, NT>::mma(kf, qf, f32x4{0.f, 0.f, 0.f, 0.f});
            t = RowFrag<T, NT>::mma(vf, gf, f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
            for (int r = 0; r < 4; ++r)
                p[r] = first + 4 * g4 + r < kr.n_valid ? __builtin_amdgcn_exp2f(fmaf(p[r], scale_log2, -l2)) : 0.f;
        };

        float D = 0.f;
#pragma unroll 2
        for (int f = ks; f < total; f += splits) {
            f32x4 p, t;
            key_group(f, p, t, [](const BlockRef &, const BlockTokens &, int) {});
#pragma unroll
            for (int r = 0; r < 4; ++r) D = fmaf(p[r], t[r], D);
        }
        D = column_sum(D);
        if (splits > 1) {                                    // uniform over the workgroup
            if (g4 == 0) part_d[wave][m] = D;
            __syncthreads();
            D = 0.f;
            for (int w = 0; w < splits; ++w) D += part_d[qw * splits + w][m];
        }
        if (q_valid && g4 == 0 && ks == 0) delta[token * g.heads + head] = D;

        f32x4 dq[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) dq[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
        for (int f = ks; f < total; f += splits) {
            f32x4 p, t;
            ColFrag<T, NT> kc;
            key_group(f, p, t, [&](const BlockRef &kr, const BlockTokens &kt, int first) {
#pragma unroll
                for (int r = 0; r < 4; ++r) kc.load(r, k + token_of(g, kr, kt, first + 4 * g4 + r) * kv_st, g.d, m);
            });
#pragma unroll
            for (int r = 0; r < 4; ++r) p[r] *= (t[r] - D) * scale;
            ColFrag<T, NT>::mma(kc, p, dq);
        }
        if (splits > 1) {
            if (ks != 0)
#pragma unroll
                for (int t = 0; t < NT; ++t) part_q[wave][t][lane] = dq[t];
            __syncthreads();
            if (ks != 0) return;
            add_parts<NT>(part_q, wave, splits, lane, dq);
        }
        if (q_valid) {
#pragma unroll
            for (int p = 0; p < NT / 2; ++p) {
                float x[8];
                channels_of(dq, p, x);
                store8(d_q + (token * g.heads + head) * g.d, 32 * p + 8 * g4, g.d, x);
            }
        }
        if (splits > 1) return;
    }
}

// ---------------------------------------------------------------------------------------------------------------
template <typename T, int NT>
__global__ __launch_bounds__(kThreads) void bwd_dkv_kernel(
    KGeom g, int kv_groups, const T *__restrict__ q, int64_t q_st, int64_t q_sh,
    const T *__restrict__ k, const T *__restrict__ v, int64_t kv_st, int64_t kv_sh,
    const int32_t *__restrict__ sel_idx, const int32_t *__restrict__ sel_cnt,
    const T *__restrict__ d_o, int64_t o_st, int64_t o_sh, const float *__restrict__ lse, const float *__restrict__ delta,
    float *__restrict__ d_k, float *__restrict__ d_v, float scale) {
    __shared__ f32x4 part[4][NT][64];
    __shared__ unsigned char kept_by[kListed];
    __shared__ uint16_t list[kListed];
    __shared__ int n_listed;
    const int kb = blockIdx.x / g.heads, head = blockIdx.x - kb * g.heads;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 15, g4 = lane >> 4;
    const int n_qb = g.q_groups * g.nb;
    const BlockRef kr = block_ref(g, kb);
    const BlockTokens kt(g, kr.vh, kr.vw);
    const int ways = row_ways(kr.n_valid, 16), splits = 4 / ways;
    const int kw = wave / splits, ks = wave - kw * splits;
    const int per_block = (g.bt + 15) >> 4;
    const float scale_log2 = scale * kLog2e;
    q += (int64_t)head * q_sh;
    d_o += (int64_t)head * o_sh;

    // rounds over the block's key rows: every wavefront takes part in every round (the lists are made together)
    for (int base = 0; base < kr.n_valid; base += ways * 16) {
        const int k0 = base + kw * 16;
        const bool key_ok = k0 + m < kr.n_valid;
        const int64_t token = token_of(g, kr, kt, k0 + m);
        RowFrag<T, NT> kf, vf;
        kf.load(k + token * kv_st + (int64_t)head * kv_sh, g.d, g4);
        vf.load(v + token * kv_st + (int64_t)head * kv_sh, g.d, g4);
        f32x4 dk[NT], dv[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) dk[t] = dv[t] = f32x4{0.f, 0.f, 0.f, 0.f};

        for (int qb0 = 0; qb0 < n_qb; qb0 += kListed) {
            // which query blocks kept this key block?  (ascending id lists: binary search)
            const int n_here = min(kListed, n_qb - qb0);
            __syncthreads();                                 // the previous list is no longer read
            for (int i = tid; i < n_here; i += kThreads) {
                const int64_t row = (int64_t)head * n_qb + qb0 + i;
                const int32_t *sel = sel_idx + row * g.topk;
                const int c = min(max(sel_cnt[row], 0), g.topk);
                int lo = 0, hi = c;
                while (lo < hi) { const int mid = (lo + hi) >> 1; if (sel[mid] < kb) lo = mid + 1; else hi = mid; }
                kept_by[i] = lo < c && sel[lo] == kb;
            }
            __syncthreads();
            if (wave == 0) {
                int n = 0;
                for (int i0 = 0; i0 < n_here; i0 += 64) {
                    const bool kept = i0 + lane < n_here && kept_by[i0 + lane];
                    const uint64_t mask = __ballot(kept);
                    if (kept) list[n + __popcll(mask & ((1ull << lane) - 1ull))] = (uint16_t)(i0 + lane);
                    n += __popcll(mask);
                }
                if (lane == 0) n_listed = n;
            }
            __syncthreads();
            const int total = n_listed * per_block;          // 16-query groups
#pragma unroll 2
            for (int f = ks; f < total; f += splits) {
                const int b = f / per_block, first = (f - b * per_block) * 16;
                const BlockRef qr = block_ref(g, __builtin_amdgcn_readfirstlane(qb0 + list[b]));
                const BlockTokens qt(g, qr.vh, qr.vw);
                const int64_t at = token_of(g, qr, qt, first + m);
                RowFrag<T, NT> qf, gf;
                qf.load(q + at * q_st, g.d, g4);
                gf.load(d_o + at * o_st, g.d, g4);
                ColFrag<T, NT> qc, gc;
                float l2[4], D[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int64_t tok = token_of(g, qr, qt, first + 4 * g4 + r);
                    qc.load(r, q + tok * q_st, g.d, m);
                    gc.load(r, first + 4 * g4 + r < qr.n_valid ? d_o + tok * o_st : (const T *)zero_row, g.d, m);
                    l2[r] = lse[tok * g.heads + head] * kLog2e;
                    D[r] = delta[tok * g.heads + head];      // written by bwd_dq_kernel, earlier on the stream
                }
                f32x4 p = RowFrag<T, NT>::mma(qf, kf, f32x4{0.f, 0.f, 0.f, 0.f});
                f32x4 u = RowFrag<T, NT>::mma(gf, vf, f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const bool ok = first + 4 * g4 + r < qr.n_valid;         // padding queries: probability zero
                    p[r] = ok ? __builtin_amdgcn_exp2f(fmaf(p[r], scale_log2, -l2[r])) : 0.f;
                    u[r] = p[r] * ((u[r] - D[r]) * scale);
                }
                ColFrag<T, NT>::mma(gc, p, dv);
                ColFrag<T, NT>::mma(qc, u, dk);
            }
        }
        if (splits > 1) {                                    // uniform over the workgroup; dk and dv take turns in `part`
#pragma unroll
            for (int turn = 0; turn < 2; ++turn) {
                f32x4 (&acc)[NT] = turn == 0 ? dk : dv;
                __syncthreads();
                if (ks != 0)
#pragma unroll
                    for (int t = 0; t < NT; ++t) part[wave][t][lane] = acc[t];
                __syncthreads();
                if (ks == 0) add_parts<NT>(part, wave, splits, lane, acc);
            }
        }
        if (key_ok && ks == 0) {
#pragma unroll
            for (int p = 0; p < NT / 2; ++p) {
                float x[8];
                channels_of(dk, p, x);
                store8(d_k + (token * g.heads + head) * g.d, 32 * p + 8 * g4, g.d, x);
                channels_of(dv, p, x);
                store8(d_v + (token * g.heads + head) * g.d, 32 * p + 8 * g4, g.d, x);
            }
        }
    }
}

template <typename T>
hipError_t launch(const KGeom &g, int kv_groups, const void *q, int64_t q_st, int64_t q_sh, const void *k, const void *v, int64_t kv_st, int64_t kv_sh,
                  const int32_t *sel_idx, const int32_t *sel_cnt, const void *d_o, int64_t o_st, int64_t o_sh, const float *lse,
                  float *d_q, float *d_k, float *d_v, float *delta, float scale, hipStream_t stream) {
    const dim3 grid_q(g.q_groups * g.nb * g.heads), grid_k(kv_groups * g.nb * g.heads);
    hipError_t e = hipSuccess;
#define LCSA_CALL(NT)                                                                                                               \
    {                                                                                                                               \
        bwd_dq_kernel<T, NT><<<grid_q, kThreads, 0, stream>>>(g, kv_groups, (const T *)q, q_st, q_sh, (const T *)k, (const T *)v,   \
                                                              kv_st, kv_sh, sel_idx, sel_cnt, (const T *)d_o, o_st, o_sh, lse,      \
                                                              d_q, delta, scale);                                                   \
        e = hipGetLastError();                                                                                                      \
        if (e != hipSuccess) return e;                                                                                              \
        bwd_dkv_kernel<T, NT><<<grid_k, kThreads, 0, stream>>>(g, kv_groups, (const T *)q, q_st, q_sh, (const T *)k, (const T *)v,  \
                                                               kv_st, kv_sh, sel_idx, sel_cnt, (const T *)d_o, o_st, o_sh, lse,     \
                                                               delta, d_k, d_v, scale);                                             \
        e = hipGetLastError();                                                                                                      \
    }
    LCSA_FOR_HEAD_DIM(g.d, LCSA_CALL)
#undef LCSA_CALL
    return e;
}

} // namespace

// No resource limit of the kernels above, whose LDS does not depend on the block or on the number of query blocks: the shapes
// whose key-block gradients, row values and query-block flags would exceed 160 KB have always been refused, and still are.
bool attn_bwd_supported(const KGeom &g) {
    return ((size_t)2 * g.bt * g.d + 8 * g.bt + 8 * g.d) * sizeof(float) + (size_t)g.q_groups * g.nb <= 160 * 1024;
}

hipError_t launch_attn_bwd(const KGeom &g, int kv_groups, const void *q, int64_t q_st, int64_t q_sh,
                           const void *k, const void *v, int64_t kv_st, int64_t kv_sh,
                           const int32_t *sel_idx, const int32_t *sel_cnt,
                           const void *d_o, int64_t o_st, int64_t o_sh, const float *lse,
                           float *d_q, float *d_k, float *d_v, float *delta, float scale, hipStream_t stream) {
    return g.bf16 ? launch<__bf16>(g, kv_groups, q, q_st, q_sh, k, v, kv_st, kv_sh, sel_idx, sel_cnt, d_o, o_st, o_sh, lse, d_q, d_k, d_v, delta, scale, stream)
                  : launch<float>(g, kv_groups, q, q_st, q_sh, k, v, kv_st, kv_sh, sel_idx, sel_cnt, d_o, o_st, o_sh, lse, d_q, d_k, d_v, delta, scale, stream);
}

} // namespace lcsa
