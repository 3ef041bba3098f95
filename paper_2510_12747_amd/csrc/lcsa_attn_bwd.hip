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
// What bounds them: latency, and address arithmetic (64-bit products and divisions run at a quarter of the rate).  Ids are turned
// into block positions 64 at a time, one per lane, a list of query blocks when it is made; row offsets are formed once for all
// unclipped blocks; several groups' operands are requested together; a short row's p and t stay in registers for the second pass.
// 2 heads, d = 32, fp32, 16-token blocks, k = 16 on a 24 x 44 grid: 19.4 + 18.7 -> 13.5 + 17.5 us in whole passes (36.0 -> 28.7 us back to back), of which
// 2.4 us are matrix work; 30 random geometries 0.84 of the time, 0.67 to 1.03.  Token-per-wavefront dot products in vector FMA with the
// key block's accumulators in LDS took 541 + 182 us there.
#include "lcsa_fp32_mma.h"
#include <type_traits>

namespace lcsa {
namespace {

using namespace fp32mma;

constexpr int kThreads = 256;
constexpr int kListed = 1024;            // query blocks whose kept flags are turned into a list at a time

struct BlockRef { int group, by, bx, vh, vw, n_valid; };
__device__ inline BlockRef block_ref(const KGeom &g, int block) {
    BlockRef b;
    b.group = g.by_nb(block);
    const int tile = block - b.group * g.nb;
    b.by = g.by_tx(tile);
    b.bx = tile - b.by * g.tx;
    b.vh = min(g.th, g.H - b.by * g.th);
    b.vw = min(g.tw, g.W - b.bx * g.tw);
    b.n_valid = g.tt * b.vh * b.vw;
    return b;
}
// A block as the loops want it: the raster token of its first token, and whether its last rows (1) or columns (2) are clipped.
struct Located { int origin, clip; };
__device__ inline Located locate(const KGeom &g, int block) {
    const BlockRef b = block_ref(g, block);
    return {(int)raster_token(g, b.group, 0, b.by * g.th, b.bx * g.tw), (b.vh < g.th ? 1 : 0) | (b.vw < g.tw ? 2 : 0)};
}
__device__ inline BlockTokens tokens_of(const KGeom &g, int clip) {
    return BlockTokens(g, clip & 1 ? g.H - (g.ty - 1) * g.th : g.th, clip & 2 ? g.W - (g.tx - 1) * g.tw : g.tw);
}
// Raster token of block token i, from the block's first one; rows beyond the valid ones repeat that one (their probability is
// zero, and what it multiplies is cleared).
__device__ inline int rel_token(const KGeom &g, const BlockTokens &bt, int i) {
    int ft, r, c;
    return bt.at(i, ft, r, c) ? (ft * g.H + r) * g.W + c : 0;
}
// Where the rows of a 16-row piece of a block lie, in raster tokens from the block's first one: this lane's row m, and rows
// 4 g4 + r.  Those of the first piece of an unclipped block are formed once; a later piece lies a uniform distance further on
// wherever 16 tokens are whole rows of the tile inside one frame of it.
struct PieceRows {
    int own, col[4];
    __device__ PieceRows(const KGeom &g, const BlockTokens &bt, int first, int m, int g4) {
        own = rel_token(g, bt, first + m);
#pragma unroll
        for (int r = 0; r < 4; ++r) col[r] = rel_token(g, bt, first + 4 * g4 + r);
    }
};
__device__ inline bool whole_rows(const KGeom &g) { return 16 % g.tw == 0 && g.ts % 16 == 0; }
// token distance of the piece that starts at token `first`, where whole_rows()
__device__ inline int piece_distance(const KGeom &g, int first) {
    if (first == 0) return 0;
    const int ft = first / g.ts;
    return (ft * g.H + (first - ft * g.ts) / g.tw) * g.W;
}
// f / n, f * n < 2^32
struct Divide {
    uint32_t m;
    __device__ explicit Divide(int n) : m(n == 1 ? 0 : 0xFFFFFFFFu / (uint32_t)n + 1u) {}
    __device__ int operator()(int f) const { return m == 0 ? f : (int)__umulhi((uint32_t)f, m); }
};

// dst (+)= the partial sums of the other wavefronts of a piece, in wavefront order; part is [4][N][64]
template <int N> __device__ inline void add_parts(const f32x4 (*part)[N][64], int wave, int splits, int lane, f32x4 (&acc)[N]) {
    for (int w = 1; w < splits; ++w)
#pragma unroll
        for (int t = 0; t < N; ++t) acc[t] += part[wave + w][t][lane];
}

// GI: 16-row groups whose operands are requested together.  HELD: rows of at most GI * HELD groups a wavefront keep p and t of all of
// them in registers, so that nothing is requested, or formed, twice; longer ones, and HELD = 0, walk their groups twice.

// ---------------------------------------------------------------------------------------------------------------
template <typename T, int NT, int GI, int HELD>
__global__ __launch_bounds__(kThreads, (HELD ? 2 : NT <= 2 ? 4 : NT <= 4 ? 3 : NT <= 8 ? 2 : 1)) void bwd_dq_kernel(
    KGeom g, int kv_groups, const T *__restrict__ q, int64_t q_st, int64_t q_sh,
    const T *__restrict__ k, const T *__restrict__ v, int64_t kv_st, int64_t kv_sh,
    const int32_t *__restrict__ sel_idx, const int32_t *__restrict__ sel_cnt,
    const T *__restrict__ d_o, int64_t o_st, int64_t o_sh, const float *__restrict__ lse,
    float *__restrict__ d_q, float *__restrict__ delta, float scale) {
    constexpr bool PIECES = sizeof(T) == 2 && GI > 1;
    __shared__ float part_d[4][16];
    __shared__ f32x4 part_q[4][NT][64];
    const int qb = g.by_heads(blockIdx.x), head = blockIdx.x - qb * g.heads;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = lane & 15, g4 = lane >> 4;
    const int n_qb = g.q_groups * g.nb;
    const int64_t row = (int64_t)head * n_qb + qb;
    const int32_t *sel = sel_idx + row * g.topk;
    const int32_t first_id = sel[min(lane, g.topk - 1)];     // requested together with the count
    const int cnt = min(max(sel_cnt[row], 0), g.topk);
    const Located own = locate(g, qb);
    const BlockTokens qt = tokens_of(g, own.clip);
    const int ways = row_ways(qt.n_valid, 16), splits = 4 / ways;
    const int qw = wave / splits, ks = wave - qw * splits;
    const int per_block = (g.bt + 15) >> 4, total = cnt * per_block;      // 16-key groups
    const Divide by_block(per_block);
    const float scale_log2 = scale * kLog2e;
    k += (int64_t)head * kv_sh;
    v += (int64_t)head * kv_sh;

    // kept blocks, 64 at a time, one per lane
    int chunk = 0;
    Located held;
    // ids outside the visible blocks must not become wild addresses
    auto take_chunk = [&](int32_t id) { held = locate(g, min(max(id, 0), kv_groups * g.nb - 1)); };
    take_chunk(first_id);
    const bool simple = NT <= 6 && whole_rows(g);            // the offsets stay in registers throughout
    const PieceRows unclipped(g, tokens_of(g, 0), 0, m, g4);

    // more than one round only where four wavefronts do not cover the block, and then splits == 1
    for (int q0 = qw * 16; q0 < qt.n_valid || splits > 1; q0 += ways * 16) {
        const bool q_valid = q0 + m < qt.n_valid;
        const int64_t token = own.origin + rel_token(g, qt, q0 + m);
        RowFrag<T, NT> qf, gf;
        qf.load_row(q + token * q_st + (int64_t)head * q_sh, g.d, g4);
        gf.load_row(d_o + token * o_st + (int64_t)head * o_sh, g.d, g4);
        const float l2 = lse[token * g.heads + head] * kLog2e;

        qf.clear_beyond(g.d, g4);
        gf.clear_beyond(g.d, g4);

        // GI groups of this wavefront, from its i0-th on: every splits-th of the row's
        struct Keys { RowFrag<T, NT> kf[GI], vf[GI]; int valid[GI]; };
        auto block_of = [&](int i, int &first) {
            const int f = min(ks + i * splits, total - 1), b = by_block(f);
            first = (f - b * per_block) * 16;
            return b;
        };
        // with(i, rows, first token's element, valid rows) for each of them
        auto each = [&](int i0, auto &&with) {
            int first_row, last_row;
            const int b0 = block_of(i0, first_row);
            if (b0 < chunk || block_of(i0 + GI - 1, last_row) >= chunk + 64) {      // uniform
                chunk = b0;
                take_chunk(chunk + lane < cnt ? sel[chunk + lane] : 0);
            }
#pragma unroll
            for (int i = 0; i < GI; ++i) {
                int first;
                const int b = block_of(i0 + i, first);
                const int origin = __builtin_amdgcn_readlane(held.origin, b - chunk), clip = __builtin_amdgcn_readlane(held.clip, b - chunk);
                const bool there = ks + (i0 + i) * splits < total;
                if (clip == 0 && simple) {                   // uniform
                    with(i, unclipped, (int64_t)(origin + piece_distance(g, first)) * kv_st, there ? g.bt - first : 0);
                } else {
                    const BlockTokens kt = tokens_of(g, clip);
                    with(i, PieceRows(g, kt, first, m, g4), (int64_t)origin * kv_st, there ? kt.n_valid - first : 0);
                }
            }
        };
        auto request = [&](int i0, Keys &keys) {
            each(i0, [&](int i, const PieceRows &rows, int64_t from, int valid) {
                keys.kf[i].load_row(k + from + rows.own * kv_st, g.d, g4);
                keys.vf[i].load_row(v + from + rows.own * kv_st, g.d, g4);
                keys.valid[i] = valid;
            });
        };
        // p and t of this lane's query and the keys 4 g4 + r of each group (p = 0 for keys that are not there)
        auto products = [&](Keys &keys, f32x4 (&p)[GI], f32x4 (&t)[GI]) {
#pragma unroll
            for (int i = 0; i < GI; ++i) {
                keys.kf[i].clear_beyond(g.d, g4);
                keys.vf[i].clear_beyond(g.d, g4);
                if (keys.valid[i] < 16 && m >= keys.valid[i]) keys.vf[i].clear();
                p[i] = RowFrag<T, NT>::mma(keys.kf[i], qf, f32x4{0.f, 0.f, 0.f, 0.f});
                t[i] = RowFrag<T, NT>::mma(keys.vf[i], gf, f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    p[i][r] = 4 * g4 + r < keys.valid[i] ? __builtin_amdgcn_exp2f(fmaf(p[i][r], scale_log2, -l2)) : 0.f;
            }
        };
        auto request_columns = [&](int i0, ColGroups<T, NT, GI> &kc, int (&valid)[GI]) {
            each(i0, [&](int i, const PieceRows &rows, int64_t from, int n) {
#pragma unroll
                for (int r = 0; r < 4; ++r) kc.load_row(i, r, k + from + rows.col[r] * kv_st, g.d, m);
                valid[i] = n;
            });
        };

        float D = 0.f;
        auto add_to_d = [&](const f32x4 (&p)[GI], const f32x4 (&t)[GI]) {
#pragma unroll
            for (int i = 0; i < GI; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) D = fmaf(p[i][r], t[i][r], D);
        };
        auto finish_d = [&]() {
            D = column_sum(D);
            if (splits > 1) {                                // uniform over the workgroup
                if (g4 == 0) part_d[wave][m] = D;
                __syncthreads();
                D = 0.f;
                for (int w = 0; w < splits; ++w) D += part_d[qw * splits + w][m];
            }
            if (q_valid && g4 == 0 && ks == 0) delta[token * g.heads + head] = D;
        };
        f32x4 dq[1][NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) dq[0][t] = f32x4{0.f, 0.f, 0.f, 0.f};
        auto add_to_dq = [&](const f32x4 (&p)[GI], const f32x4 (&t)[GI], ColGroups<T, NT, GI> &kc, const int (&valid)[GI], int pass) {
            f32x4 u[1][GI];
#pragma unroll
            for (int i = 0; i < GI; ++i) {
#pragma unroll
                for (int r = 0; r < 4; ++r) u[0][i][r] = p[i][r] * ((t[i][r] - D) * scale);
                kc.keep(i, valid[i], g4);
            }
            if (pass == 0) kc.template mma<1>(u, dq);
            else kc.template mma<1, true>(u, dq);
        };
        // Sums of pieces that are doubtful are made once more in float products alone; each pass ends here, true if it was the last.
        constexpr int PASSES = PIECES ? 2 : 1;
        auto last_pass = [&](int pass) {
            if (!PIECES || pass == 1 || !ColGroups<T, NT, GI>::doubtful(dq[0])) return true;      // uniform over the wavefront
#pragma unroll
            for (int t = 0; t < NT; ++t) dq[0][t] = f32x4{0.f, 0.f, 0.f, 0.f};
            return false;
        };
        const int mine = total > ks ? (total - ks + splits - 1) / splits : 0;      // groups of this wavefront
        if (HELD && total <= HELD * GI * splits) {           // uniform over the workgroup
            // A wavefront without groups takes the last one, with no valid rows, if there is one.
            Keys keys_a, keys_b;
            f32x4 p_a[GI], t_a[GI], p_b[GI], t_b[GI];
            ColGroups<T, NT, GI> kc_a, kc_b;
            int valid_a[GI], valid_b[GI];
            if (total > 0) {
                request(0, keys_a);
                if (HELD > 1) request(GI, keys_b);
                request_columns(0, kc_a, valid_a);
                if (HELD > 1) request_columns(GI, kc_b, valid_b);
                products(keys_a, p_a, t_a);
                add_to_d(p_a, t_a);
                if (HELD > 1) { products(keys_b, p_b, t_b); add_to_d(p_b, t_b); }
            }
            finish_d();
#pragma unroll
            for (int pass = 0; pass < PASSES; ++pass) {
                if (total > 0) {
                    if (pass == 1) {                         // the first took the large values out
                        request_columns(0, kc_a, valid_a);
                        if (HELD > 1) request_columns(GI, kc_b, valid_b);
                    }
                    add_to_dq(p_a, t_a, kc_a, valid_a, pass);
                    if (HELD > 1) add_to_dq(p_b, t_b, kc_b, valid_b, pass);
                }
                if (last_pass(pass)) break;
            }
        } else {
            Keys keys;
            f32x4 p[GI], t[GI];
            for (int i0 = 0; i0 < mine; i0 += GI) {
                request(i0, keys);
                products(keys, p, t);
                add_to_d(p, t);
            }
            finish_d();
#pragma unroll
            for (int pass = 0; pass < PASSES; ++pass) {
                for (int i0 = 0; i0 < mine; i0 += GI) {
                    ColGroups<T, NT, GI> kc;
                    int valid[GI];
                    request(i0, keys);
                    request_columns(i0, kc, valid);
                    products(keys, p, t);
                    add_to_dq(p, t, kc, valid, pass);
                }
                if (last_pass(pass)) break;
            }
        }
        if (splits > 1) {
            if (ks != 0)
#pragma unroll
                for (int t = 0; t < NT; ++t) part_q[wave][t][lane] = dq[0][t];
            __syncthreads();
            if (ks != 0) return;
            add_parts<NT>(part_q, wave, splits, lane, dq[0]);
        }
        if (q_valid) {
#pragma unroll
            for (int p = 0; p < NT / 2; ++p) {
                float x[8];
                channels_of(dq[0], p, x);
                store8(d_q + (token * g.heads + head) * g.d, 32 * p + 8 * g4, g.d, x);
            }
        }
        if (splits > 1) return;
    }
}

// ---------------------------------------------------------------------------------------------------------------
// WAVES: wavefronts a SIMD at least
template <typename T, int NT, int GI, int WAVES>
__global__ __launch_bounds__(kThreads, WAVES) void bwd_dkv_kernel(
    KGeom g, int kv_groups, const T *__restrict__ q, int64_t q_st, int64_t q_sh,
    const T *__restrict__ k, const T *__restrict__ v, int64_t kv_st, int64_t kv_sh,
    const int32_t *__restrict__ sel_idx, const int32_t *__restrict__ sel_cnt,
    const T *__restrict__ d_o, int64_t o_st, int64_t o_sh, const float *__restrict__ lse, const float *__restrict__ delta,
    float *__restrict__ d_k, float *__restrict__ d_v, float scale) {
    using Cols = ColGroups<T, NT, GI>;
    constexpr bool PIECES = sizeof(T) == 2 && GI > 1;
    constexpr int kParts = NT <= 4 ? 2 : 1;
    __shared__ f32x4 part[kParts][4][NT][64];
    __shared__ unsigned char kept_by[kListed], list_clip[kListed];
    __shared__ int list_origin[kListed];
    __shared__ int n_listed, again;
    const int kb = g.by_heads(blockIdx.x), head = blockIdx.x - kb * g.heads;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = lane & 15, g4 = lane >> 4;
    const int n_qb = g.q_groups * g.nb;
    const Located own = locate(g, kb);
    const BlockTokens kt = tokens_of(g, own.clip);
    const int ways = row_ways(kt.n_valid, 16), splits = 4 / ways;
    const int kw = wave / splits, ks = wave - kw * splits;
    const int per_block = (g.bt + 15) >> 4;
    const Divide by_block(per_block);
    const float scale_log2 = scale * kLog2e;
    q += (int64_t)head * q_sh;
    d_o += (int64_t)head * o_sh;

    const bool simple = NT <= 6 && whole_rows(g);            // the offsets stay in registers throughout
    const PieceRows unclipped(g, tokens_of(g, 0), 0, m, g4);

    if (PIECES && tid == 0) again = -1;
    // rounds over the block's key rows: every wavefront takes part in every round (the lists are made together)
    for (int base = 0; base < kt.n_valid; base += ways * 16) {
        const int k0 = base + kw * 16;
        const bool key_ok = k0 + m < kt.n_valid;
        const int64_t token = own.origin + rel_token(g, kt, k0 + m);
        RowFrag<T, NT> kf, vf;
        kf.load_row(k + token * kv_st + (int64_t)head * kv_sh, g.d, g4);
        vf.load_row(v + token * kv_st + (int64_t)head * kv_sh, g.d, g4);
        kf.clear_beyond(g.d, g4);
        vf.clear_beyond(g.d, g4);
        f32x4 dk[1][NT], dv[1][NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) dk[0][t] = dv[0][t] = f32x4{0.f, 0.f, 0.f, 0.f};
        bool again_k = true, again_v = true;                 // uniform over the wavefront
#pragma unroll
        for (int pass = 0; pass < (PIECES ? 2 : 1); ++pass) {      // the second in float products alone, for sums of pieces that are doubtful
            if (pass == 1) {
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    if (again_k) dk[0][t] = f32x4{0.f, 0.f, 0.f, 0.f};
                    if (again_v) dv[0][t] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
            }
            for (int qb0 = 0; qb0 < n_qb; qb0 += kListed) {
                // which query blocks kept this key block?  (ascending id lists)
                const int n_here = min(kListed, n_qb - qb0);
                const int64_t first_row = (int64_t)head * n_qb + qb0;
                __syncthreads();                                 // the previous list is no longer read
                if (NT <= 8 && g.topk <= 32) {                   // all ids, eight loads of a thread in flight; longer rows: a search reads less
                    for (int i = tid; i < n_here; i += kThreads) kept_by[i] = 0;
                    __syncthreads();
                    const int32_t *ids = sel_idx + first_row * g.topk;
                    const int n_ids = n_here * g.topk;
                    for (int at = tid; at < n_ids; at += 8 * kThreads) {
                        int id[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e) id[e] = at + e * kThreads < n_ids ? ids[at + e * kThreads] : -1;
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            if (id[e] == kb) {
                                const int i = (at + e * kThreads) / g.topk;
                                if (at + e * kThreads - i * g.topk < sel_cnt[first_row + i]) kept_by[i] = 1;
                            }
                    }
                } else {
                    for (int i = tid; i < n_here; i += kThreads) {
                        const int32_t *sel = sel_idx + (first_row + i) * g.topk;
                        const int c = min(max(sel_cnt[first_row + i], 0), g.topk);
                        int lo = 0, hi = c;
                        while (lo < hi) { const int mid = (lo + hi) >> 1; if (sel[mid] < kb) lo = mid + 1; else hi = mid; }
                        kept_by[i] = lo < c && sel[lo] == kb;
                    }
                }
                __syncthreads();
                if (wave == 0) {
                    int n = 0;
                    for (int i0 = 0; i0 < n_here; i0 += 64) {
                        const bool kept = i0 + lane < n_here && kept_by[i0 + lane];
                        const uint64_t mask = __ballot(kept);
                        if (kept) {
                            const int at = n + __popcll(mask & ((1ull << lane) - 1ull));
                            const Located b = locate(g, qb0 + i0 + lane);
                            list_origin[at] = b.origin;
                            list_clip[at] = (unsigned char)b.clip;
                        }
                        n += __popcll(mask);
                    }
                    if (lane == 0) n_listed = n;
                }
                __syncthreads();
                const int total = __builtin_amdgcn_readfirstlane(n_listed) * per_block;          // 16-query groups
                for (int f0 = ks; f0 < total; f0 += GI * splits) {
                    RowFrag<T, NT> qf[GI], gf[GI];
                    ColGroups<T, NT, GI> qc, gc;
                    float l2[GI][4], D[GI][4];
                    int valid[GI];
                    int origin[GI], own_at[GI], at[GI][4];       // first token, and rows m and 4 g4 + r from it
                    auto request_stats = [&]() {
#pragma unroll
                        for (int i = 0; i < GI; ++i) {
                            const float *lse_from = lse + (int64_t)origin[i] * g.heads + head, *d_from = delta + (int64_t)origin[i] * g.heads + head;
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                l2[i][r] = lse_from[(int64_t)at[i][r] * g.heads] * kLog2e;
                                D[i][r] = d_from[(int64_t)at[i][r] * g.heads];           // written by bwd_dq_kernel, earlier on the stream
                            }
                        }
                    };
                    auto request_columns = [&](ColGroups<T, NT, GI> &cols, const T *x, int64_t st) {
#pragma unroll
                        for (int i = 0; i < GI; ++i)
#pragma unroll
                            for (int r = 0; r < 4; ++r) cols.load_row(i, r, x + (int64_t)origin[i] * st + at[i][r] * st, g.d, m);
                    };
#pragma unroll
                    for (int i = 0; i < GI; ++i) {
                        const int f = min(f0 + i * splits, total - 1), b = by_block(f), first = (f - b * per_block) * 16;
                        origin[i] = __builtin_amdgcn_readfirstlane(list_origin[b]);
                        const int clip = __builtin_amdgcn_readfirstlane(list_clip[b]);
                        const bool there = f0 + i * splits < total;
                        auto request_rows = [&](const PieceRows &rows) {
                            qf[i].load_row(q + (int64_t)origin[i] * q_st + rows.own * q_st, g.d, g4);
                            own_at[i] = rows.own;
                            if (NT <= 8) gf[i].load_row(d_o + (int64_t)origin[i] * o_st + rows.own * o_st, g.d, g4);
#pragma unroll
                            for (int r = 0; r < 4; ++r) at[i][r] = rows.col[r];
                        };
                        if (clip == 0 && simple) {               // uniform
                            origin[i] += piece_distance(g, first);
                            valid[i] = there ? g.bt - first : 0;
                            request_rows(unclipped);
                        } else {
                            const BlockTokens qt = tokens_of(g, clip);
                            valid[i] = there ? qt.n_valid - first : 0;
                            request_rows(PieceRows(g, qt, first, m, g4));
                        }
                    }
                    constexpr bool COLUMNS = NT <= 2 || (NT <= 4 && WAVES == 2);         // registers for these beside the rows
                    if (NT <= 8) request_stats();
                    if (COLUMNS) { request_columns(gc, d_o, o_st); request_columns(qc, q, q_st); }
                    f32x4 p[1][GI], u[1][GI];
#pragma unroll
                    for (int i = 0; i < GI; ++i) {
                        qf[i].clear_beyond(g.d, g4);
                        p[0][i] = RowFrag<T, NT>::mma(qf[i], kf, f32x4{0.f, 0.f, 0.f, 0.f});
                        if (NT > 8) { __builtin_amdgcn_sched_barrier(0); gf[i].load_row(d_o + (int64_t)origin[i] * o_st + own_at[i] * o_st, g.d, g4); }
                        gf[i].clear_beyond(g.d, g4);
                        u[0][i] = RowFrag<T, NT>::mma(gf[i], vf, f32x4{0.f, 0.f, 0.f, 0.f});
                    }
                    if (NT > 8) { __builtin_amdgcn_sched_barrier(0); request_stats(); }
#pragma unroll
                    for (int i = 0; i < GI; ++i) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const bool ok = 4 * g4 + r < valid[i];               // padding queries: probability zero
                            p[0][i][r] = ok ? __builtin_amdgcn_exp2f(fmaf(p[0][i][r], scale_log2, -l2[i][r])) : 0.f;
                            u[0][i][r] = ok ? p[0][i][r] * ((u[0][i][r] - D[i][r]) * scale) : 0.f;
                        }
                    }
                    if (!COLUMNS) { __builtin_amdgcn_sched_barrier(0); request_columns(gc, d_o, o_st); }
#pragma unroll
                    for (int i = 0; i < GI; ++i) gc.keep(i, valid[i], g4);
                    if (pass == 0) gc.template mma<1>(p, dv);
                    else if (again_v) gc.template mma<1, true>(p, dv);
                    if (!COLUMNS) { __builtin_amdgcn_sched_barrier(0); request_columns(qc, q, q_st); }
#pragma unroll
                    for (int i = 0; i < GI; ++i) qc.keep(i, valid[i], g4);
                    if (pass == 0) qc.template mma<1>(u, dk);
                    else if (again_k) qc.template mma<1, true>(u, dk);
                }
            }
            if (PIECES && pass == 0) {
                again_k = Cols::doubtful(dk[0]);
                again_v = Cols::doubtful(dv[0]);
                if (again_k || again_v) again = base;
                __syncthreads();
                if (__builtin_amdgcn_readfirstlane(again) != base) break;      // set anew only behind the next barriers
            }
        }
        if (splits > 1) {                                    // uniform over the workgroup
#pragma unroll
            for (int turn = 0; turn < 2; ++turn) {           // dk and dv take turns in `part` where it holds only one of them
                f32x4 (&acc)[NT] = turn == 0 ? dk[0] : dv[0];
                if (turn == 0 || kParts == 1) __syncthreads();
                if (ks != 0)
#pragma unroll
                    for (int t = 0; t < NT; ++t) part[turn % kParts][wave][t][lane] = acc[t];
                if (kParts == 1) {
                    __syncthreads();
                    if (ks == 0) add_parts<NT>(part[0], wave, splits, lane, acc);
                }
            }
            if (kParts == 2) {
                __syncthreads();
                if (ks == 0) {
                    add_parts<NT>(part[0], wave, splits, lane, dk[0]);
                    add_parts<NT>(part[kParts - 1], wave, splits, lane, dv[0]);
                }
            }
        }
        if (key_ok && ks == 0) {
#pragma unroll
            for (int p = 0; p < NT / 2; ++p) {
                float x[8];
                channels_of(dk[0], p, x);
                store8(d_k + (token * g.heads + head) * g.d, 32 * p + 8 * g4, g.d, x);
                channels_of(dv[0], p, x);
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
    auto query_side = [&](auto nt, auto gi, auto held) {
        bwd_dq_kernel<T, nt, gi, held><<<grid_q, kThreads, 0, stream>>>(g, kv_groups, (const T *)q, q_st, q_sh, (const T *)k, (const T *)v, kv_st, kv_sh,
                                                                        sel_idx, sel_cnt, (const T *)d_o, o_st, o_sh, lse, d_q, delta, scale);
    };
    auto key_side = [&](auto nt, auto gi, auto waves) {
        bwd_dkv_kernel<T, nt, gi, waves><<<grid_k, kThreads, 0, stream>>>(g, kv_groups, (const T *)q, q_st, q_sh, (const T *)k, (const T *)v, kv_st, kv_sh,
                                                                          sel_idx, sel_cnt, (const T *)d_o, o_st, o_sh, lse, delta, d_k, d_v, scale);
    };
    constexpr std::integral_constant<int, 0> none{};
    constexpr std::integral_constant<int, 1> one{};
    constexpr std::integral_constant<int, 2> two{};
    constexpr std::integral_constant<int, 3> three{};
    // bf16 groups in pairs where blocks have pairs of them (8 heads, d = 64, 32-token blocks, k = 14: 60.7 / 40.7 us, of which the bf16
    // products are the larger part); 16-token blocks leave a wavefront one or two groups, and pairs half empty (1 head, d = 64, k = 5,
    // in pairs 18.2 us, 15.5 one by one; 2 heads, k = 9, 25.4 / 22.1).
    const bool pairs = sizeof(T) == 2 && g.bt > 16 && g.d <= 128;        // beyond that registers spill
    // Rows short enough to be held (d <= 32), where the registers for it leave room for all workgroups, two a unit: 264 rows of 4
    // groups a wavefront 32.9 / 30.2 us; more workgroups than that would take turns.
    const int admissible = max_candidates(g, kv_groups), kept = g.topk < admissible ? g.topk : admissible, splits = 4 / row_ways(g.bt, 16);
    const int groups = (kept * ((g.bt + 15) / 16) + splits - 1) / splits;
    const int held = (int)grid_q.x <= 2 * compute_units() ? (groups <= 2 ? 1 : groups <= 4 ? 2 : 0) : 0;
    auto call = [&](auto nt) {
        if constexpr (nt == 2) {
            if (held == 1) query_side(nt, two, one);
            else if (held == 2) query_side(nt, two, two);
        }
        if (nt != 2 || held == 0) {
            if constexpr (sizeof(T) == 2 && nt <= 8) { if (pairs) query_side(nt, two, none); }
            if (!pairs) query_side(nt, one, none);
        }
        const hipError_t launched = hipGetLastError();
        if (launched != hipSuccess) return launched;
        // as many wavefronts a SIMD as fit without spilled registers: a spill of half an address to an accumulation register and half
        // to scratch memory has come back without its first half here, an address beyond all memory (tests look for spills)
        constexpr std::integral_constant<int, nt <= 2 ? 4 : nt <= 4 ? 2 : 1> waves{};
        if constexpr (sizeof(T) == 2 && nt <= 8) { if (pairs) key_side(nt, two, std::integral_constant<int, nt <= 2 ? 3 : nt <= 4 ? 2 : 1>{}); }
        // Three workgroups a unit and the column operands requested late, where two a unit with all of them in flight would take turns
        // (1584 key blocks, d = 64, float: 50.8 / 45.7 us; 440 the other way round, 22.1 / 23.4).
        if constexpr (sizeof(T) == 4 && nt == 4) { if ((int)grid_k.x > 2 * compute_units()) { key_side(nt, one, three); return hipGetLastError(); } }
        if (!pairs) key_side(nt, one, waves);
        return hipGetLastError();
    };
#define LCSA_CALL(NT) e = call(std::integral_constant<int, NT>{});
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
