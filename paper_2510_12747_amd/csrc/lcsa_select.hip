// Block selection: coarse block-to-block scores (Sec. 3.2) restricted to the spatial local
// window (Sec. 3.3, Fig. 3), then the per-row top-k with ties going to the lower key-block
// id.  One workgroup owns one (head, query block) row: four lanes share each dot product
// against an admissible key block, then one wavefront parts the k largest scores from the rest by a
// bitwise search over order-preserving integer keys with ballot/popcount and emits the kept ids
// in ascending order with ballot prefix counts.  No sort, no atomics, fully deterministic.
#include "lcsa_block_score.h"
#include "lcsa_kernels.h"
#include "lcsa_pool.h"

namespace lcsa {
namespace {

// Monotone map float -> uint32 (larger float = larger key); -0 is folded into +0 first so
// that equal floats always get equal keys.
__device__ inline uint32_t order_key(float s) {
    uint32_t u = __float_as_uint(s + 0.0f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ inline float key_to_float(uint32_t key) {
    return __uint_as_float((key & 0x80000000u) ? (key ^ 0x80000000u) : ~key);
}

__device__ inline int wave_count(bool p) { return __popcll(__ballot(p)); }

constexpr int kSelThreads = 256;
static_assert(kSelThreads == pooling::kThreads, "the fused kernel pools with the pooling kernel's thread layout");

// VEC = 0: the pooled queries are given.  VEC = 8 (bf16) or 4 (f32): the kernel first pools its own query
// block from q, exactly as the pooling kernel would (same code, same summation order), and also writes
// the mean to pooled_out: one launch and one pass over Q less per layer call.
template <int VEC>
__global__ __launch_bounds__(kSelThreads) void select_kernel(KGeom g, KCache c, const float *__restrict__ pooled_q,
                                                             const char *__restrict__ x, int64_t st, int64_t sh,
                                                             float *__restrict__ pooled_out,
                                                             int32_t *__restrict__ sel_idx, int32_t *__restrict__ sel_cnt,
                                                             float *__restrict__ gap) {
    extern __shared__ __align__(16) float smem[];
    float *qs = smem;                                  // [d] pooled query of this row
    uint32_t *keys = (uint32_t *)(smem + g.d);         // [n] ordered keys of the admissible blocks (after pooling's partial sums)
    const int qb = g.by_heads(blockIdx.x), head = blockIdx.x - qb * g.heads;     // head-fastest, like the pooling kernels
    const int tid = threadIdx.x, lane = tid & 63;
    const int n_qb = g.q_groups * g.nb;
    const int tile = qb - g.by_nb(qb) * g.nb, by = g.by_tx(tile), bx = tile - by * g.tx;
    int y0, y1, x0, x1;
    axis_window(by, g.th, g.ty, g.rh, g.wmode, &y0, &y1);
    axis_window(bx, g.tw, g.tx, g.rw, g.wmode, &x0, &x1);
    const int wx = x1 - x0, nwin = (y1 - y0) * wx;
    const int n = c.valid * nwin;                      // admissible key blocks, in ascending id order
    const int64_t row = (int64_t)head * n_qb + qb;
    const int start = ring_start(c, g);                // requested here, needed after the pooling

    if constexpr (VEC == 0) {
        for (int i = tid; i < g.d; i += kSelThreads) qs[i] = pooled_q[row * g.d + i];
    } else {
        float *red = smem + g.d;                       // [kSelThreads * VEC] partial sums per row group
        const pooling::TileRef t = pooling::tile_ref(g, qb);
        const int lpr = g.d / VEC, rows_par = kSelThreads / lpr;
        const int rg = tid / lpr, j = tid - rg * lpr;
        float acc[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
        if (rg < rows_par) {
            pooling::accumulate_block<VEC>(g, t, x, st, sh, head, rg, j, rows_par, acc);
#pragma unroll
            for (int e = 0; e < VEC; ++e) red[rg * g.d + j * VEC + e] = acc[e];
        }
        __syncthreads();
        const int count = g.tt * t.vh * t.vw;
        for (int ch = tid; ch < g.d; ch += kSelThreads) {
            float sum = 0.f;
            for (int r = 0; r < rows_par; ++r) sum += red[r * g.d + ch];
            const float mean = sum / (float)count;
            qs[ch] = mean;
            pooled_out[row * g.d + ch] = mean;
        }
    }
    __syncthreads();

    // candidate ci -> (visible group f, tile t); key-block id = f*nb + t grows with ci
    auto tile_of = [&](int ci, int &f) {
        f = ci / nwin;
        int w = ci - f * nwin, wy = w / wx;
        return (y0 + wy) * g.tx + x0 + (w - wy * wx);
    };

    // ---- scores: four lanes per candidate
    {
        const int part = tid & 3, n4 = g.d / 4;
        for (int ci = tid >> 2; ci < ((n + 63) & ~63); ci += kSelThreads / 4) {
            float s = 0.f;
            if (ci < n) {
                int f;
                const int t = tile_of(ci, f);
                const int slot = cache_slot(c, g, start, head, f);
                const float4 *kr = (const float4 *)(c.pooled + (((int64_t)head * g.cap + slot) * g.nb + t) * g.d);
                s = quarter_score(qs, kr, part, n4);
            }
            s += __shfl_xor(s, 1);
            s += __shfl_xor(s, 2);
            if (ci < n && part == 0) keys[ci] = order_key(s);
        }
    }
    __syncthreads();
    if (tid >= 64) return;                             // the selection itself is one wavefront's work

    int32_t *out = sel_idx + row * g.topk;
    const int k = g.topk;
    const uint64_t lt_mask = (1ull << lane) - 1ull;
    int written = 0;
    float row_gap = __builtin_inff();

    if (n <= k) {
        for (int base = 0; base < n; base += 64) {
            const int ci = base + lane;
            if (ci < n) { int f; const int t = tile_of(ci, f); out[ci] = f * g.nb + t; }
        }
        written = n;
    } else {
        // Keys of the row, PER_LANE in registers of each lane; PER_LANE = 0: read from LDS each time.  The search looks at every
        // key up to 32 times, one look waiting for the other: from LDS that is a round trip per 64 keys each time (a layer
        // call with 504 candidates a row: 329 us, 313 with 8 keys per lane; up to 128 candidates were in registers before).
        // 512 candidates cover, with 6 cached frames of 8 x 16-token tiles, windows of up to 85 tiles (9 x 9: radius 32 by 64);
        // rows beyond that (12 cached frames and a 9 x 5 window: 540) take the LDS loop, as all beyond 128 did.
        uint32_t T = 0, below = 0, above = ~0u;          // bound of the kept keys; largest key < T (0 if none; keys of finite floats are > 0), least >= T
        int n_ge = 0;
        auto search = [&](auto per_lane) {
            constexpr int PER_LANE = decltype(per_lane)::value;
            uint32_t held[PER_LANE ? PER_LANE : 1];
            auto each = [&](auto &&look) {               // look(candidate, key), 64 ascending candidates at a time
                if constexpr (PER_LANE > 0) {
#pragma unroll
                    for (int i = 0; i < PER_LANE; ++i) look(i * 64 + lane, held[i]);
                } else {
                    for (int ci = lane; ci - lane < n; ci += 64) look(ci, ci < n ? keys[ci] : 0u);
                }
            };
            if constexpr (PER_LANE > 0) {
#pragma unroll
                for (int i = 0; i < PER_LANE; ++i) held[i] = i * 64 + lane < n ? keys[i * 64 + lane] : 0u;
            }
            // A bound with exactly k keys >= it, or, if ties leave none, the k-th largest key: bitwise from the top, trial > 0, so
            // the zeros beyond n never count.  It ends at the first bound that parts k keys from the rest (after
            // about 9 + log2(n) bits instead of 32 for keys spread like a normal variable; 4 heads on 48 x 88 with 24 cached frames,
            // most rows from LDS: 15.9 -> 14.8 us); unrolled, or what each step adds in scalar code costs short rows more than the steps left out give.
#pragma unroll
            for (int bit = 31; bit >= 0; --bit) {
                const uint32_t trial = T | (1u << bit);
                int cnt = 0;
                each([&](int, uint32_t key) { cnt += wave_count(key >= trial); });
                if (cnt >= k) T = trial;
                if (cnt == k) break;
            }
            int n_gt = 0;
            each([&](int ci, uint32_t key) {
                n_gt += wave_count(ci < n && key > T);
                n_ge += wave_count(ci < n && key >= T);
                if (ci < n && key < T && key > below) below = key;
                if (ci < n && key >= T && key < above) above = key;
            });
            const int need = k - n_gt;                   // how many of the blocks tied at T are kept: none if the search ended early and T is no key
            int eq_seen = 0;
            each([&](int ci, uint32_t key) {
                const bool gt = ci < n && key > T, eq = ci < n && key == T;
                const uint64_t eq_mask = __ballot(eq);
                const bool keep = gt || (eq && eq_seen + __popcll(eq_mask & lt_mask) < need);
                const uint64_t keep_mask = __ballot(keep);
                if (keep) { int f; const int t = tile_of(ci, f); out[written + __popcll(keep_mask & lt_mask)] = f * g.nb + t; }
                written += __popcll(keep_mask);
                eq_seen += __popcll(eq_mask);
            });
        };
        if (n <= 128) search(std::integral_constant<int, 2>{});
        else if (n <= 256) search(std::integral_constant<int, 4>{});
        else if (n <= 512) search(std::integral_constant<int, 8>{});
        else search(std::integral_constant<int, 0>{});
        if (gap) {
            if (n_ge > k) row_gap = 0.f;                 // the search went to the last bit: T is a key, and tied
            else {
                for (int off = 32; off > 0; off >>= 1) {
                    const uint32_t o = __shfl_xor(below, off);
                    below = o > below ? o : below;
                    const uint32_t a = __shfl_xor(above, off);
                    above = a < above ? a : above;
                }
                row_gap = key_to_float(above) - key_to_float(below);
            }
        }
    }
    for (int i = written + lane; i < k; i += 64) out[i] = -1;
    if (lane == 0) {
        sel_cnt[row] = written;
        if (gap) gap[row] = row_gap;
    }
}

} // namespace

hipError_t launch_select(const KGeom &g, const KCache &c, const float *pooled_q,
                         int32_t *sel_idx, int32_t *sel_cnt, float *gap, int max_cand, hipStream_t stream) {
    dim3 grid(g.q_groups * g.nb * g.heads);
    const size_t lds = (size_t)(g.d + max_cand) * sizeof(float);
    select_kernel<0><<<grid, kSelThreads, lds, stream>>>(g, c, pooled_q, nullptr, 0, 0, nullptr, sel_idx, sel_cnt, gap);
    return hipGetLastError();
}

hipError_t launch_pool_select(const KGeom &g, const KCache &c, const void *q, int64_t q_st, int64_t q_sh, float *pooled_q,
                              int32_t *sel_idx, int32_t *sel_cnt, float *gap, int max_cand, hipStream_t stream) {
    dim3 grid(g.q_groups * g.nb * g.heads);
    const int vec = g.bf16 ? 8 : 4;
    const size_t lds = (size_t)(g.d + (max_cand > kSelThreads * vec ? max_cand : kSelThreads * vec)) * sizeof(float);
    if (g.bf16)
        select_kernel<8><<<grid, kSelThreads, lds, stream>>>(g, c, nullptr, (const char *)q, q_st, q_sh, pooled_q, sel_idx, sel_cnt, gap);
    else
        select_kernel<4><<<grid, kSelThreads, lds, stream>>>(g, c, nullptr, (const char *)q, q_st, q_sh, pooled_q, sel_idx, sel_cnt, gap);
    return hipGetLastError();
}

} // namespace lcsa
