// Building blocks of the general attention kernels (any head_dim <= 256, any block shape, f32 or bf16 storage):
// 16 x 16 products on the matrix cores with float operands (v_mfma_f32_16x16x4_f32: float products and accumulation;
// 157 TFLOP/s, 154 of them reached by a large float matrix product).
//
// A first-level product C[m][n] = sum_c A[m][c] B[n][c] sums over channels; both operands are rows of d channels
// ("row fragments").  bf16 rows need no conversion: v_mfma_f32_16x16x32_bf16 forms the same exact products and
// accumulates them in float.  C has its column n in lane & 15 and its rows 4 g + r, g = lane >> 4, in register r.
// That is the B-operand layout of v_mfma_f32_16x16x4_f32 with the summed index m = 4 g + r in step r: a second-level
// product sum_m X[m][ch] C[m][n] takes the accumulator as it is, and its A operand is the channels of rows 4 g + r
// ("column fragment").  Which channel a matrix row stands for is free: tile t = 2 p + e of a column fragment holds
// the channels 32 p + 2 m + e, so that a lane loads two neighbouring channels of a row at a time and owns, of the
// result, the eight consecutive channels 32 p + 8 g .. + 7 (register r of tiles 2 p, 2 p + 1: channels + 2 r, + 2 r + 1).
//
// Fragments are loaded from global memory straight into registers: a float operand serves 32 cycles of matrix work per
// 256 bytes, which the caches feed without a detour through LDS (and without barriers between wavefronts).
#pragma once
#include "lcsa_kernels.h"

namespace lcsa {
namespace fp32mma {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// A row of up to 16 NT channels, spread over the four lanes (m, g = 0..3); channels from d on are zero.
template <typename T, int NT> struct RowFrag;
template <int NT> struct RowFrag<float, NT> {
    f32x4 v[NT];                                             // chunk j: channels 16 j + 4 g .. + 3
    __device__ void load(const float *row, int d, int g) {
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int c = 16 * j + 4 * g;
            v[j] = c < d ? *(const f32x4 *)(row + c) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    // a row of a tile image: `at` uniform, offset = this lane's byte offset from it, lane_offset(g) included
    __device__ static uint32_t lane_offset(int g) { return 16 * g; }
    __device__ void load_at(const char *at, uint32_t offset) {
#pragma unroll
        for (int j = 0; j < NT; ++j) v[j] = *(const f32x4 *)(at + offset + 64 * j);
    }
    __device__ void clear() {
#pragma unroll
        for (int j = 0; j < NT; ++j) v[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // a row of d channels anywhere: those from d on repeat others until clear_beyond()
    __device__ void load_row(const float *row, int d, int g) {
#pragma unroll
        for (int j = 0; j < NT; ++j) v[j] = *(const f32x4 *)(row + min(16 * j + 4 * g, d - 4));
    }
    // channels from d on: zeros instead of what was read
    __device__ void clear_beyond(int d, int g) {
        if (d == 16 * NT) return;
#pragma unroll
        for (int j = 0; j < NT; ++j)
            if (16 * j + 4 * g >= d) v[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __device__ static f32x4 mma(const RowFrag &a, const RowFrag &b, f32x4 acc) {
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[j][e], b.v[j][e], acc, 0, 0, 0);
        return acc;
    }
};
template <int NT> struct RowFrag<__bf16, NT> {
    bf16x8 v[NT / 2];                                        // chunk j: channels 32 j + 8 g .. + 7
    __device__ void load(const __bf16 *row, int d, int g) {
#pragma unroll
        for (int j = 0; j < NT / 2; ++j) {
            const int c = 32 * j + 8 * g;
            const uint4 u = c < d ? *(const uint4 *)(row + c) : make_uint4(0, 0, 0, 0);
            v[j] = __builtin_bit_cast(bf16x8, u);
        }
    }
    __device__ void clear() {
#pragma unroll
        for (int j = 0; j < NT / 2; ++j) v[j] = __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0));
    }
    __device__ void load_row(const __bf16 *row, int d, int g) {
#pragma unroll
        for (int j = 0; j < NT / 2; ++j) v[j] = __builtin_bit_cast(bf16x8, *(const uint4 *)(row + min(32 * j + 8 * g, d - 8)));
    }
    __device__ static uint32_t lane_offset(int g) { return 16 * g; }
    __device__ void load_at(const char *at, uint32_t offset) {
#pragma unroll
        for (int j = 0; j < NT / 2; ++j) v[j] = __builtin_bit_cast(bf16x8, *(const uint4 *)(at + offset + 64 * j));
    }
    __device__ void clear_beyond(int d, int g) {
        if (d == 16 * NT) return;
#pragma unroll
        for (int j = 0; j < NT / 2; ++j)
            if (32 * j + 8 * g >= d) v[j] = __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0));
    }
    __device__ static f32x4 mma(const RowFrag &a, const RowFrag &b, f32x4 acc) {
#pragma unroll
        for (int j = 0; j < NT / 2; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v[j], b.v[j], acc, 0, 0, 0);
        return acc;
    }
};

// Second-level products of GI 16-row groups with QS sets of columns: acc[s] += X^T w[s], X being the rows of the groups.
//   load_at   row 4 g + r of group i, `at` uniform, offset = this lane's byte offset from it, lane_offset(m) included (channels
//             from d on are what follows the row: they only reach channels of the result that are not stored)
//   load_row  the same from a row of d channels anywhere
//   keep      only the first n rows of group i have a weight; the others become zeros, whatever was read
//   mma       weights between 0 and 1, or NaN; sums of others have to be looked at when they are complete, and made again in
//             mma<QS, true> where they are doubtful()
template <typename T, int NT, int GI> struct ColGroups;
template <int NT, int GI> struct ColGroups<float, NT, GI> {
    f32x2 v[GI][4][NT / 2];                                  // [group][row 4 g + r][p]: channels 32 p + 2 m, + 1
    __device__ static uint32_t lane_offset(int m) { return 8 * m; }
    __device__ void load_at(int i, int r, const char *at, uint32_t offset) {
#pragma unroll
        for (int p = 0; p < NT / 2; ++p) v[i][r][p] = *(const f32x2 *)(at + offset + 128 * p);
    }
    __device__ void clear_beyond(int, int) {}
    __device__ void load_row(int i, int r, const float *row, int d, int m) {
#pragma unroll
        for (int p = 0; p < NT / 2; ++p) v[i][r][p] = *(const f32x2 *)(row + min(32 * p + 2 * m, d - 2));
    }
    __device__ void keep(int i, int n, int g) {
        if (n >= 16) return;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int p = 0; p < NT / 2; ++p)
                if (4 * g + r >= n) v[i][r][p] = f32x2{0.f, 0.f};
    }
    __device__ static bool doubtful(const f32x4 (&)[NT]) { return false; }
    template <int QS, bool FLOAT = true> __device__ void mma(const f32x4 (&w)[QS][GI], f32x4 (&acc)[QS][NT]) const {
#pragma unroll
        for (int i = 0; i < GI; ++i)
#pragma unroll
            for (int s = 0; s < QS; ++s)
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        acc[s][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[i][r][t >> 1][t & 1], w[s][i][r], acc[s][t], 0, 0, 0);
    }
};
// bf16 rows: a float weight is the sum of three bf16 values (8 bits of its 24 each, every remainder exact), and the products
// of bf16 values are exact in v_mfma_f32_16x16x32_bf16, which takes two groups at a time: three instructions of 16 cycles in
// place of eight of 32, and fewer roundings of the accumulator.  Zero and negative pieces of a weight must not meet an infinity:
// infinities and NaN go through the float products by themselves, which leaves the bits of all other channels alone.  So do values from
// 2^16 on, because the last pieces of weights below 2^-110 fall among bf16's subnormals, which count for nothing: 2^-126 of a value is lost.
// Weights that may be anything: an infinite one leaves inf - inf behind its first piece, one close to the largest float rounds to an infinity,
// and tiny ones may all lose their last pieces.  The sums tell (doubtful()): all channels of a column are infinite or NaN, or all are below
// 2^-76, where the 2^13 terms' losses are no longer below 2^-20 of them.  In the backward that costs 0 to 3 % (8 heads, d = 64, 32-token blocks, k = 16 on a
// 24 x 44 grid 107.8 / 110.2 us); looking at the weights instead, group by group, or one loop for both kinds of product, 1 to 8 %.
template <int NT, int GI> struct ColGroups<__bf16, NT, GI> {
    static_assert(GI % 2 == 0, "groups go in pairs");
    uint32_t v[GI][4][NT / 2];
    __device__ static uint32_t lane_offset(int m) { return 4 * m; }
    __device__ void load_at(int i, int r, const char *at, uint32_t offset) {
#pragma unroll
        for (int p = 0; p < NT / 2; ++p) v[i][r][p] = *(const uint32_t *)(at + offset + 64 * p);
    }
    __device__ void load_row(int i, int r, const __bf16 *row, int d, int m) {
#pragma unroll
        for (int p = 0; p < NT / 2; ++p) v[i][r][p] = *(const uint32_t *)(row + min(32 * p + 2 * m, d - 2));
    }
    __device__ void keep(int i, int n, int g) {
        if (n >= 16) return;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int p = 0; p < NT / 2; ++p)
                if (4 * g + r >= n) v[i][r][p] = 0;
    }
    // After load_at(): zeros in the channels from d on.  What follows the last row of all, means in float, would look like large values:
    // d = 200, 400 rows of 16-token blocks, k = 4, 20 us for 16.5, the one workgroup's time that meets them.
    __device__ void clear_beyond(int d, int m) {
        if (d == 16 * NT) return;
        constexpr int first = NT == 16 ? 4 : NT / 2 - 1;     // LCSA_FOR_HEAD_DIM: all channels of the words before it exist
#pragma unroll
        for (int p = first; p < NT / 2; ++p) {
            const bool beyond = 32 * p + 2 * m >= d;
#pragma unroll
            for (int i = 0; i < GI; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (beyond) v[i][r][p] = 0;
        }
    }
    static constexpr uint32_t kLarge = 0x4780;               // bf16 of 2^16
    __device__ bool large() const {                          // wavefront-uniform
        typedef __attribute__((ext_vector_type(2))) uint16_t u16x2;
        u16x2 most = {0, 0};
#pragma unroll
        for (int i = 0; i < GI; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int p = 0; p < NT / 2; ++p)
                    most = __builtin_elementwise_max(most, __builtin_bit_cast(u16x2, v[i][r][p] & 0x7fff7fffu));
        return __ballot(most[0] >= kLarge || most[1] >= kLarge) != 0;
    }
    __device__ static bool doubtful(const f32x4 (&acc)[NT]) {      // wavefront-uniform
        uint32_t most = 0, least = 0x7fffffffu;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t bits = __float_as_uint(acc[t][r]) & 0x7fffffffu;
                most = max(most, bits);
                least = min(least, bits);
            }
        // a column's channels lie in lanes m, m + 16, m + 32, m + 48
        auto all_four = [](uint64_t lanes) { lanes &= lanes >> 32; return lanes & lanes >> 16 & 0xffffu; };
        return all_four(__ballot(least >= 0x7f800000u)) != 0 ||
               (all_four(__ballot(most < 0x19800000u)) & ~all_four(__ballot(most == 0))) != 0;
    }
    // the two weights of a word as bf16, and what they leave
    __device__ static uint32_t piece(float &a, float &b) {
        typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
        const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
        a -= __uint_as_float(w << 16);
        b -= __uint_as_float(w & 0xffff0000u);
        return w;
    }
    template <int QS, bool FLOAT = false> __device__ void mma(const f32x4 (&w)[QS][GI], f32x4 (&acc)[QS][NT]) {
        if (FLOAT || large())                                // these by themselves, and zeros in their place below
#pragma unroll
            for (int i = 0; i < GI; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        uint32_t &u = v[i][r][t >> 1];
                        const uint32_t half = t & 1 ? u & 0xffff0000u : u << 16;
                        const bool odd = FLOAT || (half & 0x7fffffffu) >= kLarge << 16;
                        if (odd) u &= t & 1 ? 0xffffu : 0xffff0000u;
#pragma unroll
                        for (int s = 0; s < QS; ++s)
                            acc[s][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(odd ? __uint_as_float(half) : 0.f, w[s][i][r], acc[s][t], 0, 0, 0);
                    }
        if constexpr (FLOAT) return;
#pragma unroll
        for (int i = 0; i < GI; i += 2) {
            bf16x8 pieces[QS][3];                            // largest first
#pragma unroll
            for (int s = 0; s < QS; ++s) {
                uint32_t x[3][4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    float a = w[s][i + (j >> 1)][2 * (j & 1)], b = w[s][i + (j >> 1)][2 * (j & 1) + 1];
#pragma unroll
                    for (int n = 0; n < 3; ++n) x[n][j] = piece(a, b);
                }
#pragma unroll
                for (int n = 0; n < 3; ++n) pieces[s][n] = __builtin_bit_cast(bf16x8, make_uint4(x[n][0], x[n][1], x[n][2], x[n][3]));
            }
#pragma unroll
            for (int p = 0; p < NT / 2; ++p) {
                bf16x8 rows[2];                              // element j: row 4 g + (j & 3) of group i + (j >> 2), of channels 32 p + 2 m, + 1
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    uint32_t x[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        x[j] = __builtin_amdgcn_perm(v[i + (j >> 1)][2 * (j & 1) + 1][p], v[i + (j >> 1)][2 * (j & 1)][p], e ? 0x07060302u : 0x05040100u);
                    rows[e] = __builtin_bit_cast(bf16x8, make_uint4(x[0], x[1], x[2], x[3]));
                }
#pragma unroll
                for (int n = 2; n >= 0; --n)
#pragma unroll
                    for (int e = 0; e < 2; ++e)
#pragma unroll
                        for (int s = 0; s < QS; ++s)
                            acc[s][2 * p + e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(rows[e], pieces[s][n], acc[s][2 * p + e], 0, 0, 0);
            }
        }
    }
};

// One group by itself: half of a bf16 instruction's sum would be empty, and taking weights apart takes as long as the float products.
template <int NT> struct ColGroups<__bf16, NT, 1> {
    uint32_t v[4][NT / 2];
    __device__ void load_row(int, int r, const __bf16 *row, int d, int m) {
#pragma unroll
        for (int p = 0; p < NT / 2; ++p) v[r][p] = *(const uint32_t *)(row + min(32 * p + 2 * m, d - 2));
    }
    __device__ void keep(int, int n, int g) {
        if (n >= 16) return;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int p = 0; p < NT / 2; ++p)
                if (4 * g + r >= n) v[r][p] = 0;
    }
    __device__ static bool doubtful(const f32x4 (&)[NT]) { return false; }
    template <int QS, bool FLOAT = true> __device__ void mma(const f32x4 (&w)[QS][1], f32x4 (&acc)[QS][NT]) const {
#pragma unroll
        for (int s = 0; s < QS; ++s)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    acc[s][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(t & 1 ? v[r][t >> 1] & 0xffff0000u : v[r][t >> 1] << 16), w[s][0][r], acc[s][t], 0, 0, 0);
    }
};

// The lane's eight consecutive channels 32 p + 8 g .. + 7 of a second-level result.
template <int NT> __device__ inline void channels_of(const f32x4 (&acc)[NT], int p, float (&out)[8]) {
#pragma unroll
    for (int r = 0; r < 4; ++r) { out[2 * r] = acc[2 * p][r]; out[2 * r + 1] = acc[2 * p + 1][r]; }
}
// Stores those of them that exist (d is a multiple of 4, of 8 for bf16); row and its stride are 16-byte aligned.
__device__ inline void store8(float *row, int c, int d, const float (&x)[8]) {
    if (c < d) *(f32x4 *)(row + c) = f32x4{x[0], x[1], x[2], x[3]};
    if (c + 4 < d) *(f32x4 *)(row + c + 4) = f32x4{x[4], x[5], x[6], x[7]};
}
__device__ inline void store8(__bf16 *row, int c, int d, const float (&x)[8]) {
    if (c >= d) return;
    bf16x8 w;
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = (__bf16)x[i];
    *(bf16x8 *)(row + c) = w;
}

// over the four lanes (m, 0..3) that share a column
__device__ inline float column_sum(float x) { x += __shfl_xor(x, 16); return x + __shfl_xor(x, 32); }
__device__ inline float column_max(float x) { x = fmaxf(x, __shfl_xor(x, 16)); return fmaxf(x, __shfl_xor(x, 32)); }

// How the four wavefronts of a workgroup share a block of n rows (n > 0) against a list of row groups: `ways` of them
// take 16-row pieces (16 * S rows each) of the block, and 4 / ways share each piece's list.
__host__ __device__ inline int row_ways(int n, int rows_per_wave) { return n > 2 * rows_per_wave ? 4 : n > rows_per_wave ? 2 : 1; }

// head_dim -> number of 16-channel tiles the kernels are built for
#define LCSA_FOR_HEAD_DIM(d, call)                                                                                    \
    if ((d) <= 32) { call(2) } else if ((d) <= 64) { call(4) } else if ((d) <= 96) { call(6) }                          \
    else if ((d) <= 128) { call(8) } else { call(16) }

} // namespace fp32mma
} // namespace lcsa
