// Backward of the block-sparse attention on the gfx950 matrix cores (bf16, d = 128, 128-token blocks).
// Same mathematics as lcsa_attn_bwd.hip (selection held fixed; Sec. 3.2 "Stage 2", eq. 1):
//     p_ij = exp(scale q_i.k_j - lse_i),  t_ij = g_i.v_j,  D_i = sum_j p_ij t_ij,  u_ij = scale p_ij (t_ij - D_i),
//     dq_i = sum_j u_ij k_j,   dk_j = sum_i u_ij q_i,   dv_j = sum_i p_ij g_i          (g = dL/do)
// with every product a v_mfma_f32_32x32x16_bf16 (float accumulation); p and u enter the second-level products
// rounded to bf16, everything else (exponentials, D, the accumulators, the results) is float.  Fixed summation
// orders, no atomics: results are reproducible bit for bit.
//
// Tiles.  A 128-token x 128-channel bf16 tile lives in LDS as 128 rows of 256 bytes, the 16-byte chunk j of row r
// at chunk position j ^ sw(r), sw(r) = the low four bits of r with their halves exchanged.  It is copied there straight
// from the raster tensor by direct-to-LDS loads (a wavefront instruction moves 4 rows: lane t lands at byte 16 t of
// them and fetches the chunk that belongs there), ahead of the computation: the query-side kernel copies a step's K and
// V rows into one of two buffers, the key-side kernel streams units of 32 rows of Q and dO through a ring.
// All products have the form C[m][n] = sum_k A[m][k] B[n][k].  Where the summed index runs along the rows of the
// tile (first level: over channels), an operand fragment is one ds_read_b128 of a row; where it runs down the
// columns (second level: over keys or queries), the fragment comes from two transposing reads (ds_read_b64_tr_b16:
// 16 lanes fetch 4 rows x 16 columns and each receives 4 consecutive rows of one column), so no transposed copy of
// a tile is ever built.  sw() spreads both kinds of read over the banks: 16 rows with distinct low bits map to 16
// distinct chunk positions, and 4 consecutive rows map to 4 distinct 64-byte positions: 64 banks of 4 bytes serve half a
// wavefront's transposing read at a time.  No conflicts of either kind (0.17 and 0.24 of the LDS index cycles with 32-byte
// positions, which 16 lanes at a time would have been content with).
//
// Operand reuse without LDS round trips: the rows fed to the matrix rows of a first-level product (S or S^T) are
// permuted (bits 2 and 3 of the row index swapped), which makes the 8 accumulator registers 8s..8s+7 of a lane
// hold 8 consecutive indices of the summed dimension of the second-level product: the accumulator, rounded to
// bf16, IS the A operand of that product.
//
//   bwd_dq_mfma_kernel    workgroup = (head, query block) or half of one, two passes over the kept key blocks:
//                         D_i = sum_j p_ij t_ij (stored in `delta`), formed from unrounded p and t in float; then u from D
//                         and dQ += u K.
//   bwd_dkv_mfma_kernel   workgroup = (head, key block).  Walks the query blocks that kept this block (ascending):
//                         dV += P^T dO, dK += U^T Q.
// Every matrix instruction takes one 1 KB operand fragment from LDS, and 64 KB of tiles per block pair come from L2 for each
// of the three passes.
//
// Paper scale (12 heads, 48 x 88 tokens, k = 32): 483 to 509 us + 464 to 482 us, by the card (632 + 668 before their copies and addresses were trimmed; as
// three kernels, D and dQ apart and dK, dV with four wavefronts, one per SIMD, 312 + 506 + 761 us).
#include "lcsa_kernels.h"
#include <utility>

namespace lcsa {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) short i16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kMaxQueryBlocks = 8192;        // more query blocks go to the float kernels.  No limit of the kernels below (they list any
                                             // number, kListed at a time); it keeps the arithmetic that callers of such sizes have had
constexpr int kLast = 256;                   // flag beside a step's number of keys: a pass over the kept blocks ends with it
constexpr int kListed = 512;                 // query blocks whose kept flags are turned into a list at a time

#define LCSA_LDS __attribute__((address_space(3)))

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
// raster token of the first token of a block; token i of the block lies rel_token(i) further on
__device__ inline int64_t block_origin(const KGeom &g, const BlockRef &b) { return raster_token(g, b.group, 0, b.by * g.th, b.bx * g.tw); }
// distance, in raster tokens, from a block's first token to its i-th valid token (valid tokens first, in
// (frame, row, column) order over the block's clipped extent); 0 beyond the valid tokens
__device__ inline int rel_token(const KGeom &g, const BlockTokens &bt, int i) {
    int ft, r, c;
    return bt.at(i, ft, r, c) ? (ft * g.H + r) * g.W + c : 0;
}

// chunk position swizzle of a tile image and the byte offset of 16-byte chunk `chunk` of row `row`
__device__ inline int sw(int row) { return ((row & 3) << 2) | ((row >> 2) & 3); }
__device__ inline int img_off(int row, int chunk) { return row * 256 + ((chunk ^ sw(row)) << 4); }
// matrix row m of a first-level product reads tile row swap23(m)
__device__ inline int swap23(int m) { return (m & 0x13) | ((m & 4) << 1) | ((m & 8) >> 1); }

// Operand fragments of a 32-row unit of a tile (`unit` = the tile's address in LDS + 8192 * the unit; tiles are 256-byte
// aligned, so every address is one XOR away from a per-lane base).
//
// Along a row: lane (n = lane & 31, half = lane >> 5) receives elements 16 ks + 8 half .. + 7 of row swap23(n).
__device__ inline int row_base(int lane) {
    const int row = swap23(lane & 31);
    return img_off(row, lane >> 5);
}
// Units start at multiples of 256 bytes and the XORs reach bits 4 to 7: unit and base are added once, and
// every fragment is one XOR further on.
__device__ inline uint32_t lds_address(const void *p) { return (uint32_t)(uintptr_t)((LCSA_LDS const unsigned char *)p); }
__device__ inline bf16x8 frag(uint32_t at, int ks) { return *(LCSA_LDS const bf16x8 *)(uintptr_t)(at ^ (ks << 5)); }
// Down a column: lane (n, half) receives column 32 nt + n, rows 16 kk + 8 half .. + 7.  A transposing read serves 16 lanes
// at a time: lane i of the 16 points at 4 elements of row (first + i / 4), columns (c16 + 4 (i % 4) ..), and receives rows
// first .. first + 3 of column c16 + i.
__device__ inline int column_base(int lane) {
    const int i = lane & 15, row = 8 * (lane >> 5) + (i >> 2), chunk = 2 * ((lane >> 4) & 1) + ((i >> 1) & 1);
    return img_off(row, chunk) + (i & 1) * 8;
}
__device__ inline bf16x8 frag_down(uint32_t at, int nt, int kk) {
    // rows + 4: four rows further, and bit 0 of sw() flips
    const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LCSA_LDS i16x4 *)(uintptr_t)((at ^ (nt << 6)) + 4096 * kk));
    const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LCSA_LDS i16x4 *)(uintptr_t)((at ^ (nt << 6) ^ 16) + 4096 * kk + 1024));
    typedef __attribute__((ext_vector_type(8))) short i16x8;
    const i16x8 both = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, both);
}
// The address in a unit; hides where it came from, so that the XORs are formed where they are used instead of kept in registers.
__device__ inline uint32_t fresh(uint32_t unit, int base) { uint32_t a = unit + base; asm volatile("" : "+v"(a)); return a; }

// B-operand fragments of the 32 rows a wavefront owns, straight from the raster tensor: lane (n, half) holds
// x[token(first + n)][16 ks + 8 half .. + 8] for ks = 0..7; rows beyond the block's valid tokens are zeros
__device__ inline void load_own_rows(const KGeom &g, const BlockRef &b, const __bf16 *__restrict__ x, int64_t st, int64_t sh, int head,
                                     int first, int lane, bf16x8 (&f)[8]) {
    const int n = lane & 31, half = lane >> 5;
    const bool ok = first + n < b.n_valid;
    const __bf16 *p = x + (block_origin(g, b) + rel_token(g, BlockTokens(g, b.vh, b.vw), first + n)) * st + (int64_t)head * sh + half * 8;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
        const uint4 u = ok ? *(const uint4 *)(p + ks * 16) : make_uint4(0, 0, 0, 0);
        f[ks] = __builtin_bit_cast(bf16x8, u);
    }
}

// ---- tile copies -------------------------------------------------------------------------------------------------
// In the query-side kernel a wavefront copies 16 rows of K and of V a step with 4 instructions per tensor; instruction i moves
// rows first + 4 i .. + 3 of the block, lane t supplying row (t >> 4), chunk position (t & 15).
// plan[] holds, for the 4 rows of a lane, the distance of the lane's 16 bytes from a whole block's first token (the
// host sends blocks that reach 4 GB or more to the float kernels); clipped blocks take theirs from a table in LDS.  Rows
// beyond the block's valid tokens are copied as zeros: their probabilities are zero, and zero times an infinity of another row
// would not be.
// byte offset of a block's i-th token from its first one
constexpr uint32_t kNoRow = 0xfffffe00u;
__device__ inline uint32_t row_offset(const KGeom &g, const BlockTokens &bt, int i, int64_t st) { return i < bt.n_valid ? (uint32_t)(rel_token(g, bt, i) * st * 2) : kNoRow; }
// One copy instruction: 64 lanes x 16 bytes from per-lane byte offsets of a scalar base to LDS bytes lds_rows + 16 lane; an
// offset of kNoRow or more brings zeros.  The load stays in flight (counted by vmcnt) until waited for; nothing else orders it.
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
__device__ inline u32x4 rows_from(const void *base) {
    const uint64_t a = (uint64_t)base;
    return u32x4{(uint32_t)a, (uint32_t)(a >> 32), kNoRow, 0x00020000u};      // addresses have 48 bits: no stride above them
}
template <int AT> __device__ inline void copy_rows_to_lds(const u32x4 &from, uint32_t offset, uint32_t lds_rows) {      // to lds_rows + AT, scalar
    asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds" :: "v"(offset), "s"(from), "s"(lds_rows), "i"(AT) : "memory", "m0", "scc");
}
// Piece i of a wavefront's copies of two tensors: rows 4 (i >> 1) .. + 3 of one or, SECOND bytes further on, the other.
template <int SECOND> __device__ inline void copy_piece_to_lds(int piece, const u32x4 &first, const u32x4 &second, uint32_t offset, uint32_t lds_rows) {
    switch (piece) {                                         // a constant where this is called
    case 0: copy_rows_to_lds<0>(first, offset, lds_rows); break;
    case 1: copy_rows_to_lds<SECOND>(second, offset, lds_rows); break;
    case 2: copy_rows_to_lds<1024>(first, offset, lds_rows); break;
    case 3: copy_rows_to_lds<SECOND + 1024>(second, offset, lds_rows); break;
    case 4: copy_rows_to_lds<2048>(first, offset, lds_rows); break;
    case 5: copy_rows_to_lds<SECOND + 2048>(second, offset, lds_rows); break;
    case 6: copy_rows_to_lds<3072>(first, offset, lds_rows); break;
    default: copy_rows_to_lds<SECOND + 3072>(second, offset, lds_rows); break;
    }
}

// A block as the loops want it: raster token of its first token, its valid tokens and how it is clipped.
// A block has one of four extents: whole, last column, last row or both clipped (0 to 3).
__device__ inline BlockTokens tokens_of_extent(const KGeom &g, int e) { return BlockTokens(g, e & 2 ? g.H - (g.ty - 1) * g.th : g.th, e & 1 ? g.W - (g.tx - 1) * g.tw : g.tw); }
__device__ inline int extent_of(const KGeom &g, const BlockRef &b) { return (b.vh < g.th) * 2 + (b.vw < g.tw); }
struct Located { int origin, valid; };                       // valid tokens | extent << 8
__device__ inline Located locate(const KGeom &g, int block) {
    const BlockRef b = block_ref(g, block);
    return {(int)block_origin(g, b), b.n_valid | extent_of(g, b) << 8};
}

// all of this wavefront's tile copies have landed; then a workgroup barrier: everybody's have, and everybody is
// done with the buffer that the next copies will overwrite
__device__ inline void tiles_ready() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
// this wavefront's tile copies have landed
__device__ inline void wait_copies() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// this wavefront's LDS writes so far are done
__device__ inline void lds_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
// a barrier for LDS traffic only: tile copies stay in flight
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Launch order.  Workgroups are dealt to the 8 XCDs round-robin, each with an L2 of its own; workgroup ids are
// mapped so that an XCD walks a contiguous run of (head, tile, frame group) items: neighbouring tiles of a head keep
// (or are kept by) nearly the same blocks, whose tiles are then found in that XCD's L2.
// `pieces` workgroups to an item, one or two, follow one another.
struct Deal { int groups, per_xcd; Quotient by_blocks, by_groups; };         // blocks = groups*nb
Deal deal(const KGeom &g, int groups, int pieces) {
    return {groups, (groups * g.nb * g.heads * pieces + 7) / 8, quotient_by(groups * g.nb), quotient_by(groups)};
}
__device__ inline bool work_item(const KGeom &g, const Deal &d, int pieces, int &head, int &block, int &piece) {
    int item = (blockIdx.x & 7) * d.per_xcd + (blockIdx.x >> 3);
    if (item >= g.heads * d.groups * g.nb * pieces) return false;
    piece = item & (pieces - 1);
    item >>= pieces - 1;
    head = d.by_blocks(item);
    const int rem = item - head * d.groups * g.nb;
    const int tile = d.by_groups(rem), grp = rem - tile * d.groups;
    block = grp * g.nb + tile;
    return true;
}

__device__ inline void zero(f32x16 &a) {
#pragma unroll
    for (int i = 0; i < 16; ++i) a[i] = 0.f;
}

// f(FIRST), f(FIRST + 1), ... with constants: what selects a register by row_value() needs them
template <int FIRST, class F, int... R> __device__ inline void in_turn(F &&f, std::integer_sequence<int, R...>) { (f(std::integral_constant<int, FIRST + R>{}), ...); }
template <int FIRST, int COUNT, class F> __device__ inline void in_turn(F &&f) { in_turn<FIRST>(f, std::make_integer_sequence<int, COUNT>{}); }

// First-level products of the 32 rows mt of two tiles with two sets of register operands, operand fragments read kAhead
// pairs ahead of the matrix instructions that use them.
constexpr int kAhead = 3, kRing = kAhead + 1;
// also(ks), ks = 0 .. 7: what goes along with the matrix instructions.
template <int SECOND, class Also>
__device__ inline void first_level(uint32_t x_unit, int base, const bf16x8 (&xf)[8], const bf16x8 (&yf)[8], f32x16 &xs, f32x16 &ys, Also &&also) {
    bf16x8 xa[kRing], ya[kRing];
    const uint32_t x_at = fresh(x_unit, base);
    auto frag_v = [](uint32_t at, int ks) { return *(LCSA_LDS const bf16x8 *)(uintptr_t)((at ^ (ks << 5)) + SECOND); };      // the same rows of the second tile
#pragma unroll
    for (int n = 0; n < kAhead; ++n) { xa[n] = frag(x_at, n); ya[n] = frag_v(x_at, n); }
    zero(xs); zero(ys);
    in_turn<0, 8>([&](auto step) {
        constexpr int ks = step;
        __builtin_amdgcn_sched_barrier(0);
        xs = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xa[ks % kRing], xf[ks], xs, 0, 0, 0);
        if constexpr (ks + kAhead < 8) {
            xa[(ks + kAhead) % kRing] = frag(x_at, ks + kAhead);
            ya[(ks + kAhead) % kRing] = frag_v(x_at, ks + kAhead);
        }
        also(step);
        __builtin_amdgcn_sched_barrier(0);
        ys = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ya[ks % kRing], yf[ks], ys, 0, 0, 0);
    });
    __builtin_amdgcn_sched_barrier(0);
}
// Keeps the work that formed a value from moving past this point.
__device__ inline void pin(bf16x8 (&v)[2]) { asm volatile("" : "+v"(v[0]), "+v"(v[1])); }
// Row fragments of a unit
__device__ inline void read_rows(uint32_t unit, int base, bf16x8 (&a)[8]) {
    const uint32_t at = fresh(unit, base);
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) a[ks] = frag(at, ks);
}
__device__ inline void first_level(uint32_t x_unit, int base, const bf16x8 (&xf)[8], f32x16 &xs) {
    bf16x8 xa[8];
    read_rows(x_unit, base, xa);
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) xs = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xa[ks], xf[ks], xs, 0, 0, 0);
}
// A value per row of a unit beside the accumulators of a first-level product: register 8 kk + j of a lane's accumulator is row
// 16 kk + 8 half + j; lane (n, half) holds the value of row 16 (n >> 3 & 1) + 8 half + (n & 7), and register r takes it from
// lane r of its row of 16 lanes (a move or an addition with row_newbcast): one register and one LDS read of four bytes a lane, where
// quads of the values took eight 16-byte reads a unit.
template <int R> __device__ inline float row_value(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x150 + R, 0xf, 0xf, true));
}
template <int R> __device__ inline float add_row(const f32x16 &x, float v) { return x[R] + row_value<R>(v); }

// ---------------------------------------------------------------------------------------------------------------
// D_i = sum_j p_ij t_ij over the kept key blocks, then once more over them for dQ += u K.  A workgroup of QG x KH wavefronts
// takes 32 QG queries of a block and walks the kept key blocks in steps of kKeys keys; wavefront w owns queries 32 (w / KH) ..
// + 31 of them and, of every step, each KH-th 32-key unit; the KH partial results of a query meet in LDS.
// Which of them when: bwd_query_form().  4 x 1 has 64 KB of tiles, so that two workgroups share a unit; 2 x 4 copies the keys
// twice for a block's queries, where units would be idle otherwise (54 items, 16 blocks a row: 75 -> 60 us).  Four wavefronts for 32 queries,
// four workgroups a block, did no better with the units that still are (0.96 at rows of up to 4 blocks, 1.00 from 16 on): a step
// is as long as one wavefront's chain of reads, products and exponentials, with or without its copies (0.97 in a timing-only build).
// What bounds it: instructions, as on the key side (457 vector and 69 matrix instructions a wavefront and block before, of which
// neither hid the other; 4.0 vector, 2.0 scalar and 1.2 LDS instructions beside each matrix one now, one issued every 7.6 cycles a
// SIMD, matrix pipe busy 0.49); paper scale 632 -> 483 us.  Tried without gain: the element-wise part of a unit beside the
// products of the next one, more operands ahead, copies spread over both units.
template <int QG, int KH>
__global__ __launch_bounds__(64 * QG * KH, 2) void bwd_dq_mfma_kernel(
    KGeom g, int kv_groups, const __bf16 *__restrict__ q, int64_t q_st, int64_t q_sh,
    const __bf16 *__restrict__ k, const __bf16 *__restrict__ v, int64_t kv_st, int64_t kv_sh,
    const int32_t *__restrict__ sel_idx, const int32_t *__restrict__ sel_cnt,
    const __bf16 *__restrict__ d_o, int64_t o_st, int64_t o_sh, const float *__restrict__ lse,
    float *__restrict__ d_q, float *__restrict__ delta, float scale, Deal items) {
    constexpr int kKeys = 16 * QG * KH, kUnits = kKeys / 32 / KH, kStepBytes = kKeys * 256;
    __shared__ __attribute__((aligned(256))) unsigned char img[2][2][kStepBytes];      // [buffer][K, V]
    __shared__ float part[KH][32 * QG];
    __shared__ uint32_t row_at[4][128];                      // byte offsets of a key block's tokens from its first one, by extent
    int qb, head, piece;
    if (!work_item(g, items, 4 / QG, head, qb, piece)) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), qg = wave % QG, kh = wave / QG, first_query = 32 * (QG * piece + qg);
    const int ql = lane & 31, half = lane >> 5;
    const int n_qb = g.q_groups * g.nb;
    const BlockRef qr = block_ref(g, qb);
    if (32 * QG * piece >= qr.n_valid) return;               // a clipped block without a second half: nothing to write
    const int64_t row = (int64_t)head * n_qb + qb;
    const int cnt = min(max(sel_cnt[row], 0), g.topk);
    const int32_t *sel = sel_idx + row * g.topk;
    const float scale_log2 = scale * kLog2e;
    const uint32_t lds_img = lds_address(&img[0][0][0]);
    k += (int64_t)head * kv_sh;
    v += (int64_t)head * kv_sh;
    // Formed once: divisions and products anew for every clipped block were a quarter of its step, 900 cycles.  Backward of 3 heads on
    // 21 x 37 tokens in (1, 8, 16) blocks, 16 kept: 84.5 -> 78.0 us, and 75.8 with a wavefront's first unit left out where it holds no key; 16 heads on
    // 21 x 45 142 -> 139, whole blocks within 0.3 % (one more barrier).
    for (int i = tid; i < 512; i += 64 * QG * KH) row_at[i >> 7][i & 127] = row_offset(g, tokens_of_extent(g, i >> 7), i & 127, kv_st);
    // this lane's rows of a whole block's step, and where they stand in row_at; its chunk of each
    const int own_row = 16 * wave + (lane >> 4);
    const BlockTokens whole_block(g, g.th, g.tw);
    uint32_t plan[4], from[4], lane_chunk[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        lane_chunk[i] = ((lane & 15) ^ sw(own_row + 4 * i)) * 16;
        plan[i] = row_offset(g, whole_block, own_row + 4 * i, kv_st) + lane_chunk[i];
    }
    // the second half of an unclipped block: 64 tokens on, which are whole rows or whole frames of the tile or half of its only row
    const uint32_t half_block = __builtin_amdgcn_readfirstlane(row_offset(g, whole_block, 64, kv_st));

    // kept blocks of this row, 64 at a time, one per lane
    Located chunk = {0, 0};
    auto refill = [&](int b0) {
        // ids outside the visible blocks must not become wild addresses
        if (b0 + lane < cnt) chunk = locate(g, min(max(sel[b0 + lane], 0), kv_groups * g.nb - 1));
    };
    // The steps follow one another through the two tile buffers, in both passes.  A step's copies, 8 instructions per
    // wavefront, go along with the first unit's products of the step before: a copy holds the issuing wavefront while the
    // memory pipeline accepts it, and all at once held everybody for 1000 to 2500 cycles a block.
    // What they need is found out a step earlier still.  The requests simply go on behind the second pass.
    u32x4 k_from, v_from;
    uint32_t copy_to = 0;
    int ask = 0, ask_half = 0, asked = 0;
    auto locate_next = [&]() {                               // returns the valid keys of the step, + kLast if it ends a pass
        if ((ask & 63) == 0 && ask_half == 0 && cnt > 64) refill(ask);
        const Located kr = {__builtin_amdgcn_readlane(chunk.origin, ask & 63), __builtin_amdgcn_readlane(chunk.valid, ask & 63)};
        const int extent = kr.valid >> 8;
        const bool whole = extent == 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) from[i] = plan[i];
        if (!whole) {
#pragma unroll
            for (int i = 0; i < 4; ++i) from[i] = row_at[extent][own_row + 64 * ask_half + 4 * i] + lane_chunk[i];
        }
        const uint64_t at = (uint64_t)(uint32_t)kr.origin * (uint32_t)(kv_st * 2) + (whole && ask_half ? half_block : 0);
        k_from = rows_from((const char *)k + at);
        v_from = rows_from((const char *)v + at);
        copy_to = __builtin_amdgcn_readfirstlane(lds_img + (asked & 1) * 2 * kStepBytes + wave * 4096);
        ++asked;
        int n = (kr.valid & 255) - 64 * ask_half;
        ask_half = kKeys == 64 && ask_half == 0 && n > 64;
        if (!ask_half && ++ask == cnt) { ask = 0; n += kLast; }
        return n;
    };
    auto copy_piece = [&](int piece) { copy_piece_to_lds<kStepBytes>(piece, k_from, v_from, from[piece >> 1], copy_to); };
    refill(0);
    lds_barrier();                                           // row_at is there
    int n_keys = 0, n_next = 0;                              // of the step at work and of the one behind it
    if (cnt > 0) {
        n_next = locate_next();
#pragma unroll
        for (int i = 0; i < 8; ++i) copy_piece(i);
    }

    // this wavefront's queries: Q and dO fragments (B operands), lse and the token to write to
    bf16x8 qf[8], gf[8];
    load_own_rows(g, qr, q, q_st, q_sh, head, first_query, lane, qf);
    load_own_rows(g, qr, d_o, o_st, o_sh, head, first_query, lane, gf);
    const bool q_ok = first_query + ql < qr.n_valid;
    const BlockTokens qt(g, qr.vh, qr.vw);
    const int64_t q_token = block_origin(g, qr) + rel_token(g, qt, first_query + ql);
    // padding queries: an infinite reference makes every probability zero
    const float l2 = q_ok ? lse[q_token * g.heads + head] * kLog2e : __builtin_inff();
    const bool wave_on = first_query < qr.n_valid;           // else only copies and barriers
    // All loads so far are waited for here, where the compiler sees it: left to itself it would wait at their first
    // use inside the loop, on every trip, and each such wait also drains the tile copies in flight (they share the counter).
    __builtin_amdgcn_s_waitcnt(0x0F70);                      // vmcnt(0)
    const int rows = row_base(lane), columns = column_base(lane);
    int n_located = cnt > 0 ? locate_next() : 0;

    // Lane = query ql; register 8 kk + j = key 16 kk + 8 half + j of a 32-key unit.  Of every step the wavefront takes unit kh if
    // that holds a key, and kh + KH if the first of the later units does.  Keys beyond the valid ones must get probability zero.
    auto mask_keys = [&](f32x16 &s, int left) {
        if (left < 32) {                                     // uniform
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if ((r >> 3) * 16 + (r & 7) + 8 * half >= left) s[r] = -__builtin_inff();
        }
    };
    auto prob = [&](float s) { return __builtin_amdgcn_exp2f(fmaf(s, scale_log2, -l2)); };

    uint32_t tiles = lds_img;
    int step = 0;
    bool last = false;
    auto begin_step = [&]() {
        tiles_ready();                                       // the step's tiles have landed; everybody is done with the other buffer
        tiles = lds_img + (step & 1) * 2 * kStepBytes;
        ++step;
        n_keys = n_next & (kLast - 1);
        last = n_next & kLast;
        n_next = n_located;
    };
    // S and T of unit kh + KH * U; the first unit's products take the copies of the next step along
    f32x16 s, t;
    auto products = [&](auto U) {
        __builtin_amdgcn_s_setprio(1);
        first_level<kStepBytes>(tiles + (kh + KH * U) * 8192, rows, qf, gf, s, t, [&](auto ks) {
            if constexpr (U == 0) copy_piece(ks);
        });
        __builtin_amdgcn_s_setprio(0);
        mask_keys(s, n_keys - 32 * (kh + KH * U));
    };
    // One pass over the steps; work(U) is given S and T of a unit.
    auto walk = [&](auto &&work) {
        if (cnt == 0) return;
        do {
            begin_step();
            if (wave_on && n_keys > 32 * kh) {               // unit kh of a clipped block may hold no key
                products(std::integral_constant<int, 0>{});
                work(std::integral_constant<int, 0>{});
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) copy_piece(i);
            }
            n_located = locate_next();
            if constexpr (kUnits == 2)
                if (wave_on && n_keys > 32 * KH) {
                    products(std::integral_constant<int, 1>{});
                    work(std::integral_constant<int, 1>{});
                }
        } while (!last);
    };

    float dsum[2] = {0.f, 0.f};                              // KH = 1: one per unit, which makes the sums those of 4 x 2
    walk([&](auto U) {
        float &sum = dsum[KH == 1 ? U : 0];
#pragma unroll
        for (int r = 0; r < 16; ++r) sum = fmaf(prob(s[r]), t[r], sum);
    });
    float D = dsum[0] + __shfl_xor(dsum[0], 32);             // the two half-waves hold the two halves of a unit's keys
    if constexpr (KH == 1) D += dsum[1] + __shfl_xor(dsum[1], 32);
    if constexpr (KH > 1) {
        if (half == 0) part[kh][32 * qg + ql] = D;
        lds_barrier();
        D = part[0][32 * qg + ql];
#pragma unroll
        for (int i = 1; i < KH; ++i) D += part[i][32 * qg + ql];
    }
    if (kh == 0 && half == 0 && q_ok) delta[q_token * g.heads + head] = D;

    f32x16 dq[4];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) zero(dq[nt]);
    const float d_scaled = D * scale;
    walk([&](auto U) {
        bf16x8 u[2], kc[kRing];
#pragma unroll
        for (int r = 0; r < 16; ++r) u[r >> 3][r & 7] = (__bf16)(prob(s[r]) * fmaf(t[r], scale, -d_scaled));
        pin(u);
        const uint32_t at_columns = fresh(tiles + (kh + KH * U) * 8192, columns);
#pragma unroll
        for (int n = 0; n < kAhead; ++n) kc[n] = frag_down(at_columns, n >> 1, n & 1);
        in_turn<0, 8>([&](auto at) {
            constexpr int n = at;
            __builtin_amdgcn_sched_barrier(0);
            dq[n >> 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(u[n & 1], kc[n % kRing], dq[n >> 1], 0, 0, 0);
            if constexpr (n + kAhead < 8) kc[(n + kAhead) % kRing] = frag_down(at_columns, (n + kAhead) >> 1, (n + kAhead) & 1);
        });
        __builtin_amdgcn_sched_barrier(0);
    });

    tiles_ready();                                           // nobody reads the tiles any more, and no copy may land later
    // The KH wavefronts of a query group: wavefront kh finishes channel groups kOut kh .. and gets the others' parts of them.
    constexpr int kOut = 4 / KH;
    float *x = (float *)&img[0][0][0];                       // [wavefront][channel group][register][lane]
    if constexpr (KH > 1) {
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
            if (nt / kOut != kh)                             // uniform
#pragma unroll
                for (int r = 0; r < 16; ++r) x[((wave * 4 + nt) * 16 + r) * 64 + lane] = dq[nt][r];
        lds_barrier();
    }
    // dq tile nt: lane = channel nt*32 + ql, register r = query row 8 (r >> 2) + 4 half + (r & 3) of this wavefront
    const int64_t origin = block_origin(g, qr);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int qi = first_query + 8 * (r >> 2) + 4 * half + (r & 3);
        if (qi < qr.n_valid) {
            float *out = d_q + ((origin + rel_token(g, qt, qi)) * g.heads + head) * 128 + ql;
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
                if (KH == 1 || nt / kOut == kh) {
                    float sum = dq[nt][r];
#pragma unroll
                    for (int i = 0; i < KH; ++i)
                        if (i != kh) sum += x[(((i * QG + qg) * 4 + nt) * 16 + r) * 64 + lane];
                    out[nt * 32] = sum;
                }
        }
    }
}

// ---------------------------------------------------------------------------------------------------------------
// Eight wavefronts, two per SIMD, in two roles: wavefront w < 4 forms S and P of its 32 keys and dV += P^T dO, wavefront
// w + 4 forms T = dO V^T of the same keys, U from T and from the P that wavefront w leaves in LDS, and dK += U^T Q.  Each
// role needs half of the register operands and accumulators, so two wavefronts fit a SIMD.
// The query rows stream through LDS in units of 32 (Q and dO rows: 16 KB), kStages of them at a time, one unit per slot and
// one barrier per slot; a role's element-wise work stands beside matrix work of its own that does not depend on it:
//     slot t   w < 4:  exponentials of S(t), P(t) -> LDS  beside  dV += P(t - 1)^T dO;   then S(t + 1)
//              w >= 4: T(t - 1);   then U(t - 1) from T(t - 1), P(t - 1)  beside  dK += U(t - 2)^T Q
// Slot t reads units t - 2 .. t + 1, and unit t + 4 is requested into the place of unit t - 3.
// What bounds it is the number of instructions: a wavefront issues one every five cycles or so, and with 64-bit address
// products, branches and a spilled operand in each slot (whose reload drained the copies in flight) a slot took 2640 cycles
// for 1024 of matrix work; it took 1840 without them (paper scale 668 -> 464 us; 6.6 vector, 2.5 scalar and 2.0
// LDS instructions beside each matrix one, one issued every 6.6 cycles a SIMD, matrix pipe busy 0.39).
constexpr int kStages = 7, kLead = kStages - 3;
constexpr int kUnitBytes = 32 * 256;
constexpr int kThreads = 512;

struct KeySideLds {
    __attribute__((aligned(256))) unsigned char img[kStages][2][kUnitBytes];      // [stage][Q, dO]
    float4 p[2][4][4][64];                                   // P on its way to the second role: [slot parity][key group][register quad][lane]
    float rows[kStages][2][32];                              // [stage][-lse log2(e), -D][query of the unit]
    uint32_t row_at[3][4][128];                              // [tokens, bytes of Q, of dO][clipped rows, columns][token of the block]: see below
    unsigned char kept_by[kListed];
    uint16_t list[4 * kListed];                              // units: 4 * query block + unit of the block
    int n_listed;
};

// Two paths of their own, loops over the lists included: with the roles side by side in one loop the compiler kept the
// accumulators twice and reloaded spilled operands in every slot.
template <bool P_ROLE>
__device__ __forceinline__ void key_side(
    KeySideLds &lds, int kb, int head, const KGeom &g, const __bf16 *__restrict__ q, int64_t q_st, int64_t q_sh,
    const __bf16 *__restrict__ kv, int64_t kv_st, int64_t kv_sh, const int32_t *__restrict__ sel_idx, const int32_t *__restrict__ sel_cnt,
    const __bf16 *__restrict__ d_o, int64_t o_st, int64_t o_sh, const float *__restrict__ lse, const float *__restrict__ delta,
    float *__restrict__ out, float scale) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), kg = wave & 3;
    const int ql = lane & 31, half = lane >> 5;
    const int n_qb = g.q_groups * g.nb;
    const BlockRef kr = block_ref(g, kb);
    const float scale_log2 = scale * kLog2e;
    const uint32_t lds_img = lds_address(&lds.img[0][0][0]);
    auto unit_at = [&](int stage, int which) { return lds_img + stage * 2 * kUnitBytes + which * kUnitBytes; };     // which: 0 = Q, 1 = dO
    q += (int64_t)head * q_sh;
    d_o += (int64_t)head * o_sh;
    // How far token i of a block lies from its first one, for the four extents a block can have (whole; last column, last row
    // or both clipped): formed once, because the divisions and 64-bit products of every unit took a third of the vector work.
    {
        const int e = tid >> 7;
        const BlockTokens bt = tokens_of_extent(g, e);
        lds.row_at[0][e][tid & 127] = (uint32_t)rel_token(g, bt, tid & 127);
        lds.row_at[1][e][tid & 127] = (uint32_t)(rel_token(g, bt, tid & 127) * q_st * 2);
        lds.row_at[2][e][tid & 127] = row_offset(g, bt, tid & 127, o_st);
    }
    const uint32_t lane_chunk = ((lane & 15) ^ sw(8 * kg + (lane >> 4))) * 16;
    const float *stat_from = (lane & 8 ? delta : lse) + head;
    const float stat_factor = lane & 8 ? -1.f : -kLog2e;
    const int stat_row = lane & 8 ? -1 : 8 * kg + (lane & 7);                    // D of a padding query is that of another one, finite or not: p is zero
    float *stat_to = &lds.rows[0][lane >> 3 & 1][8 * kg + (lane & 7)];
    const float *stat_at = &lds.rows[0][0][2 * (lane & 8) + 8 * half + (lane & 7)];
    float4 *p_to = &lds.p[0][kg][0][lane];
    const uint32_t *own_rows = &lds.row_at[1][0][8 * kg + (lane >> 4)], *stat_row_at = &lds.row_at[0][0][8 * kg + (lane & 7)];

    // this wavefront's keys: K or V fragments (B operands of the first-level products)
    bf16x8 own[8];
    load_own_rows(g, kr, kv, kv_st, kv_sh, head, 32 * kg, lane, own);
    f32x16 acc[4];                                           // dV or dK
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) zero(acc[nt]);
    const bool wave_on = 32 * kg < kr.n_valid;               // else only copies and barriers
    const int rows = row_base(lane), columns = column_base(lane);

    for (int qb0 = 0; qb0 < n_qb; qb0 += kListed) {
        // which query blocks kept this key block?  (ascending id lists)
        const int n_here = min(kListed, n_qb - qb0);
        for (int i = tid; i < n_here; i += kThreads) lds.kept_by[i] = 0;
        tiles_ready();                                       // the previous list and its units are no longer read, and no copy is in flight
        const int64_t first_row = (int64_t)head * n_qb + qb0;
        if (g.topk <= 128) {
            // all ids, eight loads of a thread in flight: with 72 rows of 32 ids one latency instead of three (12 k cycles to
            // the list, 7 k now); beyond 128 ids a row a search of the row reads less
            const int32_t *ids = sel_idx + first_row * g.topk;
            const int total = n_here * g.topk;
            for (int base = tid; base < total; base += 8 * kThreads) {
                int id[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) id[e] = base + e * kThreads < total ? ids[base + e * kThreads] : -1;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (id[e] == kb) {
                        const int i = (base + e * kThreads) / g.topk;
                        if (base + e * kThreads - i * g.topk < sel_cnt[first_row + i]) lds.kept_by[i] = 1;
                    }
            }
        } else {                                             // a binary search per row
            for (int i = tid; i < n_here; i += kThreads) {
                const int32_t *sel = sel_idx + (first_row + i) * g.topk;
                const int c = min(max(sel_cnt[first_row + i], 0), g.topk);
                int lo = 0, hi = c;
                while (lo < hi) { const int mid = (lo + hi) >> 1; if (sel[mid] < kb) lo = mid + 1; else hi = mid; }
                lds.kept_by[i] = lo < c && sel[lo] == kb;
            }
        }
        __syncthreads();
        if (wave == 0) {                                     // the kept blocks' units that hold valid queries, in order
            int n = 0;
            for (int i0 = 0; i0 < n_here; i0 += 64) {
                const int i = i0 + lane;
                const bool kept = i < n_here && lds.kept_by[i];
                const int units = kept ? (block_ref(g, qb0 + i).n_valid + 31) >> 5 : 0;
                int before = units;                          // inclusive prefix sum
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) { const int x = __shfl_up(before, off); before += lane >= off ? x : 0; }
                for (int u = 0; u < units; ++u) lds.list[n + before - units + u] = (uint16_t)(4 * i + u);
                n += __shfl(before, 63);
            }
            if (lane == 0) lds.n_listed = n;
        }
        __syncthreads();
        const int n_units = __builtin_amdgcn_readfirstlane(lds.n_listed);
        __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0), where the compiler sees it (see the query-side kernel)
        if (n_units == 0) continue;

        // Units 64 at a time, one per lane: raster token of the block's first token, and where the unit's rows start in row_at |
        // how many of them hold valid queries << 16.
        int unit_origin = 0, unit_rows = 0;
        auto refill = [&](int t) {
            if ((t & 63) == 0 && t + lane < n_units) {
                const int e = lds.list[t + lane];
                const BlockRef b = block_ref(g, qb0 + (e >> 2));
                unit_origin = (int)block_origin(g, b);
                unit_rows = extent_of(g, b) * 128 + (e & 3) * 32 | min(b.n_valid - (e & 3) * 32, 32) << 16;
            }
        };
        // Unit t on its way into stage `stage`: 8 rows of Q and of dO per wavefront of the second role (lane t supplies row
        // t >> 4 of four), four instructions.  Rows beyond the block's valid queries repeat its first one in Q (an infinity
        // there makes the gradients of the same keys NaN in any case) and are zeros in dO.
        // A unit beyond the last one is the last one again: its stage is free, and the loop has no branch that would keep the
        // scheduler from spreading a slot's work over its matrix instructions.
        u32x4 q_from, o_from;
        uint32_t row_off[4], copy_to = 0;
        auto locate_rows = [&](int t, int stage) {           // refill(t) has been called
            t = min(t, n_units - 1);
            const int origin = __builtin_amdgcn_readlane(unit_origin, t & 63), rows_of = __builtin_amdgcn_readlane(unit_rows, t & 63);
            q_from = rows_from((const char *)q + (uint64_t)(uint32_t)origin * (uint32_t)(q_st * 2));
            o_from = rows_from((const char *)d_o + (uint64_t)(uint32_t)origin * (uint32_t)(o_st * 2));
            copy_to = lds_img + stage * 2 * kUnitBytes + 8 * kg * 256;
            const uint32_t *at = own_rows + (rows_of & 0xffff);
#pragma unroll
            for (int i = 0; i < 2; ++i) { row_off[2 * i] = at[4 * i]; row_off[2 * i + 1] = at[512 + 4 * i]; }
        };
        auto copy_rows = [&](int piece) {                    // sw(8 kg + 4 i + row) = sw(8 kg + row) ^ i
            copy_piece_to_lds<kUnitBytes>(piece, q_from, o_from, row_off[piece] + (lane_chunk ^ 16 * (piece >> 1)), copy_to);
        };
        auto request_rows = [&](int t, int stage) {
            refill(t);
            locate_rows(t, stage);
#pragma unroll
            for (int i = 0; i < 4; ++i) copy_rows(i);
        };
        // lse (lanes 0..7) and D (lanes 8..15) of 8 rows per wavefront of the first role: an ordinary load, stored to the
        // stage a slot later.  (As direct-to-LDS loads of single dwords these made every slot twice as long.)  Stored as the
        // kernel uses them, -lse log2(e) and -D; padding queries get an infinite lse: probability zero.
        // Lanes 16.. repeat lanes 0..15.
        float stat = 0.f;
        int stat_rel = 0, stat_origin = 0, stat_rows = 0, rows_held = 0;
        auto locate_stats = [&](int t) {                     // refill(t) has been called
            t = min(t, n_units - 1);
            stat_origin = __builtin_amdgcn_readlane(unit_origin, t & 63);
            const int rows_of = __builtin_amdgcn_readlane(unit_rows, t & 63);
            stat_rows = rows_of >> 16;
            stat_rel = (int)stat_row_at[rows_of & 0xffff];
        };
        auto request_stats = [&]() {                         // of the unit located last
            stat = stat_from[(int64_t)(stat_origin + stat_rel) * g.heads];
            rows_held = stat_rows;
        };
        auto store_stats = [&](int stage) { stat_to[stage * 64] = stat_row >= rows_held ? -__builtin_inff() : stat * stat_factor; };
        // what row_value() hands to this lane's accumulator registers
        auto row_stat = [&](int stage, int which) { return stat_at[stage * 64 + which * 32]; };
        // The second role's copies of all units but the two requested last have landed, and every wavefront is done with the slot.
        auto end_of_slot = [&]() {
            if constexpr (P_ROLE) asm volatile("s_barrier" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(8)\n\ts_barrier" ::: "memory");
        };
        auto wrap = [](int stage) { return stage >= kStages ? stage - kStages : stage; };

        if constexpr (P_ROLE) {
            refill(0);
            for (int t = 0; t < 2; ++t) { locate_stats(t); request_stats(); store_stats(t); }
            locate_stats(2); request_stats();
            locate_stats(3);
            lds_done();
        } else {
            for (int t = 0; t < kLead; ++t) request_rows(t, t);
        }
        end_of_slot();                                       // units 0 and 1 are in LDS

        // The slots are alike; what a first or last one would take from a unit that does not exist is either multiplied by
        // the zeros p and u start with (dO rows: zeros too; Q rows: of unit 0 instead) or never used.
        // Lane = key ql of this wavefront; register 8 kk + j = query 16 kk + 8 half + j of the unit.
        bf16x8 w[2];                                         // P(t - 1) or U(t - 2)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) w[i][j] = (__bf16)0.f;
        f32x16 x;                                            // S(t) or T(t - 1)
        zero(x);
        if (!wave_on) {
#pragma unroll 1
            for (int t = 0, now = 0; t < n_units + 2; ++t, now = wrap(now + 1)) {
                if constexpr (P_ROLE) { refill(t + 4); store_stats(wrap(now + 2)); request_stats(); locate_stats(t + 4); lds_done(); }
                else request_rows(t + kLead, wrap(now + kLead));
                end_of_slot();
            }
        } else if constexpr (P_ROLE) {
            float l_now = row_stat(0, 0);
            first_level(unit_at(0, 0), rows, own, x);
            bf16x8 cols[8];                                  // of unit t - 1
#pragma unroll
            for (int n = 0; n < 8; ++n)
#pragma unroll
                for (int j = 0; j < 8; ++j) cols[n][j] = (__bf16)0.f;
#pragma unroll 1
            for (int t = 0, now = 0; t <= n_units; ++t, now = wrap(now + 1)) {
                refill(t + 4);
                bf16x8 xa[8], wn[2];
                const uint32_t next = fresh(unit_at(wrap(now + 1), 0), rows);
                float l_next;
                in_turn<0, 8>([&](auto step) {
                    constexpr int n = step;
                    __builtin_amdgcn_sched_barrier(0);
                    acc[n >> 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[n & 1], cols[n], acc[n >> 1], 0, 0, 0);
                    xa[n] = frag(next, n);
                    if (n == 0) l_next = row_stat(wrap(now + 1), 0);
                    in_turn<2 * n, 2>([&](auto reg) {
                        constexpr int e = reg;
                        x[e] = __builtin_amdgcn_exp2f(fmaf(x[e], scale_log2, row_value<e>(l_now)));
                        wn[e >> 3][e & 7] = (__bf16)x[e];
                    });
                    if (n & 1) p_to[t & 1 ? 1024 + 64 * (n >> 1) : 64 * (n >> 1)] = make_float4(x[2 * n - 2], x[2 * n - 1], x[2 * n], x[2 * n + 1]);
                    if (n == 4) store_stats(wrap(now + 2));
                    if (n == 5) request_stats();
                    if (n == 6) locate_stats(t + 4);
                });
                pin(wn);
                asm volatile("" ::: "memory");               // P(t) and the row values are written before the column reads below
                const uint32_t down = fresh(unit_at(now, 1), columns);
                zero(x);
#pragma unroll
                for (int n = 0; n < 8; ++n) {
                    __builtin_amdgcn_sched_barrier(0);
                    x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xa[n], own[n], x, 0, 0, 0);
                    cols[n] = frag_down(down, n >> 1, n & 1);      // for the next slot: these need not wait for the barrier
                }
                __builtin_amdgcn_sched_barrier(0);
                w[0] = wn[0]; w[1] = wn[1];
                l_now = l_next;
                // LDS operations of a wavefront end in order, and 16 of them (the column reads) follow the writes of P(t) and of
                // the row values: with at most 14 in flight both writes are done.  (The counter has four bits: 15 is no wait.)
                asm volatile("s_waitcnt lgkmcnt(14)" ::: "memory");
                end_of_slot();
            }
            end_of_slot();
        } else {
            // T(t - 1) first, then U(t - 1) beside dK: while the first role's wavefront of the SIMD is at its exponentials this
            // one has matrix work only, and the other way round.
            bf16x8 cols[8], xa[8];                           // of unit t - 2, of unit t - 1
            read_rows(unit_at(0, 1), rows, xa);
            request_rows(kLead, kLead);
            end_of_slot();
#pragma unroll 1
            for (int t = 1, now = 1, last = 0, before = 0; t < n_units + 2; ++t, before = last, last = now, now = wrap(now + 1)) {
                refill(t + kLead);
                bf16x8 wn[2];
                float4 p4[4];
                float d_last;
                const float4 *p_from = p_to + (t & 1 ? 0 : 1024);
                const uint32_t down = fresh(unit_at(before, 0), columns);
                zero(x);
                in_turn<0, 8>([&](auto step) {
                    constexpr int n = step;
                    __builtin_amdgcn_sched_barrier(0);
                    x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xa[n], own[n], x, 0, 0, 0);
                    cols[n] = frag_down(down, n >> 1, n & 1);
                    if (n == 0) locate_rows(t + kLead, wrap(now + kLead));
                    if constexpr (n >= 4) p4[n - 4] = p_from[64 * (n - 4)];
                    if (n == 4) d_last = row_stat(last, 1);
                    if (n == 3 || n == 6) copy_rows(n / 6);
                });
                const uint32_t across = fresh(unit_at(now, 1), rows);
                in_turn<0, 8>([&](auto step) {
                    constexpr int n = step;
                    __builtin_amdgcn_sched_barrier(0);
                    acc[n >> 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[n & 1], cols[n], acc[n >> 1], 0, 0, 0);
                    xa[n] = frag(across, n);
                    if constexpr (n >= 2 && n < 6)
                        in_turn<4 * (n - 2), 4>([&](auto reg) { constexpr int e = reg; wn[e >> 3][e & 7] = (__bf16)((&p4[e >> 2].x)[e & 3] * add_row<e>(x, d_last)); });
                    if (n == 1 || n == 6) copy_rows(2 + n / 6);
                });
                pin(wn);
                __builtin_amdgcn_sched_barrier(0);
                w[0] = wn[0]; w[1] = wn[1];
                end_of_slot();
            }
        }
    }
    wait_copies();                                           // none may land after the workgroup has gone
    const float factor = P_ROLE ? 1.f : scale;               // u enters dK without it
    const BlockTokens kt(g, kr.vh, kr.vw);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int ki = 32 * kg + 8 * (r >> 2) + 4 * half + (r & 3);
        if (ki < kr.n_valid) {
            const int64_t o = ((block_origin(g, kr) + rel_token(g, kt, ki)) * g.heads + head) * 128 + ql;
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) out[o + nt * 32] = acc[nt][r] * factor;
        }
    }
}

__global__ __launch_bounds__(512, 2) void bwd_dkv_mfma_kernel(
    KGeom g, int kv_groups, const __bf16 *__restrict__ q, int64_t q_st, int64_t q_sh,
    const __bf16 *__restrict__ k, const __bf16 *__restrict__ v, int64_t kv_st, int64_t kv_sh,
    const int32_t *__restrict__ sel_idx, const int32_t *__restrict__ sel_cnt,
    const __bf16 *__restrict__ d_o, int64_t o_st, int64_t o_sh, const float *__restrict__ lse, const float *__restrict__ delta,
    float *__restrict__ d_k, float *__restrict__ d_v, float scale, Deal items) {
    __shared__ KeySideLds lds;
    int kb, head, whole;
    if (!work_item(g, items, 1, head, kb, whole)) return;
    if (__builtin_amdgcn_readfirstlane(threadIdx.x) < 256)
        key_side<true>(lds, kb, head, g, q, q_st, q_sh, k, kv_st, kv_sh, sel_idx, sel_cnt, d_o, o_st, o_sh, lse, delta, d_v, scale);
    else
        key_side<false>(lds, kb, head, g, q, q_st, q_sh, v, kv_st, kv_sh, sel_idx, sel_cnt, d_o, o_st, o_sh, lse, delta, d_k, scale);
}

} // namespace

bool attn_bwd_mfma_supported(const KGeom &g, int64_t q_st, int64_t kv_st, int64_t o_st) {
    // byte offsets inside a block are 32-bit, up to kNoRow, and so is the distance of two tokens (also where a block has only one)
    const int64_t last = ((int64_t)(g.tt - 1) * g.H + min(g.th, g.H) - 1) * g.W + min(g.tw, g.W) - 1;
    for (const int64_t st : {q_st, kv_st, o_st})
        if (st > ((int64_t)kNoRow - 256) / 2 / (last > 1 ? last : 1)) return false;
    return g.bf16 && g.d == 128 && g.bt == 128 && g.q_groups * g.nb <= kMaxQueryBlocks;
}

hipError_t launch_attn_bwd_mfma(const KGeom &g, int kv_groups, const void *q, int64_t q_st, int64_t q_sh,
                                const void *k, const void *v, int64_t kv_st, int64_t kv_sh,
                                const int32_t *sel_idx, const int32_t *sel_cnt,
                                const void *d_o, int64_t o_st, int64_t o_sh, const float *lse,
                                float *d_q, float *d_k, float *d_v, float *delta, float scale, hipStream_t stream) {
    const Deal keys = deal(g, kv_groups, 1);
    const int items = g.q_groups * g.nb * g.heads;
    auto query_side = [&](auto QG, auto KH) {
        const Deal to = deal(g, g.q_groups, 4 / QG);
        bwd_dq_mfma_kernel<QG, KH><<<dim3(to.per_xcd * 8), 64 * QG * KH, 0, stream>>>(
            g, kv_groups, (const __bf16 *)q, q_st, q_sh, (const __bf16 *)k, (const __bf16 *)v, kv_st, kv_sh, sel_idx, sel_cnt,
            (const __bf16 *)d_o, o_st, o_sh, lse, d_q, delta, scale, to);
    };
    constexpr std::integral_constant<int, 1> one{};
    constexpr std::integral_constant<int, 2> two{};
    constexpr std::integral_constant<int, 4> four{};
    const int admissible = max_candidates(g, kv_groups);
    const BwdQueryForm form = bwd_query_form(items, compute_units(), g.topk < admissible ? g.topk : admissible);
    if (form == kBwd4x1) query_side(four, one);
    else if (form == kBwd4x2) query_side(four, two);
    else query_side(two, four);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    bwd_dkv_mfma_kernel<<<dim3(keys.per_xcd * 8), 512, 0, stream>>>(g, kv_groups, (const __bf16 *)q, q_st, q_sh, (const __bf16 *)k, (const __bf16 *)v,
                                                                 kv_st, kv_sh, sel_idx, sel_cnt, (const __bf16 *)d_o, o_st, o_sh, lse, delta,
                                                                 d_k, d_v, scale, keys);
    return hipGetLastError();
}

} // namespace lcsa
