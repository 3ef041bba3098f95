// Block-sparse flash attention on the gfx950 matrix cores (bf16, d = 128, 128-token blocks).
//
// Work item = one (head, query block): 128 query rows against its selected key blocks.
// A workgroup has 8 wavefronts = two GROUPS of 4, each with its own K and V tile buffers in LDS;
// wavefront w of a group owns query rows 32w .. 32w+31.  By the size of the launch (lcsa_attn_form.h)
// each group owns one work item (the two query blocks of the same spatial tile, which share their
// window), or both share one item's selected blocks, or one group owns the only item.  Launches of
// at most half an item per compute unit take a kernel of their own (attn_mfma_few_kernel), if their
// blocks hold more than 64 tokens in the mean.
//
// Per selected key block a group runs
//     QK   S^T = K Q^T        v_mfma_f32_32x32x16_bf16  (keys on the row axis, queries on lanes)
//     SM   online softmax     VALU, fp32 (eq. 1; scale folded into exp2; lazily updated reference)
//     PV   O^T += V^T P^T     v_mfma_f32_32x32x16_f16   (channels on the row axis, queries on lanes)
// as four phases (two matrix, two vector), every phase ending in a workgroup barrier, and the
// two groups run two phases apart: each SIMD holds one wavefront of either group, so while one
// issues matrix instructions the other issues vector instructions.  Left to themselves two
// independent wavefronts fall into step (both want the matrix pipe, then both want the vector
// pipe); the fixed stagger keeps the two pipes busy together.
//
// A block clipped by the grid border holds its valid tokens first: only the 32-key groups (and
// 32-query wavefronts) that contain valid tokens are computed, and at most one 16-key fragment
// per block needs a mask.
//
// Transposed products put every query column in one lane (and its partner lane^32): the
// softmax statistics need one cross-lane exchange per block, the rescale factor of O is a
// per-lane scalar, and the accumulator of S^T is already in B-operand layout for the second
// product.  K rows fed to MFMA row m are permuted (bits 2 and 3 of m swapped) so that
// accumulator registers 8s..8s+7 of a lane hold 8 consecutive keys: the P fragment for
// k-step s is those registers packed, the matching V^T fragment one 16-byte LDS read.
//
// The second product runs in IEEE half (same matrix-core rate as bf16): probabilities lie in
// [0,1] and need mantissa rather than range, which cuts the kernel's dominant rounding error
// (bf16 P) by 8x; V was converted to half, exactly for all normal-range values, at append time.
//
// K and V tiles are 32 KB byte-for-byte LDS images prepared by the cache append (16-byte
// chunk j of row r at chunk position j ^ (r & 15): conflict-free ds_read_b128 operand reads)
// and are streamed in with direct-to-LDS loads that stay in flight across barriers:
// V(i) arrives during QK(i)+SM(i), K(i+1) during SM(i)+PV(i).
#include "lcsa_kernels.h"

namespace lcsa {

// Built with -DLCSA_TIMERS=1 (only the benchmark's measurement aids do that) the kernel also records, per
// workgroup, the shader-clock counter and the constant 100 MHz counter at entry, before and after the main
// loop and at exit (-DLCSA_TIMERS=2: at entry and exit only; the inner stamps perturb the loop's schedule
// measurably), plus the hardware id of the compute unit: 10 x uint64 per workgroup at *d_attn_timers
// (a device-side pointer variable rather than a kernel argument, which would cost scalar registers for the
// whole kernel; null = no stamps).
#ifdef LCSA_TIMERS
__device__ uint64_t *d_attn_timers;
hipError_t set_attn_timers(uint64_t *device_buffer) {
    return hipMemcpyToSymbol(HIP_SYMBOL(d_attn_timers), &device_buffer, sizeof(device_buffer));
}
#define LCSA_STAMP(slot)                                                                                     \
    if ((LCSA_TIMERS == 1 || (slot) == 0 || (slot) == 3) && threadIdx.x == 0) {                                                                                  \
        uint64_t *timers = d_attn_timers;                                                                    \
        if (timers) {                                                                                        \
            timers[(size_t)blockIdx.x * 10 + 2 * (slot)] = __builtin_readcyclecounter();                     \
            timers[(size_t)blockIdx.x * 10 + 2 * (slot) + 1] = __builtin_amdgcn_s_memrealtime();             \
            if ((slot) == 0)      /* HW_ID (compute unit, shader engine) and, above it, XCC_ID (which of the 8 dies) */ \
                timers[(size_t)blockIdx.x * 10 + 8] = (uint64_t)__builtin_amdgcn_s_getreg(4 | (31 << 11)) |  \
                                                      (uint64_t)__builtin_amdgcn_s_getreg(20 | (31 << 11)) << 32; \
        }                                                                                                    \
    }
#else
#define LCSA_STAMP(slot)
#endif

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int kTileBytes = 128 * 256;
constexpr int kAhead = 3;            // operand fragments in flight ahead of the matrix instruction using them
constexpr int kRing = kAhead + 1;
constexpr int kSplit = 4;            // softmax fragments (of 8) done in the first vector phase; the rest in the second
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

#define LCSA_LDS __attribute__((address_space(3)))

// Synchronisation inside the main loop is inline assembly on purpose.  The tile copies are
// direct-to-LDS loads that stay in flight across workgroup barriers; __syncthreads() and the
// compiler's own bookkeeping for LDS-writing loads would drain them (vmcnt(0)) at every
// barrier and before unrelated LDS reads, which serialises copy and compute.  Arrival of a
// tile is established by an explicit vmcnt wait; the barrier itself only orders LDS traffic.
__device__ inline void stage_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
// wait until at most N of this wavefront's vector-memory loads are still in flight
__device__ inline void wait_vm0() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ inline void wait_vm8() { asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); }

// One of the 8 copy instructions of a wavefront's quarter tile: 64 lanes x 16 bytes, lane t lands at
// LDS address dst + 1024*piece + 16*t (M0 + immediate + 16*t).  The source is scalar base (the tile, wavefront-uniform) +
// per-lane byte offset `voff` (wavefront quarter + 16*lane, loop invariant) + an immediate, so the
// copies cost no vector arithmetic.  A load to LDS must not be the instruction right behind the write of M0 (one wait state,
// which the compiler does not put into inline assembly).
__device__ inline void copy_piece_to_lds(const char *tile, uint32_t voff, uint32_t dst, int piece) {
    const char *base = tile + (piece >> 2) * 4096;        // immediates reach 4095 bytes
    const uint32_t m0v = dst + (piece >> 2) * 4096;        // the immediate offset is added to the LDS address too
    switch (piece & 3) {
    case 0: asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" :: "v"(voff), "s"(base), "s"(m0v) : "memory", "m0"); break;
    case 1: asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:1024" :: "v"(voff), "s"(base), "s"(m0v) : "memory", "m0"); break;
    case 2: asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:2048" :: "v"(voff), "s"(base), "s"(m0v) : "memory", "m0"); break;
    default: asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:3072" :: "v"(voff), "s"(base), "s"(m0v) : "memory", "m0"); break;
    }
}

// exp2 of 8 scores of one accumulator (registers first..first+7 = 8 consecutive keys), rounded to
// half for the second matrix product; the row sum is kept in float.  (Plain adds on purpose: the
// dot-product instructions v_dot2* run on the matrix pipeline and do not overlap with MFMAs of the
// other wavefront on the SIMD, ordinary vector instructions do.)
__device__ inline void softmax_fragment(const f32x16 &sc, int first, float scale_log2, float m, float &l, f16x8 &out) {
#pragma unroll
    for (int j = 0; j < 8; j += 2) {
        const float p0 = __builtin_amdgcn_exp2f(fmaf(sc[first + j], scale_log2, -m));
        const float p1 = __builtin_amdgcn_exp2f(fmaf(sc[first + j + 1], scale_log2, -m));
        l += p0 + p1;
        out[j] = (_Float16)p0;
        out[j + 1] = (_Float16)p1;
    }
}

// Largest score of each query column over the block's first nf 16-key fragments (both lanes of a
// query agree); nf is wavefront-uniform.
__device__ inline float block_row_max(const f32x16 (&sc)[4], int nf) {
    float mx = -__builtin_inff();
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
        if (ks < nf) {
#pragma unroll
            for (int j = 0; j < 8; ++j) mx = fmaxf(mx, sc[ks >> 1][(ks & 1) * 8 + j]);
        }
    return fmaxf(mx, __shfl_xor(mx, 32));
}

// A selected key block as the loop wants it: ring-slot tile index and its number of valid keys.
//   bits 0..23 tile index (slot*nb + tile), bits 24..30 valid keys - 1
__device__ inline uint32_t pack_block(const KGeom &g, const KCache &c, int start, int head, int kb, int ph, int pw) {
    kb = min(max(kb, 0), c.valid * g.nb - 1);          // ids outside the cache (corrupt input) must not become wild addresses
    const int f = g.by_nb(kb), kt = kb - f * g.nb;
    const int kby = g.by_tx(kt), kbx = kt - kby * g.tx;
    const int vh = kby == g.ty - 1 ? ph : g.th, vw = kbx == g.tx - 1 ? pw : g.tw;
    return (uint32_t)(cache_slot(c, g, start, head, f) * g.nb + kt) | (uint32_t)(g.tt * vh * vw - 1) << 24;
}
__device__ inline int block_keys(uint32_t blk) { return (int)(blk >> 24) + 1; }

// FORM: kAttnPairs, or one work item per workgroup.  Split: the item's selected blocks are dealt out to the two groups in turn
// (group g takes blocks g, g + 2, ...), each group with a softmax of its own; at the end the groups exchange halves of their
// accumulators through LDS and each finishes 64 of the 128 channels.  Alone: group 1 only keeps the barriers company.
template <AttnForm FORM>
__global__ __launch_bounds__(512, 2) void attn_mfma_kernel(
    KGeom g, KCache c, const __bf16 *__restrict__ q, int64_t q_st, int64_t q_sh,
    const int32_t *__restrict__ sel_idx, const int32_t *__restrict__ sel_cnt,
    __bf16 *__restrict__ o, int64_t o_st, int64_t o_sh, float *__restrict__ lse,
    float scale_log2, int total_items, int wg_per_xcd) {
    __shared__ __attribute__((aligned(16))) unsigned char lds_all[2][2][kTileBytes];   // [group][K, V]
    constexpr bool SPLIT = FORM == kAttnSplit, ALONE = FORM == kAttnAlone;
    __shared__ float2 softmax_all[SPLIT ? 2 : 1][128];                                 // SPLIT: [group][query] reference and sum
    LCSA_STAMP(0)

    // Workgroups are dealt to the 8 XCDs round-robin; give each XCD a contiguous run of work
    // items (same head, neighbouring tiles, both query frames) so that K/V tiles shared by
    // neighbouring windows are found in that XCD's L2.
    const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
    const int work = FORM == kAttnPairs ? (total_items + 1) >> 1 : total_items;        // workgroups with work
    const int wg = xcd * wg_per_xcd + idx;
    if (wg >= work) return;

    const int tid = threadIdx.x, lane = tid & 63;
    const int grp8 = __builtin_amdgcn_readfirstlane(tid >> 8);        // which group of 4 wavefronts
    const int wave = __builtin_amdgcn_readfirstlane((tid >> 6) & 3);  // wavefront within the group
    unsigned char *k_lds = lds_all[grp8][0], *v_lds = lds_all[grp8][1];
    const int ql = lane & 31, half = lane >> 5;
    const int n_qb = g.q_groups * g.nb;

    // this group's item, and how many blocks the other group has (the stage clock is shared)
    auto item_row = [&](int item, int &head, int &qb) {
        head = g.by_n_qb(item);
        const int rem = item - head * n_qb;
        const int t = g.by_q_groups(rem), fq = rem - t * g.q_groups;   // items ordered (head, tile, group)
        qb = fq * g.nb + dealt_tile(g, t);
    };
    const int item = SPLIT ? wg : ALONE ? (grp8 == 0 ? wg : total_items) : 2 * wg + grp8;
    const int other = SPLIT ? wg : ALONE ? (grp8 == 0 ? total_items : wg) : 2 * wg + (grp8 ^ 1);
    // entry of the row's id list that is this group's block number i
    auto listed = [&](int i) { return SPLIT ? 2 * i + grp8 : i; };
    const bool active = item < total_items;
    int head = 0, qb = 0, cnt = 0, other_cnt = 0;
    const int start = ring_start(c, g);    // requested together with the counts and ids below
    int32_t first_ids = -1;                // selected block `lane` of this row, requested together with the count
    if (active) {
        item_row(item, head, qb);
        cnt = sel_cnt[(int64_t)head * n_qb + qb];
        if (listed(lane) < g.topk) first_ids = sel_idx[((int64_t)head * n_qb + qb) * g.topk + listed(lane)];
    }
    if (!SPLIT && other < total_items) { int h2, q2; item_row(other, h2, q2); other_cnt = sel_cnt[(int64_t)h2 * n_qb + q2]; }
    const int fq = g.by_nb(qb), tile = qb - fq * g.nb;
    const int by = g.by_tx(tile), bx = tile - by * g.tx;
    const int qvh = min(g.th, g.H - by * g.th), qvw = min(g.tw, g.W - bx * g.tw);

    // ---- Q fragments (B operand of S^T = K Q^T), requested before the counts are waited for:
    // lane holds query ql of this wavefront, channels 16s+8*half..+8
    const int tq = wave * 32 + ql;
    int qft, qr, qc;
    const BlockTokens q_tokens(g, qvh, qvw);
    const bool q_valid = q_tokens.at(tq, qft, qr, qc) && active;
    const int64_t token = q_valid ? raster_token(g, fq, qft, by * g.th + qr, bx * g.tw + qc)
                                  : raster_token(g, fq, 0, by * g.th, bx * g.tw);       // clamp padding rows
    // a wavefront whose 32 query rows are all padding only takes part in the copies and barriers
    const bool wave_on = active && wave * 32 < g.tt * qvh * qvw;
    bf16x8 bq[8];
    {
        const __bf16 *qp = q + token * q_st + (int64_t)head * q_sh + half * 8;
#pragma unroll
        for (int s = 0; s < 8; ++s) bq[s] = *(const bf16x8 *)(qp + s * 16);
    }

    cnt = min(max(__builtin_amdgcn_readfirstlane(cnt), 0), g.topk);            // a row holds at most topk ids
    other_cnt = min(max(__builtin_amdgcn_readfirstlane(other_cnt), 0), g.topk);
    if (SPLIT) { other_cnt = (cnt + grp8) >> 1; cnt = (cnt + 1 - grp8) >> 1; }
    const int n_iter = max(cnt, other_cnt);
    const int64_t row = (int64_t)head * n_qb + qb;
    const int32_t *sel = sel_idx + row * g.topk;

    // ---- the first K tile is requested as soon as its id is known so that its latency overlaps the set-up.
    // Wavefront w copies rows 32w..32w+31 of a K tile, which are only read if they hold valid keys.
    const char *k_head = (const char *)c.k + (int64_t)head * g.cap * g.nb * kTileBytes;
    const char *v_head = (const char *)c.v + (int64_t)head * g.cap * g.nb * kTileBytes;
    auto tile_off = [](uint32_t blk) { return (int64_t)(blk & 0xffffffu) * kTileBytes; };
    auto key_groups = [](uint32_t blk) { return (block_keys(blk) + 31) >> 5; };
    const uint32_t copy_voff = wave * 8192 + lane * 16;     // this lane's byte offset inside any tile image
    const uint32_t kdst = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)((LCSA_LDS unsigned char *)k_lds) + wave * 8192);
    const uint32_t vdst = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)((LCSA_LDS unsigned char *)v_lds) + wave * 8192);
    // selected blocks of this row, 64 at a time, one per lane, already turned into tile indices
    const int ph = g.H - (g.ty - 1) * g.th, pw = g.W - (g.tx - 1) * g.tw;   // extent of clipped edge tiles
    uint32_t blk_chunk = lane < cnt ? pack_block(g, c, start, head, first_ids, ph, pw) : 0u;
    uint32_t blk = __builtin_amdgcn_readfirstlane(blk_chunk);
    if (cnt > 0 && wave < key_groups(blk)) {
#pragma unroll
        for (int piece = 0; piece < 8; ++piece) copy_piece_to_lds(k_head + tile_off(blk), copy_voff, kdst, piece);
    }

    // ---- per-lane LDS offsets
    // K operand: MFMA row m = ql reads key row pi(ql) of each 32-key group (bits 2,3 swapped)
    const int krow = (ql & 0x13) | ((ql & 4) << 1) | ((ql & 8) >> 1);
    // byte offset of the 16-byte chunk (2s + half) of this lane's row: row*256 + (((2s+half) ^ (row&15)) << 4)
    //   = base ^ (s << 5) with base = row*256 + (((half ^ row) & 15) << 4): one XOR per read, two registers
    const int k_base = krow * 256 + (((half ^ krow) & 15) << 4);     // + 8192 * key group
    const int v_base = ql * 256 + (((half ^ ql) & 15) << 4);         // + 8192 * channel group
    auto k_off = [&](int s) { return k_base ^ (s << 5); };
    auto v_off = [&](int s) { return v_base ^ (s << 5); };

    f32x16 oacc[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[dt][i] = 0.f;
    float m_run = -__builtin_inff(), l_run = 0.f;

    __builtin_amdgcn_s_waitcnt(0x0F70);    // vmcnt(0), visible to the compiler: Q fragments, ids and the first K tile have arrived
    stage_barrier();                       // first K tiles of both groups are in LDS
    if (grp8 == 1) { stage_barrier(); stage_barrier(); }   // group 1 runs two phases behind group 0

    LCSA_STAMP(1)
    f16x8 pfrag[8];                        // P^T fragments of the previous block: [key group*2 + k-step]
    uint32_t blk_next = 0;
    bool has_next = false;
    float l_before = 0.f;
    int ng = 4, ng_prev = 4;               // 32-key groups of the current / previous block that hold valid keys

    // O^T += V^T P^T over the first `groups` 32-key groups (2 k-steps each) x 4 channel groups.
    // Operand fragments are read kAhead matrix instructions ahead through a register ring; a group
    // without valid keys ends the product (its operands, already requested, are dropped).
    auto pv_phase = [&](int groups) {
        f16x8 va[kRing];
#pragma unroll
        for (int n = 0; n < kAhead; ++n) va[n % kRing] = *(const f16x8 *)(v_lds + (n & 3) * 8192 + v_off(n >> 2));
        __builtin_amdgcn_sched_group_barrier(0x100, kAhead, 0);
#pragma unroll
        for (int kg = 0; kg < 4; ++kg)
            if (kg < groups) {
#pragma unroll
                for (int n = 8 * kg; n < 8 * kg + 8; ++n) {
                    const int ks = n >> 2, dt = n & 3;
                    if (n + kAhead < 32) {
                        va[(n + kAhead) % kRing] = *(const f16x8 *)(v_lds + ((n + kAhead) & 3) * 8192 + v_off((n + kAhead) >> 2));
                        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    }
                    oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va[n % kRing], pfrag[ks], oacc[dt], 0, 0, 0);
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                }
            }
    };

    // Four phases per block, each ending in a workgroup barrier:
    //   P1  PV(i-1)            matrix     P3  softmax(i), first fragments   vector
    //   P2  QK(i)              matrix     P4  softmax(i), the rest + check  vector
    // Group 1 is two phases behind, so every SIMD always holds one wavefront in a matrix phase and
    // one in a vector phase.  Tile copies: V(i) is issued during P2(i) and needed at P1(i+1);
    // K(i+1) is issued during P3(i) and P4(i) and needed at P2(i+1): two to three phases of lead.  The eight
    // copy instructions of a tile are spread through the phase because each one can hold the
    // issuing wavefront while the memory pipeline accepts it.
    for (int it = 0; it <= n_iter; ++it) {
        const bool pv_on = it >= 1 && it - 1 < cnt;   // wavefront-uniform
        const bool on = it < cnt;
        f32x16 sacc[4];                    // S^T of this block: produced in P2, consumed in P3 and P4

        // S^T = K Q^T over the first `groups` key groups x 8 k-steps; the 8 copy instructions of V(i) go along
        auto qk_phase = [&](int groups, const char *vsrc) {
            bf16x8 ka[kRing];
#pragma unroll
            for (int n = 0; n < kAhead; ++n) ka[n % kRing] = *(const bf16x8 *)(k_lds + (n >> 3) * 8192 + k_off(n & 7));
            __builtin_amdgcn_sched_group_barrier(0x100, kAhead, 0);
#pragma unroll
            for (int kg = 0; kg < 4; ++kg) {
                if (kg < groups) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) sacc[kg][i] = 0.f;
#pragma unroll
                    for (int n = 8 * kg; n < 8 * kg + 8; ++n) {
                        const int s = n & 7;
                        if ((n & 3) == 0) copy_piece_to_lds(vsrc, copy_voff, vdst, n >> 2);     // one copy instruction per 4 MFMAs
                        if (n + kAhead < 32) {
                            ka[(n + kAhead) % kRing] = *(const bf16x8 *)(k_lds + ((n + kAhead) >> 3) * 8192 + k_off((n + kAhead) & 7));
                            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                        }
                        sacc[kg] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[n % kRing], bq[s], sacc[kg], 0, 0, 0);
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    }
                } else {
                    copy_piece_to_lds(vsrc, copy_voff, vdst, 2 * kg);
                    copy_piece_to_lds(vsrc, copy_voff, vdst, 2 * kg + 1);
                }
            }
        };

        // ================= P1: O^T += V^T P^T of the previous block ===================================
        if (pv_on && wave_on) {
            __builtin_amdgcn_s_setprio(2);
            pv_phase(ng_prev);
            __builtin_amdgcn_s_setprio(0);
        }
        if (on) wait_vm0();                // K(i) (this wavefront's part) has landed
        __builtin_amdgcn_sched_barrier(0);
        stage_barrier();
        __builtin_amdgcn_sched_barrier(0);

        // ================= P2: S^T = K Q^T; V(i) copy issued alongside ================================
        if (on) {
            blk = it == 0 ? blk : blk_next;
            ng = key_groups(blk);
            const char *vsrc = v_head + tile_off(blk);
            if (wave_on) {
                __builtin_amdgcn_s_setprio(2);
                qk_phase(ng, vsrc);
                __builtin_amdgcn_s_setprio(0);
            } else {
#pragma unroll
                for (int piece = 0; piece < 8; ++piece) copy_piece_to_lds(vsrc, copy_voff, vdst, piece);
            }
            // next block; every 64 iterations the per-lane chunk is refilled (the read of the fresh
            // value sits inside the branch so that the wait for that load does too)
            has_next = it + 1 < cnt;
            if (has_next) {
                if (((it + 1) & 63) == 0) {
                    blk_chunk = (it + 1 + lane) < cnt ? pack_block(g, c, start, head, sel[listed(it + 1 + lane)], ph, pw) : 0u;
                    blk_next = __builtin_amdgcn_readlane(blk_chunk, 0);
                } else {
                    blk_next = __builtin_amdgcn_readlane(blk_chunk, (it + 1) & 63);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        stage_barrier();
        __builtin_amdgcn_sched_barrier(0);

        // ================= P3: online softmax, first half; K(i+1) copy issued alongside ===============
        const char *ksrc = k_head + tile_off(blk_next);
        const bool k_copy = on && has_next && wave < key_groups(blk_next);    // this wavefront's rows of K(i+1) hold keys
        const int nv = block_keys(blk);
        const int nf = (nv + 15) >> 4;     // 16-key fragments that hold valid keys
        // everyone in the group is done reading K: the next K tile may overwrite it
        if (k_copy) { copy_piece_to_lds(ksrc, copy_voff, kdst, 0); copy_piece_to_lds(ksrc, copy_voff, kdst, 1); }
        if (on && wave_on) {
            // Padding keys get weight exactly zero.  Valid keys come first in a block, so only the last
            // fragment can be mixed: accumulator register j of fragment ks is key 16*ks + 8*half + j.
            if (nv & 15) {
                const int thr = (nv & 15) - half * 8;      // registers j >= thr of the last fragment are padding
#pragma unroll
                for (int ks = 0; ks < 8; ++ks)
                    if (ks == nf - 1) {
#pragma unroll
                        for (int j = 0; j < 8; ++j)
                            if (j >= thr) sacc[ks >> 1][(ks & 1) * 8 + j] = -__builtin_inff();
                    }
            }
            // Reference point of the exponentials.  Any per-query reference gives the same softmax after
            // the final normalisation; it only has to keep 2^(score - reference) inside half's range.
            // The first block sets it to its exact row maximum; later blocks reuse it without looking
            // for their maximum (which would cost a pass over all scores) and are checked afterwards:
            // see the end of P4.  It is kept finite: a first block whose scores are all -inf (masked keys) weighs nothing,
            // and the check moves the reference to the first block that does.
            if (it == 0) m_run = fmaxf(block_row_max(sacc, nf) * scale_log2, -__FLT_MAX__);
        }
        if (k_copy) { copy_piece_to_lds(ksrc, copy_voff, kdst, 2); copy_piece_to_lds(ksrc, copy_voff, kdst, 3); }
        if (on && wave_on) {
            l_before = l_run;
            // probabilities -> half for the matrix product; row sum in float
#pragma unroll
            for (int ks = 0; ks < kSplit; ++ks) {
                if (ks < nf) softmax_fragment(sacc[ks >> 1], (ks & 1) * 8, scale_log2, m_run, l_run, pfrag[ks]);
                else pfrag[ks] = f16x8{0, 0, 0, 0, 0, 0, 0, 0};
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        stage_barrier();
        __builtin_amdgcn_sched_barrier(0);

        // ================= P4: online softmax, second half =============================================
        if (k_copy) { copy_piece_to_lds(ksrc, copy_voff, kdst, 4); copy_piece_to_lds(ksrc, copy_voff, kdst, 5); }
        if (on && wave_on) {
#pragma unroll
            for (int ks = kSplit; ks < 8; ++ks) {
                if (ks < nf) softmax_fragment(sacc[ks >> 1], (ks & 1) * 8, scale_log2, m_run, l_run, pfrag[ks]);
                else pfrag[ks] = f16x8{0, 0, 0, 0, 0, 0, 0, 0};
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (k_copy) { copy_piece_to_lds(ksrc, copy_voff, kdst, 6); copy_piece_to_lds(ksrc, copy_voff, kdst, 7); }
        if (on && wave_on) {
            // Check of the reference: this lane's probabilities of the block sum to less than 2^14, hence none
            // of them left half's range.  Otherwise (a block whose scores tower over everything seen before, or
            // non-finite input) redo the block against its exact maximum, rescaling the running sums.
            if (__ballot(!(l_run - l_before < 16384.f))) {
                const float m_new = fmaxf(m_run, block_row_max(sacc, nf) * scale_log2);
                const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
                l_run = l_before * alpha;
#pragma unroll
                for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                    for (int i = 0; i < 16; ++i) oacc[dt][i] *= alpha;
                m_run = m_new;
#pragma unroll
                for (int ks = 0; ks < 8; ++ks)
                    if (ks < nf) softmax_fragment(sacc[ks >> 1], (ks & 1) * 8, scale_log2, m_run, l_run, pfrag[ks]);
            }
        }
        if (on) {
            // V(i) has landed (the 8 newer copies in flight are this wavefront's part of the next K tile, if any)
            if (k_copy) wait_vm8(); else wait_vm0();
            ng_prev = ng;
        }
        __builtin_amdgcn_sched_barrier(0);
        stage_barrier();
        __builtin_amdgcn_sched_barrier(0);
    }
    if (grp8 == 0) { stage_barrier(); stage_barrier(); }   // matches group 1's two extra barriers at the start
    LCSA_STAMP(2)

    // ---- epilogue: normalise, transpose through this wavefront's own quarter of its group's K buffer, store.
    // No LDS reads of other wavefronts are outstanding: the last stage ended in a barrier.
    if (!active) return;
    float l_tot = l_run + __shfl_xor(l_run, 32);
    constexpr int kOut = SPLIT ? 2 : 4;                    // channel groups of 32 that this group finishes: first_dt ..
    const int first_dt = SPLIT ? 2 * grp8 : 0;
    f32x16 out[kOut];
    if constexpr (SPLIT) {
        // Each group passes the 64 channels it does not finish to the other one, through its own V and K buffers: a
        // wavefront's 8 KB of either, register quad by register quad, 16 bytes per lane.
        unsigned char *mine = v_lds + wave * 8192, *theirs = lds_all[grp8 ^ 1][1] + wave * 8192;
        f32x16 give[2];
#pragma unroll
        for (int dt = 0; dt < 2; ++dt) {
            out[dt] = grp8 ? oacc[2 + dt] : oacc[dt];
            give[dt] = grp8 ? oacc[dt] : oacc[2 + dt];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            typedef __attribute__((ext_vector_type(4))) float f32x4;
            const f32x16 &from = give[i >> 2];
            const int r = (i & 3) * 4;
            *(f32x4 *)(mine + i * 1024 + lane * 16) = f32x4{from[r], from[r + 1], from[r + 2], from[r + 3]};
        }
        if (half == 0) softmax_all[grp8][tq] = make_float2(m_run, l_tot);
        stage_barrier();
        const float2 o_ml = softmax_all[grp8 ^ 1][tq];
        const float m_all = fmaxf(m_run, o_ml.x), ref = m_all == -__builtin_inff() ? 0.f : m_all;   // a group without blocks: reference -inf, sum 0
        const float a_own = __builtin_amdgcn_exp2f(m_run - ref), a_other = __builtin_amdgcn_exp2f(o_ml.x - ref);
        l_tot = l_tot * a_own + o_ml.y * a_other;
        m_run = m_all;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            typedef __attribute__((ext_vector_type(4))) float f32x4;
            const f32x4 x = *(const f32x4 *)(theirs + i * 1024 + lane * 16);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float &y = ((float *)&out[i >> 2])[(i & 3) * 4 + j];
                y = y * a_own + x[j] * a_other;
            }
        }
    } else {
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) out[dt] = oacc[dt];
    }
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
    // lane owns query row tq; accumulator register i of channel group dt is channel
    // dt*32 + (i>>2)*8 + half*4 + (i&3): 4 consecutive channels = 8 bytes
#pragma unroll
    for (int dt = 0; dt < kOut; ++dt)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
            bf16x4 w;
#pragma unroll
            for (int j = 0; j < 4; ++j) w[j] = (__bf16)(out[dt][i4 * 4 + j] * inv);
            const int chunk = dt * 4 + i4;
            *(bf16x4 *)(k_lds + tq * 256 + ((chunk ^ (tq & 15)) << 4) + half * 8) = w;
        }
    if (lse && half == 0 && q_valid && (!SPLIT || grp8 == 0))
        lse[token * g.heads + head] = l_tot > 0.f ? (m_run + __builtin_amdgcn_logf(l_tot)) * kLn2 : -__builtin_inff();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // rows written by this wavefront are read by it only
    {
        constexpr int kLanes = kOut * 4, kRows = 64 / kLanes;     // lanes x 16 bytes per row, rows per pass
        const int rg = lane / kLanes, j = lane % kLanes;
#pragma unroll
        for (int itr = 0; itr < 32 / kRows; ++itr) {
            const int t = wave * 32 + rg + kRows * itr;
            int ft, r, cc;
            if (q_tokens.at(t, ft, r, cc)) {
                const int64_t tok = raster_token(g, fq, ft, by * g.th + r, bx * g.tw + cc);
                const uint4 u = *(const uint4 *)(k_lds + t * 256 + ((j ^ (t & 15)) << 4));
                *(uint4 *)(o + tok * o_st + (int64_t)head * o_sh + first_dt * 32 + j * 8) = u;
            }
        }
    }
    LCSA_STAMP(3)
}

// Few items: a workgroup takes 64 of a block's 128 queries, so that two workgroups work on an item.  Wavefront w owns queries
// 32 (w >> 2) .. + 31 of them and, of every selected block, the 32 keys of unit w & 3, with a softmax of its own over the keys
// it sees; the four partial results of a query meet in LDS at the end.  One barrier a block; the next block's copies go along
// with the first product.
// What bounds it: the arrival of the copies, 64 KB a block for half the queries, one block ahead (0.93 us a block; issued later,
// or with the values waited for apart, it is 10 to 15 % slower); it is used only where units would be idle otherwise.
__global__ __launch_bounds__(512, 2) void attn_mfma_few_kernel(
    KGeom g, KCache c, const __bf16 *__restrict__ q, int64_t q_st, int64_t q_sh,
    const int32_t *__restrict__ sel_idx, const int32_t *__restrict__ sel_cnt,
    __bf16 *__restrict__ o, int64_t o_st, int64_t o_sh, float *__restrict__ lse,
    float scale_log2, int total_items, int wg_per_xcd) {
    __shared__ __attribute__((aligned(256))) unsigned char lds[2][2][kTileBytes];      // [stage][K, V]; at the end the partial results
    __shared__ float2 softmax_all[4][64];                                              // [unit][query] reference and sum
    const int wg = (blockIdx.x & 7) * wg_per_xcd + (blockIdx.x >> 3);
    if (wg >= 2 * total_items) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), qg = wave >> 2, unit = wave & 3;
    const int ql = lane & 31, half = lane >> 5;
    const int n_qb = g.q_groups * g.nb;
    const int item = wg >> 1, head = g.by_n_qb(item), rem = item - head * n_qb;
    const int tile = g.by_q_groups(rem), fq = rem - tile * g.q_groups, qb = fq * g.nb + tile;    // items ordered (head, tile, group)
    const int by = g.by_tx(tile), bx = tile - by * g.tx;
    const int qvh = min(g.th, g.H - by * g.th), qvw = min(g.tw, g.W - bx * g.tw);
    const int first_query = 64 * (wg & 1);
    if (first_query >= g.tt * qvh * qvw) return;             // a clipped block without a second half

    const int64_t row = (int64_t)head * n_qb + qb;
    const int32_t *sel = sel_idx + row * g.topk;
    const int start = ring_start(c, g);
    int cnt = sel_cnt[row];
    const int32_t first_ids = lane < g.topk ? sel[lane] : -1;
    const int tq = first_query + 32 * qg + ql;
    int qft, qr, qc;
    const BlockTokens q_tokens(g, qvh, qvw);
    const bool q_valid = q_tokens.at(tq, qft, qr, qc);
    const int64_t token = q_valid ? raster_token(g, fq, qft, by * g.th + qr, bx * g.tw + qc)
                                  : raster_token(g, fq, 0, by * g.th, bx * g.tw);       // padding rows: the block's first token
    bf16x8 bq[8];
    {
        const __bf16 *qp = q + token * q_st + (int64_t)head * q_sh + half * 8;
#pragma unroll
        for (int s = 0; s < 8; ++s) bq[s] = *(const bf16x8 *)(qp + s * 16);
    }
    cnt = min(max(__builtin_amdgcn_readfirstlane(cnt), 0), g.topk);
    const char *k_head = (const char *)c.k + (int64_t)head * g.cap * g.nb * kTileBytes;
    const char *v_head = (const char *)c.v + (int64_t)head * g.cap * g.nb * kTileBytes;
    const int ph = g.H - (g.ty - 1) * g.th, pw = g.W - (g.tx - 1) * g.tw;   // extent of clipped edge tiles
    const uint32_t copy_voff = wave * 4096 + lane * 16;
    const uint32_t lds_at = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)((LCSA_LDS unsigned char *)&lds[0][0][0]));
    uint32_t blk_chunk = lane < cnt ? pack_block(g, c, start, head, first_ids, ph, pw) : 0u;
    // piece of this wavefront's eighths of a block's K and V tiles
    auto copy_piece = [&](uint32_t blk, int stage, int piece) {
        const int64_t off = (int64_t)(blk & 0xffffffu) * kTileBytes;
        const uint32_t dst = lds_at + stage * 2 * kTileBytes + wave * 4096;
        if (piece < 4) copy_piece_to_lds(k_head + off, copy_voff, dst, piece);
        else copy_piece_to_lds(v_head + off, copy_voff, dst + kTileBytes, piece - 4);
    };
    uint32_t blk = 0, blk_next = __builtin_amdgcn_readfirstlane(blk_chunk);
    if (cnt > 0)
#pragma unroll
        for (int piece = 0; piece < 8; ++piece) copy_piece(blk_next, 0, piece);

    // operand offsets as in the kernel above, for this wavefront's 32 keys
    const int krow = (ql & 0x13) | ((ql & 4) << 1) | ((ql & 8) >> 1);
    const int k_base = (32 * unit + krow) * 256 + (((half ^ krow) & 15) << 4);
    const int v_base = kTileBytes + ql * 256 + (((4 * unit + half) ^ (ql & 15)) << 4);
    f32x16 oacc[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[dt][i] = 0.f;
    float m_run = -__builtin_inff(), l_run = 0.f;
    bool started = false;                                    // this wavefront has seen a key
    __builtin_amdgcn_s_waitcnt(0x0F70);                      // vmcnt(0), visible to the compiler

    for (int it = 0; it < cnt; ++it) {
        wait_vm0();                                          // the block's tiles have landed,
        stage_barrier();                                     // everybody's, and everybody is done with the other stage
        blk = blk_next;
        if (((it + 1) & 63) == 0 && it + 1 < cnt)
            blk_chunk = it + 1 + lane < cnt ? pack_block(g, c, start, head, sel[it + 1 + lane], ph, pw) : 0u;
        blk_next = __builtin_amdgcn_readlane(blk_chunk, min(it + 1, cnt - 1) & 63);       // behind the last block itself again
        const unsigned char *tiles = lds[it & 1][0];
        const int nv = block_keys(blk) - 32 * unit;          // valid keys from this unit on
        f32x16 sacc;
        {
            __builtin_amdgcn_s_setprio(2);
            bf16x8 ka[kRing];
#pragma unroll
            for (int n = 0; n < kAhead; ++n) ka[n] = *(const bf16x8 *)(tiles + (k_base ^ (n << 5)));
#pragma unroll
            for (int i = 0; i < 16; ++i) sacc[i] = 0.f;
#pragma unroll
            for (int n = 0; n < 8; ++n) {
                __builtin_amdgcn_sched_barrier(0);
                sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[n % kRing], bq[n], sacc, 0, 0, 0);
                if (n + kAhead < 8) ka[(n + kAhead) % kRing] = *(const bf16x8 *)(tiles + (k_base ^ ((n + kAhead) << 5)));
                copy_piece(blk_next, (it + 1) & 1, n);
            }
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(0);
        }
        if (nv <= 0) continue;                               // uniform over the wavefront
        if (nv < 32) {
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if ((i >> 3) * 16 + (i & 7) + 8 * half >= nv) sacc[i] = -__builtin_inff();
        }
        // reference as in the kernel above: exact for the first keys, kept finite, checked afterwards
        auto row_max = [&]() {
            float mx = sacc[0];
#pragma unroll
            for (int i = 1; i < 16; ++i) mx = fmaxf(mx, sacc[i]);
            return fmaxf(mx, __shfl_xor(mx, 32));
        };
        if (!started) { m_run = fmaxf(row_max() * scale_log2, -__FLT_MAX__); started = true; }
        f16x8 pfrag[2];
        const float l_before = l_run;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) softmax_fragment(sacc, 8 * ks, scale_log2, m_run, l_run, pfrag[ks]);
        if (__ballot(!(l_run - l_before < 16384.f))) {
            const float m_new = fmaxf(m_run, row_max() * scale_log2);
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
            l_run = l_before * alpha;
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                for (int i = 0; i < 16; ++i) oacc[dt][i] *= alpha;
            m_run = m_new;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) softmax_fragment(sacc, 8 * ks, scale_log2, m_run, l_run, pfrag[ks]);
        }
        __builtin_amdgcn_s_setprio(2);
        f16x8 va[kRing];
#pragma unroll
        for (int n = 0; n < kAhead; ++n) va[n] = *(const f16x8 *)(tiles + (n >> 1) * 8192 + (v_base ^ ((n & 1) << 5)));
#pragma unroll
        for (int n = 0; n < 8; ++n) {
            __builtin_amdgcn_sched_barrier(0);
            oacc[n >> 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va[n % kRing], pfrag[n & 1], oacc[n >> 1], 0, 0, 0);
            if (n + kAhead < 8) va[(n + kAhead) % kRing] = *(const f16x8 *)(tiles + ((n + kAhead) >> 1) * 8192 + (v_base ^ (((n + kAhead) & 1) << 5)));
        }
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(0);
    }

    // ---- epilogue: wavefront (qg, unit) finishes channels 32 unit .. + 31 of its queries from the four partial results
    float l_tot = l_run + __shfl_xor(l_run, 32);
    if (half == 0) softmax_all[unit][32 * qg + ql] = make_float2(m_run, l_tot);
    wait_vm0();
    stage_barrier();                                         // nobody reads the tiles any more, and no copy may land later
    typedef __attribute__((ext_vector_type(4))) float f32x4;
    f32x4 *part = (f32x4 *)&lds[0][0][0];                    // [wavefront][channel group][register quad][lane]
    f32x16 out;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
        if (dt == unit) out = oacc[dt];                      // uniform
        else
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4)
                part[((wave * 4 + dt) * 4 + i4) * 64 + lane] = f32x4{oacc[dt][4 * i4], oacc[dt][4 * i4 + 1], oacc[dt][4 * i4 + 2], oacc[dt][4 * i4 + 3]};
    }
    stage_barrier();
    float m_all = -__builtin_inff();
#pragma unroll
    for (int u = 0; u < 4; ++u) m_all = fmaxf(m_all, softmax_all[u][32 * qg + ql].x);
    const float ref = m_all == -__builtin_inff() ? 0.f : m_all;      // no keys at all
    l_tot = 0.f;
    f32x16 sum;
#pragma unroll
    for (int i = 0; i < 16; ++i) sum[i] = 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const float2 ml = softmax_all[u][32 * qg + ql];
        const float a = __builtin_amdgcn_exp2f(ml.x - ref);
        l_tot = fmaf(ml.y, a, l_tot);
        if (u == unit) {
#pragma unroll
            for (int i = 0; i < 16; ++i) sum[i] = fmaf(out[i], a, sum[i]);
        } else {
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const f32x4 x = part[(((4 * qg + u) * 4 + unit) * 4 + i4) * 64 + lane];
#pragma unroll
                for (int j = 0; j < 4; ++j) sum[4 * i4 + j] = fmaf(x[j], a, sum[4 * i4 + j]);
            }
        }
    }
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
    if (lse && unit == 0 && half == 0 && q_valid)
        lse[token * g.heads + head] = l_tot > 0.f ? (m_all + __builtin_amdgcn_logf(l_tot)) * kLn2 : -__builtin_inff();
    stage_barrier();                                         // the partial results have been read
    // register i is channel 32 unit + (i >> 2) * 8 + half * 4 + (i & 3): rows of 256 bytes, 16-byte chunk j of row r at j ^ (r & 15)
    unsigned char *rows = &lds[0][0][0];
    const int r64 = 32 * qg + ql;
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
        bf16x4 w;
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j] = (__bf16)(sum[4 * i4 + j] * inv);
        *(bf16x4 *)(rows + r64 * 256 + (((4 * unit + i4) ^ (r64 & 15)) << 4) + half * 8) = w;
    }
    stage_barrier();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = (tid >> 4) + 32 * i, j = tid & 15;
        int ft, rr, cc;
        if (q_tokens.at(first_query + r, ft, rr, cc)) {
            const int64_t tok = raster_token(g, fq, ft, by * g.th + rr, bx * g.tw + cc);
            *(uint4 *)(o + tok * o_st + (int64_t)head * o_sh + j * 8) = *(const uint4 *)(rows + r * 256 + ((j ^ (r & 15)) << 4));
        }
    }
}

} // namespace

AttnLaunch attn_mfma_launch(const KGeom &g, const KCache &c) {
    const int n_cu = compute_units();
    const int total = g.heads * g.nb * g.q_groups, admissible = max_candidates(g, c.valid);
    AttnForm form = attn_form(total, n_cu, g.topk < admissible ? g.topk : admissible);
#ifndef LCSA_TIMERS                                          // the other forms are the ones with stamps
    if (attn_few(total, n_cu, (int64_t)g.tt * g.H * g.W, g.nb)) form = kAttnFew;
#endif
    return {form, total, (attn_workgroups(form, total) + 7) / 8};
}

hipError_t launch_attn_mfma(const KGeom &g, const KCache &c, const void *q, int64_t q_st, int64_t q_sh,
                            const int32_t *sel_idx, const int32_t *sel_cnt,
                            void *o, int64_t o_st, int64_t o_sh, float *lse, float scale, hipStream_t stream) {
    const auto [form, total, per_xcd] = attn_mfma_launch(g, c);
#define LCSA_CALL(FORM)                                                                                                    \
    attn_mfma_kernel<FORM><<<dim3(per_xcd * 8), 512, 0, stream>>>(g, c, (const __bf16 *)q, q_st, q_sh, sel_idx, sel_cnt,     \
                                                                  (__bf16 *)o, o_st, o_sh, lse, scale * kLog2e, total, per_xcd)
    if (form == kAttnPairs) LCSA_CALL(kAttnPairs);
    else if (form == kAttnSplit) LCSA_CALL(kAttnSplit);
    else if (form == kAttnAlone) LCSA_CALL(kAttnAlone);
    else
        attn_mfma_few_kernel<<<dim3(per_xcd * 8), 512, 0, stream>>>(g, c, (const __bf16 *)q, q_st, q_sh, sel_idx, sel_cnt,
                                                                    (__bf16 *)o, o_st, o_sh, lse, scale * kLog2e, total, per_xcd);
#undef LCSA_CALL
    return hipGetLastError();
}

} // namespace lcsa
