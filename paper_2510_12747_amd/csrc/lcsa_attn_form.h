// How launches of the matrix-core attention kernels deal their work items (one per (head, query block)) out to workgroups, and
// the general append its tiles.  Host arithmetic only.
#pragma once
#include <stdint.h>

namespace lcsa {

enum AttnForm {
    kAttnPairs = 0,      // two items per workgroup, one per group of four wavefronts
    kAttnSplit = 1,      // one item per workgroup, its blocks shared between the groups, the partial results merged
    kAttnAlone = 2,      // one item per workgroup on one group, the other only keeps the barriers company
    kAttnFew = 3,        // two workgroups to an item, half its queries each (a kernel of its own)
};

// A workgroup holds a compute unit to itself, so a launch takes rounds = ceil(workgroups / units), each as long as the blocks
// of one workgroup plus a set-up and an epilogue.  2 n + 1 rounds of split items against n + 1 of pairs save the last half
// round and pay n more set-ups; with any other numbers of rounds splitting saves nothing.  Set-up and epilogue cost about
// 2.5 blocks, which would make split items shorter for k > 5 n (k: blocks of a full row); the more rounds, the further the
// workgroups have drifted apart and the less there is of a last round, hence k > n (9 + n) / 2, and pairs from n = 6 on.
// Medians of split / pairs over 1900 launches of random geometry on 256 units (all of it in profiles/): n = 1, k = 4 1.04,
// k = 6 0.985, k = 13 .. 20 0.87; n = 2, k = 9 .. 10 1.01, k = 11 .. 12 0.98; n = 3, k = 16 .. 18 1.00, k = 19 .. 21 0.99;
// n = 4, k = 21 .. 24 1.01, k = 25 .. 28 1.00; n = 6, k = 43 .. 54 1.02, k = 55 .. 72 1.01.  Single geometries lie up to 10 % away,
// most of them grids whose last row or column of tiles is a sliver.
// Up to one item per unit a split item always ends earlier than a pair, and than an item on one group (k = 2 0.99, k = 4
// 0.89), except that one block cannot be shared: k = 1 1.08.
inline AttnForm attn_form(int items, int units, int k) {
    const int rounds_split = (items + units - 1) / units, rounds_pairs = ((items + 1) / 2 + units - 1) / units;
    if (rounds_split <= 1) return k <= 1 ? kAttnAlone : kAttnSplit;
    const int n = rounds_pairs - 1;
    return rounds_split == 2 * n + 1 && n <= 5 && k > n * (9 + n) / 2 ? kAttnSplit : kAttnPairs;
}

// Before the rule above: where two workgroups an item still leave nobody waiting, an item is faster in two halves of its
// queries than in two of its keys, which spares the second half of the blocks one after the other.  Split / two halves, us on 256
// units, full blocks: 9 items of one, two, four and 16 blocks 9.5 / 7.9 (alone: 8.5), 10.8 / 8.8, 13.4 / 10.7, 27.9 / 21.2; 72 of 16
// 29.5 / 23.5, of 64 89.8 / 70.7; 126 of 16 31.1 / 26.2, of 64 93.8 / 81.4; 135 of 16 30.8 / 45.8.
// Only if a block holds more than 64 tokens in the mean (tokens of a frame group / its blocks): with fewer there is little for a
// second workgroup to do, and this kernel copies all of every tile, the other forms only the keys there are.  Over 400 random
// geometries of at most 128 items it takes 0.84 of the other form's time at 112 tokens and more, 0.88 at 80 to 95, 0.92 at 64
// to 79, 0.97 (single ones 1.13) at 48 to 63, 1.00 at 32 to 47, 1.18 (up to 1.49) below 16.
inline bool attn_few(int items, int units, int64_t tokens, int blocks) { return items <= units / 2 && tokens > (int64_t)64 * blocks; }

inline int attn_workgroups(AttnForm form, int items) { return form == kAttnPairs ? (items + 1) / 2 : form == kAttnFew ? 2 * items : items; }

// Query-side backward: wavefronts of a workgroup = query groups of 32 x shares of the keys.
enum BwdQueryForm {
    kBwd4x1 = 0,         // a block's four query groups; two workgroups share a unit
    kBwd4x2 = 1,         // the same with the keys shared by two wavefronts each: a workgroup has a unit to itself
    kBwd2x4 = 2,         // half a block's queries, the keys shared by four
};

// k: blocks a row keeps, at most.  Whole backward in us on 256 units, 4 x 1 / 4 x 2 / 2 x 4, rows of k full blocks:
//   up to half an item a unit   126 items: k = 1 44 / 45 / 44, 4 66 / 63 / 60, 16 149 / 129 / 116, 32 257 / 213 / 189
//   up to one                   144 items: k = 1 44 / 46 / 56, 4 69 / 66 / 79, 16 159 / 141 / 164;  252 of 32 343 / 318 / 341
//   two rounds of 4 x 2         288 items: k = 1 64 / 74 / 82, 16 240 / 264 / 262, 32 417 / 458 / 440;  504 of 32 617 / 627 / 685
//   three                       576 items: k = 1 122 / 136 / 152, 4 195 / 209 / 224, 16 451 / 445 / 460, 32 814 / 778 / 783;  756 of 16
//                               548 / 555 / 601, of 32 950 / 936 / 1025
//   more                        864 items of 32 1084 / 1136 / 1171, 1152 of 32 1465 / 1461 / 1598, 1728 of 32 2129 / 2166 / 2341
// Two workgroups of 4 x 1 share a unit and do not wait at each other's barriers, which wins wherever units have two of them
// to the end; three rounds of 4 x 2 take less than two of 4 x 1, of which the second is half full, only where rows are long (five
// rounds, 1080 of 32: 1408 / 1406).
inline BwdQueryForm bwd_query_form(int items, int units, int k) {
    const int rounds = (items + units - 1) / units;
    if (rounds <= 1) return 2 * items <= units ? kBwd2x4 : kBwd4x2;
    return rounds == 3 && k > 16 ? kBwd4x2 : kBwd4x1;
}

// General append into the ring: whether four tiles share a workgroup of 1024 threads.  What they share is a ticket, 10 ns each and one
// after the other; what it costs is that a tile's threads move together with three others', in fewer workgroups.  So by the bytes of a tile
// (each of K and V; the shape does not matter) and by how evenly the units are filled.  One / four a workgroup, us on 256 units (all of it in
// profiles/):
//   to 16 KB     the tickets are most of it: 200 tiles of 16 KB 7.0 / 6.8, of 4 KB 5.4 / 4.5; 576 of 4 KB 10.4 / 6.1; 2400 of 16 KB 53 / 39
//   to 32 KB     once units have a tile each: 200 tiles of 32 KB 9.2 / 9.7, 224 9.8 / 9.8, 256 10.4 / 10.2, 1152 44.8 / 42.3, 2400 83 / 71
//   more         where four to a workgroup fill more than half of the units, all of them at once, and the single ones take turns: 576 to
//                1024 tiles of 48 KB 31.4 / 30.0 to 52.7 / 44.4, of 256 KB 137 / 136 to 231 / 226; not 512 (26.3 / 27.9, 120 / 138) or
//                1152 (61.1 / 61.5, 266 / 308); 224 tiles of 64 KB would take 1.13 and of 256 KB 1.6 times as long.  Beyond five tiles a unit
//                the unevenness fades: 64 KB 1408 91.6 / 87.4, 2048 127 / 113; from 128 KB on it does not pay for itself (1408 169 / 170).
inline bool append_shares(int items, int units, int64_t tile_bytes) {
    if (tile_bytes <= 16384) return items > units * 3 / 4;
    if (tile_bytes <= 32768) return items >= units;
    return (items > 2 * units && items <= 4 * units) || (tile_bytes <= 65536 && items > 5 * units);
}

} // namespace lcsa
