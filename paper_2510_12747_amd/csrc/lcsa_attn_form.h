// How a launch of the matrix-core attention kernel deals its work items (one per (head, query block)) out to workgroups.
// Host arithmetic only.
#pragma once

namespace lcsa {

enum AttnForm {
    kAttnPairs = 0,      // two items per workgroup, one per group of four wavefronts
    kAttnSplit = 1,      // one item per workgroup, its blocks shared between the groups, the partial results merged
    kAttnAlone = 2,      // one item per workgroup on one group, the other only keeps the barriers company
};

// A workgroup holds a compute unit to itself, so a launch takes rounds = ceil(workgroups / units), each as long as the blocks
// of one workgroup plus a set-up and an epilogue that cost about 3.5 blocks: rounds_pairs * (k + 3.5) for pairs,
// rounds_split * (ceil(k / 2) + 3.5) for split items (k: blocks of a full row).  Split only where that is less, i.e. for
// items in (2 n, 2 n + 1] x units and k > 7 n.  Measured on 256 units, pairs / split in us (more in profiles/): 768 items
// (3 rounds of split items for 2 of pairs) k = 4 47.8 / 50.7, k = 8 72.6 / 70.9, k = 32 219 / 194; 1080 items (5 for 3)
// k = 6 90.8 / 97.8, k = 32 329 / 306; 2160 items (9 for 5) k = 16 335 / 348, k = 32 602 / 596.  From 11 rounds on the
// workgroups have drifted apart and there is no last round to even out: 2816 items (11 for 6) k = 64 1540 / 1552, 3328
// items (13 for 7) k = 64 1745 / 1780: pairs.
// Up to one item per unit a split item always ends earlier than a pair; with one or two blocks there is nothing to share
// out and the merge costs more than it saves: 256 items, alone / split, k = 1 10.2 / 11.0 us, k = 2 13.2 / 13.5, k = 3
// 16.7 / 16.5, k = 16 50.8 / 39.8.
inline AttnForm attn_form(int items, int units, int k) {
    const int rounds_split = (items + units - 1) / units, rounds_pairs = ((items + 1) / 2 + units - 1) / units;
    if (rounds_split <= 1) return k <= 2 ? kAttnAlone : kAttnSplit;
    if (rounds_split > 9) return kAttnPairs;
    return (long long)rounds_split * (2 * ((k + 1ll) / 2) + 7) < (long long)rounds_pairs * (2ll * k + 7) ? kAttnSplit : kAttnPairs;
}

inline int attn_workgroups(AttnForm form, int items) { return form == kAttnPairs ? (items + 1) / 2 : items; }

} // namespace lcsa
