// The packing of a batch (pack_kernels.hip) as a share of a kernel's threads.
#pragma once

#include "aug_internal.h"

namespace aug {

// Threads per utterance (a power of two): a few when there are many utterances, more when one utterance may own all
// the items.
__host__ __device__ inline int pack_lanes(const PackArgs& a) { return a.n_utt < 32 ? 256 : 16; }
inline int64_t pack_threads(const PackArgs& a) { return ((int64_t)a.n_utt + 1) * pack_lanes(a); }

// thread `at` of pack_threads
__device__ inline void pack_utterances(const PackArgs& a, int at) {
    const int lanes = pack_lanes(a);
    const int u = at / lanes, l = at % lanes;
    if (u > a.n_utt) return;
    const bool last = u == a.n_utt;                     // entry n_utt of every array, no items
    int64_t off = 0, foff = 0;
    int c0 = 0, c1 = 0, f0 = 0, f1 = 0;
    if (l == 0 && a.offsets) off = a.offsets[u];
    if (l == 0 && a.frame_offsets) foff = a.frame_offsets[u];
    if (a.conv_first) {
        c0 = a.conv_first[u];
        c1 = last ? c0 : a.conv_first[u + 1];
    }
    if (a.frame_first) {
        f0 = a.frame_first[u];
        f1 = last ? f0 : a.frame_first[u + 1];
    }
    if (l == 0) {
        if (a.offsets) a.d_offsets[u] = off;
        if (a.frame_offsets) a.d_frame_offsets[u] = foff;
        if (a.conv_first) a.d_conv_first[u] = c0;
    }
    for (int i = l; i < c1 - c0; i += lanes) a.conv_items[c0 + i] = make_int2(u, i);
    if (f1 > f0) {
        // the groups whose first unit is one of this utterance's
        const FrameShares& s = a.shares;
        const int of_longer = s.longer * (s.per_group + 1);
        auto group_at = [&](int unit) {                 // the first group that begins at this unit or behind it (units < 2^30)
            return unit <= of_longer ? (int)((unsigned int)(unit + s.per_group) / (unsigned int)(s.per_group + 1))
                                     : s.longer + (int)((unsigned int)(unit - of_longer + s.per_group - 1) / (unsigned int)s.per_group);
        };
        const int end = group_at(f1);
        for (int g = group_at(f0) + l; g < end; g += lanes) {
            const int first = g * s.per_group + (g < s.longer ? g : s.longer);
            a.frame_items[g] = make_int2(u, first - f0);
        }
    }
}

}  // namespace aug
