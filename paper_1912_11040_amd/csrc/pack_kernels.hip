// Work-item tables of a packed batch.
//
// The example queue of Sec. 2.2 hands over a new padded batch, with new utterance lengths, at every step,
// so the tables that cut a batch into convolution blocks and frame groups are rebuilt per call:
//   first[u]  = number of items of utterances 0..u-1 (exclusive prefix sum of per-utterance item counts)
//   items[i]  = (u, index of item i within utterance u, times `step`)
// Per-utterance item counts: ceil(len_u / conv_block) convolution blocks, ceil(rows_u / frames_per_group)
// frame groups (rows_u = output rows the utterance owns).
//
// The host, which counts the items anyway to size the grids, leaves the offsets and the prefix sums in pinned
// memory; one kernel reads them from there, writes the device copies and spreads the items.  It is bound by
// latency (one round trip over the bus, a few KB): two copy commands, a scan and an items kernel per table
// took 25 us of the stream's time on a batch of 256 utterances, this kernel takes 6.

#include "aug_internal.h"

namespace aug {
namespace {

constexpr int kPackThreads = 256;

// `lanes` threads per utterance (a power of two): a few when there are many utterances, the whole group when one
// utterance may own all the items.
__global__ __launch_bounds__(kPackThreads) void pack_kernel(PackArgs a, int lanes) {
    const int at = (int)(blockIdx.x * blockDim.x + threadIdx.x);
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
    for (int i = l; i < f1 - f0; i += lanes) a.frame_items[f0 + i] = make_int2(u, i * a.frames_per_group);
}

}  // namespace

hipError_t launch_pack(hipStream_t s, const PackArgs& a) {
    if (a.n_utt <= 0) return hipSuccess;
    const int lanes = a.n_utt < 32 ? kPackThreads : 16;
    const int64_t threads = ((int64_t)a.n_utt + 1) * lanes;
    pack_kernel<<<dim3((unsigned)((threads + kPackThreads - 1) / kPackThreads)), dim3(kPackThreads), 0, s>>>(a, lanes);
    return hipGetLastError();
}

}  // namespace aug
