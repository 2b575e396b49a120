// Work-item tables of a packed batch.
//
// The example queue of Sec. 2.2 hands over a new padded batch, with new utterance lengths, at every step,
// so the tables that cut a batch into convolution blocks and frame groups are rebuilt per call:
//   first[u]  = number of items of utterances 0..u-1 (exclusive prefix sum of per-utterance item counts)
//   items[i]  = (u, index of item i within utterance u)
// Per-utterance item counts: ceil(len_u / conv_block) convolution blocks, and units of the front end (FrameShares), whose table
// has an entry per work group only: where its equal share of all units begins.
//
// The host, which counts the items anyway to size the grids, leaves the offsets and the prefix sums in pinned
// memory; one kernel reads them from there, writes the device copies and spreads the items.  It is bound by
// latency (one round trip over the bus, a few KB): two copy commands, a scan and an items kernel per table
// took 25 us of the stream's time on a batch of 256 utterances, this kernel takes 6.  (Where a call builds other small
// tables too, this is a share of that kernel's groups: see mel_setup_kernel.)

#include "pack_device.h"

namespace aug {
namespace {

constexpr int kPackThreads = 256;

__global__ __launch_bounds__(kPackThreads) void pack_kernel(PackArgs a) {
    pack_utterances(a, (int)(blockIdx.x * blockDim.x + threadIdx.x));
}

}  // namespace

hipError_t launch_pack(hipStream_t s, const PackArgs& a) {
    if (a.n_utt <= 0) return hipSuccess;
    const int64_t threads = pack_threads(a);
    pack_kernel<<<dim3((unsigned)((threads + kPackThreads - 1) / kPackThreads)), dim3(kPackThreads), 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace aug
