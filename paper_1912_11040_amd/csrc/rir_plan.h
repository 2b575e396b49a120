// The plan of the image sum: a response's taps cut into work items of about equal work.  Here because a call with a front end plans
// an ordinary batch in the launch that sets up the front end (mel_setup_plan_kernel); rir_kernels.hip has the other kernels.
// (Whether the compiler contracts multiplications and additions may move a cut by a tap between the two; responses do not depend on
// where they are cut.)
#pragma once

#include "aug_internal.h"

namespace aug {

constexpr int kMaxTaps = 5568;            // taps owned by one item (LDS: 8 bytes each)
constexpr int kMinTaps = 64;
// Work per item, in image visits (see WorkModel): the batch's estimated work divided by the number of
// persistent groups and by kItemsPerGroup, within limits.  Thick shells visit fewer (x, y) columns per image
// (every shell sets up all columns inside its outer radius), thin ones even out the groups' finishing
// times; every response yields at least one item, so the groups still get several items each.  Whole calls against
// 600000 at every batch: 3072 responses of 32768 taps (1024 utterances of 10 s) 7.8 -> 6.7 ms, 128 of 8000 (64 of 4 s) 180 -> 134 us.
constexpr float kItemsPerGroup = 1.25f;
// (the lower limit matters for small batches only, where items must be small for all groups to get one: 64 utterances of 4 s
// with two responses of 8000 taps each take 156 us at 300000, 130 at 50000, and the image sum alone 43.5 us anywhere from 10000 to
// 50000.  With fewer than a quarter as many responses as groups it falls with their number: most groups would have nothing, and the time is that
// of the heaviest item.  Image sum of 16 responses of 4096 taps: 19.4 us at 64000, 15.2 at 50000, 13.4 at 20000, 12.9 at 10000.)
constexpr float kMinTargetWork = 50000.f, kLeastTargetWork = 10000.f, kMaxTargetWork = 8000000.f;
constexpr float kWorkUnit = 4096.f;       // the batch total is summed in integers of this many visits
constexpr int kMaxShells = 96;            // shells per response, before those wider than kMaxTaps are split

// A usable room has sides of at least 10 cm (else the image lattice is unbounded) and a reflection
// coefficient in [0, 1] (amplitudes are summed as unsigned fixed point and must not grow with the
// reflection count); the comparisons are false for values that are not numbers.
__device__ inline bool room_ok(const float* g) {
    return (g[0] >= 0.1f) && (g[1] >= 0.1f) && (g[2] >= 0.1f) && (g[0] * g[1] * g[2] < 1e30f) &&
           (g[9] >= 0.f) && (g[9] <= 1.f);
}

// The geometry of one response: its room's row, with the microphone replaced where a room has several.
struct Room { float g[10]; };
__device__ inline Room load_room(const Rooms& rooms, int rir) {
    const float* row = rooms.geom + (size_t)(rooms.mics ? rir / rooms.n_mic : rir) * 10;
    Room r;
#pragma unroll
    for (int i = 0; i < 10; ++i) r.g[i] = row[i];
    if (rooms.mics)
#pragma unroll
        for (int i = 0; i < 3; ++i) r.g[6 + i] = rooms.mics[(size_t)rir * 3 + i];
    return r;
}

struct Item { int rir, n0, n1, cls; };

// Barrier of the work group, with the wait for this wavefront's LDS operations spelled out.  With __syncthreads the compiler
// (ROCm 7.2) emits two of the image kernel's barriers without one, that behind the candidates and that of a further go, where it
// takes every operation on the paths to them for waited for.  Reading those paths finds nothing in flight either; spelled out,
// the wait costs nothing and does not rest on that.  (The other kernels keep __syncthreads: the wait stands before all of
// their barriers but the last of the spectrum kernels' loops, where every value read has been used.)
__device__ inline void group_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0xc07f);                    // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// inclusive sum over the lanes of a wavefront: shifts within rows of sixteen lanes, then the rows' last lanes passed on
__device__ inline int wave_inclusive_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);      // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);      // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);      // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);      // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);     // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);     // row_bcast:31 into rows 2 and 3
    return v;
}

constexpr int kClasses = 32;            // cost classes for the order in which items are handed out
// ctrl: [0] number of items, [1] next item to hand out, [2 .. 2+kClasses) items per class,
// [2+kClasses .. 2+2 kClasses) next free slot of each class in the sorted table, then the batch's
// estimated work in units of kWorkUnit
constexpr int kCtrlWork = 2 + 2 * kClasses;
constexpr int kCtrlInts = kCtrlWork + 1;

// Estimate of the work in a response's taps, in units of one image visit: the images it keeps plus, for every live (x image, y
// image) column inside an item's outer radius, twelve visits' worth of set-up and of images visited in vain at its ends, and
// for every item what its tables cost.
// What the reflection cut keeps: an image in direction u at distance d has about d (|ux|/Lx + |uy|/Ly + |uz|/Lz)
// reflections, so it is the share of directions whose reflections per metre stay under cut / d.  Over an octant that
// sum runs from the smallest of the 1/L to the length of the vector (1/Lx, 1/Ly, 1/Lz); the share below a fraction x of
// that range is x^2.5 to within 0.02 on average over rooms of 3 x 3 x 2.4 to 10 x 8 x 4 m.  (Counting a lattice of
// directions for every item, with library divisions and powers, took most of the plan's time.)
// The kept images within a radius are summed up at kKnots radii; between two of them the share is taken as constant.
// (Eight knots plan no better and take 2000 responses 1.5 us more.)
constexpr int kKnots = 4;
constexpr float kColumnWork = 12.f, kItemWork = 13500.f;
struct WorkModel {
    float images, columns;       // per cubic tap, per square tap
    float metres, inv_log2_beta; // per tap; 0: no cut
    float least, inv_range;      // of the reflections per metre
    float step;                  // taps between knots
    float kept[kKnots + 1];      // images kept within i steps
    float column_work[kKnots];   // of an item that ends in the middle of step i
    // the fraction x of the range of reflections per metre that the cut leaves at tap n
    __device__ float fraction(float n) const {
        const float d = n * metres;
        if (!(inv_log2_beta < 0.f) || d < 1e-3f) return 1.f;
        const float per_metre = (__builtin_amdgcn_logf(12.566371f * d) - 57.f) * inv_log2_beta * __builtin_amdgcn_rcpf(d);
        // (0.19^2.5 = 1/64: the estimate is poor below)
        return fminf(fmaxf((per_metre - least) * inv_range, 0.19f), 1.f);
    }
    __device__ float columns_within(float n) const {
        const float x = fraction(0.7f * n);
        return columns * n * n * x * __builtin_amdgcn_sqrtf(x);
    }
    __device__ float item(float n0, float n1) const {
        const float x = fraction(0.5f * (n0 + n1));
        return images * (n1 * n1 * n1 - n0 * n0 * n0) * x * x * __builtin_amdgcn_sqrtf(x) + columns_within(n1) + kItemWork;
    }
    __device__ float total(float rir_len) const { return kept[kKnots] + columns_within(rir_len); }
};

__device__ inline WorkModel work_model(const float* g, int rir_len, double k_fs_c) {
    WorkModel m;
    m.metres = __builtin_amdgcn_rcpf((float)k_fs_c);
    const float ix = __builtin_amdgcn_rcpf(g[0]), iy = __builtin_amdgcn_rcpf(g[1]), iz = __builtin_amdgcn_rcpf(g[2]);
    m.images = 4.18879f * (m.metres * m.metres) * m.metres * ix * iy * iz;
    m.columns = kColumnWork * 3.14159265f * (m.metres * m.metres) * ix * iy;
    m.inv_log2_beta = (g[9] > 0.f && g[9] < 1.f) ? __builtin_amdgcn_rcpf(__builtin_amdgcn_logf(g[9])) : 0.f;
    m.least = fminf(fminf(ix, iy), iz);
    m.inv_range = __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(ix * ix + iy * iy + iz * iz) - m.least);
    m.step = (float)rir_len * (1.f / kKnots);
    m.kept[0] = 0.f;
#pragma unroll
    for (int i = 0; i < kKnots; ++i) {
        const float x = m.fraction(m.step * ((float)i + 0.5f));
        const float n = m.step * ((float)i + 0.5f), root = x * __builtin_amdgcn_sqrtf(x);
        m.kept[i + 1] = m.kept[i] + m.images * m.step * m.step * m.step * (float)(3 * i * (i + 1) + 1) * x * root;
        m.column_work[i] = m.columns * n * n * root + kItemWork;
    }
    return m;
}

// estimated work of a whole response (0 for a room that is not usable)
__device__ inline float response_work(const float* g, int rir_len, double k_fs_c) {
    return room_ok(g) ? work_model(g, rir_len, k_fs_c).total((float)rir_len) : 0.f;
}

// Work per item that a batch of `units` work units (kWorkUnit visits each) aims at.
__device__ inline float item_target(int units, int n_groups, int n_rir) {
    const float least = fminf(fmaxf(kMinTargetWork * 4.f * (float)n_rir / (float)n_groups, kLeastTargetWork), kMinTargetWork);
    return fminf(fmaxf(kWorkUnit * (float)units / ((float)n_groups * kItemsPerGroup), least), kMaxTargetWork);
}

// Cut the taps of a response into shells of about equal work, and those wider than kMaxTaps into parts: calls
// take(lower, upper) for the shells lane, lane + lanes, ...; returns their number.
// A shell pays for all columns inside its outer radius, so the outer ones get fewer images: the number of shells per image kept
// goes as 1 / (target - columns' work).  (Shells of equal volume left the ones at middle distance, before the cut takes most
// images away, several times the work of the others: 32 responses of 32768 taps waited for one item, five times the mean of a
// work group.)  The bounds are a closed form, so that a response's shells can be shared among threads: one after the
// other they took 0.6 us each.
// Callers that first count and then write run it twice rather than keep a table of bounds.
template <class Take>
__device__ inline int cut_shells(const WorkModel& model, bool ok, int rir_len, float target, int lane, int lanes, Take take) {
    const float most = fminf((float)kMaxShells, fmaxf((float)(rir_len / kMinTaps), 1.f));
    float within[kKnots + 1];                             // shells up to the knots
    within[0] = 0.f;
#pragma unroll
    for (int i = 0; i < kKnots; ++i)
        within[i + 1] = within[i] + (model.kept[i + 1] - model.kept[i]) * __builtin_amdgcn_rcpf(fmaxf(target - model.column_work[i], 0.25f * target));
    const int shells = ok ? (int)fminf(fmaxf(ceilf(model.total((float)rir_len) / target), 1.f), most) : 1;
    const float share = within[kKnots] / (float)shells;
    auto bound = [&](int j) {
        if (j == 0 || j >= shells) return j == 0 ? 0 : rir_len;
        const float w = share * (float)j;
        float from = 0.f, to = within[1], begin = 0.f;
#pragma unroll
        for (int i = 1; i < kKnots; ++i)
            if (w >= within[i]) {
                from = within[i];
                to = within[i + 1];
                begin = model.step * (float)i;
            }
        const float end = begin + model.step, b3 = begin * begin * begin;
        const float n3 = b3 + (end * end * end - b3) * (w - from) * __builtin_amdgcn_rcpf(fmaxf(to - from, 1e-20f));
        return n3 > 0.f ? min((int)__builtin_amdgcn_exp2f(__builtin_amdgcn_logf(n3) * (1.f / 3.f)), rir_len) : 0;
    };
    int count = 0;
#pragma unroll 1
    for (int j = lane; j < shells; j += lanes) {
        int ends[2];
#pragma unroll 1
        for (int e = 0; e < 2; ++e) {
            ends[0] = ends[1];
            ends[1] = bound(j + e);
        }
        // (from the outside in: every shell sets up all columns inside its outer radius, so that what is left over belongs at
        // the centre)
        int to = ends[1];
#pragma unroll 1
        while (to > ends[0]) {                            // (not where two bounds round to one tap)
            const int from = max(ends[0], to - kMaxTaps);
            take(from, to);
            to = from;
            ++count;
        }
    }
    return count;
}

// cost class of an item (0 = heaviest)
__device__ inline int item_class(const WorkModel& model, bool ok, int n0, int n1) {
    if (!ok) return kClasses - 1;
    return min(max((int)(2.5f * (24.93f - __builtin_amdgcn_logf(model.item((float)n0, (float)n1)))), 0), kClasses - 1);     // 2^24.93 = 3.2e7
}

// The whole plan in one work group, for batches of at most kPlanMost responses (beyond, the four launches of the kernels
// around this one).  As many threads per response as there are, up to 64: first the batch's work, then the shells, their places
// in the table from a counter, and their classes, then all threads over the items for the counting sort.  Between the two the
// items lie in LDS, or in `unsorted` if there are more than it holds.  Leaves ctrl[0] = number of items, ctrl[1] = 0.
// Latency bound: the 16 waves of one CU, and instructions that no launch before has left in the cache, so the code is kept
// short (unrolled, with passes of their own for counting and writing, 16 responses took 12 us instead of 6).
constexpr int kPlanItems = 8192;
static_assert(AUG_MAX_RIR_LEN < 1 << 16 && kPlanMost <= 1 << 12 && kClasses <= 1 << 5, "the packing of items in LDS");
// What it keeps in LDS.
struct PlanShared {
    unsigned long long held[kPlanItems];
    int census[kClasses], cursor[kClasses];
    int units, items;
};
__device__ inline void plan_all(PlanShared& sh, int n_rir, const Rooms& rooms, int rir_len, double k_fs_c, Item* __restrict__ sorted,
                                Item* __restrict__ unsorted, int* __restrict__ ctrl, int n_groups) {
    unsigned long long* const held = sh.held;
    int *const census = sh.census, *const cursor = sh.cursor, &s_units = sh.units, &s_items = sh.items;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid < kClasses) census[tid] = 0;
    if (tid == 0) s_units = s_items = 0;
    group_sync();

    int lg = 0;
    while (lg < 6 && n_rir << (lg + 1) <= kPlanThreads) ++lg;
    const int lanes = 1 << lg, n = n_rir << lg;
    auto units_of = [&](const WorkModel& model, bool ok) {
        return ok ? (int)fminf(model.total((float)rir_len) * (1.f / kWorkUnit), 500000.f) + 1 : 1;
    };
    auto write_items = [&](const WorkModel& model, bool ok, int r, int share, float target) {
        cut_shells(model, ok, rir_len, target, share, lanes, [&](int lo, int hi) {
            const int cls = item_class(model, ok, lo, hi), at = atomicAdd(&s_items, 1);
            if (at < kPlanItems) held[at] = (unsigned long long)(unsigned int)(lo | hi << 16) | (unsigned long long)(unsigned int)(r | cls << 12) << 32;
            else unsorted[at] = Item{r, lo, hi, cls};
            atomicAdd(&census[cls], 1);
        });
    };
    if (n_rir <= kPlanThreads) {                          // each thread has one response, or a share of one
        const int r = min(tid >> lg, n_rir - 1), share = tid & (lanes - 1);
        const Room room = load_room(rooms, r);
        const bool ok = room_ok(room.g);
        const WorkModel model = work_model(room.g, rir_len, k_fs_c);
        if (share == 0 && tid < n) atomicAdd(&s_units, units_of(model, ok));
        group_sync();
        if (tid < n) write_items(model, ok, r, share, item_target(s_units, n_groups, n_rir));
    } else {
#pragma unroll 1
        for (int pass = 0; pass < 2; ++pass) {
            int units = 0;
#pragma unroll 1
            for (int r = tid; r < n_rir; r += kPlanThreads) {
                const Room room = load_room(rooms, r);
                const bool ok = room_ok(room.g);
                const WorkModel model = work_model(room.g, rir_len, k_fs_c);
                if (pass == 0) units += units_of(model, ok);
                else write_items(model, ok, r, 0, item_target(s_units, n_groups, n_rir));
            }
            if (pass == 0) {
                atomicAdd(&s_units, units);
                group_sync();
            }
        }
    }
    group_sync();                                          // (the group's writes to `unsorted` are visible to it)
    const int n_items = s_items;
    if (wave == 0) {
        const int mine = lane < kClasses ? census[lane] : 0;
        const int incl_classes = wave_inclusive_scan(mine);
        if (lane < kClasses) cursor[lane] = incl_classes - mine;
        if (lane == 0) {
            ctrl[0] = n_items;
            ctrl[1] = 0;
        }
    }
    group_sync();
    for (int i = tid; i < n_items; i += kPlanThreads) {
        Item it;
        if (i < kPlanItems) {
            const unsigned int lo = (unsigned int)held[i], hi = (unsigned int)(held[i] >> 32);
            it = Item{(int)(hi & 4095u), (int)(lo & 65535u), (int)(lo >> 16), (int)(hi >> 12)};
        } else {
            it = unsorted[i];
        }
        sorted[atomicAdd(&cursor[it.cls], 1)] = it;
    }
}

}  // namespace aug
