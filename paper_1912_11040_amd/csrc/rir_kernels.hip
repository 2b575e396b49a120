// Image-method room impulse responses (the acoustic simulator of Sec. 2.3 computes
// them on the fly for every training example).
//
// h[n] = sum over image sources with floor(d fs/c + 0.5) == n of beta^k / (4 pi d),
// d = distance image -> microphone, k = number of wall reflections of that image.
// Along one axis the images of a source at s between walls at 0 and L are
// (1 - 2q) s + 2 n L, q in {0,1}, n integer, reflected |n - q| + |n| times.
//
// The tap index is integer work decided by floating point, so it follows one fixed
// fp64 recipe with no contraction:
//     d2 = (dx*dx + dy*dy) + dz*dz;  idx = floor(sqrt(d2) * (fs/c) + 0.5)
// An estimate of sqrt from the hardware's double-precision rsq decides the index whenever the result is
// farther from a rounding boundary than the estimate's error bound; the images nearer to one take a Newton
// step more, and those that this leaves open, rarely, the exact correctly-rounded sqrt.
//
// Layout of the work
//   * plan kernels: one thread per response cuts its taps into shells [n0, n1) of about
//     equal image count (equal volume of the spherical shell) and at most kMaxTaps taps; the shell size
//     follows the batch's estimated work per persistent group.  Every shell gets an estimate of its work
//     and a counting sort orders the items heaviest first.
//   * image kernel: persistent work groups fetch items from a counter.  An item owns its
//     taps, so sums live in LDS and are stored once, without global atomics.
//     The z images of the response (both q, both signs) are merged into one LDS table sorted by
//     dz*dz, so the images of an (x image, y image) column that can fall inside the shell are one
//     contiguous range of that table between r_in^2 - a and r_out^2 - a, whose ends are counted from the
//     two arithmetic progressions that the axis's images form rather than searched for.
//     The y images are sorted the same way, so the live columns of an x image are a prefix of the
//     y table; a prefix sum over the x images numbers the live columns and dead ones are never seen.
//     A wave takes 64 live columns at a time; their z ranges are cut into pieces of at most kPiece
//     images, a wave scan numbers the pieces, and lanes take pieces 64 at a time (a piece finds its column by
//     counting bits in a map of the columns' first pieces) and walk them, two images side by side.
//     Bound by issue and by LDS about equally (256 x 16000 taps: vector units 0.80, LDS 0.75 of the time, half of that
//     conflicts of reads at scattered table entries and of sums at scattered taps).
//     Rooms so flat or narrow that an axis has more images than the tables hold, and positions far outside
//     the room, take a plain path (all columns of the bounding box, every z image of a live column).
//   * amplitudes accumulate as 64-bit fixed point (2^-56, each increment rounded to the nearest unit)
//     with integer LDS atomics: gfx950 executes float LDS atomics about thirty times slower than integer
//     ones, and integer sums do not depend on the order of arrival nor on how a batch is cut into items.

#include "aug_internal.h"

namespace aug {
namespace {

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kMaxTaps = 5632;            // taps owned by one item (LDS: 8 bytes each)
constexpr int kMinTaps = 64;
constexpr int kPow = 1024;                // beta^k table entries held in LDS
constexpr int kAxisCap = 320;             // y or z images per q held in the sorted LDS tables 
// Images per piece, even (two are worked on side by side).  A column's pieces start kPiece sixteen-byte entries apart, so
// the number also decides which LDS banks neighbouring lanes read: 2000 responses of 8000 taps take 312 us at 10 and
// 14, 320 at 12, 318 at 18, 395 at 16 (all lanes of a column on the same banks).
constexpr int kPiece = 14;
constexpr int kStartWords = 32;           // pieces are dealt in chunks of 32 * kStartWords (one bit each in LDS)
// Work per item, in image visits (see item_cost): the batch's estimated work divided by the number of
// persistent groups and by kItemsPerGroup, within limits.  Thick shells visit fewer (x, y) columns per image
// (every shell sets up all columns inside its outer radius), thin ones even out the groups' finishing
// times; every response yields at least one item, so the groups still get several items each.  Measured:
// 16000-tap batch 0.89 -> 0.80 ms, 32768-tap batch 12.8 -> 7.6 ms against a fixed 600000.
constexpr float kItemsPerGroup = 1.25f;
// (the lower limit matters for small batches only, where items must be small for all groups to get one:
// 64 utterances with 8000-tap responses take 0.122 ms at 300000, 0.080 ms at 50000)
constexpr float kMinTargetWork = 50000.f, kMaxTargetWork = 8000000.f;
constexpr float kWorkUnit = 4096.f;       // the batch total is summed in integers of this many visits
constexpr int kMaxShells = 96;            // volume-balanced shells per response, at most

#pragma clang fp contract(off)

struct Axis {
    double room, src, mic;
};

// delta of image (q, n) to the microphone along one axis, in the reference operation order
__device__ inline double axis_delta(const Axis& a, int q, int n) {
    const double sgn = q ? -1.0 : 1.0;
    const double coord = __dadd_rn(__dmul_rn(sgn, a.src), __dmul_rn(__dmul_rn(2.0, (double)n), a.room));
    return __dsub_rn(coord, a.mic);
}

__device__ inline int iabs(int v) { return v < 0 ? -v : v; }

// A value that every lane of the wavefront has computed alike, moved to scalar registers: what an item's
// geometry determines is the same in all lanes and would otherwise occupy vector registers for the whole item.
__device__ inline int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline float uni(float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); }
__device__ inline double uni(double v) { return __hiloint2double(uni(__double2hiint(v)), uni(__double2loint(v))); }

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

__device__ inline void wave_sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
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

// Estimate of the work in a response's taps [n0, n1), in units of one image visit: the images it keeps plus about twelve
// visits' worth of set-up for every live (x image, y image) column inside its outer radius.
// What the reflection cut keeps: an image in direction u at distance d has about d (|ux|/Lx + |uy|/Ly + |uz|/Lz)
// reflections, so it is the share of directions whose reflections per metre stay under cut / d.  Over an octant that
// sum runs from the smallest of the 1/L to the length of the vector (1/Lx, 1/Ly, 1/Lz); the share below a fraction x of
// that range is x^2.5 to within 0.02 on average over rooms of 3 x 3 x 2.4 to 10 x 8 x 4 m.  (Counting a lattice of
// directions for every item, with library divisions and powers, took most of the plan's time.)
struct WorkModel {
    float images, columns;       // per cubic tap, per square tap
    float metres, inv_log2_beta; // per tap; 0: no cut
    float least, inv_range;      // of the reflections per metre
    __device__ float operator()(float n0, float n1) const {
        float kept = 1.f, kept_columns = 1.f;
        const float d = 0.5f * (n0 + n1) * metres;
        if (inv_log2_beta < 0.f && d > 1e-3f) {
            const float per_metre = (__builtin_amdgcn_logf(12.566371f * d) - 57.f) * inv_log2_beta * __builtin_amdgcn_rcpf(d);
            const float x = fminf(fmaxf((per_metre - least) * inv_range, 0.19f), 1.f);     // (0.19^2.5 = 1/64)
            const float root = __builtin_amdgcn_sqrtf(x);
            kept = x * x * root;
            kept_columns = x * root;
        }
        return images * (n1 * n1 * n1 - n0 * n0 * n0) * kept + columns * n1 * n1 * kept_columns;
    }
};

__device__ inline WorkModel work_model(const float* g, double k_fs_c) {
    WorkModel m;
    m.metres = __builtin_amdgcn_rcpf((float)k_fs_c);
    const float ix = __builtin_amdgcn_rcpf(g[0]), iy = __builtin_amdgcn_rcpf(g[1]), iz = __builtin_amdgcn_rcpf(g[2]);
    m.images = 4.18879f * (m.metres * m.metres) * m.metres * ix * iy * iz;
    m.columns = 12.f * 3.14159265f * (m.metres * m.metres) * ix * iy;
    m.inv_log2_beta = (g[9] > 0.f && g[9] < 1.f) ? __builtin_amdgcn_rcpf(__builtin_amdgcn_logf(g[9])) : 0.f;
    m.least = fminf(fminf(ix, iy), iz);
    m.inv_range = __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(ix * ix + iy * iy + iz * iz) - m.least);
    return m;
}

// estimated work of a whole response (0 for a room that is not usable)
__device__ inline float response_work(const float* g, int rir_len, double k_fs_c) {
    return room_ok(g) ? work_model(g, k_fs_c)(0.f, (float)rir_len) : 0.f;
}

// one thread per response: the batch's estimated work (an integer sum, so it does not depend on the order)
__global__ void rir_work_kernel(int n_rir, Rooms rooms, int rir_len, double k_fs_c,
                                int* __restrict__ ctrl) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    int units = 0;
    if (r < n_rir) units = (int)fminf(response_work(load_room(rooms, r).g, rir_len, k_fs_c) / kWorkUnit, 500000.f) + 1;
    for (int off = 32; off > 0; off >>= 1) units += __shfl_down(units, off, 64);      // one atomic per wavefront
    if ((threadIdx.x & 63) == 0 && units) atomicAdd(&ctrl[kCtrlWork], units);
}

// Work per item that a batch of `units` work units (kWorkUnit visits each) aims at.
__device__ inline float item_target(int units, int n_groups) {
    return fminf(fmaxf(kWorkUnit * (float)units / ((float)n_groups * kItemsPerGroup), kMinTargetWork), kMaxTargetWork);
}

// Cut the taps of a response of estimated work `work` into shells of about equal image count (equal volume), at most
// kMaxTaps wide: calls take(lower, upper) for every shell, outermost first; returns their number.
// Shells are cut from the outside in: every shell sets up all (x, y) columns inside its outer radius, so
// where the tap limit, not the work, decides the width it is the inner shells, with few columns, that
// should be the many and the narrow ones, and the left-over sliver belongs at the centre.
// (Single precision: the cuts need not be exact, and the library's cube root in double precision took a microsecond
// per shell.  Callers that first count and then write run it twice rather than keep a table of bounds.)
template <class Take>
__device__ inline int cut_shells(float work, int rir_len, float target, int items_per_rir, Take take) {
    const float shells = fminf(fmaxf(ceilf(work / target), 1.f), (float)kMaxShells);
    const float step = (float)rir_len * (float)rir_len * (float)rir_len / shells;
    int count = 0, hi = rir_len;
    while (hi > 0 && count < items_per_rir - 1) {
        const float inner = (float)hi * (float)hi * (float)hi - step;
        int lo = inner > 0.f ? (int)__builtin_amdgcn_exp2f(__builtin_amdgcn_logf(inner) * (1.f / 3.f)) : 0;
        lo = min(lo, hi - kMinTaps);
        lo = max(max(lo, hi - kMaxTaps), 0);
        if (lo < kMinTaps && hi <= kMaxTaps) lo = 0;              // no sliver at the centre
        take(lo, hi);
        ++count;
        hi = lo;
    }
    while (hi > 0 && count < items_per_rir) {                       // out of table space: cannot happen with the
        const int lo = max(hi - kMaxTaps, 0);                       // sizes chosen by the host
        take(lo, hi);
        ++count;
        hi = lo;
    }
    return count;
}

// cost class of an item (0 = heaviest)
__device__ inline int item_class(const WorkModel& model, bool ok, int n0, int n1) {
    if (!ok) return kClasses - 1;
    const float cost = model((float)n0, (float)n1);
    return min(max((int)(2.5f * (24.93f - __builtin_amdgcn_logf(fmaxf(cost, 1.f)))), 0), kClasses - 1);     // 2^24.93 = 3.2e7
}

// One thread per response: cut its taps into shells and append them to the unsorted item table, with their cost classes
// and the class census (taken in LDS first: one global atomic per class and group, not per item).
__global__ void rir_plan_kernel(int n_rir, Rooms rooms, int rir_len, double k_fs_c, Item* __restrict__ unsorted,
                                int items_per_rir, int* __restrict__ ctrl, int n_groups) {
    __shared__ int census[kClasses];
    if (threadIdx.x < kClasses) census[threadIdx.x] = 0;
    __syncthreads();
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r < n_rir) {
        const Room room = load_room(rooms, r);
        const float work = response_work(room.g, rir_len, k_fs_c), target = item_target(ctrl[kCtrlWork], n_groups);
        const int count = cut_shells(work, rir_len, target, items_per_rir, [](int, int) {});
        const WorkModel model = work_model(room.g, k_fs_c);
        const bool ok = room_ok(room.g);
        int at = atomicAdd(&ctrl[0], count);
        cut_shells(work, rir_len, target, items_per_rir, [&](int lo, int hi) {
            const int cls = item_class(model, ok, lo, hi);
            unsorted[at++] = Item{r, lo, hi, cls};
            atomicAdd(&census[cls], 1);
        });
    }
    __syncthreads();
    if (threadIdx.x < kClasses && census[threadIdx.x]) atomicAdd(&ctrl[2 + threadIdx.x], census[threadIdx.x]);
}

// The whole plan in one work group, for batches of at most kPlanRows * kPlanThreads responses (beyond, the four launches
// of the kernels around this one).  A thread per
// response, up to kPlanRows in turn, for the batch's work, the shells (their places in the table by a scan, not by
// atomics) and their classes, then all threads over the items for the counting sort.  Between the two the items lie in
// LDS, or in `unsorted` if there are more than it holds.  Leaves ctrl[0] = number of items, ctrl[1] = 0.
// Latency bound: the 16 waves of one CU.
constexpr int kPlanThreads = 1024, kPlanRows = 4;
constexpr int kPlanItems = 8192;
static_assert(AUG_MAX_RIR_LEN < 1 << 16 && kPlanRows * kPlanThreads <= 1 << 12 && kClasses <= 1 << 5, "the packing of items in LDS");
__global__ __launch_bounds__(kPlanThreads) void rir_plan_all_kernel(
    int n_rir, Rooms rooms, int rir_len, double k_fs_c, Item* __restrict__ sorted,
    Item* __restrict__ unsorted, int items_per_rir, int* __restrict__ ctrl, int n_groups) {
    __shared__ unsigned long long held[kPlanItems];
    __shared__ int part[2][kPlanThreads / 64];
    __shared__ int census[kClasses], cursor[kClasses];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid < kClasses) census[tid] = 0;

    float work[kPlanRows];
    int units = 0;
#pragma unroll
    for (int k = 0; k < kPlanRows; ++k) {
        const int r = tid + k * kPlanThreads;
        work[k] = 0.f;
        if (r < n_rir) {
            work[k] = response_work(load_room(rooms, r).g, rir_len, k_fs_c);
            units += (int)fminf(work[k] * (1.f / kWorkUnit), 500000.f) + 1;
        }
    }
    units = wave_inclusive_scan(units);
    if (lane == 63) part[0][wave] = units;
    __syncthreads();
    int total_units = 0;
    for (int w = 0; w < kPlanThreads / 64; ++w) total_units += part[0][w];
    const float target = item_target(total_units, n_groups);

    int count = 0;
#pragma unroll
    for (int k = 0; k < kPlanRows; ++k)
        if (tid + k * kPlanThreads < n_rir) count += cut_shells(work[k], rir_len, target, items_per_rir, [](int, int) {});
    const int incl = wave_inclusive_scan(count);
    if (lane == 63) part[1][wave] = incl;
    __syncthreads();
    int at = incl - count, n_items = 0;
    for (int w = 0; w < kPlanThreads / 64; ++w) {
        if (w < wave) at += part[1][w];
        n_items += part[1][w];
    }
    const bool in_lds = n_items <= kPlanItems;
    auto pack = [](const Item& it) {
        return (unsigned long long)(unsigned int)(it.n0 | it.n1 << 16) | (unsigned long long)(unsigned int)(it.rir | it.cls << 12) << 32;
    };
    auto get = [&](int i) {
        if (!in_lds) return unsorted[i];
        const unsigned int lo = (unsigned int)held[i], hi = (unsigned int)(held[i] >> 32);
        return Item{(int)(hi & 4095u), (int)(lo & 65535u), (int)(lo >> 16), (int)(hi >> 12)};
    };
#pragma unroll
    for (int k = 0; k < kPlanRows; ++k) {
        const int r = tid + k * kPlanThreads;
        if (r >= n_rir) continue;
        const Room room = load_room(rooms, r);
        const WorkModel model = work_model(room.g, k_fs_c);
        const bool ok = room_ok(room.g);
        cut_shells(work[k], rir_len, target, items_per_rir, [&](int lo, int hi) {
            const Item it{r, lo, hi, item_class(model, ok, lo, hi)};
            if (in_lds) held[at] = pack(it);
            else unsorted[at] = it;
            ++at;
            atomicAdd(&census[it.cls], 1);
        });
    }
    __syncthreads();                                   // (the group's writes to `unsorted` are visible to it)
    if (wave == 0) {
        const int mine = lane < kClasses ? census[lane] : 0;
        const int incl_classes = wave_inclusive_scan(mine);
        if (lane < kClasses) cursor[lane] = incl_classes - mine;
        if (lane == 0) {
            ctrl[0] = n_items;
            ctrl[1] = 0;
        }
    }
    __syncthreads();
    for (int i = tid; i < n_items; i += kPlanThreads) {
        const Item it = get(i);
        sorted[atomicAdd(&cursor[it.cls], 1)] = it;
    }
}

// Items move to their class's stretch of the sorted table, heaviest class first: persistent groups then take
// the heaviest items first and finish on the light ones, which evens out their finishing times.
// ctrl[2 + c] is the census of class c, ctrl[2 + kClasses + c] the cursor within its stretch.
__global__ void rir_sort_items_kernel(const Item* __restrict__ unsorted, Item* __restrict__ sorted, int* __restrict__ ctrl) {
    // (a work group numbers its items of a class in LDS and takes their places in the class's stretch with
    // one global atomic per class)
    __shared__ int first_slot[kClasses], mine[kClasses];
    if (threadIdx.x < kClasses) mine[threadIdx.x] = 0;
    if (threadIdx.x == 0) {
        int at = 0;
        for (int c = 0; c < kClasses; ++c) {
            first_slot[c] = at;
            at += ctrl[2 + c];
        }
    }
    __syncthreads();
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const bool have = i < ctrl[0];
    Item it;
    int rank = 0;
    if (have) {
        it = unsorted[i];
        rank = atomicAdd(&mine[it.cls], 1);
    }
    __syncthreads();
    if (threadIdx.x < kClasses && mine[threadIdx.x])
        first_slot[threadIdx.x] += atomicAdd(&ctrl[2 + kClasses + threadIdx.x], mine[threadIdx.x]);
    __syncthreads();
    if (have) sorted[first_slot[it.cls] + rank] = it;
}

// per-column record shared through LDS between the lane that built it and the lanes that walk its pieces
struct __align__(16) Column {
    double a;                    // dx*dx + dy*dy
    float bxy;                   // beta^(reflections along x and y)
    int place;                   // of the range of the sorted z table that can fall inside the shell: its end, and above
                                 // bit 10 its start less kPiece times the column's first piece, so that piece p
                                 // starts at that number plus kPiece p
};
static_assert(sizeof(Column) == 16, "column records are packed");
static_assert(2 * kAxisCap < 1024 && kPiece % 2 == 0, "the fields of Column::place, and pairs of images");

// One image along an axis, as stored in the sorted tables: key = squared distance to the microphone
// along that axis (reference operation order); aux = beta^reflections (z axis) or the reflection count
// (y axis).  Sixteen bytes: one LDS read per entry.
struct __align__(16) AxisImage {
    double key;
    double aux;
};

struct WalkCtx {
    double k_fs_c;
    double beta;
    double quick_k;         // fs/c, less the middle of the hardware estimate's error
    double quick_shift;     // 0.5 + margin - (n0 - 1) + kQuickMagic
    int quick_margin2;      // quick estimates whose 16-bit fraction is below this are settled by tap_slot
    double shift;           // 0.5 + guard - (n0 - 1)
    double guard2;
    int n0, n1;             // the item's taps.  Slots are tap - n0 + 1: slot 0 takes what belongs below the item, slot
                            // n1 - n0 + 1 what belongs above it; neither is read
};

// the reference recipe, out of line so that the table walk stays short
__device__ __attribute__((noinline)) int exact_tap(double d2, double k_fs_c) {
    const double d = __dsqrt_rn(d2);
    return (int)__dadd_rn(__dmul_rn(d, k_fs_c), 0.5);     // positive: truncation is floor
}

// Largest reflection count k whose amplitude beta^k / (4 pi d) can still add to a sum in the 2^-56 fixed
// point at distance d_min or beyond.  Increments are rounded to the nearest unit (or truncated, in the
// innermost item), so an amplitude below half a unit adds exactly zero; the cut is taken at 2^-57.5, a
// margin of a factor 1.41 under that, plus one count of slack, which covers the rounding of this estimate
// for every beta that the limit of 10^6 counts lets through.  "No limit" when beta is 0, >= 1
// (log2_beta == 0 encodes both) or d_min is tiny.
__device__ inline int reflection_cut(float log2_beta, float d_min) {
    if (!(log2_beta < 0.f) || !(d_min > 1e-3f)) return 1 << 20;
    // beta^k >= 4 pi d 2^-57.5  <=>  k <= (log2(4 pi d) - 57.5) / log2(beta)
    const float k = (__log2f(12.566371f * d_min) - 57.5f) / log2_beta;
    return k > 1.0e6f ? (1 << 20) : (int)k + 2;
}

// Slot (tap - n0 + 1) of an image at squared distance d2, given y, the hardware's estimate of 1/sqrt(d2).
// One Newton step on the root leaves d fs/c good to ~1e-10 taps; shifted up by the guard, its fraction falls below
// 2 guard exactly when the true value may lie within the guard of a rounding boundary, and only then is the
// reference recipe evaluated.
__device__ inline int tap_slot(const WalkCtx& w, double d2, double y) {
    const double s0 = __dmul_rn(d2, y);                    // sqrt(d2) to 2^-24
    const double res = fma(-s0, s0, d2);                   // exact residual
    const double s1 = fma(__dmul_rn(res, y), 0.5, s0);     // one Newton step: ~4e-15 relative
    const double t = fma(s1, w.k_fs_c, w.shift);
    int slot = (int)t;
    if (__builtin_amdgcn_fract(t) < w.guard2) slot = exact_tap(d2, w.k_fs_c) - (w.n0 - 1);
    return slot;
}

// The table walk first asks for less.  d2 rsq(d2) without the Newton step is the distance to within the hardware
// estimate's own error, which over all 2^31 leading mantissas of [1, 4) (three fillings of the remaining bits) lies
// between -3.24 and +7.10 units of 2^-27; with the middle of that range taken out of fs/c the error is below
// 5.2 * 2^-27: 3e-4 taps at tap 8000.  Adding 1.5 * 2^36 leaves slot and fraction as two sixteen-bit halves of the
// sum's low word: the address is a shift and a mask, the test one 16-bit comparison, and the Newton step,
// conversion, fraction and double-precision comparison are not needed (40 instead of 60 issue cycles, without rsq,
// per image).  y ~ 1/sqrt(d2) is enough for the amplitude.
constexpr double kAmplitude = 0.07957747154594767 * 0x1p56;      // 1 / (4 pi) in the sums' fixed point
constexpr double kQuickMagic = 0x1.8p36;
constexpr double kQuickMiddle = 1.93 * 0x1p-27, kQuickError = 5.2 * 0x1p-27;
__device__ inline unsigned int quick_estimate(const WalkCtx& w, double d2, double& y) {
    y = __builtin_amdgcn_rsq(d2);
    return (unsigned int)__double2loint(fma(__dmul_rn(d2, y), w.quick_k, w.quick_shift));
}

// amp2 = amplitude * 2^56, rounded to an integer, goes to the tap's 64-bit integer sum.  Below 2^51 (every
// image farther than 2.55 m) adding 1.5 * 2^52 rounds the exact product to an integer in the sum's own
// mantissa, whose low 51 bits are then the increment; larger ones are rounded and split in two exact steps
// (amp2 < 2^64: images at least a third of a millimetre away).  Which of the two an image takes depends on
// its own amplitude only, so a response does not depend on how the batch was cut into items.
// FAR: the image lies beyond kNearMetres, the test is not needed.  slot8 is the slot times eight.
constexpr double kNearMetres = 2.6;
template <bool COUNT, bool FAR>
__device__ inline void deposit(unsigned int slot8, double a, double y, unsigned long long* hist) {
    if (COUNT) {
        atomicAdd((unsigned int*)((char*)hist + slot8 / 2), 1u);
        return;
    }
    unsigned int hi, lo;
    if (FAR || __dmul_rn(a, y) < 0x1p51) {
        const double m = fma(a, y, 0x1.8p52);
        hi = (unsigned int)__double2hiint(m) & 0x7ffffu;
        lo = (unsigned int)__double2loint(m);
    } else {
        const double amp2 = rint(__dmul_rn(a, y));
        hi = (unsigned int)__dmul_rn(amp2, 0x1p-32);
        lo = (unsigned int)fma(-(double)hi, 0x1p32, amp2);
    }
    atomicAdd((unsigned long long*)((char*)hist + slot8), ((unsigned long long)hi << 32) | lo);
}

// The images z[first .. first + len) of a column, 1 <= len <= kPiece, all beyond kNearMetres unless images are counted.
// Every one lies inside the item's shell up to the slack of the closed-form table positions (a fifth of a tap), so
// its slot is one of 0 .. taps + 1 and needs no test.
// Two images at a time, so that each lane has two independent chains of arithmetic in flight (three or four measured
// no better); the pair of the next round is requested before the current one is worked on.  Walked from the far end
// so that the LDS address is also the loop's condition (the sums are integers: the order does not matter), and opaque
// to the compiler so that it is not split into a counter plus an offset.  An odd piece's top pair is its last image
// twice, the second time with amplitude zero (where images are counted, in slot 0, which is never read).  The last
// round requests the pair below the piece: the table has spare entries in front.
template <bool COUNT>
__device__ inline void walk_piece_table(const WalkCtx& w, double a, double bxy, const AxisImage* z, int first, int len,
                                        unsigned long long* hist) {
    typedef const AxisImage __attribute__((address_space(3))) * LdsImages;
    constexpr unsigned int kE = (unsigned int)sizeof(AxisImage);
    struct Pair { AxisImage e[2]; };
    auto load = [](unsigned int at, unsigned int partner) {
        const LdsImages p = (LdsImages)(uintptr_t)at, q = (LdsImages)(uintptr_t)partner;
        Pair g;
        g.e[0].key = p->key;
        g.e[0].aux = p->aux;
        g.e[1].key = q->key;
        g.e[1].aux = q->aux;
        return g;
    };
    auto step = [&](const Pair& g) {
        double d2[2], y[2];
        unsigned int slot8[2];
        bool redo = false;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            d2[i] = __dadd_rn(a, g.e[i].key);
            const unsigned int t = quick_estimate(w, d2[i], y[i]);
            slot8[i] = t >> 13 & 0x7fff8u;
            redo |= (unsigned short)t < (unsigned short)w.quick_margin2;
        }
        if (redo) {       // (one test for both, so that the estimates are complete before the branch)
#pragma unroll
            for (int i = 0; i < 2; ++i) slot8[i] = 8u * (unsigned int)tap_slot(w, d2[i], y[i]);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) deposit<COUNT, true>(slot8[i], COUNT ? 0.0 : __dmul_rn(g.e[i].aux, bxy), y[i], hist);
    };
    const unsigned int bottom = (unsigned int)(uintptr_t)(LdsImages)z + (unsigned int)first * kE;
    const bool odd = len & 1;
    unsigned int cur = bottom + ((unsigned int)(len - 1) & ~1u) * kE;      // the top pair
    Pair g0 = load(cur, cur + (odd ? 0u : kE)), g1;
    if (COUNT) {
        if (odd) g0.e[1].key = __longlong_as_double(0x7ff8000000000000ll);      // not a number: slot 0
    } else {
        // (the upper half alone: what is left of the number is below 2^-1022 and adds nothing)
        g0.e[1].aux = __hiloint2double(odd ? 0 : __double2hiint(g0.e[1].aux), __double2loint(g0.e[1].aux));
    }
    for (;;) {
        const bool last0 = cur == bottom;
        cur -= 2 * kE;
        asm("" : "+v"(cur));
        g1 = load(cur, cur + kE);
        step(g0);
        if (last0) break;
        const bool last1 = cur == bottom;
        cur -= 2 * kE;
        asm("" : "+v"(cur));
        g0 = load(cur, cur + kE);
        step(g1);
        if (last1) break;
    }
}

// beta^k for reflection counts past the LDS table; out of line so that the double-precision pow does not
// weigh on the register allocation of the loops that call it once in a long while
__device__ __attribute__((noinline)) float beta_pow_slow(double beta, int k) { return (float)pow(beta, (double)k); }

// (out of line for the same reason: only rooms too flat or narrow for the tables come here)
template <bool COUNT>
__device__ __attribute__((noinline)) void walk_column_direct(const WalkCtx w, const Axis az, double a, double cxy, int nmz,
                                                             unsigned long long* hist) {
    for (int q = 0; q < 2; ++q)
        for (int n = -nmz; n <= nmz; ++n) {
            const double dz = axis_delta(az, q, n);
            const double d2 = __dadd_rn(a, __dmul_rn(dz, dz));
            const double y = __builtin_amdgcn_rsq(d2);
            const int slot = tap_slot(w, d2, y);
            if ((unsigned int)slot > (unsigned int)(w.n1 - w.n0 + 1)) continue;          // outside the item
            double bz = 0.0;
            if (!COUNT) bz = (double)beta_pow_slow(w.beta, iabs(n - q) + iabs(n));
            deposit<COUNT, false>(8u * (unsigned int)slot, __dmul_rn(bz, cxy), y, hist);
        }
}

// The images z[first .. last) of a column, with the test for amplitudes too large for the fast rounding.
__device__ __attribute__((noinline)) void walk_near(const WalkCtx w, double a, double bxy, const AxisImage* z, int first,
                                                    int last, unsigned long long* hist) {
    for (int i = first; i < last; ++i) {
        const double d2 = __dadd_rn(a, z[i].key), y = __builtin_amdgcn_rsq(d2);
        const int slot = tap_slot(w, d2, y);
        if ((unsigned int)slot <= (unsigned int)(w.n1 - w.n0 + 1))
            deposit<false, false>(8u * (unsigned int)slot, __dmul_rn(z[i].aux, bxy), y, hist);
    }
}

// Source and microphone lie between the walls, or not so far outside that an axis' images stop beginning within 2 L of
// the microphone (false where a position is not a number).  Rows beyond that are not refused: they take the plain path,
// which tests every tap.
__device__ inline bool axis_in_order(const Axis& a) {
    return fabs(a.src - a.mic) <= 2.0 * a.room && fabs(a.src + a.mic) <= 2.0 * a.room;
}

// All images (1 - 2q) s + 2 n L - m, q in {0,1}, |n| <= nm, of one axis, written to `out` in order of
// squared distance.  For each q the signed distance grows with n, so the images with negative
// distance (walked towards smaller n) and those with non-negative distance are two sorted lists.  All four lists step
// by 2 L and begin within 2 L of the microphone, so the merged order is known: element p of a list follows every
// list's elements 0 .. p-1 and, of the elements p, those of the lists that begin nearer (ties: the lower list).
// That takes an axis_in_order.
// (Searching the other lists for every entry's place, eight steps each, took a sixth of all the kernel's instructions.)
// aux(q, n) supplies the entry's second field.
template <class Aux>
__device__ inline void build_sorted_images(const Axis& ax, int nm, AxisImage* out, int tid, Aux aux) {
    const int per_q = 2 * nm + 1, n_all = 2 * per_q;
    // list 2 q + side: its first distance and its length.  The first image at a non-negative distance is n = 0 or 1
    // while source and microphone lie between the walls.
    double begin[4];
    int length[4];
    int split[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int n = axis_delta(ax, q, 0) >= 0.0 ? 0 : 1;
        split[q] = n + nm;                        // index of that image; nm >= 1
        begin[2 * q] = -axis_delta(ax, q, n - 1);
        begin[2 * q + 1] = axis_delta(ax, q, n);
        length[2 * q] = n + nm;
        length[2 * q + 1] = nm - n + 1;
    }
    for (int i = tid; i < n_all; i += kThreads) {
        const int q = i >= per_q, t = i - q * per_q, sp = q ? split[1] : split[0];
        const int side = t >= sp, own = 2 * q + side;
        const double d = axis_delta(ax, q, t - nm);
        const int p = side ? t - sp : sp - 1 - t;
        const double mine = own == 0 ? begin[0] : own == 1 ? begin[1] : own == 2 ? begin[2] : begin[3];
        int rank = p;
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            if (l == own) continue;
            const bool nearer = begin[l] < mine || (begin[l] == mine && l < own);
            rank += min(p + (nearer ? 1 : 0), length[l]);
        }
        AxisImage e;
        e.key = __dmul_rn(d, d);
        e.aux = aux(q, t - nm);
        out[rank] = e;
    }
}

// Position in an axis's sorted table without searching it.  The table holds the images c_q + 2 n L,
// q in {0,1}, |n| <= nm, ordered by squared distance, so the number of entries within distance s of the
// microphone is the number of terms of the two arithmetic progressions that lie in [-s, s].
// Single precision is enough: a bound is widened (or narrowed) by `slack`, a fifth of a tap plus two millionths of the
// distance, which covers the rounding of these counts for every axis of up to 4e5 taps (longer ones take the plain
// path).  An entry that close to a bound is then visited although it may lie outside; it lands, less than half a tap
// away, in one of the two slots that are never read.
constexpr double kMaxAxisTaps = 4e5;
struct AxisCount {
    float k0, k1;        // -c_q / (2 L), c_q = (1 - 2q) src - mic
    float inv2l;         // 1 / (2 L)
    float nm;
    float slack;         // metres
};

__device__ inline AxisCount axis_count(const Axis& a, int nm, double k_fs_c) {
    const double inv2l = 1.0 / (2.0 * a.room);
    return AxisCount{uni((float)(-(a.src - a.mic) * inv2l)), uni((float)(-(-a.src - a.mic) * inv2l)), uni((float)inv2l),
                     uni((float)nm), uni((float)(0.2 / k_fs_c))};
}

// terms n of c_q + 2 n L, |n| <= nm, within [-s, s]: (-s - c_q) / 2L <= n <= (s - c_q) / 2L
__device__ inline int count_within(const AxisCount& a, float s) {
    float total = 0.f;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const float k = q ? a.k1 : a.k0;
        const float hi = fminf(floorf(fmaf(s, a.inv2l, k)), a.nm);
        const float minus_lo = fminf(floorf(fmaf(s, a.inv2l, -k)), a.nm);
        total += fmaxf(hi + minus_lo + 1.f, 0.f);
    }
    return (int)total;
}

// number of entries with key <= bound, or a few more
__device__ inline int count_not_above(const AxisCount& a, int n, double bound) {
    if (!(bound >= 0.0)) return 0;
    const float s = __builtin_amdgcn_sqrtf((float)bound);
    return min(count_within(a, fmaf(s, 1.000002f, a.slack)), n);
}
// number of entries with key < bound, or a few fewer
__device__ inline int count_below(const AxisCount& a, double bound) {
    const float s = fmaf(__builtin_amdgcn_sqrtf(fmaxf((float)bound, 0.f)), 0.999998f, -a.slack);
    return s > 0.f ? count_within(a, s) : 0;
}

// VISITS: a measuring instantiation that also adds the number of images it walked to *visits.
template <bool COUNT, bool VISITS = false>
__global__ __launch_bounds__(kThreads, 4) void rir_image_kernel(
    Rooms rooms, int rir_len, double k_fs_c, const Item* __restrict__ items,
    int* __restrict__ ctrl, float* __restrict__ rir_out,
    int32_t* __restrict__ cnt_out, unsigned long long* __restrict__ visits = nullptr) {
    __shared__ unsigned long long hist[(COUNT ? kMaxTaps / 2 : kMaxTaps) + 2];     // first and last slot are never read
    __shared__ float bpow[COUNT ? 1 : kPow];
    __shared__ AxisImage ztab_store[2 * kAxisCap + 2];
    AxisImage* const ztab = ztab_store + 2;        // z images sorted by dz*dz (spare entries in front)
    __shared__ AxisImage ytab[2 * kAxisCap];       // y images sorted by dy*dy
    __shared__ int row_pfx[2 * kAxisCap];          // per x image: inclusive prefix of live column counts
    __shared__ Column cols[kWaves][64];
    __shared__ __align__(8) unsigned int piece_starts[kWaves][kStartWords];
    __shared__ int s_item, s_batch;
    unsigned int* hist32 = reinterpret_cast<unsigned int*>(hist);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n_items = ctrl[0];
    unsigned long long walked = 0;

    for (;;) {
        if (tid == 0) {
            s_item = atomicAdd(&ctrl[1], 1);
            s_batch = kWaves;
        }
        __syncthreads();
        const int it = uni(s_item);
        if (it >= n_items) break;
        const Item item = items[it];
        const int n0 = item.n0, n1 = item.n1, n_taps = n1 - n0;
        const Room room = load_room(rooms, uni(item.rir));
        const float* g = room.g;

        if (COUNT) {
            for (int i = tid; i <= n_taps + 1; i += kThreads) hist32[i] = 0u;
        } else {
            for (int i = tid; i <= n_taps + 1; i += kThreads) hist[i] = 0ull;
        }
        if (room_ok(g)) {
            const Axis ax{uni((double)g[0]), uni((double)g[3]), uni((double)g[6])};
            const Axis ay{uni((double)g[1]), uni((double)g[4]), uni((double)g[7])};
            const Axis az{uni((double)g[2]), uni((double)g[5]), uni((double)g[8])};
            const double beta = uni((double)g[9]);
            // every image of this item lies in r_in <= d < r_out (half a tap of slack on either side)
            const double r_out = uni((double)n1 / k_fs_c);
            const double r_in = n0 > 0 ? uni((double)(n0 - 1) / k_fs_c) : 0.0;
            const double r_out2 = uni(r_out * r_out), r_in2 = uni(r_in * r_in);
            // An image reflected k times adds beta^k / (4 pi d) * 2^56, rounded to an integer, to its
            // tap; once beta^k < 2 pi d 2^-56 that is exactly zero, so such images are never visited.
            // log2_beta < 0 enables the cut (amplitude sums only; tap counts visit every image).
            const float log2_beta = (!COUNT && g[9] > 0.f && g[9] < 1.f) ? uni(__log2f(g[9])) : 0.f;
            const int k_cut_item = uni(reflection_cut(log2_beta, (float)r_in));
            int nmx = uni((int)ceil(r_out / (2.0 * ax.room)) + 1);
            int nmy = uni((int)ceil(r_out / (2.0 * ay.room)) + 1);
            const int nmz = uni((int)ceil(r_out / (2.0 * az.room)) + 1);
            nmx = min(nmx, k_cut_item / 2 + 1);          // |n - q| + |n| >= 2 |n| - 1
            nmy = min(nmy, k_cut_item / 2 + 1);
            const int nix = 2 * (2 * nmx + 1), niy = 2 * (2 * nmy + 1), niz = 2 * (2 * nmz + 1);
            const AxisCount cy = axis_count(ay, nmy, k_fs_c), cz = axis_count(az, nmz, k_fs_c);
            Column* wc = cols[wave];
            WalkCtx wctx;
            wctx.k_fs_c = k_fs_c;
            // (in whole units of the estimate's 2^-16 tap, so that adding it to the magic number is exact; one unit
            // for the sum's rounding)
            const double margin = ceil(kQuickError * 65536.0 * (double)(n1 + 2)) + 1.0;
            wctx.quick_k = uni(k_fs_c * (1.0 - kQuickMiddle));
            wctx.quick_shift = kQuickMagic + (0.5 + margin * 0x1p-16 - (double)(n0 - 1));
            wctx.quick_margin2 = uni((int)(2.0 * margin) + 1);
            const double guard = 1e-12 * (double)(n1 + 1) + 1e-13;
            wctx.shift = (0.5 + guard) - (double)(n0 - 1);
            wctx.guard2 = uni(2.0 * guard);
            wctx.n0 = n0;
            wctx.n1 = n1;
            // beyond 2.6 m every amplitude is below 2^-5 (see deposit); the few images of the innermost items that may be
            // nearer are walked apart.  (The table positions that separate the two are off by less than 0.25 taps.)
            const double r_near = kNearMetres + 0.25 / k_fs_c, r_near2 = uni(r_near * r_near);
            const bool near_item = !COUNT && r_in < r_near;
            const double r_walk2 = near_item ? r_near2 : r_in2;
            wctx.beta = beta;
            const float y0_max = uni(fmaxf(fabsf((float)(ay.src - ay.mic)), fabsf((float)(ay.src + ay.mic))));
            const float z0_max = uni(fmaxf(fabsf((float)(az.src - az.mic)), fabsf((float)(az.src + az.mic))));
            const float lyf = uni((float)ay.room), lzf = uni((float)az.room);
            // every image with at most k reflections along an axis lies within max|c_q| + (k + 1) L of the
            // microphone on that axis; squared, with a little slack, this bounds the table range to visit
            auto reach2 = [](float c_max, float room, int k) {
                const float r = c_max + (float)(k + 1) * room;
                return (double)(r * r * 1.0001f + 1e-3f);
            };

            // fast path: the y and z images fit the LDS tables and so do the x rows, and the closed forms hold
            const bool fast = axis_in_order(ax) && axis_in_order(ay) && axis_in_order(az) &&
                              nix <= 2 * kAxisCap && niy <= 2 * kAxisCap && niz <= 2 * kAxisCap &&
                              fmax(ay.room, az.room) * k_fs_c < kMaxAxisTaps;
            int n_cand;
            if (!COUNT) {
                // beta^k by squaring (k < 1024: ten steps, a few units in the last place of the double, far inside
                // the float it is kept as; the library pow is some ten times the instructions), for the counts that
                // can be asked for: those of the z images, and of a column at most the cut or all there are
                const int k_most = max(2 * nmz + 1, min(k_cut_item, 2 * (nmx + nmy) + 2));
                for (int i = tid; i <= min(k_most, kPow - 1); i += kThreads) {
                    double b = beta, acc = 1.0;
#pragma unroll
                    for (int bit = 0; bit < 10; ++bit) {
                        if ((i >> bit) & 1) acc *= b;
                        b *= b;
                    }
                    bpow[i] = (float)acc;
                }
            }
            __syncthreads();
            if (fast) {
                build_sorted_images(az, nmz, ztab, tid, [&](int q, int n) {
                    if (COUNT) return 0.0;
                    const int k = iabs(n - q) + iabs(n);
                    // beta^k / (4 pi) * 2^56
                    return (double)(k < kPow ? bpow[k] : beta_pow_slow(beta, k)) * kAmplitude;
                });
                build_sorted_images(ay, nmy, ytab, tid, [&](int q, int n) { return (double)(iabs(n - q) + iabs(n)); });
                // live columns of x image ix: the y images with dy^2 <= r_out^2 - dx^2 that the reflection
                // cut can still reach -- a prefix of the sorted y table
                for (int ix = tid; ix < nix; ix += kThreads) {
                    const int qx = ix & 1, nx = (ix >> 1) - nmx;
                    const double dx = axis_delta(ax, qx, nx);
                    double bound = r_out2 - __dmul_rn(dx, dx);
                    const int ky_max = k_cut_item - (iabs(nx - qx) + iabs(nx));
                    if (ky_max < (1 << 18)) bound = fmin(bound, reach2(y0_max, lyf, ky_max));
                    row_pfx[ix] = (bound >= 0.0 && ky_max >= 0) ? count_not_above(cy, niy, bound) : 0;
                }
                __syncthreads();
                if (wave == 0) {                              // inclusive scan over the rows, 64 at a time
                    int carry = 0;
                    for (int base = 0; base < nix; base += 64) {
                        const int i = base + lane;
                        const int v = wave_inclusive_scan(i < nix ? row_pfx[i] : 0) + carry;
                        if (i < nix) row_pfx[i] = v;
                        carry = __shfl(v, 63, 64);
                    }
                }
                __syncthreads();
                n_cand = row_pfx[nix - 1];
            } else {
                n_cand = nix * niy;
            }
            if (fast && near_item) {
                // the columns within r_near: y images up to that, of the x images with |n| <= n_near
                const int n_near = min((int)(r_near / (2.0 * ax.room)) + 1, nmx), n_rows = 2 * (2 * n_near + 1);
                const int n_y = count_not_above(cy, niy, r_near2);
                for (int i = tid; i < n_rows * n_y; i += kThreads) {
                    const int ix = i / n_y, qx = ix & 1, nx = (ix >> 1) - n_near;
                    const AxisImage ye = ytab[i - ix * n_y];
                    const double dx = axis_delta(ax, qx, nx);
                    const double a = __dadd_rn(__dmul_rn(dx, dx), ye.key);
                    const int first = count_below(cz, r_in2 - a);
                    const int last = min(count_below(cz, r_near2 - a), count_not_above(cz, niz, r_out2 - a));
                    const int kxy = iabs(nx - qx) + iabs(nx) + (int)ye.aux;
                    // (past the cut the amplitudes are zero, and bpow has not been formed)
                    if (last <= first || kxy > k_cut_item) continue;
                    walk_near(wctx, a, (double)(kxy < kPow ? bpow[kxy] : beta_pow_slow(beta, kxy)), ztab, first, last, hist);
                    if (VISITS) walked += (unsigned long long)(last - first);
                }
            }
            const int n_batch = (n_cand + 63) / 64;

            // Batches are taken from a counter (they differ in work by their columns' ranges; dealt in turn, a wave in
            // eight waited an eighth of the time for the others); the next one is asked for while this one is worked on.
            int row_lo = 0;          // row of the batch's first candidate: it only moves up from batch to batch
            for (int batch = wave, next = 0; batch < n_batch; batch = uni(next)) {
                if (lane == 0) next = atomicAdd(&s_batch, 1);
                // ---- each lane describes one candidate column ----
                const int cand = batch * 64 + lane;
                if (fast)
                    while (row_pfx[row_lo] <= batch * 64) ++row_lo;       // (the same in every lane; batch * 64 < n_cand)
                Column col;
                col.a = 0.0;
                int kxy = 0, z_first = 0, z_len = 0;
                int pieces = 0;
                if (cand < n_cand) {
                    if (fast) {
                        // smallest row with row_pfx > cand: a short walk from the row of the batch's first
                        // column, since 64 consecutive columns span few rows
                        int lo = row_lo;
                        while (row_pfx[lo] <= cand) ++lo;
                        const int ix = lo, qx = ix & 1, nx = (ix >> 1) - nmx;
                        const AxisImage ye = ytab[cand - (ix ? row_pfx[ix - 1] : 0)];
                        const double dx = axis_delta(ax, qx, nx);
                        col.a = __dadd_rn(__dmul_rn(dx, dx), ye.key);
                        kxy = iabs(nx - qx) + iabs(nx) + (int)ye.aux;
                    } else {
                        const int ix = cand / niy, iy = cand - ix * niy;
                        const int qx = ix & 1, nx = (ix >> 1) - nmx;
                        const int qy = iy & 1, ny = (iy >> 1) - nmy;
                        const double dx = axis_delta(ax, qx, nx);
                        const double dy = axis_delta(ay, qy, ny);
                        col.a = __dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy));
                        kxy = iabs(nx - qx) + iabs(nx) + iabs(ny - qy) + iabs(ny);
                    }
                    // reflections left for the z axis before this column's images vanish
                    // (beyond the first shell the shell's own inner radius bounds the distance well enough)
                    const int kz_max = (n0 > 0 ? k_cut_item : reflection_cut(log2_beta, sqrtf((float)col.a))) - kxy;
                    if (col.a < r_out2 && kz_max >= 0) {
                        if (fast) {
                            // images with r_in^2 - a <= dz^2 <= r_out^2 - a within reach of the reflection cut:
                            // one contiguous range of the sorted z table (the few images past the cut that it
                            // keeps add exactly zero)
                            double hi2 = r_out2 - col.a;
                            if (kz_max < (1 << 18)) hi2 = fmin(hi2, reach2(z0_max, lzf, kz_max));
                            const double lo2 = r_walk2 - col.a;
                            const int first = lo2 > 0.0 ? count_below(cz, lo2) : 0;     // entries with dz2 < lo2
                            const int last = count_not_above(cz, niz, hi2);
                            if (last > first) {
                                z_first = first;
                                z_len = last - first;
                                pieces = (z_len + kPiece - 1) / kPiece;
                            }
                        } else {
                            pieces = 1;                        // one lane walks every z image of the column
                        }
                    }
                }
                const int pfx = wave_inclusive_scan(pieces);
                const int my_first = pfx - pieces;             // this column's first piece
                col.place = (z_first - kPiece * my_first) * 1024 + (z_first + z_len);
                if (!COUNT) col.bxy = kxy < kPow ? bpow[kxy] : (pieces ? beta_pow_slow(beta, kxy) : 0.f);
                const int n_pieces = __builtin_amdgcn_readlane(pfx, 63);
                // columns with pieces, packed in order
                const unsigned long long live = __ballot(pieces > 0);
                if (pieces > 0)
                    wc[__builtin_amdgcn_mbcnt_hi((unsigned int)(live >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)live, 0u))] = col;

                // ---- pieces are dealt to lanes ----
                // Piece p belongs to the last column that starts at or before it.  Every column but a chunk's first sets
                // bit f - 1 of a bit map, f its first piece; a piece's column is then a count of the bits below it.
                unsigned int* starts = piece_starts[wave];
                constexpr int kChunk = 32 * kStartWords;
                for (int chunk = 0; chunk < n_pieces; chunk += kChunk) {
                    if (lane < kStartWords) starts[lane] = 0u;
                    wave_sync_lds();
                    const int bit = my_first - chunk - 1;
                    if (pieces > 0 && bit >= 0 && bit < kChunk) atomicOr(&starts[bit >> 5], 1u << (bit & 31));
                    int before = __popcll(__ballot(pieces > 0 && bit < 0)) - 1;       // the column of the chunk's first piece
                    wave_sync_lds();
                    const int chunk_end = min(n_pieces, chunk + kChunk);
                    for (int p0 = chunk; p0 < chunk_end; p0 += 64) {
                        const uint2 m = *reinterpret_cast<const uint2*>(&starts[(p0 - chunk) >> 5]);   // pieces p0 .. p0 + 63
                        const int mine = (int)__builtin_amdgcn_mbcnt_hi(m.y, __builtin_amdgcn_mbcnt_lo(m.x, (unsigned int)before));
                        const int p = p0 + lane;
                        if (p < chunk_end) {
                            const Column c = wc[mine];
                            if (fast) {
                                const int first = (c.place >> 10) + __mul24(kPiece, p);
                                const int len = min(kPiece, (c.place & 1023) - first);
                                walk_piece_table<COUNT>(wctx, c.a, (double)c.bxy, ztab, first, len, hist);
                                if (VISITS) walked += (unsigned long long)len;
                            } else {
                                walk_column_direct<COUNT>(wctx, az, c.a, (double)c.bxy * kAmplitude, nmz, hist);
                                if (VISITS) walked += (unsigned long long)niz;
                            }
                        }
                        before += __popc(m.x) + __popc(m.y);
                    }
                    wave_sync_lds();
                }
            }
        }
        __syncthreads();

        if (COUNT) {
            int32_t* out = cnt_out + (size_t)item.rir * rir_len + n0;
            for (int i = tid; i < n_taps; i += kThreads) out[i] = (int32_t)hist32[i + 1];
        } else {
            float* out = rir_out + (size_t)item.rir * rir_len + n0;
            for (int i = tid; i < n_taps; i += kThreads) {
                const unsigned long long v = hist[i + 1];
                const double d = (double)(unsigned int)(v >> 32) * 4294967296.0 + (double)(unsigned int)v;
                out[i] = (float)(d * 1.3877787807814457e-17);       // 2^-56
            }
        }
        __syncthreads();
    }
    if (VISITS) {
        for (int off = 32; off > 0; off >>= 1) walked += __shfl_down(walked, off, 64);
        if (lane == 0 && walked) atomicAdd(visits, walked);
    }
}

__global__ void fill_u32_kernel(uint32_t* p, uint32_t v, int64_t n) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

}  // namespace

hipError_t launch_fill_u32(hipStream_t s, void* p, uint32_t v, int64_t n) {
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    fill_u32_kernel<<<dim3((unsigned)blocks), dim3(256), 0, s>>>(static_cast<uint32_t*>(p), v, n);
    return hipGetLastError();
}

int rir_items_per_response(int rir_len) { return kMaxShells + rir_len / kMaxTaps + 2; }
size_t rir_item_bytes() { return sizeof(Item); }

int rir_ctrl_ints() { return kCtrlInts; }

hipError_t launch_rir_plan(hipStream_t s, int n_groups, int n_rir, const Rooms& rooms, int rir_len, double fs_over_c,
                           void* items, int* ctrl) {
    if (n_rir <= 0) return hipSuccess;
    // `items` holds the sorted table followed by the unsorted one
    const int per_rir = rir_items_per_response(rir_len);
    Item* sorted = static_cast<Item*>(items);
    Item* unsorted = sorted + (size_t)n_rir * per_rir;
    if (n_rir <= kPlanRows * kPlanThreads) {                 // one launch instead of four
        rir_plan_all_kernel<<<dim3(1), dim3(kPlanThreads), 0, s>>>(n_rir, rooms, rir_len, fs_over_c, sorted, unsorted,
                                                                    per_rir, ctrl, n_groups);
        return hipGetLastError();
    }
    hipError_t e = launch_fill_u32(s, ctrl, 0u, kCtrlInts);
    if (e != hipSuccess) return e;
    rir_work_kernel<<<dim3((n_rir + 127) / 128), dim3(128), 0, s>>>(n_rir, rooms, rir_len, fs_over_c, ctrl);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    rir_plan_kernel<<<dim3((n_rir + 127) / 128), dim3(128), 0, s>>>(n_rir, rooms, rir_len, fs_over_c, unsorted, per_rir, ctrl,
                                                                    n_groups);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t max_items = (size_t)n_rir * per_rir;
    const int item_groups = (int)((max_items + 255) / 256);
    rir_sort_items_kernel<<<dim3((unsigned)item_groups), dim3(256), 0, s>>>(unsorted, sorted, ctrl);
    return hipGetLastError();
}

hipError_t launch_rir(hipStream_t s, int n_groups, int n_rir, const Rooms& rooms, int rir_len, double fs_over_c,
                      const void* items, int* ctrl, float* rir_out, int32_t* cnt_out,
                      bool restart, unsigned long long* visits) {
    if (n_rir <= 0) return hipSuccess;
    hipError_t e = hipSuccess;
    if (restart) {                                           // another pass over the same plan
        e = launch_fill_u32(s, ctrl + 1, 0u, 1);
        if (e != hipSuccess) return e;
    }
    const Item* it = static_cast<const Item*>(items);
    if (rir_out && visits)
        rir_image_kernel<false, true><<<dim3((unsigned)n_groups), dim3(kThreads), 0, s>>>(
            rooms, rir_len, fs_over_c, it, ctrl, rir_out, nullptr, visits);
    else if (rir_out)
        rir_image_kernel<false><<<dim3((unsigned)n_groups), dim3(kThreads), 0, s>>>(
            rooms, rir_len, fs_over_c, it, ctrl, rir_out, nullptr);
    else
        rir_image_kernel<true><<<dim3((unsigned)n_groups), dim3(kThreads), 0, s>>>(
            rooms, rir_len, fs_over_c, it, ctrl, nullptr, cnt_out);
    return hipGetLastError();
}

}  // namespace aug
