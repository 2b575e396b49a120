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
//   * plan kernels: a response's taps are cut into shells [n0, n1) of about equal estimated work, at most kMaxTaps taps
//     wide; the shell size follows the batch's work per persistent group.  Every shell gets an estimate of its work
//     and a counting sort orders the items heaviest first.
//   * image kernel: persistent work groups fetch items from a counter.  An item owns its
//     taps, so sums live in LDS and are stored once, without global atomics.
//     The y images of the response (both q, both signs) lie in an LDS table in order of distance, so the columns (x image,
//     y image) of an x image that can still reach the shell are the first of that table; a prefix sum over the x images
//     numbers the columns and dead ones are never seen.
//     Along z the images are four arithmetic progressions of one step, 2 L.  A column's images inside the shell are
//     therefore those of a range of steps p, with up to three more at either end, and a lane walks a column from the
//     first p to the last, four images a step, without reading any table of images: distances are formed from the step,
//     amplitudes by two multiplications a step.  Columns are sorted by length, some thousand at a time, so that the 64 lanes of a
//     wavefront walk columns of one length.
//     Rooms so flat or narrow that an axis has more images than the tables hold, rooms of more than 4e5 taps along y or z,
//     and positions far outside the room take a plain path (all columns of the bounding box, of a live column the z
//     images about the shell, every tap tested).
//   * amplitudes accumulate as 64-bit fixed point (2^-56, each increment rounded to the nearest unit)
//     with integer LDS atomics: gfx950 executes float LDS atomics far slower than integer
//     ones, and integer sums do not depend on the order of arrival nor on how a batch is cut into items.
//
// What bounds it: vector issue (a double-precision operation takes four cycles, its rsq sixteen: 55 per image with four
// wavefronts per SIMD) and LDS (64 adds of 64 bits to scattered places take the CU 13 to 16 cycles, six if no two meet in a
// bank).  Measured on 2000 responses of 8000 taps, plan included: a walk of pieces of 14 images read from a sorted table of z images, which
// were dealt to lanes as a wavefront's 64 columns gave them, 289 us (a quarter of the lanes idle in the mean, up to half
// in small batches); this walk, 261; the item's constants formed by one wavefront while the others walk, 239; rows found by
// comparing 64 at once and the near images walked last, 224; the ends of a column walked like its middle, with a
// slot per lane for what lies outside, 215.  Groups of 1024 threads with 64 registers
// took 294.  Without its walk (the sums left empty) the kernel alone takes 85 of 212 us there, 102 of 378 for 1024 responses of 16000
// taps and 21 of 34 for 128 of 8000: candidates, tables, sorting, stores and barriers, so these count nearly as much as the walk does.
// What the long responses wanted cost this batch 9 of those us: six candidate columns per thread and chunk instead of
// four (four again now), rows with a gap where the cut leaves their middle empty, and shells of equal work (the plan is 16 us instead of 10).
// Other whole calls with amplitudes from a table of z powers and a chunk's columns in registers while they were walked, and now:
// 1 response of 1000 taps 15.6 -> 12.5 us, 600 of 1000 25.0 -> 26.2, 3000 of 1000 64.2 -> 64.1, 16 of 4096 24.4 -> 17.9, 128 of 8000 43.1 ->
// 38.9, 2000 of 8000 222 -> 220, 384 of 16000 205 -> 197, 16 of 32768 118 -> 87.

#include "rir_plan.h"

#include <type_traits>

namespace aug {
namespace {

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
// beta^k held in LDS (see power): the first kPow and from there every kPowStep-th.  (Two tables of 256 and every 64th, the next
// item's filled by the wavefront that prepares it: that wavefront is what an item of few images waits for, 3000 responses of 1000 taps
// 65.3 us instead of 63.9, and columns that begin past 256 multiplied up to 63 times, 64 responses of 8000 taps of rooms of 0.6 to 1 m
// with beta 0.95 2790 us instead of 2317.)
constexpr int kPow = 504, kPowStep = 16;
constexpr int kPowMost = 1024;            // more reflections than an image of the fast walk can have
constexpr int kPowTable = kPow + (kPowMost - kPow + kPowStep - 1) / kPowStep;
static_assert(kPow % 8 == 0, "form_powers");
constexpr int kAxisCap = 320;             // x or y images per q held in the LDS tables
constexpr int kYCap = 2 * kAxisCap + 8;
constexpr int kMaxP = 160;                // steps of 2 L along z (see walk_step) that the fast walk takes
constexpr int kPerThread = 4;             // candidate columns per thread and chunk (described two and two)
// Sums and columns share LDS: columns that there is room for behind the sums of the widest item; items of fewer taps have room for
// more, and a chunk is as many candidates as are sure to have it.  (Columns with LDS of their own and a chunk walked in as many
// goes as that took kept what was found out about the chunk in registers meanwhile, and the compiler spilled.  Six candidates per
// thread it spills too: 2000 responses of 8000 taps 282 us.)
constexpr int kColumns = 3 * kThreads;
constexpr int kPool = kMaxTaps + 66 + kColumns * 3 / 2;        // words of eight bytes
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

// the same from 2 n
__device__ inline double axis_delta_2n(const Axis& a, int q, int n2) {
    return __dsub_rn(__dadd_rn(q ? -a.src : a.src, __dmul_rn((double)n2, a.room)), a.mic);
}

// reflections of image (q, n) along its axis: |n - q| + |n|
__device__ inline int reflections(int q, int n) {
    const int v = 2 * n - q;
    return v < 0 ? -v : v;
}

// A value that every lane of the wavefront has computed alike, moved to scalar registers: what an item's
// geometry determines is the same in all lanes and would otherwise occupy vector registers for the whole item.
__device__ inline int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline float uni(float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); }
__device__ inline double uni(double v) { return __hiloint2double(uni(__double2hiint(v)), uni(__double2loint(v))); }

__device__ inline void wave_sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
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

// One thread per response: cut its taps into shells and append them to the unsorted item table, with their cost classes
// and the class census (taken in LDS first: one global atomic per class and group, not per item).
__global__ void rir_plan_kernel(int n_rir, Rooms rooms, int rir_len, double k_fs_c, Item* __restrict__ unsorted,
                                int* __restrict__ ctrl, int n_groups) {
    __shared__ int census[kClasses];
    if (threadIdx.x < kClasses) census[threadIdx.x] = 0;
    __syncthreads();
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r < n_rir) {
        const Room room = load_room(rooms, r);
        const float target = item_target(ctrl[kCtrlWork], n_groups, n_rir);
        const WorkModel model = work_model(room.g, rir_len, k_fs_c);
        const bool ok = room_ok(room.g);
        const int count = cut_shells(model, ok, rir_len, target, 0, 1, [](int, int) {});
        int at = atomicAdd(&ctrl[0], count);
        cut_shells(model, ok, rir_len, target, 0, 1, [&](int lo, int hi) {
            const int cls = item_class(model, ok, lo, hi);
            unsorted[at++] = Item{r, lo, hi, cls};
            atomicAdd(&census[cls], 1);
        });
    }
    __syncthreads();
    if (threadIdx.x < kClasses && census[threadIdx.x]) atomicAdd(&ctrl[2 + threadIdx.x], census[threadIdx.x]);
}

__global__ __launch_bounds__(kPlanThreads) void rir_plan_all_kernel(int n_rir, Rooms rooms, int rir_len, double k_fs_c, Item* __restrict__ sorted,
                                                                    Item* __restrict__ unsorted, int* __restrict__ ctrl, int n_groups) {
    __shared__ PlanShared shared;
    plan_all(shared, n_rir, rooms, rir_len, k_fs_c, sorted, unsorted, ctrl, n_groups);
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

// Source and microphone lie between the walls, or not so far outside that an axis' images stop beginning within 2 L of
// the microphone (false where a position is not a number).  Rows beyond that are not refused: they take the plain path,
// which tests every tap.
__device__ inline bool axis_in_order(const Axis& a) {
    return fabs(a.src - a.mic) <= 2.0 * a.room && fabs(a.src + a.mic) <= 2.0 * a.room;
}

// The images (1 - 2q) s + 2 n L - m, q in {0,1}, of an axis in order of distance.  For each q the signed distance grows
// with n, so the images with negative distance (walked towards smaller n) and those with non-negative distance are two
// sorted lists, 2 q and 2 q + 1.  All four lists step by 2 L and begin within 2 L of the microphone (that takes an
// axis_in_order), so the merged order is known: element p of every list in the order in which the lists begin, then the
// elements p + 1.
struct AxisOrder {
    unsigned int lists;         // list of rank r in bits 4 r, 4 r + 1
    int first_n[2];             // the first image at a non-negative distance, per q
};
__device__ inline AxisOrder axis_order(const Axis& ax) {
    AxisOrder o;
    double begin[4];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int n = axis_delta(ax, q, 0) >= 0.0 ? 0 : 1;          // (0 or 1 while source and microphone lie between the walls)
        o.first_n[q] = n;
        begin[2 * q] = -axis_delta(ax, q, n - 1);
        begin[2 * q + 1] = axis_delta(ax, q, n);
    }
    o.lists = 0;
#pragma unroll
    for (int l = 0; l < 4; ++l) {
        int rank = 0;
#pragma unroll
        for (int m = 0; m < 4; ++m)
            if (m != l && (begin[m] < begin[l] || (begin[m] == begin[l] && m < l))) ++rank;
        o.lists |= (unsigned int)l << 4 * rank;
    }
    return o;
}
// image i of that order: q and n
__device__ inline void ordered_image(const AxisOrder& o, int i, int& q, int& n) {
    const int list = (int)(o.lists >> 4 * (i & 3)) & 3, p = i >> 2;
    q = list >> 1;
    n = list & 1 ? o.first_n[q] + p : o.first_n[q] - 1 - p;
}

// The number of images of an axis within distance s of the microphone, c_q = (1 - 2q) src - mic: the number of terms of
// the two arithmetic progressions c_q + 2 n L that lie in [-s, s].
// Single precision is enough: a bound is widened by `slack`, a fifth of a tap plus two millionths of the
// distance, which covers the rounding of these counts for every axis of up to 4e5 taps (longer ones take the plain
// path).  An image that close to a bound is then visited although it may lie outside; it lands, less than half a tap
// away, in one of the two slots that are never read.  The same goes for the ends of a column's range (see the kernel).
constexpr double kMaxAxisTaps = 4e5;
// An image of a column's first or last four lies up to 2 L outside the shell; where that is so far that its slot may come round
// to the item's in sixteen bits, its distance is tested (128 responses of 32768 taps of rooms 400 m high: 109 us, 357 on the plain
// path).  And L must not be so few taps that the slack is more than L.
constexpr double kWrapTaps = 16384.0, kMinHeightTaps = 0.25;
struct AxisCount {
    float k0, k1;        // -c_q / (2 L)
    float inv2l;         // 1 / (2 L)
    float slack;         // metres
};
__device__ inline AxisCount axis_count(const Axis& a, double k_fs_c) {
    const double inv2l = 1.0 / (2.0 * a.room);
    return AxisCount{(float)(-(a.src - a.mic) * inv2l), (float)(-(-a.src - a.mic) * inv2l), (float)inv2l, (float)(0.2 / k_fs_c)};
}
// images within a distance, or a few more: (-s - c_q) / 2L <= n <= (s - c_q) / 2L.  SLACK -1: or a few fewer
template <int SLACK = 1>
__device__ inline int count_within(const AxisCount& a, float distance) {
    const float s = fmaf(distance, SLACK > 0 ? 1.000002f : 0.999998f, SLACK > 0 ? a.slack : -a.slack) * a.inv2l;
    const float one = floorf(s + a.k0) + floorf(s - a.k0) + 1.f, two = floorf(s + a.k1) + floorf(s - a.k1) + 1.f;
    return (int)(fmaxf(one, 0.f) + fmaxf(two, 0.f));
}

// One item, prepared by one wavefront for the whole group and kept in LDS: what each phase needs is read there at its start
// (computed by every wavefront, and held in registers from phase to phase, it took a seventh of the kernel's instructions
// and made it spill).
struct ItemCtx {
    int kind;               // one of the kinds below
    int rir, n0, n1;
    unsigned int top8;      // eight times the last slot.  Slots are tap - n0 + 1: slot 0 takes what belongs below the item, the
                            // last, n1 - n0 + 1, what belongs above it, and this and the 63 behind it what the lanes
                            // drop; none of these is read
    int k_cut;              // reflections from which on nothing can add to a sum (see reflection_cut)
    int nmx, nmy, nmz;      // images |n| <= nm of each axis
    Axis ax, ay, az;
    double beta, r_out2, walk2;      // walk2: squared distance from which images are walked
    float inv_log2_beta;    // 0: no cut
    int near_item;          // images nearer than kNearMetres are walked apart
    int tested;             // the ends of columns drop what lies outside by its distance
    int edges;              // steps of a column that may hold images outside the shell: its first, last, second, last but one, ...

    // taps
    double k_fs_c;
    double quick_k;         // fs/c, less the middle of the hardware estimate's error
    double quick_shift;     // 0.5 + margin - (n0 - 1) + kQuickMagic
    int quick_margin2;      // quick estimates whose 16-bit fraction is below this are formed again (see walk_step)
    double shift;           // 0.5 + guard - (n0 - 1)
    double guard2;
    double settle_shift;    // the same in units of 2^-32 tap (see walk_step)
    unsigned int settle_guard2;

    // the z axis (see walk_step) and the range of a column in steps of 2 L:
    // first p = ceil(lo[0] sqrt(walk2 - a) + lo[1]), last p = floor(hi[0] sqrt(r_out2 - a) + hi[1])
    double two_l, begin[4];
    float lo[2], hi[2];
    // An image (q, n) with k reflections lies at most k L + max(|s - m|, |L - s - m|) from the microphone along its axis:
    // with k of them, no y image is beyond y_reach[0] k + y_reach[1] metres, and with k for y and z together, no z image of
    // the y image at |dy| is beyond z_reach[0] k + z_reach[1] - z_reach[2] |dy|.
    float y_reach[2], z_reach[3];
    AxisCount cy;
    AxisOrder y_order;
};
// Images of the y table: a row's bound lies within y_reach of the cut, or r_out, both less than 2 (nmy + 2) L.
__device__ inline int y_images(int nmy) { return 4 * (nmy + 2); }
// two consecutive taps; only their 4-byte alignment is promised
struct __attribute__((aligned(4))) TapPair { float x, y; };
constexpr int kEnd = -1, kSilent = 0, kFast = 1, kPlain = 2;      // no more items; a room that is not usable; the walk; the plain walk

// the reference recipe, out of line so that the walk stays short
__device__ __attribute__((noinline)) int exact_tap(double d2, double k_fs_c) {
    const double d = __dsqrt_rn(d2);
    return (int)__dadd_rn(__dmul_rn(d, k_fs_c), 0.5);     // positive: truncation is floor
}

// Largest reflection count k whose amplitude beta^k / (4 pi d) can still add to a sum in the 2^-56 fixed
// point at distance d_min or beyond.  Increments are rounded to the nearest unit, so an amplitude below half a unit adds
// exactly zero; the cut is taken at 2^-57.5, a
// margin of a factor 1.41 under that, plus one count of slack, which covers the rounding of this estimate
// for every beta that the limit of 10^6 counts lets through.  "No limit" when beta is 0, >= 1
// (inv_log2_beta == 0 encodes both) or d_min is tiny.
constexpr int kNoCut = 1 << 20;
__device__ inline int reflection_cut(float inv_log2_beta, float d_min) {
    if (!(inv_log2_beta < 0.f) || !(d_min > 1e-3f)) return kNoCut;
    // beta^k >= 4 pi d 2^-57.5  <=>  k <= (log2(4 pi d) - 57.5) / log2(beta)
    const float k = (__builtin_amdgcn_logf(12.566371f * d_min) - 57.5f) * inv_log2_beta;
    return k > 1.0e6f ? kNoCut : (int)k + 2;
}

// Slot (tap - n0 + 1) of an image at squared distance d2, given y, the hardware's estimate of 1/sqrt(d2).
// One Newton step on the root leaves d fs/c good to ~1e-10 taps; shifted up by the guard, its fraction falls below
// 2 guard exactly when the true value may lie within the guard of a rounding boundary, and only then is the
// reference recipe evaluated, on the reference's own d2 (that of the walk may differ in the last bit).
template <class Taps, class ExactD2>
__device__ inline int tap_slot(const Taps& w, double d2, double y, ExactD2 exact_d2) {
    const double s0 = __dmul_rn(d2, y);                    // sqrt(d2) to 2^-24
    const double res = fma(-s0, s0, d2);                   // exact residual
    const double s1 = fma(__dmul_rn(res, y), 0.5, s0);     // one Newton step: ~4e-15 relative
    const double t = fma(s1, w.k_fs_c, w.shift);
    int slot = (int)t;
    if (__builtin_amdgcn_fract(t) < w.guard2) slot = exact_tap(exact_d2(), w.k_fs_c) - (w.n0 - 1);
    return slot;
}

// The walk first asks for less.  d2 rsq(d2) without the Newton step is the distance to within the hardware
// estimate's own error, which over all 2^31 leading mantissas of [1, 4) (three fillings of the remaining bits) lies
// between -3.24 and +7.10 units of 2^-27; with the middle of that range taken out of fs/c the error is below
// 5.2 * 2^-27: 3e-4 taps at tap 8000.  Adding 1.5 * 2^36 leaves slot and fraction as two sixteen-bit halves of the
// sum's low word: the address is a shift of one half, the test a comparison of the other, and the Newton step,
// conversion, fraction and double-precision comparison are not needed (40 instead of 60 issue cycles, without rsq,
// per image).  y ~ 1/sqrt(d2) is enough for the amplitude.
constexpr double kAmplitude = 0.07957747154594767 * 0x1p56;      // 1 / (4 pi) in the sums' fixed point
constexpr double kQuickMagic = 0x1.8p36, kSettleMagic = 0x1.8p20;
constexpr int kSettleHigh = 0x41380000;                          // high word of kSettleMagic
constexpr double kQuickMiddle = 1.93 * 0x1p-27, kQuickError = 5.2 * 0x1p-27;
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

// The z images of a response are four arithmetic progressions of step 2 L, at distances u + begin[list], u = 2 L p,
// from the microphone's plane (L the room's height, s and m the heights of source and microphone):
//   list 0: |s - m|,        2 p reflections       list 2: s + m,        2 p + 1
//   list 1: 2 L - |s - m|,  2 p + 2               list 3: 2 L - (s + m), 2 p + 1
// (for |s + m| <= 2 L and |s - m| <= 2 L, so that every list begins between 0 and 2 L; below the floor, s + m < 0, list 2
// begins with an image at |s + m| on the other side, and list 3 beyond 2 L).  u is exact in double precision, a multiple of a
// 24-bit number below 2^12 of them.
// squared distance of image (list, p) by the reference recipe; a: of the column
__device__ __attribute__((noinline)) double exact_z_image(Axis az, double a, double u, int list) {
    const int p = (int)rint(u / (2.0 * az.room));
    const bool below = az.src < az.mic;
    const int n = list == 0 ? (below ? -p : p) : list == 1 ? (below ? 1 + p : -1 - p) : list == 2 ? -p : 1 + p;
    const double dz = axis_delta(az, list >> 1, n);
    return __dadd_rn(a, __dmul_rn(dz, dz));
}

// fma(a, b, c) with c left as it is: the compiler takes the two-address form, which destroys c, and copies it first for
// each of four uses
__device__ inline double fma_keep(double a, double b, double c) {
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ inline double fma_keep_uniform(double a, double b_uniform, double c) {
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "s"(b_uniform), "v"(c));
    return r;
}
struct WalkRegs {           // what every step needs of the item, moved to scalar registers for the length of a chunk
    double begin[4], quick_k, quick_shift, beta, k_fs_c, settle_shift;
    unsigned int settle_guard2;
    unsigned short quick_margin2;
    __device__ explicit WalkRegs(const ItemCtx& c)
        : begin{uni(c.begin[0]), uni(c.begin[1]), uni(c.begin[2]), uni(c.begin[3])}, quick_k(uni(c.quick_k)), quick_shift(c.quick_shift),
          beta(uni(c.beta)), k_fs_c(uni(c.k_fs_c)), settle_shift(uni(c.settle_shift)), settle_guard2((unsigned int)uni((int)c.settle_guard2)),
          quick_margin2((unsigned short)uni(c.quick_margin2)) {}
};
// The four images of a column at u = 2 L p.  amp = beta^(kxy + 2 p) / (4 pi) 2^56; leaves that of the next step.
// Four independent chains of arithmetic; no memory is read.  EDGE: some of the images may lie outside the item's
// shell and go to the lane's own slot for such (dropped8), with `tested` by their distance (see ItemCtx::tested); else every one
// lies inside, up to the slack of the closed form (a fifth of a tap), so its slot is one of 0 .. taps + 1 and needs no test.
template <bool COUNT, bool EDGE>
__device__ inline int walk_step(const ItemCtx& w, const WalkRegs& k, bool tested, double a, double u, double& amp,
                                unsigned int dropped8, unsigned long long* hist) {
    double d2[4], y[4];
    unsigned int slot8[4];
    unsigned short fraction[4];
#pragma unroll
    for (int l = 0; l < 4; ++l) {
        const double dz = __dadd_rn(u, k.begin[l]);
        d2[l] = fma_keep(dz, dz, a);
        y[l] = __builtin_amdgcn_rsq(d2[l]);
        const unsigned int t = (unsigned int)__double2loint(fma_keep_uniform(__dmul_rn(d2[l], y[l]), k.quick_k, k.quick_shift));
        slot8[l] = t >> 13 & 0x7fff8u;
        fraction[l] = (unsigned short)t;
    }
    // (one test for all, so that the estimates are complete before the branch)
    if (min(min(fraction[0], fraction[1]), min(fraction[2], fraction[3])) < k.quick_margin2) {
#pragma unroll
        for (int l = 0; l < 4; ++l)
            if (fraction[l] < k.quick_margin2) {
                const double s0 = __dmul_rn(d2[l], y[l]), s1 = fma(__dmul_rn(fma(-s0, s0, d2[l]), y[l]), 0.5, s0);
                const double t = fma(s1, k.k_fs_c, k.settle_shift);
                int slot = __double2hiint(t) - kSettleHigh;
                if ((unsigned int)__double2loint(t) < k.settle_guard2) slot = exact_tap(exact_z_image(w.az, a, u, l), k.k_fs_c) - (w.n0 - 1);
                slot8[l] = 8u * (unsigned int)slot;
            }
    }
    int walked = 0;
    if (EDGE) {
#pragma unroll
        for (int l = 0; l < 4; ++l) slot8[l] = min(slot8[l], dropped8);
        if (tested) {
#pragma unroll
            for (int l = 0; l < 4; ++l) slot8[l] = d2[l] < w.walk2 || d2[l] >= w.r_out2 ? dropped8 : slot8[l];
        }
#pragma unroll
        for (int l = 0; l < 4; ++l) walked += slot8[l] < w.top8;
    }
    const double amp_odd = __dmul_rn(amp, k.beta), amp_far = __dmul_rn(amp_odd, k.beta);
#pragma unroll
    for (int l = 0; l < 4; ++l) deposit<COUNT, true>(slot8[l], l == 0 ? amp : l == 1 ? amp_far : amp_odd, y[l], hist);
    amp = amp_far;
    return walked;
}

// beta^k / (4 pi) in the sums' fixed point: what a walk that multiplies by beta from one reflection to the next comes to, wherever
// it began, so that an image's amplitude does not depend on where its response was cut.  `table` holds the first kPow and from
// there every kPowStep-th.
__device__ inline double power(const double* table, double beta, int k) {
    double v = table[k < kPow ? k : kPow + (k - kPow) / kPowStep];
    if (k >= kPow)
        for (int i = (k - kPow) % kPowStep; i > 0; --i) v *= beta;
    return v;
}
// The same for the plain walk, whose images come in no order of their reflections: those past kPow one by one, in the LDS that the
// fast walk has its y images in.  (Out of line and multiplied up from every 64th for each image, 16 responses of 16000 taps of rooms
// of 1 to 2 m without a cut took 18.8 ms, 4.8 so.)
__device__ __attribute__((noinline)) double pow_far(double beta, int k) { return pow(beta, (double)k) * kAmplitude; }
__device__ inline double power_any(const double* table, const double* past, double beta, int k) {
    return k < kPowMost ? *(k < kPow ? table + k : past + (k - kPow)) : pow_far(beta, k);
}
// by one wavefront, from `table`
__device__ inline void form_powers_past(const double* table, double* past, double beta, int lane) {
    static_assert(kPowMost - kPow <= (kYCap < 64 * kPowStep ? kYCap : 64 * kPowStep), "a lane forms kPowStep of them");
    const int begin = kPowStep * lane, end = min(begin + kPowStep, kPowMost - kPow);
    if (begin >= end) return;
    double v = table[kPow + lane];
    for (int i = begin; i < end; ++i, v *= beta) past[i] = v;
}

// Items that the closed forms do not take (rooms too flat or narrow for the tables, positions far outside): every column of
// the bounding box, of a live column the z images about the item's shell, every tap tested.  (All z images of every column: 16
// responses of 16000 taps of rooms of 1 to 2 m without a cut took 112 ms, 4.8 so.)  Out of line for the same reason as the power.
// Distance and amplitude of an image are formed as walk_step forms them, step for step: whether an item fits the tables
// depends on where the batch's plan has cut the response, and the response must not.
template <bool COUNT>
__device__ __attribute__((noinline)) unsigned int walk_plain(const ItemCtx& w, int rir_len, const double* powers, const double* powers_past, unsigned long long* hist) {
    unsigned int walked = 0;
    // Of positions far outside, no shell's radius bounds the numbers of its images: those of the whole response's radius, in
    // whatever item they land.  (Formed here, where they are asked for: in prepare_item they took 2048 responses of 1000 taps of ordinary
    // rooms 51 us instead of 49.5.)
    auto most_n = [&](const Axis& ax, int within, int most) {
        return axis_in_order(ax) ? within : min((int)ceil((double)rir_len / w.k_fs_c / (2.0 * ax.room)) + 1, most);
    };
    const int nmx = most_n(w.ax, w.nmx, w.k_cut / 2 + 1), nmy = most_n(w.ay, w.nmy, w.k_cut / 2 + 1), nmz = most_n(w.az, w.nmz, kNoCut);
    const int niy = 2 * (2 * nmy + 1);
    // (what every image needs, in scalar registers: read from LDS again behind every add to the sums, one value after the other, it took
    // those 16 responses 7.0 ms instead of 4.8)
    struct { double k_fs_c, shift, guard2; int n0; } const taps{uni(w.k_fs_c), uni(w.shift), uni(w.guard2), uni(w.n0)};
    const Axis az{uni(w.az.room), uni(w.az.src), uni(w.az.mic)};
    const double begin[4] = {uni(w.begin[0]), uni(w.begin[1]), uni(w.begin[2]), uni(w.begin[3])};
    const double two_l = uni(w.two_l), beta = uni(w.beta);
    const unsigned int last_slot = (unsigned int)uni((int)w.top8) / 8u;
    const bool below = az.src < az.mic, in_steps = axis_in_order(az);
    const long long n_columns = 2ll * (2 * nmx + 1) * niy;
    const double r_in = w.n0 > 0 ? (double)(w.n0 - 1) / w.k_fs_c : 0.0, inv_2l = 1.0 / w.two_l;
    // what the recipe's operations may move an image of the z axis by: positions so far outside that it is more than a room's
    // height put several images in one place, or none
    const double rounding = 0x1p-50 * (fabs(w.az.src) + fabs(w.az.mic) + w.two_l * (double)(nmz + 1));
    for (long long cand = threadIdx.x; cand < n_columns; cand += kThreads) {
        const int ix = (int)(cand / niy), iy = (int)(cand - (long long)ix * niy);
        const int qx = ix & 1, nx = (ix >> 1) - nmx, qy = iy & 1, ny = (iy >> 1) - nmy;
        const double dx = axis_delta(w.ax, qx, nx), dy = axis_delta(w.ay, qy, ny);
        const double a = __dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy));
        const int kxy = reflections(qx, nx) + reflections(qy, ny);
        // (beyond the first shell the shell's own inner radius bounds the distance well enough)
        const int kz_max = (w.n0 > 0 ? w.k_cut : reflection_cut(w.inv_log2_beta, sqrtf((float)a))) - kxy;
        if (!(a < w.r_out2) || kz_max < 0) continue;
        const double far = sqrt(w.r_out2 - a) + rounding, near = fmax(sqrt(fmax(r_in * r_in - a, 0.0)) - rounding, 0.0);
        const int nz = min(nmz, kz_max / 2 + 1);                     // |n - q| + |n| >= 2 |n| - 1
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            // the images from -far to far but for those between -near and near, and one more at every end for rounding
            const double at_zero = axis_delta(az, q, 0);
            auto below_distance = [&](double dz) { return (int)fmin(fmax(floor((dz - at_zero) * inv_2l), -(double)nz - 2.0), (double)nz + 2.0); };
            const int first = max(below_distance(-far), -nz), last = min(below_distance(far) + 1, nz);
            const int hole_first = below_distance(-near) + 2, hole_last = below_distance(near) - 1;
            for (int n = first; n <= last; ++n) {
                if (n >= hole_first && n <= hole_last) {
                    n = hole_last;
                    continue;
                }
                // image (q, n) as element p of its list (see walk_step)
                const bool up = q ? n > 0 : n && (n > 0) == below;
                const int p = up ? abs(n) - 1 : abs(n);
                const double dz = axis_delta(az, q, n), recipe = __dadd_rn(a, __dmul_rn(dz, dz));
                // (the recipe rounds positions far outside to less than the tap's guard allows: there it is what counts)
                const double step = __dadd_rn(__dmul_rn(two_l, (double)p), up ? begin[2 * q + 1] : begin[2 * q]);
                const double d2 = in_steps ? fma(step, step, a) : recipe;
                const double y = __builtin_amdgcn_rsq(d2);
                const int slot = tap_slot(taps, d2, y, [&] { return recipe; });
                if ((unsigned int)slot > last_slot) continue;       // (eight times a slot beyond 2^29 would come round)
                const double amp = COUNT ? 0.0 : power_any(powers, powers_past, beta, kxy + 2 * p + (q ? 1 : up ? 2 : 0));
                deposit<COUNT, false>(8u * (unsigned int)slot, amp, y, hist);
                ++walked;
            }
        }
    }
    return walked;
}

// The images within kNearMetres, with the test for amplitudes too large for the fast rounding: of the columns of the x images
// |n| <= n_near and the first n_y images along y, those at steps p < n_p along z.
struct NearImages {
    int n_near, n_y, n_p, n;
    __device__ explicit NearImages(const ItemCtx& w) {
        const float r_near = __builtin_amdgcn_sqrtf((float)w.walk2) * 1.0001f;
        n_near = min((int)(r_near / (2.f * (float)w.ax.room)) + 1, w.nmx);
        n_y = min(count_within(w.cy, r_near), y_images(w.nmy));
        n_p = min((int)(r_near / (float)w.two_l) + 1, w.nmz) + 1;
        n = 2 * (2 * n_near + 1) * n_y * n_p * 4;
    }
};
__device__ __attribute__((noinline)) unsigned int walk_near(const ItemCtx& w, int n_near, int n_y, int n_p, int i, const double* ykey, const unsigned short* ycount,
                                                            const double* powers, unsigned long long* hist) {
    const int l = i & 3, column = (i >> 2) / n_p, p = (i >> 2) - column * n_p, ix = column / n_y, iy = column - ix * n_y;
    const int qx = ix & 1, nx = (ix >> 1) - n_near;
    const double dx = axis_delta(w.ax, qx, nx);
    const double a = __dadd_rn(__dmul_rn(dx, dx), ykey[iy]);
    const int kxy = reflections(qx, nx) + ycount[iy];
    const double u = w.two_l * (double)p, dz = __dadd_rn(u, w.begin[l]), d2 = fma(dz, dz, a);
    // (past the cut the amplitudes are zero, and their powers have not been formed)
    if (!(d2 < w.walk2) || kxy > w.k_cut) return 0;
    const double y = __builtin_amdgcn_rsq(d2);
    const int slot = tap_slot(w, d2, y, [&] { return exact_z_image(w.az, a, u, l); });
    if (8u * (unsigned int)slot > w.top8) return 0;
    deposit<false, false>(8u * (unsigned int)slot, power(powers, w.beta, kxy + 2 * p + (l == 0 ? 0 : l == 1 ? 2 : 1)), y, hist);
    return 1;
}

// The powers of an item's reflection coefficient, by one wavefront, for the counts that an image can have: at most the cut (which
// steps near the microphone are not held to) or all there are.  One multiplication after the other (see power): formed while
// others set up the item's y images and rows.
template <bool COUNT>
__device__ inline void form_powers(const ItemCtx& c, double* powers, int lane) {
    if (COUNT || lane || c.kind == kSilent || c.kind == kEnd) return;
    const double beta = c.beta;
    const int near_steps = c.near_item ? (int)((float)kNearMetres * 1.1f * c.lo[0]) + 4 : 0;       // (lo[0] ~ 1 / 2 L)
    const int k_all = c.kind == kPlain ? kPowMost : 2 * (c.nmx + c.nmy + c.nmz) + 8;
    const int k_most = min(min(c.k_cut + 2 * near_steps + 8, k_all), kPowMost - 1);
    double v = kAmplitude;
    for (int k = 0; k <= min(k_most, kPow - 1); k += 8) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            powers[k + i] = v;
            v *= beta;
        }
    }
    for (int k = kPow; k <= k_most; k += kPowStep) {
        powers[kPow + (k - kPow) / kPowStep] = v;
#pragma unroll
        for (int i = 0; i < kPowStep; ++i) v *= beta;
    }
}

// Prepares item `it`: all lanes of one wavefront compute the same, lane 0 writes.
template <bool COUNT>
__device__ inline void prepare_item(ItemCtx& ctx, const Rooms& rooms, double k_fs_c, const Item* __restrict__ items, int it, int n_items, int lane) {
    ItemCtx c{};
    c.kind = kEnd;
    if (it < n_items) {
        const Item item = items[it];
        const Room room = load_room(rooms, uni(item.rir));
        const float* g = room.g;
        const int n0 = item.n0, n1 = item.n1;
        c.kind = kSilent;
        c.rir = item.rir;
        c.n0 = n0;
        c.n1 = n1;
        c.top8 = 8u * (unsigned int)(n1 - n0 + 1);
        if (room_ok(g)) {
            const Axis ax{(double)g[0], (double)g[3], (double)g[6]}, ay{(double)g[1], (double)g[4], (double)g[7]},
                az{(double)g[2], (double)g[5], (double)g[8]};
            c.ax = ax;
            c.ay = ay;
            c.az = az;
            c.beta = (double)g[9];
            // every image of this item lies in r_in <= d < r_out (half a tap of slack on either side)
            const double r_out = (double)n1 / k_fs_c, r_in = n0 > 0 ? (double)(n0 - 1) / k_fs_c : 0.0;
            c.r_out2 = r_out * r_out;
            // An image reflected k times adds beta^k / (4 pi d) * 2^56, rounded to an integer, to its
            // tap; once beta^k < 2 pi d 2^-56 that is exactly zero, so such images are never visited.
            // (amplitude sums only; tap counts visit every image)
            c.inv_log2_beta = (!COUNT && g[9] > 0.f && g[9] < 1.f) ? 1.f / __log2f(g[9]) : 0.f;
            c.k_cut = reflection_cut(c.inv_log2_beta, (float)r_in);
            c.nmx = min((int)ceil(r_out / (2.0 * ax.room)) + 1, c.k_cut / 2 + 1);          // |n - q| + |n| >= 2 |n| - 1
            c.nmy = min((int)ceil(r_out / (2.0 * ay.room)) + 1, c.k_cut / 2 + 1);
            c.nmz = (int)ceil(r_out / (2.0 * az.room)) + 1;
            c.k_fs_c = k_fs_c;
            // (in whole units of the estimate's 2^-16 tap, so that adding it to the magic number is exact; one unit
            // for the sum's rounding)
            const double margin = ceil(kQuickError * 65536.0 * (double)(n1 + 2)) + 1.0;
            c.quick_k = k_fs_c * (1.0 - kQuickMiddle);
            c.quick_shift = kQuickMagic + (0.5 + margin * 0x1p-16 - (double)(n0 - 1));
            c.quick_margin2 = (int)(2.0 * margin) + 1;
            const double guard = 1e-12 * (double)(n1 + 1) + 1e-13;
            c.shift = (0.5 + guard) - (double)(n0 - 1);
            c.guard2 = 2.0 * guard;
            const double settle = ceil(guard * 0x1p32) + 1.0;
            c.settle_shift = kSettleMagic + (0.5 + settle * 0x1p-32 - (double)(n0 - 1));
            c.settle_guard2 = (unsigned int)(2.0 * settle) + 1u;
            c.two_l = 2.0 * az.room;
            const double apart = fabs(az.src - az.mic), both = az.src + az.mic;
            c.begin[0] = apart;
            c.begin[1] = c.two_l - apart;
            c.begin[2] = both;
            c.begin[3] = c.two_l - both;
            // beyond 2.6 m every amplitude is below 2^-5 (see deposit); the few images of the innermost items that may be
            // nearer are walked apart
            const double r_near = kNearMetres + 0.25 / k_fs_c;
            c.near_item = !COUNT && r_in < r_near;
            c.walk2 = c.near_item ? r_near * r_near : r_in * r_in;
            // the fast walk: the x and y images fit the LDS tables, the steps along z a column's record, and the closed forms hold
            const double height_taps = az.room * k_fs_c;
            const bool fast = axis_in_order(ax) && axis_in_order(ay) && axis_in_order(az) && 2 * (2 * c.nmx + 1) <= 2 * kAxisCap && y_images(c.nmy) <= kYCap && c.nmz <= kMaxP &&
                              fmax(ay.room, az.room) * k_fs_c < kMaxAxisTaps && height_taps >= kMinHeightTaps;
            c.tested = c.near_item || height_taps > kWrapTaps || both < 0.0;
            // (the lists begin within 2 L of each other, or, with positions below the floor, 6 L; next to images that are walked
            // apart the bound counts to the last bit, and its slack is worth another step)
            c.edges = (both < 0.0 ? 6 : 2) + (c.near_item ? 1 : 0);
            c.kind = fast ? kFast : kPlain;
            c.cy = axis_count(ay, k_fs_c);
            c.y_order = axis_order(ay);
            const float slack = c.cy.slack, inv2l = (float)(1.0 / c.two_l), z_per_y = (float)(az.room / ay.room);
            auto farthest = [](const Axis& ax1) {
                return 1.0001f * fmaxf(fabsf((float)(ax1.src - ax1.mic)), fabsf((float)(ax1.room - ax1.src - ax1.mic))) + 1e-3f;
            };
            c.y_reach[0] = 1.0001f * (float)ay.room;
            c.y_reach[1] = farthest(ay);
            c.z_reach[0] = 1.0001f * (float)az.room;
            c.z_reach[1] = farthest(az) + c.y_reach[1] * z_per_y;
            c.z_reach[2] = 0.9999f * z_per_y;
            // the nearest and the farthest beginning of a list, in units of 2 L
            const float least = (float)(fmin(fmin(apart, c.begin[1]), fmin(both, c.begin[3])) / c.two_l);
            const float most = (float)(fmax(fmax(apart, c.begin[1]), fmax(both, c.begin[3])) / c.two_l);
            c.lo[0] = 0.999998f * inv2l;
            c.lo[1] = -slack * inv2l - most;
            c.hi[0] = 1.000002f * inv2l;
            c.hi[1] = slack * inv2l - least;
        }
    }
    if (lane == 0) ctx = c;
}

// What a group of the kernel below keeps in LDS: two must fit a compute unit, or the 2 n_cu persistent groups run in two rounds.
constexpr size_t kImageLds = 8 * (size_t)kPool + 8 * kPowTable + 10 * kYCap + 10 * 2 * kAxisCap + 4 * (2 * kAxisCap / 64 + 5 + 2 * 64 + 1) + 2 * sizeof(ItemCtx) + 16;      // (the last: alignment)
static_assert(kImageLds <= 80 * 1024 && 2 * kThreads <= 4 * 4 * 64, "two groups on a compute unit");

// VISITS: a measuring instantiation that also adds the number of images it walked to *visits.
template <bool COUNT, bool VISITS = false>
__global__ __launch_bounds__(kThreads, 4) void rir_image_kernel(
    Rooms rooms, int rir_len, double k_fs_c, const Item* __restrict__ items,
    int* __restrict__ ctrl, float* __restrict__ rir_out,
    int32_t* __restrict__ cnt_out, unsigned long long* __restrict__ visits = nullptr) {
    __shared__ __align__(16) unsigned long long hist[kPool];       // tap sums, and behind them the live columns of a chunk
    __shared__ __align__(16) double s_powers[COUNT ? 1 : kPowTable];    // beta^k / (4 pi) 2^56
    __shared__ double ykey[kYCap];                 // y images in order of distance: dy*dy
    __shared__ unsigned short ycount[kYCap];       // and reflections
    __shared__ unsigned short row_count[2 * kAxisCap];     // live columns per x image, summed up within every 64 of them
    __shared__ int row_part[2 * kAxisCap / 64];    // the totals of those
    __shared__ unsigned int row_gap[2 * kAxisCap];         // y images before the dead ones, and how many these are << 16
    __shared__ int row_begin[2 * kAxisCap + 5];    // the first column of every x image (and what is read past the last)
    __shared__ int census[2][64];                  // columns per length
    __shared__ int s_round;
    __shared__ ItemCtx s_ctx[2];
    unsigned int* hist32 = reinterpret_cast<unsigned int*>(hist);

    int tid = threadIdx.x, lane = tid & 63;
    const int wave = uni(tid >> 6), n_items = ctrl[0];
    unsigned long long walked = 0;
    // by one wavefront.  A group begins with the item of its own number: 512 groups that ask one counter wait for each other (128 responses of
    // 500 taps 17.9 us instead of 14.8; 600 of 1000, where all ask for their second item at once, 24.6 instead of 26.2).
    auto prepare_next = [&](ItemCtx& ctx) {
        int it = 0;
        if (lane == 0) it = (int)gridDim.x + atomicAdd(&ctrl[1], 1);
        prepare_item<COUNT>(ctx, rooms, k_fs_c, items, uni(it), n_items, lane);
    };

    // sums start at zero and are left at zero where an item is written out (and where the next one's lie over its columns)
    if (COUNT) {
        for (int i = tid; i < kMaxTaps + 65; i += kThreads) hist32[i] = 0u;
    } else {
        for (int i = tid; i < kMaxTaps + 65; i += kThreads) hist[i] = 0ull;
    }
    if (wave == kWaves - 1) prepare_item<COUNT>(s_ctx[0], rooms, k_fs_c, items, (int)blockIdx.x, n_items, lane);

    for (int now = 0, items_done = 0;; now ^= 1, ++items_done) {
        group_sync();                              // s_ctx[now] is there, and the sums of the item before are complete
        // (opaque: addresses are formed anew for every item, kept from one to the next they do not fit the registers)
        asm volatile("" : "+v"(tid));
        lane = tid & 63;
        const ItemCtx& c = s_ctx[now];
        if (items_done > 0) {
            const ItemCtx& before = s_ctx[now ^ 1];
            const int n_taps = uni(before.n1 - before.n0), n_clear = max(n_taps, uni(c.n1 - c.n0)) + 65;
            const size_t to = (size_t)uni(before.rir) * rir_len + uni(before.n0) - 1;
            if (COUNT) {
                for (int i = tid; i < n_clear; i += kThreads) {
                    const unsigned int v = hist32[i];
                    hist32[i] = 0u;
                    if (i > 0 && i <= n_taps) cnt_out[to + i] = (int32_t)v;
                }
            } else {
                // two slots per thread and round
                float* const out = rir_out + to;
                ulonglong2* const pairs = reinterpret_cast<ulonglong2*>(hist);
                auto value = [](unsigned long long v) {
                    return (float)(fma((double)(unsigned int)(v >> 32), 0x1p32, (double)(unsigned int)v) * 0x1p-56);
                };
#pragma unroll 3
                for (int i = tid; 2 * i < n_clear; i += kThreads) {
                    const ulonglong2 v = pairs[i];
                    pairs[i] = make_ulonglong2(0ull, 0ull);
                    const TapPair t{value(v.x), value(v.y)};
                    if (i > 0 && 2 * i + 1 <= n_taps) {
                        *reinterpret_cast<TapPair*>(out + 2 * i) = t;
                    } else {
                        if (i > 0 && 2 * i <= n_taps) out[2 * i] = t.x;
                        if (2 * i + 1 <= n_taps) out[2 * i + 1] = t.y;
                    }
                }
            }
        }
        const int kind = uni(c.kind);
        if (kind == kEnd) break;

        const int nmx = uni(c.nmx), nmy = uni(c.nmy), nmz = uni(c.nmz), k_cut = uni(c.k_cut);
        const int nix = 2 * (2 * nmx + 1), n_yimages = y_images(nmy), segments = (nix + 63) / 64;
        const double* const powers = s_powers;
        if (wave == 0) form_powers<COUNT>(c, s_powers, lane);
        if (kind == kFast) {
            for (int i = tid ^ 64; i < n_yimages; i += kThreads) {
                int q, n;
                ordered_image(c.y_order, i, q, n);
                const double dy = axis_delta(c.ay, q, n);
                ykey[i] = __dmul_rn(dy, dy);
                ycount[i] = (unsigned short)reflections(q, n);
            }
            // Columns of x image ix that may be live: the y images with dy^2 <= r_out^2 - dx^2 that the reflection
            // cut can still reach -- the first of the y table --, but for those in a gap: what reflections they leave does
            // not take their z images as far as the shell's inner radius, A - B |dy| < sqrt(R^2 - dy^2), an interval of |dy|.
            // (Five of six columns of 32 responses of 32768 taps, half of those of 3072.)  The wavefronts from the other
            // end: those have no y image.
            for (int seg = kWaves - 1 - wave; seg < segments; seg += kWaves) {
                const int ix = 64 * seg + lane, qx = ix & 1, nx = (ix >> 1) - nmx;
                const double dx = axis_delta(c.ax, qx, nx), dx2 = __dmul_rn(dx, dx);
                const float outer = (float)(c.r_out2 - dx2), inner = (float)(c.walk2 - dx2) * 0.9999f;
                const int k_left = k_cut - reflections(qx, nx);
                const float reach = fmaf((float)k_left, c.y_reach[0], c.y_reach[1]);
                int count = 0;
                unsigned int gap = 0;
                if (outer >= 0.f && k_left >= 0 && ix < nix) {
                    count = min(count_within(c.cy, fminf(__builtin_amdgcn_sqrtf(outer), reach)), n_yimages);
                    const float A = fmaf((float)k_left, c.z_reach[0], c.z_reach[1]), B = c.z_reach[2], s = fmaf(B, B, 1.f);
                    const float D = fmaf(inner, s, -A * A);
                    if (D > 0.f) {
                        const float root = __builtin_amdgcn_sqrtf(D), scale = __builtin_amdgcn_rcpf(s);
                        const float from = (A * B - root) * scale, to = (A * B + root) * scale;
                        const int first = from > 0.f ? min(count_within(c.cy, from), count) : 0;
                        const int last = min(count_within<-1>(c.cy, to * 0.99999f), count);
                        if (last > first) {
                            gap = (unsigned int)(first | (last - first) << 16);
                            count -= last - first;
                        }
                    }
                }
                const int part = wave_inclusive_scan(count);
                if (ix < nix) {
                    row_count[ix] = (unsigned short)part;
                    row_gap[ix] = gap;
                }
                if (lane == 63) row_part[seg] = part;
            }
            if (tid < 128) census[tid >> 6][lane] = 0;
        } else if (!COUNT && kind == kPlain && wave == 0) {
            wave_sync_lds();
            form_powers_past(powers, ykey, c.beta, lane);
        }
        group_sync();

        bool prepared = false;
        if (kind == kFast) {
            // the rows' prefix sums: every wavefront forms all of them (and writes what the others write), so that none
            // waits for another
            const int my_part = lane < segments ? row_part[lane] : 0, up_to_part = wave_inclusive_scan(my_part);
            const int n_cand = __builtin_amdgcn_readlane(up_to_part, 63);
            for (int seg = 0; seg < segments; ++seg) {
                const int i = 64 * seg + lane;
                if (i < nix) row_begin[i + 1] = (int)row_count[i] + (seg ? __builtin_amdgcn_readlane(up_to_part, seg - 1) : 0);
            }
            if (lane < 4) row_begin[lane ? nix + lane : 0] = lane ? 0x7fffffff : 0;
            wave_sync_lds();
            const bool near_item = uni(c.near_item) != 0, tested = uni(c.tested) != 0;
            const int edges = uni(c.edges);

            // Columns are worked through a chunk at a time: as many candidates as there is certainly room for behind the sums.
            // Each thread describes kPerThread of them (the wavefronts' stretches of 64 side by side, so that a wavefront's rows
            // only move up), two at a time so that one's loads and roots are under way with the other's; the live ones
            // are sorted by length, in LDS, and taken 64 at a time, longest first, from a counter.
            // (The images near the microphone are walked after the last chunk's columns.  An item that has such images takes one
            // chunk also where the gaps leave it no column: they remove the columns whose images all lie that near.)
            const int behind = uni(c.n1 - c.n0) + 66 & ~1, room = (kPool - behind) * 2 / 3 & ~1, chunk = min(room / kThreads, kPerThread) * kThreads;
            double* const col_a = reinterpret_cast<double*>(hist + behind);       // the columns, longest first: dx*dx + dy*dy
            unsigned int* const col_range = reinterpret_cast<unsigned int*>(col_a + room);      // first p, last p less that << 8, reflections << 16
            for (int base = 0, parity = 0; base < n_cand || (base == 0 && near_item); base += chunk, parity ^= 1) {
                double a[kPerThread];
                unsigned int range[kPerThread];
                int place[kPerThread];                    // length << 16 | number among those of that length, -1: not live
                // the rows of the stretches' first columns
                int first_row[kPerThread];
#pragma unroll
                for (int j = 0; j < kPerThread; ++j) {
                    first_row[j] = 0;
                    place[j] = -1;
                }
                if (base < n_cand)
                    for (int seg = 0; seg < segments; ++seg) {
                        const int i = 64 * seg + lane, end = i < nix ? row_begin[i + 1] : 0x7fffffff;
#pragma unroll
                        for (int j = 0; j < kPerThread; ++j)
                            first_row[j] += __popcll(__ballot(end <= min(base + 64 * (kWaves * j + wave), n_cand - 1)));
                    }
                const Axis ax{uni(c.ax.room), uni(c.ax.src), uni(c.ax.mic)};
                const double r_out2 = uni(c.r_out2), walk2 = uni(c.walk2);
                const float lo0 = uni(c.lo[0]), lo1 = uni(c.lo[1]), hi0 = uni(c.hi[0]), hi1 = uni(c.hi[1]), inv_log2_beta = uni(c.inv_log2_beta);
                const bool inner_item = uni(c.n0) == 0;
                // candidates `pair` .. `pair` + N - 1
                auto describe = [&](auto pair_constant, auto n_constant) {
                    constexpr int pair = decltype(pair_constant)::value, N = decltype(n_constant)::value;
                    // the lanes' own rows, from there: 64 consecutive columns span few rows, so the next four are compared at once
                    int cand[N], ix[N], ahead[N][4];
#pragma unroll
                    for (int e = 0; e < N; ++e)
#pragma unroll
                        for (int k = 0; k < 4; ++k) ahead[e][k] = row_begin[first_row[pair + e] + 1 + k];
                    bool farther = false;
#pragma unroll
                    for (int e = 0; e < N; ++e) {
                        cand[e] = min(base + 64 * (kWaves * (pair + e) + wave) + lane, n_cand - 1);
                        ix[e] = first_row[pair + e];
#pragma unroll
                        for (int k = 0; k < 4; ++k) ix[e] += ahead[e][k] <= cand[e];
                        farther |= ahead[e][3] <= cand[e];
                    }
                    if (farther) {                        // (seldom)
#pragma unroll
                        for (int e = 0; e < N; ++e)
                            while (row_begin[ix[e] + 1] <= cand[e]) ++ix[e];
                    }
                    int length[N];
#pragma unroll
                    for (int e = 0; e < N; ++e) {
                        const int j = pair + e;
                        const unsigned int gap = row_gap[ix[e]];
                        const int qx = ix[e] & 1, n2 = (ix[e] & ~1) - 2 * nmx, nth = cand[e] - row_begin[ix[e]];
                        const int iy = nth + (nth >= (int)(gap & 0xffffu) ? (int)(gap >> 16) : 0);
                        const double dx = axis_delta_2n(ax, qx, n2);
                        a[j] = __dadd_rn(__dmul_rn(dx, dx), ykey[iy]);
                        const int kxy = abs(n2 - qx) + ycount[iy];
                        // reflections left for the z axis before this column's images vanish
                        // (beyond the first shell the shell's own inner radius bounds the distance well enough)
                        const int cut = inner_item ? reflection_cut(inv_log2_beta, __builtin_amdgcn_sqrtf((float)a[j])) : k_cut;
                        const float outer = (float)(r_out2 - a[j]), inner = (float)(walk2 - a[j]);
                        // The images with r_in^2 <= a + dz^2 <= r_out^2 and reflections left: from the first p at which some
                        // list has begun to the last at which not all have ended.
                        const float to = fmaf(__builtin_amdgcn_sqrtf(fmaxf(outer, 0.f)), hi0, hi1);
                        const float from = fmaf(__builtin_amdgcn_sqrtf(fmaxf(inner, 0.f)), lo0, lo1);
                        const int p1 = min(min((int)floorf(to), (cut - kxy) >> 1), nmz), p0 = max((int)ceilf(from), 0);
                        range[j] = (unsigned int)(p0 | (p1 - p0) << 8 | kxy << 16);
                        const bool mine = base + 64 * (kWaves * j + wave) + lane < n_cand && kThreads * j < chunk;
                        length[e] = mine && outer > 0.f && cut >= kxy && p1 >= p0 ? min(p1 - p0, 63) : -1;
                    }
#pragma unroll
                    for (int e = 0; e < N; ++e)
                        if (length[e] >= 0) place[pair + e] = atomicAdd(&census[parity][63 - length[e]], 1) | (63 - length[e]) << 16;
                };
                const std::integral_constant<int, 1> one;
                const std::integral_constant<int, 2> two;
                const auto any = [&](int j) { return base + 64 * (kWaves * j + wave) < n_cand && kThreads * j < chunk; };
                // (a wavefront with one stretch is not kept by a second that is empty: 3000 responses of 1000 taps, whose items have some 70
                // candidates, took 68 us instead of 64)
                if (any(1)) describe(std::integral_constant<int, 0>(), two);
                else if (any(0)) describe(std::integral_constant<int, 0>(), one);
                if (any(2)) describe(two, two);
                group_sync();                             // also: every column of the chunk before has been walked
                const int of_length = census[parity][lane], up_to = wave_inclusive_scan(of_length);
                const int n_live = __builtin_amdgcn_readlane(up_to, 63), first = up_to - of_length;
                if (wave == 0) census[parity ^ 1][lane] = 0;
#pragma unroll
                for (int j = 0; j < kPerThread; ++j) {
                    if (base + kThreads * j >= n_cand) continue;
                    const int at = __shfl(first, (place[j] >> 16) & 63, 64) + (place[j] & 0xffff);
                    place[j] = place[j] >= 0 ? at : -1;
                }
                const WalkRegs regs(c);
                const double two_l = uni(c.two_l);
                const unsigned int dropped8 = uni((int)c.top8) + 8u * (unsigned int)lane;      // (slots apart: adds to one place queue up)
#pragma unroll
                for (int j = 0; j < kPerThread; ++j)
                    if (place[j] >= 0) {
                        col_a[place[j]] = a[j];
                        col_range[place[j]] = range[j];
                    }
                // behind the last chunk's candidates a wavefront prepares the next item before it joins in
                const bool last = base + chunk >= n_cand, apart = last && wave == kWaves - 1;
                if (tid == 0) s_round = last ? kWaves - 1 : kWaves;
                group_sync();
                const int column_rounds = (n_live + 63) / 64;
                int round = wave;
                auto next_round = [&] {
                    int next = 0;
                    if (lane == 0) next = atomicAdd(&s_round, 1);
                    return uni(next);
                };
                if (apart) {
                    prepare_next(s_ctx[now ^ 1]);
                    round = next_round();
                }
                prepared |= last;
                for (; round < column_rounds; round = next_round()) {
                    const int mine = 64 * round + lane;
                    if (mine < n_live) {
                        const double col = col_a[mine];
                        const unsigned int r = col_range[mine];
                        const int p0 = (int)(r & 255u), n = (int)(r >> 8 & 255u);
                        double amp = COUNT ? 0.0 : power(powers, regs.beta, (int)(r >> 16) + 2 * p0), u = two_l * (double)p0;
                        // its first steps, those between and its last, in this order so that the amplitude goes on from step to step
                        int at = 0;
#pragma unroll 1
                        for (int stop = min((edges + 1) >> 1, n + 1);; stop = n + 1) {
                            for (; at < stop; ++at, u += two_l) {
                                const int in = walk_step<COUNT, true>(c, regs, tested, col, u, amp, dropped8, hist);
                                if (VISITS) walked += in;
                            }
                            if (at > n) break;
                            int left = n + 1 - (edges >> 1) - at;
                            if (left > 0) {
                                if (VISITS) walked += 4 * left;
                                at += left;
                                do {
                                    walk_step<COUNT, false>(c, regs, false, col, u, amp, 0u, hist);
                                    u += two_l;
                                } while (--left > 0);
                            }
                        }
                    }
                }
                if (last && near_item) {
                    const NearImages near(c);
                    for (; 64 * (round - column_rounds) < near.n; round = next_round()) {
                        const int i = 64 * (round - column_rounds) + lane;
                        if (i < near.n) {
                            const unsigned int in = walk_near(c, near.n_near, near.n_y, near.n_p, i, ykey, ycount, powers, hist);
                            if (VISITS) walked += in;
                        }
                    }
                }
            }
        } else if (kind == kPlain) {
            walked += walk_plain<COUNT>(c, rir_len, powers, ykey, hist);
        }
        if (!prepared && wave == kWaves - 1) prepare_next(s_ctx[now ^ 1]);
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
    const PlanArgs p = rir_plan_args(n_groups, n_rir, rooms, rir_len, fs_over_c, items, ctrl);
    Item *const sorted = static_cast<Item*>(p.items), *const unsorted = static_cast<Item*>(p.unsorted);
    if (n_rir <= kPlanMost) {                                // one launch instead of four
        rir_plan_all_kernel<<<dim3(1), dim3(kPlanThreads), 0, s>>>(n_rir, rooms, rir_len, fs_over_c, sorted, unsorted,
                                                                    ctrl, n_groups);
        return hipGetLastError();
    }
    hipError_t e = launch_fill_u32(s, ctrl, 0u, kCtrlInts);
    if (e != hipSuccess) return e;
    rir_work_kernel<<<dim3((n_rir + 127) / 128), dim3(128), 0, s>>>(n_rir, rooms, rir_len, fs_over_c, ctrl);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    rir_plan_kernel<<<dim3((n_rir + 127) / 128), dim3(128), 0, s>>>(n_rir, rooms, rir_len, fs_over_c, unsorted, ctrl,
                                                                    n_groups);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t max_items = (size_t)n_rir * rir_items_per_response(rir_len);
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
