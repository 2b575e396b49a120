// Front end (Sec. 2.3): framed power spectrum, VTLP-warped mel filterbank, power law.
//
// P_t[k] = |DFT_K(hamming * x[t hop .. t hop + win))[k]|^2, k = 0..K/2;
// E_t[m] = sum_k Tri_m(f'_k) P_t[k] with f'_k the Eq. (1) bilinear warp of bin k;
// feature = E^(power).
//
// Adjacent unit-peak triangles share their edges, so a bin whose warped frequency
// falls between band edges c and c+1 feeds only filter c (rising side, weight w) and
// filter c-1 (falling side, weight 1-w).  A small kernel writes (c, w) per bin and
// utterance and how the filters are dealt to the matrix cores (MelPlan); the main kernel runs each K-point
// real transform as a K/2-point complex FFT (16 lanes per frame, two radix-16 passes with one exchange
// through LDS), forms the bin powers in registers and projects them with 4x4x1 matrix instructions.  Other
// epilogues of the same energies (log-mel, MFCC) and the on-the-fly mixture of reverberated sources
// are options of the kernel.

#include "fft_lds.h"
#include "pack_device.h"
#include "rir_plan.h"

namespace aug {
namespace {

constexpr int kMelThreads = 256;

// sample i of the symmetric Hamming window
__device__ inline float hamming(int i, int win) {
    double s, c;
    sincospi(2.0 * (double)i / (double)(win - 1), &s, &c);
    return (float)(0.54 - 0.46 * c);
}

// ---- per-utterance tables -----------------------------------------------------------------------------------

// The projection is done by v_mfma_f32_4x4x1_16b_f32: sixteen independent products of a 4 x 1 with a 1 x 4
// matrix, added to sixteen 4 x 4 accumulators.  The rows are the four frames of a wavefront, the columns four
// consecutive mel channels (a "quad"); the sixteen blocks run through different stretches of bins.  The bins of
// a quad are contiguous (five bands of them); they are cut into pieces of `steps` bins, a block each, in `rounds`
// times sixteen pieces over all quads.  rounds and steps are chosen per utterance so that the number of
// instructions is least: 24 for 40 channels, where a dense product would need 161.  There is no plan where the bins are
// not in the order of their bands (warp factors outside (0, 2), for which Eq. (1) does not increase and puts the bins at or
// beyond the ends of the band), or where more than a hundred channels meet a strong warp (the nearest to 1 that were
// found: 0.64 and 1.39); the kernel then sums over all bins.
constexpr int kMaxRounds = 4;
constexpr int kMaxQuads = AUG_MAX_MEL / 4;
constexpr int kMaxSteps = 32;                // rounds x steps that the kernel has room for
constexpr unsigned short kNoPiece = 0xffff;
struct MelPlan {
    unsigned char rounds, steps;             // steps: a multiple of 4; rounds = 0: no plan
    unsigned char first_piece[kMaxQuads + 6];     // of quad g; entry n_quads is the number of pieces
    unsigned short piece[16 * kMaxRounds];   // first bin (a multiple of 4) | quad << 10, kNoPiece where unused
};
static_assert(sizeof(MelPlan) % sizeof(float2) == 0, "the plan follows the bins in an array of float2");
constexpr int kPlanEntries = sizeof(MelPlan) / sizeof(float2);

// Where Eq. (1) puts bin k on the mel scale: its band c and the weight w of filter c; band -1 below f_lo and
// n_mel + 1 above f_hi.  `edges`: the n_mel + 2 band edges in Hz.
__device__ inline int mel_band(const MelTableArgs& a, const double* edges, float alpha_u, int k, float& w) {
    const double one_minus = 1.0 - (double)alpha_u;
    double sn, cs;
    sincospi(2.0 * (double)k / (double)a.cfg.nfft, &sn, &cs);
    const double omega = 2.0 * M_PI * (double)k / (double)a.cfg.nfft;
    const double warped = omega + 2.0 * atan(one_minus * sn / (1.0 - one_minus * cs));          // Eq. (1)
    const double f = warped * (double)a.cfg.fs / (2.0 * M_PI);
    w = 0.f;
    if (f < (double)a.cfg.f_lo) return -1;
    if (!(f <= (double)a.cfg.f_hi)) return a.cfg.n_mel + 1;
    // the band from the logarithm in single precision, then by the edges themselves (a bin on an edge has weight 0
    // in the band above it or 1 in the band below, which is the same)
    int c = (int)((2595.f * 0.30102999566f * __log2f(1.f + (float)f * (1.f / 700.f)) - a.mel_lo) * a.inv_step);
    c = c < 0 ? 0 : (c > a.cfg.n_mel ? a.cfg.n_mel : c);
    while (c > 0 && f < edges[c]) --c;
    while (c < a.cfg.n_mel && f >= edges[c + 1]) ++c;
    const double x = (f - edges[c]) / (edges[c + 1] - edges[c]);
    w = (float)(x < 0.0 ? 0.0 : (x > 1.0 ? 1.0 : x));
    return c;
}

// The tables of utterance u, by `threads` threads, five wavefronts or one; all threads of the work group call (u < 0: nothing to
// do).  An entry is a chain of double-precision library calls: with few
// utterances a group has a thread per bin (K = 512) so that the chains run side by side, with many a single wavefront,
// which fills the chip anyway.  The band edges come from the host (a power each: here they were two thirds of the time).
constexpr int kMelTableThreads = 320;
struct MelTableShared {
    double edges[AUG_MAX_MEL + 2];
    short band[2050];
    int first_bin[AUG_MAX_MEL + 8];                   // first bin of band c or higher
    MelPlan plan;
    bool unordered;
};
__device__ inline void mel_table(MelTableShared& sh, const MelTableArgs& a, int stride, int u, int tid, int threads) {
    double* const edges = sh.edges;
    short* const band = sh.band;
    int* const first_bin = sh.first_bin;
    MelPlan& plan = sh.plan;
    bool& unordered = sh.unordered;
    const int bins = u < 0 ? 0 : a.cfg.nfft / 2 + 1, n_mel = a.cfg.n_mel;
    float2* t = a.tab + (size_t)max(u, 0) * stride;
    const float alpha_u = a.alpha[max(u, 0)];
    for (int i = tid; i < n_mel + 2; i += threads) edges[i] = a.edges[i];
    for (int i = tid; i < n_mel + 8; i += threads) first_bin[i] = bins;
    for (int i = tid; i < 16 * kMaxRounds; i += threads) plan.piece[i] = kNoPiece;
    if (tid == 0) unordered = false;
    __syncthreads();
    for (int k = tid; k < bins; k += threads) {
        float w;
        const int c = mel_band(a, edges, alpha_u, k, w);
        band[k] = (short)c;
        t[k] = make_float2(c <= n_mel ? (float)c : -2.f, w);
    }
    __syncthreads();
    for (int k = tid; k < bins; k += threads) {
        const int below = k ? (int)band[k - 1] : -1;
        if (band[k] < below) unordered = true;
        for (int c = below + 1; c <= band[k]; ++c) first_bin[c] = k;
    }
    __syncthreads();
    if (tid < 64 && u >= 0) {
        // a quad's stretch in units of four bins, on lane g
        const int n_quads = (n_mel + 3) / 4, lane = tid;
        int lo4 = 0, len4 = 0;
        if (lane < n_quads) {
            const int lo = first_bin[4 * lane], hi = first_bin[min(4 * lane + 5, n_mel + 1)];
            lo4 = lo / 4;
            len4 = hi > lo ? (hi + 3) / 4 - lo4 : 0;
        }
        // lane i counts the pieces that steps = 4 (i + 1) would give.  A quad without bins owns a piece too, with zero
        // weights: quad g's first sum is then at or behind place 4 g, which the cepstra rely on (see mel_kernel).
        const float inv = 1.f / (float)(lane + 1);
        int count = 0;
        for (int g = 0; g < n_quads; ++g) count += max((int)ceilf((float)__shfl(len4, g, 64) * inv - 1e-4f), 1);
        int best = 1 << 20, rounds = 0, steps4 = 1;
        for (int r = 1; r <= kMaxRounds && !unordered; ++r) {
            const unsigned long long fits = __ballot(count <= 16 * r);
            if (!fits) continue;
            const int s4 = __ffsll((unsigned long long)fits);           // the smallest: lane + 1
            // (a round's own cost: its stores, and more pieces to add up)
            if (4 * r * s4 + 6 * r < best && 4 * r * s4 <= kMaxSteps) {
                best = 4 * r * s4 + 6 * r;
                rounds = r;
                steps4 = s4;
            }
        }
        const int mine = lane < n_quads ? max((len4 + steps4 - 1) / steps4, 1) : 0;
        int incl = mine;
        for (int off = 1; off < 64; off <<= 1) {
            const int up = __shfl_up(incl, off, 64);
            if (lane >= off) incl += up;
        }
        if (lane <= n_quads) plan.first_piece[lane] = (unsigned char)(incl - mine);
        if (rounds)
            for (int i = 0; i < mine; ++i) plan.piece[incl - mine + i] = (unsigned short)(4 * (lo4 + i * steps4) | lane << 10);
        if (lane == 0) {
            plan.rounds = (unsigned char)rounds;
            plan.steps = (unsigned char)(4 * steps4);
        }
    }
    __syncthreads();
    for (int i = tid; i < kPlanEntries && u >= 0; i += threads) t[bins + i] = reinterpret_cast<const float2*>(&plan)[i];
}

// Constants of the sixteen lanes of a frame, [value][lane]: the second pass's twiddles exp(-2 pi i lane m / 256) and,
// for k = lane + 16 i, tangent and cosine of the split's twiddle exp(-i pi k / 256).
constexpr int kMelLanes = 16;                            // lanes per frame
constexpr int kLanePairs = 8;
constexpr int kMelTwFloats = 2 * kTw4Floats;
constexpr int kLaneConsts = kMelTwFloats + 2 * kLanePairs;
__device__ inline void mel_lane_value(int i, float* out) {
    const int lane = i % kMelLanes, f = i / kMelLanes;
    if (f < kMelTwFloats) {                              // the two factor sets of a Tw16Short
        const double x = (double)lane / 128.0;
        const Tw4 w = make_tw4(f < kTw4Floats ? 4.0 * x : x);
        const float v[kTw4Floats] = {w.t1, w.t2, w.t3, w.c1, w.c2, w.r};
        float pick = v[0];
        for (int k = 1; k < kTw4Floats; ++k) pick = f % kTw4Floats == k ? v[k] : pick;
        out[i] = pick;
    } else {
        const int pair = (f - kMelTwFloats) / 2;
        double s, c;
        sincospi(-(double)(lane + kMelLanes * pair) / 256.0, &s, &c);
        out[i] = (f - kMelTwFloats) % 2 ? (float)c : (float)(s / c);
    }
}

// element i of the orthonormal DCT-II rows
__device__ inline float dct_value(int i, int n_mel) {
    const int q = i / n_mel, m = i % n_mel;
    const double s = q == 0 ? sqrt(1.0 / (double)n_mel) : sqrt(2.0 / (double)n_mel);
    return (float)(s * cos(M_PI * (double)q * ((double)m + 0.5) / (double)n_mel));
}

// Everything a front-end call needs before its main kernel, in one launch: the utterances' tables (a group each), the
// batch's packing if its offsets are new, the constants that are not there yet.  Each of these was a launch of its own:
// five of them and two copies took 40 us before a static call's main kernel.
// The rest of the set-up, by groups behind those of the tables.
__device__ inline void mel_setup_rest(const MelSetupArgs& a, int pack_groups, int group) {
    const int threads = (int)blockDim.x;
    if (group < pack_groups) {
        pack_utterances(a.pack, group * threads + (int)threadIdx.x);
        return;
    }
    int i = (group - pack_groups) * threads + (int)threadIdx.x;
    const int n_lanes = a.lane_consts ? kLaneConsts * kMelLanes : 0, n_window = a.window ? a.table.cfg.win : 0;
    const int n_dct = a.dct ? a.table.cfg.n_ceps * a.table.cfg.n_mel : 0;
    if (i < n_lanes) {
        mel_lane_value(i, a.lane_consts);
        return;
    }
    i -= n_lanes;
    if (i < n_window) {
        a.window[i] = hamming(i, a.table.cfg.win);
        return;
    }
    i -= n_window;
    if (i < n_dct) a.dct[i] = dct_value(i, a.table.cfg.n_mel);
}

__global__ __launch_bounds__(kMelTableThreads) void mel_setup_kernel(MelSetupArgs a, int stride, int pack_groups) {
    __shared__ MelTableShared shared;
    const int group = (int)blockIdx.x;
    if (group < a.n_utt) mel_table(shared, a.table, stride, group, (int)threadIdx.x, (int)blockDim.x);
    else mel_setup_rest(a, pack_groups, group - a.n_utt);
}

// The same with the image sum's plan as its first group, which has nothing to do with the others but is a launch of 6 us for
// a few responses and 14 for 1024 otherwise: eight utterances of 1 s with one noise 51.7 -> 46.9 us, 64 of 4 s 132.7 -> 127.2.  The
// plan's groups are large, so one makes the tables of three utterances.
constexpr int kTablesPerGroup = kPlanThreads / kMelTableThreads;
__global__ __launch_bounds__(kPlanThreads) void mel_setup_plan_kernel(MelSetupArgs a, int stride, int pack_groups) {
    __shared__ union { PlanShared plan; MelTableShared table[kTablesPerGroup + 1]; } shared;      // (the last for the threads left over)
    const int table_groups = (a.n_utt + kTablesPerGroup - 1) / kTablesPerGroup, group = (int)blockIdx.x - 1, tid = (int)threadIdx.x;
    if (group < 0) {
        const PlanArgs& p = a.plan;
        plan_all(shared.plan, p.n_rir, p.rooms, p.rir_len, p.fs_over_c, static_cast<Item*>(p.items), static_cast<Item*>(p.unsorted), p.ctrl, p.n_groups);
    } else if (group < table_groups) {
        const int part = tid / kMelTableThreads, u = group * kTablesPerGroup + part;
        mel_table(shared.table[part], a.table, stride, part < kTablesPerGroup && u < a.n_utt ? u : -1, tid - part * kMelTableThreads, kMelTableThreads);
    } else {
        mel_setup_rest(a, pack_groups, group - table_groups);
    }
}

// ---- the front end ------------------------------------------------------------------------------------------

// A frame's buffer in LDS, in floats: the transform's exchange (real parts, then imaginary parts: 16 rows of 17), then,
// over it, the bin powers P[0..259] (three zeros behind the last bin), then the pieces' sums.  Frames of a
// wavefront start sixteen banks apart: its 64 lanes then hit 64 banks in every access of the exchange.
constexpr int kSlotFloats = 272;
static_assert(kSlotFloats * 4 >= 64 * 4 * 4 && kSlotFloats >= 64 * kMaxRounds + 12 && kSlotFloats % 64 == 16, "frame buffer");
constexpr int kBinsPadded = 260;
constexpr int kMelSlots = kMelThreads / kMelLanes;       // frames in flight per work group

// two consecutive samples; only their 4-byte alignment is promised (global loads of two dwords need no more)
struct __attribute__((aligned(4))) SamplePair { float x, y; };
struct __attribute__((aligned(4))) SampleQuad { float x, y, z, w; };
constexpr int kStageLoads = 4;                           // 16-byte loads per lane that stage four frames (1024 samples)
constexpr int kAheadExtra = 3;                           // sources beside the first that are requested a pass ahead
constexpr int kStagedHop = (64 * 4 * kStageLoads - 400) / 3;      // largest hop of a 400-sample window that they cover

// e^power for e > 0 as exp2(power log2 e) on the hardware's base-2 logarithm and exponential (about one
// unit in the last place each; the library's pow spends some 150 instructions on its last bit).  The
// logarithm instruction does not take denormal inputs, so tiny energies are scaled into range first.
__device__ inline float power_law(float e, float power) {
    const bool tiny = e < 0x1p-100f;
    return __builtin_amdgcn_exp2f(power * (__builtin_amdgcn_logf(e * (tiny ? 0x1p+64f : 1.f)) - (tiny ? 64.f : 0.f)));
}

// the value that lane (16 - i) mod 16 of a row of sixteen lanes holds, for lane i: mirrored, then rotated by one
__device__ inline float row_negate(float x) {
    const int m = __builtin_amdgcn_mov_dpp(__float_as_int(x), 0x140, 0xf, 0xf, true);          // row_mirror
    return __int_as_float(__builtin_amdgcn_mov_dpp(m, 0x121, 0xf, 0xf, true));                 // row_ror:1
}

typedef float vec4 __attribute__((ext_vector_type(4)));

// The gain of a source.  Out of line: in the loop over a group's utterances the constants of its exponential were kept in registers all
// along, or spilled for it (16 of them with a window of 400 samples, 36 with others; so 8 or none, 18): with three noises 256 utterances of
// 8 s 151 -> 147 us, of 4 s with a hop of 240 78 -> 72, with a window of 320 115 -> 106.
__device__ __attribute__((noinline)) float source_gain(double e0, double ej, float snr_db) {
    const double e[2] = {e0, ej};
    return snr_gain(e, 0, snr_db);
}

// 4-point DFT of windowed inputs x_m w_m, m < 4 (or 3): the window's factors ride on the additions
template <bool FOUR>
__device__ inline void dft4_windowed(float2& a0, float2& a1, float2& a2, float2& a3, float2 w0, float2 w1, float2 w2, float2 w3) {
    const float2 m0 = make_float2(a0.x * w0.x, a0.y * w0.y), m1 = make_float2(a1.x * w1.x, a1.y * w1.y);
    const float2 s02 = make_float2(fmaf(a2.x, w2.x, m0.x), fmaf(a2.y, w2.y, m0.y));
    const float2 d02 = make_float2(fmaf(-a2.x, w2.x, m0.x), fmaf(-a2.y, w2.y, m0.y));
    const float2 s13 = FOUR ? make_float2(fmaf(a3.x, w3.x, m1.x), fmaf(a3.y, w3.y, m1.y)) : m1;
    const float2 d13 = rot90<false>(FOUR ? make_float2(fmaf(-a3.x, w3.x, m1.x), fmaf(-a3.y, w3.y, m1.y)) : m1);
    a0 = cadd(s02, s13);
    a1 = cadd(d02, d13);
    a2 = csub(s02, s13);
    a3 = csub(d02, d13);
}

// K = 512: a 256-point complex FFT per frame, 16 lanes per frame, 16 frames per pass of the group.
// WIN: the window length when it is known at compile time (the paper's front end uses 400), else 0.  MIX: the signal is
// mixed on the fly.  STAGED: by way of LDS (see the launcher).
//
// A group takes an equal share of the batch's frames (FrameShares), utterance by utterance.
//
// What bounds it: vector issue (655 vector instructions per pass of four frames, 0.97 of one in four cycles on
// 4096 utterances of 8 s, at a clock that falls to 1.8 GHz under them), with the LDS busy half the time.  The first design sent the
// second pass's outputs through
// LDS to pair the bins and summed the bands from step lists there: 770 vector and 126 LDS instructions, a third
// of the LDS's cycles bank conflicts.  Pairing by row permutations, twiddles folded into multiply-adds and the
// projection on the matrix cores, which read every power once and need no vector arithmetic, took that batch from
// 1500 to 1080-1140 us; cepstra from a cosine table in LDS instead of global memory, 256 padded utterances from 350
// to 134 us, and equal shares, set up from loads that are all on their way at once, to 99.  With a mixture it waits for memory:
// 148 us for four sources of 256 utterances of 1-16 s (0.56 GB).
// (The first radix-16 pass on the matrix cores as well measured slower, 1350 us: products of 32-bit
// floats there take the vector units' time.  Requesting a frame's samples a pass ahead without a mixture as well does not fit
// the registers of four wavefronts per SIMD: 4096 utterances 1251 us.)
template <int WIN, bool MIX, bool STAGED>
__global__ __launch_bounds__(kMelThreads, mel_waves(WIN == 400, MIX)) void mel_kernel(MelArgs a, int tab_stride) {
    constexpr int NC = 256;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_wide;                               // some channel has more than four pieces
    const int n_mel = a.cfg.n_mel;
    const int feature = a.cfg.feature;
    const int n_out = feature == AUG_FEAT_MFCC ? a.cfg.n_ceps : n_mel;     // values per output row
    float* const slots = reinterpret_cast<float*>(smem);                     // [kMelSlots][kSlotFloats]
    vec4* const s_weight = reinterpret_cast<vec4*>(slots + kMelSlots * kSlotFloats);       // [kMaxSteps / 4][64]
    int4* const s_pieces = reinterpret_cast<int4*>(s_weight + kMaxSteps / 4 * 64);          // [n_mel]: a channel's sums (see energy)
    float2* const s_pair = reinterpret_cast<float2*>(s_pieces + AUG_MAX_MEL);               // [kLanePairs][kMelLanes]
    float2* const s_window = s_pair + kLanePairs * kMelLanes;                               // [256]
    float* const s_gains = reinterpret_cast<float*>(s_window + NC);                         // [AUG_MAX_NOISE]
    vec4* const s_dct = reinterpret_cast<vec4*>(s_gains + AUG_MAX_NOISE);                             // [n_mel / 4][n_out up to 16s]

    int tid = threadIdx.x, lane = tid & 63, slot = tid / kMelLanes, sub = tid % kMelLanes;
    // Group ids are dealt round-robin to the eight XCDs.  XCD x takes the x-th contiguous eighth of the shares, so that groups
    // that read neighbouring frames of an utterance share an L2.
    const unsigned int xcd = blockIdx.x % 8u, nth = blockIdx.x / 8u;
    const unsigned int item = xcd * (gridDim.x / 8u) + min(xcd, gridDim.x % 8u) + nth;
    int u = a.items[item].x, unit = a.items[item].y;
    const int win = WIN ? WIN : a.cfg.win, hop = a.cfg.hop;
    const float power = a.cfg.power;
    // Window samples, z[n] = w[2n] x[2n] + i w[2n+1] x[2n+1], halved: the even/odd split below then needs no halves of
    // its own.  Lane sub takes n = sub + 16 m.
    constexpr int kRows = WIN ? (WIN + 2 * kMelLanes - 1) / (2 * kMelLanes) : 16;     // rows m with any sample in the window
    static_assert(kRows == 16 || kRows == 13, "the first butterflies are written for 13 or 16 rows");
    const float2 window = make_float2(2 * tid < win ? 0.5f * a.window[2 * tid] : 0.f, 2 * tid + 1 < win ? 0.5f * a.window[2 * tid + 1] : 0.f);
    Tw16Short tw;
    {
        float f[2 * kTw4Floats];
#pragma unroll
        for (int i = 0; i < 2 * kTw4Floats; ++i) f[i] = a.lane_consts[i * kMelLanes + sub];
        tw.outer = Tw4{f[0], f[1], f[2], f[3], f[4], f[5]};
        tw.inner = Tw4{f[6], f[7], f[8], f[9], f[10], f[11]};
    }
    // The window and the tangents and cosines of the split's twiddles are read from LDS where they are used: in registers
    // they would cost a wavefront per SIMD, and a wavefront alone issues a vector instruction only every six cycles
    // where the SIMD could take one every two.
    const int pair = 2 * (tid / kMelLanes % kLanePairs) + kMelTwFloats;
    const float2 pair_consts = make_float2(a.lane_consts[pair * kMelLanes + sub], a.lane_consts[(pair + 1) * kMelLanes + sub]);
    // The group's share: consecutive units of the utterances' frames (see FrameShares), the first of them unit `unit` of utterance u;
    // its part of an utterance is a stretch.
    int left = a.shares.per_group + ((int)item < a.shares.longer ? 1 : 0);
    const int shift = a.shares.shift + kLgUnitFrames;
    // what changes from utterance to utterance
    const float *x, *extra = nullptr;
    int len, n_frames_u;
    [[maybe_unused]] const bool even_win = (win & 1) == 0;
    const float* gains = s_gains;

    // With STAGED the samples of a wavefront's four frames, which overlap, are staged: 16 bytes
    // per lane and load, each sample of each source once, mixed while still in registers, into the frames' buffers and
    // from there into the butterflies.  They are requested a pass ahead, when the registers of the transform are free.  What lies past the
    // utterance's end is not read: frames that do not exist compute something, and it is dropped.
    static_assert(!STAGED || (WIN == 400 && MIX), "staging is written for a mixture and 400 samples");
    constexpr int kMore = MIX ? kAheadExtra : 0;
    const int staged = STAGED ? (3 * hop + 400 + 3) & ~3 : 0;
    // where this lane's i-th four samples lie among those of the frames t_wave .. t_wave + 3 (the last four that exist, if
    // there are no more)
    auto limit = [&](int t_wave) { return min(staged, len - t_wave * hop) - 4; };
    auto place = [&](int i, int most) { return min(4 * lane + 256 * i, most); };
    auto load = [&](SampleQuad (&q)[kStageLoads], const float* src, int t_wave) {
        const char* base = reinterpret_cast<const char*>(src + t_wave * hop);
        const int most = limit(t_wave);
#pragma unroll
        for (int i = 0; i < kStageLoads; ++i) q[i] = *reinterpret_cast<const SampleQuad*>(base + 4u * (uint32_t)place(i, most));
    };
    SampleQuad ahead[kStageLoads], more[kMore ? kMore : 1][kStageLoads];
    // (every register is assigned on every path, so that none is kept for its old value)
    auto request = [&](int t_wave) {
        const bool any = t_wave < n_frames_u;
        if (any) {
            load(ahead, x, t_wave);
        } else {
#pragma unroll
            for (int i = 0; i < kStageLoads; ++i) ahead[i] = SampleQuad{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int j = 0; j < kMore; ++j) {
            if (any && j < a.n_extra) {
                load(more[j], extra + (size_t)j * a.extra_stride, t_wave);
            } else {
#pragma unroll
                for (int i = 0; i < kStageLoads; ++i) more[j][i] = SampleQuad{0.f, 0.f, 0.f, 0.f};
            }
        }
    };

    // What the next stretch needs, all loads side by side: the utterance's table and plan, from which the weights are formed in LDS
    // (where the frames' buffers will be), its energies, a lane of the last wavefront per gain, and the first samples.
    float2* const s_tab = reinterpret_cast<float2*>(slots);                                 // [NC + 1 + kPlanEntries]
    static_assert(NC + 1 + kPlanEntries <= 2 * kMelThreads && sizeof(float2) * 2 * kMelThreads <= sizeof(float) * kMelSlots * kSlotFloats, "the table in LDS");
    float2 tab0, tab1;
    double energies[2];
    float snr;
    int units, units_u, frame_units_u, wave_first;
    int64_t rows_u;
    float* feats;
    auto has_gain = [&] { return MIX && tid >= kMelThreads - 64 && tid - (kMelThreads - 64) < a.n_extra; };
    auto begin_stretch = [&] {
        // The utterance owns rows of the output; the first n_frames_u hold its frames and the rest, if the caller reserved
        // more (padded batches), are set to zero.  (Utterances are shorter than 2^30 samples: checked on the host.)
        const int64_t start = a.offsets[u], first_row = a.frame_offsets[u];
        rows_u = a.frame_offsets[u + 1] - first_row;
        len = (int)(a.offsets[u + 1] - start);
        const float2* g_tab = a.mel_tab + (size_t)u * tab_stride;
        tab0 = g_tab[tid];
        tab1 = g_tab[min(tid + kMelThreads, NC + kPlanEntries)];
        if (has_gain()) {
            const double* const e = a.energy + (size_t)u * (a.n_extra + 1);
            energies[0] = e[0];
            energies[1] = e[1 + tid - (kMelThreads - 64)];
            snr = a.snr_db[(size_t)u * a.n_extra + tid - (kMelThreads - 64)];
        } else {
            energies[0] = energies[1] = 0.0;
            snr = 0.f;
        }
        x = a.wave + start;
        if (MIX) extra = a.extra + start;
        feats = a.feats + first_row * n_out;
        n_frames_u = len >= win ? 1 + (len - win) / hop : 0;
        frame_units_u = (n_frames_u + ((1 << shift) - 1)) >> shift;
        units_u = max(frame_units_u + (int)((rows_u - n_frames_u) >> (a.shares.shift + a.shares.lg_rows)), 1);      // (see frame_units)
        units = min(left, units_u - unit);
        // (a stretch of rows without frames only: past every frame)
        wave_first = __builtin_amdgcn_readfirstlane(unit < frame_units_u ? (unit << shift) + (slot & ~3) : 0x7fffffff);
        if (STAGED) request(wave_first);
    };
    begin_stretch();
    s_window[tid] = window;
    if (tid < kLanePairs * kMelLanes) s_pair[tid] = pair_consts;
    const int q_pad = (n_out + kMelLanes - 1) & ~(kMelLanes - 1);
    if (feature == AUG_FEAT_MFCC) {                       // cosine rows by fours of channels, zero past the last
        for (int e = tid; e < (n_mel + 3) / 4 * q_pad; e += kMelThreads) {
            const int m4 = e / q_pad, q = e - m4 * q_pad;
            vec4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (q < n_out && 4 * m4 + i < n_mel) d[i] = a.dct[q * n_mel + 4 * m4 + i];
            s_dct[e] = d;
        }
    }
    for (;;) {
    // (opaque: addresses are formed anew for every stretch, kept from one to the next they do not fit the registers)
    asm volatile("" : "+v"(tid));
    lane = tid & 63;
    slot = tid / kMelLanes;
    sub = tid % kMelLanes;
    float* const buf = slots + slot * kSlotFloats;       // the frame's buffer
    float* const wave_buf = slots + (slot & ~3) * kSlotFloats;     // the four frames of this wavefront
    const float2* const g_tab = a.mel_tab + (size_t)u * tab_stride;
    if (tid == 0) s_wide = 0;
    s_tab[tid] = tab0;
    if (tid + kMelThreads < NC + 1 + kPlanEntries) s_tab[tid + kMelThreads] = tab1;
    // this stretch's part of the rows without frames
    if (const int64_t spare = rows_u - n_frames_u; spare > 0) {
        const int64_t each = spare / units_u, more_rows = spare - each * units_u;
        const int64_t from = n_frames_u + each * unit + min((int64_t)unit, more_rows), to = from + each * units + max(min(more_rows - unit, (int64_t)units), (int64_t)0);
        for (int64_t i = from * n_out + tid; i < to * n_out; i += kMelThreads) feats[i] = 0.f;
    }
    __syncthreads();
    // from the plan, the weights in the order in which the lanes use them
    const MelPlan* plan = reinterpret_cast<const MelPlan*>(s_tab + (NC + 1));
    const int rounds = __builtin_amdgcn_readfirstlane(plan->rounds), steps = __builtin_amdgcn_readfirstlane(plan->steps);
    for (int e = tid; e < rounds * (steps / 4) * 64; e += kMelThreads) {
        const int l = e & 63, q = e >> 6, s4 = steps / 4, r = (q >= s4) + (q >= 2 * s4) + (q >= 3 * s4), s0 = 4 * (q - r * s4);
        static_assert(kMaxRounds == 4, "the round of a step");
        const int piece = plan->piece[16 * r + (l >> 2)];
        vec4 w = {0.f, 0.f, 0.f, 0.f};
        if (piece != kNoPiece) {
            const int begin = piece & 1023, m = 4 * (piece >> 10) + (l & 3);
            const int k0 = min(begin, kBinsPadded - steps) + s0;             // (a piece at the end starts earlier, to stay inside)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int k = k0 + i;
                const float2 cw = s_tab[min(k, NC)];
                const int c = (int)cw.x;
                const float weight = c == m ? cw.y : (c == m + 1 ? 1.f - cw.y : 0.f);
                w[i] = k >= begin && k <= NC ? weight : 0.f;
            }
        }
        s_weight[q * 64 + l] = w;
    }
    for (int m = tid; m < n_mel; m += kMelThreads) {
        const int p0 = plan->first_piece[m / 4], p1 = plan->first_piece[m / 4 + 1];
        const int n = p1 - p0;
        s_pieces[m] = make_int4(4 * p0 + (m & 3), n > 1 ? -1 : 0, n > 2 ? -1 : 0, n > 3 ? (n > 4 ? n : -1) : 0);
        if (n > 4) s_wide = 1;
    }
    if (has_gain()) s_gains[tid - (kMelThreads - 64)] = source_gain(energies[0], energies[1], snr);
    // where this lane's block starts to read powers, per round
    int at[kMaxRounds];
#pragma unroll
    for (int r = 0; r < kMaxRounds; ++r) {
        const int piece = r < rounds ? plan->piece[16 * r + (lane >> 2)] : kNoPiece;
        at[r] = (lane & 3) * kSlotFloats + (piece == kNoPiece ? 0 : min(piece & 1023, kBinsPadded - steps));
    }
    __syncthreads();

    const bool wide = __builtin_amdgcn_readfirstlane(s_wide) != 0;
    const int passes = max(min(units, frame_units_u - unit), 0) << (shift - kLgUnitFrames);
    for (int it = 0; it < passes; ++it) {
        const int t_wave = wave_first + it * kMelSlots, t = t_wave + (slot & 3);
        if (t_wave >= n_frames_u) break;                  // (no barrier before the stretch's end)
        const bool live = t < n_frames_u;
        float2 v[16];
        // With MIX the analysed signal is formed here, in source order: x + sum_j gains[j] extra_j.
        if constexpr (STAGED) {
            auto add = [&](const SampleQuad (&e)[kStageLoads], float gain) {
#pragma unroll
                for (int i = 0; i < kStageLoads; ++i) {
                    ahead[i].x += gain * e[i].x;
                    ahead[i].y += gain * e[i].y;
                    ahead[i].z += gain * e[i].z;
                    ahead[i].w += gain * e[i].w;
                }
            };
#pragma unroll
            for (int j = 0; j < kMore; ++j)
                if (j < a.n_extra) add(more[j], gains[j]);
            const int most = limit(t_wave);
            if (MIX)
                for (int j = kMore; j < a.n_extra; ++j) {
                    load(more[0], extra + (size_t)j * a.extra_stride, t_wave);
                    add(more[0], gains[j]);
                }
#pragma unroll
            for (int i = 0; i < kStageLoads; ++i) {
                float* to = wave_buf + place(i, most);
                if (most == staged - 4) *reinterpret_cast<vec4*>(to) = vec4{ahead[i].x, ahead[i].y, ahead[i].z, ahead[i].w};
                else *reinterpret_cast<SampleQuad*>(to) = ahead[i];
            }
            fft_sync();
            const float2* mine = reinterpret_cast<const float2*>(wave_buf + (slot & 3) * hop);      // (the hop is even)
#pragma unroll
            for (int i = 0; i < kRows; ++i) v[i] = mine[min(sub + kMelLanes * i, WIN / 2 - 1)];    // (past the window: times zero)
            fft_sync();
        } else {
            // Loads are unconditional: a slot past the utterance's last frame recomputes that last frame (its result is
            // dropped) and inputs past the window are read from the frame's last samples and meet a zero window weight.
            const int x0 = (live ? t : n_frames_u - 1) * hop;
            // (opaque in the general kernel, whose clamped positions would otherwise all be kept in registers)
            int at_sub = sub;
            if (!WIN) asm volatile("" : "+v"(at_sub));
            if (even_win) {                                   // one 8-byte load per complex input
#pragma unroll
                for (int i = 0; i < kRows; ++i) {
                    const int i0 = min(2 * (at_sub + kMelLanes * i), win - 2);
                    const SamplePair s2 = *reinterpret_cast<const SamplePair*>(x + (x0 + i0));
                    v[i] = make_float2(s2.x, s2.y);
                }
                if (MIX) {
                    for (int j = 0; j < a.n_extra; ++j) {
                        const float g = gains[j];
                        const float* xj = extra + (size_t)j * a.extra_stride;
                        // all loads of a source are issued before the first of them is used (the
                        // scheduler may otherwise pair every load with its wait to save registers)
                        SamplePair s2[kRows];
#pragma unroll
                        for (int i = 0; i < kRows; ++i) {
                            const int i0 = min(2 * (at_sub + kMelLanes * i), win - 2);
                            s2[i] = *reinterpret_cast<const SamplePair*>(xj + (x0 + i0));
                        }
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int i = 0; i < kRows; ++i) {
                            v[i].x += g * s2[i].x;
                            v[i].y += g * s2[i].y;
                        }
                    }
                }
            } else {
#pragma unroll
                for (int i = 0; i < kRows; ++i) {
                    const int i0 = 2 * (at_sub + kMelLanes * i);
                    v[i] = make_float2(x[x0 + min(i0, win - 1)], x[x0 + min(i0 + 1, win - 1)]);
                }
                if (MIX) {
                    for (int j = 0; j < a.n_extra; ++j) {
                        const float g = gains[j];
                        const float* xj = extra + (size_t)j * a.extra_stride;
#pragma unroll
                        for (int i = 0; i < kRows; ++i) {
                            const int i0 = 2 * (at_sub + kMelLanes * i);
                            v[i].x += g * xj[x0 + min(i0, win - 1)];
                            v[i].y += g * xj[x0 + min(i0 + 1, win - 1)];
                        }
                    }
                }
            }
        }
        // 256 = 16 x 16: first pass without twiddles (inputs past the window are zero), exchange through LDS,
        // second pass with this lane's fixed twiddles
        float2 wnd[kRows];
#pragma unroll
        for (int m = 0; m < kRows; ++m) wnd[m] = s_window[sub + kMelLanes * m];
        if constexpr (kRows == 16) {
#pragma unroll
            for (int m = 0; m < 4; ++m)
                dft4_windowed<true>(v[m], v[m + 4], v[m + 8], v[m + 12], wnd[m], wnd[m + 4], wnd[m + 8], wnd[m + 12]);
        } else {
            dft4_windowed<true>(v[0], v[4], v[8], v[12], wnd[0], wnd[4], wnd[8], wnd[12]);
#pragma unroll
            for (int m = 1; m < 4; ++m)
                dft4_windowed<false>(v[m], v[m + 4], v[m + 8], v[m + 12], wnd[m], wnd[m + 4], wnd[m + 8], wnd[m + 8]);
        }
        dft16_inner<false, false>(v, 1.f, 1.f, 1.f);
        dft16_transpose(v);
        {
            // lane sub's outputs are elements 16 sub + r, its next inputs sub + 16 m; element i lives at i + i / 16
            float* const to = buf + 17 * sub;
            const float* const from = buf + sub;
#pragma unroll
            for (int r = 0; r < 16; ++r) to[r] = v[r].x;
            fft_sync();                   // a frame's 16 lanes share a wavefront
#pragma unroll
            for (int m = 0; m < 16; ++m) v[m].x = from[17 * m];
            fft_sync();
#pragma unroll
            for (int r = 0; r < 16; ++r) to[r] = v[r].y;
            fft_sync();
#pragma unroll
            for (int m = 0; m < 16; ++m) v[m].y = from[17 * m];
            fft_sync();
        }
        dft16_twiddled<false>(v, tw);

        // v[i] = Z[k], k = sub + 16 i.  Bin powers, two at a time: with A = Z[k], B = conj Z[N-k] (halved inputs),
        // E = A + B, O = -i (A - B) and w = exp(-i pi k / N):  X[k] = E + w O and conj(X[N-k]) = E - w O.  Z[N-k] is
        // v[15 - i] of lane 16 - sub (lane 0 finds its own in v[16 - i]).
#pragma unroll
        for (int i = 0; i < kLanePairs; ++i) {
            const float2 other = sub == 0 ? v[(16 - i) & 15] : v[15 - i];
            const float2 B = make_float2(row_negate(other.x), -row_negate(other.y));
            const float2 E = cadd(v[i], B), d = csub(v[i], B);
            const float2 tc = s_pair[i * kMelLanes + sub];
            const float2 wO = tilt<false>(make_float2(d.y, -d.x), tc.x);                 // awaits the cosine
            // sums first, then squares: a weak bin next to a strong mirror bin keeps its relative accuracy
            const float2 Xk = cfma(tc.y, wO, E), Xn = cfma(-tc.y, wO, E);
            buf[sub + kMelLanes * i] = fmaf(Xk.x, Xk.x, Xk.y * Xk.y);
            buf[NC - (sub + kMelLanes * i)] = fmaf(Xn.x, Xn.x, Xn.y * Xn.y);             // k = 0: P[N] (from Z[0] too)
        }
        // bin N/2 is its own partner; the three places behind bin N meet zero weights and must be finite
        if (sub < 4) buf[sub == 0 ? NC / 2 : NC + sub] = sub == 0 ? 4.f * fmaf(v[8].x, v[8].x, v[8].y * v[8].y) : 0.f;
        if (STAGED) request(it + 1 < passes ? t_wave + kMelSlots : 0x7fffffff);
        fft_sync();

        // pieces of the projection: row i of a block is frame i of the wavefront, column j channel 4 quad + j
        if (rounds) {
            // (opaque: comparisons with them are made where they are used, not kept in scalar registers all along)
            int n_rounds = rounds, n_steps = steps;
            asm volatile("" : "+s"(n_rounds), "+s"(n_steps));
            vec4 sums[kMaxRounds];
            const vec4* wq = s_weight + lane;
#pragma unroll
            for (int r = 0; r < kMaxRounds; ++r) {
                if (r >= n_rounds) break;
                const vec4* pq = reinterpret_cast<const vec4*>(wave_buf + at[r]);
                vec4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int q = 0; q < kMaxSteps / 4; ++q) {
                    if (4 * q >= n_steps) break;
                    const vec4 p = pq[q], w = wq[64 * q];
                    acc0 = __builtin_amdgcn_mfma_f32_4x4x1f32(p[0], w[0], acc0, 0, 0, 0);
                    acc1 = __builtin_amdgcn_mfma_f32_4x4x1f32(p[1], w[1], acc1, 0, 0, 0);
                    acc0 = __builtin_amdgcn_mfma_f32_4x4x1f32(p[2], w[2], acc0, 0, 0, 0);
                    acc1 = __builtin_amdgcn_mfma_f32_4x4x1f32(p[3], w[3], acc1, 0, 0, 0);
                }
                wq += 64 * (n_steps / 4);
                sums[r] = acc0 + acc1;
            }
            fft_sync();                   // the powers are read before the sums take their place
#pragma unroll
            for (int r = 0; r < kMaxRounds; ++r) {
                if (r >= n_rounds) break;
                float* to = wave_buf + 64 * r + lane;
#pragma unroll
                for (int i = 0; i < 4; ++i) to[i * kSlotFloats] = sums[r][i];
            }
            fft_sync();
        }
        // energy of channel m: the sum of its pieces, without a plan a plain sum over all bins
        auto energy = [&](int m) {
            float e = 0.f;
            if (rounds) {
                // (the first four at once, the few pieces of a wider quad after them; what lies behind a quad's last piece
                // is read and masked out)
                const int4 pc = s_pieces[m];
                const float* from = buf + pc.x;
                auto masked = [](float v, int mask) { return __int_as_float(__float_as_int(v) & mask); };
                const float e0 = from[0], e1 = from[4], e2 = from[8], e3 = from[12];
                e = (e0 + masked(e1, pc.y)) + (masked(e2, pc.z) + masked(e3, wide && pc.w ? -1 : pc.w));
                if (wide)
                    for (int i = 4; i < pc.w; ++i) e += from[4 * i];
            } else {
                for (int k = 0; k <= NC; ++k) {
                    const float2 cw = g_tab[k];
                    if ((int)cw.x == m) e = fmaf(cw.y, buf[k], e);
                    else if ((int)cw.x == m + 1) e = fmaf(1.f - cw.y, buf[k], e);
                }
            }
            return e;
        };
        // For cepstra the log energies go over the sums: channel m at place m, which is at or before its own sums (every
        // quad owns a piece, so those of quad g begin at 4 g or later), so what a later channel still has to read is not
        // overwritten.
        const bool to_lds = feature == AUG_FEAT_MFCC && rounds;
        const int m_end = to_lds ? (n_mel + 3) & ~3 : feature == AUG_FEAT_MFCC ? 0 : n_mel;
#pragma unroll 1
        for (int m = sub; m < m_end; m += kMelLanes) {
            const float e = m < n_mel ? energy(m) : 0.f;
            if (feature == AUG_FEAT_POWER_LAW) {
                if (live) feats[(int64_t)t * n_mel + m] = e > 0.f ? power_law(e, power) : 0.f;
            } else {
                const float le = m < n_mel ? logf(fmaxf(e, a.cfg.log_floor)) : 0.f;
                if (to_lds) {
                    fft_sync();
                    buf[m] = le;
                } else if (live) {
                    feats[(int64_t)t * n_mel + m] = le;
                }
            }
        }
        if (feature == AUG_FEAT_MFCC) {
            // every lane takes the dot products of its coefficients with the whole vector, four channels at a time
            fft_sync();
            const vec4* lq = reinterpret_cast<const vec4*>(buf);
#pragma unroll 1
            for (int q = sub; q < q_pad; q += kMelLanes) {
                vec4 acc = {0.f, 0.f, 0.f, 0.f};
                if (to_lds) {
                    for (int m4 = 0; m4 < m_end / 4; ++m4) {
                        const vec4 l = lq[m4], d = s_dct[m4 * q_pad + q];
#pragma unroll
                        for (int i = 0; i < 4; ++i) acc[i] = fmaf(l[i], d[i], acc[i]);
                    }
                } else {
                    for (int m = 0; m < n_mel; ++m) acc[0] = fmaf(logf(fmaxf(energy(m), a.cfg.log_floor)), s_dct[(m / 4) * q_pad + q][m & 3], acc[0]);
                }
                if (live && q < n_out) feats[(int64_t)t * n_out + q] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
            }
        }
        fft_sync();                       // everything is read before the next frame's exchange
    }
    left -= units;
    if (left == 0) break;
    do ++u;
    while (a.frame_offsets[u + 1] == a.frame_offsets[u]);
    unit = 0;
    begin_stretch();
    __syncthreads();                      // every wavefront is done with the tables and its frames
    }
}

}  // namespace

int mel_lane_floats() { return kLaneConsts * kMelLanes; }

int mel_table_stride(int nfft) { return nfft / 2 + 1 + kPlanEntries; }   // (c, w) per bin, then the plan

void mel_edges(const aug_frontend_cfg& cfg, MelTableArgs& a) {
    const double mel_lo = 2595.0 * log10(1.0 + (double)cfg.f_lo / 700.0);
    const double mel_hi = 2595.0 * log10(1.0 + (double)cfg.f_hi / 700.0);
    const double step = (mel_hi - mel_lo) / (double)(cfg.n_mel + 1);
    for (int c = 0; c < cfg.n_mel + 2; ++c) a.edges[c] = 700.0 * (pow(10.0, (mel_lo + c * step) / 2595.0) - 1.0);
    a.mel_lo = (float)mel_lo;
    a.inv_step = (float)(1.0 / step);
    a.cfg = cfg;
}

hipError_t launch_mel_setup(hipStream_t s, const MelSetupArgs& a) {
    const bool plan = a.plan.n_rir > 0;
    const int threads = plan ? kPlanThreads : a.n_utt >= 1024 ? 64 : kMelTableThreads;
    const int64_t pack = a.pack.n_utt > 0 ? (pack_threads(a.pack) + threads - 1) / threads : 0;
    const int64_t consts = (a.lane_consts ? kLaneConsts * kMelLanes : 0) + (a.window ? a.table.cfg.win : 0) +
                           (a.dct ? a.table.cfg.n_ceps * a.table.cfg.n_mel : 0);
    const int64_t groups = (plan ? (a.n_utt + kTablesPerGroup - 1) / kTablesPerGroup : a.n_utt) + pack + (consts + threads - 1) / threads;
    if (plan) {
        mel_setup_plan_kernel<<<dim3((unsigned)groups + 1), dim3(threads), 0, s>>>(a, mel_table_stride(a.table.cfg.nfft), (int)pack);
        return hipGetLastError();
    }
    if (groups <= 0) return hipSuccess;
    mel_setup_kernel<<<dim3((unsigned)groups), dim3(threads), 0, s>>>(a, mel_table_stride(a.table.cfg.nfft), (int)pack);
    return hipGetLastError();
}

hipError_t launch_mel(hipStream_t s, const MelArgs& a) {
    if (a.n_items <= 0) return hipSuccess;
    if (a.cfg.nfft != 512) return hipErrorInvalidValue;
    constexpr int NC = 256;
    static_assert(kMelThreads == NC, "a thread per pair of window samples");
    static_assert(kMelThreads == 4 * 64, "a group is a wavefront on every SIMD (mel_slots)");
    static_assert(kMelSlots == kUnitFrames && sizeof(float) * kSlotFloats == 4 * 272 && sizeof(vec4) * (kMaxSteps / 4) == 16 * 8 &&
                  kLanePairs * kMelLanes == 8 * 16 && sizeof(int4) == 16, "mel_lds_bytes");
    const size_t lds = mel_lds_bytes(a.cfg);
    const bool mix = a.n_extra > 0;
    // A window of 400 samples has kernels of its own for every hop; its mixtures are staged where the loads cover four frames
    // and the samples of a frame start on a pair.  (With hops of 161 and 240 the general kernel, 16 rows of inputs instead of
    // 13 and without a mixture a wavefront per SIMD fewer, took 334 and 236 us where these take 287 and 205 for 1024 utterances of 8 s,
    // and 105 and 80 us where these take 93 and 72 for a mixture of 256 x 4 s with three noises.)
    const bool staged = a.cfg.hop <= kStagedHop && a.cfg.hop % 2 == 0;
    auto k = a.cfg.win == 400 ? (!mix ? &mel_kernel<400, false, false> : staged ? &mel_kernel<400, true, true> : &mel_kernel<400, true, false>)
                              : (mix ? &mel_kernel<0, true, false> : &mel_kernel<0, false, false>);
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    // (launched by address, not called through the pointer: see the convolution's launcher)
    MelArgs by_value = a;
    int tab_stride = mel_table_stride(a.cfg.nfft);
    void* args[] = {&by_value, &tab_stride};
    return hipLaunchKernel(reinterpret_cast<const void*>(k), dim3((unsigned)a.n_items), dim3(kMelThreads), args, lds, s);
}

}  // namespace aug
