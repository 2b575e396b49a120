// Vocal tract length perturbation on the waveform (Sec. 2.3): the utterance is analysed in short
// frames, each frame's spectrum is moved along the frequency axis by the bilinear rule of Eq. (1)
// with the utterance's warp factor, and the frames are overlap-added back into a waveform that the
// acoustic simulator then takes as its input.
//
// What the paper leaves to a cited work is fixed as follows.  Frames of 800 samples (50 ms, the best
// window length of Sec. 4, Table 2) under the periodic Hann window, every 400 samples, frame t centred on sample
// 400 t, so that each sample lies in two frames whose weights add up to one.  The frame is laid out
// around time zero of a 2048-point transform.  Output bin k' reads the input spectrum, by linear
// interpolation between the two nearest bins, at the frequency that Eq. (1) maps onto k':
//     omega = omega' - 2 atan(a sin omega' / (1 + a cos omega')),  a = 1 - alpha, omega' = 2 pi k' / 2048.
// All 2048 samples of the inverse transform are added at the frame's position.  alpha = 1 returns the input.
//
// One wavefront per frame.  The 2048-point real transform is a 1024-point complex one of the even/odd
// packing in place (fft_inplace.h with steps of 16, 16 and 4), done by 64 lanes with 16 values each in LDS (wave-level fences
// only); the frame's samples go from HBM straight into the first butterflies' registers.  The last step's butterflies come in
// mirrored pairs, so the real spectrum is formed in registers and only the warp itself, which gathers from it, needs it in
// LDS; the warped spectrum goes from registers into the inverse's first step.
// A wavefront works through a run of consecutive frames and overlap-adds them in a sliding window of 2048 samples in its
// registers: a lane owns every 64th pair of output samples, which moves by eight columns of the transform from frame to
// frame.  The 400 samples that leave the window after each frame are written out.  Only the ends of
// a run, where the frames of the neighbouring runs also land, go to HBM with float atomics; measured on
// the chip, sending every sample through HBM atomics more than doubled the kernel's time.
// Per utterance a table holds, for every output bin, the lower source bin and the interpolation weight;
// both come from fp64 arithmetic so that the choice of the bin pair matches a double-precision evaluation.
//
// What bounds it: vector issue, with room for three wavefronts per SIMD (the window's 32
// registers, factors that do not differ from frame to frame in LDS, 53.7 KB for four wavefronts), and in batches that do not
// fill the chip many times the last round of groups: 256 utterances of 1-16 s are 1.95 rounds of 768 groups.  On that batch the whole call takes
// 303 us, the vector units busy 0.87 of the time with 1480 instructions per frame, set-up and the ends of runs included, and 128 of the LDS,
// where transforms in natural order, with the spectrum's split, the product and the window (8 KB) in LDS and so two
// wavefronts per SIMD, took 480, busy 0.52 of the time with 1440 and 217: the third wavefront is what it gains by; 768 utterances of 640 frames take 2.6 ns a frame.
// Runs of at most 10, 12, 14, 20, 24 and 32 frames: 407, 312, 331, 389, 318, 343 us, by how full the last round is; plain
// stores instead of the atomics would give 14 us, cheaper constants at a group's start nothing.

#include "aug_internal.h"
#include "fft_inplace.h"

namespace aug {
namespace {

constexpr int kWin = 800, kHop = 400, kFft = 2048;
constexpr int kN = kFft / 2;                       // complex transform length
constexpr int kBins = kN + 1;                      // real-spectrum bins 0..1024
constexpr int kWaves = 4, kThreads = 64 * kWaves;
constexpr int kRun = 16;                           // consecutive frames overlap-added by one wavefront, at most
constexpr int kMinRun = 8;                         // and at least: with runs of six or more no sample gets more than two shares
constexpr int kFramesPerGroup = kRun * kWaves;
using T1024 = InPlace<kN>;
constexpr int kSlot = T1024::kPadded;              // a wavefront's transform buffer; the real spectrum, of kBins, lies in it too
static_assert(T1024::T == 64 && kSlot >= kBins && kSlot % 2 == 0, "a transform per wavefront");
constexpr int kReach = kFft / 2;                   // a frame adds to [centre - kReach, centre + kReach)

// two consecutive output samples; only their 4-byte alignment is promised
struct __attribute__((aligned(4))) SamplePair { float x, y; };

// One thread per (utterance, output bin): lower source bin j (as a float, exact) and weight f of bin j + 1.
__global__ void vtlp_table_kernel(int n_utt, const float* __restrict__ alpha, float2* __restrict__ tab) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_utt * kBins) return;
    const int u = i / kBins, k = i % kBins;
    const double a = 1.0 - (double)alpha[u];
    const double w = M_PI * (double)k / (double)kN;
    const double src = w - 2.0 * atan(a * sin(w) / (1.0 + a * cos(w)));
    // fmin/fmax drop a NaN operand, so a warp factor that is not a number cannot produce an index out of range
    const double kappa = fmin(fmax(src * (double)kN / M_PI, 0.0), (double)kN);
    int j = (int)floor(kappa);
    if (j > kN - 1) j = kN - 1;
    tab[i] = make_float2((float)j, (float)(kappa - (double)j));
}

__device__ inline int frame_count(int len) { return len > 0 ? (len - 1) / kHop + 2 : 0; }

// How an utterance's frames are shared: groups of kWaves runs, `run` frames each (the last ones fewer or none).
struct Share { int n_groups, run; };
__device__ inline Share share_frames(int n_frames) {
    const int n_groups = (n_frames + kFramesPerGroup - 1) / kFramesPerGroup;
    return Share{n_groups, max((n_frames + n_groups * kWaves - 1) / max(n_groups * kWaves, 1), kMinRun)};
}

// Zeros where runs meet: the samples that two of them add to.  All others are stored by the kernel below.  (Clearing the
// whole output cost a write of it; this is a quarter.)  Same grid as below.
__global__ __launch_bounds__(kThreads) void vtlp_clear_kernel(const int64_t* __restrict__ offsets, float* __restrict__ out) {
    const int u = blockIdx.y;
    const int64_t start = offsets[u];
    const int len = (int)(offsets[u + 1] - start);
    const int n_frames = frame_count(len);
    const Share share = share_frames(n_frames);
    if ((int)blockIdx.x >= share.n_groups) return;
    float* const y = out + start;
    for (int w = 0; w < kWaves; ++w) {
        const int t = ((int)blockIdx.x * kWaves + w) * share.run;       // first frame of a run
        if (t == 0 || t >= n_frames) continue;
        const int lo = max(t * kHop - kReach, 0), hi = min(t * kHop + (kReach - kHop), len);
        for (int p = lo + (int)threadIdx.x; p < hi; p += kThreads) y[p] = 0.f;
    }
}

// Value of output bin q of the warped spectrum; X is in natural order in buf.  The table in LDS holds the place of the
// lower source bin in bytes and the weight of the one behind it.
__device__ inline float2 warped_bin(const float2* buf, const float2* s_tab, int q) {
    const float2 e = s_tab[q];
    const float2* const at = reinterpret_cast<const float2*>(reinterpret_cast<const char*>(buf) + __float_as_int(e.x));
    const float2 lo = at[0], hi = at[1];
    return make_float2(fmaf(e.y, hi.x - lo.x, lo.x), fmaf(e.y, hi.y - lo.y, lo.y));
}

__device__ inline Tw4 tw4_of(const float2* __restrict__ tw, int k) {       // w = tw[k]
    float c[3], t[3];
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        const float2 w = tw[(m + 1) * k];
        c[m] = fabsf(w.x) < 0x1p-40f ? copysignf(0x1p-40f, w.x) : w.x;
        t[m] = w.y / c[m];
    }
    return Tw4{t[0], t[1], t[2], c[0], c[1], c[2] / c[0]};
}
__device__ inline Tw16Short tw16_of(const float2* __restrict__ tw, int k) { return Tw16Short{tw4_of(tw, 4 * k), tw4_of(tw, k)}; }

// Forward 16-point DFT of values of which those in places 4 .. 11 are zero.
__device__ inline void dft16_outer_inputs(float2 (&v)[16]) {
#pragma unroll
    for (int m2 = 0; m2 < 4; ++m2) {
        const float2 a = v[m2], b = v[m2 + 12], ib = make_float2(-b.y, b.x);
        v[m2] = cadd(a, b);
        v[m2 + 4] = cadd(a, ib);
        v[m2 + 8] = csub(a, b);
        v[m2 + 12] = csub(a, ib);
    }
    dft16_inner<false, false>(v, 1.f, 1.f, 1.f);
    dft16_transpose(v);
}

// Factors kept in LDS, three float4 each: of the inverse's last step by column, of step B by row, of the inverse's step B by t.
constexpr int kOfB = 64, kOfInverseB = kOfB + 16, kFactors = kOfInverseB + 4;
__device__ inline Tw16Short read_factors(const float4* f) {
    const float4 f0 = f[0], f1 = f[1], f2 = f[2];
    return Tw16Short{{f0.x, f0.y, f0.z, f0.w, f1.x, f1.y}, {f1.z, f1.w, f2.x, f2.y, f2.z, f2.w}};
}

// Step B of the forward transform or its counterpart of the inverse: the sixteen values t + 4 m of row k1, lane 4 k1 + t
template <bool INV>
__device__ inline void step_b(float2* buf, const float4* factors, int lane) {
    const Tw16Short w = read_factors(factors);
    float2* const at = buf + T1024::pad(T1024::M) * (lane >> 2) + (lane & 3);
    float2 v[16];
#pragma unroll
    for (int m = 0; m < 16; ++m) v[m] = at[T1024::pad(4 * m)];
    dft16_twiddled<INV>(v, w);
#pragma unroll
    for (int m = 0; m < 16; ++m) at[T1024::pad(4 * m)] = v[m];
}

// grid: (frame groups of the longest utterance, utterances); `out` as vtlp_clear_kernel leaves it
__global__ __launch_bounds__(kThreads, 3) void vtlp_resynth_kernel(
    const int64_t* __restrict__ offsets, const float* __restrict__ wave, const float2* __restrict__ tab,
    const float2* __restrict__ tw, float* __restrict__ out) {
    extern __shared__ __align__(16) float2 smem[];
    constexpr int RD = T1024::RD;
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;
    const int u = blockIdx.y;
    const int64_t start = offsets[u];
    const int len = (int)(offsets[u + 1] - start);      // utterances are shorter than 2^30 samples (checked on the host)
    const int n_frames = frame_count(len);
    const Share share = share_frames(n_frames);
    if ((int)blockIdx.x >= share.n_groups) return;           // the whole group leaves together
    float2* const buf = smem + wv * kSlot;
    float4* const s_window = reinterpret_cast<float4*>(smem + kWaves * kSlot);       // [3][64]: of inputs 2 i and 2 i + 1 of a lane
    float4* const s_factors = s_window + 3 * 64;                                     // [84][3], see read_factors
    float4* const s_step_d = s_factors + 3 * kFactors;                               // [3][64]
    float2* const s_tab = reinterpret_cast<float2*>(s_step_d + 3 * 64);              // [kBins + 1]
    float2* const s_window6 = s_tab + kBins + 1;                                     // [64]: of input 6
    for (int k = tid; k < kBins; k += kThreads) {
        const float2 jf = tab[(size_t)u * kBins + k];
        s_tab[k] = make_float2(__int_as_float((int)sizeof(float2) * (int)jf.x), jf.y);
    }

    // Lane l holds packed inputs m = l + 64 i, i.e. frame offsets tau = 2m, 2m + 1 for m < 200 and
    // tau = 2m - 2048, 2m - 2047 for m >= 824; everything else in the 2048-point buffer is zero.  So i is 0 .. 3 or
    // 12 .. 15, of i = 3 the first eight lanes have one and of i = 12 the last eight: these two are input 3 of a lane.
    // Input s of a lane lies 2 l + tau0(s) from the frame's centre.  The window weight of offset tau is 0.5 + 0.5 cos(pi tau / 400).
    auto tau0 = [](int s) { return s < 3 ? 128 * s : 128 * (s + 9) - kFft; };        // (s = 3: that of the last lanes)
    const bool head = lane < 8, tail = lane >= 56;           // what input 3 is
    const int tau3 = head ? 2 * lane + 384 : tail ? 2 * lane + tau0(3) : 0;
    if (wv == 0) {
        float2 w[7];
#pragma unroll
        for (int s = 0; s < 7; ++s) {
            const int tau = s == 3 ? tau3 : 2 * lane + tau0(s);
            w[s] = make_float2(0.5f + 0.5f * cospif((float)tau / (float)kHop), 0.5f + 0.5f * cospif((float)(tau + 1) / (float)kHop));
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) s_window[64 * i + lane] = make_float4(w[2 * i].x, w[2 * i].y, w[2 * i + 1].x, w[2 * i + 1].y);
        s_window6[lane] = w[6];
    }
    if (tid >= kThreads - kFactors) {
        const int i = tid - (kThreads - kFactors);
        const Tw16Short w = tw16_of(tw, i < kOfB ? i : i < kOfInverseB ? 4 * (i - kOfB) : 16 * (i - kOfInverseB));
        s_factors[3 * i] = make_float4(w.outer.t1, w.outer.t2, w.outer.t3, w.outer.c1);
        s_factors[3 * i + 1] = make_float4(w.outer.c2, w.outer.r, w.inner.t1, w.inner.t2);
        s_factors[3 * i + 2] = make_float4(w.inner.t3, w.inner.c1, w.inner.c2, w.inner.r);
    }
    // A lane's units of step D are the butterflies j = lane and j = lane + 64 with their mirror images; lane 0 has 128 and 0
    // in the first (see inplace_step_d).  Their twiddles are kept in LDS, the places are formed anew for every frame.
    auto butterfly = [](int l, int i) { return i == 0 && l == 0 ? 128 : l + 64 * i; };
    auto mirrored = [](int l, int i) { return i == 0 && l == 0 ? 0 : 256 - (l + 64 * i); };
    auto position = [](int j) { return (j & 15) * 16 + (j >> 4); };
    if (wv == 2) {
        const Tw4 w0 = tw4_of(tw, butterfly(lane, 0)), w1 = tw4_of(tw, butterfly(lane, 1));
        s_step_d[lane] = make_float4(w0.t1, w0.t2, w0.t3, w0.c1);
        s_step_d[64 + lane] = make_float4(w1.t1, w1.t2, w1.t3, w1.c1);
        s_step_d[128 + lane] = make_float4(w0.c2, w0.r, w1.c2, w1.r);
    }
    // bins k of unit 0's pairs, and exp(-i pi k / N) of them; those of unit 1 are lane + 64 + 256 s, of whose factors the
    // last two are the first two times -i
    auto bin0 = [](int l, int s) { return l ? l + 256 * s : s < 2 ? 128 + 256 * s : s == 2 ? 256 : 0; };
    float2 split0[RD], split1[2];
#pragma unroll
    for (int s = 0; s < RD; ++s) {
        const int k = bin0(lane, s);
        split0[s] = tw[kN + (k > kN / 2 ? kN - k : k)];
        if (k > kN / 2) split0[s].x = -split0[s].x;
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) split1[s] = tw[kN + lane + 64 + 256 * s];
    auto split = [&](int i, int s) { return i == 0 ? split0[s] : s < 2 ? split1[s] : rot90<false>(split1[s - 2]); };
    __syncthreads();

    // this wavefront's run of frames, and the positions that only its frames reach
    const int t_first = ((int)blockIdx.x * kWaves + wv) * share.run;
    if (t_first >= n_frames) return;                     // no barriers below
    const int t_last = min(t_first + share.run, n_frames) - 1;
    const int excl_lo = t_first == 0 ? -(1 << 30) : t_first * kHop + (kReach - kHop);
    const int excl_hi = t_last == n_frames - 1 ? (1 << 30) : t_last * kHop - (kReach - kHop);

    const float* const x = wave + start;
    float* const y = out + start;
    // the lane's seven sample pairs of frame t (unweighted)
    auto load_frame = [&](float2 (&xs)[7], int t) {
        if (t > 0 && (t + 1) * kHop <= len) {          // the whole frame lies in the utterance
            const float* const at = x + t * kHop;
#pragma unroll
            for (int s = 0; s < 7; ++s) {
                const SamplePair p = *reinterpret_cast<const SamplePair*>(at + (s == 3 ? tau3 : 2 * lane + tau0(s)));
                xs[s] = make_float2(p.x, p.y);
            }
            return;
        }
#pragma unroll
        for (int s = 0; s < 7; ++s) {                  // (unsigned compares fold in the test for positions before the utterance)
            const int g = t * kHop + (s == 3 ? tau3 : 2 * lane + tau0(s));
            xs[s] = make_float2((unsigned)g < (unsigned)len ? x[g] : 0.f, (unsigned)(g + 1) < (unsigned)len ? x[g + 1] : 0.f);
        }
    };
    // Output pairs [p, p + 1] at positions p: those in [excl_lo, excl_hi) receive nothing from other runs and are stored,
    // the rest is added atomically.  p, excl_lo and excl_hi are even, so a pair never straddles a boundary.
    auto write_pair = [&](int p, float2 s) {
        if (p >= excl_lo && p < excl_hi) {
            if (p >= 0 && p + 1 < len) {
                *reinterpret_cast<SamplePair*>(y + p) = SamplePair{s.x, s.y};
            } else {
                if ((unsigned)p < (unsigned)len) y[p] = s.x;
                if ((unsigned)(p + 1) < (unsigned)len) y[p + 1] = s.y;
            }
        } else {
            if ((unsigned)p < (unsigned)len) atomicAdd(&y[p], s.x);
            if ((unsigned)(p + 1) < (unsigned)len) atomicAdd(&y[p + 1], s.y);
        }
    };

    // The sliding window in registers.  Output pairs of frame t are numbered A = 200 t + m, m in [-512, 512); a lane owns those
    // with A mod 64 = lane, i.e. m = column + 64 (row - 8) with column = (lane - 200 t) mod 64: the inverse transform's
    // last step is taken by columns that move from frame to frame by eight lanes.  Rows 0 .. 2, in the columns below
    // eight also row 3, are complete after the frame, and the others move up by three or four.
    float2 acc[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = make_float2(0.f, 0.f);
    int column = (lane - 8 * t_first) & 63;
    bool four = false;                                   // the rows' last move was one of four
    float2 next_x[7];
    load_frame(next_x, t_first);
    for (int t = t_first;; ++t) {
        // (opaque: addresses are formed anew for every frame rather than kept in registers from one to the next)
        int l = lane;
        asm volatile("" : "+v"(l));
        float2 v[16];
        {
            float2 in[7];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const float4 w = s_window[64 * i + l];
                in[2 * i] = make_float2(next_x[2 * i].x * w.x, next_x[2 * i].y * w.y);
                in[2 * i + 1] = make_float2(next_x[2 * i + 1].x * w.z, next_x[2 * i + 1].y * w.w);
            }
            const float2 w6 = s_window6[l];
            in[6] = make_float2(next_x[6].x * w6.x, next_x[6].y * w6.y);
#pragma unroll
            for (int s = 0; s < 3; ++s) v[s] = in[s];
            v[3] = make_float2(head ? in[3].x : 0.f, head ? in[3].y : 0.f);
            v[12] = make_float2(tail ? in[3].x : 0.f, tail ? in[3].y : 0.f);
#pragma unroll
            for (int s = 4; s < 7; ++s) v[s + 9] = in[s];
        }
        if (t < t_last) load_frame(next_x, t + 1);       // arrives while this frame is transformed
        dft16_outer_inputs(v);
        {
            float2* const col = buf + T1024::pad(l);
#pragma unroll
            for (int i = 0; i < 16; ++i) col[T1024::pad(T1024::M) * i] = v[i];
        }
        fft_sync();
        step_b<false>(buf, s_factors + 3 * (kOfB + (l >> 2)), l);
        fft_sync();
        float2 a[2][RD], b[2][RD], mid = make_float2(0.f, 0.f), unused = make_float2(0.f, 0.f);
        {
            const float4 d0 = s_step_d[l], d1 = s_step_d[64 + l], d2 = s_step_d[128 + l], none = make_float4(0.f, 0.f, 0.f, 0.f);
            const float4 q0[] = {d0, make_float4(d2.x, d2.y, 0.f, 0.f), none}, q1[] = {d1, make_float4(d2.z, d2.w, 0.f, 0.f), none};
            inplace_step_d<kN, true>(a[0], b[0], mid, buf, position(butterfly(l, 0)), position(mirrored(l, 0)), q0, l == 0);
            inplace_step_d<kN, false>(a[1], b[1], unused, buf, position(butterfly(l, 1)), position(mirrored(l, 1)), q1, false);
        }
        fft_sync();

        // Packed transform Z -> twice the real spectrum X, in natural order: with A = Z[k], B = conj Z[N-k], E = A + B,
        // O = -i (A - B), w = exp(-i pi k / N):  X[k] = E + w O,  X[N-k] = conj(E - w O).  (The halves of both splits are
        // left to the scale of the output.)  k = 0 yields X[0] and X[N].
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int s = 0; s < RD; ++s) {
                const float2 A = a[i][s], B = cconj(b[i][RD - 1 - s]);
                const float2 E = cadd(A, B), O = make_float2(A.y - B.y, B.x - A.x), wO = cmul(split(i, s), O);
                const int k = i == 0 ? bin0(l, s) : l + 64 + 256 * s;
                buf[k] = cadd(E, wO);
                buf[kN - k] = cconj(csub(E, wO));
            }
        if (l == 0) buf[kN / 2] = make_float2(2.f * mid.x, -2.f * mid.y);
        fft_sync();

        // Warped spectrum Y (two interpolated bins per pair), packed for the inverse transform:
        // Ye = Y[k] + conj Y[N-k], Yo = conj(w) (Y[k] - conj Y[N-k]), Z'[k] = Ye + i Yo,
        // Z'[N-k] = conj(Ye) + i conj(Yo).  All reads of X finish before the buffer is overwritten.
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int s = 0; s < RD; ++s) {
                const int k = i == 0 ? bin0(l, s) : l + 64 + 256 * s;
                const float2 Yk = warped_bin(buf, s_tab, k), Yn = cconj(warped_bin(buf, s_tab, kN - k));
                const float2 Ye = cadd(Yk, Yn), Yo = cmul_conj(csub(Yk, Yn), split(i, s));
                a[i][s] = make_float2(Ye.x - Yo.y, Ye.y + Yo.x);
                b[i][RD - 1 - s] = make_float2(Ye.x + Yo.y, Yo.x - Ye.y);
            }
        if (l == 0) {
            const float2 Y = warped_bin(buf, s_tab, kN / 2);
            mid = make_float2(2.f * Y.x, -2.f * Y.y);
        }
        fft_sync();
        inplace_step_d_inverse<kN, true>(a[0], b[0], mid, buf, position(butterfly(l, 0)), position(mirrored(l, 0)), l == 0);
        inplace_step_d_inverse<kN, false>(a[1], b[1], unused, buf, position(butterfly(l, 1)), position(mirrored(l, 1)), false);
        fft_sync();
        step_b<true>(buf, s_factors + 3 * (kOfInverseB + (l & 3)), l);
        fft_sync();
        {
            const float2* const col = buf + T1024::pad(column);
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = col[T1024::pad(T1024::M) * i];
            dft16_twiddled<true>(v, read_factors(s_factors + 3 * column));
        }
        // v[i] is packed output m = column + 64 i times 4 N, m >= 512 standing for m - 1024
        constexpr float scale = 0.25f / (float)kN;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float2 zero = make_float2(0.f, 0.f);
            const float2 three = i < 13 ? acc[i + 3 < 16 ? i + 3 : 0] : zero, more = i < 12 ? acc[i + 4 < 16 ? i + 4 : 0] : zero;
            acc[i] = cfma(scale, v[(i + 8) & 15], make_float2(four ? more.x : three.x, four ? more.y : three.y));
        }
        const int p0 = 2 * (200 * t + column) - kReach;      // position of the lane's row 0
        if (t == t_last) {
#pragma unroll
            for (int i = 0; i < 16; ++i) write_pair(p0 + 128 * i, acc[i]);
            break;
        }
        // the next frame starts kHop later: the first kHop positions of the window are complete for this run
        four = column < 8;
        const int lo = t * kHop - kReach;
        if (lo >= max(excl_lo, 0) && lo + kHop <= min(excl_hi, len)) {      // the usual case, alike for the whole wavefront
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (i < 3 || four) *reinterpret_cast<SamplePair*>(y + p0 + 128 * i) = SamplePair{acc[i].x, acc[i].y};
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (i < 3 || four) write_pair(p0 + 128 * i, acc[i]);
        }
        column = (column - 8) & 63;
        fft_sync();                       // the next frame reuses the transform buffer
    }
}

}  // namespace

int vtlp_table_entries() { return kBins; }
int vtlp_fft_size() { return kN; }
bool vtlp_supported(int win, int hop, int nfft) { return win == kWin && hop == kHop && nfft == kFft; }

hipError_t launch_vtlp_table(hipStream_t s, int n_utt, const float* alpha, float2* tab) {
    const int64_t n = (int64_t)n_utt * kBins;
    if (n <= 0) return hipSuccess;
    vtlp_table_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s>>>(n_utt, alpha, tab);
    return hipGetLastError();
}

hipError_t launch_vtlp_resynth(hipStream_t s, int n_utt, const int64_t* d_offsets, int64_t max_len,
                               const float* wave, const float2* tab, const float2* twiddle, float* out) {
    if (n_utt <= 0 || max_len <= 0) return hipSuccess;
    const int64_t frames = (max_len - 1) / kHop + 2;
    const int64_t groups = (frames + kFramesPerGroup - 1) / kFramesPerGroup;
    const size_t lds = sizeof(float2) * (size_t)(kWaves * kSlot + kBins + 1 + 64) + sizeof(float4) * (6 * 64 + 3 * kFactors);
    vtlp_clear_kernel<<<dim3((unsigned)groups, (unsigned)n_utt), dim3(kThreads), 0, s>>>(d_offsets, out);
    vtlp_resynth_kernel<<<dim3((unsigned)groups, (unsigned)n_utt), dim3(kThreads), lds, s>>>(
        d_offsets, wave, tab, twiddle, out);
    return hipGetLastError();
}

}  // namespace aug
