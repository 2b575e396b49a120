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
// packing, done by 64 lanes with 16 values each in LDS (wave-level fences only); the frame's samples go
// from HBM straight into the first butterflies' registers.  A wavefront works through a run of consecutive
// frames and overlap-adds them in a 2048-sample sliding window of its own in LDS (plain read-modify-write,
// no atomics); the 400 samples that leave the window after each frame are written out.  Only the ends of
// a run, where the frames of the neighbouring runs also land, go to HBM with float atomics; measured on
// the chip, sending every sample through HBM atomics more than doubled the kernel's time.
// Per utterance a table holds, for every output bin, the lower source bin and the interpolation weight;
// both come from fp64 arithmetic so that the choice of the bin pair matches a double-precision evaluation.
//
// What bounds it: latency.  The windows and transform buffers leave room for two wavefronts per SIMD, whose
// vector units are busy half the time and the LDS two fifths of it (1440 vector and 217 LDS instructions per frame on 256
// utterances of 1-16 s).  Twiddles folded into multiply-adds, zero inputs skipped, mirrored bins at constant distances from
// two places and frames inside the utterance without range tests took that batch from 530 to 506 us, an utterance's
// frames shared evenly among its wavefronts instead of in runs of 16 and a rest to 495, zeros only where runs meet to 484.  Longer runs would save
// atomics and lose in balance (at most 24 frames: 506 us against 495; 32: 479, but a single utterance then has half the wavefronts).

#include "aug_internal.h"
#include "fft_lds.h"

namespace aug {
namespace {

constexpr int kWin = 800, kHop = 400, kFft = 2048;
constexpr int kN = kFft / 2;                       // complex transform length
constexpr int kBins = kN + 1;                      // real-spectrum bins 0..1024
constexpr int kWaves = 4, kThreads = 64 * kWaves;
constexpr int kRun = 16;                           // consecutive frames overlap-added by one wavefront, at most
constexpr int kMinRun = 8;                         // and at least: with runs of six or more no sample gets more than two shares
constexpr int kFramesPerGroup = kRun * kWaves;
constexpr int kSlot = lds_padded_size(kN) + 2;     // a wavefront's transform buffer plus the slot of bin 1024
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

// Value of output bin q of the warped spectrum; X is in natural order in buf, bin 1024 in the extra slot.  The table in
// LDS holds the places of the two source bins in bytes, sixteen bits each, and the weight.
__device__ inline float2 warped_bin(const float2* buf, const float2* s_tab, int q) {
    const float2 e = s_tab[q];
    const unsigned int at = (unsigned int)__float_as_int(e.x);
    const float2 lo = *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(buf) + (at & 0xffffu));
    const float2 hi = *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(buf) + (at >> 16));
    return make_float2(lo.x + e.y * (hi.x - lo.x), lo.y + e.y * (hi.y - lo.y));
}
static_assert(sizeof(float2) * kSlot < 1 << 16, "places in the buffer have sixteen bits");

// A lane's twiddles, the same for every frame: of the 1024 = 16 x 16 x 4 point transform's second pass w = W256^(lane mod
// 16), of its third w = W1024^(lane + 64 i) for butterfly i.  From the table of W1024.
struct LaneTwiddles {
    Tw16Short second;
    Tw4 third[4];
};
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
__device__ inline LaneTwiddles lane_twiddles(const float2* __restrict__ tw, int lane) {
    LaneTwiddles w;
    w.second.outer = tw4_of(tw, 16 * (lane & 15));
    w.second.inner = tw4_of(tw, 4 * (lane & 15));
#pragma unroll
    for (int i = 0; i < 4; ++i) w.third[i] = tw4_of(tw, lane + 64 * i);
    return w;
}

// A wavefront's 1024-point transform after its first butterflies; on return v[i] is output fft_out_index(lane, i).
template <bool INV>
__device__ inline void later_passes(float2 (&v)[16], float2* buf, const LaneTwiddles& w, int lane) {
    fft_store<kN, 64, 16, 1>(v, buf, lane);
    fft_sync();
    fft_load<kN, 64, 16>(v, buf, lane);
    fft_sync();
    dft16_twiddled<INV>(v, w.second);
    fft_store<kN, 64, 16, 16>(v, buf, lane);
    fft_sync();
    fft_load<kN, 64, 4>(v, buf, lane);
    fft_sync();
#pragma unroll
    for (int i = 0; i < 4; ++i) dft4_twiddled<INV>(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3], w.third[i]);
}

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

// Write positions [p0, p0 + 2 count) of the wavefront's window to the output and clear them.  Positions in
// [excl_lo, excl_hi) receive nothing from other runs and are stored; the rest is added atomically.
// p0, excl_lo and excl_hi are even, so a pair never straddles a boundary.
__device__ inline void flush_window(float* acc, float* y, int len, int p0, int count, int excl_lo, int excl_hi, int lane) {
    const int p1 = p0 + 2 * count;
    if (p0 >= max(excl_lo, 0) && p1 <= min(excl_hi, len)) {      // the usual case, alike for the whole wavefront
        for (int i = lane; i < count; i += 64) {
            const int p = p0 + 2 * i;
            float2* slot = reinterpret_cast<float2*>(acc + (p & (kFft - 1)));
            const float2 s = *slot;
            *slot = make_float2(0.f, 0.f);
            *reinterpret_cast<SamplePair*>(y + p) = SamplePair{s.x, s.y};
        }
        return;
    }
    for (int i = lane; i < count; i += 64) {
        const int p = p0 + 2 * i;
        float2* slot = reinterpret_cast<float2*>(acc + (p & (kFft - 1)));
        const float2 s = *slot;
        *slot = make_float2(0.f, 0.f);
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
    }
}

// grid: (frame groups of the longest utterance, utterances); `out` as vtlp_clear_kernel leaves it
__global__ __launch_bounds__(kThreads, 2) void vtlp_resynth_kernel(
    const int64_t* __restrict__ offsets, const float* __restrict__ wave, const float2* __restrict__ tab,
    const float2* __restrict__ tw, float* __restrict__ out) {
    extern __shared__ float2 smem[];
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;
    const int u = blockIdx.y;
    const int64_t start = offsets[u];
    const int len = (int)(offsets[u + 1] - start);      // utterances are shorter than 2^30 samples (checked on the host)
    const int n_frames = frame_count(len);
    const Share share = share_frames(n_frames);
    if ((int)blockIdx.x >= share.n_groups) return;           // the whole group leaves together
    float2* buf = smem + wv * kSlot;
    float2* s_tab = smem + kWaves * kSlot;
    float* acc = reinterpret_cast<float*>(s_tab + kBins + 1) + wv * kFft;     // [waves][2048], 8-byte aligned
    for (int k = tid; k < kBins; k += kThreads) {
        const float2 jf = tab[(size_t)u * kBins + k];
        const int j = (int)jf.x;
        s_tab[k] = make_float2(__int_as_float((int)sizeof(float2) * (lds_pad(j) | lds_pad(j + 1) << 16)), jf.y);
    }
    for (int k = lane; k < kFft / 2; k += 64) reinterpret_cast<float2*>(acc)[k] = make_float2(0.f, 0.f);

    // Lane l holds packed inputs m = l + 64 i, i.e. frame offsets tau = 2m, 2m + 1 for m < 200 and
    // tau = 2m - 2048, 2m - 2047 for m >= 824; everything else in the 2048-point buffer is zero.
    // Slots 0..3 are i = 0..3, slots 4..7 are i = 12..15.  The window weight of offset tau is
    // 0.5 + 0.5 cos(pi tau / 400).
    int tau0[8];
    float2 wnd[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const int m = lane + 64 * (s < 4 ? s : s + 8);
        const bool used = s < 4 ? m < kHop / 2 : m >= kN - kHop / 2;
        tau0[s] = s < 4 ? 2 * m : 2 * m - kFft;
        wnd[s] = used ? make_float2(0.5f + 0.5f * cospif((float)tau0[s] / (float)kHop),
                                    0.5f + 0.5f * cospif((float)(tau0[s] + 1) / (float)kHop))
                      : make_float2(0.f, 0.f);
    }
    // twiddles of this lane's butterflies and of its bin pairs are the same for every frame
    const LaneTwiddles lane_tw = lane_twiddles(tw, lane);
    float2 pair_tw[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) pair_tw[i] = tw[kN + lane + 64 * i];     // exp(-i pi k / N), k = lane + 64 i
    const float2 quarter_tw = make_float2(0.f, -1.f);                   // k = N/2
    __syncthreads();

    // this wavefront's run of frames, and the positions that only its frames reach
    const int t_first = ((int)blockIdx.x * kWaves + wv) * share.run;
    if (t_first >= n_frames) return;                     // no barriers below
    const int t_last = min(t_first + share.run, n_frames) - 1;
    const int excl_lo = t_first == 0 ? -(1 << 30) : t_first * kHop + (kReach - kHop);
    const int excl_hi = t_last == n_frames - 1 ? (1 << 30) : t_last * kHop - (kReach - kHop);

    const float* x = wave + start;
    float* y = out + start;
    // the lane's eight sample pairs of frame t (unweighted); a zero window weight marks inputs the lane does
    // not have, and unsigned compares fold the test for positions before the utterance in
    auto load_frame = [&](float2 (&xs)[8], int t) {
        if (t > 0 && (t + 1) * kHop <= len) {          // the whole frame lies in the utterance
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const bool used = wnd[s].x != 0.f || wnd[s].y != 0.f;
                const SamplePair p = *reinterpret_cast<const SamplePair*>(x + t * kHop + (used ? tau0[s] : 0));
                xs[s] = make_float2(used ? p.x : 0.f, used ? p.y : 0.f);
            }
            return;
        }
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int g = t * kHop + tau0[s];
            const bool used = wnd[s].x != 0.f || wnd[s].y != 0.f;
            xs[s] = make_float2(used && (unsigned)g < (unsigned)len ? x[g] : 0.f,
                                used && (unsigned)(g + 1) < (unsigned)len ? x[g + 1] : 0.f);
        }
    };
    float2 next_x[8];
    load_frame(next_x, t_first);
    for (int t = t_first; t <= t_last; ++t) {
        const int centre = t * kHop;
        // (opaque: addresses are formed anew for every frame rather than kept in registers from one to the next)
        int l = lane;
        asm volatile("" : "+v"(l));
        float2 v[16];
#pragma unroll
        for (int s = 0; s < 8; ++s) v[s < 4 ? s : s + 8] = make_float2(next_x[s].x * wnd[s].x, next_x[s].y * wnd[s].y);
        if (t < t_last) load_frame(next_x, t + 1);       // arrives while this frame is transformed
        dft16_outer_inputs(v);
        later_passes<false>(v, buf, lane_tw, l);
        fft_store_natural<kN, 64>(v, buf, l);
        fft_sync();

        // Packed transform Z -> twice the real spectrum X, in place: with A = Z[k], B = conj Z[N-k], E = A + B,
        // O = -i (A - B), w = exp(-i pi k / N):  X[k] = E + w O,  X[N-k] = conj(E - w O).  (The halves of both splits are
        // left to the scale of the output.)
        // A lane owns the pairs (k, N-k), k = l + 64 i: one place below and one above plus constants.  k = 0 yields X[0]
        // and X[N], the latter kept in the extra slot.
        float2* const below = buf + lds_pad(l);
        float2* const above = buf + lds_pad(64 - l);
        auto unpack = [&](float2* at_k, float2* at_n, const float2* from_n, float2 w) {
            const float2 A = *at_k, B = cconj(*from_n);
            const float2 E = cadd(A, B), O = make_float2(A.y - B.y, B.x - A.x);
            const float2 wO = cmul(w, O);
            *at_k = cadd(E, wO);
            *at_n = cconj(csub(E, wO));
        };
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            float2* const at_n = above + lds_pad(kN - 64 - 64 * i);
            unpack(below + lds_pad(64 * i), at_n, i == 0 && l == 0 ? buf : at_n, pair_tw[i]);
        }
        if (l == 0) unpack(buf + lds_pad(kN / 2), buf + lds_pad(kN / 2), buf + lds_pad(kN / 2), quarter_tw);
        fft_sync();

        // Warped spectrum Y (two interpolated bins per pair), packed for the inverse transform:
        // Ye = Y[k] + conj Y[N-k], Yo = conj(w) (Y[k] - conj Y[N-k]), Z'[k] = Ye + i Yo,
        // Z'[N-k] = conj(Ye) + i conj(Yo).  All reads of X finish before the buffer is overwritten.
        float2 zk[9], zn[9];
        auto pack = [&](int k, int slot, float2 w) {
            const float2 Yk = warped_bin(buf, s_tab, k), Yn = cconj(warped_bin(buf, s_tab, kN - k));
            const float2 Ye = cadd(Yk, Yn), Yo = cmul_conj(csub(Yk, Yn), w);
            zk[slot] = make_float2(Ye.x - Yo.y, Ye.y + Yo.x);
            zn[slot] = make_float2(Ye.x + Yo.y, Yo.x - Ye.y);
        };
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            pack(l + 64 * i, i, pair_tw[i]);
        }
        if (l == 0) pack(kN / 2, 8, quarter_tw);
        fft_sync();
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            below[lds_pad(64 * i)] = zk[i];
            if (i || l) above[lds_pad(kN - 64 - 64 * i)] = zn[i];
        }
        if (l == 0) buf[lds_pad(kN / 2)] = zk[8];
        fft_sync();

        fft_load_natural<kN, 64>(v, buf, l);
        fft_sync();
        dft16<true>(v);
        later_passes<true>(v, buf, lane_tw, l);
        // v[i] is packed output m = fft_out_index(l, i) times 4 N: samples at offsets 2m, 2m + 1 (m < N/2)
        // or 2m - 2048, 2m - 2047 from the frame centre; position p lives at window slot p mod 2048, and the
        // centre is even, so a pair is one aligned float2 of the window
        constexpr float scale = 0.25f / (float)kN;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int m = fft_out_index<kN, 64>(l, i);
            float2* slot = reinterpret_cast<float2*>(acc + ((centre + 2 * m) & (kFft - 1)));
            float2 a = *slot;
            a.x += v[i].x * scale;
            a.y += v[i].y * scale;
            *slot = a;
        }
        fft_sync();
        // the next frame starts kHop later: the first kHop positions of the window are complete for this run
        flush_window(acc, y, len, centre - kReach, kHop / 2, excl_lo, excl_hi, l);
        fft_sync();                       // also: the next frame reuses the transform buffer
    }
    flush_window(acc, y, len, t_last * kHop - kReach + kHop, (kFft - kHop) / 2, excl_lo, excl_hi, lane);
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
    const size_t lds = sizeof(float2) * (size_t)(kWaves * kSlot + kBins + 1) + sizeof(float) * kWaves * kFft;
    vtlp_clear_kernel<<<dim3((unsigned)groups, (unsigned)n_utt), dim3(kThreads), 0, s>>>(d_offsets, out);
    vtlp_resynth_kernel<<<dim3((unsigned)groups, (unsigned)n_utt), dim3(kThreads), lds, s>>>(
        d_offsets, wave, tab, twiddle, out);
    return hipGetLastError();
}

}  // namespace aug
