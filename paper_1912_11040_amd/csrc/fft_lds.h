// Complex FFT of a power-of-two length N held in LDS and worked on by T = N/16 threads,
// and the butterflies that the library's transforms share: the convolution for responses of up to 2048 taps
// (N = 1024, 2048) runs the passes below, the front end, the convolution for longer
// responses and the waveform VTLP (fft_inplace.h) have passes of their own.
//
// Stockham autosort passes: a pass of radix R over sub-transforms of length NS reads, for
// butterfly j < N/R, x[j + m N/R] (m < R), multiplies by exp(-+2 pi i (j mod NS) m / (NS R)),
// takes an R-point DFT and writes y[(j div NS) NS R + (j mod NS) + r NS].  Input and output
// are in natural order.  The transform runs in place: every thread keeps its 16 values of a
// pass in registers, so all reads of a pass complete before its writes begin.
// Radix 16 while four or more bits remain, then radix 4 and/or 2.
//
// Twiddles come from a table in LDS (RowTwiddles), from per-lane factors folded into the butterflies' additions
// (dft16_twiddled), or, in the convolution's column step, from one table value per butterfly whose powers are formed by
// at most four successive complex products.  The inverse uses conjugates and is unscaled.
//
// All threads of one transform sit in one wavefront, so a wave-level fence separates the reads and writes of a
// pass (LDS operations of a wave complete in order).  The convolution's transforms are split as N = 16 x M: one
// radix-16 step across the group, with barriers, then 16 independent M-point row transforms of at most 64 lanes
// each, which need none and so overlap each other's LDS and ALU phases (see fft_columns_*).
//
// LDS addressing is padded by one complex per 16 (element i lives at lds_pad(i)) so that both
// the unit-stride reads and the stride-NS writes of every pass spread over all banks.
#pragma once

#include <hip/hip_runtime.h>

namespace aug {

__device__ __host__ constexpr int lds_pad(int i) { return i + (i >> 4); }
__device__ __host__ constexpr int lds_padded_size(int n) { return n + (n >> 4); }

__host__ __device__ inline float2 cmul(float2 a, float2 b) {
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__host__ __device__ inline float2 cmul_conj(float2 a, float2 b) {   // a * conj(b)
    return make_float2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}
__host__ __device__ inline float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__host__ __device__ inline float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__host__ __device__ inline float2 cconj(float2 a) { return make_float2(a.x, -a.y); }
// multiply by -i (forward) or +i (inverse)
template <bool INV> __host__ __device__ inline float2 rot90(float2 a) {
    return INV ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x);
}

// 4-point DFT, natural order in and out; INV uses exp(+2 pi i / 4).
template <bool INV>
__host__ __device__ inline void dft4(float2& a0, float2& a1, float2& a2, float2& a3) {
    const float2 s02 = cadd(a0, a2), d02 = csub(a0, a2);
    const float2 s13 = cadd(a1, a3), d13 = rot90<INV>(csub(a1, a3));
    a0 = cadd(s02, s13);
    a1 = cadd(d02, d13);
    a2 = csub(s02, s13);
    a3 = csub(d02, d13);
}

// R-point DFT of v[0..R), natural order in and out.
template <int R, bool INV> struct SmallDft;

template <bool INV> struct SmallDft<2, INV> {
    __device__ static inline void run(float2* v) {
        const float2 a = v[0], b = v[1];
        v[0] = cadd(a, b);
        v[1] = csub(a, b);
    }
};

template <bool INV> struct SmallDft<4, INV> {
    __device__ static inline void run(float2* v) { dft4<INV>(v[0], v[1], v[2], v[3]); }
};

template <bool INV> struct SmallDft<16, INV> {
    // m = m2 + 4 m1, r = r1 + 4 r2:
    // y[r1 + 4 r2] = sum_{m2} W4^{m2 r2} W16^{m2 r1} sum_{m1} x[m2 + 4 m1] W4^{m1 r1}
    __device__ static inline void run(float2* v) {
        constexpr float c1 = 0.92387953251128674f, s1 = 0.38268343236508977f;   // cos, sin(pi/8)
        constexpr float h = 0.70710678118654752f;
        // W16^e = exp(-2 pi i e / 16) for e = 0..9 (forward sign)
        const float2 w[10] = {{1.f, 0.f}, {c1, -s1}, {h, -h}, {s1, -c1}, {0.f, -1.f},
                              {-s1, -c1}, {-h, -h}, {-c1, -s1}, {-1.f, 0.f}, {-c1, s1}};
#pragma unroll
        for (int m2 = 0; m2 < 4; ++m2) {
            dft4<INV>(v[m2], v[m2 + 4], v[m2 + 8], v[m2 + 12]);     // now v[m2 + 4 r1]
#pragma unroll
            for (int r1 = 1; r1 < 4; ++r1) {
                if (m2 == 0) continue;
                const float2 t = w[m2 * r1];
                v[m2 + 4 * r1] = INV ? cmul_conj(v[m2 + 4 * r1], t) : cmul(v[m2 + 4 * r1], t);
            }
        }
#pragma unroll
        for (int r1 = 0; r1 < 4; ++r1)
            dft4<INV>(v[4 * r1 + 0], v[4 * r1 + 1], v[4 * r1 + 2], v[4 * r1 + 3]);  // v[4 r1 + r2] = y[r1 + 4 r2]
#pragma unroll
        for (int r1 = 0; r1 < 4; ++r1)
#pragma unroll
            for (int r2 = r1 + 1; r2 < 4; ++r2) {
                const float2 t = v[4 * r1 + r2];
                v[4 * r1 + r2] = v[4 * r2 + r1];
                v[4 * r2 + r1] = t;
            }
    }
};

// ---- radix-4 and radix-16 steps with their twiddles folded into multiply-adds ----------------------------
// A twiddle w = c (1 + i t), t = tan of its angle, costs two fused multiply-adds if the factor c is left for
// the additions that follow, where it is the multiplier of a fused multiply-add and costs nothing: a radix-4
// step on twiddled inputs takes 22 instructions instead of 12 + 16, a radix-16 step 176 instead of 228.
// Results round as those of the plain form do: where c is small, t is large and the sum inside is the term
// that survives the product with c.  (c is kept at 2^-40 or above in magnitude, so that t and the ratio of
// two such factors stay far from overflow; the twiddle is then off by 2^-40, a 2^-16th of its rounding.)
struct Tw4 {
    float t1, t2, t3;      // tangents of w1, w2 = w1^2, w3 = w1^3
    float c1, c2, r;       // cosines of w1, w2; cosine of w3 over that of w1
};
constexpr int kTw4Floats = sizeof(Tw4) / sizeof(float);

// w1 = exp(-i pi x), evaluated in double precision
__host__ __device__ inline Tw4 make_tw4(double x) {
    double c[3], t[3];
    for (int m = 0; m < 3; ++m) {
        double sn;
        sincospi(-x * (double)(m + 1), &sn, &c[m]);
        if (fabs(c[m]) < 0x1p-40) c[m] = c[m] < 0.0 ? -0x1p-40 : 0x1p-40;
        t[m] = sn / c[m];
    }
    return Tw4{(float)t[0], (float)t[1], (float)t[2], (float)c[0], (float)c[1], (float)(c[2] / c[0])};
}

// a (1 + i t), the twiddle conjugated for the inverse
template <bool INV> __host__ __device__ inline float2 tilt(float2 a, float t) {
    return INV ? make_float2(fmaf(t, a.y, a.x), fmaf(-t, a.x, a.y)) : make_float2(fmaf(-t, a.y, a.x), fmaf(t, a.x, a.y));
}
__host__ __device__ inline float2 cfma(float k, float2 b, float2 a) { return make_float2(fmaf(k, b.x, a.x), fmaf(k, b.y, a.y)); }

// 4-point DFT of a0, c1 a1, c2 a2, c1 r a3
template <bool INV>
__host__ __device__ inline void dft4_scaled(float2& a0, float2& a1, float2& a2, float2& a3, float c1, float c2, float r) {
    const float2 s02 = cfma(c2, a2, a0), d02 = cfma(-c2, a2, a0);
    const float2 s13 = cfma(r, a3, a1), d13 = rot90<INV>(cfma(-r, a3, a1));
    a0 = cfma(c1, s13, s02);
    a1 = cfma(c1, d13, d02);
    a2 = cfma(-c1, s13, s02);
    a3 = cfma(-c1, d13, d02);
}
template <bool INV>
__host__ __device__ inline void dft4_twiddled(float2& a0, float2& a1, float2& a2, float2& a3, const Tw4& w) {
    a1 = tilt<INV>(a1, w.t1);
    a2 = tilt<INV>(a2, w.t2);
    a3 = tilt<INV>(a3, w.t3);
    dft4_scaled<INV>(a0, a1, a2, a3, w.c1, w.c2, w.r);
}

// The four inner butterflies of a 16-point DFT, on v[4 r1 + m2] with the constant twiddles W16^{r1 m2} and, in
// the SHARED form, inputs that still await the factors c1, c2, c1 r of a twiddle common to all four.
// cos and sin of pi/8 and 3 pi/8 over each other:
constexpr float kTan8 = 0.41421356237309505f, kCot8 = 2.414213562373095f, kCos8 = 0.92387953251128674f, kSin8 = 0.38268343236508977f;
constexpr float kHalfRoot = 0.70710678118654752f;
template <bool INV, bool SHARED>
__host__ __device__ inline void dft16_inner(float2* v, float c1, float c2, float r) {
    if (!SHARED) c1 = c2 = r = 1.f;
    if (SHARED) dft4_scaled<INV>(v[0], v[1], v[2], v[3], c1, c2, r);
    else dft4<INV>(v[0], v[1], v[2], v[3]);
    // r1 = 1: angles pi/8, pi/4, 3 pi/8
    v[5] = tilt<INV>(v[5], -kTan8);
    v[6] = tilt<INV>(v[6], -1.f);
    v[7] = tilt<INV>(v[7], -kCot8);
    dft4_scaled<INV>(v[4], v[5], v[6], v[7], kCos8 * c1, kHalfRoot * c2, kTan8 * r);
    // r1 = 2: pi/4, pi/2, 3 pi/4
    v[9] = tilt<INV>(v[9], -1.f);
    v[10] = rot90<INV>(v[10]);
    v[11] = tilt<INV>(v[11], 1.f);
    dft4_scaled<INV>(v[8], v[9], v[10], v[11], kHalfRoot * c1, c2, -r);
    // r1 = 3: 3 pi/8, 3 pi/4, 9 pi/8
    v[13] = tilt<INV>(v[13], -kCot8);
    v[14] = tilt<INV>(v[14], 1.f);
    v[15] = tilt<INV>(v[15], -kTan8);
    dft4_scaled<INV>(v[12], v[13], v[14], v[15], kSin8 * c1, -kHalfRoot * c2, -kCot8 * r);
}
// v[4 r1 + r2] = y[r1 + 4 r2] -> natural order (register names only)
__host__ __device__ inline void dft16_transpose(float2* v) {
#pragma unroll
    for (int r1 = 0; r1 < 4; ++r1)
#pragma unroll
        for (int r2 = r1 + 1; r2 < 4; ++r2) {
            const float2 t = v[4 * r1 + r2];
            v[4 * r1 + r2] = v[4 * r2 + r1];
            v[4 * r2 + r1] = t;
        }
}

// 16-point DFT, natural order in and out: 144 instructions
template <bool INV> __host__ __device__ inline void dft16(float2* v) {
#pragma unroll
    for (int m2 = 0; m2 < 4; ++m2) dft4<INV>(v[m2], v[m2 + 4], v[m2 + 8], v[m2 + 12]);      // v[m2 + 4 r1]
    dft16_inner<INV, false>(v, 1.f, 1.f, 1.f);
    dft16_transpose(v);
}

// 16-point DFT of v[m] w^m from twelve factors, for w that differ from thread to thread: the first four butterflies share
// the twiddles w^4, w^8, w^12; the second four take w^{m2} and the constant W16^{r1 m2} one after the other.  199
// instructions.
struct Tw16Short { Tw4 outer, inner; };
template <bool INV> __host__ __device__ inline void dft16_twiddled(float2* v, const Tw16Short& w) {
#pragma unroll
    for (int m2 = 0; m2 < 4; ++m2) dft4_twiddled<INV>(v[m2], v[m2 + 4], v[m2 + 8], v[m2 + 12], w.outer);
#pragma unroll
    for (int r1 = 0; r1 < 4; ++r1) {
        v[4 * r1 + 1] = tilt<INV>(v[4 * r1 + 1], w.inner.t1);
        v[4 * r1 + 2] = tilt<INV>(v[4 * r1 + 2], w.inner.t2);
        v[4 * r1 + 3] = tilt<INV>(v[4 * r1 + 3], w.inner.t3);
    }
    dft16_inner<INV, true>(v, w.inner.c1, w.inner.c2, w.inner.r);
    dft16_transpose(v);
}

// v[m] *= w^m for m = 1..15, powers by products of depth <= 4
__device__ inline void twiddle_inputs(float2* v, float2 w1) {
    // powers are formed and used in an order that keeps few of them alive: w1..w8, then w8 w_m
    const float2 w2 = cmul(w1, w1);
    const float2 w3 = cmul(w2, w1);
    const float2 w4 = cmul(w2, w2);
    v[1] = cmul(v[1], w1);
    v[2] = cmul(v[2], w2);
    v[3] = cmul(v[3], w3);
    v[4] = cmul(v[4], w4);
    const float2 w5 = cmul(w4, w1);
    const float2 w6 = cmul(w4, w2);
    const float2 w7 = cmul(w4, w3);
    const float2 w8 = cmul(w4, w4);
    v[5] = cmul(v[5], w5);
    v[6] = cmul(v[6], w6);
    v[7] = cmul(v[7], w7);
    v[8] = cmul(v[8], w8);
    v[9] = cmul(v[9], cmul(w8, w1));
    v[10] = cmul(v[10], cmul(w8, w2));
    v[11] = cmul(v[11], cmul(w8, w3));
    v[12] = cmul(v[12], cmul(w8, w4));
    v[13] = cmul(v[13], cmul(w8, w5));
    v[14] = cmul(v[14], cmul(w8, w6));
    v[15] = cmul(v[15], cmul(w8, w7));
}

constexpr int ilog2(int n) { return n <= 1 ? 0 : 1 + ilog2(n >> 1); }

template <int N>
struct FftPlan {
    static constexpr int kLog = ilog2(N);
    static constexpr int kN16 = kLog / 4;
    static constexpr int kRem = kLog % 4;
    static constexpr int kPasses = kN16 + (kRem >= 2 ? 1 : 0) + (kRem & 1);
    static constexpr int radix(int p) { return p < kN16 ? 16 : ((p == kN16 && kRem >= 2) ? 4 : 2); }
    static constexpr int ns(int p) {
        int s = 1;
        for (int i = 0; i < p; ++i) s *= radix(i);
        return s;
    }
    static constexpr int kLastRadix = radix(kPasses - 1);
};

// lds_pad(a + b) = lds_pad(a) + lds_pad(b) whenever b is a multiple of 16; the address code below
// uses this to keep one padded base per thread plus compile-time offsets.

// Each thread owns 16 values per pass: 16 / R butterflies j = tid + bi T.
template <int N, int T, int R>
__device__ inline void fft_load(float2 (&v)[16], const float2* buf, int tid) {
    static_assert(N == 16 * T, "sixteen values per thread");
    if constexpr (T % 16 == 0 && (N / R) % 16 == 0) {
        const float2* base = buf + lds_pad(tid);
#pragma unroll
        for (int bi = 0; bi < 16 / R; ++bi)
#pragma unroll
            for (int m = 0; m < R; ++m) v[bi * R + m] = base[lds_pad(bi * T + m * (N / R))];
    } else {
#pragma unroll
        for (int bi = 0; bi < 16 / R; ++bi)
#pragma unroll
            for (int m = 0; m < R; ++m) v[bi * R + m] = buf[lds_pad(tid + bi * T + m * (N / R))];
    }
}

template <int N, int T, int R, int NS>
__device__ inline void fft_store(const float2 (&v)[16], float2* buf, int tid) {
#pragma unroll
    for (int bi = 0; bi < 16 / R; ++bi) {
        const int j = tid + bi * T;
        const int k = j % NS;
        const int j0 = (j / NS) * NS * R + k;
        if constexpr (NS % 16 == 0) {
            float2* base = buf + lds_pad(j0);
#pragma unroll
            for (int r = 0; r < R; ++r) base[lds_pad(r * NS)] = v[bi * R + r];
        } else if constexpr (NS == 1 && R == 16) {
            float2* base = buf + 17 * j;                 // lds_pad(16 j + r) = 17 j + r
#pragma unroll
            for (int r = 0; r < R; ++r) base[r] = v[bi * R + r];
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) buf[lds_pad(j0 + r * NS)] = v[bi * R + r];
        }
    }
}

// what the wavefront wrote to LDS before is there for the reads after
__device__ inline void fft_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Natural index of value v[bi R + r] after the last pass, and before the first pass of input v[bi R + m].
template <int N, int T>
__device__ inline int fft_out_index(int tid, int i) {
    constexpr int R = FftPlan<N>::kLastRadix;
    return tid + (i / R) * T + (i % R) * (N / R);
}
template <int N, int T>
__device__ inline int fft_in_index(int tid, int i) {
    constexpr int R = FftPlan<N>::radix(0);
    return tid + (i / R) * T + (i % R) * (N / R);
}

// Store the last pass's outputs in natural order.
template <int N, int T>
__device__ inline void fft_store_natural(const float2 (&v)[16], float2* buf, int tid) {
    constexpr int R = FftPlan<N>::kLastRadix;
    if constexpr (T % 16 == 0 && (N / R) % 16 == 0) {
        float2* base = buf + lds_pad(tid);
#pragma unroll
        for (int i = 0; i < 16; ++i) base[lds_pad((i / R) * T + (i % R) * (N / R))] = v[i];
    } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) buf[lds_pad(fft_out_index<N, T>(tid, i))] = v[i];
    }
}

// Load the first pass's inputs from a natural-order buffer.
template <int N, int T>
__device__ inline void fft_load_natural(float2 (&v)[16], const float2* buf, int tid) {
    constexpr int R = FftPlan<N>::radix(0);
    if constexpr (T % 16 == 0 && (N / R) % 16 == 0) {
        const float2* base = buf + lds_pad(tid);
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = base[lds_pad((i / R) * T + (i % R) * (N / R))];
    } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = buf[lds_pad(fft_in_index<N, T>(tid, i))];
    }
}

// ---- N = 16 x M split -------------------------------------------------------------------
// X[k1 + 16 k2] = sum_{n2 < M} W_M^{n2 k2} W_N^{n2 k1} sum_{n1 < 16} x[n2 + M n1] W_16^{n1 k1}.
// Thread n2 of the M = N/16 threads holds x[n2 + M n1] in v[n1]; after the column step v[k1] belongs
// to row k1, column n2.  Row k1 lives at buf[lds_pad(k1 M + .)] and is transformed by M/16 lanes of
// one wavefront.  After the forward transform frequency k = k1 + 16 k2 sits at row k1, column k2.

// forward column step on registers: v[n1] -> v[k1] (twiddled), to be stored at row k1, column n2
template <int N>
__device__ inline void fft_columns_forward(float2 (&v)[16], const float2* __restrict__ tw, int n2) {
    SmallDft<16, false>::run(v);
    twiddle_inputs(v, tw[n2]);
}

// inverse column step: v[k1] (row k1, column n2) -> v[n1] = N x[n2 + M n1]
template <int N>
__device__ inline void fft_columns_inverse(float2 (&v)[16], const float2* __restrict__ tw, int n2) {
    float2 w1 = tw[n2];
    w1.y = -w1.y;
    twiddle_inputs(v, w1);
    SmallDft<16, true>::run(v);
}

template <int N, int T>
__device__ inline void fft_columns_store(const float2 (&v)[16], float2* buf, int n2) {
    static_assert((N / 16) % 16 == 0, "rows are whole padding groups");
    float2* base = buf + lds_pad(n2);
#pragma unroll
    for (int k1 = 0; k1 < 16; ++k1) base[lds_pad(k1 * (N / 16))] = v[k1];
}
template <int N, int T>
__device__ inline void fft_columns_load(float2 (&v)[16], const float2* buf, int n2) {
    const float2* base = buf + lds_pad(n2);
#pragma unroll
    for (int k1 = 0; k1 < 16; ++k1) v[k1] = base[lds_pad(k1 * (N / 16))];
}

// ---- row-pass twiddles with their powers, held in LDS ---------------------------------------
// A persistent kernel fills the table once and its row transforms then read every factor they need
// (pass P of radix R and sub-length NS: exp(-2 pi i k m / (NS R)) at [k][m - 1], k < NS, m = 1..R-1) instead of
// loading one factor from global memory and forming its powers by chained products.  That removes the
// products, and it removes global loads from the row transforms, so loads issued ahead of them are not
// waited for there (a wave's global loads complete in order).
template <int M>
struct RowTwiddles {
    using Plan = FftPlan<M>;
    static constexpr int offset(int p) {
        int o = 0;
        for (int q = 1; q < p; ++q) o += Plan::ns(q) * (Plan::radix(q) - 1);
        return o;
    }
    static constexpr int kEntries = offset(Plan::kPasses);
    // tw: exp(-2 pi i t / (M TWS)); all threads of the group call, then synchronise
    template <int TWS, int P = 1>
    __device__ static inline void fill(float2* tab, const float2* __restrict__ tw, int tid, int n_threads) {
        if constexpr (P < Plan::kPasses) {
            constexpr int R = Plan::radix(P), NS = Plan::ns(P);
            for (int e = tid; e < NS * (R - 1); e += n_threads) {
                const int k = e / (R - 1), m = e % (R - 1) + 1;
                tab[offset(P) + e] = tw[k * m * (M / (NS * R)) * TWS];
            }
            fill<TWS, P + 1>(tab, tw, tid, n_threads);
        }
    }
};

// All passes, with every twiddle factor read from a RowTwiddles table in LDS.  On entry v holds the inputs of the first
// (fft_in_index order); on return it holds the outputs of the last (fft_out_index order), not yet stored.  All T threads of
// the transform must call; buf contents are overwritten.
template <int M, int T, bool INV, int P = 0>
__device__ inline void fft_passes_table(float2 (&v)[16], float2* buf, const float2* tab, int tid) {
    using Plan = FftPlan<M>;
    constexpr int R = Plan::radix(P), NS = Plan::ns(P);
#pragma unroll
    for (int bi = 0; bi < 16 / R; ++bi) {
        if constexpr (NS > 1) {
            const float2* e = tab + RowTwiddles<M>::offset(P) + ((tid + bi * T) % NS) * (R - 1);
#pragma unroll
            for (int m = 1; m < R; ++m)
                v[bi * R + m] = INV ? cmul_conj(v[bi * R + m], e[m - 1]) : cmul(v[bi * R + m], e[m - 1]);
        }
        SmallDft<R, INV>::run(&v[bi * R]);
    }
    if constexpr (P + 1 < Plan::kPasses) {
        fft_store<M, T, R, NS>(v, buf, tid);
        fft_sync();
        fft_load<M, T, Plan::radix(P + 1)>(v, buf, tid);
        fft_sync();
        fft_passes_table<M, T, INV, P + 1>(v, buf, tab, tid);
    }
}

// The 16 row transforms, in place in natural order within each row, with the twiddles of a RowTwiddles<N / 16> table;
// wave-level synchronisation only.  Thread tid works on row tid / (M/16) as lane tid % (M/16).  Rows must be complete
// (barrier) before.
template <int N, bool INV>
__device__ inline void fft_rows_table(float2* buf, const float2* tab, int tid) {
    constexpr int M = N / 16, LANES = M / 16;
    static_assert(LANES >= 1 && LANES <= 64, "a row is transformed inside one wavefront");
    float2* row = buf + lds_pad((tid / LANES) * M);
    const int lane = tid % LANES;
    float2 v[16];
    fft_load_natural<M, LANES>(v, row, lane);
    fft_sync();
    fft_passes_table<M, LANES, INV>(v, row, tab, lane);
    fft_store_natural<M, LANES>(v, row, lane);
}

}  // namespace aug
