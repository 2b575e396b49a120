// Complex FFT of N = 4096, 8192 or 16384 points in LDS by T = N / 16 threads, in place, for the overlap-save
// convolution, and of 1024 points by one wavefront for the waveform VTLP (which has its own steps A and B, with no barrier,
// and no step C): the forward transform leaves its output in digit-reversed order, the inverse takes it from there, and
// the product between them happens in the registers that the forward transform's last step and the inverse's first
// step share.
//
// N = 16 x 16 x RC x RD.  Time index n = n' + M mA (M = N/16), n' = t' + M2 mB (M2 = N/256), t' = t'' + RD mC;
// frequency k = k1 + 16 kB + 256 kC + 256 RC kD.  Steps: A over mA (thread n' = tid), B over mB, C over mC, D over t''.
// Each step's outputs replace its inputs, so value (k1, kB, kC, kD) ends at ((k1 16 + kB) RC + kC) RD + kD and a step's
// stores meet no other thread's loads.  B and C work inside rows of M values that one wavefront owns: they need no
// barrier between them.  A thread's values of step A (inverse: its last step) are its own from one block to the next.
//
// Twiddles ride on the next step's inputs: what a step leaves to be multiplied is, for the inputs m of one butterfly of
// the next step, a constant (passed on once more) times w^m:
//   B: w = W256^k1     C: w = W(256 RC)^(k1 + 16 kB)     D: w = WN^j, j = k1 + 16 kB + 256 kC
// and for the inverse, conjugated, C: w = W(M2)^t''     B: w = WM^(t'' + RD mC)     A: w = WN^n'.
// (dft16_twiddled / dft4_twiddled take such powers as part of their additions.)
//
// Step D's butterfly j makes the bins j + (N / RD) kD; the mirror images N - k of its bins are those of butterfly
// N / RD - j in reverse order.  A thread takes both ("a unit", 8 / RD of them per thread), so the even/odd split of a
// real transform, which pairs k with N - k, needs no exchange.  Row 0 has two butterflies that are their own mirror
// images (j = 0 and N / (2 RD)); they form unit 0 of thread 0.
//
// LDS traffic per transform pair: 12 passes over the block, where transforms in natural order with the product from LDS
// took 16.
#pragma once

#include "fft_lds.h"

namespace aug {

template <int N>
struct InPlace {
    static_assert(N == 1024 || N == 4096 || N == 8192 || N == 16384, "transform size");
    static constexpr int T = N / 16, M = N / 16, M2 = N / 256;
    static constexpr int RD = N == 8192 ? 2 : 4, RC = M2 / RD;
    static constexpr int Y = 16 * RC;                   // butterflies of step D in a row
    static constexpr int Units = 8 / RD;                // per thread
    static constexpr int RowLanes = M / 16;             // lanes that own a row

    // two complex values of padding per 32: 16-byte accesses stay aligned, and step C's stride of M2 values spreads over
    // all banks
    __host__ __device__ static constexpr int pad(int p) { return p + 2 * (p >> 5); }
    static constexpr int kPadded = N + N / 16;

    // The pair that unit i of thread tid makes in slot s < RD: bins k and, mirrored, N - k (k = 0: bins 0 and N).
    // Slot RD of thread 0 is the bin in the middle, N / 2.
    __host__ __device__ static int pair_bin(int tid, int i, int s) {
        if (s == RD) return N / 2;
        if (tid == 0 && i == 0) {                       // p: j = N / (2 RD); q: j = 0
            if (s < RD / 2) return N / (2 * RD) + N / RD * s;
            return s == RD - 1 ? 0 : N / RD;            // (RD = 4: q1 with q3, then q0)
        }
        int a, b;
        unit(tid, i, a, b);
        return bin(a) + N / RD * s;
    }
    // step-D butterfly index (position / RD) -> j
    __host__ __device__ static int bin(int at) {
        const int k1 = at / Y, y = at % Y;
        return k1 + 16 * (y / RC) + 256 * (y % RC);
    }
    // the two butterflies of a unit, as positions / RD.  (Within a row positions count kB RC + kC.)
    __host__ __device__ static inline void unit(int tid, int i, int& a, int& b) {
        const int p = tid + T * i;
        if (p >= Y) {                                   // rows k1 and 16 - k1
            const int k1 = p / Y, at = p % Y;
            a = k1 * Y + at;
            b = (16 - k1) * Y + (Y - 1 - at);
        } else if (p >= Y / 2) {                        // row 8
            const int at = p - Y / 2;
            a = 8 * Y + at;
            b = 8 * Y + (Y - 1 - at);
        } else {                                        // row 0: frequencies 16 y and 16 (Y - y)
            const int y = p ? p : Y / 2, z = p ? Y - p : 0;
            a = (y % 16) * RC + y / 16;
            b = (z % 16) * RC + z / 16;
        }
    }

    // ---- twiddle tables, in floats ----
    // first kept in LDS: step B [16][12], C [Y 16][12 or 6], inverse C [RD][12 or 6], inverse B [M2][12]; then, read
    // from memory, per thread: inverse A [3][T][4] and step D with the pairs' tangents [Units][kDQuads][T][4]
    static constexpr int kShort = 2 * kTw4Floats;       // floats of a Tw16Short
    static constexpr int kC = RC == 16 ? kShort : kTw4Floats;
    static constexpr int kB0 = 0, kC0 = kB0 + 16 * kShort, kCi0 = kC0 + 256 * kC, kBi0 = kCi0 + RD * kC;
    static constexpr int kLdsFloats = (kBi0 + M2 * kShort + 3) & ~3;
    static constexpr int kDQuads = RD == 4 ? 3 : 1;     // RD 4: six factors and four tangents; RD 2: two and two
    static constexpr int kA0 = kLdsFloats, kD0 = kA0 + 12 * T;
    static constexpr int kFloats = kD0 + Units * kDQuads * 4 * T;
};

// ---- device code ----------------------------------------------------------------------------------------

template <int N>
__device__ inline float inplace_table_value(int e) {
    using P = InPlace<N>;
    auto of_tw4 = [](double x, int f) {
        const Tw4 w = make_tw4(x);
        const float v[kTw4Floats] = {w.t1, w.t2, w.t3, w.c1, w.c2, w.r};
        float pick = v[0];
        for (int k = 1; k < kTw4Floats; ++k) pick = f == k ? v[k] : pick;
        return pick;
    };
    auto of_short = [&](double x, int f) { return f < kTw4Floats ? of_tw4(4.0 * x, f) : of_tw4(x, f - kTw4Floats); };
    auto of_c = [&](double x, int f) { return P::RC == 16 ? of_short(x, f) : of_tw4(x, f); };
    if (e < P::kC0) return of_short((double)(e / P::kShort) / 128.0, e % P::kShort);                       // W256^k1
    if (e < P::kCi0) return of_c((double)((e - P::kC0) / P::kC) / (128.0 * P::RC), (e - P::kC0) % P::kC);
    if (e < P::kBi0) return of_c(2.0 * (double)((e - P::kCi0) / P::kC) / (double)P::M2, (e - P::kCi0) % P::kC);
    if (e < P::kA0) return of_short(2.0 * (double)((e - P::kBi0) / P::kShort) / (double)P::M, (e - P::kBi0) % P::kShort);
    if (e < P::kD0) {
        const int i = e - P::kA0, quad = i / (4 * P::T), tid = i / 4 % P::T;
        return of_short(2.0 * (double)tid / (double)N, 4 * quad + i % 4);
    }
    const int i = e - P::kD0, tid = i / 4 % P::T, quad = i / (4 * P::T), unit = quad / P::kDQuads;
    const int f = 4 * (quad % P::kDQuads) + i % 4, n_tw = P::RD == 4 ? kTw4Floats : 2;
    if (f < n_tw) {
        int a, b;
        P::unit(tid, unit, a, b);
        const double x = 2.0 * (double)P::bin(a) / (double)N;
        if (P::RD == 4) return of_tw4(x, f);
        return f == 0 ? of_tw4(x, 0) : of_tw4(x, 3);                            // t1, c1
    }
    if (f >= n_tw + P::RD) return 0.f;
    double s, c;                                                                // tangent of the pair's split twiddle
    sincospi(-(double)P::pair_bin(tid, unit, f - n_tw) / (double)N, &s, &c);
    return (float)(s / c);
}

__device__ inline Tw4 read_tw4(const float* f) { return Tw4{f[0], f[1], f[2], f[3], f[4], f[5]}; }
__device__ inline Tw16Short read_short(const float* f) {         // 16-byte aligned
    const float4 a = *reinterpret_cast<const float4*>(f), b = *reinterpret_cast<const float4*>(f + 4), c = *reinterpret_cast<const float4*>(f + 8);
    return Tw16Short{{a.x, a.y, a.z, a.w, b.x, b.y}, {b.z, b.w, c.x, c.y, c.z, c.w}};
}

// positions of step C's inputs: butterfly g < 16 / RC of this thread, inputs at + RD m
template <int N>
struct StepC {
    using P = InPlace<N>;
    int row, kb[16 / P::RC], low;                       // row k1, the blocks kB, t''
    __device__ inline explicit StepC(int tid) {
        row = tid / P::RowLanes;
        const int l = tid % P::RowLanes;
        low = l % P::RD;
#pragma unroll
        for (int g = 0; g < 16 / P::RC; ++g) kb[g] = l / P::RD + (P::RowLanes / P::RD) * g;
    }
    __device__ inline int at(int g) const { return row * P::M + kb[g] * P::M2 + low; }
};

// Steps A and B: v[mA] = input n' + M mA of thread n' = tid.  All threads call.  `tab`: the tables in LDS.
template <int N>
__device__ inline void inplace_forward_ab(float2 (&v)[16], float2* buf, const float* tab, int tid) {
    using P = InPlace<N>;
    dft16<false>(v);
    {
        float2* col = buf + P::pad(tid);
#pragma unroll
        for (int i = 0; i < 16; ++i) col[P::pad(P::M) * i] = v[i];               // (M is a multiple of 32)
    }
    __syncthreads();
    {
        const int row = tid / P::RowLanes, l = tid % P::RowLanes;
        const Tw16Short w = read_short(tab + P::kB0 + P::kShort * row);
        // the row's values l + M2 m
        float2* at = buf + P::pad(P::M) * row;
#pragma unroll
        for (int m = 0; m < 16; ++m) v[m] = at[P::pad(l) + P::pad(P::M2 * m)];
        dft16_twiddled<false>(v, w);
#pragma unroll
        for (int m = 0; m < 16; ++m) at[P::pad(l) + P::pad(P::M2 * m)] = v[m];
    }
    fft_sync();
}

// Step C: the values are left in LDS for step D, which needs a barrier before it.
template <int N>
__device__ inline void inplace_forward_c(float2 (&v)[16], float2* buf, const float* tab, int tid) {
    using P = InPlace<N>;
    const StepC<N> c(tid);
#pragma unroll
    for (int g = 0; g < 16 / P::RC; ++g)
#pragma unroll
        for (int m = 0; m < P::RC; ++m) v[P::RC * g + m] = buf[P::pad(c.at(g)) + P::pad(P::RD * m)];
    if constexpr (P::RC == 16) {
        dft16_twiddled<false>(v, read_short(tab + P::kC0 + P::kC * (c.row + 16 * c.kb[0])));
    } else {
#pragma unroll
        for (int g = 0; g < 16 / P::RC; ++g)
            dft4_twiddled<false>(v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3], read_tw4(tab + P::kC0 + P::kC * (c.row + 16 * c.kb[g])));
    }
#pragma unroll
    for (int g = 0; g < 16 / P::RC; ++g)
#pragma unroll
        for (int m = 0; m < P::RC; ++m) buf[P::pad(c.at(g)) + P::pad(P::RD * m)] = v[P::RC * g + m];
}

// Steps C to A of the inverse, from the values that the first step left in LDS (a barrier before): v[mA] = N x[n' + M mA].
// `wa`: the thread's factors of step A.
template <int N>
__device__ inline void inplace_inverse(float2 (&v)[16], float2* buf, const float* tab, int tid, const Tw16Short& wa) {
    using P = InPlace<N>;
    {
        const StepC<N> c(tid);
#pragma unroll
        for (int g = 0; g < 16 / P::RC; ++g)
#pragma unroll
            for (int m = 0; m < P::RC; ++m) v[P::RC * g + m] = buf[P::pad(c.at(g)) + P::pad(P::RD * m)];
        if constexpr (P::RC == 16) {
            dft16_twiddled<true>(v, read_short(tab + P::kCi0 + P::kC * c.low));
        } else {
            const Tw4 w = read_tw4(tab + P::kCi0 + P::kC * c.low);
#pragma unroll
            for (int g = 0; g < 16 / P::RC; ++g) dft4_twiddled<true>(v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3], w);
        }
#pragma unroll
        for (int g = 0; g < 16 / P::RC; ++g)
#pragma unroll
            for (int m = 0; m < P::RC; ++m) buf[P::pad(c.at(g)) + P::pad(P::RD * m)] = v[P::RC * g + m];
    }
    fft_sync();
    {
        const int row = tid / P::RowLanes, l = tid % P::RowLanes;
        const Tw16Short w = read_short(tab + P::kBi0 + P::kShort * l);
        float2* at = buf + P::pad(P::M) * row;
#pragma unroll
        for (int m = 0; m < 16; ++m) v[m] = at[P::pad(l) + P::pad(P::M2 * m)];
        dft16_twiddled<true>(v, w);
#pragma unroll
        for (int m = 0; m < 16; ++m) at[P::pad(l) + P::pad(P::M2 * m)] = v[m];
    }
    __syncthreads();
    const float2* col = buf + P::pad(tid);
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = col[P::pad(P::M) * i];
    dft16_twiddled<true>(v, wa);
}

// Step D of unit i: the two butterflies' inputs from LDS, outputs a[kD] and b[kD] with a[s] and b[RD - 1 - s] mirror
// images of each other.  q[..]: the unit's factors.  FIRST: unit 0, which in thread 0 is not like the others.
template <int N, bool FIRST>
__device__ inline void inplace_step_d(float2 (&a)[InPlace<N>::RD], float2 (&b)[InPlace<N>::RD], float2& mid, const float2* buf, int pos_a,
                                      int pos_b, const float4 (&q)[InPlace<N>::kDQuads], bool thread0) {
    using P = InPlace<N>;
    constexpr int RD = P::RD;
    const float4* pa = reinterpret_cast<const float4*>(buf + P::pad(RD * pos_a));
    const float4* pb = reinterpret_cast<const float4*>(buf + P::pad(RD * pos_b));
#pragma unroll
    for (int m = 0; m < RD / 2; ++m) {
        const float4 x = pa[m], y = pb[m];
        a[2 * m] = make_float2(x.x, x.y);
        a[2 * m + 1] = make_float2(x.z, x.w);
        b[2 * m] = make_float2(y.x, y.y);
        b[2 * m + 1] = make_float2(y.z, y.w);
    }
    // the mirrored butterfly's twiddles are W_RD^m conj(w^m): the conjugates, with outputs moved on by one
    if constexpr (RD == 4) {
        const Tw4 w{q[0].x, q[0].y, q[0].z, q[0].w, q[1].x, q[1].y};
        Tw4 z = w;
        if (FIRST && thread0) z = Tw4{0.f, 0.f, 0.f, 1.f, 1.f, 1.f};             // j = 0
        dft4_twiddled<false>(a[0], a[1], a[2], a[3], w);
        b[1] = tilt<true>(b[1], z.t1);
        b[2] = tilt<true>(b[2], z.t2);
        b[3] = tilt<true>(b[3], z.t3);
        dft4_scaled<false>(b[0], b[1], b[2], b[3], z.c1, z.c2, z.r);
        const float2 first = b[0];
        b[0] = b[1];
        b[1] = b[2];
        b[2] = b[3];
        b[3] = first;
        if (FIRST && thread0) {                          // b = q1 q2 q3 q0, a = p0 .. p3
            mid = b[1];
            const float2 q1 = b[0], q3 = b[2], q0 = b[3];
            b[3] = a[3];
            b[2] = a[2];
            b[1] = q3;
            b[0] = q0;
            a[2] = q1;
            a[3] = q0;
        }
    } else {
        const float2 x = tilt<false>(a[1], q[0].x);
        const float c = q[0].y;
        a[1] = cfma(-c, x, a[0]);
        a[0] = cfma(c, x, a[0]);
        const float tz = FIRST && thread0 ? 0.f : q[0].x, cz = FIRST && thread0 ? 1.f : c;
        const float2 y = tilt<true>(b[1], tz);
        const float2 plus = cfma(cz, y, b[0]), minus = cfma(-cz, y, b[0]);
        b[0] = minus;                                    // outputs moved on by one
        b[1] = plus;
        if (FIRST && thread0) {                          // b = q1 q0, a = p0 p1
            mid = b[0];
            const float2 q0 = b[1];
            b[1] = a[1];
            a[1] = q0;
            b[0] = q0;
        }
    }
}

// The inverse's first step: undo the arrangement above and store both butterflies in place.
template <int N, bool FIRST>
__device__ inline void inplace_step_d_inverse(float2 (&a)[InPlace<N>::RD], float2 (&b)[InPlace<N>::RD], float2 mid, float2* buf, int pos_a,
                                              int pos_b, bool thread0) {
    using P = InPlace<N>;
    constexpr int RD = P::RD;
    if (FIRST && thread0) {
        if constexpr (RD == 4) {                         // slots: (p0,p3) (p1,p2) (q1,q3) (q0,-)
            const float2 p2 = b[2], p3 = b[3], q0 = a[3], q1 = a[2], q3 = b[1];
            a[2] = p2;
            a[3] = p3;
            b[0] = q0;
            b[1] = q1;
            b[2] = mid;
            b[3] = q3;
        } else {                                         // slots: (p0,p1) (q0,-)
            const float2 p1 = b[1], q0 = a[1];
            a[1] = p1;
            b[0] = q0;
            b[1] = mid;
        }
    }
    if constexpr (RD == 4) {
        dft4<true>(a[0], a[1], a[2], a[3]);
        dft4<true>(b[0], b[1], b[2], b[3]);
    } else {
        const float2 x = a[0], y = b[0];
        a[0] = cadd(x, a[1]);
        a[1] = csub(x, a[1]);
        b[0] = cadd(y, b[1]);
        b[1] = csub(y, b[1]);
    }
    float4* pa = reinterpret_cast<float4*>(buf + P::pad(RD * pos_a));
    float4* pb = reinterpret_cast<float4*>(buf + P::pad(RD * pos_b));
#pragma unroll
    for (int m = 0; m < RD / 2; ++m) {
        pa[m] = make_float4(a[2 * m].x, a[2 * m].y, a[2 * m + 1].x, a[2 * m + 1].y);
        pb[m] = make_float4(b[2 * m].x, b[2 * m].y, b[2 * m + 1].x, b[2 * m + 1].y);
    }
}

// ---- products of packed real transforms --------------------------------------------------------------------
// Two real sequences packed even/odd into complex ones transform to Z; with A = Z[k], B = conj Z[N-k] and the response's
// spectrum H of the 2N-point real transform, the packed product is
//     Z'[k] = (S A + D X) / 2,  conj Z'[N-k] = (S B - D Y) / 2,   X = tau A + i B,  Y = tau B + i A,
// S = H[k] + conj H[N-k], D = cos(pi k / N) (H[k] - conj H[N-k]), tau = -tan(pi k / N): twenty multiply-adds per pair,
// and no twiddle to be formed.  (S, D) take the place of H[k], H[N-k]: the same memory.
// ADD: the result is added to what is there (the response's second partition).
template <bool ADD>
__device__ inline void product_pair(float2 A, float2 B, float4 sd, float tau, float2& zk, float2& zn_conj) {
    const float2 X = make_float2(fmaf(tau, A.x, -B.y), fmaf(tau, A.y, B.x));
    const float2 Y = make_float2(fmaf(tau, B.x, -A.y), fmaf(tau, B.y, A.x));
    const float2 k0 = ADD ? make_float2(fmaf(sd.x, A.x, zk.x), fmaf(sd.x, A.y, zk.y)) : make_float2(sd.x * A.x, sd.x * A.y);
    const float2 n0 = ADD ? make_float2(fmaf(sd.x, B.x, zn_conj.x), fmaf(sd.x, B.y, zn_conj.y)) : make_float2(sd.x * B.x, sd.x * B.y);
    zk.x = fmaf(-sd.w, X.y, fmaf(sd.z, X.x, fmaf(-sd.y, A.y, k0.x)));
    zk.y = fmaf(sd.w, X.x, fmaf(sd.z, X.y, fmaf(sd.y, A.x, k0.y)));
    zn_conj.x = fmaf(sd.w, Y.y, fmaf(-sd.z, Y.x, fmaf(-sd.y, B.y, n0.x)));
    zn_conj.y = fmaf(-sd.w, Y.x, fmaf(-sd.z, Y.y, fmaf(sd.y, B.x, n0.y)));
}

// Spectrum entries: pair s of unit i of thread tid is entry (i RD + s) T + tid of N / 2; entry N / 2 holds what the bin in
// the middle, k = N / 2, is multiplied by.
template <int N> __device__ __host__ constexpr int inplace_spectrum_entries() { return N / 2 + 1; }

}  // namespace aug
