// Reverberation and SNR mixing (acoustic simulator, Sec. 2.3).
//
// y_j[n] = sum_{k < L} h_j[k] x_j[n-k] is evaluated by uniformly partitioned
// overlap-save: the response is cut into partitions of P taps, each transformed once
// (2P-point real FFT); an output block of P samples is the inverse transform of
// sum_p X_{b-p} H_p, X_w the transform of input samples [(w-1)P, (w+1)P).  Where one partition holds the response,
// a window gives more than its last P samples, and the blocks are as long as that (see conv_plan).
// A 2P-point real transform is run as a P-point complex FFT of the even/odd packed
// sequence, entirely in LDS, split as 16 x P/16: the radix-16 column step reads its inputs
// straight from HBM (and, inverse, writes the block straight back); the 16 row transforms
// run one per wavefront without work-group barriers.
//
// Work groups are persistent and walk along the reverberated signals block after block (see
// convolve_kernel); each block's energy is added to E[u][j] (fp64 atomics).  A response of two partitions
// costs one forward and one inverse transform per block as well: the previous window's spectrum stays in
// registers.  The gains g_j = sqrt(E_0 / (E_j 10^(snr_j/10))) (zero where an energy is zero) are formed where they are
// used: the mixture y_0 + sum_j g_j y_j is written by mix_kernel when the caller wants it, and formed by
// the front end on the fly otherwise.

#include <type_traits>

#include "aug_internal.h"
#include "fft_inplace.h"

namespace aug {
namespace {

constexpr int conv_threads(int n) { return n / 16; }

__host__ __device__ constexpr int twiddle_count(int n) { return n + n / 2 + 1 + n / 32; }

__global__ void twiddle_kernel(int n, float2* tw) {
    // tw[t] = exp(-2 pi i t / n), t < n;  tw[n + k] = exp(-i pi k / n), k <= n/2;
    // tw[n + n/2 + 1 + j] = exp(-i pi 16 j / n), j < n/32
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= twiddle_count(n)) return;
    double s, c;
    if (i < n) sincospi(-2.0 * (double)i / (double)n, &s, &c);
    else if (i < n + n / 2 + 1) sincospi(-(double)(i - n) / (double)n, &s, &c);
    else sincospi(-16.0 * (double)(i - n - n / 2 - 1) / (double)n, &s, &c);
    tw[i] = make_float2((float)c, (float)s);
}

// Even/odd split of the packed transform: from A = Z[k] and B = conj(Z[N-k]) give
// W[k] and conj(W[N-k]) of the 2N-point real transform; w = exp(-i pi k / N).
__device__ inline void unpack_pair(float2 A, float2 B, float2 w, float2& Wk, float2& WNk_conj) {
    const float2 E = make_float2(0.5f * (A.x + B.x), 0.5f * (A.y + B.y));
    const float2 d = csub(A, B);
    const float2 O = make_float2(0.5f * d.y, -0.5f * d.x);     // -(i/2)(A - B)
    const float2 wO = cmul(w, O);
    Wk = cadd(E, wO);
    WNk_conj = csub(E, wO);
}

// Bins are visited as k = k1 + 16 k2 (row k1, column k2 of the split transform), k < N/2, each with
// its partner N - k.  Thread tid owns column k2 = tid mod M/2 of rows k1 = 8 (tid div M/2) + i.
template <int N>
struct PairIndex {
    static constexpr int M = N / 16;
    int k, pos, pos_partner, h_partner;     // LDS/spectrum position of k and of N-k (spectrum: H[N] sits at N)
    __device__ inline PairIndex(int k1, int k2) {
        k = k1 + 16 * k2;
        pos = k1 * M + k2;
        pos_partner = k1 ? (16 - k1) * M + (M - 1 - k2) : ((M - k2) & (M - 1));
        h_partner = k ? pos_partner : N;
    }
};

template <int N> __device__ inline float2 pair_twiddle(const float2* __restrict__ tw, int k1, int k2) {
    return cmul(tw[N + k1], tw[N + N / 2 + 1 + k2]);           // exp(-i pi (k1 + 16 k2) / N)
}

// Spectra of the response partitions, stored in the split order (k at (k mod 16) N/16 + k div 16, k = N last)
// and scaled by 1/(4N): 1/N for the unnormalised inverse, 1/4 for the halves that multiply_pair leaves out.
// Work groups are persistent: each takes every gridDim.x-th partition and requests the taps of its next one
// before the row transforms of the current one, whose twiddles come from a table in LDS (no global load of
// theirs then stands between the requested taps and the arithmetic).
template <int N>
__device__ inline int load_taps(float2 (&v)[8], const float* __restrict__ h, int rir_len, int p, int tid) {
    constexpr int M = N / 16;
    int first = 0x7fffffff;                          // index of this thread's first non-zero tap
#pragma unroll
    for (int n1 = 7; n1 >= 0; --n1) {                // taps of this partition: [pN, (p+1)N), then N zeros
        const int t = p * N + 2 * (tid + M * n1);
        const float a = t < rir_len ? h[t] : 0.f, b = t + 1 < rir_len ? h[t + 1] : 0.f;
        v[n1] = make_float2(a, b);
        if (b != 0.f) first = t + 1;
        if (a != 0.f) first = t;
    }
    return first;
}

template <int N, int T>
__global__ __launch_bounds__(T) void rir_spectrum_kernel(
    const float* __restrict__ rir, int rir_len, int n_part, int n_work, const float2* __restrict__ tw,
    float2* __restrict__ spec, int* __restrict__ first_tap, double* __restrict__ energy) {
    extern __shared__ float2 buf[];
    __shared__ int wave_first[(T + 63) / 64];
    constexpr int M = N / 16;
    float2* const row_tw = buf + lds_padded_size(N);
    RowTwiddles<M>::template fill<16>(row_tw, tw, threadIdx.x, T);
    const int tid0 = threadIdx.x;
    int work = blockIdx.x;
    if (work >= n_work) return;
    float2 taps[8];
    int first = load_taps<N>(taps, rir + (size_t)(work / n_part) * rir_len, rir_len, work % n_part, tid0);
    __syncthreads();                                 // the twiddle table is complete
    for (;;) {
        int tid = tid0;
        asm volatile("" : "+v"(tid));
        const int r = work / n_part, p = work % n_part;
        // the response is zero before its first non-zero tap, and so is everything convolved with it
        // (a partition's first tap is its group's alone to write, so the array needs no reset, and the response's
        // energy, which the convolution adds to later, gets its zero here)
        for (int off = 32; off > 0; off >>= 1) first = min(first, __shfl_down(first, off, 64));
        if ((tid & 63) == 0) wave_first[tid >> 6] = first;
        float2 v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = i < 8 ? taps[i] : make_float2(0.f, 0.f);
        fft_columns_forward<N>(v, tw, tid);
        fft_columns_store<N, T>(v, buf, tid);
        __syncthreads();
        if (tid == 0) {
            int f = wave_first[0];
            for (int i = 1; i < (T + 63) / 64; ++i) f = min(f, wave_first[i]);
            first_tap[work] = f;
            if (p == 0) energy[r] = 0.0;
        }
        const int next = work + (int)gridDim.x;
        if (next < n_work)
            first = load_taps<N>(taps, rir + (size_t)(next / n_part) * rir_len, rir_len, next % n_part, tid);
        fft_rows_table<N, false>(buf, row_tw, tid);
        __syncthreads();
        asm volatile("" : "+v"(tid));
        float2* out = spec + ((size_t)r * n_part + p) * (N + 1);
        const float scale = 0.25f / (float)N;
        const int k2 = tid % (M / 2), half = tid / (M / 2);
#pragma unroll
        for (int i = 0; i <= 8; ++i) {
            if (i == 8 && tid != 0) break;
            const PairIndex<N> ix(i == 8 ? 0 : half * 8 + i, i == 8 ? M / 2 : k2);
            const float2 A = buf[lds_pad(ix.pos)];
            const float2 B = cconj(buf[lds_pad(ix.pos_partner)]);
            const float2 w = i == 8 ? tw[N + N / 2] : pair_twiddle<N>(tw, half * 8 + i, k2);
            float2 Hk, HNk_conj;
            unpack_pair(A, B, w, Hk, HNk_conj);
            out[ix.pos] = make_float2(Hk.x * scale, Hk.y * scale);
            if (i < 8) out[ix.h_partner] = make_float2(HNk_conj.x * scale, -HNk_conj.y * scale);
        }
        if (next >= n_work) break;
        work = next;
        __syncthreads();                             // every bin is read before the next column store
    }
}

// Z'[k] and Z'[N-k] of the packed output block from Z[k] = A, conj(Z[N-k]) = B and the response
// spectrum: Y = W H on the 2N-point real transform, repacked for the N-point inverse.  The halves of the
// even/odd split (two on the way in, two on the way out) are left out here: the stored response spectrum
// carries the factor 1/4 for them (powers of two: the result is the same bit for bit).
__device__ inline void multiply_pair(float2 A, float2 B, float2 w, float2 Hk, float2 HNk, float2& Zk, float2& ZNk) {
    const float2 E = cadd(A, B);
    const float2 d = csub(A, B);
    const float2 O = make_float2(d.y, -d.x);         // -i (A - B)
    const float2 wO = cmul(w, O);
    const float2 Yk = cmul(Hk, cadd(E, wO));
    const float2 YNk_conj = cmul_conj(csub(E, wO), HNk);
    const float2 Ye = cadd(Yk, YNk_conj);
    const float2 Yo = cmul_conj(csub(Yk, YNk_conj), w);      // conj(w) (Y[k] - conj Y[N-k])
    Zk = make_float2(Ye.x - Yo.y, Ye.y + Yo.x);      // Ye + i Yo
    ZNk = make_float2(Ye.x + Yo.y, Yo.x - Ye.y);     // conj(Ye) + i conj(Yo)
}

// two consecutive samples; only their 4-byte alignment is promised (global accesses of two dwords need no more)
struct __attribute__((aligned(4))) SamplePair { float x, y; };

// Accesses at a per-lane 32-bit byte offset from a wave-uniform base: the address is then a scalar register
// pair plus one vector register, with no 64-bit vector arithmetic per access.
// The place `bytes` behind a wave-uniform base, itself kept in scalar registers: of rows a constant apart the compiler would otherwise
// add the constants to the vector address, two instructions and a wait state per access.  (With that, and without the copies that
// the first wavefront's special case and zeros for no next window cost all: 58 700 vector instructions per wavefront instead of 63 500
// on 256 utterances of 1-16 s with three noises, whose kernel takes its 1.09 million cycles with either (see convolve_inplace_kernel).  Without
// the windows' traffic it would take 4.5 % less, without the stores' 4.2.)
typedef const __attribute__((address_space(1))) char* GlobalRow;
__device__ inline GlobalRow row_at(const void* base, uint32_t bytes) {
    GlobalRow p = (GlobalRow)base + bytes;
    asm("" : "+s"(p));
    return p;
}
typedef float Pair __attribute__((ext_vector_type(2), aligned(4)));
typedef float Quad __attribute__((ext_vector_type(4)));
__device__ inline SamplePair load_pair(const float* base, uint32_t byte_off) {
    return *reinterpret_cast<const SamplePair*>(reinterpret_cast<const char*>(base) + byte_off);
}
__device__ inline float load_sample(const float* base, uint32_t byte_off) {
    return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + byte_off);
}
// element tid of row i, T elements a row
template <int T>
__device__ inline float4 load_quad(const float4* base, int i, int tid) {
    const Quad v = *(const __attribute__((address_space(1))) Quad*)(row_at(base, 16u * T * (uint32_t)i) + 16u * (uint32_t)tid);
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ inline float2 load_bin(const float2* base, uint32_t byte_off) {
    return *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(base) + byte_off);
}

// One block of one (utterance, source): everything here is the same for all lanes.
struct ConvBlock {
    const float* x;          // the source's signal, first sample of the utterance
    const float2* H;         // the response's spectra, partition 0
    float* y;                // reverberated signal, first sample of the utterance
    double* energy;          // E[u][j]
    int len;                 // samples of the utterance
    int first;               // first non-zero tap of the response
    int b;                   // block index: rows [b rows, (b+1) rows) of the utterance are its outputs (see window_row)
};

// Rows: the 2 N samples of a window in sixteenths, row n1 in v[n1] (two samples per thread).  A block's outputs are the
// last `rows` rows of its window, those that no tap reaches from beyond its start, and block b + 1 begins that many rows
// later; so window and outputs of block b are the rows window_row(b, rows) + n1 of the utterance.
__device__ inline int window_row(int b, int rows) { return (b + 1) * rows - 16; }

// The window from row `row`, as the inputs of the column step: v[n1] = (x[2n], x[2n+1]), n = tid + M n1; zeros before the
// utterance and past its end.  The rows before the block's own are all there or, in the first window, all before the utterance,
// and its own never are before it.  Only a window that reaches past the end tests its samples: what a branch loads without looking
// at it stays on its way behind the transform that follows.
template <int N, int ROWS>
__device__ inline void load_window(float2 (&v)[16], const float* x, int len, int row, int tid) {
    constexpr int M = N / 16, kOwn = 16 - ROWS;
    const int from = row * (2 * M);                        // (signals are shorter than 2^30 samples)
    const float* at = x + from;
    const uint32_t lane_off = 8u * (uint32_t)tid;
    auto whole_row = [&](int n1) {
        const Pair s2 = *(const __attribute__((address_space(1))) Pair*)(row_at(at, 8 * M * n1) + lane_off);
        v[n1] = make_float2(s2.x, s2.y);
    };
    if (row >= 0) {
#pragma unroll
        for (int n1 = 0; n1 < kOwn; ++n1) whole_row(n1);
    } else {
#pragma unroll
        for (int n1 = 0; n1 < kOwn; ++n1) v[n1] = make_float2(0.f, 0.f);
    }
    if (from + 32 * M <= len) {
#pragma unroll
        for (int n1 = kOwn; n1 < 16; ++n1) whole_row(n1);
    } else if (ROWS == 8 || len < 2) {
        // addresses are clamped to the utterance's last sample, values past it are zero
#pragma unroll
        for (int n1 = kOwn; n1 < 16; ++n1) {
            const int g = from + 2 * M * n1 + 2 * tid;
            const float x0 = load_sample(x, 4u * (uint32_t)min(g, len - 1));
            const float x1 = load_sample(x, 4u * (uint32_t)min(g + 1, len - 1));
            v[n1] = make_float2(g < len ? x0 : 0.f, g + 1 < len ? x1 : 0.f);
        }
    } else {
        // pairs clamped to the utterance's last, whose second sample is then the one wanted (half as many loads: 96
        // signals with 12001 taps 155 us, not 159)
#pragma unroll
        for (int n1 = kOwn; n1 < 16; ++n1) {
            const SamplePair s2 = load_pair(x, 4u * (uint32_t)min(from + 2 * M * n1 + 2 * tid, len - 2));
            v[n1] = make_float2(s2.x, s2.y);
        }
#pragma unroll
        for (int n1 = kOwn; n1 < 16; ++n1) {
            const int r = from + 2 * M * n1, g = r + 2 * tid;
            if (r + 2 * M <= len) continue;                // (the same for all threads)
            asm volatile("");                              // a branch, not selects in every row: those took 1 us a window
            const float first = g == len - 1 ? v[n1].y : v[n1].x;
            v[n1] = make_float2(g < len ? first : 0.f, g + 1 < len ? v[n1].y : 0.f);
        }
    }
}

// The outputs of a block, v[n1] = (y[n], y[n+1]) in its last rows (see window_row), go to HBM; returns the
// lane's share of the block's energy.  Samples before the response's first non-zero tap are exact zeros
// (the transforms leave rounding noise there, which the power law of the front end would magnify).
template <int N, int ROWS>
__device__ inline float store_block(const float2 (&v)[16], const ConvBlock& c, int tid) {
    constexpr int M = N / 16, kOwn = 16 - ROWS;
    const int row = window_row(c.b, ROWS);
    float* yb = c.y + (int64_t)row * (2 * M);              // (row 0 of the window, which may lie before the utterance)
    const int first = min(c.first, c.len) - row * (2 * M); // first live sample (a silent response has none: its first tap is 2^31 - 1)
    const int left = c.len - row * (2 * M);                // samples up to the utterance's end
    float e[2] = {0.f, 0.f};                               // (chains of sixteen squares, however many rows there are)
    if (left >= 32 * M && first <= kOwn * (2 * M)) {     // whole and live: two-sample stores
        const uint32_t lane_off = 8u * (uint32_t)tid;
#pragma unroll
        for (int n1 = kOwn; n1 < 16; ++n1) {
            const Pair s2 = {v[n1].x, v[n1].y};
            *(__attribute__((address_space(1))) Pair*)(row_at(yb, 8 * M * n1) + lane_off) = s2;
            e[n1 / 8] = fmaf(s2.x, s2.x, fmaf(s2.y, s2.y, e[n1 / 8]));
        }
    } else {
#pragma unroll
        for (int n1 = kOwn; n1 < 16; ++n1) {
            const int g = 2 * tid + 2 * M * n1;
            const float s0 = g >= first ? v[n1].x : 0.f, s1 = g + 1 >= first ? v[n1].y : 0.f;
            if (g < left) { yb[g] = s0; e[n1 / 8] += s0 * s0; }
            if (g + 1 < left) { yb[g + 1] = s1; e[n1 / 8] += s1 * s1; }
        }
    }
    return e[0] + e[1];
}

// A wavefront's energy in lane 0: 1024 squares in fp32, however many rows a block has, the rest in fp64.  (Sixteen squares per
// lane with eight rows, up to 32 with more: then the two halves of the wavefront are joined in fp64.)
template <int ROWS>
__device__ inline double wave_energy(float e) {
    for (int off = ROWS == 8 ? 32 : 16; off > 0; off >>= 1) e += __shfl_down(e, off, 64);
    if (ROWS == 8) return (double)e;
    return (double)e + (double)__uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(e), 32));
}

// Work groups are persistent and take their blocks from the list of all blocks ordered by (utterance, source, block).
// With one partition, the groups that share an L2 (the hardware deals group ids round-robin to the eight XCDs) take one
// contiguous eighth of the list together and go through it side by side, group s of the 32 on blocks s, s + 32, ...: at
// any time they are on a few neighbouring signals, so a response spectrum and the halves that neighbouring windows have
// in common are fetched from HBM once and found in L2 by the other groups, not re-read by one group a whole block later.
// With two partitions (CONTIGUOUS) a group needs consecutive blocks of a signal, so it takes one contiguous range.
// What a block needs of the tables comes by scalar loads (nothing here writes them), asked for a block ahead: by vector loads, where
// it was needed, three round trips to the L2 and the wait for whatever was on its way before them stood between two barriers
// of every block.  (With the scalar addresses, whole calls with one noise: 64 utterances of 4 s with 8000 taps 59.3 -> 57.2 us,
// 256 of 2 s with 16000 105.9 -> 102.8.)
template <class T>
__device__ inline T scalar_load(const T* p) { return *(const __attribute__((address_space(4))) T*)p; }

template <bool CONTIGUOUS>
struct ConvWalk {
    const ConvArgs& a;
    int at, end, step;       // list position, end of the share, stride
    int u, nb, j, b;         // utterance, blocks of each of its sources, source, block
    int64_t start;           // the utterance's first sample
    int len;                 // and its length: utterances are shorter than 2^30 samples (checked on the host)
    // of the next block: utterance, its prefix of the block table, its offsets; and the utterance of the block after that
    int u1, f0, f1, u2;
    int64_t o0, o1;

    __device__ inline explicit ConvWalk(const ConvArgs& args) : a(args) {
        const int total = (int)(a.n_items * a.n_src);      // (the launcher refuses lists of 2^31 blocks or more)
        if (CONTIGUOUS) {
            at = (int)((int64_t)total * blockIdx.x / gridDim.x);
            end = (int)((int64_t)total * (blockIdx.x + 1) / gridDim.x);
            step = 1;
        } else {
            const int teams = gridDim.x % 8 == 0 ? 8 : 1;
            const int team = blockIdx.x % teams, slot = blockIdx.x / teams;
            at = (int)((int64_t)total * team / teams) + slot;
            end = (int)((int64_t)total * (team + 1) / teams);
            step = (int)gridDim.x / teams;
        }
        if (at >= end) return;
        u2 = utterance_at(at);
        ask(u2);
        arrive();
        if (!CONTIGUOUS) u2 = utterance_ahead(step);
    }
    // the utterance that holds a block is the one that holds block at / n_src of the per-source table
    __device__ inline int utterance_at(int block) const {
        return scalar_load(reinterpret_cast<const int*>(a.items) + 2 * (size_t)((unsigned int)block / (unsigned int)a.n_src));
    }
    __device__ inline int utterance_ahead(unsigned int by) const { return utterance_at((int)min((unsigned int)at + by, (unsigned int)end - 1u)); }
    __device__ inline void ask(int of) {
        u1 = of;
        f0 = scalar_load(a.first + of);
        f1 = scalar_load(a.first + of + 1);
        o0 = scalar_load(a.offsets + of);
        o1 = scalar_load(a.offsets + of + 1);
    }
    // what was asked for is where `at` is
    __device__ inline void arrive() {
        u = u1;
        nb = f1 - f0;
        start = o0;
        len = (int)(o1 - o0);
        const unsigned int r = (unsigned int)(at - f0 * a.n_src);
        j = (int)(r / (unsigned int)nb);
        b = (int)r - j * nb;
    }
    __device__ inline bool more() const { return at + step < end; }
    // at the beginning of a block: the next block's tables are asked for
    __device__ inline void look_ahead() {
        if (CONTIGUOUS) return;
        ask(u2);
        u2 = utterance_ahead(2u * (unsigned int)step);
    }
    // to the next block; more() must hold
    __device__ inline void next() {
        at += step;
        if (!CONTIGUOUS) {
            arrive();
        } else if (++b == nb) {
            b = 0;
            if (++j == a.n_src) {
                j = 0;
                do {
                    ask(u + 1);
                    u = u1;
                    nb = f1 - f0;
                } while (nb == 0);
                start = o0;
                len = (int)(o1 - o0);
            }
        }
    }
    // spec_stride: float2 entries per partition
    __device__ inline ConvBlock describe(size_t spec_stride) const {
        ConvBlock c;
        const size_t uj = (size_t)u * a.n_src + j;
        c.len = len;
        c.x = (j == 0 ? a.speech : a.noise + (size_t)(j - 1) * a.total) + start;
        c.H = a.spec + uj * a.n_part * spec_stride;
        c.y = a.reverb + (size_t)j * a.reverb_stride + start;
        c.energy = a.energy + uj;
        c.first = scalar_load(a.first_tap + uj * a.n_part);
        if (CONTIGUOUS) c.first = min(c.first, scalar_load(a.first_tap + uj * a.n_part + 1));
        c.b = b;
        return c;
    }
};

// Responses of up to 2048 taps: transforms in natural order (ROWS as in convolve_inplace_kernel).  While a block's
// inverse transform runs, the inputs of the next block are already on their way from HBM, and the response
// spectrum is requested before the forward row transforms that precede its use: the loads' latency is
// hidden behind arithmetic instead of being paid at either end of a short-lived group.
template <int N, int T, int ROWS>
__global__ __launch_bounds__(T) void convolve_kernel(ConvArgs a, const float2* __restrict__ tw) {
    extern __shared__ float2 buf[];
    __shared__ double red[(T + 63) / 64];
    constexpr int M = N / 16;
    static_assert(T == M, "one thread per column of the split transform");
    // behind the transform buffer: the row transforms' twiddles with their powers, and the two factors of
    // the even/odd split's twiddle exp(-i pi (k1 + 16 k2) / N) = split_lo[k1] split_hi[k2]
    float2* const row_tw = buf + lds_padded_size(N);
    float2* const split_lo = row_tw + RowTwiddles<M>::kEntries;
    float2* const split_hi = split_lo + 16;
    RowTwiddles<M>::template fill<16>(row_tw, tw, threadIdx.x, T);
    for (int i = threadIdx.x; i < 16 + M / 2; i += T) split_lo[i] = i < 16 ? tw[N + i] : tw[N + N / 2 + 1 + (i - 16)];
    // (the first barrier of the loop below comes before any of these is read)
    const int tid0 = threadIdx.x;
    ConvWalk<false> walk(a);
    if (walk.at >= walk.end) return;
    ConvBlock cur = walk.describe(N + 1);
    float2 v[16];
    load_window<N, ROWS>(v, cur.x, cur.len, window_row(cur.b, ROWS), tid0);

    for (;;) {
        // The thread index is made opaque in every round so that twiddle powers and addresses are not
        // hoisted out of the loop, where they would sit on top of the transforms' registers.
        int tid = tid0;
        asm volatile("" : "+v"(tid));
        walk.look_ahead();
        fft_columns_forward<N>(v, tw, tid);
        fft_columns_store<N, T>(v, buf, tid);
        __syncthreads();
        const bool more = walk.more();
        ConvBlock nxt = cur;
        if (more) {
            walk.next();
            nxt = walk.describe(N + 1);
        }

        // the response spectrum of this thread's bins, requested now, used after the row transforms
        float2 hk[8], hn[8];
        {
            const int k2 = tid % (M / 2), half = tid / (M / 2);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const PairIndex<N> ix(half * 8 + i, k2);
                hk[i] = load_bin(cur.H, 8u * (uint32_t)ix.pos);
                hn[i] = load_bin(cur.H, 8u * (uint32_t)ix.h_partner);
            }
        }
        fft_rows_table<N, false>(buf, row_tw, tid);
        __syncthreads();
        // (opaque again: bin positions are recomputed here rather than kept in registers across the transform)
        asm volatile("" : "+v"(tid));
        const int k2 = tid % (M / 2), half = tid / (M / 2);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const PairIndex<N> ix(half * 8 + i, k2);
            const float2 A = buf[lds_pad(ix.pos)];
            const float2 B = cconj(buf[lds_pad(ix.pos_partner)]);
            const float2 wk = cmul(split_lo[half * 8 + i], split_hi[k2]);
            float2 Zk, ZNk;
            multiply_pair(A, B, wk, hk[i], hn[i], Zk, ZNk);
            buf[lds_pad(ix.pos)] = Zk;                     // both positions belong to this thread alone
            if (ix.k != 0) buf[lds_pad(ix.pos_partner)] = ZNk;
        }
        if (tid == 0) {                                    // the bin in the middle, k = N / 2, is its own partner
            const PairIndex<N> ix(0, M / 2);
            const float2 A = buf[lds_pad(ix.pos)];
            const float2 wk = tw[N + N / 2];
            float2 Zk, ZNk;
            multiply_pair(A, cconj(A), wk, cur.H[ix.pos], cur.H[ix.h_partner], Zk, ZNk);
            buf[lds_pad(ix.pos)] = Zk;
        }
        __syncthreads();

        // the next block of the share: its inputs are requested now and arrive during the inverse transform
        asm volatile("" : "+v"(tid));
        if (more) {
            load_window<N, ROWS>(v, nxt.x, nxt.len, window_row(nxt.b, ROWS), tid);
        } else {
            // (assigned on this path too, so that the old inputs do not stay alive in registers up to here; to nothing, since zeros
            // would be written ahead of the branch, in every round)
#pragma unroll
            for (int i = 0; i < 16; ++i) asm volatile("" : "=v"(v[i].x), "=v"(v[i].y));
        }

        fft_rows_table<N, true>(buf, row_tw, tid);
        __syncthreads();
        float2 o[16];
        fft_columns_load<N, T>(o, buf, tid);
        fft_columns_inverse<N>(o, tw, tid);
        const double es = wave_energy<ROWS>(store_block<N, ROWS>(o, cur, tid));
        if ((tid & 63) == 0) red[tid >> 6] = es;
        __syncthreads();                                   // also: every thread has read its columns from LDS
        if (tid == 0) {
            double tot = 0.0;
            for (int i = 0; i < (T + 63) / 64; ++i) tot += red[i];
            atomicAdd(cur.energy, tot);
        }
        if (!more) break;
        cur = nxt;
    }
}

// ---- responses of more than 2048 taps: in-place transforms (fft_inplace.h) ------------------------------------

template <int N>
__global__ void inplace_table_kernel(float* tab) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < InPlace<N>::kFloats) tab[i] = inplace_table_value<N>(i);
}

// the tables that the transforms read from LDS
template <int N>
__device__ inline void copy_tables(float* lds, const float* __restrict__ tab, int tid) {
    for (int i = tid; i < InPlace<N>::kLdsFloats / 4; i += InPlace<N>::T)
        reinterpret_cast<float4*>(lds)[i] = reinterpret_cast<const float4*>(tab)[i];
}

template <int N>
__device__ inline void load_step_d(float4 (&q)[InPlace<N>::Units][InPlace<N>::kDQuads], const float* __restrict__ tab, int tid) {
    using P = InPlace<N>;
    const float4* const d = reinterpret_cast<const float4*>(tab + P::kD0);
#pragma unroll
    for (int i = 0; i < P::Units; ++i)
#pragma unroll
        for (int k = 0; k < P::kDQuads; ++k) q[i][k] = load_quad<P::T>(d, i * P::kDQuads + k, tid);
}

// tangent of pair s (see inplace_table_value)
template <int N>
__device__ inline float pair_tangent(const float4 (&q)[InPlace<N>::kDQuads], int s) {
    if constexpr (InPlace<N>::RD == 4) return s == 0 ? q[1].z : s == 1 ? q[1].w : s == 2 ? q[2].x : q[2].y;
    else return s == 0 ? q[0].z : q[0].w;
}

// Spectra of the response partitions as the products need them: (S, D) per pair of bins (see product_pair), scaled by
// 1/(2N) (1/N for the unnormalised inverse, 1/2 from the product).  Persistent groups, each taking every gridDim.x-th
// partition; the next one's taps are requested before the current one's transform.  Bound by the traffic (N 8 bytes
// written per N taps read).
template <int N>
__global__ __launch_bounds__(InPlace<N>::T) void rir_spectrum_inplace_kernel(
    const float* __restrict__ rir, int rir_len, int n_part, int n_work, const float* __restrict__ tab,
    float4* __restrict__ spec, int* __restrict__ first_tap, double* __restrict__ energy) {
    using P = InPlace<N>;
    constexpr int T = P::T, RD = P::RD;
    extern __shared__ __align__(16) float2 buf[];
    __shared__ int wave_first[T / 64];
    float* const lds_tab = reinterpret_cast<float*>(buf + P::kPadded);
    const int tid0 = threadIdx.x;
    copy_tables<N>(lds_tab, tab, tid0);
    int work = blockIdx.x;
    if (work >= n_work) return;
    float2 taps[8];
    int first = load_taps<N>(taps, rir + (size_t)(work / n_part) * rir_len, rir_len, work % n_part, tid0);
    for (;;) {
        int tid = tid0;
        asm volatile("" : "+v"(tid));
        const int r = work / n_part, p = work % n_part;
        // the response is zero before its first non-zero tap, and so is everything convolved with it
        for (int off = 32; off > 0; off >>= 1) first = min(first, __shfl_down(first, off, 64));
        if ((tid & 63) == 0) wave_first[tid >> 6] = first;
        float2 v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = i < 8 ? taps[i] : make_float2(0.f, 0.f);
        const int next = work + (int)gridDim.x;
        if (next < n_work)
            first = load_taps<N>(taps, rir + (size_t)(next / n_part) * rir_len, rir_len, next % n_part, tid);
        inplace_forward_ab<N>(v, buf, lds_tab, tid);
        inplace_forward_c<N>(v, buf, lds_tab, tid);
        __syncthreads();
        if (tid == 0) {
            int f = wave_first[0];
            for (int i = 1; i < T / 64; ++i) f = min(f, wave_first[i]);
            first_tap[work] = f;
            if (p == 0) energy[r] = 0.0;
        }
        asm volatile("" : "+v"(tid));
        float4 q[P::Units][P::kDQuads];
        load_step_d<N>(q, tab, tid);
        float4* out = spec + (size_t)work * inplace_spectrum_entries<N>();
        const float scale = 0.5f / (float)N;
#pragma unroll
        for (int i = 0; i < P::Units; ++i) {
            int pos_a, pos_b;
            P::unit(tid, i, pos_a, pos_b);
            float2 a[RD], b[RD], mid = make_float2(0.f, 0.f);
            if (i == 0) inplace_step_d<N, true>(a, b, mid, buf, pos_a, pos_b, q[i], tid == 0);
            else inplace_step_d<N, false>(a, b, mid, buf, pos_a, pos_b, q[i], false);
#pragma unroll
            for (int s = 0; s < RD; ++s) {
                // E = A + B is H[k] + conj H[N-k]; -i w (A - B) is their difference, w = c (1 + i tau)
                const float2 A = a[s], B = cconj(b[RD - 1 - s]), d = csub(A, B);
                const float tau = pair_tangent<N>(q[i], s);
                const float2 D = tilt<false>(make_float2(d.y, -d.x), tau);
                const float cc = scale / fmaf(tau, tau, 1.f);                   // c^2
                out[(i * RD + s) * T + tid] = make_float4(scale * (A.x + B.x), scale * (A.y + B.y), cc * D.x, cc * D.y);
            }
            if (i == 0 && tid == 0) out[N / 2] = make_float4(2.f * scale * mid.x, 2.f * scale * mid.y, 0.f, 0.f);
        }
        if (next >= n_work) break;
        work = next;
        __syncthreads();                             // every value is read before the next step A
    }
}

// What bounds it: one group of sixteen wavefronts fills a compute unit (the block is 128 KB of LDS) and its barriers keep the
// wavefronts in step.  On 256 utterances of 1-16 s with three noises the vector units are busy 0.86 of the time and the LDS 0.48, so the
// two overlap; a wavefront issues for 0.30 of its time, waits to issue for 0.31 and waits for memory, LDS or a barrier for 0.38.  Vector issue
// alone is not the limit: with 7.6 % fewer instructions (0.86 busy instead of 0.93) it takes the same cycles.  What does limit it is
// not known.  About 1680 vector instructions per thread and block, all told.  Against transforms in natural
// order, with the product from LDS between them, this one makes 12 passes over the block in LDS instead of 16, has four
// barriers per block instead of five, and two thirds of the vector instructions: twiddles
// folded into the butterflies' additions, the product in twenty multiply-adds per pair from the registers that the last
// forward and the first inverse step share.
// While a block's inverse transform runs, the inputs of the next block are already on their way from HBM; the response
// spectrum is requested before the step that precedes its use.
// MULTI: the response has two partitions.  Block b is then the inverse transform of H_0 W_b + H_1 W_{b-1}; W_{b-1} is the
// window spectrum of the block this group finished just before, and each thread keeps its sixteen bins of it in
// registers, so a block still costs one forward and one inverse transform (plus one forward transform at the start of a
// group's share).  The kept spectrum takes the registers that the single-partition kernel spends on inputs requested
// ahead of time; they are then loaded where they are used.
// ROWS: a block's rows (the last step's other outputs are never formed).
template <int N, bool MULTI, int ROWS>
__global__ __launch_bounds__(InPlace<N>::T) void convolve_inplace_kernel(ConvArgs a, const float* __restrict__ tab) {
    using P = InPlace<N>;
    constexpr int T = P::T, RD = P::RD;
    constexpr bool AHEAD = !MULTI;
    constexpr size_t kEntries = inplace_spectrum_entries<N>();
    extern __shared__ __align__(16) float2 buf[];
    __shared__ double red[2][T / 64];                      // energies per wavefront of this block and the one before
    float* const lds_tab = reinterpret_cast<float*>(buf + P::kPadded);
    const int tid0 = threadIdx.x;
    copy_tables<N>(lds_tab, tab, tid0);                    // (a barrier of the loop below comes before these are read)
    ConvWalk<MULTI> walk(a);
    if (walk.at >= walk.end) return;
    ConvBlock cur = walk.describe(2 * kEntries);

    float2 v[16];
    float2 prev_a[MULTI ? 8 : 1], prev_b[MULTI ? 8 : 1], prev_mid = make_float2(0.f, 0.f);
    bool have_prev = false;         // prev_* hold the window spectrum of block cur.b - 1 of this signal
    if (MULTI) {
#pragma unroll
        for (int i = 0; i < 8; ++i) prev_a[i] = prev_b[i] = make_float2(0.f, 0.f);
        have_prev = cur.b == 0;     // the window before the first block is all zeros, and so is its spectrum
    }
    if (AHEAD) load_window<N, ROWS>(v, cur.x, cur.len, window_row(cur.b, ROWS), tid0);
    double* done_energy = nullptr;  // where the energies in red[parity ^ 1] belong
    int parity = 0;
    // the energy of the block before this one
    auto flush_energy = [&](int tid) {
        if (tid == 0 && done_energy) {
            double tot = 0.0;
            for (int i = 0; i < T / 64; ++i) tot += red[parity ^ 1][i];
            atomicAdd(done_energy, tot);
        }
    };

    for (;;) {
        // The thread index is made opaque in every round so that addresses are not hoisted out of the loop, where they
        // would sit on top of the transforms' registers.
        int tid = tid0;
        asm volatile("" : "+v"(tid));
        const bool warm_up = MULTI && !have_prev;          // this pass only produces the spectrum of window b - 1
        if (!AHEAD) load_window<N, ROWS>(v, cur.x, cur.len, window_row(warm_up ? cur.b - 1 : cur.b, ROWS), tid);

        walk.look_ahead();
        inplace_forward_ab<N>(v, buf, lds_tab, tid);
        flush_energy(tid);
        done_energy = nullptr;
        const bool more = !warm_up && walk.more();
        ConvBlock nxt = cur;
        if (more) {
            walk.next();
            nxt = walk.describe(2 * kEntries);
        }
        const float4 middle = reinterpret_cast<const float4*>(cur.H)[N / 2];     // (used by thread 0 alone, which it must not keep waiting)
        float4 middle1 = middle;
        if (MULTI) middle1 = reinterpret_cast<const float4*>(cur.H)[kEntries + N / 2];
        float4 q[P::Units][P::kDQuads];
        load_step_d<N>(q, tab, tid);
        inplace_forward_c<N>(v, buf, lds_tab, tid);
        asm volatile("" : "+v"(tid));
        const float4* H = reinterpret_cast<const float4*>(cur.H);
        float4 sd[AHEAD ? 8 : 1];
        if (AHEAD) {
#pragma unroll
            for (int i = 0; i < 8; ++i) sd[i] = load_quad<T>(H, i, tid);
        }
        __syncthreads();

        // (thread 0's unit 0 is not like the others: the first wavefront has code of its own for it, which the others neither run
        // nor make room for)
        auto unit = [&](auto first, int i) {
            constexpr bool FIRST = decltype(first)::value;
            int pos_a, pos_b;
            P::unit(tid, i, pos_a, pos_b);
            float2 x[RD], y[RD], mid = make_float2(0.f, 0.f);
            const bool thread0 = FIRST && tid == 0;
            inplace_step_d<N, FIRST>(x, y, mid, buf, pos_a, pos_b, q[i], thread0);
            if (warm_up) {
#pragma unroll
                for (int s = 0; s < RD; ++s) {
                    prev_a[MULTI ? i * RD + s : 0] = x[s];
                    prev_b[MULTI ? i * RD + s : 0] = cconj(y[RD - 1 - s]);
                }
                if (FIRST) prev_mid = mid;
                return;
            }
#pragma unroll
            for (int s = 0; s < RD; ++s) {
                const float2 A = x[s], B = cconj(y[RD - 1 - s]);
                const float tau = pair_tangent<N>(q[i], s);
                float2 zk, zn;
                product_pair<false>(A, B, AHEAD ? sd[AHEAD ? i * RD + s : 0] : load_quad<T>(H, i * RD + s, tid), tau, zk, zn);
                if (MULTI) {
                    float2& pa = prev_a[MULTI ? i * RD + s : 0];
                    float2& pb = prev_b[MULTI ? i * RD + s : 0];
                    product_pair<true>(pa, pb, load_quad<T>(H + kEntries, i * RD + s, tid), tau, zk, zn);
                    pa = A;
                    pb = B;
                }
                x[s] = zk;
                y[RD - 1 - s] = cconj(zn);
            }
            if (thread0) {                                 // the bin in the middle
                float2 z = cmul(mid, make_float2(middle.x, middle.y));
                if (MULTI) {
                    z = cadd(z, cmul(prev_mid, make_float2(middle1.x, middle1.y)));
                    prev_mid = mid;
                }
                mid = z;
            }
            inplace_step_d_inverse<N, FIRST>(x, y, mid, buf, pos_a, pos_b, thread0);
        };
        if (__builtin_amdgcn_readfirstlane(tid) == 0) unit(std::true_type{}, 0);
        else unit(std::false_type{}, 0);
#pragma unroll
        for (int i = 1; i < P::Units; ++i) unit(std::false_type{}, i);
        if (warm_up) {
            have_prev = true;
            __syncthreads();                               // all values are read before the next step A
            continue;
        }
        asm volatile("" : "+v"(tid));
        float4 wa[3];                                      // the last step's factors, requested before the next inputs
#pragma unroll
        for (int i = 0; i < 3; ++i) wa[i] = load_quad<T>(reinterpret_cast<const float4*>(tab + P::kA0), i, tid);
        __syncthreads();

        // the next block of the share: its inputs are requested now and arrive during the inverse transform
        if (AHEAD && more) {
            load_window<N, ROWS>(v, nxt.x, nxt.len, window_row(nxt.b, ROWS), tid);
        } else if (AHEAD) {
            // (assigned on this path too, so that the old inputs do not stay alive in registers up to here; to nothing, since zeros
            // would be written ahead of the branch, in every round)
#pragma unroll
            for (int i = 0; i < 16; ++i) asm volatile("" : "=v"(v[i].x), "=v"(v[i].y));
        }

        float2 o[16];
        const Tw16Short w{{wa[0].x, wa[0].y, wa[0].z, wa[0].w, wa[1].x, wa[1].y}, {wa[1].z, wa[1].w, wa[2].x, wa[2].y, wa[2].z, wa[2].w}};
        inplace_inverse<N>(o, buf, lds_tab, tid, w);
        const double es = wave_energy<ROWS>(store_block<N, ROWS>(o, cur, tid));
        if ((tid & 63) == 0) red[parity][tid >> 6] = es;
        done_energy = cur.energy;
        parity ^= 1;
        if (!more) break;
        if (MULTI && nxt.b == 0) {                         // a new signal starts: nothing precedes its first window
#pragma unroll
            for (int i = 0; i < 8; ++i) prev_a[i] = prev_b[i] = make_float2(0.f, 0.f);
            prev_mid = make_float2(0.f, 0.f);
        }
        cur = nxt;
    }
    __syncthreads();
    flush_energy(tid0);
}

// One thread per (utterance, noise source), for callers that want the gains but not the mixture.
__global__ void gain_kernel(int n_utt, int n_src, const double* __restrict__ energy, const float* __restrict__ snr_db,
                            float* __restrict__ gains_out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int n_noise = n_src - 1;
    if (i >= n_utt * n_noise) return;
    const int u = i / n_noise;
    gains_out[i] = snr_gain(energy + (size_t)u * n_src, i - u * n_noise, snr_db[i]);
}

// mixed = y_0 + sum_j g_j y_j, kMixChunk samples of one utterance per work group, four consecutive ones per thread and
// round.  The group forms the utterance's gains itself, while its first samples are on their way (a launch for the
// gains took 5 us); the first group of an utterance also writes them out.  Bound by HBM.
constexpr int kMixThreads = 256, kMixRounds = 4, kMixChunk = kMixThreads * 4 * kMixRounds;
struct __attribute__((aligned(4))) SampleQuad { float x, y, z, w; };
__global__ __launch_bounds__(kMixThreads) void mix_kernel(
    const int64_t* __restrict__ offsets, int64_t stride, int n_src, const float* __restrict__ reverb,
    const double* __restrict__ energy, const float* __restrict__ snr_db, float* __restrict__ mixed,
    float* __restrict__ gains_out) {
    __shared__ float gains[AUG_MAX_NOISE];
    const int u = blockIdx.y;
    const int64_t start = offsets[u];
    const int64_t len = offsets[u + 1] - start;
    const int64_t first = (int64_t)blockIdx.x * kMixChunk;
    if (first >= len && blockIdx.x > 0) return;
    const float* y0 = reverb + start;
    float* out = mixed + start;
    auto load = [&](const float* y, int64_t n) {
        if (n + 4 <= len) return *reinterpret_cast<const SampleQuad*>(y + n);
        return SampleQuad{n < len ? y[n] : 0.f, n + 1 < len ? y[n + 1] : 0.f, n + 2 < len ? y[n + 2] : 0.f, 0.f};
    };
    SampleQuad acc[kMixRounds];
#pragma unroll
    for (int i = 0; i < kMixRounds; ++i) acc[i] = load(y0, first + 4 * ((int64_t)i * kMixThreads + threadIdx.x));
    if ((int)threadIdx.x < n_src - 1) {
        const int j = threadIdx.x;
        const float g = snr_gain(energy + (size_t)u * n_src, j, snr_db[(size_t)u * (n_src - 1) + j]);
        gains[j] = g;
        if (gains_out && blockIdx.x == 0) gains_out[(size_t)u * (n_src - 1) + j] = g;
    }
    __syncthreads();
    for (int j = 1; j < n_src; ++j) {
        const float g = gains[j - 1];
        const float* y = y0 + (size_t)j * stride;
        SampleQuad e[kMixRounds];
#pragma unroll
        for (int i = 0; i < kMixRounds; ++i) e[i] = load(y, first + 4 * ((int64_t)i * kMixThreads + threadIdx.x));
#pragma unroll
        for (int i = 0; i < kMixRounds; ++i) {
            acc[i].x += g * e[i].x;
            acc[i].y += g * e[i].y;
            acc[i].z += g * e[i].z;
            acc[i].w += g * e[i].w;
        }
    }
#pragma unroll
    for (int i = 0; i < kMixRounds; ++i) {
        const int64_t n = first + 4 * ((int64_t)i * kMixThreads + threadIdx.x);
        if (n + 4 <= len) {
            *reinterpret_cast<SampleQuad*>(out + n) = acc[i];
        } else {
            if (n < len) out[n] = acc[i].x;
            if (n + 1 < len) out[n + 1] = acc[i].y;
            if (n + 2 < len) out[n + 2] = acc[i].z;
        }
    }
}

constexpr bool in_place(int n) { return n >= 4096; }

// As many persistent groups of T threads as the chip holds at once: per compute unit, what the 160 KB of LDS and
// sixteen wavefronts (128 registers each) allow.
int64_t groups_at_once(int n_cu, size_t lds, int threads) {
    const int by_lds = (int)((160 * 1024) / (lds + 256));
    const int by_waves = 16 / ((threads + 63) / 64);
    const int per_cu = by_lds < 1 ? 1 : (by_lds < by_waves ? by_lds : by_waves);
    return (int64_t)n_cu * per_cu;
}

// (launched by address, not called through the pointer: the call form is what undefined-behaviour
// sanitizers of the host code instrument, and with them it was seen to launch nothing)
hipError_t launch_groups(hipStream_t s, const void* kernel, int n_cu, int64_t work, int threads, size_t lds, void** args) {
    hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    int64_t groups = groups_at_once(n_cu, lds, threads);
    if (groups > work) groups = work;
    return hipLaunchKernel(kernel, dim3((unsigned)groups), dim3(threads), args, lds, s);
}

template <int N>
size_t inplace_lds() { return sizeof(float2) * InPlace<N>::kPadded + sizeof(float) * InPlace<N>::kLdsFloats; }

template <int N>
hipError_t spectrum_n(hipStream_t s, int n_rir, const float* rir, int rir_len, const float2* tw,
                      float2* spec, int* first_tap, double* energy, int n_cu) {
    int n_part = (rir_len + N - 1) / N;
    int n_work = n_rir * n_part;
    void* args[] = {&rir, &rir_len, &n_part, &n_work, &tw, &spec, &first_tap, &energy};
    if constexpr (in_place(N)) {
        return launch_groups(s, reinterpret_cast<const void*>(&rir_spectrum_inplace_kernel<N>), n_cu, n_work, InPlace<N>::T,
                             inplace_lds<N>(), args);
    } else {
        constexpr int T = conv_threads(N);
        return launch_groups(s, reinterpret_cast<const void*>(&rir_spectrum_kernel<N, T>), n_cu, n_work, T,
                             sizeof(float2) * (lds_padded_size(N) + RowTwiddles<N / 16>::kEntries), args);
    }
}

// The kernel for blocks of that many rows.  (One for any number tested every row and formed all sixteen: calls of a few signals
// took up to 2 us longer with it, one signal of 8000 samples 18.9 -> 20.5 us with 1100 taps and 27.9 -> 29.2 with 12001, 32
// of 16000 with 3300 taps 23.3 -> 24.1.)  A response longer than half a transform leaves
// at most twelve rows; shorter ones exist at the smallest transform only.
template <int N, int ROWS = 8>
const void* convolve_of_rows(int rows) {
    if (rows == ROWS) {
        if constexpr (in_place(N)) return reinterpret_cast<const void*>(&convolve_inplace_kernel<N, false, ROWS>);
        else return reinterpret_cast<const void*>(&convolve_kernel<N, conv_threads(N), ROWS>);
    }
    if constexpr (ROWS < (N == 1024 ? 16 : 12)) return convolve_of_rows<N, ROWS + 1>(rows);
    else return nullptr;
}

template <int N>
hipError_t convolve_n(hipStream_t s, const float2* tw, const ConvArgs& a, int n_cu) {
    const int64_t total = a.n_items * a.n_src;
    if (total > 0x7fffffffLL) return hipErrorInvalidValue;
    ConvArgs by_value = a;
    void* args[] = {&by_value, &tw};
    const void* k = convolve_of_rows<N>(a.rows);
    if constexpr (in_place(N)) {
        // responses longer than one partition exist only at the largest transform size (conv_fft_size)
        if (a.n_part > 1) {
            if (N != 16384 || a.n_part != 2 || a.rows != 8) return hipErrorInvalidValue;
            k = reinterpret_cast<const void*>(&convolve_inplace_kernel<16384, true, 8>);
        }
        if (!k) return hipErrorInvalidValue;
        return launch_groups(s, k, n_cu, total, InPlace<N>::T, inplace_lds<N>(), args);
    } else {
        if (a.n_part > 1 || !k) return hipErrorInvalidValue;
        return launch_groups(s, k, n_cu, total, conv_threads(N),
                             sizeof(float2) * (lds_padded_size(N) + RowTwiddles<N / 16>::kEntries + 16 + N / 32), args);
    }
}

}  // namespace

int conv_fft_size(int rir_len) {
    int n = 1024;                       // at least one full wave of sixteen-point butterflies
    while (n < rir_len && n < 16384) n <<= 1;
    return n;
}

int conv_table_entries(int n) {
    switch (n) {
        case 4096: return InPlace<4096>::kFloats / 2;
        case 8192: return InPlace<8192>::kFloats / 2;
        case 16384: return InPlace<16384>::kFloats / 2;
        default: return twiddle_count(n);
    }
}
size_t conv_spectrum_entries(int n) { return in_place(n) ? (size_t)n + 2 : (size_t)n + 1; }

hipError_t launch_conv_table(hipStream_t s, int n, float2* tab) {
    float* f = reinterpret_cast<float*>(tab);
    const dim3 grid((unsigned)((2 * conv_table_entries(n) + 255) / 256)), block(256);
    switch (n) {
        case 4096: inplace_table_kernel<4096><<<grid, block, 0, s>>>(f); break;
        case 8192: inplace_table_kernel<8192><<<grid, block, 0, s>>>(f); break;
        case 16384: inplace_table_kernel<16384><<<grid, block, 0, s>>>(f); break;
        default: return launch_twiddle(s, n, tab);
    }
    return hipGetLastError();
}

int twiddle_entries(int n) { return twiddle_count(n); }

hipError_t launch_twiddle(hipStream_t s, int n, float2* tw) {
    const int count = twiddle_count(n);
    twiddle_kernel<<<dim3((count + 255) / 256), dim3(256), 0, s>>>(n, tw);
    return hipGetLastError();
}

#define AUG_FFT_DISPATCH(n, CALL)                                  \
    switch (n) {                                                   \
        case 1024: return CALL(1024);                              \
        case 2048: return CALL(2048);                              \
        case 4096: return CALL(4096);                              \
        case 8192: return CALL(8192);                              \
        case 16384: return CALL(16384);                            \
        default: return hipErrorInvalidValue;                      \
    }

hipError_t launch_rir_spectrum(hipStream_t s, int n_rir, const float* rir, int rir_len, int fft_n,
                               const float2* twiddle, float2* spec, int* first_tap, double* energy, int n_cu) {
    if (n_rir <= 0) return hipSuccess;
#define CALL(NN) spectrum_n<NN>(s, n_rir, rir, rir_len, twiddle, spec, first_tap, energy, n_cu)
    AUG_FFT_DISPATCH(fft_n, CALL)
#undef CALL
}

hipError_t launch_convolve(hipStream_t s, int fft_n, const float2* twiddle, const ConvArgs& a, int n_cu) {
    if (a.n_items <= 0) return hipSuccess;
#define CALL(NN) convolve_n<NN>(s, twiddle, a, n_cu)
    AUG_FFT_DISPATCH(fft_n, CALL)
#undef CALL
}

hipError_t launch_gains(hipStream_t s, int n_utt, int n_src, const double* energy, const float* snr_db, float* gains_out) {
    const int n = n_utt * (n_src - 1);
    if (n <= 0) return hipSuccess;
    gain_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s>>>(n_utt, n_src, energy, snr_db, gains_out);
    return hipGetLastError();
}

hipError_t launch_mix(hipStream_t s, int n_utt, const int64_t* d_offsets, int64_t stride, int n_src, const float* reverb,
                      const double* energy, const float* snr_db, float* mixed_out, float* gains_out, int64_t max_len) {
    if (n_utt <= 0) return hipSuccess;
    int64_t chunks = (max_len + kMixChunk - 1) / kMixChunk;
    if (chunks < 1) chunks = 1;
    mix_kernel<<<dim3((unsigned)chunks, (unsigned)n_utt), dim3(kMixThreads), 0, s>>>(
        d_offsets, stride, n_src, reverb, energy, snr_db, mixed_out, gains_out);
    return hipGetLastError();
}

}  // namespace aug
