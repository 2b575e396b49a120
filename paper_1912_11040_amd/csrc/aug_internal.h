// Internal declarations shared by the library's translation units (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <utility>
#include <vector>

#include "aug.h"

namespace aug {

// A grow-only device buffer owned by the context.
struct DeviceBuffer {
    void* ptr = nullptr;
    size_t bytes = 0;
    hipError_t reserve(size_t need);
    void release();
    template <class T> T* as() const { return static_cast<T*>(ptr); }
};

// The framing of a front-end call, the values of an output row and the number of work groups that the chip runs at once of its kernel.
struct Framing {
    int win = 0, hop = 0, width = 0, slots = 0;
    bool operator==(const Framing& o) const { return win == o.win && hop == o.hop && width == o.width && slots == o.slots; }
};

// How the front end's work is shared among its groups.  An utterance's frames are cut into units of 16 << shift, its rows without
// frames into units of 1 << lg_rows + shift, some 8000 to 16000 values (an utterance with rows has one at least), numbered in the utterances' order; group g takes those from
// g per_group + min(g, longer), per_group of them, the first `longer` groups one more.  The rows without frames, which are set to zero,
// go with all of their utterance's units evenly.  (Counted by their frames alone, four empty utterances of 20000 rows each were four
// groups' work, 457 us instead of 50.)
struct FrameShares {
    int n_groups = 0, per_group = 0, longer = 0, shift = 0, lg_rows = 0;
};
constexpr int kUnitFrames = 16, kLgUnitFrames = 4;       // the frames that a group of the front end has in flight
static_assert(1 << kLgUnitFrames == kUnitFrames, "units");
inline int unit_lg_rows(int width) {
    int lg = 13;
    while (width > 1) width >>= 1, --lg;
    return lg;
}
inline int64_t frame_units(int64_t len, int64_t rows, const Framing& f, int shift) {
    if (rows <= 0) return 0;
    const int64_t frames = len < f.win ? 0 : 1 + (len - f.win) / f.hop;
    const int64_t units = ((frames + (((int64_t)kUnitFrames << shift) - 1)) >> (kLgUnitFrames + shift)) + ((rows - frames) >> (unit_lg_rows(f.width) + shift));
    return units > 0 ? units : 1;
}

// The batch's units shared out evenly, in consecutive stretches, among as many groups as run at once (fewer if there are not
// that many units), so that a group meets few utterances and all end together.  In groups of so many rows of one utterance,
// as many as made eight rounds, the last round was half empty and every group set up an utterance's tables for four passes of
// sixteen frames: 256 padded utterances of 1-16 s 131 us, 99 so.  Shares of more than kUnitsPerGroup units are cut further: with
// 200 each, 4096 utterances of 8 s waited for the slowest groups (1151 us; in twice as many 1132, four times 1097, eight times
// 1100), while with 13 each every set-up counts (110, 115, 124, 138 us).  `limit`: no more units than that.
constexpr int kUnitsPerGroup = 40;
inline FrameShares share_frames(int n_utt, const int64_t* offsets, const int64_t* frame_offsets, const Framing& f, int64_t limit = 1 << 30) {
    FrameShares s;
    s.lg_rows = unit_lg_rows(f.width);
    for (;; ++s.shift) {                                     // (units of more frames where 31 bits would not number them)
        int64_t units = 0;
        for (int u = 0; u < n_utt; ++u) units += frame_units(offsets[u + 1] - offsets[u], frame_offsets[u + 1] - frame_offsets[u], f, s.shift);
        if (units >= limit) continue;
        const int64_t per_round = (int64_t)f.slots * kUnitsPerGroup, groups = f.slots * (units < per_round ? 1 : units / per_round);
        s.n_groups = (int)(units < groups ? units : groups);
        if (s.n_groups > 0) {
            s.per_group = (int)(units / s.n_groups);
            s.longer = (int)(units % s.n_groups);
        }
        return s;
    }
}

// Host-side description of how the packed utterances are cut into work items;
// rebuilt only when the offsets of a call differ from the cached ones.
struct Packing {
    std::vector<int64_t> offsets;        // n_utt + 1
    std::vector<int64_t> frame_offsets;  // n_utt + 1 (empty if not a front-end call)
    int conv_block = 0;                  // output samples per convolution block the tables were built for
    int64_t n_conv_blocks = 0;           // sum over utterances of ceil(len / conv_block)
    // How the front end's work on these offsets is shared out, one table of beginnings on the device for each framing asked for:
    // a call that takes other slots (with the mixture on the fly or not, another feature) must not rewrite the table that
    // a captured call reads.
    struct Framed {
        Framing framing;
        FrameShares shares;
    };
    static constexpr int kTables = 16;   // (with more framings of one batch than this the oldest table goes)
    Framed framed[kTables];              // unused ones have no framing
    int next_table = 0;                  // the next to be made
    int table = 0;                       // that of the present call
    const FrameShares& shares() const { return framed[table].shares; }
};

// Pinned host staging for the offset arrays: a call writes its arrays into the next slot and the packing kernel
// reads them there, so the caller's arrays are free when the call returns and nothing waits for the stream.
// A slot is reused only after the kernel that read it has finished: one event for every kPerEvent slots in
// turn, recorded behind the last of them and waited for before the first is written again.
struct HostRing {
    static constexpr int kSlots = 16, kPerEvent = 4;
    unsigned char* host = nullptr;       // kSlots slots of `bytes` each
    unsigned char* device = nullptr;     // the same memory as the device addresses it
    hipEvent_t done[kSlots / kPerEvent] = {};
    size_t bytes = 0;
    int next = 0;
};

// Device copies of a batch's offsets and its item tables, from the arrays that the host has left in pinned
// memory: offsets, frame offsets and the exclusive prefix sums of the items per utterance (blocks of the
// convolution; units of the front end, see FrameShares), n_utt + 1 entries each.  A null source is skipped.
struct PackArgs {
    int n_utt;
    FrameShares shares;
    const int64_t* offsets;          // pinned host memory, as the device sees it
    const int64_t* frame_offsets;
    const int* conv_first;
    const int* frame_first;
    int64_t* d_offsets;              // device
    int64_t* d_frame_offsets;
    int* d_conv_first;
    int2* conv_items;                // (utterance, block)
    int2* frame_items;               // (utterance, unit of it) at which a group begins
};
// Per-utterance (band, weight) table of the warped mel bank followed by how the filters are dealt to the matrix
// cores: tab float2 [n_utt][mel_table_stride(nfft)].  mel_edges fills in what depends on the configuration only.
struct MelTableArgs {
    double edges[AUG_MAX_MEL + 2];   // band edges, Hz
    float mel_lo, inv_step;          // f_lo in mel, 1 / spacing of the edges in mel
    aug_frontend_cfg cfg;
    const float* alpha;
    float2* tab;
};
}  // namespace aug

struct aug_ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    std::string last_error;

    // device copies of the host offset arrays and the work-item tables derived from them
    aug::Packing packing;
    aug::DeviceBuffer d_offsets;         // int64 [n_utt+1]
    aug::DeviceBuffer d_frame_offsets;   // int64 [n_utt+1]
    aug::DeviceBuffer d_conv_items;      // int2 [n_conv_blocks]: (utterance, block)
    aug::DeviceBuffer d_frame_items[aug::Packing::kTables];      // int2 [shares.n_groups]: (utterance, unit of it) at which a group begins
    aug::DeviceBuffer d_conv_first;      // int [n_utt+1]: blocks of the utterances before u
    aug::HostRing ring;
    unsigned char* scratch = nullptr;    // this device's copy of the library's static scratch array

    // image-method work list
    int n_cu = 0;                        // compute units of the device
    aug::DeviceBuffer rir_items;         // Item [n_rir * items_per_response]
    aug::DeviceBuffer rir_ctrl;          // int [rir_ctrl_ints()]: item count, next item, class counters
    aug::DeviceBuffer visits;            // one 64-bit counter (aug_rir_visited_images)

    // intermediate results
    aug::DeviceBuffer rir;               // float [n_rir][rir_len]            (pipeline only)
    aug::DeviceBuffer rir_spec;          // float2 [n_rir][n_part][conv_spectrum_entries]
    aug::DeviceBuffer reverb;            // float [1+n_noise][total rounded up to even]
    aug::DeviceBuffer energy;            // double [n_utt][1+n_noise]: energies of the reverberated signals
    aug::DeviceBuffer first_tap;         // int [n_utt][1+n_noise][n_part]
    aug::DeviceBuffer mel_tab;           // float2 [n_utt][mel_table_stride(nfft)]: (band, weight) per bin, then the plan
    aug::DeviceBuffer mel_lanes;         // float [mel_lane_floats()], filled once
    aug::DeviceBuffer twiddle[16];       // per log2(n): float2 [twiddle_entries(n)] FFT twiddles
    aug::DeviceBuffer conv_tab[16];      // per log2(n): float2 [conv_table_entries(n)] tables of the convolution
    aug::DeviceBuffer window;            // float [win]
    aug::DeviceBuffer dct;               // float [n_ceps][n_mel]
    int dct_ceps = 0, dct_mel = 0;       // shape the table was built for
    aug::DeviceBuffer vtlp_tab;          // float2 [n_utt][vtlp_table_entries()]: (source bin, weight) per output bin
    int window_n = 0;
    aug::MelTableArgs mel_args{};        // band edges of the last front-end configuration seen
    bool have_mel_args = false;
    bool have_lanes = false;             // mel_lanes is filled

    // stage timing: events recorded in stream order, each tagged with the stage it ends (-1 = a start mark)
    bool profiling = false;
    std::vector<std::pair<hipEvent_t, int>> marks;
};

namespace aug {

// ---- kernels' host launchers (each checks nothing; arguments are validated by the API layer) ----

// Image-method impulse responses.  launch_rir_plan cuts every response into items (tap ranges of
// about equal image count) ordered heaviest first and resets ctrl (item count,
// next item, class counters: rir_ctrl_ints() ints); `items` needs room for 2 n_rir rir_items_per_response items;
// launch_rir then runs n_groups persistent work groups over the items (restart: once more over the
// same plan), writing either
// rir_out float [n_rir][rir_len] or, if rir_out is null, tap counts cnt_out int32 [n_rir][rir_len].
// With `visits` (device, one 64-bit counter, zero on entry) the amplitude pass runs in a measuring
// instantiation that adds the number of images it walked.
// Response r is that of geometry row r, or, with mics (float [n_rir][3]), of row r / n_mic with its microphone replaced
// by mics[r].
struct Rooms {
    const float* geom;           // device, float [n_rir / n_mic][10]
    const float* mics;           // device, may be null
    int n_mic;                   // used with mics
};
int rir_items_per_response(int rir_len);
size_t rir_item_bytes();
int rir_ctrl_ints();
hipError_t launch_rir_plan(hipStream_t s, int n_groups, int n_rir, const Rooms& rooms, int rir_len, double fs_over_c,
                           void* items, int* ctrl);
hipError_t launch_rir(hipStream_t s, int n_groups, int n_rir, const Rooms& rooms, int rir_len, double fs_over_c,
                      const void* items, int* ctrl, float* rir_out, int32_t* cnt_out,
                      bool restart, unsigned long long* visits = nullptr);


// Smallest transform the convolution kernels are built for that holds a response (16384 points if none does).
int conv_fft_size(int rir_len);

// Size of the convolution's transforms (N complex points) and outputs per block, in rows of N / 8 samples: of the sixteen
// rows of a window those that no tap reaches from beyond its start, 8 .. 16.  (12001 taps at N = 16384 leave ten: three sources
// of 96 signals took 139 us with eight rows at every length, 120 now; 14000 leave nine: three sources of 96 signals of up to 100000
// samples 118 us with eight, 108 so, 256 of 64000 alone 197 and 188, 1000 of 9000 no difference.)
// Every number of rows has a kernel of its own (see convolve_of_rows).
// Size and rows follow from the response's length alone, so that a signal's reverberation does not depend on the batch it is in, and
// the window is the smallest that there is: a transform spreads its rounding error over its whole window, at the level of the
// window's loudest part.  (The largest transform at every length that fills the chip took 256 signals of 64000 samples with 4096
// taps from 189 us to 158, and put 1.8e-7 of the loud part where 3.7e-8 had been in a pause 8000 samples behind it.)
struct ConvPlan {
    int fft_n, rows;
    int block() const { return rows * (fft_n / 8); }
};
inline ConvPlan conv_plan(int rir_len) {
    const int fft_n = conv_fft_size(rir_len), row = fft_n / 8;
    return {fft_n, rir_len > fft_n ? 8 : 16 - (rir_len - 1 + row - 1) / row};      // more than one partition: whole blocks of N
}

// The tables that the transforms of that size read (float2 [conv_table_entries(fft_n)]), and the size of a partition's
// spectrum, in float2.
int conv_table_entries(int fft_n);
hipError_t launch_conv_table(hipStream_t s, int fft_n, float2* tab);
size_t conv_spectrum_entries(int fft_n);

// Spectra of the zero-padded partitions of each response: spec float2 [n_rir][n_part][conv_spectrum_entries(fft_n)];
// first_tap[n_rir][n_part] gets the index of every partition's first non-zero tap (INT_MAX: none), energy[n_rir] zeros.
hipError_t launch_rir_spectrum(hipStream_t s, int n_rir, const float* rir, int rir_len, int fft_n,
                               const float2* twiddle, float2* spec, int* first_tap, double* energy, int n_cu);

// Overlap-save convolution of every (utterance, source) with its response; adds the block's energy
// to energy[u][j] (double, must be zero on entry).  src_base[j] points at source j's packed signal.
struct ConvArgs {
    const int64_t* offsets;      // device
    const int2* items;           // device (utterance, block)
    const int* first;            // device [n_utt+1]: blocks of the utterances before u
    int64_t n_items;             // blocks of one source, all utterances
    int n_src;
    const float* speech;
    const float* noise;          // [n_src-1][total]
    int64_t total;
    const float2* spec;          // [n_utt][n_src][n_part][conv_spectrum_entries]
    int rows;                    // ConvPlan::rows
    int n_part;
    float* reverb;               // [n_src][reverb_stride]
    int64_t reverb_stride;
    double* energy;              // [n_utt][n_src] of the reverberated signals
    const int* first_tap;        // [n_utt][n_src][n_part] first non-zero tap of each partition
};
// n_cu: compute units of the device (the kernel runs as persistent work groups)
hipError_t launch_convolve(hipStream_t s, int fft_n, const float2* twiddle, const ConvArgs& a, int n_cu);

// The gain that puts noise j at its target SNR against the speech, from the energies [n_src] of one utterance's
// reverberated signals; zero energy on either side gives gain 0.  (A source whose direct path arrives after the
// utterance has ended has exactly zero energy: the convolution writes exact zeros before the response's first
// non-zero tap.)
__device__ inline float snr_gain(const double* energy, int j, float snr_db) {
    const double e0 = energy[0], ej = energy[1 + j];
    return e0 > 0.0 && ej > 0.0 ? (float)sqrt(e0 / (ej * exp10(0.1 * (double)snr_db))) : 0.f;
}
// gains_out [n_utt][n_src - 1]
hipError_t launch_gains(hipStream_t s, int n_utt, int n_src, const double* energy, const float* snr_db, float* gains_out);
// mixed = reverb[0] + sum_j gain_j reverb[j]; source j of the reverberated signals starts at j * stride; gains_out may be null
hipError_t launch_mix(hipStream_t s, int n_utt, const int64_t* d_offsets, int64_t stride, int n_src, const float* reverb,
                      const double* energy, const float* snr_db, float* mixed_out, float* gains_out, int64_t max_len);

void mel_edges(const aug_frontend_cfg& cfg, MelTableArgs& a);
int mel_table_stride(int nfft);
int mel_lane_floats();               // the front end's per-lane constants

// The image sum's plan as a share of another launch (rir_plan_fits): what launch_rir_plan does for these arguments.
struct PlanArgs {
    int n_rir = 0;               // 0: no plan
    Rooms rooms;
    int rir_len;
    double fs_over_c;
    void *items, *unsorted;      // the two tables in `items` of launch_rir_plan
    int* ctrl;
    int n_groups;
};
inline PlanArgs rir_plan_args(int n_groups, int n_rir, const Rooms& rooms, int rir_len, double fs_over_c, void* items, int* ctrl) {
    PlanArgs p;
    p.n_rir = n_rir;
    p.rooms = rooms;
    p.rir_len = rir_len;
    p.fs_over_c = fs_over_c;
    p.items = items;
    p.unsorted = static_cast<unsigned char*>(items) + rir_item_bytes() * (size_t)n_rir * rir_items_per_response(rir_len);
    p.ctrl = ctrl;
    p.n_groups = n_groups;
    return p;
}
constexpr int kPlanThreads = 1024, kPlanMost = 4 * kPlanThreads;
inline bool rir_plan_fits(int n_rir) { return n_rir <= kPlanMost; }      // one work group plans so many responses

// Everything a front-end call needs before its main kernel, in one launch: the utterances' tables, the packing if
// pack.n_utt > 0, the image sum's plan if plan.n_rir > 0, and those of the constants whose pointer is given (per-lane constants, Hamming window of
// table.cfg.win samples, orthonormal DCT-II rows [n_ceps][n_mel]).
struct MelSetupArgs {
    int n_utt;
    MelTableArgs table;
    PackArgs pack;
    PlanArgs plan;
    float* lane_consts;
    float* window;
    float* dct;
};
hipError_t launch_mel_setup(hipStream_t s, const MelSetupArgs& a);

// tw[t] = exp(-2 pi i t / n), t < n, then tw[n + k] = exp(-i pi k / n), k <= n/2, then
// exp(-i pi 16 j / n), j < n/32; each computed in fp64 and rounded once.
int twiddle_entries(int n);
hipError_t launch_twiddle(hipStream_t s, int n, float2* tw);

// The front end's LDS per group in bytes: frame buffers of 272 floats, weights, pieces, constants, for cepstra the cosine table.
inline size_t mel_lds_bytes(const aug_frontend_cfg& cfg) {
    size_t lds = 4 * kUnitFrames * 272 + 16 * 8 * 64 + 16 * AUG_MAX_MEL + 8 * (8 * 16 + 256) + 4 * AUG_MAX_NOISE;
    if (cfg.feature == AUG_FEAT_MFCC) lds += 16 * (size_t)((cfg.n_mel + 3) / 4) * ((cfg.n_ceps + 15) & ~15);
    return lds;
}
// Wavefronts per SIMD that the front end's kernels are built for (their launch bounds): four with a window of 400 samples and no mixture,
// three otherwise.
constexpr int mel_waves(bool own_window, bool mix) { return own_window && !mix ? 4 : 3; }
// Groups of the front end that the chip runs at once, by that and by what the LDS allows.
inline int mel_slots(int n_cu, const aug_frontend_cfg& cfg, bool mix) {
    const int by_waves = mel_waves(cfg.win == 400, mix), by_lds = (int)((160 * 1024) / (mel_lds_bytes(cfg) + 1280));
    return n_cu * (by_lds < 1 ? 1 : by_lds < by_waves ? by_lds : by_waves);
}
inline Framing mel_framing(int n_cu, const aug_frontend_cfg& cfg, bool mix) {
    return {cfg.win, cfg.hop, cfg.feature == AUG_FEAT_MFCC ? cfg.n_ceps : cfg.n_mel, mel_slots(n_cu, cfg, mix)};
}

// STFT power -> warped mel -> power law.
struct MelArgs {
    const int64_t* offsets;        // device
    const int64_t* frame_offsets;  // device
    const int2* items;             // device (utterance, unit of it) at which a group begins
    int64_t n_items;               // shares.n_groups
    FrameShares shares;
    const float* wave;
    // Mixing on the fly: when n_extra > 0 the analysed signal is
    // wave[n] + sum_j gain[u][j] * extra[j * extra_stride + n], j < n_extra, with the gains of snr_gain.
    const float* extra;
    int64_t extra_stride;
    const double* energy;          // [n_utt][1 + n_extra]
    const float* snr_db;           // [n_utt][n_extra]
    int n_extra;
    const float2* mel_tab;
    const float* dct;              // [n_ceps][n_mel] orthonormal DCT-II rows (AUG_FEAT_MFCC), else null
    const float* window;
    const float* lane_consts;
    aug_frontend_cfg cfg;
    float* feats;
};
hipError_t launch_mel(hipStream_t s, const MelArgs& a);

// Waveform VTLP: per-utterance table of (lower source bin, interpolation weight) for every output bin,
// then analysis, warp and overlap-add, one wavefront per frame; `out` must be zero on entry.
int vtlp_table_entries();
int vtlp_fft_size();                 // length of the complex transform whose twiddle table the kernel needs
bool vtlp_supported(int win, int hop, int nfft);
hipError_t launch_vtlp_table(hipStream_t s, int n_utt, const float* alpha, float2* tab);
hipError_t launch_vtlp_resynth(hipStream_t s, int n_utt, const int64_t* d_offsets, int64_t max_len,
                               const float* wave, const float2* tab, const float2* twiddle, float* out);

hipError_t launch_pack(hipStream_t s, const PackArgs& a);

// fill n 32-bit words with a value (used instead of memset so that calls stay graph-capturable)
hipError_t launch_fill_u32(hipStream_t s, void* p, uint32_t v, int64_t n);

}  // namespace aug
