// What a graph that holds a front-end call reads on replay: the call's kernel arguments, kept, and the table of its groups'
// beginnings as other calls on the same batch have left it.  The API layer on a host runtime; built by test_frame_tables.py with
// the host compiler.
#include <cstdlib>

#include "../../paper_1912_11040_amd/csrc/aug_api.hip"
#include "../../paper_1912_11040_amd/csrc/pack_device.h"

static aug::MelArgs g_mel;                // of the last front-end call
static bool g_capturing = false;

// ---- the runtime ----
extern "C" {
hipError_t hipMalloc(void** p, size_t n) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipFree(void*) { return hipSuccess; }          // (kept: a table that has been moved is looked at again below)
hipError_t hipHostMalloc(void** p, size_t n, unsigned int) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned int) { *d = h; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* s) { *p = const_cast<void*>(s); return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
    *s = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = reinterpret_cast<hipEvent_t>(8); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
}

// ---- the launchers ----
namespace aug {
hipError_t launch_pack(hipStream_t, const PackArgs& a) {
    for (int64_t t = 0; t < pack_threads(a); ++t) pack_utterances(a, (int)t);
    return hipSuccess;
}
hipError_t launch_mel_setup(hipStream_t s, const MelSetupArgs& a) { return a.pack.n_utt > 0 ? launch_pack(s, a.pack) : hipSuccess; }
hipError_t launch_mel(hipStream_t, const MelArgs& a) { g_mel = a; return hipSuccess; }
hipError_t launch_convolve(hipStream_t, int, const float2*, const ConvArgs&, int) { return hipSuccess; }
hipError_t launch_conv_table(hipStream_t, int, float2*) { return hipSuccess; }
hipError_t launch_twiddle(hipStream_t, int, float2*) { return hipSuccess; }
hipError_t launch_mix(hipStream_t, int, const int64_t*, int64_t, int, const float*, const double*, const float*, float*, float*, int64_t) { return hipSuccess; }
hipError_t launch_vtlp_resynth(hipStream_t, int, const int64_t*, int64_t, const float*, const float2*, const float2*, float*) { return hipSuccess; }
hipError_t launch_vtlp_table(hipStream_t, int, const float*, float2*) { return hipSuccess; }
hipError_t launch_gains(hipStream_t, int, int, const double*, const float*, float*) { return hipSuccess; }
hipError_t launch_fill_u32(hipStream_t, void*, uint32_t, int64_t) { return hipSuccess; }
hipError_t launch_rir_spectrum(hipStream_t, int, const float*, int, int, const float2*, float2*, int*, double*, int) { return hipSuccess; }
hipError_t launch_rir_plan(hipStream_t, int, int, const Rooms&, int, double, void*, int*) { return hipSuccess; }
hipError_t launch_rir(hipStream_t, int, int, const Rooms&, int, double, const void*, int*, float*, int32_t*, bool, unsigned long long*) { return hipSuccess; }
void mel_edges(const aug_frontend_cfg&, MelTableArgs&) {}
int mel_table_stride(int) { return 278; }
int mel_lane_floats() { return 448; }
int conv_fft_size(int) { return 1024; }
int conv_table_entries(int n) { return 2 * n; }
size_t conv_spectrum_entries(int n) { return (size_t)n + 1; }
int twiddle_entries(int n) { return 2 * n; }
int vtlp_table_entries() { return 1025; }
int vtlp_fft_size() { return 1024; }
bool vtlp_supported(int, int, int) { return true; }
int rir_items_per_response(int) { return 8; }
size_t rir_item_bytes() { return 16; }
int rir_ctrl_ints() { return 67; }
}  // namespace aug

static std::vector<int64_t> g_offsets{0}, g_frames{0};

static int run(aug_ctx* ctx, int kind) {
    float* const p = reinterpret_cast<float*>(64);       // (not read here)
    const int n = (int)g_offsets.size() - 1;
    aug_frontend_cfg fe{16000.f, 400, 160, 512, 40, 0.f, 8000.f, 1.f / 15.f, AUG_FEAT_POWER_LAW, 13, 1e-6f};
    if (kind == 2) {                                     // fewer groups by its LDS
        fe.feature = AUG_FEAT_MFCC;
        fe.n_mel = fe.n_ceps = 128;
    }
    if (kind == 3) fe.hop = 200;
    if (kind >= 4) fe.hop = 400 + kind;
    if (kind == 1) return aug_pipeline_batch(ctx, n, g_offsets.data(), p, 1, p, p, 100, 16000.f, 343.f, p, p, &fe, g_frames.data(), p, nullptr, nullptr, nullptr);
    return aug_vtlp_mel_batch(ctx, n, g_offsets.data(), p, p, &fe, g_frames.data(), p);
}

// groups of `a` that do not begin where the one before ends (the first: at the first unit), and units not shared out
static int faults(const aug::MelArgs& a) {
    int bad = 0, g = 0, next = 0, unit = 0;
    for (size_t u = 0; u + 1 < g_offsets.size(); ++u) {
        const int64_t n = aug::frame_units(g_offsets[u + 1] - g_offsets[u], g_frames[u + 1] - g_frames[u], aug::Framing{a.cfg.win, a.cfg.hop, aug_feature_dim(&a.cfg), 0}, a.shares.shift);
        for (int i = 0; i < n; ++i, ++unit)
            if (unit == next && g < a.shares.n_groups) {
                if (a.items[g].x != (int)u || a.items[g].y != i) ++bad;
                next += a.shares.per_group + (g < a.shares.longer ? 1 : 0);
                ++g;
            }
    }
    return bad + (g != a.shares.n_groups) + (next != unit) + (a.n_items != a.shares.n_groups);
}

int main() {
    for (int u = 0; u < 40; ++u) {
        g_offsets.push_back(g_offsets.back() + 100000 + 37 * u);
        g_frames.push_back(g_frames.back() + 1000);
    }
    int wrong = 0, refused = 0;
    for (int first = 0; first < 4; ++first)
        for (int second = 0; second < 4; ++second) {
            aug_ctx* ctx = nullptr;
            if (aug_create(&ctx, 0, nullptr) != AUG_OK || run(ctx, first) != AUG_OK) return 2;
            const aug::MelArgs kept = g_mel;
            if (faults(kept) || kept.shares.n_groups < 256) return 3;
            if (run(ctx, second) != AUG_OK || faults(g_mel)) return 4;
            if (faults(kept)) { printf("call %d, then call %d: the first one's groups begin elsewhere\n", first, second); ++wrong; }
            g_capturing = true;                          // both have been made once
            if (run(ctx, first) != AUG_OK || faults(g_mel) || run(ctx, second) != AUG_OK || faults(g_mel)) { printf("calls %d and %d: refused while capturing\n", first, second); ++refused; }
            g_capturing = false;
            aug_destroy(ctx);
        }
    // more framings of one batch than there are tables: the latest are there, and every call has its own
    aug_ctx* ctx = nullptr;
    if (aug_create(&ctx, 0, nullptr) != AUG_OK) return 2;
    for (int kind = 4; kind < 44; ++kind)
        if (run(ctx, kind) != AUG_OK || faults(g_mel)) ++wrong;
    g_capturing = true;
    for (int kind = 43; kind > 43 - 16; --kind)
        if (run(ctx, kind) != AUG_OK || faults(g_mel)) ++refused;
    if (run(ctx, 4) == AUG_OK) ++wrong;
    g_capturing = false;
    aug_destroy(ctx);
    printf("%d stale, %d refused\n", wrong, refused);
    return wrong || refused;
}
