// The API layer on a host runtime whose allocations fail when told to: after a call that ran out of memory the context's
// records of what its tables hold must be true, so that the call before it, made again, finds its tables whole.  Built by
// test_out_of_memory.py with the host compiler; the kernels' launchers below check what they are given.
#include <cstdlib>

#include "../../paper_1912_11040_amd/csrc/aug_api.hip"
#include "../../paper_1912_11040_amd/csrc/pack_device.h"

static int g_until_failure = -1;         // allocations that still succeed; -1: all
static int g_faults = 0;
static const int64_t* g_offsets;         // of the call under way
static const int64_t* g_frame_offsets;
static int g_n_utt;

#define EXPECT(cond)                                                       \
    do {                                                                   \
        if (!(cond)) { ++g_faults; printf("line %d: %s\n", __LINE__, #cond); } \
    } while (0)

// ---- the runtime ----
extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
    if (g_until_failure == 0) return hipErrorOutOfMemory;
    if (g_until_failure > 0) --g_until_failure;
    *p = malloc(n);
    memset(*p, 0xa5, n);
    return hipSuccess;
}
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned int) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned int) { *d = h; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* s) { *p = const_cast<void*>(s); return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
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
static void check_offsets(const int64_t* d) { EXPECT(d && !memcmp(d, g_offsets, sizeof(int64_t) * (g_n_utt + 1))); }
static void check_items(const int2* items, int64_t n) {
    for (int64_t i = 0; items && i < n; ++i)
        if (items[i].x < 0 || items[i].x >= g_n_utt) { EXPECT(!"an item of no utterance"); return; }
    EXPECT(items || !n);
}
hipError_t launch_pack(hipStream_t, const PackArgs& a) {
    for (int64_t t = 0; t < pack_threads(a); ++t) pack_utterances(a, (int)t);
    return hipSuccess;
}
hipError_t launch_mel_setup(hipStream_t s, const MelSetupArgs& a) {
    if (a.pack.n_utt > 0) (void)launch_pack(s, a.pack);
    if (a.lane_consts) a.lane_consts[0] = 7.f;
    for (int i = 0; a.window && i < a.table.cfg.win; ++i) a.window[i] = (float)a.table.cfg.win;
    for (int i = 0; a.dct && i < a.table.cfg.n_ceps * a.table.cfg.n_mel; ++i) a.dct[i] = (float)a.table.cfg.n_ceps;
    return hipSuccess;
}
hipError_t launch_mel(hipStream_t, const MelArgs& a) {
    check_offsets(a.offsets);
    EXPECT(a.frame_offsets && !memcmp(a.frame_offsets, g_frame_offsets, sizeof(int64_t) * (g_n_utt + 1)));
    check_items(a.items, a.n_items);
    EXPECT(a.lane_consts[0] == 7.f);
    for (int i = 0; i < a.cfg.win; ++i)
        if (a.window[i] != (float)a.cfg.win) { EXPECT(!"window"); break; }
    for (int i = 0; a.dct && i < a.cfg.n_ceps * a.cfg.n_mel; ++i)
        if (a.dct[i] != (float)a.cfg.n_ceps) { EXPECT(!"cosine table"); break; }
    return hipSuccess;
}
hipError_t launch_convolve(hipStream_t, int, const float2* tab, const ConvArgs& a, int) {
    check_offsets(a.offsets);
    check_items(a.items, a.n_items);
    EXPECT(tab && tab[0].x == 3.f);
    EXPECT(a.first && a.first[0] == 0 && a.first[g_n_utt] == (int)a.n_items);
    return hipSuccess;
}
hipError_t launch_conv_table(hipStream_t, int, float2* t) { t[0].x = 3.f; return hipSuccess; }
hipError_t launch_twiddle(hipStream_t, int, float2*) { return hipSuccess; }
hipError_t launch_mix(hipStream_t, int, const int64_t* o, int64_t, int, const float*, const double*, const float*, float*, float*, int64_t) { check_offsets(o); return hipSuccess; }
hipError_t launch_vtlp_resynth(hipStream_t, int, const int64_t* o, int64_t, const float*, const float2*, const float2*, float*) { check_offsets(o); return hipSuccess; }
hipError_t launch_vtlp_table(hipStream_t, int, const float*, float2*) { return hipSuccess; }
hipError_t launch_gains(hipStream_t, int, int, const double*, const float*, float*) { return hipSuccess; }
hipError_t launch_fill_u32(hipStream_t, void*, uint32_t, int64_t) { return hipSuccess; }
hipError_t launch_rir_spectrum(hipStream_t, int, const float*, int, int, const float2*, float2*, int*, double*, int) { return hipSuccess; }
hipError_t launch_rir_plan(hipStream_t, int, int, const Rooms&, int, double, void*, int*) { return hipSuccess; }
hipError_t launch_rir(hipStream_t, int, int, const Rooms&, int, double, const void*, int*, float*, int32_t*, bool, unsigned long long*) { return hipSuccess; }
void mel_edges(const aug_frontend_cfg&, MelTableArgs&) {}
int mel_table_stride(int) { return 278; }
int mel_lane_floats() { return 448; }
int mel_rows_per_group(int, int64_t) { return 64; }
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

struct Batch {
    std::vector<int64_t> offsets{0}, frames{0};
    aug_frontend_cfg fe{16000.f, 400, 160, 512, 40, 0.f, 8000.f, 1.f / 15.f, AUG_FEAT_MFCC, 13, 1e-6f};
    Batch(int n_utt, int64_t len, int win, int n_ceps) {
        fe.win = win;
        fe.n_ceps = n_ceps;
        for (int u = 0; u < n_utt; ++u) {
            offsets.push_back(offsets.back() + len + u % 7);
            frames.push_back(frames.back() + aug_frame_count(len + u % 7, win, 160));
        }
    }
    int run(aug_ctx* ctx, int entry) const {
        float* const p = reinterpret_cast<float*>(64);       // (not read here)
        const int n = (int)offsets.size() - 1;
        const aug_vtlp_cfg vc{800, 400, 2048};
        g_offsets = offsets.data();
        g_frame_offsets = frames.data();
        g_n_utt = n;
        switch (entry) {
            case 0: return aug_vtlp_mel_batch(ctx, n, g_offsets, p, p, &fe, g_frame_offsets, p);
            case 1: return aug_convolve_mix_batch(ctx, n, g_offsets, p, 1, p, p, 100, p, p, nullptr);
            case 2: return aug_pipeline_batch(ctx, n, g_offsets, p, 1, p, p, 100, 16000.f, 343.f, p, p, &fe, g_frame_offsets, p, nullptr, nullptr, nullptr);
            default: return aug_vtlp_resynth_batch(ctx, n, g_offsets, p, p, &vc, p + ((int64_t)1 << 32));
        }
    }
};

int main() {
    const Batch small(3, 4000, 400, 13), large(5200, 500, 480, 40);
    int refused = 0;
    for (int first = 0; first < 4; ++first)
        for (int second = 0; second < 4; ++second)
            for (int k = 0;; ++k) {
                aug_ctx* ctx = nullptr;
                EXPECT(aug_create(&ctx, 0, nullptr) == AUG_OK);
                EXPECT(small.run(ctx, first) == AUG_OK);
                g_until_failure = k;                         // every allocation after the next k fails
                const int rc = large.run(ctx, second);
                g_until_failure = -1;
                EXPECT(rc == AUG_OK || rc == AUG_ERR_NOMEM);
                refused += rc == AUG_ERR_NOMEM;
                const int before = g_faults;
                EXPECT(small.run(ctx, first) == AUG_OK);
                EXPECT(large.run(ctx, second) == AUG_OK);
                if (g_faults != before) printf("entry points %d and %d, allocation %d\n", first, second, k);
                aug_destroy(ctx);
                if (rc == AUG_OK) break;
            }
    printf("%d calls out of memory, %d faults\n", refused, g_faults);
    return g_faults || refused < 16;
}
