// Top-m selection for callers that cannot allocate (code under HIP graph capture, tight serving loops, harnesses that
// forbid hipMalloc): the radix-select work space lives in a file-scope device array instead of a per-call allocation.
// See sage_topm_static in include/sage.h.
#include <mutex>

#include "sage_internal.h"
#include "topm_kept.h"

namespace {

// Work space of one top-m run over at most SAGE_TOPM_STATIC_MAX_N keys: the histograms, the state, and two counters and a table
// for every block of keys that such a run has.
constexpr int64_t MAX_N = SAGE_TOPM_STATIC_MAX_N;
constexpr int64_t MAX_BLOCKS = sage::topm_work_blocks(MAX_N);
constexpr size_t SCRATCH_WORDS = sage::topm_work_words(MAX_BLOCKS);

// One copy per GPU, at that GPU's own address; host code never uses this name as a pointer (it is a host-side stand-in
// there): it asks the runtime for the device address once per device and keeps it.
static __device__ __align__(256) uint32_t scratch[SCRATCH_WORDS];

constexpr int MAX_DEVICES = 64;
std::mutex g_lock;
uint32_t* g_ptr[MAX_DEVICES] = {nullptr};
sage::KeptHistograms g_kept[MAX_DEVICES];

// Device address of `scratch` on the current device (looked up on the first call per device).
int scratch_ptr(uint32_t** out, int& dev) {
    dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return SAGE_ERR_HIP;
    }
    if (dev < 0 || dev >= MAX_DEVICES) return SAGE_ERR_ARG;
    std::lock_guard<std::mutex> hold(g_lock);
    if (!g_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return SAGE_ERR_HIP;
        }
        g_ptr[dev] = (uint32_t*)p;
    }
    *out = g_ptr[dev];
    return SAGE_OK;
}

}  // namespace

extern "C" int sage_topm_static(const float* alpha, int64_t N, int64_t m, int64_t* out_idx, void* hip_stream) {
    if (N < 0 || m < 0 || m > N || (N > 0 && !alpha) || (m > 0 && !out_idx)) return SAGE_ERR_ARG;
    if (N > MAX_N) return SAGE_ERR_CAPACITY;
    if (m == 0) return SAGE_OK;
    uint32_t* base = nullptr;
    int dev = -1, rc = scratch_ptr(&base, dev);
    if (rc != SAGE_OK) return rc;
    const sage::SelectWork w = sage::select_work_at(base, MAX_BLOCKS);
    // The histograms are zero when the module is loaded and when a run is over (two that overlapped too, once both are: each
    // clears them after its own additions), but for runs that were cut short: see topm_kept.h. The state, every per-block counter
    // and every table that is read are written earlier in the same run. So nothing of the previous call's contents is used.
    const hipStream_t st = (hipStream_t)hip_stream;
    const bool many = sage::topm_needs_work(N);  // (else one launch, which uses none of it)
    bool eager = true;
    if (many) {
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        eager = hipStreamIsCapturing(st, &cs) == hipSuccess && cs == hipStreamCaptureStatusNone;
        if (!eager) (void)hipGetLastError();
    }
    const bool clear = many && !g_kept[dev].clear_first(eager);
    if (sage::launch_topm(alpha, N, m, out_idx, w, clear, st) != hipSuccess) {
        (void)hipGetLastError();
        if (many) g_kept[dev].refused();
        return SAGE_ERR_HIP;
    }
    return SAGE_OK;
}
