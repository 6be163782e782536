// C ABI of the SAGE hot-path library: context, state machine and kernel sequencing. See include/sage.h.
#include <math.h>
#include <new>
#include <stdlib.h>
#include <string.h>
#include <chrono>
#include <mutex>
#include <type_traits>
#include <unistd.h>

#include "fd_defer_plan.h"
#include "sage_internal.h"

using namespace sage;

namespace {

constexpr int NCLASS = 9;
constexpr int MAX_HALVES = GRAM_TOPS - 1;  // of the ring of new rows; a block's products are with all but one of them and the top
constexpr int64_t SCORE_CHUNK = 2048;  // rows per projection launch
enum { K_GRAM = 0, K_REDUCE, K_EIG, K_REBUILD = 4, K_INSERT, K_PROJECT, K_FINALIZE, K_SELECT };

}  // namespace

// What a context needs from the driver besides memory. Creating and destroying it costs more than a small context's first
// cycles (a stream and a pinned word: 100 us and more, 0.6 ms at destruction), so a few kits are kept for the next context
// on the same device (kit_take, kit_give).
struct SideKit {
    hipStream_t stream = nullptr;
    hipEvent_t mark = nullptr, side[2] = {nullptr, nullptr};
    int* host = nullptr;  // pinned words: [1], [2] report of the class-balanced selection, [16] signal
    unsigned token = 0;   // of the last signal
};

// Where device memory comes from (sage_set_allocator); a context keeps the pair it was created with.
struct Allocator {
    sage_alloc_fn alloc = nullptr;  // null: hipMalloc and hipFree
    sage_free_fn free = nullptr;
    void* user = nullptr;
};

// Chunk images of the basis for the bf16 projection (score_split.hip), built when rows first ask for them.
struct BasisImages {
    void* mem = nullptr;
    size_t bytes = 0;
    bool current = false;  // they are of the basis in Vblk
};

struct sage_ctx {
    Allocator mem{};
    Dims d{};
    int dtype = SAGE_F32;
    hipStream_t st = nullptr;
    int num_cu = 256;

    // The 2*ell-row buffer is kept as two half buffers of LP rows each (column-slab layout): `top` holds buffer rows
    // 0 .. ell-1 (after a shrink: the rows it wrote), half df.cur of the ring holds buffer rows ell .. 2*ell-1 as they arrive.
    // Two of the ring's halves alternate so that the rows of the next cycle can be stored, and their own Gram block formed, on a
    // side stream while the eigensolve of the current cycle runs; the others hold blocks whose shrink is deferred (see below).
    float* top = nullptr;
    float* ring = nullptr;
    int64_t half_floats = 0;
    int halves = 0;
    float* nw(int i) const { return ring + i * half_floats; }
    DeferPlan df{};  // df.cur: the current half
    int par = 0;                       // of the cycle: which of gram_partial_new, ev_side and gp_side_used are those of half cur
    SideKit kit{};                               // the stream, events and host word the next five name
    hipStream_t st2 = nullptr;                   // side stream (only when the Gram has >= 2 row panels)
    hipEvent_t ev_mark = nullptr;                // context stream: the Gram matrix of the current cycle is complete
    hipEvent_t ev_side[2] = {nullptr, nullptr};  // side stream: rows stored ahead and their Gram block formed, by par
    int* side_hole = nullptr;                    // the place its launches leave out (spare_unit_at)
    bool pending_shrink = false;   // the buffer is full, its shrink waits for the next update call (see sage_fd_update)
    bool pre_stored = false;       // the next ell rows of the running call are stored in half cur already
    bool new_block_ready = false;  // ... and their Gram block is (or will be, see ev_side) in gram_partial_new[par]
    // Deferred shrinks (fd_defer.hip). The buffer's top rows are W [top; the blocks of df], with blocks only inside an update call: it
    // ends with the rows written, so that everything else finds them in `top`.
    double* coef[5] = {nullptr, nullptr, nullptr, nullptr, nullptr};  // M and W, by the numbers of df
    const double* last_M() const { return coef[df.m]; }
    const double* W() const { return coef[df.w]; }
    int ldw() const { return df.w < df.MS ? d.NP : (1 + df.max) * d.LP; }
    int ldk = 0;
    double* K = nullptr;        // products of the next block's rows with [W [top; blocks]; cur], then those with top and blocks
    double* C_next = nullptr;   // the Gram matrix of the next cycle, as far as it is known
    bool C_ready = false;       // ew.C is the whole Gram matrix of the coming shrink
    bool marked = false;        // ev_mark is recorded after the last work of the context stream that the side stream must wait for
    GramPlan gp{};        // whole lower triangle
    GramPlan gp_skip{};   // without the top x top block (known after a shrink)
    GramPlan gp_cross{};  // new rows x top rows
    // ... and their counterparts for the split-arithmetic kernels (tiles = 0: not available for this sketch size)
    GramPlan gp_cross_split{}, gp_new_split{}, gp_new2_split{};
    GramPlan gp_cross_side{};  // (that on the side stream)
    const GramPlan* gp_side_used[2] = {nullptr, nullptr};  // the plan the launch into gram_partial_new[i] used
    GramPlan gp_new{};    // new rows x new rows, one work-group per CU (it shares the chip with the eigensolve)
    GramPlan gp_new2{};   // the same block with the chip to itself (context stream, when there was nothing to look ahead to)
    bool top_shrunk = false;  // top holds exactly what the last shrink wrote
    float* gram_partial = nullptr;
    float* gram_partial_new[2] = {nullptr, nullptr};
    EigWork ew{};
    char* eig_mem = nullptr;  // what ew points into
    float* Mt = nullptr;
    void* Mt3 = nullptr;   // the rebuild's coefficients split into bf16 parts (SAGE_MM_SPLIT)
    int mm_mode = SAGE_MM_SPLIT;
    // Rows of a bf16 stream are kept as fp32 but have one bf16 part, not three: the split-arithmetic kernels then skip
    // the products with the new rows' mid and lo parts (exact zeros; same bits). nw_bf16[i]: every row in use in half i
    // came from a bf16 batch (row-major or factored; not sage_fd_merge's fp32 rows). one_part: the shortcut is allowed (off under SAGE_MM_SPLIT_ALL_PARTS).
    bool nw_bf16[MAX_HALVES] = {};
    bool nw_half[MAX_HALVES] = {};  // half i is kept in pieces of bf16 (half16), not as fp32
    bool one_part = true;
    double* acc = nullptr;  // [0] sum_delta [1] frob2 [2] last_delta [4] EigWork::redone

    bool poisoned = false;   // a HIP call failed while work of a call was partly enqueued: the state is not trustworthy
    int fail_in = 0;         // test hook (sage_debug_fail_launch): the fail_in-th launch from now fails without running
    bool debug_checks = false;      // sage_set_debug_checks: scan caller batches for non-finite values
    unsigned* dbg_count = nullptr;  // device counter of that scan

    int xcd_slot = -1;        // registered use of an XCD by this context's eigensolves (-1: they need none)
    int device = 0;

    int fill_top = 0, fill_new = 0;  // rows in use in top (0..ell) and in nw[cur] (0..ell)
    int cnt_top = 0, cnt_new = 0;    // of those, rows already counted in frob2
    int64_t rows_seen = 0, n_shrinks = 0;

    bool has_basis = false;
    int k = 0, KP = 0;
    float* Vblk = nullptr;
    int Vblk_KP = 0;
    BasisImages img[2];        // in two and in three bf16 parts
    bool img_ok = false;       // those of two parts serve row-major batches of this D
    void* stage = nullptr;     // factored rows written out, for shapes the factored projection does not take
    size_t stage_bytes = 0;
    int proj_mode = SAGE_PROJ_AUTO;
    float* zhat = nullptr;
    int64_t cap_rows = 0, n_scored = 0;
    bool store_zhat = true;   // false: zhat is not kept; alpha comes from a second pass over the rows (sage_rescore)
    int64_t n_rescored = 0;
    int* labels = nullptr;       // class label of every scored row (sage_score_labeled), same capacity as zhat
    int64_t n_labeled = 0;       // rows of the current pass that came with a label
    void* cb_work = nullptr;     // work space of the class-balanced selection
    size_t cb_work_bytes = 0;
    bool fixed_cap = false;
    float* proj_partial = nullptr;
    size_t proj_partial_floats = 0;
    double* cons_partial = nullptr;
    double* ssum = nullptr;      // (the first batch of a pass sets it)
    unsigned* ticket = nullptr;  // beside it
    float* alpha = nullptr;
    int64_t alpha_cap = 0, alpha_n = 0;
    SelectWork sw{};

    bool prof = false;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    double prof_ms[NCLASS] = {0};
    int64_t prof_n[NCLASS] = {0};
};

namespace {

// A HIP call that fails in the middle of a library call leaves work of that call partly enqueued: the context is
// marked poisoned (every later call except sage_destroy returns SAGE_ERR_STATE). `c` must be in scope.
inline int hip_failed(sage_ctx* c) {
    (void)hipGetLastError();
    c->poisoned = true;
    return SAGE_ERR_HIP;
}
#define HIPCHK(expr)                                 \
    do {                                             \
        hipError_t e_ = (expr);                      \
        if (e_ != hipSuccess) return hip_failed(c);  \
    } while (0)

// first statement of every call on a context
#define ALIVE(c)                                                                       \
    do {                                                                               \
        if (!(c)) return SAGE_ERR_ARG;                                                 \
        if ((c)->poisoned) return SAGE_ERR_STATE;                                      \
    } while (0)

std::mutex g_mem_lock;
Allocator g_mem;

bool dev_alloc(const Allocator& m, hipStream_t st, void** p, size_t bytes) {
    *p = nullptr;
    if (m.alloc) {
        *p = m.alloc(bytes, (void*)st, m.user);
        return *p != nullptr;
    }
    if (hipMalloc(p, bytes) == hipSuccess) return true;
    (void)hipGetLastError();
    *p = nullptr;
    return false;
}
void dev_free(const Allocator& m, void* p) {
    if (!p) return;
    if (m.free) m.free(p, m.user);
    else (void)hipFree(p);
}

int give_up_halves(sage_ctx* c);
// ... for what a context comes to need after its creation
bool late_alloc(sage_ctx* c, void** p, size_t bytes) {
    while (!dev_alloc(c->mem, c->st, p, bytes))
        if (give_up_halves(c) != SAGE_OK) return false;
    return true;
}
#define NO_MEMORY(c) ((c)->poisoned ? SAGE_ERR_HIP : SAGE_ERR_ALLOC)
// (`c` must be in scope)
#define ALLOC(ptr, bytes)                                                      \
    do {                                                                       \
        if (!late_alloc(c, (void**)&(ptr), (bytes))) return NO_MEMORY(c);      \
    } while (0)
#define FREE(ptr)                       \
    do {                                \
        dev_free(c->mem, (void*)(ptr)); \
        (ptr) = nullptr;                \
    } while (0)

// Of the halves that only rows stored ahead (64 buffer rows) and deferred shrinks take, those that the next smaller plan does without
// (DeferPlan::fewer), given back where memory is short after all: between calls none of them is in use but, perhaps, the current one. The ring is one allocation, so what remains takes the place of
// it, by way of the host where the two do not fit side by side. SAGE_ERR_ALLOC: there is nothing to give.
bool capturing(hipStream_t st);
int give_up_halves(sage_ctx* c) {
    DeferPlan less = c->df;
    less.give_up();
    int keep = c->d.NP == 64 ? 1 : less.halves();
    if (c->halves <= keep || c->df.count > 0 || c->df.captured || capturing(c->st)) return SAGE_ERR_ALLOC;
    HIPCHK(hipStreamSynchronize(c->st));
    if (c->st2) HIPCHK(hipStreamSynchronize(c->st2));
    const size_t half = (size_t)c->half_floats * sizeof(float);
    const int cur = c->df.cur;
    const bool rows = c->fill_new > 0;
    auto copy = [&](void* dst, const void* src, hipMemcpyKind kind) {
        return !rows || (hipMemcpyAsync(dst, src, half, kind, c->st) == hipSuccess && hipStreamSynchronize(c->st) == hipSuccess);
    };
    float* ring = nullptr;
    bool ok;
    if (dev_alloc(c->mem, c->st, (void**)&ring, keep * half)) {
        ok = copy(ring, c->nw(cur), hipMemcpyDeviceToDevice);
        if (ok) FREE(c->ring);
    } else {
        void* const host = rows ? malloc(half) : nullptr;
        if (rows && !host) return SAGE_ERR_ALLOC;
        ok = copy(host, c->nw(cur), hipMemcpyDeviceToHost);
        if (ok) {
            FREE(c->ring);
            // (no more than what has just been given back; should some of that be gone, there may be room for fewer)
            while (!(ok = dev_alloc(c->mem, c->st, (void**)&ring, keep * half)) && less.max > 0) {
                less.give_up();
                keep = less.halves();
            }
            ok = ok && copy(ring, host, hipMemcpyHostToDevice);
        }
        free(host);
    }
    if (!ok) {
        FREE(ring);
        return hip_failed(c);
    }
    c->ring = ring;
    c->halves = keep;
    c->nw_bf16[0] = c->nw_bf16[cur];
    c->nw_half[0] = c->nw_half[cur];
    for (int i = 1; i < MAX_HALVES; ++i) c->nw_bf16[i] = c->nw_half[i] = false;
    c->df = less;
    return SAGE_OK;
}

// The end of the work that sets `done`: a short spin on the host's word, then (the stream has much to do before it, or
// something failed) the runtime's own wait.
hipError_t wait_signal(const HostSignal& done, hipStream_t st) {
    using clock = std::chrono::steady_clock;
    const auto until = clock::now() + std::chrono::microseconds(500);
    do {
        for (int i = 0; i < 64; ++i) {
            if (__atomic_load_n(done.word, __ATOMIC_ACQUIRE) == done.token) return hipSuccess;
            __builtin_ia32_pause();
        }
    } while (clock::now() < until);
    return hipStreamSynchronize(st);
}

// Words for calls without a context: one pinned page for the process, at most 32 calls at a time (the others use the
// runtime's wait).
struct SignalPage {
    std::mutex lock;
    unsigned* words = nullptr;
    unsigned used = 0, token = 0;
    bool failed = false;
} g_signals;
bool signal_take(HostSignal& s) {
    std::lock_guard<std::mutex> hold(g_signals.lock);
    if (!g_signals.words && !g_signals.failed) {
        g_signals.failed = hipHostMalloc((void**)&g_signals.words, 32 * 64, hipHostMallocPortable) != hipSuccess;
        if (g_signals.failed) (void)hipGetLastError();
        else memset(g_signals.words, 0, 32 * 64);
    }
    if (g_signals.failed || g_signals.used == 0xFFFFFFFFu) return false;
    const int i = __builtin_ctz(~g_signals.used);
    g_signals.used |= 1u << i;
    s.word = g_signals.words + 16 * i;  // a line of its own
    s.token = ++g_signals.token;
    if (s.token == 0) s.token = ++g_signals.token;
    return true;
}
void signal_give(const HostSignal& s) {
    if (!s.word) return;
    std::lock_guard<std::mutex> hold(g_signals.lock);
    g_signals.used &= ~(1u << ((s.word - g_signals.words) / 16));
}

// run a launcher, optionally bracketed by events of kernel class `cls`
template <typename F>
int run(sage_ctx* c, int cls, F&& f) {
    if (c->fail_in > 0 && --c->fail_in == 0) return hip_failed(c);  // sage_debug_fail_launch
    if (c->prof) {
        if (!c->ev0) HIPCHK(hipEventCreate(&c->ev0));
        if (!c->ev1) HIPCHK(hipEventCreate(&c->ev1));
        HIPCHK(hipEventRecord(c->ev0, c->st));
    }
    HIPCHK(f());
    if (c->prof) {
        HIPCHK(hipEventRecord(c->ev1, c->st));
        HIPCHK(hipEventSynchronize(c->ev1));
        float ms = 0.f;
        HIPCHK(hipEventElapsedTime(&ms, c->ev0, c->ev1));
        c->prof_ms[cls] += ms;
        c->prof_n[cls] += 1;
    }
    return SAGE_OK;
}

#define RUN(cls, call)                                         \
    do {                                                       \
        int rc_ = run(c, cls, [&]() -> hipError_t { return (call); }); \
        if (rc_ != SAGE_OK) return rc_;                        \
    } while (0)

int pad_pow2_32(int v) {
    int p = 32;
    while (p < v) p *= 2;
    return p;
}

bool use_side(const sage_ctx* c) { return c->st2 != nullptr; }

// Where rows come from: a row-major batch, or the two factors of last-layer gradient rows (sage_fd_update_outer).
struct RowSrc {
    const void* G = nullptr;  // rows x D, or
    const void* E = nullptr;  // rows x C logit errors and
    const void* H = nullptr;  // rows x dh features
    int64_t C = 0, dh = 0;
    int dtype = SAGE_F32;
    bool outer() const { return G == nullptr; }
    RowSrc after(int64_t rows, int64_t D) const {
        const size_t esz = dtype == SAGE_BF16 ? 2 : 4;
        RowSrc r = *this;
        if (outer()) {
            r.E = (const char*)E + (size_t)rows * C * esz;
            r.H = (const char*)H + (size_t)rows * dh * esz;
        } else {
            r.G = (const char*)G + (size_t)rows * D * esz;
        }
        return r;
    }
};

hipError_t insert_rows(const RowSrc& s, int64_t rows, int row0, float* half, int half_rows, const Dims& d, bool to16,
                       hipStream_t st, const int* hole = nullptr) {
    if (s.outer()) return launch_insert_outer(s.E, s.H, s.dtype, s.C, s.dh, rows, row0, half, half_rows, d, to16, hole, st);
    return launch_insert(s.G, s.dtype, rows, row0, half, half_rows, d, to16, hole, st);
}

// Before the top half is read while the stream has not filled it yet: its other rows count as zero.
int clear_top(sage_ctx* c) {
    if (c->fill_top < c->d.ell) HIPCHK(launch_zero_rows(c->top, c->d.LP, c->fill_top, c->d.ell, c->d, c->st));
    return SAGE_OK;
}

bool split_grams(const sage_ctx* c) {
    return c->mm_mode == SAGE_MM_SPLIT && c->gp_cross_split.tiles > 0 && c->gp_new2_split.tiles > 0;
}

// Half i of the ring as fp32 (on the context stream; the side stream is done with it): for the kernels that know no other form.
int widen(sage_ctx* c, int i) {
    if (!c->nw_half[i]) return SAGE_OK;
    if (c->st2 && i == c->df.cur) HIPCHK(hipStreamWaitEvent(c->st, c->ev_side[c->par], 0));  // (never recorded: nothing to wait for)
    HIPCHK(launch_widen(c->nw(i), c->d, c->st));
    c->nw_half[i] = false;
    return SAGE_OK;
}

HostSignal next_signal(sage_ctx* c) {
    HostSignal s;
    s.word = (unsigned*)c->kit.host + 16;
    s.token = ++c->kit.token;
    if (s.token == 0) s.token = ++c->kit.token;
    return s;
}

// Rows of `s` are about to be stored in half i from row row0 on (by the context stream unless row0 = 0).
int note_new_rows(sage_ctx* c, int i, int row0, const RowSrc& s) {
    const bool b = s.dtype == SAGE_BF16;  // factored rows of a bf16 context are rounded to bf16 when they are stored
    if (row0 == 0) c->nw_half[i] = b && c->d.NP == 512 && c->one_part && split_grams(c) && c->Mt3;
    else if (!b)
        if (int rc = widen(c, i); rc != SAGE_OK) return rc;
    c->nw_bf16[i] = row0 == 0 ? b : (c->nw_bf16[i] && b);
    return SAGE_OK;
}
// (at NP = 512 the kernels that take one part read pieces of bf16)
bool new_one(const sage_ctx* c, int i) { return c->one_part && c->nw_bf16[i] && (c->d.NP < 512 || c->nw_half[i]); }

// The reduction of a 128-, 256- or 512-row eigensolve keeps 16 or 32 work-groups of one XCD in step, so all of them must be
// resident together (where they are not, the solve takes milliseconds longer), and at 512 rows they fill the registers of
// its 32 CUs. Contexts are spread over the XCDs; where two share one, each reduction waits for the one before it on that
// XCD, by an event that is recorded after it, or, if the XCD was not shared yet, when the other context comes to wait.
struct XcdSlot {
    int users = 0;
    hipEvent_t last = nullptr;        // kept for the life of the process (at most 8 per device)
    const sage_ctx* owner = nullptr;  // whose reduction was the last one
    bool marked = false;              // ... and `last` is recorded after it
};
constexpr int MAX_DEVICES = 64;
std::mutex g_xcd_lock;
XcdSlot g_xcd[MAX_DEVICES][8];

constexpr int KITS_KEPT = 4;  // per device
constexpr int KIT_WORDS = 32;
std::mutex g_kit_lock;
SideKit g_kit[MAX_DEVICES][KITS_KEPT];
int g_kits[MAX_DEVICES] = {0};

void kit_destroy(SideKit& k) {
    if (k.stream) (void)hipStreamDestroy(k.stream);
    for (hipEvent_t e : {k.mark, k.side[0], k.side[1]})
        if (e) (void)hipEventDestroy(e);
    if (k.host) (void)hipHostFree(k.host);
    k = SideKit{};
}
// (the current device is `device`)
bool kit_take(int device, SideKit& k) {
    if (device >= 0 && device < MAX_DEVICES) {
        std::lock_guard<std::mutex> hold(g_kit_lock);
        if (g_kits[device] > 0) {
            k = g_kit[device][--g_kits[device]];
            return true;
        }
    }
    k = SideKit{};
    bool ok = hipStreamCreateWithFlags(&k.stream, hipStreamNonBlocking) == hipSuccess;
    // These order data between streams (the caller's rows; rows and partial sums of the side stream) on a chip with an L2
    // per XCD: they keep the release that a recorded event has. (hipEventDisableSystemFence is for events that only time.)
    for (hipEvent_t* e : {&k.mark, &k.side[0], &k.side[1]})
        ok = ok && hipEventCreateWithFlags(e, hipEventDisableTiming) == hipSuccess;
    ok = ok && hipHostMalloc((void**)&k.host, KIT_WORDS * sizeof(int), hipHostMallocDefault) == hipSuccess;
    if (!ok) {
        (void)hipGetLastError();
        kit_destroy(k);
        return false;
    }
    memset(k.host, 0, KIT_WORDS * sizeof(int));  // (the signal word must not hold a token to come)
    return true;
}
// (everything enqueued with it is complete)
void kit_give(int device, SideKit& k, bool reuse) {
    if (!k.stream) return;
    if (reuse && device >= 0 && device < MAX_DEVICES) {
        std::lock_guard<std::mutex> hold(g_kit_lock);
        if (g_kits[device] < KITS_KEPT) {
            g_kit[device][g_kits[device]++] = k;
            k = SideKit{};
            return;
        }
    }
    kit_destroy(k);
}

// The XCD for a context's reductions; where there is no telling which work-groups share one, it needs none.
void xcd_take(sage_ctx* c) {
    if (c->d.NP < 128 || c->device < 0 || c->device >= MAX_DEVICES) return;
    const XcdMap& map = xcd_map();
    c->ew.period = map.period;
    if (map.period == 0) return;
    std::lock_guard<std::mutex> hold(g_xcd_lock);
    int best = -1;
    for (int i = 0; i < 8; ++i) {
        const int x = ((int)(getpid() & 7) + i) & 7;  // other processes on the GPU most likely start at another one
        bool there = false;
        for (int p = 0; p < map.period; ++p) there = there || map.id[p] == x;
        if (there && (best < 0 || g_xcd[c->device][x].users < g_xcd[c->device][best].users)) best = x;
    }
    g_xcd[c->device][best].users += 1;
    c->xcd_slot = best;
    c->ew.xcd = best;
}
void xcd_release(sage_ctx* c) {
    if (c->xcd_slot < 0) return;
    std::lock_guard<std::mutex> hold(g_xcd_lock);
    XcdSlot& x = g_xcd[c->device][c->xcd_slot];
    x.users -= 1;
    if (x.owner == c) x.owner = nullptr;  // the context's stream has been waited for
    c->xcd_slot = -1;
}

// What a captured stream holds runs later, if at all: it has no place in the order of reductions on an XCD.
bool capturing(hipStream_t st) {
    hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &s) == hipSuccess) return s != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return false;
}
// A call that stores to the halves or reads them: if it is captured, they must be found where they are now by every replay. (And what
// is known of a pending shrink here is not what a replay leaves.)
void note_capture(sage_ctx* c) {
    if (c->df.captured || !capturing(c->st)) return;
    c->df.captured = true;
    c->C_ready = false;
}

// Eigensolve of the Gram matrix of fill_top + fill_new rows; the `count` leading eigenvectors are formed, or (cf given) the
// coefficients made from its own count of them.
hipError_t eigensolve(sage_ctx* c, int m0, int n, int count, const CoeffArgs* cf = nullptr, const RowJob* job = nullptr) {
    if (n < 1) m0 = n = 1;  // an empty buffer: one zero row
    if (c->xcd_slot < 0) return launch_eig(c->ew, c->d.NP, m0, n, count, cf, c->st, job);
    std::unique_lock<std::mutex> hold(g_xcd_lock);
    XcdSlot& x = g_xcd[c->device][c->xcd_slot];
    const bool shared = x.users > 1 && !capturing(c->st);
    if (shared) {
        if (!x.last && hipEventCreateWithFlags(&x.last, hipEventDisableTiming) != hipSuccess) return hipErrorUnknown;
        if (x.owner && x.owner != c) {
            if (!x.marked && !capturing(x.owner->st)) {
                if (hipError_t e = hipEventRecord(x.last, x.owner->st); e != hipSuccess) return e;
                x.marked = true;
            }
            if (x.marked)
                if (hipError_t e = hipStreamWaitEvent(c->st, x.last, 0); e != hipSuccess) return e;
        }
    }
    hipError_t e = launch_tridiag(c->ew, c->d.NP, m0, n, c->st);
    if (shared && e == hipSuccess) e = hipEventRecord(x.last, c->st);
    x.owner = c;
    x.marked = shared && e == hipSuccess;
    hold.unlock();
    if (e == hipSuccess) e = launch_dc(c->ew, c->d.NP, n, c->st);
    if (e == hipSuccess) e = launch_tri_back(c->ew, c->d.NP, m0, n, count, cf, c->st);
    return e;
}

// The Gram matrix of a buffer of which no block is known, with the split-arithmetic kernels: new x top, new x new and, by
// the latter's kernel, top x top (at D = 2,049,000 the fp32 kernel took 5.4 ms for it, this takes 2.6 for bf16 and 2.9 for fp32 rows). The side stream
// is idle here.
int gram_whole_split(sage_ctx* c, hipEvent_t mark = nullptr) {
    const int i = c->par, o = i ^ 1;
    const bool one = new_one(c, c->df.cur);
    RUN(K_GRAM, launch_gram(c->top, c->top, c->fill_top, c->gram_partial_new[o], c->gp_new2_split, c->d, c->st));
    RUN(K_GRAM, launch_gram(c->top, c->nw(c->df.cur), c->fill_new, c->gram_partial_new[i], c->gp_new2_split, c->d, c->st, one));
    RUN(K_GRAM, launch_gram(c->top, c->nw(c->df.cur), c->fill_new, c->gram_partial, c->gp_cross_split, c->d, c->st, one));
    RUN(K_REDUCE, launch_gram_reduce(c->gram_partial, c->gp_cross_split, c->gram_partial_new[i], &c->gp_new2_split, c->ew.C,
                                     false, c->ew.known, c->d, c->st, c->gram_partial_new[o], &c->gp_new2_split, mark));
    return SAGE_OK;
}

// After a shrink the Gram matrix of the top rows is known (diagonal lambda_j - delta, recorded by the shrink). At 64 buffer rows no plan
// leaves that block out (gram64_kernel forms it with the others), and there even a buffer that was just shrunk is decomposed anew for a basis: a
// solve of some 65 us, once a stream.
bool top_known(const sage_ctx* c) { return c->top_shrunk && c->gp_skip.t0 > 0; }

// Gram + eigensolve of the buffer as it stands, and the coefficients of a basis. A block that is known is not recomputed.
int decompose(sage_ctx* c, const CoeffArgs& cf) {
    if (int rc = clear_top(c); rc != SAGE_OK) return rc;
    const bool skip = top_known(c);
    if (!skip && split_grams(c) && !c->new_block_ready && !c->pre_stored) {
        if (int rc = gram_whole_split(c); rc != SAGE_OK) return rc;
    } else if (skip && split_grams(c) && !c->new_block_ready && !c->pre_stored) {
        // the two blocks that are not known, with the split-arithmetic kernels (the side stream is idle here: its
        // partial buffer of the current half is free)
        const bool one = new_one(c, c->df.cur);
        RUN(K_GRAM, launch_gram(c->top, c->nw(c->df.cur), c->fill_new, c->gram_partial, c->gp_cross_split, c->d, c->st, one));
        RUN(K_GRAM, launch_gram(c->top, c->nw(c->df.cur), c->fill_new, c->gram_partial_new[c->par], c->gp_new2_split, c->d,
                                c->st, one));
        RUN(K_REDUCE, launch_gram_reduce(c->gram_partial, c->gp_cross_split, c->gram_partial_new[c->par], &c->gp_new2_split,
                                         c->ew.C, true, c->ew.known, c->d, c->st));
    } else {
        const GramPlan& gp = skip ? c->gp_skip : c->gp;
        if (int rc = widen(c, c->df.cur); rc != SAGE_OK) return rc;
        RUN(K_GRAM, launch_gram(c->top, c->nw(c->df.cur), c->fill_new, c->gram_partial, gp, c->d, c->st));
        RUN(K_REDUCE, launch_gram_reduce(c->gram_partial, gp, nullptr, nullptr, c->ew.C, skip, c->ew.known, c->d, c->st));
    }
    RUN(K_EIG, eigensolve(c, c->fill_top, c->fill_top + c->fill_new, cf.count, &cf));
    return SAGE_OK;
}

// The side stream goes on after what the context stream has been given so far.
int side_follow(sage_ctx* c) {
    if (!c->marked || capturing(c->st)) HIPCHK(hipEventRecord(c->ev_mark, c->st));  // (else it rode on the last launch)
    HIPCHK(hipStreamWaitEvent(c->st2, c->ev_mark, 0));
    return SAGE_OK;
}

// The next ell rows of the running call into another half and their own Gram block, on the side stream.
int side_ahead(sage_ctx* c, const RowSrc* next, const int* hole) {
    const int LP = c->d.LP, ell = c->d.ell, o = c->df.next = c->df.free_half(), pn = c->par ^ 1;
    if (int rc = note_new_rows(c, o, 0, *next); rc != SAGE_OK) return rc;
    c->gp_side_used[pn] = c->mm_mode == SAGE_MM_SPLIT && c->gp_new_split.tiles > 0 ? &c->gp_new_split : &c->gp_new;
    if (c->nw_half[o] && !next->outer() && gram_rows_ok(*c->gp_side_used[pn], c->d)) {
        HIPCHK(launch_gram_rows16(next->G, ell, c->nw(o), c->gram_partial_new[pn], *c->gp_side_used[pn], c->d, hole, c->st2));
        return SAGE_OK;
    }
    HIPCHK(insert_rows(*next, ell, 0, c->nw(o), LP, c->d, c->nw_half[o], c->st2, hole));
    HIPCHK(launch_gram(c->top, c->nw(o), ell, c->gram_partial_new[pn], *c->gp_side_used[pn], c->d, c->st2, new_one(c, o), hole));
    return SAGE_OK;
}

// Whether this shrink may leave its rows unwritten: the block and the next one are kept in the same form.
bool may_defer(const sage_ctx* c, const RowSrc& next) {
    return c->df.max > 0 && c->mm_mode == SAGE_MM_SPLIT && next.dtype == c->dtype &&
           c->nw_bf16[c->df.cur] == (c->dtype == SAGE_BF16) &&
           (c->d.NP < 512 || (c->Mt3 && split_grams(c) && c->nw_half[c->df.cur] == (c->one_part && c->dtype == SAGE_BF16)));
}
// (the blocks are all in the form that may_defer asks for)
bool blocks_one_part(const sage_ctx* c) { return c->one_part && c->dtype == SAGE_BF16; }

// W takes in the last shrink's M.
hipError_t fold_shrink(sage_ctx* c, hipStream_t st) {
    const int n = c->df.count;
    if (n < 1 || n > c->df.max) return hipErrorInvalidValue;  // (what the buffers are made for)
    const double* const from = c->W();
    const int ldf = c->ldw();
    const DeferPlan::Fold f = c->df.fold();
    if (f.out < 0) return hipSuccess;
    return launch_defer_compose(c->last_M(), from, ldf, n * c->d.LP, c->coef[f.out], c->ldw(), c->d, st);
}

// The rows of the deferred shrinks: top <- W [top; blocks].
hipError_t write_rows(sage_ctx* c, hipStream_t st, const int* hole) {
    const int LP = c->d.LP;
    if (!c->df.folded)
        if (hipError_t e = fold_shrink(c, st); e != hipSuccess) return e;
    const NewBlocks b{c->ring, c->half_floats, c->df.slots, c->df.count};
    if (b.count < 1 || b.count > c->df.max) return hipErrorInvalidValue;
    c->df.written();
    if (hipError_t e = launch_defer_coeffs(c->W(), c->ldw(), (1 + b.count) * LP, c->Mt, c->Mt3, c->d, st); e != hipSuccess) return e;
    if (c->Mt3) return launch_rebuild_split(c->top, b, c->d.ell, c->Mt3, c->top, LP, LP, c->d, st, blocks_one_part(c), hole);
    return launch_rebuild(c->top, b, c->d.ell, c->Mt, c->top, LP, LP, c->d, st, hole);
}

// Products of the rows of half o with `top` and with the blocks b, partial tiles one after the other.
const GramPlan& cross_plan(const sage_ctx* c, hipStream_t st) {
    if (c->gp_cross_split.tiles == 0) return c->gp_cross;
    return st == c->st2 ? c->gp_cross_side : c->gp_cross_split;
}
int64_t cross_stride(const sage_ctx* c) { return (int64_t)c->gp_cross.partial_floats; }  // (no plan has more)
hipError_t cross_top(sage_ctx* c, int o, hipStream_t st, const int* hole) {
    return launch_gram_tops(GramTops{{c->top}, 0, c->d.ell}, 1, c->nw(o), c->d.ell, c->gram_partial, cross_plan(c, st), c->d, st,
                            new_one(c, o), hole);
}
hipError_t cross_blocks(sage_ctx* c, int o, const NewBlocks& b, hipStream_t st, const int* hole) {
    const GramPlan& gp = cross_plan(c, st);
    GramTops tops{};
    tops.rows = c->d.ell;
    tops.stride = cross_stride(c);
    for (int j = 0; j < b.count; ++j) tops.p[j] = b.at(j);
    if (c->d.NP == 512 && blocks_one_part(c))
        return launch_gram_blocks(tops, b.count, c->nw(o), c->d.ell, c->gram_partial + tops.stride, gp, c->d, st, hole);
    return launch_gram_tops(tops, b.count, c->nw(o), c->d.ell, c->gram_partial + tops.stride, gp, c->d, st, false, hole);
}
// ... with both, in one launch where their rows have the same form
hipError_t cross_all(sage_ctx* c, int o, const NewBlocks& b, hipStream_t st, const int* hole) {
    if (c->d.NP == 512 && blocks_one_part(c)) {
        if (hipError_t e = cross_top(c, o, st, hole); e != hipSuccess) return e;
        return cross_blocks(c, o, b, st, hole);
    }
    GramTops tops{};
    tops.rows = c->d.ell;
    tops.stride = cross_stride(c);
    tops.p[0] = c->top;
    for (int j = 0; j < b.count; ++j) tops.p[1 + j] = b.at(j);
    return launch_gram_tops(tops, 1 + b.count, c->nw(o), c->d.ell, c->gram_partial, cross_plan(c, st), c->d, st, false, hole);
}
// (the products with the blocks were formed on the side stream, those with the top by the same stream as this)
hipError_t cross_reduce(sage_ctx* c, int sources, const int* col, hipStream_t st) {
    const int pn = c->par ^ 1;
    return launch_defer_reduce(c->gram_partial, cross_stride(c), sources, col, cross_plan(c, st).groups, cross_plan(c, c->st2).groups,
                               c->gram_partial_new[pn], *c->gp_side_used[pn], c->K, c->ldk, c->C_next, c->d, st);
}

// The blocks whose shrink is deferred, with the current one.
NewBlocks blocks_and_cur(const sage_ctx* c) { return NewBlocks{c->ring, c->half_floats, c->df.slots_with_cur(), c->df.count + 1}; }

// Beside the eigensolve of a shrink that will be deferred, on the side stream: the rows of earlier ones where it is time, the
// next block, and its products with the buffer of the running shrink (columns 0 .. 2 LP - 1 of K).
int side_defer(sage_ctx* c, const RowSrc* next, bool write_first, const int* hole) {
    const int LP = c->d.LP;
    if (!c->df.folded) HIPCHK(fold_shrink(c, c->st2));
    if (write_first) HIPCHK(write_rows(c, c->st2, hole));
    if (int rc = side_ahead(c, next, hole); rc != SAGE_OK) return rc;
    const int n = c->df.count;
    HIPCHK(cross_all(c, c->df.next, blocks_and_cur(c), c->st2, hole));
    int col[GRAM_TOPS];
    col[0] = n > 0 ? 2 * LP : 0;
    for (int j = 0; j < n; ++j) col[1 + j] = (3 + j) * LP;
    col[n + 1] = LP;
    HIPCHK(cross_reduce(c, n + 2, col, c->st2));
    if (n > 0) HIPCHK(launch_defer_fold(c->K + 2 * LP, c->ldk, c->W(), c->ldw(), (1 + n) * LP, c->K, c->ldk, c->d, c->st2));
    return SAGE_OK;
}

// The buffer is full: shrink it (Method, FD paragraph). Leaves top = the ell new rows and another new half current.
// next / next_rows: what is left of the running update call after this buffer. If a whole further cycle of rows is
// there, they are stored in another new half and their own Gram block is formed on the side stream while the
// eigensolve runs on the context stream (neither needs its result, and the eigensolve leaves most of the chip idle). Where
// shrinks are deferred (fd_defer.hip), so are the products with the buffer, and the rows may stay unwritten.
int shrink(sage_ctx* c, const RowSrc* next, int64_t next_rows) {
    const int LP = c->d.LP, ell = c->d.ell;
    const bool ahead = use_side(c) && !c->prof && next && next_rows >= ell;
    const bool cap = capturing(c->st);
    const DeferPlan::Step step = c->df.step(ahead, ahead && may_defer(c, *next), next_rows, ell);
    const hipEvent_t mark = ahead && !cap ? c->ev_mark : nullptr;
    const bool have_C = c->C_ready;
    c->C_ready = false;
    if (have_C) {
        // formed after the last eigensolve
    } else if (c->new_block_ready || (c->top_shrunk && c->gp_cross.tiles > 0)) {
        // The top x top block is known. The new x new block came from the side stream, or is formed here when there
        // was nothing to look ahead to (first cycle of a call); then only new x top is left.
        const bool split = c->mm_mode == SAGE_MM_SPLIT;
        const GramPlan* gn = c->gp_side_used[c->par];
        if (c->new_block_ready) {
            HIPCHK(hipStreamWaitEvent(c->st, c->ev_side[c->par], 0));
        } else {
            gn = split && c->gp_new2_split.tiles > 0 ? &c->gp_new2_split : &c->gp_new2;
            RUN(K_GRAM, launch_gram(c->top, c->nw(c->df.cur), ell, c->gram_partial_new[c->par], *gn, c->d, c->st,
                                    new_one(c, c->df.cur)));
        }
        const GramPlan& gc = split && c->gp_cross_split.tiles > 0 ? c->gp_cross_split : c->gp_cross;
        RUN(K_GRAM, launch_gram(c->top, c->nw(c->df.cur), ell, c->gram_partial, gc, c->d, c->st, new_one(c, c->df.cur)));
        RUN(K_REDUCE, launch_gram_reduce(c->gram_partial, gc, c->gram_partial_new[c->par], gn, c->ew.C, true,
                                         c->ew.known, c->d, c->st, nullptr, nullptr, mark));
        c->marked = mark != nullptr;
    } else if (!c->top_shrunk && split_grams(c)) {
        if (int rc = gram_whole_split(c, mark); rc != SAGE_OK) return rc;
        c->marked = mark != nullptr;
    } else {
        const bool skip = c->top_shrunk && c->gp_skip.t0 > 0;
        const GramPlan& gp = skip ? c->gp_skip : c->gp;
        if (int rc = widen(c, c->df.cur); rc != SAGE_OK) return rc;
        RUN(K_GRAM, launch_gram(c->top, c->nw(c->df.cur), ell, c->gram_partial, gp, c->d, c->st));
        RUN(K_REDUCE, launch_gram_reduce(c->gram_partial, gp, nullptr, nullptr, c->ew.C, skip, c->ew.known, c->d, c->st, nullptr, nullptr, mark));
        c->marked = mark != nullptr;
    }
    c->new_block_ready = false;
    if (ahead) {
        // after the Gram launches of this cycle: started beside them, the side stream's work (all of it, or the insert
        // alone) slowed the cross block more than it gained under the eigensolve (28.4 k against 29.7 k rows/s at
        // D = 2,049,000, both ways)
        if (int rc = side_follow(c); rc != SAGE_OK) return rc;
        int* const hole = c->ew.period == 8 ? c->side_hole : nullptr;
        if (hole) HIPCHK(launch_xcd_place(c->ew.xcd, hole, c->st2));
        if (int rc = step.defer && c->df.beside ? side_defer(c, next, step.write_first, hole) : side_ahead(c, next, hole); rc != SAGE_OK) return rc;
        if (step.defer && !c->df.beside && !step.last) HIPCHK(cross_blocks(c, c->df.next, blocks_and_cur(c), c->st2, hole));
        HIPCHK(hipEventRecord(c->ev_side[c->par ^ 1], c->st2));
    } else if (step.write_first) {
        RUN(K_REBUILD, write_rows(c, c->st, nullptr));
    } else if (c->df.count > 0 && !c->df.folded) {
        RUN(K_REDUCE, fold_shrink(c, c->st));  // (with the count it was made for)
    }
    const bool split_rb = c->mm_mode == SAGE_MM_SPLIT && c->Mt3, write_now = !step.defer && c->df.count == 0;
    CoeffArgs cf{LP, ell - 1, 0, c->d.n, ell, c->cnt_top, c->fill_top, LP + c->cnt_new, LP + c->fill_new, c->Mt,
                 split_rb ? c->Mt3 : nullptr, c->acc};  // (row ell - 1 of the result is zero)
    if (!write_now) cf.M = c->coef[c->df.next_m()];
    // At 64 buffer rows the reduction's launch stores them (`inline_rows`), into the half that is not in use.
    const bool inline_rows = c->d.NP == 64 && c->halves > 1 && !c->prof && next && next_rows >= ell && !cap;
    RowJob job{};
    if (inline_rows) {
        job = RowJob{next->G, next->E, next->H, next->C, next->dh, next->dtype, ell, c->nw(c->df.cur ^ 1), c->d};
        if (int rc = note_new_rows(c, c->df.cur ^ 1, 0, *next); rc != SAGE_OK) return rc;
    }
    RUN(K_EIG, eigensolve(c, ell, 2 * ell, cf.count, &cf, inline_rows ? &job : nullptr));
    const NewBlocks one{c->ring, c->half_floats, (unsigned)c->df.cur, 1};
    c->marked = false;
    if (inline_rows) {
        RUN(K_REBUILD, launch_rebuild_gram(c->top, c->nw(c->df.cur), c->nw(c->df.cur ^ 1), c->Mt, c->gram_partial, c->gp, c->d, c->st));
        RUN(K_REDUCE, launch_gram_reduce(c->gram_partial, c->gp, nullptr, nullptr, c->ew.C, false, c->ew.known, c->d, c->st));
        c->C_ready = true;
    } else if (write_now) {
        if (split_rb)
            RUN(K_REBUILD, launch_rebuild_split(c->top, one, ell, c->Mt3, c->top, LP, LP, c->d, c->st, new_one(c, c->df.cur)));
        else
            RUN(K_REBUILD, launch_rebuild(c->top, one, ell, c->Mt, c->top, LP, LP, c->d, c->st));
    } else {
        c->df.push();
        c->df.made_m();
        const double* W = c->last_M();
        int ldw = c->d.NP, len = 2 * LP;
        if (step.defer && !c->df.beside) {
            RUN(K_REDUCE, fold_shrink(c, c->st));
            if (!step.last) {
                HIPCHK(hipStreamWaitEvent(c->st, c->ev_side[c->par ^ 1], 0));
                RUN(K_GRAM, cross_top(c, c->df.next, c->st, nullptr));
                int col[GRAM_TOPS];
                for (int j = 0; j <= c->df.count; ++j) col[j] = j * LP;
                RUN(K_REDUCE, cross_reduce(c, 1 + c->df.count, col, c->st));
                W = c->W();
                ldw = c->ldw();
                len = (1 + c->df.count) * LP;
                c->C_ready = true;
            }
        } else if (step.defer) {
            HIPCHK(hipStreamWaitEvent(c->st, c->ev_side[c->par ^ 1], 0));
            c->C_ready = true;
        }
        if (c->C_ready) {
            RUN(K_REDUCE, launch_defer_cross(c->K, c->ldk, W, ldw, len, c->C_next, c->ew.known, c->d, c->st, c->ev_mark));
            double* const C = c->ew.C;
            c->ew.C = c->C_next;
            c->C_next = C;
            c->marked = true;
        }
        if (!step.defer || step.last) {
            RUN(K_REBUILD, write_rows(c, c->st, nullptr));
            c->marked = false;
        }
    }
    if (use_side(c)) {
        c->df.advance(ahead);
        c->par ^= 1;
    } else {
        c->df.cur = inline_rows ? c->df.cur ^ 1 : 0;  // (0 whenever a call ends, so that a captured one can be replayed)
    }
    c->fill_top = ell;
    c->cnt_top = ell;
    c->fill_new = 0;
    c->cnt_new = 0;
    c->pre_stored = ahead || inline_rows;
    c->new_block_ready = ahead;
    c->n_shrinks += 1;
    c->top_shrunk = true;
    return SAGE_OK;
}

// A shrink that was left for the next update call: do it now (something wants to see the sketch).
int flush_pending(sage_ctx* c) {
    if (!c->pending_shrink) return SAGE_OK;
    c->pending_shrink = false;
    return shrink(c, nullptr, 0);
}

void reset_scoring(sage_ctx* c) {
    c->n_scored = 0;
    c->n_rescored = 0;
    c->n_labeled = 0;
    c->alpha_n = 0;
}

int ensure_score_buffers(sage_ctx* c) {
    if (!c->ssum) {
        ALLOC(c->ssum, 128 * sizeof(double) + 256);
        c->ticket = (unsigned*)(c->ssum + 128);
        HIPCHK(hipMemsetAsync(c->ssum, 0, 128 * sizeof(double) + 256, c->st));
    }
    if (!c->cons_partial) ALLOC(c->cons_partial, (size_t)(SCORE_CHUNK / 4) * 128 * sizeof(double));  // one per 4 rows
    return SAGE_OK;
}

int ensure_vblk(sage_ctx* c, int KP) {
    if (c->Vblk && c->Vblk_KP == KP) return SAGE_OK;
    if (c->Vblk) {
        HIPCHK(hipStreamSynchronize(c->st));
        FREE(c->Vblk);
    }
    ALLOC(c->Vblk, (size_t)c->d.S * KP * DC * sizeof(float));
    c->Vblk_KP = KP;
    return SAGE_OK;
}

// The images of the basis in Vblk in so many bf16 parts (score_split.hip). Either number has memory of its own, so that a pass
// that takes factored rows and row-major rows of another alignment in turn does not make them anew each time; where there is not
// room for both, the other one's is given up.
int ensure_images(sage_ctx* c, int parts) {
    BasisImages& im = c->img[parts - 2];
    if (im.current) return SAGE_OK;
    const size_t need = basis_image_bytes(c->KP, c->dtype, parts, c->d);
    if (need > im.bytes) {
        BasisImages& other = c->img[3 - parts];
        if (im.mem) HIPCHK(hipStreamSynchronize(c->st));
        FREE(im.mem);
        im.bytes = 0;
        if (!late_alloc(c, &im.mem, need)) {
            if (!other.mem || c->poisoned) return NO_MEMORY(c);
            HIPCHK(hipStreamSynchronize(c->st));
            FREE(other.mem);
            other = BasisImages{};
            ALLOC(im.mem, need);
        }
        im.bytes = need;
    }
    RUN(K_REBUILD, launch_basis_split(c->Vblk, c->KP, c->dtype, parts, im.mem, c->d, c->st));
    im.current = true;
    return SAGE_OK;
}

// After Vblk holds a new basis: build the images when the split projection can be used for row-major batches of
// this D (factored rows, and rows of other widths, build theirs on first use).
int finish_basis(sage_ctx* c) {
    c->img_ok = false;
    for (BasisImages& im : c->img) im.current = false;
    if (c->proj_mode == SAGE_PROJ_F32) return SAGE_OK;
    if (!split_path_ok(nullptr, c->dtype, c->d)) return SAGE_OK;  // nullptr is "aligned": only D is judged here
    int rc = ensure_images(c, 2);
    if (rc != SAGE_OK) return rc;
    c->img_ok = true;
    return SAGE_OK;
}

// Which contexts defer shrinks (fd_defer.hip). Us a cycle, at once / deferred, for calls of four cycles, medians of seven in turn; runs of
// one side differ by 3%.
// Beside the eigensolves while all work on the rows of a cycle is done before an eigensolve is; it then takes the insert, rectangles,
// a triangle and the rebuild on seven XCDs instead of one rectangle and the rebuild in series. The lines lie where the two cross:
//   ell = 64, fp32 rows:  216 / 200 (D = 131,072), 228 / 222 (163,840), 240 / 250 (196,608), 262 / 306 (262,144)
//   ell = 100:            368 / 342, 395 / 390, 410 / 435, 451 / 544        ell = 128: 414 / 369, 436 / 402, 457 / 450, 496 / 560
//   (bf16 rows the same within 3%)
//   ell = 256, fp32 rows: 863 / 835 (65,536), 931 / 914 (98,304), 945 / 961 (114,688), 967 / 1071 (131,071)
//   ell = 200:            718 / 695, 795 / 761, 807 / 798, 809 / 878        ell = 136: 540 / 521, 611 / 593, 624 / 618, 642 / 683
// Three blocks where that costs next to nothing: the rows are rounded to fp32 a third as often. At 512 buffer rows it would cost a tenth
// (bf16, 131,072: 946 where one block takes 853).
// Beyond, several at a time where that is less work: rows with one part cost three products per element in a rebuild, the top's six,
// so two shrinks at once take 12 where one by one they take 18, for one more rectangle of one product (1,048,576: 2332 / 1994).
// Against one beside each eigensolve (bf16, beside / two at a time): ell = 256, 852 / 864 (131,072), 910 / 929 (163,840),
// 954 / 939 (196,608), 1082 / 1034 (262,144), 1189 / 1069 (327,680); ell = 200, 725 / 735, 762 / 775, 786 / 781, 886 / 835, 992 / 911. For
// rows of three parts it would be as much work as before. Up to four at once take 18 where two by two they take 24, for three rectangles
// more, which are formed beside the eigensolves as long as these last; and two halves more of memory. Two / up to four at a time, calls
// of 4 cycles: ell = 256, 942 / 945 (190,000), 1081 / 1075 (300,000), 1424 / 1372 (600,000), 3190 / 3100 (2,049,000); ell = 200, 852 / 837
// (260,000), 1644 / 1500 (1,000,000); calls of 3 and of 5 cycles gain more (an odd one is not left alone).
// Below 524,288 columns what four gain over two, half a per cent to two, is less than runs of one side differ by: not worth the memory.
void defer_plan(sage_ctx* c) {
    const int64_t D = c->d.D;
    if (c->d.NP < 128) return;
    const bool one = c->dtype == SAGE_BF16 && c->d.NP == 512;
    c->df.beside = D <= (c->d.NP < 512 ? 196608 : one ? 180224 : 98304);
    c->df.max = c->df.beside ? (c->d.NP < 512 ? 3 : 1) : one ? (D < 524288 ? 2 : 4) : 0;
}

int64_t keep_count(double keep_rate, int64_t N) {
    double x = floor(keep_rate * (double)N + 0.5);
    int64_t m = (int64_t)x;
    if (m < 0) m = 0;
    if (m > N) m = N;
    return m;
}

// one allocation: histograms, state, counters and tables
size_t select_work_bytes(int64_t N) { return topm_work_words(topm_work_blocks(N)) * sizeof(uint32_t); }

}  // namespace

extern "C" {

const char* sage_strerror(int code) {
    switch (code) {
        case SAGE_OK: return "ok";
        case SAGE_ERR_ARG: return "bad argument";
        case SAGE_ERR_STATE: return "call not allowed in this state";
        case SAGE_ERR_ALLOC: return "allocation failed";
        case SAGE_ERR_HIP: return "HIP runtime error";
        case SAGE_ERR_CAPACITY: return "capacity exceeded";
        default: return "unknown status";
    }
}

int sage_set_allocator(sage_alloc_fn alloc, sage_free_fn free_, void* user) {
    if ((alloc == nullptr) != (free_ == nullptr)) return SAGE_ERR_ARG;
    std::lock_guard<std::mutex> hold(g_mem_lock);
    g_mem.alloc = alloc;
    g_mem.free = free_;
    g_mem.user = user;
    return SAGE_OK;
}

// less: how many plans smaller than the usual one, for the halves that storing rows ahead (64 buffer rows) and deferring shrinks take.
// more: there is a smaller one still.
static int create(sage_ctx** out, int ell, int64_t D, sage_dtype in_dtype, int64_t max_rows, void* hip_stream, int less, bool& more) {
    *out = nullptr;
    more = false;
    if (ell < 2 || ell > 256 || D < 1 || max_rows < 0) return SAGE_ERR_ARG;
    if (in_dtype != SAGE_F32 && in_dtype != SAGE_BF16) return SAGE_ERR_ARG;
    sage_ctx* c = new (std::nothrow) sage_ctx();
    if (!c) return SAGE_ERR_ALLOC;
    c->d.ell = ell;
    c->d.n = 2 * ell;
    c->d.LP = pad_pow2_32(ell);
    c->d.NP = 2 * c->d.LP;
    c->d.D = D;
    c->d.S = (D + DC - 1) / DC;
    c->d.Dp = c->d.S * DC;
    c->dtype = in_dtype;
    c->st = (hipStream_t)hip_stream;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        (void)hipGetLastError();
        delete c;
        return SAGE_ERR_HIP;
    }
    c->device = dev;
    c->num_cu = cus > 0 ? cus : 256;
    {
        std::lock_guard<std::mutex> hold(g_mem_lock);
        c->mem = g_mem;
    }
    const int P = c->d.NP / 64;
    c->gp = gram_plan(c->d, c->num_cu, 0, false, 2);
    c->gp_skip = gram_plan(c->d, c->num_cu, 0, P >= 2, 2);
    if (P >= 2) {
        c->gp_cross = gram_plan(c->d, c->num_cu, 1, false, 2);
        c->gp_new = gram_plan(c->d, c->num_cu, 2, false, 1);
        c->gp_new2 = gram_plan(c->d, c->num_cu, 2, false, 2);
        c->gp_cross_split = gram_plan_split(c->gp_cross, c->d, 0);
        c->gp_new2_split = gram_plan_split(c->gp_new2, c->d, 0);
        // beside the eigensolve: one work-group per CU of the seven XCDs that it leaves alone, so that the kernels after
        // the reduction find room beside them
        const int side = c->num_cu > 32 ? c->num_cu / 8 * 7 : 8;
        c->gp_new_split = gram_plan_split(c->gp_new2, c->d, side);
        // The new x top kernels fill a CU, and the kernels after the reduction that do not fit beside them (divide and conquer's
        // blocks: 77 KB of LDS) come to all XCDs: one CU of each is left to them (those blocks of 512 rows 290 -> 60 us; a launch for
        // two or three blocks of a wide bf16 stream has as many again for each and leaves none: 300 us). As many
        // work-groups as the whole chip holds took two rounds of the 224 CUs.
        c->gp_cross_side = gram_plan_split(c->gp_cross, c->d, side > 56 ? side - 7 : side);
    }
    c->fixed_cap = max_rows > 0;
    c->cap_rows = max_rows > 0 ? max_rows : 65536;

    auto fail = [&](int rc) {
        sage_destroy(c);
        return rc;
    };
    const int NP = c->d.NP;
    size_t hbytes = (size_t)c->d.S * c->d.LP * DC * sizeof(float);  // one half buffer
    if (!kit_take(dev, c->kit)) return fail(SAGE_ERR_HIP);
#define CALLOC(ptr, bytes)                                                        \
    do {                                                                          \
        if (!dev_alloc(c->mem, c->st, (void**)&(ptr), (bytes))) return fail(SAGE_ERR_ALLOC); \
    } while (0)
    defer_plan(c);
    for (int i = 0; i < less; ++i) c->df.max = c->df.fewer();
    more = less == 0 || c->df.max > 0;
    c->half_floats = (int64_t)(hbytes / sizeof(float));
    c->halves = less > 0 && c->d.NP == 64 ? 1 : c->df.halves();
    CALLOC(c->top, hbytes);
    CALLOC(c->ring, (size_t)c->halves * hbytes);
    {
        size_t pf = c->gp.partial_floats;
        if (c->gp_skip.partial_floats > pf) pf = c->gp_skip.partial_floats;
        // deferred shrinks: a block's products with the top and up to defer_max blocks
        const size_t pc = c->gp_cross.partial_floats * (1 + c->df.max);
        if (pc > pf) pf = pc;
        CALLOC(c->gram_partial, pf * sizeof(float));
    }
    if (P >= 2) {
        const size_t pn = c->gp_new.partial_floats > c->gp_new2.partial_floats ? c->gp_new.partial_floats
                                                                                : c->gp_new2.partial_floats;
        CALLOC(c->gram_partial_new[0], pn * sizeof(float));
        CALLOC(c->gram_partial_new[1], pn * sizeof(float));
        c->st2 = c->kit.stream;
        c->ev_mark = c->kit.mark;
        for (int i = 0; i < 2; ++i) c->ev_side[i] = c->kit.side[i];
    }
    {
        // work space of the eigensolve: one allocation, every array on a multiple of 256 bytes
        size_t bytes = 0;
        auto take = [&](auto*& p, size_t count) {
            if (c->eig_mem) p = (std::remove_reference_t<decltype(p)>)(c->eig_mem + bytes);
            bytes += (count * sizeof(*p) + 255) / 256 * 256;
        };
        for (int pass = 0; pass < 2; ++pass) {
            const size_t n1 = (size_t)NP, n2 = n1 * n1;
            EigWork& w = c->ew;
            bytes = 0;
            take(w.xch, 8 * n1);
            take(w.stat, 32);
            take(w.C, n2);
            if (c->df.max > 0) {
                const size_t lp = (size_t)c->d.LP;
                c->ldk = (c->df.max + 2) * c->d.LP;
                take(c->C_next, n2);
                for (int i = 0; i < c->df.MS; ++i) take(c->coef[i], lp * n1);
                for (int i = 0; i < 2; ++i) take(c->coef[c->df.MS + i], lp * lp * (1 + c->df.max));
                take(c->K, lp * c->ldk);
            }
            take(w.Yt, n2);
            take(w.V, n2);
            take(w.Tw, 8 * n1);
            for (int i = 0; i < 2; ++i) take(w.Z[i], n2);
            for (int i = 0; i < 2; ++i) take(w.dI[i], n1);
            for (double** p : {&w.dT, &w.eT, &w.tauT, &w.known, &w.dc.dk, &w.dc.zk, &w.dc.org, &w.dc.tau, &w.dc.val, &w.dc.zh, &w.dc.rc, &w.dc.rs})
                take(*p, n1);
            for (int** p : {&w.dc.col, &w.dc.half, &w.dc.npos, &w.dc.from, &w.dc.ra, &w.dc.rb, &w.dc.K, &w.dc.k1, &w.dc.dense, &w.dc.nrot}) take(*p, n1);
            if (pass == 0) CALLOC(c->eig_mem, bytes);
        }
        xcd_take(c);
    }
    const int brows = (c->df.max > 1 ? 1 + c->df.max : 2) * c->d.LP;
    CALLOC(c->Mt, (size_t)brows * c->d.LP * sizeof(float));
    if (rebuild_split_ok(c->d.LP)) CALLOC(c->Mt3, rebuild_split_bytes(brows, c->d.LP));
    CALLOC(c->acc, 8 * sizeof(double));
    c->ew.redone = c->acc + 4;
    c->ew.claim = (unsigned*)(c->ew.stat + 16);
    c->side_hole = (int*)(c->ew.stat + 24);
#undef CALLOC
    // Rows of the top half that the stream never fills are zero. (Those it has not filled yet are cleared when something
    // looks at them, see clear_top; rows of a new half beyond its fill are never used.)
    if (ell < c->d.LP && launch_zero_rows(c->top, c->d.LP, ell, c->d.LP, c->d, c->st) != hipSuccess) return fail(SAGE_ERR_HIP);
    if (hipMemsetAsync(c->acc, 0, 8 * sizeof(double), c->st) != hipSuccess) return fail(SAGE_ERR_HIP);
    if (hipMemsetAsync(c->ew.stat, 0, 32 * sizeof(double), c->st) != hipSuccess) return fail(SAGE_ERR_HIP);
    if (hipMemsetAsync(c->ew.xch, 0xFF, (size_t)8 * NP * sizeof(double), c->st) != hipSuccess) return fail(SAGE_ERR_HIP);
    *out = c;
    return SAGE_OK;
}

int sage_fd_create_ex(sage_ctx** out, int ell, int64_t D, sage_dtype in_dtype, int64_t max_rows, void* hip_stream) {
    if (!out) return SAGE_ERR_ARG;
    int rc = SAGE_ERR_ALLOC;
    bool more = true;
    for (int less = 0; rc == SAGE_ERR_ALLOC && more; ++less) rc = create(out, ell, D, in_dtype, max_rows, hip_stream, less, more);
    return rc;
}

int sage_fd_create(sage_ctx** out, int ell, int64_t D) { return sage_fd_create_ex(out, ell, D, SAGE_F32, 0, nullptr); }

void sage_destroy(sage_ctx* c) {
    if (!c) return;
    (void)hipStreamSynchronize(c->st);
    if (c->st2) (void)hipStreamSynchronize(c->st2);
    void* ptrs[] = {c->top,     c->ring,     c->gram_partial, c->gram_partial_new[0], c->gram_partial_new[1],
                    c->eig_mem, c->Mt,       c->acc,    c->Vblk,         c->img[0].mem, c->img[1].mem,
                    c->zhat,    c->proj_partial, c->cons_partial, c->ssum, c->alpha, c->labels, c->cb_work, c->stage, c->Mt3, c->dbg_count};
    for (void* p : ptrs) dev_free(c->mem, p);
    xcd_release(c);
    kit_give(c->device, c->kit, !c->poisoned);
    dev_free(c->mem, c->sw.hist);
    if (c->ev0) (void)hipEventDestroy(c->ev0);
    if (c->ev1) (void)hipEventDestroy(c->ev1);
    delete c;
}

int sage_sync(sage_ctx* c) {
    ALIVE(c);
    HIPCHK(hipStreamSynchronize(c->st));
    return SAGE_OK;
}

// Rows of type `dtype` (the context's own for sage_fd_update, fp32 for sage_fd_merge) go through the insert / shrink cycle.
static int update_rows(sage_ctx* c, RowSrc g, int64_t rows) {
    ALIVE(c);
    if (rows < 0) return SAGE_ERR_ARG;
    if (rows == 0) return SAGE_OK;
    c->has_basis = false;
    note_capture(c);
    const int ell = c->d.ell, LP = c->d.LP;
    if (c->pending_shrink) {
        // the buffer filled up exactly at the end of the previous call: with this call's rows at hand the shrink can
        // look ahead
        c->pending_shrink = false;
        int rc = shrink(c, &g, rows);
        if (rc != SAGE_OK) return rc;
    }
    while (rows > 0) {
        int take;
        if (c->fill_top < ell) {
            // first fill of the buffer: rows go into the top half
            take = (int)((int64_t)(ell - c->fill_top) < rows ? (ell - c->fill_top) : rows);
            RUN(K_INSERT, insert_rows(g, take, c->fill_top, c->top, LP, c->d, false, c->st));
            c->fill_top += take;
        } else if (c->pre_stored) {
            // the previous shrink of this call has had these ell rows stored already
            take = ell;
            c->pre_stored = false;
            c->fill_new = ell;
        } else {
            take = (int)((int64_t)(ell - c->fill_new) < rows ? (ell - c->fill_new) : rows);
            if (int rc = note_new_rows(c, c->df.cur, c->fill_new, g); rc != SAGE_OK) return rc;
            RUN(K_INSERT, insert_rows(g, take, c->fill_new, c->nw(c->df.cur), LP, c->d, c->nw_half[c->df.cur], c->st));
            c->fill_new += take;
        }
        c->rows_seen += take;
        g = g.after(take, c->d.D);
        rows -= take;
        if (c->fill_new == ell) {
            if (rows == 0 && use_side(c) && c->top_shrunk && !c->prof) {
                // Nothing to look ahead to: leave the shrink to the next update call, which brings rows (whoever
                // looks at the sketch first does it otherwise). The side stream may still be reading this batch for
                // the half just completed: the context stream waits for it, so that the batch is free once this
                // call's work is complete there.
                c->pending_shrink = true;
                if (c->new_block_ready) HIPCHK(hipStreamWaitEvent(c->st, c->ev_side[c->par], 0));
            } else {
                int rc = shrink(c, &g, rows);
                if (rc != SAGE_OK) return rc;
            }
        }
    }
    return SAGE_OK;
}

// sage_set_debug_checks: a batch with a non-finite entry is refused before anything is enqueued for it (the scan
// waits for the stream; the context is left as it was).
static int check_finite(sage_ctx* c, const void* p, int dtype, int64_t n) {
    if (!c->debug_checks || n <= 0 || !p) return SAGE_OK;
    if (!c->dbg_count) ALLOC(c->dbg_count, sizeof(unsigned));
    unsigned bad = 0;
    HIPCHK(hipMemsetAsync(c->dbg_count, 0, sizeof(unsigned), c->st));
    HIPCHK(launch_count_nonfinite(p, dtype, n, c->dbg_count, c->st));
    HIPCHK(hipMemcpyAsync(&bad, c->dbg_count, sizeof(unsigned), hipMemcpyDeviceToHost, c->st));
    HIPCHK(hipStreamSynchronize(c->st));
    return bad ? SAGE_ERR_ARG : SAGE_OK;
}

static RowSrc dense_src(const void* G, int dtype) {
    RowSrc s;
    s.G = G;
    s.dtype = dtype;
    return s;
}

// factored rows must tile the context's row exactly: D = C * (dh + 1)
static bool outer_src(const sage_ctx* c, const void* E, const void* H, int64_t C, int64_t dh, RowSrc& s) {
    if (!E || !H || C < 1 || dh < 1 || dh > ((int64_t)1 << 40) / C || C * (dh + 1) != c->d.D) return false;
    s.E = E;
    s.H = H;
    s.C = C;
    s.dh = dh;
    s.dtype = c->dtype;
    return true;
}

int sage_fd_update(sage_ctx* c, const void* G_batch, int64_t rows) {
    ALIVE(c);
    if (rows > 0 && !G_batch) return SAGE_ERR_ARG;
    if (int rc = check_finite(c, G_batch, c->dtype, rows * c->d.D); rc != SAGE_OK) return rc;
    return update_rows(c, dense_src(G_batch, c->dtype), rows);
}

int sage_fd_update_outer(sage_ctx* c, const void* E, const void* H, int64_t rows, int64_t n_classes, int64_t n_features) {
    ALIVE(c);
    if (rows < 0) return SAGE_ERR_ARG;
    if (rows == 0) return SAGE_OK;
    RowSrc s;
    if (!outer_src(c, E, H, n_classes, n_features, s)) return SAGE_ERR_ARG;
    if (int rc = check_finite(c, E, c->dtype, rows * n_classes); rc != SAGE_OK) return rc;
    if (int rc = check_finite(c, H, c->dtype, rows * n_features); rc != SAGE_OK) return rc;
    return update_rows(c, s, rows);
}

int sage_fd_merge(sage_ctx* c, const float* B_other, int64_t rows) {
    ALIVE(c);
    if (rows > 0 && !B_other) return SAGE_ERR_ARG;
    if (int rc = check_finite(c, B_other, SAGE_F32, rows * c->d.D); rc != SAGE_OK) return rc;
    return update_rows(c, dense_src(B_other, SAGE_F32), rows);
}

static int basis_impl(sage_ctx* c, int k, bool weighted);

int sage_fd_basis(sage_ctx* c, int k) { return basis_impl(c, k, false); }

int sage_fd_basis_weighted(sage_ctx* c, int k) { return basis_impl(c, k, true); }

static int basis_impl(sage_ctx* c, int k, bool weighted) {
    ALIVE(c);
    if (k < 1 || k > c->d.ell - 1 || k > 128) return SAGE_ERR_ARG;
    const int KP = pad_pow2_32(k);
    note_capture(c);
    int rc = flush_pending(c);
    if (rc != SAGE_OK) return rc;
    rc = ensure_vblk(c, KP);
    if (rc != SAGE_OK) return rc;
    const bool shrunk = top_known(c) && c->fill_new == 0;  // only the rows the last shrink wrote are there: nothing to decompose
    const bool split_rb = c->mm_mode == SAGE_MM_SPLIT && c->Mt3 && rebuild_split_ok(KP) && KP <= c->d.LP;
    const CoeffArgs cf{KP, k, weighted ? 2 : 1, c->d.n, c->d.ell, c->cnt_top, c->fill_top, c->d.LP + c->cnt_new,
                       c->d.LP + c->fill_new, c->Mt, split_rb ? c->Mt3 : nullptr, c->acc};
    if (!shrunk) {  // (of a shrunk buffer's rows all are counted in ||A||_F^2)
        rc = decompose(c, cf);
        if (rc != SAGE_OK) return rc;
    }
    c->cnt_top = c->fill_top;
    c->cnt_new = c->fill_new;
    const NewBlocks rows{c->ring, c->half_floats, (unsigned)c->df.cur, 1};
    if (shrunk)
        RUN(K_REBUILD, launch_basis_rows(c->top, c->ew.known, k, cf.mode, c->Vblk, KP, c->d, c->st));
    else if (split_rb)
        RUN(K_REBUILD, launch_rebuild_split(c->top, rows, c->fill_new, c->Mt3, c->Vblk, KP, KP, c->d, c->st,
                                            c->fill_new > 0 && new_one(c, c->df.cur)));
    else {
        if (c->fill_new > 0)
            if (int rcw = widen(c, c->df.cur); rcw != SAGE_OK) return rcw;
        RUN(K_REBUILD, launch_rebuild(c->top, rows, c->fill_new, c->Mt, c->Vblk, KP, KP, c->d, c->st));
    }
    c->k = k;
    c->KP = KP;
    rc = finish_basis(c);
    if (rc != SAGE_OK) return rc;
    c->has_basis = true;
    reset_scoring(c);
    return ensure_score_buffers(c);
}

int sage_set_projection_mode(sage_ctx* c, int mode) {
    ALIVE(c);
    if ((mode != SAGE_PROJ_AUTO && mode != SAGE_PROJ_F32)) return SAGE_ERR_ARG;
    c->proj_mode = mode;
    c->has_basis = false;
    return SAGE_OK;
}

int sage_set_update_arithmetic(sage_ctx* c, int mode) {
    ALIVE(c);
    if (mode != SAGE_MM_F32 && mode != SAGE_MM_SPLIT && mode != SAGE_MM_SPLIT_ALL_PARTS) return SAGE_ERR_ARG;
    c->mm_mode = mode == SAGE_MM_F32 ? SAGE_MM_F32 : SAGE_MM_SPLIT;
    c->one_part = mode != SAGE_MM_SPLIT_ALL_PARTS;
    c->C_ready = false;  // a shrink that is pending forms its products in the new arithmetic
    if (mode != SAGE_MM_SPLIT)
        for (int i = 0; i < c->halves; ++i)
            if (int rc = widen(c, i); rc != SAGE_OK) return rc;
    return SAGE_OK;
}

int sage_set_basis(sage_ctx* c, const float* Vt, int k) {
    ALIVE(c);
    if (!Vt || k < 1 || k > 128) return SAGE_ERR_ARG;
    const int KP = pad_pow2_32(k);
    int rc = ensure_vblk(c, KP);
    if (rc != SAGE_OK) return rc;
    HIPCHK(launch_import_rows(Vt, k, c->Vblk, KP, c->d, c->st));
    c->k = k;
    c->KP = KP;
    rc = finish_basis(c);
    if (rc != SAGE_OK) return rc;
    c->has_basis = true;
    reset_scoring(c);
    return ensure_score_buffers(c);
}

// split-K partial projections of one launch
static int ensure_partial(sage_ctx* c, size_t need) {
    if (need <= c->proj_partial_floats) return SAGE_OK;
    if (c->proj_partial) {
        HIPCHK(hipStreamSynchronize(c->st));
        FREE(c->proj_partial);
        c->proj_partial_floats = 0;
    }
    size_t want = (size_t)512 * 128 * 128 > need ? (size_t)512 * 128 * 128 : need;
    ALLOC(c->proj_partial, want * sizeof(float));
    c->proj_partial_floats = want;
    return SAGE_OK;
}

// staging memory of the factored scoring calls
static int ensure_stage(sage_ctx* c, size_t need) {
    if (need <= c->stage_bytes) return SAGE_OK;
    if (c->stage) {
        HIPCHK(hipStreamSynchronize(c->st));
        FREE(c->stage);
        c->stage_bytes = 0;
    }
    ALLOC(c->stage, need);
    c->stage_bytes = need;
    return SAGE_OK;
}

// The projection partials of R rows (R <= SCORE_CHUNK) in proj_partial; *slots = partial slots to sum.
static int project_rows(sage_ctx* c, const RowSrc& src, int64_t R, int* slots) {
    const void* g = src.G;
    if (src.outer()) {
        if (c->proj_mode != SAGE_PROJ_F32 && outer_path_ok(src.E, src.H, src.dtype, src.C, src.dh)) {
            int rc = ensure_images(c, 2);
            if (rc != SAGE_OK) return rc;
            rc = ensure_stage(c, outer_work_bytes(R, src.dtype, src.C));
            if (rc != SAGE_OK) return rc;
            ScorePlan p = score_outer_plan(R, src.dtype, src.C, src.dh, c->num_cu);
            rc = ensure_partial(c, (size_t)(p.splits + p.bias_slots) * R * c->KP);
            if (rc != SAGE_OK) return rc;
            RUN(K_PROJECT, launch_project_outer(src.E, src.H, src.dtype, R, src.C, src.dh, c->stage, c->img[0].mem, c->Vblk,
                                                c->KP, c->proj_partial, p, c->st));
            *slots = p.splits + p.bias_slots;
            return SAGE_OK;
        }
        // any other shape: write the rows out and project them like a row-major batch
        int rc = ensure_stage(c, (size_t)R * c->d.D * (src.dtype == SAGE_BF16 ? 2 : 4));
        if (rc != SAGE_OK) return rc;
        RUN(K_INSERT, launch_expand_outer(src.E, src.H, src.dtype, src.C, src.dh, R, c->stage, c->d, c->st));
        g = c->stage;
    }
    int parts = c->img_ok && split_path_ok(g, c->dtype, c->d) ? 2 : 0;
    if (!parts && c->proj_mode != SAGE_PROJ_F32 && any_path_ok(g, c->dtype, c->d)) parts = 3;
    if (parts) {
        if (int rc = ensure_images(c, parts); rc != SAGE_OK) return rc;
    }
    ScorePlan p = parts ? score_split_plan(R, c->dtype, c->d, c->num_cu) : score_plan(R, c->d, c->num_cu);
    int rc = ensure_partial(c, (size_t)p.splits * R * c->KP);
    if (rc != SAGE_OK) return rc;
    if (parts)
        RUN(K_PROJECT, launch_project_split(g, c->dtype, R, parts, c->img[parts - 2].mem, c->KP, c->proj_partial, p, c->d, c->st));
    else
        RUN(K_PROJECT, launch_project(g, c->dtype, R, c->Vblk, c->KP, c->proj_partial, p, c->d, c->st));
    *slots = p.splits;
    return SAGE_OK;
}

static int score_impl(sage_ctx* c, RowSrc g, const int* labels, int64_t rows);

int sage_score(sage_ctx* c, const void* G_batch, int64_t rows) {
    ALIVE(c);
    if (rows > 0 && !G_batch) return SAGE_ERR_ARG;
    if (int rc = check_finite(c, G_batch, c->dtype, rows * c->d.D); rc != SAGE_OK) return rc;
    return score_impl(c, dense_src(G_batch, c->dtype), nullptr, rows);
}

int sage_score_labeled(sage_ctx* c, const void* G_batch, const int32_t* labels, int64_t rows) {
    ALIVE(c);
    if (rows > 0 && (!labels || !G_batch)) return SAGE_ERR_ARG;
    if (int rc = check_finite(c, G_batch, c->dtype, rows * c->d.D); rc != SAGE_OK) return rc;
    return score_impl(c, dense_src(G_batch, c->dtype), labels, rows);
}

int sage_score_outer(sage_ctx* c, const void* E, const void* H, const int32_t* labels, int64_t rows, int64_t n_classes,
                     int64_t n_features) {
    ALIVE(c);
    if (rows < 0) return SAGE_ERR_ARG;
    if (!c->has_basis) return SAGE_ERR_STATE;
    if (rows == 0) return SAGE_OK;
    RowSrc s;
    if (!outer_src(c, E, H, n_classes, n_features, s)) return SAGE_ERR_ARG;
    if (int rc = check_finite(c, E, c->dtype, rows * n_classes); rc != SAGE_OK) return rc;
    if (int rc = check_finite(c, H, c->dtype, rows * n_features); rc != SAGE_OK) return rc;
    return score_impl(c, s, labels, rows);
}

static int score_impl(sage_ctx* c, RowSrc g, const int* labels, int64_t rows) {
    ALIVE(c);
    if (rows < 0) return SAGE_ERR_ARG;
    if (!c->has_basis) return SAGE_ERR_STATE;
    if (rows == 0) return SAGE_OK;
    if (!c->store_zhat && (labels || c->n_rescored > 0)) return SAGE_ERR_STATE;  // no labels without zhat; pass 2 is over
    if (c->store_zhat && !c->zhat) ALLOC(c->zhat, (size_t)c->cap_rows * 128 * sizeof(float));
    if (c->store_zhat && c->n_scored + rows > c->cap_rows) {
        if (c->fixed_cap) return SAGE_ERR_CAPACITY;
        int64_t ncap = c->cap_rows;
        while (ncap < c->n_scored + rows) ncap *= 2;
        float* nz = nullptr;
        ALLOC(nz, (size_t)ncap * 128 * sizeof(float));
        if (hipMemcpyAsync(nz, c->zhat, (size_t)c->n_scored * c->k * sizeof(float), hipMemcpyDeviceToDevice, c->st) !=
                hipSuccess ||
            hipStreamSynchronize(c->st) != hipSuccess) {
            FREE(nz);
            return hip_failed(c);
        }
        FREE(c->zhat);
        c->zhat = nz;
        if (c->labels) {
            int* nl = nullptr;
            ALLOC(nl, (size_t)ncap * sizeof(int));
            if (hipMemcpyAsync(nl, c->labels, (size_t)c->n_scored * sizeof(int), hipMemcpyDeviceToDevice, c->st) !=
                    hipSuccess ||
                hipStreamSynchronize(c->st) != hipSuccess) {
                FREE(nl);
                return hip_failed(c);
            }
            FREE(c->labels);
            c->labels = nl;
        }
        c->cap_rows = ncap;
    }
    if (labels) {
        if (!c->labels) ALLOC(c->labels, (size_t)c->cap_rows * sizeof(int));
        if (c->n_labeled == c->n_scored) c->n_labeled += rows;  // stays behind for good once an unlabeled batch came
    }
    while (rows > 0) {
        int64_t R = rows < SCORE_CHUNK ? rows : SCORE_CHUNK;
        int slots = 0;
        int rcp = project_rows(c, g, R, &slots);
        if (rcp != SAGE_OK) return rcp;
        RUN(K_FINALIZE, launch_score_finalize(c->proj_partial, R, c->KP, c->k, slots,
                                             c->store_zhat ? c->zhat + (size_t)c->n_scored * c->k : nullptr,
                                             c->cons_partial, c->ticket, c->ssum, c->store_zhat ? 0 : 1, c->n_scored == 0,
                                             nullptr, labels, labels ? c->labels + c->n_scored : nullptr, c->st));
        if (labels) labels += R;
        c->n_scored += R;
        g = g.after(R, c->d.D);
        rows -= R;
    }
    c->alpha_n = 0;
    return SAGE_OK;
}

// alpha capacity for N rows (and the selection work space that goes with it)
static int ensure_alpha(sage_ctx* c, int64_t N) {
    if (N <= c->alpha_cap) return SAGE_OK;
    float* na = nullptr;
    void* work = nullptr;
    int64_t ncap = N > c->cap_rows ? N : c->cap_rows;
    ALLOC(na, (size_t)ncap * sizeof(float));
    if (!late_alloc(c, &work, select_work_bytes(ncap))) {
        FREE(na);
        return NO_MEMORY(c);
    }
    if (c->alpha) {
        // keep what a running rescoring pass has written
        if (hipMemcpyAsync(na, c->alpha, (size_t)c->alpha_cap * sizeof(float), hipMemcpyDeviceToDevice, c->st) != hipSuccess ||
            hipStreamSynchronize(c->st) != hipSuccess) {
            FREE(na);
            FREE(work);
            return hip_failed(c);
        }
        FREE(c->alpha);
        FREE(c->sw.hist);
    }
    c->alpha = na;
    c->sw = select_work_at((uint32_t*)work, topm_work_blocks(ncap));
    c->alpha_cap = ncap;
    return SAGE_OK;
}

int sage_set_score_store(sage_ctx* c, int store_zhat) {
    ALIVE(c);
    c->store_zhat = store_zhat != 0;
    reset_scoring(c);
    return SAGE_OK;
}

static int rescore_impl(sage_ctx* c, RowSrc g, int64_t rows) {
    ALIVE(c);
    if (!c->has_basis || c->store_zhat) return SAGE_ERR_STATE;
    if (c->n_rescored + rows > c->n_scored) return SAGE_ERR_STATE;  // more rows than the first pass saw
    if (rows == 0) return SAGE_OK;
    int rc = ensure_alpha(c, c->n_scored);
    if (rc != SAGE_OK) return rc;
    while (rows > 0) {
        int64_t R = rows < SCORE_CHUNK ? rows : SCORE_CHUNK;
        int slots = 0;
        rc = project_rows(c, g, R, &slots);
        if (rc != SAGE_OK) return rc;
        RUN(K_FINALIZE, launch_score_finalize(c->proj_partial, R, c->KP, c->k, slots, nullptr, c->cons_partial, c->ticket,
                                             c->ssum, 2, false, c->alpha + c->n_rescored, nullptr, nullptr, c->st));
        c->n_rescored += R;
        g = g.after(R, c->d.D);
        rows -= R;
    }
    c->alpha_n = c->n_rescored == c->n_scored ? c->n_scored : 0;
    return SAGE_OK;
}

int sage_rescore(sage_ctx* c, const void* G_batch, int64_t rows) {
    ALIVE(c);
    if (rows < 0 || (rows > 0 && !G_batch)) return SAGE_ERR_ARG;
    return rescore_impl(c, dense_src(G_batch, c->dtype), rows);
}

int sage_rescore_outer(sage_ctx* c, const void* E, const void* H, int64_t rows, int64_t n_classes, int64_t n_features) {
    ALIVE(c);
    if (rows < 0) return SAGE_ERR_ARG;
    if (rows == 0) return rescore_impl(c, RowSrc{}, 0);
    RowSrc s;
    if (!outer_src(c, E, H, n_classes, n_features, s)) return SAGE_ERR_ARG;
    return rescore_impl(c, s, rows);
}

int sage_select(sage_ctx* c, double keep_rate, int64_t* out_idx, int64_t cap, int64_t* out_m) {
    ALIVE(c);
    if (!out_m || cap < 0 || !(keep_rate >= 0.0 && keep_rate <= 1.0)) return SAGE_ERR_ARG;
    if (!c->has_basis) return SAGE_ERR_STATE;
    const int64_t N = c->n_scored;
    const int64_t m = keep_count(keep_rate, N);
    *out_m = m;
    if (m > cap) return SAGE_ERR_CAPACITY;
    if (m > 0 && !out_idx) return SAGE_ERR_ARG;
    if (!c->store_zhat && c->n_rescored != N) return SAGE_ERR_STATE;  // the rescoring pass is not complete
    {
        int rc = ensure_alpha(c, N);
        if (rc != SAGE_OK) return rc;
    }
    if (c->store_zhat) RUN(K_SELECT, launch_cosine(c->zhat, N, c->k, c->ssum, c->alpha, c->st));
    c->alpha_n = N;
    const HostSignal done = next_signal(c);
    RUN(K_SELECT, launch_topm(c->alpha, N, m, out_idx, c->sw, false, c->st, done));
    HIPCHK(topm_signals(N, m) ? wait_signal(done, c->st) : hipStreamSynchronize(c->st));
    return SAGE_OK;
}

int sage_select_cb(sage_ctx* c, double keep_rate, int n_classes, int64_t* out_idx, int64_t cap, int64_t* out_m) {
    return sage_select_cb_ex(c, keep_rate, n_classes, SAGE_CB_PROPORTIONAL, out_idx, cap, out_m);
}

int sage_select_cb_ex(sage_ctx* c, double keep_rate, int n_classes, int rule, int64_t* out_idx, int64_t cap,
                      int64_t* out_m) {
    ALIVE(c);
    if (!out_m || cap < 0 || !(keep_rate >= 0.0 && keep_rate <= 1.0) || n_classes < 1 || n_classes > 65536 ||
        (rule != SAGE_CB_PROPORTIONAL && rule != SAGE_CB_EQUAL))
        return SAGE_ERR_ARG;
    if (!c->has_basis) return SAGE_ERR_STATE;
    const int64_t N = c->n_scored;
    if (!c->store_zhat || c->n_labeled != N) return SAGE_ERR_STATE;  // needs zhat, and a label for every row of the pass
    *out_m = 0;
    {
        int rc = ensure_alpha(c, N);
        if (rc != SAGE_OK) return rc;
    }
    const size_t need = cb_work_bytes(n_classes, N);
    if (need > c->cb_work_bytes) {
        if (c->cb_work) {
            HIPCHK(hipStreamSynchronize(c->st));
            FREE(c->cb_work);
            c->cb_work_bytes = 0;
        }
        ALLOC(c->cb_work, need);
        c->cb_work_bytes = need;
    }
    const CbWork w = cb_work_layout(c->cb_work, n_classes, N);
    uint32_t* report = (uint32_t*)c->kit.host + 1;
    RUN(K_SELECT, launch_cb_select(c->zhat, c->labels, N, c->k, n_classes, keep_rate, rule, c->alpha, cap, out_idx, report, w,
                                   c->st));
    c->alpha_n = N;
    HIPCHK(hipStreamSynchronize(c->st));
    if (((volatile uint32_t*)report)[1]) return SAGE_ERR_ARG;  // a label outside [0, n_classes)
    const int64_t m = (int64_t)((volatile uint32_t*)report)[0];
    *out_m = m;
    if (m > cap) return SAGE_ERR_CAPACITY;
    if (m > 0 && !out_idx) return SAGE_ERR_ARG;
    return SAGE_OK;
}

int sage_topm(const float* alpha, int64_t N, int64_t m, int64_t* out_idx, void* hip_stream) {
    if (N < 0 || m < 0 || m > N || (N > 0 && !alpha) || (m > 0 && !out_idx)) return SAGE_ERR_ARG;
    if (m == 0) return SAGE_OK;
    hipStream_t st = (hipStream_t)hip_stream;
    Allocator mem;
    {
        std::lock_guard<std::mutex> hold(g_mem_lock);
        mem = g_mem;
    }
    SelectWork w{};
    if (topm_needs_work(N)) {
        void* p = nullptr;
        if (!dev_alloc(mem, st, &p, select_work_bytes(N))) return SAGE_ERR_ALLOC;
        w = select_work_at((uint32_t*)p, topm_work_blocks(N));
    }
    HostSignal done;
    if (topm_signals(N, m)) (void)signal_take(done);
    hipError_t e = launch_topm(alpha, N, m, out_idx, w, false, st, done);
    hipError_t e2 = e == hipSuccess && done.word ? wait_signal(done, st) : hipStreamSynchronize(st);
    signal_give(done);
    dev_free(mem, w.hist);
    if (e == hipSuccess && e2 == hipSuccess) return SAGE_OK;
    (void)hipGetLastError();
    return SAGE_ERR_HIP;
}

int sage_fd_sketch_export(sage_ctx* c, float* B_out) {
    ALIVE(c);
    if (!B_out) return SAGE_ERR_ARG;
    int rcf = flush_pending(c);
    if (rcf != SAGE_OK) return rcf;
    const int ell = c->d.ell;
    if (int rc = clear_top(c); rc != SAGE_OK) return rc;
    if (c->fill_new > 0)
        if (int rc = widen(c, c->df.cur); rc != SAGE_OK) return rc;
    HIPCHK(launch_export_rows(c->top, c->d.LP, ell, B_out, c->d, c->st));
    HIPCHK(launch_export_rows(c->nw(c->df.cur), c->d.LP, c->fill_new, B_out + (size_t)ell * c->d.D, c->d, c->st));
    if (c->fill_new < ell)
        HIPCHK(hipMemsetAsync(B_out + (size_t)(ell + c->fill_new) * c->d.D, 0,
                              (size_t)(ell - c->fill_new) * c->d.D * sizeof(float), c->st));
    HIPCHK(hipStreamSynchronize(c->st));
    return SAGE_OK;
}

int sage_basis_export(sage_ctx* c, float* Vt_out) {
    ALIVE(c);
    if (!Vt_out) return SAGE_ERR_ARG;
    if (!c->has_basis) return SAGE_ERR_STATE;
    HIPCHK(launch_export_rows(c->Vblk, c->KP, c->k, Vt_out, c->d, c->st));
    HIPCHK(hipStreamSynchronize(c->st));
    return SAGE_OK;
}

int sage_scores(sage_ctx* c, const float** alpha, int64_t* n) {
    ALIVE(c);
    if (!alpha || !n) return SAGE_ERR_ARG;
    if (!c->has_basis || c->alpha_n != c->n_scored) return SAGE_ERR_STATE;
    *alpha = c->alpha;
    *n = c->alpha_n;
    return SAGE_OK;
}

int sage_scores_export(sage_ctx* c, float* alpha_out) {
    ALIVE(c);
    if ((!alpha_out && c->n_scored > 0)) return SAGE_ERR_ARG;
    if (!c->has_basis || c->alpha_n != c->n_scored) return SAGE_ERR_STATE;
    if (c->alpha_n > 0 && c->alpha_n <= COPY_SIGNAL_MAX) {
        const HostSignal done = next_signal(c);
        HIPCHK(launch_copy_signal(c->alpha, (int)c->alpha_n, alpha_out, done, c->st));
        HIPCHK(wait_signal(done, c->st));
        return SAGE_OK;
    }
    if (c->alpha_n > 0)
        HIPCHK(hipMemcpyAsync(alpha_out, c->alpha, (size_t)c->alpha_n * sizeof(float), hipMemcpyDeviceToDevice, c->st));
    HIPCHK(hipStreamSynchronize(c->st));
    return SAGE_OK;
}

int sage_zhat_export(sage_ctx* c, float* zhat_out) {
    ALIVE(c);
    if ((!zhat_out && c->n_scored > 0)) return SAGE_ERR_ARG;
    if (!c->has_basis || !c->store_zhat) return SAGE_ERR_STATE;
    if (c->n_scored > 0)
        HIPCHK(hipMemcpyAsync(zhat_out, c->zhat, (size_t)c->n_scored * c->k * sizeof(float), hipMemcpyDeviceToDevice,
                              c->st));
    HIPCHK(hipStreamSynchronize(c->st));
    return SAGE_OK;
}

int sage_stats(sage_ctx* c, sage_stats_t* out) {
    ALIVE(c);
    if (!out) return SAGE_ERR_ARG;
    int rcf = flush_pending(c);
    if (rcf != SAGE_OK) return rcf;
    double acc[8];
    HIPCHK(hipMemcpyAsync(acc, c->acc, sizeof(acc), hipMemcpyDeviceToHost, c->st));
    HIPCHK(hipStreamSynchronize(c->st));
    double pending = 0.0;
    if (c->cnt_top < c->fill_top || c->cnt_new < c->fill_new) {
        // rows inserted since the last decomposition: add their squared norms from a Gram of the buffer
        hipError_t e = hipSuccess;
        if (int rc = clear_top(c); rc != SAGE_OK) return rc;
        if (split_grams(c) && !c->new_block_ready && !c->pre_stored) {
            if (int rc = gram_whole_split(c); rc != SAGE_OK) return rc;
        } else {
            if (int rc = widen(c, c->df.cur); rc != SAGE_OK) return rc;
            e = launch_gram(c->top, c->nw(c->df.cur), c->fill_new, c->gram_partial, c->gp, c->d, c->st);
            if (e == hipSuccess)
                e = launch_gram_reduce(c->gram_partial, c->gp, nullptr, nullptr, c->ew.C, false, c->ew.known, c->d, c->st);
            if (e != hipSuccess) return hip_failed(c);
        }
        const int NP = c->d.NP, LP = c->d.LP;
        double* diag = (double*)malloc(sizeof(double) * NP);
        if (!diag) return SAGE_ERR_ALLOC;
        e = hipMemcpy2DAsync(diag, sizeof(double), c->ew.C, (size_t)(NP + 1) * sizeof(double), sizeof(double), NP,
                             hipMemcpyDeviceToHost, c->st);
        if (e == hipSuccess) e = hipStreamSynchronize(c->st);
        if (e != hipSuccess) {
            free(diag);
            return hip_failed(c);
        }
        for (int r = c->cnt_top; r < c->fill_top; ++r) pending += diag[r];
        for (int r = c->cnt_new; r < c->fill_new; ++r) pending += diag[LP + r];
        free(diag);
    }
    out->rows_seen = c->rows_seen;
    out->n_shrinks = c->n_shrinks;
    out->n_scored = c->n_scored;
    out->sum_delta = acc[0];
    out->frob2 = acc[1] + pending;
    out->last_delta = acc[2];
    out->last_sweeps = 0;  // the eigensolve is direct
    out->n_unconverged = (int64_t)acc[4];
    out->last_offdiag = 0.0;
    out->fill = c->fill_top + c->fill_new;
    return SAGE_OK;
}

int sage_probe_gram_eig(sage_ctx* c, double* C_out, int eig, double* Y_out, double* lam_out, int* n_pad) {
    ALIVE(c);
    const int NP = c->d.NP, LP = c->d.LP, ell = c->d.ell;
    if (n_pad) *n_pad = NP;
    if (!C_out && !eig) return SAGE_OK;
    int rcf = flush_pending(c);
    if (rcf != SAGE_OK) return rcf;
    if (int rc = clear_top(c); rc != SAGE_OK) return rc;
    if (int rc = widen(c, c->df.cur); rc != SAGE_OK) return rc;
    HIPCHK(launch_gram(c->top, c->nw(c->df.cur), c->fill_new, c->gram_partial, c->gp, c->d, c->st));
    HIPCHK(launch_gram_reduce(c->gram_partial, c->gp, nullptr, nullptr, c->ew.C, false, c->ew.known, c->d, c->st));
    // Inside the library matrix index LP + j stands for buffer row ell + j; the probe reports buffer-row order
    // (rows 0 .. 2*ell-1, padding last).
    if (C_out) HIPCHK(launch_probe_permute(c->ew.C, C_out, NP, LP, ell, true, c->st));
    if (eig) {
        HIPCHK(eigensolve(c, LP, NP, NP));
        HIPCHK(launch_eig_export(c->ew, NP, Y_out ? c->ew.V : nullptr, lam_out, nullptr, c->st));
        if (Y_out) HIPCHK(launch_probe_permute(c->ew.V, Y_out, NP, LP, ell, false, c->st));
    }
    HIPCHK(hipStreamSynchronize(c->st));
    return SAGE_OK;
}

int sage_probe_gram_split(sage_ctx* c, double* C_out, int* n_pad) {
    ALIVE(c);
    const int NP = c->d.NP, LP = c->d.LP, ell = c->d.ell;
    if (n_pad) *n_pad = NP;
    if (c->gp_cross_split.tiles <= 0 || c->gp_new2_split.tiles <= 0) return SAGE_ERR_STATE;
    if (!C_out) return SAGE_OK;
    int rcf = flush_pending(c);
    if (rcf != SAGE_OK) return rcf;
    if (c->new_block_ready || c->pre_stored) return SAGE_ERR_STATE;  // (never after flush_pending)
    if (int rc = clear_top(c); rc != SAGE_OK) return rc;
    const bool one = c->fill_new > 0 && new_one(c, c->df.cur);
    HIPCHK(launch_gram(c->top, c->nw(c->df.cur), c->fill_new, c->gram_partial, c->gp_cross_split, c->d, c->st, one));
    HIPCHK(launch_gram(c->top, c->nw(c->df.cur), c->fill_new, c->gram_partial_new[c->par], c->gp_new2_split, c->d, c->st, one));
    HIPCHK(launch_gram_reduce(c->gram_partial, c->gp_cross_split, c->gram_partial_new[c->par], &c->gp_new2_split, c->ew.C,
                              false, c->ew.known, c->d, c->st));
    HIPCHK(launch_probe_permute(c->ew.C, C_out, NP, LP, ell, true, c->st));
    HIPCHK(hipStreamSynchronize(c->st));
    return SAGE_OK;
}

int sage_probe_eig_matrix(sage_ctx* c, const double* C_in, double* Y_out, double* lam_out, double* sweep_stat_out) {
    ALIVE(c);
    if (!C_in) return SAGE_ERR_ARG;
    const int NP = c->d.NP;
    c->C_ready = false;  // (C_in takes its place: a shrink that is pending forms the products again)
    HIPCHK(hipMemcpyAsync(c->ew.C, C_in, (size_t)NP * NP * sizeof(double), hipMemcpyDeviceToDevice, c->st));
    HIPCHK(eigensolve(c, NP / 2, NP, NP));
    HIPCHK(launch_eig_export(c->ew, NP, Y_out, lam_out, sweep_stat_out, c->st));
    HIPCHK(hipStreamSynchronize(c->st));
    return SAGE_OK;
}

int sage_set_sweep_policy(sage_ctx* c, int policy) {
    ALIVE(c);
    if (policy != SAGE_SWEEPS_ADAPTIVE && policy != SAGE_SWEEPS_ALL) return SAGE_ERR_ARG;
    return SAGE_OK;  // the eigensolve is direct: there is nothing to choose
}

int sage_set_debug_checks(sage_ctx* c, int on) {
    ALIVE(c);
    c->debug_checks = on != 0;
    return SAGE_OK;
}

int sage_debug_fail_launch(sage_ctx* c, int nth) {
    ALIVE(c);
    if (nth < 0) return SAGE_ERR_ARG;
    c->fail_in = nth;
    return SAGE_OK;
}

int sage_debug_impatient_solves(sage_ctx* c, int on) {
    ALIVE(c);
    if (on < 0 || on > 3) return SAGE_ERR_ARG;
    c->ew.impatient = on == 1;
    if (c->xcd_slot >= 0) c->ew.xcd = on == 3 ? 8 : c->xcd_slot;
    c->ew.period = on == 2 || c->xcd_slot < 0 ? 0 : xcd_map().period;
    return SAGE_OK;
}

int sage_copy_probe(void* dst, const void* src, int64_t bytes, void* hip_stream) {
    if (!dst || !src || bytes < 0 || bytes % 16 != 0 || ((uintptr_t)dst | (uintptr_t)src) % 16 != 0) return SAGE_ERR_ARG;
    if (launch_plain_copy(src, dst, bytes, (hipStream_t)hip_stream) != hipSuccess) return SAGE_ERR_HIP;
    return SAGE_OK;
}

int sage_profile_enable(sage_ctx* c, int on) {
    ALIVE(c);
    c->prof = on != 0;
    return SAGE_OK;
}

int sage_profile_read(sage_ctx* c, int which, double* ms, int64_t* launches) {
    ALIVE(c);
    if (which < 0 || which >= NCLASS || !ms || !launches) return SAGE_ERR_ARG;
    HIPCHK(hipStreamSynchronize(c->st));
    *ms = c->prof_ms[which];
    *launches = c->prof_n[which];
    c->prof_ms[which] = 0.0;
    c->prof_n[which] = 0;
    return SAGE_OK;
}

}  // extern "C"
