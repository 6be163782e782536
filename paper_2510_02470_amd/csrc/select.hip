// Scoring pass, second half (Algorithm 1, Phase II: "u <- zbar/||zbar||", "alpha_i <- <zhat_i, u>",
// "Select top-k by alpha_i"): consensus direction, cosine scores, radix-select of the m-th largest score and a
// stable compaction of the selected indices in ascending order.
#include "score_ops.h"
#include "select_ops.h"

namespace sage {

// alpha_i = clamp(<zhat_i, u>, -1, 1), -0 stored as +0, with u = ssum / ||ssum|| made by every wave. A wave takes a row per
// group of L = KP / 4 lanes, four times over.
template <int L>
__global__ __launch_bounds__(256) void cosine_kernel(const float* __restrict__ zhat, int64_t N, int k,
                                                     const double* __restrict__ ssum, float* __restrict__ alpha) {
    constexpr int G = 64 / L, U = 4;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane / L, c0 = (lane % L) * 4;
    const int64_t r0 = ((int64_t)blockIdx.x * 4 + wave) * (U * G) + g;
    double z[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int c = 0; c < 4; ++c)
            z[u][c] = r0 + u * G < N && c0 + c < k ? (double)zhat[(r0 + u * G) * k + c0 + c] : 0.0;
    double cu[4];
    consensus_unit<L>(ssum, k, c0, cu);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const float f = clamp_score(row_dot<L>(z[u], cu));
        if (r0 + u * G < N && lane % L == 0) alpha[r0 + u * G] = f;
    }
}

hipError_t launch_cosine(const float* zhat, int64_t N, int k, const double* ssum, float* alpha, hipStream_t st) {
    if (N <= 0) return hipSuccess;
    const int L = k <= 32 ? 8 : (k <= 64 ? 16 : 32);
    const unsigned blocks = (unsigned)((N * L + 1023) / 1024);
    switch (L) {
        case 8: hipLaunchKernelGGL(cosine_kernel<8>, dim3(blocks), dim3(256), 0, st, zhat, N, k, ssum, alpha); break;
        case 16: hipLaunchKernelGGL(cosine_kernel<16>, dim3(blocks), dim3(256), 0, st, zhat, N, k, ssum, alpha); break;
        default: hipLaunchKernelGGL(cosine_kernel<32>, dim3(blocks), dim3(256), 0, st, zhat, N, k, ssum, alpha); break;
    }
    return hipGetLastError();
}

// ---- top-m ----------------------------------------------------------------------------------------------------------
// Radix select of the m-th largest key, 12 + 10 + 10 bits from the top, then compaction in ascending index. All the data
// there is to move is 4 N bytes, so what counts is the number of launches (about 3 us each with its gap) and serial work
// inside them:
//   N <= TOPM_ONE: one work-group does everything, keys in registers, histograms in LDS; one launch, no work space;
//   else: two histograms, the third with a table for each block of keys, emit. Every work-group of the next kernel
//         reads the histogram and finds the digit itself (a scan over the bins by 1024 threads), so there are no kernels
//         between them. Each run clears a histogram after its last reader, so that work space that is kept is clear for the
//         next run, which may then do without the launch for that (eager calls of sage_topm_static: a million keys 18.1 us, 20.0
//         with it). All other calls begin with it. The tables answer, whatever the last digit turns out to be, how many keys of a block are above it and
//         how many equal it, which took a kernel of its own between the last histogram and emit (a million keys: 24.2 us
//         with it, 22.4 without, 19.9 with fewer work-groups for the histograms, see launch_topm).
// The first digit has 12 bits because scores crowd into a few binary orders of magnitude: with 8 bits most lanes of a wave
// add to one of two or three LDS words and the adds are done one after the other.
// (One digit of 8 bits per launch with a one-thread pick kernel after each took 13 launches: 86 us at N = 2048 and 80 us at
// a million, host and waiting included.)
constexpr int BINS1 = 4096, BINS2 = 1024;
constexpr int TOPM_T = 1024;  // threads of every kernel below

// one work-group, N <= 1024 C
template <int C>
__global__ __launch_bounds__(TOPM_T) void topm_one_kernel(const float* __restrict__ alpha, int N, uint32_t m,
                                                          int64_t* __restrict__ out_idx, HostSignal done) {
    static_assert(C <= 32, "emit_keys packs counts of 16 bits");
    __shared__ uint32_t h[BINS1 + 2 * BINS2];
    __shared__ uint32_t cnt[16 * C], tot[16];
    __shared__ PickWork pw;
    const int tid = threadIdx.x;
    uint32_t key[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int i = c * TOPM_T + tid;
        key[c] = i < N ? score_key(alpha[i]) : 0u;
    }
    for (int b = tid; b < BINS1 + 2 * BINS2; b += TOPM_T) h[b] = 0;
    __syncthreads();
#pragma unroll
    for (int c = 0; c < C; ++c)
        if (c * TOPM_T + tid < N) atomicAdd(&h[key[c] >> 20], 1u);
    __syncthreads();
    uint32_t d1, d2, d3, rest;
    pick_bin<TOPM_T, BINS1>(h, m, pw, d1, rest);
#pragma unroll
    for (int c = 0; c < C; ++c)
        if (c * TOPM_T + tid < N && (key[c] >> 20) == d1) atomicAdd(&h[BINS1 + ((key[c] >> 10) & 1023u)], 1u);
    __syncthreads();
    pick_bin<TOPM_T, BINS2>(h + BINS1, rest, pw, d2, rest);
    const uint32_t p2 = (d1 << 10) | d2;
#pragma unroll
    for (int c = 0; c < C; ++c)
        if (c * TOPM_T + tid < N && (key[c] >> 10) == p2) atomicAdd(&h[BINS1 + BINS2 + (key[c] & 1023u)], 1u);
    __syncthreads();
    pick_bin<TOPM_T, BINS2>(h + BINS1 + BINS2, rest, pw, d3, rest);
    emit_keys<TOPM_T, C>(key, 0, (p2 << 10) | d3, rest, 0u, 0u, cnt, tot, out_idx);
    signal_host(done);
}

// hist: BINS1 + 2 BINS2 words. (The third part needs no clearing here, but new work space is all the same to this launch.)
__global__ __launch_bounds__(TOPM_T) void topm_clear_kernel(uint32_t* __restrict__ hist) {
    hist[blockIdx.x * TOPM_T + threadIdx.x] = 0;
}

// Histogram of digit P (0: bits 31..20, 1: bits 19..10) of the keys that share the digits found so far. state[0], state[1]: the
// first digit and the count left, found from the first histogram, left for the next kernel. P = 0 also clears the third histogram.
template <int P>
__global__ __launch_bounds__(TOPM_T) void topm_hist_kernel(const float* __restrict__ alpha, int64_t N, uint32_t m,
                                                           uint32_t* __restrict__ hist, uint32_t* __restrict__ state) {
    constexpr int BINS = P == 0 ? BINS1 : BINS2;
    __shared__ uint32_t h[BINS];
    __shared__ PickWork pw;
    const int tid = threadIdx.x;
    for (int b = tid; b < BINS; b += TOPM_T) h[b] = 0;
    uint32_t prefix = 0;
    if constexpr (P > 0) {
        uint32_t rest;
        pick_bin<TOPM_T, BINS1>(hist, m, pw, prefix, rest);
        if (blockIdx.x == 0 && tid == 0) {
            state[0] = prefix;
            state[1] = rest;
        }
    } else {
        if (blockIdx.x == 0) hist[BINS1 + BINS2 + tid] = 0;
        __syncthreads();
    }
    const int64_t stride = (int64_t)gridDim.x * TOPM_T;
    for (int64_t i0 = (int64_t)blockIdx.x * TOPM_T + tid; i0 < N; i0 += 4 * stride) {
        float a[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] = i0 + u * stride < N ? alpha[i0 + u * stride] : 0.f;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t key = score_key(a[u]);
            if (i0 + u * stride >= N) continue;
            if (P == 0) atomicAdd(&h[key >> 20], 1u);
            if (P == 1 && (key >> 20) == prefix) atomicAdd(&h[(key >> 10) & 1023u], 1u);
        }
    }
    __syncthreads();
    uint32_t* g = hist + (P == 0 ? 0 : BINS1);
    for (int b = tid; b < BINS; b += TOPM_T)
        if (const uint32_t v = h[b]) atomicAdd(&g[b], v);
}

// Histogram of the last digit (bits 9..0), and for each block of 1024 C keys: blk_gt, how many are above all that share
// the first 22 bits, blk_in, how many share them, and if any do, table[d], how many of those have a last digit of d or more. Clears
// the first histogram, which has been read.
template <int C>
__global__ __launch_bounds__(TOPM_T) void topm_table_kernel(const float* __restrict__ alpha, int64_t N,
                                                            uint32_t* __restrict__ hist, uint32_t* __restrict__ state,
                                                            uint32_t* __restrict__ blk_gt, uint32_t* __restrict__ blk_in,
                                                            uint16_t* __restrict__ table) {
    static_assert(BINS2 == TOPM_T && C * TOPM_T < 65536, "a bin a thread, counts of 16 bits");
    __shared__ uint32_t h[BINS2], tot[16], sg, si;
    __shared__ PickWork pw;
    const int tid = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * (C * TOPM_T) + tid;
    uint32_t key[C];
#pragma unroll
    for (int c = 0; c < C; ++c) key[c] = base + c * TOPM_T < N ? score_key(alpha[base + c * TOPM_T]) : 0u;
    h[tid] = 0;
    if (tid == 0) sg = si = 0;
    if (blockIdx.x < BINS1 / TOPM_T) hist[blockIdx.x * TOPM_T + tid] = 0;
    uint32_t digit, rest;
    pick_bin<TOPM_T, BINS2>(hist + BINS1, state[1], pw, digit, rest);
    const uint32_t prefix = (state[0] << 10) | digit;
    if (blockIdx.x == 0 && tid == 0) {
        state[2] = prefix;
        state[3] = rest;
    }
    uint32_t g = 0, i = 0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const bool in = base + c * TOPM_T < N, eq = in && (key[c] >> 10) == prefix;
        g += (uint32_t)__popcll(__ballot(in && (key[c] >> 10) > prefix));
        i += (uint32_t)__popcll(__ballot(eq));
        if (eq) atomicAdd(&h[key[c] & 1023u], 1u);
    }
    if ((tid & 63) == 0) {
        if (g) atomicAdd(&sg, g);
        if (i) atomicAdd(&si, i);
    }
    __syncthreads();
    if (tid == 0) {
        blk_gt[blockIdx.x] = sg;
        blk_in[blockIdx.x] = si;
    }
    if (si == 0) return;
    const int d = BINS2 - 1 - tid;
    const uint32_t v = h[d];
    if (v) atomicAdd(&hist[BINS1 + BINS2 + d], v);
    table[(int64_t)blockIdx.x * BINS2 + d] = (uint16_t)block_scan<TOPM_T>(v, tot);
}

// every work-group adds up the counts of the blocks before its own; the second histogram, which has been read, is cleared
template <int C>
__global__ __launch_bounds__(TOPM_T) void topm_emit_kernel(const float* __restrict__ alpha, int64_t N,
                                                           uint32_t* __restrict__ hist, const uint32_t* __restrict__ state,
                                                           const uint32_t* __restrict__ blk_gt,
                                                           const uint32_t* __restrict__ blk_in,
                                                           const uint16_t* __restrict__ table, int64_t* __restrict__ out_idx) {
    __shared__ uint32_t cnt[16 * C], tot[16], sg, se;
    __shared__ PickWork pw;
    const int64_t base = (int64_t)blockIdx.x * (C * TOPM_T);
    uint32_t key[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int64_t i = base + c * TOPM_T + threadIdx.x;
        key[c] = i < N ? score_key(alpha[i]) : 0u;
    }
    if (threadIdx.x == 0) sg = se = 0;
    if (blockIdx.x == 0) hist[BINS1 + threadIdx.x] = 0;
    uint32_t digit, rest;
    pick_bin<TOPM_T, BINS2>(hist + BINS1 + BINS2, state[3], pw, digit, rest);
    uint32_t g = 0, e = 0;
    for (unsigned b = threadIdx.x; b < blockIdx.x; b += TOPM_T) {
        g += blk_gt[b];
        if (blk_in[b]) {
            const uint16_t* t = table + (int64_t)b * BINS2 + digit;
            const uint32_t above = digit + 1 < BINS2 ? t[1] : 0u;
            g += above;
            e += t[0] - above;
        }
    }
    g = wave_scan(g);
    e = wave_scan(e);
    if ((threadIdx.x & 63) == 63 && (g | e)) {
        atomicAdd(&sg, g);
        atomicAdd(&se, e);
    }
    __syncthreads();
    emit_keys<TOPM_T, C>(key, base, (state[2] << 10) | digit, rest, sg, se, cnt, tot, out_idx);
}

// One work-group up to 32 keys a thread, as many as fit its registers; beyond, the width of four or five launches wins.
constexpr int64_t TOPM_ONE = 32 * TOPM_T;

// Small copies for a caller that waits: one work-group, then the signal.
__global__ __launch_bounds__(TOPM_T) void copy_signal_kernel(const float* __restrict__ src, int n, float* __restrict__ dst,
                                                             HostSignal done) {
    for (int i = threadIdx.x; i < n; i += TOPM_T) dst[i] = src[i];
    signal_host(done);
}
hipError_t launch_copy_signal(const float* src, int n, float* dst, HostSignal done, hipStream_t st) {
    hipLaunchKernelGGL(copy_signal_kernel, dim3(1), dim3(TOPM_T), 0, st, src, n, dst, done);
    return hipGetLastError();
}

bool topm_needs_work(int64_t N) { return N > TOPM_ONE; }

bool topm_signals(int64_t N, int64_t m) { return m > 0 && N > 0 && N <= TOPM_ONE; }

hipError_t launch_topm(const float* alpha, int64_t N, int64_t m, int64_t* out_idx, const SelectWork& w, bool clear,
                       hipStream_t st, HostSignal done) {
    if (m <= 0 || N <= 0) return hipSuccess;
    if (N <= TOPM_ONE) {
#define SAGE_ONE(C) \
    hipLaunchKernelGGL(topm_one_kernel<C>, dim3(1), dim3(TOPM_T), 0, st, alpha, (int)N, (uint32_t)m, out_idx, done)
        if (N <= 2 * TOPM_T) SAGE_ONE(2);
        else if (N <= 4 * TOPM_T) SAGE_ONE(4);
        else if (N <= 8 * TOPM_T) SAGE_ONE(8);
        else if (N <= 16 * TOPM_T) SAGE_ONE(16);
        else SAGE_ONE(32);
#undef SAGE_ONE
        return hipGetLastError();
    }
    const int64_t nblk = topm_blocks(N);
    if (nblk > w.nblk_cap) return hipErrorInvalidValue;
    // Work-groups of the histograms: 16,384 keys each, 64 at least while there are as many blocks (their adds to the same few words
    // of memory are done one after the other: a million keys 22.4 us with 244 work-groups, 19.9 with 64; 4 million, waiting
    // included, 56.0 with 512, 49.8 with 244).
    const int64_t blocks = (N + SELECT_BLOCK - 1) / SELECT_BLOCK, wide = blocks / 4;
    const int64_t hw = wide < 64 ? (blocks < 64 ? blocks : 64) : wide < 512 ? wide : 512;
    static_assert(BINS2 == TOPM_T && BINS1 / TOPM_T <= TOPM_ONE / SELECT_BLOCK, "a bin a thread; as many blocks as clear bins");
    if (!clear) hipLaunchKernelGGL(topm_clear_kernel, dim3(TOPM_HIST_WORDS / TOPM_T), dim3(TOPM_T), 0, st, w.hist);
    hipLaunchKernelGGL(topm_hist_kernel<0>, dim3((unsigned)hw), dim3(TOPM_T), 0, st, alpha, N, (uint32_t)m, w.hist, w.state);
    hipLaunchKernelGGL(topm_hist_kernel<1>, dim3((unsigned)hw), dim3(TOPM_T), 0, st, alpha, N, (uint32_t)m, w.hist, w.state);
#define SAGE_TAIL(C)                                                                                                          \
    do {                                                                                                                      \
        hipLaunchKernelGGL(topm_table_kernel<C>, dim3((unsigned)nblk), dim3(TOPM_T), 0, st, alpha, N, w.hist, w.state,         \
                           w.blk_gt, w.blk_in, w.table);                                                                      \
        hipLaunchKernelGGL(topm_emit_kernel<C>, dim3((unsigned)nblk), dim3(TOPM_T), 0, st, alpha, N, w.hist, w.state,          \
                           w.blk_gt, w.blk_in, w.table, out_idx);                                                             \
    } while (0)
    if (topm_long(N)) SAGE_TAIL(SELECT_LONG / TOPM_T);
    else SAGE_TAIL(SELECT_BLOCK / TOPM_T);
#undef SAGE_TAIL
    return hipGetLastError();
}

}  // namespace sage
