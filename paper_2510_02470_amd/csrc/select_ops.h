// What the selection kernels share: keys, scans over a work-group, the digit of a radix select, compaction.
#pragma once
#include "sage_internal.h"

namespace sage {

// order-preserving key: larger alpha <-> larger key; -0 and +0 share a key
__device__ __forceinline__ uint32_t score_key(float a) {
    uint32_t b = __float_as_uint(a);
    if (b == 0x80000000u) b = 0u;
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// inclusive sum over the wave
__device__ __forceinline__ uint32_t wave_scan(uint32_t x) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true);  // row_shr 1, 2, 4, 8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);  // row_bcast 15 into rows 1 and 3
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);  // row_bcast 31 into rows 2 and 3
    return x;
}

// inclusive sum over the T threads of the work-group; tot: 16 words of LDS
template <int T>
__device__ __forceinline__ uint32_t block_scan(uint32_t x, uint32_t* tot) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    x = wave_scan(x);
    if (lane == 63) tot[wave] = x;
    __syncthreads();
    const uint32_t t = lane < T / 64 ? tot[lane] : 0u;
    const uint32_t before = wave_scan(t) - t;
    return x + (uint32_t)__builtin_amdgcn_readlane((int)before, __builtin_amdgcn_readfirstlane(wave));
}

struct PickWork {
    uint32_t tot[16];
    uint32_t digit, rest;
};
// The bin that holds the want-th largest key (want >= 1, at most the sum of the bins) and how many keys of that bin are
// among the want largest. Ends with a barrier.
template <int T, int BINS>
__device__ __forceinline__ void pick_bin(const uint32_t* hist, uint32_t want, PickWork& w, uint32_t& digit, uint32_t& rest) {
    constexpr int PER = BINS / T;
    const int top = BINS - 1 - (int)threadIdx.x * PER;  // thread t takes bins top, top - 1, ..
    uint32_t v[PER], sum = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        v[u] = hist[top - u];
        sum += v[u];
    }
    const uint32_t incl = block_scan<T>(sum, w.tot);
    uint32_t cum = incl - sum;
    if (cum < want && want <= incl) {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            if (cum < want && want <= cum + v[u]) {
                w.digit = (uint32_t)(top - u);
                w.rest = want - cum;
            }
            cum += v[u];
        }
    }
    __syncthreads();
    digit = w.digit;
    rest = w.rest;
}

__device__ __forceinline__ uint32_t lanes_below(unsigned long long mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Slice c of a work-group's keys: index base + c * T + thread. A key is kept when it is above thr, or equal to thr with
// fewer than `take` equal keys before it; its slot is (#greater before) + min(#equal before, take), so the output ascends.
// gt0, eq0: such keys before the work-group's first. Keys at and beyond N are 0 and come last, so they are never kept.
template <int T, int C>
__device__ __forceinline__ void emit_keys(const uint32_t (&key)[C], int64_t base, uint32_t thr, uint32_t take, uint32_t gt0,
                                          uint32_t eq0, uint32_t* cnt /* C T / 64 words */, uint32_t* tot,
                                          int64_t* __restrict__ out_idx) {
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    unsigned long long mg[C], me[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        mg[c] = __ballot(key[c] > thr);
        me[c] = __ballot(key[c] == thr);
        // (a work-group has at most 32768 keys: both counts fit 16 bits)
        if (lane == 0) cnt[c * (T / 64) + wave] = (uint32_t)__popcll(mg[c]) | ((uint32_t)__popcll(me[c]) << 16);
    }
    __syncthreads();
    static_assert(C * (T / 64) <= T, "one counter a thread");
    const uint32_t mine = tid < C * (T / 64) ? cnt[tid] : 0u;
    const uint32_t incl = block_scan<T>(mine, tot);
    if (tid < C * (T / 64)) cnt[tid] = incl - mine;
    __syncthreads();
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const uint32_t b = cnt[c * (T / 64) + wave];
        const uint32_t g = gt0 + (b & 0xFFFFu) + lanes_below(mg[c]), e = eq0 + (b >> 16) + lanes_below(me[c]);
        if (key[c] > thr || (key[c] == thr && e < take)) out_idx[g + (e < take ? e : take)] = base + c * T + tid;
    }
}

// Called by every thread at the end of a kernel of ONE work-group: its stores are made visible to the whole system, then the
// host's word is set.
__device__ __forceinline__ void signal_host(const HostSignal& done) {
    if (!done.word) return;
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence_system();
        __hip_atomic_store(done.word, done.token, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

}  // namespace sage
