// Class-balanced selection (Algorithm 1, "if class balance required"; "Agreement Scoring and Selection", CB-SAGE):
// per class c the unit centroid u_c of the normalised projections of its rows, alpha_i = <zhat_i, u_c(i)>, and the
// top k_c rows of every class. The k_c share out the budget m = floor(keep * N + 0.5) of the plain selection in
// proportion to the class sizes (largest-remainder rule, see cb_quota_kernel), so that sum_c k_c = m as Algorithm 1
// requires.
//
// Everything that decides the result is integer work, so the outcome does not depend on timing:
//   * class sums are accumulated in 64-bit fixed point (zhat * 2^40, |zhat| <= 1, up to 2^23 rows per class) with
//     integer atomics -- addition of integers is associative, unlike floating point;
//   * the k_c largest of a class are found by rank or radix select on order-preserving 32-bit keys, ties at the threshold
//     going to the lowest row indices;
//   * the selected rows are compacted in ascending row order (per-block counts, emit).
//
// The rows are listed by class first (count, scan, scatter; the order inside a class is arbitrary). Then a wave sums 32 rows
// of one class in registers before it touches memory (an atomic per row and coordinate was 66 us at 20,000 rows), and a
// work-group has a whole class to select from: one launch where a histogram and a pick per byte and for all classes at
// once were 17 (of 21 us each for the picks). Nine launches and one wait in all.
#include <type_traits>

#include "select_ops.h"

namespace sage {

constexpr double CB_SCALE = 1099511627776.0;  // 2^40
constexpr int CB_LDS_CLASSES = 4096;          // up to here a work-group counts its rows in LDS before it counts in memory

__global__ __launch_bounds__(256) void cb_zero_kernel(uint32_t* __restrict__ counts, long long* __restrict__ sums,
                                                      uint32_t* __restrict__ misc, int C) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < C) counts[i] = 0;
    if (i < (int64_t)C * 128) sums[i] = 0;
    if (i < 4) misc[i] = 0;  // [0] total kept, [1] a label was out of range
}

// rows per class
__global__ __launch_bounds__(1024) void cb_count_kernel(const int* __restrict__ labels, int64_t N, int C,
                                                        uint32_t* __restrict__ counts, uint32_t* __restrict__ misc) {
    __shared__ uint32_t h[CB_LDS_CLASSES];
    const bool lds = C <= CB_LDS_CLASSES;
    if (lds)
        for (int c = threadIdx.x; c < C; c += 1024) h[c] = 0;
    __syncthreads();
    for (int64_t i = (int64_t)blockIdx.x * 1024 + threadIdx.x; i < N; i += (int64_t)gridDim.x * 1024) {
        const int c = labels[i];
        if (c < 0 || c >= C) misc[1] = 1;
        else if (lds) atomicAdd(&h[c], 1u);
        else atomicAdd(&counts[c], 1u);
    }
    __syncthreads();
    if (lds)
        for (int c = threadIdx.x; c < C; c += 1024)
            if (const uint32_t v = h[c]) atomicAdd(&counts[c], v);
}

// The rows of every class, one class after the other (cursor[c]: first free place of class c). 4 rows a thread.
__global__ __launch_bounds__(1024) void cb_scatter_kernel(const int* __restrict__ labels, int64_t N, int C,
                                                          uint32_t* __restrict__ cursor, uint32_t* __restrict__ ord,
                                                          float* __restrict__ alpha) {
    __shared__ uint32_t h[CB_LDS_CLASSES];
    const bool lds = C <= CB_LDS_CLASSES;
    const int64_t i0 = (int64_t)blockIdx.x * 4096 + threadIdx.x;
    int c[4];
    uint32_t rank[4];
    if (lds)
        for (int j = threadIdx.x; j < C; j += 1024) h[j] = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int64_t i = i0 + u * 1024;
        c[u] = i < N ? labels[i] : -1;
        if (c[u] < 0 || c[u] >= C) {
            if (i < N) alpha[i] = 0.f;  // (the call reports the label)
            c[u] = -1;
        }
        rank[u] = c[u] < 0 ? 0u : (lds ? atomicAdd(&h[c[u]], 1u) : atomicAdd(&cursor[c[u]], 1u));
    }
    if (lds) {
        __syncthreads();
        for (int j = threadIdx.x; j < C; j += 1024)
            if (const uint32_t v = h[j]) h[j] = atomicAdd(&cursor[j], v);
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (c[u] >= 0) ord[(lds ? h[c[u]] : 0u) + rank[u]] = (uint32_t)(i0 + u * 1024);
}

constexpr int CB_RUN = 32;  // listed rows a wave goes through

// class sums, fixed point
__global__ __launch_bounds__(256) void cb_sum_kernel(const float* __restrict__ zhat, const int* __restrict__ labels,
                                                     const uint32_t* __restrict__ ord, int64_t N, int k, int C,
                                                     long long* __restrict__ sums, const uint32_t* __restrict__ misc) {
    if (misc[1]) return;  // (fewer than N rows are listed)
    const int lane = threadIdx.x & 63;
    const int64_t p0 = ((int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * CB_RUN;
    if (p0 >= N) return;
    const int64_t left = N - p0;
    const int cnt = left < CB_RUN ? (int)left : CB_RUN;
    const uint32_t myrow = lane < cnt ? ord[p0 + lane] : 0u;
    const int mycls = lane < cnt ? labels[myrow] : -1;
    long long s0 = 0, s1 = 0;
    for (int g = 0; g < cnt; g += 8) {
        float z0[8], z1[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float* z = zhat + (int64_t)(uint32_t)__builtin_amdgcn_readlane((int)myrow, g + u) * k;
            z0[u] = g + u < cnt && lane < k ? z[lane] : 0.f;
            z1[u] = g + u < cnt && lane + 64 < k ? z[lane + 64] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (g + u >= cnt) break;
            s0 += __double2ll_rn((double)z0[u] * CB_SCALE);
            s1 += __double2ll_rn((double)z1[u] * CB_SCALE);
            const int c = __builtin_amdgcn_readlane(mycls, g + u);
            const int next = g + u + 1 < cnt ? __builtin_amdgcn_readlane(mycls, (g + u + 1) & 63) : -1;
            if (c != next) {
                unsigned long long* s = reinterpret_cast<unsigned long long*>(sums + (int64_t)c * 128);
                if (lane < k) atomicAdd(&s[lane], (unsigned long long)s0);
                if (lane + 64 < k) atomicAdd(&s[lane + 64], (unsigned long long)s1);
                s0 = s1 = 0;
            }
        }
    }
}

// alpha_i = clamp(<zhat_i, u_c>, -1, 1), -0 stored as +0, u_c = S_c / ||S_c|| (0 if S_c = 0), and the keys in list order
__global__ __launch_bounds__(256) void cb_cosine_kernel(const float* __restrict__ zhat, const int* __restrict__ labels,
                                                        const uint32_t* __restrict__ ord, int64_t N, int k, int C,
                                                        const long long* __restrict__ sums,
                                                        const uint32_t* __restrict__ misc, float* __restrict__ alpha,
                                                        uint32_t* __restrict__ skey) {
    if (misc[1]) return;
    const int lane = threadIdx.x & 63;
    const int64_t p0 = ((int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * CB_RUN;
    if (p0 >= N) return;
    const int64_t left = N - p0;
    const int cnt = left < CB_RUN ? (int)left : CB_RUN;
    const uint32_t myrow = lane < cnt ? ord[p0 + lane] : 0u;
    const int mycls = lane < cnt ? labels[myrow] : -1;
    int cls = -1;
    double u0 = 0.0, u1 = 0.0;
    float mine = 0.f;
    for (int g = 0; g < cnt; g += 8) {
        float z0[8], z1[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float* z = zhat + (int64_t)(uint32_t)__builtin_amdgcn_readlane((int)myrow, g + u) * k;
            z0[u] = g + u < cnt && lane < k ? z[lane] : 0.f;
            z1[u] = g + u < cnt && lane + 64 < k ? z[lane + 64] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (g + u >= cnt) break;
            const int c = __builtin_amdgcn_readlane(mycls, g + u);
            if (c != cls) {
                cls = c;
                u0 = lane < k ? (double)sums[(int64_t)c * 128 + lane] / CB_SCALE : 0.0;
                u1 = lane + 64 < k ? (double)sums[(int64_t)c * 128 + lane + 64] / CB_SCALE : 0.0;
                double q2 = u0 * u0 + u1 * u1;
                for (int o = 32; o >= 1; o >>= 1) q2 += __shfl_xor(q2, o);
                const double nrm = sqrt(q2);
                u0 = nrm > 0.0 ? u0 / nrm : 0.0;
                u1 = nrm > 0.0 ? u1 / nrm : 0.0;
            }
            double a = (double)z0[u] * u0 + (double)z1[u] * u1;
            for (int o = 32; o >= 1; o >>= 1) a += __shfl_xor(a, o);
            if (a > 1.0) a = 1.0;
            if (a < -1.0) a = -1.0;
            float f = (float)a;
            if (f == 0.f) f = 0.f;
            if (lane == g + u) mine = f;
        }
    }
    if (lane < cnt) {
        alpha[myrow] = mine;
        skey[p0 + lane] = score_key(mine);
    }
}

// exclusive scan of the class counts into start and cursor, by the 1024 threads of a work-group (every thread owns a
// contiguous run of classes); red: 1024 words
__device__ __forceinline__ void cb_starts(const uint32_t* __restrict__ counts, int C, uint32_t* __restrict__ start,
                                          uint32_t* __restrict__ cursor, unsigned long long* red) {
    const int t = threadIdx.x, chunk = (C + 1023) / 1024;
    const int c0 = t * chunk, c1 = c0 + chunk < C ? c0 + chunk : C;
    uint32_t sum = 0;
    for (int c = c0; c < c1; ++c) sum += counts[c];
    __syncthreads();
    uint32_t at = block_scan<1024>(sum, (uint32_t*)red) - sum;
    for (int c = c0; c < c1; ++c) {
        start[c] = at;
        cursor[c] = at;
        at += counts[c];
    }
}

// The class budgets (Algorithm 1, class-balanced branch: sum_c k_c = k). With N_c rows in class c and N in all,
// m = floor(keep * N + 0.5) as in the plain selection, quota q_c = keep * N_c (fp64), k_c = floor(q_c), and the
// m - sum_c floor(q_c) rows still to hand out go one each to the classes with the largest fractional part
// q_c - floor(q_c) (equal parts: the lower class first) among those with k_c < N_c. All of it is exact integer or
// correctly rounded fp64 work, so the host-side definition gives the same numbers. One work-group of 1024 threads;
// also sets the places of the classes in the list and misc[0] = sum_c k_c.
__global__ __launch_bounds__(1024) void cb_quota_kernel(const uint32_t* __restrict__ counts, int C, double keep,
                                                        uint32_t* __restrict__ kc, uint32_t* __restrict__ start,
                                                        uint32_t* __restrict__ cursor, uint32_t* __restrict__ misc) {
#pragma clang fp contract(off)
    __shared__ unsigned long long red[1024];
    __shared__ uint32_t hist[1024];
    __shared__ PickWork pw;
    const int t = threadIdx.x;
    auto block_sum = [&](unsigned long long v) {
        for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
        if ((t & 63) == 0) red[t >> 6] = v;
        __syncthreads();
        unsigned long long r = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) r += red[w];
        __syncthreads();
        return r;
    };
    // The product keep * N_c must be rounded before floor() is subtracted from it. Contracted into a fused
    // multiply-add (the compiler's default, and __dmul_rn does not stop it) the difference comes from the unrounded
    // product: other bits than the host-side definition, even a negative "fraction" when keep * N_c rounds up to an
    // integer.
    auto quota = [&](uint32_t n) {
#pragma clang fp contract(off)
        return keep * (double)n;
    };
    auto frac_key = [&](uint32_t n) {  // order-preserving bits of the fractional part (a double in [0, 1))
#pragma clang fp contract(off)
        const double q = keep * (double)n;
        const double f = q - floor(q);
        return (unsigned long long)__double_as_longlong(f);
    };
    unsigned long long nsum = 0, bsum = 0, cand = 0;
    for (int c = t; c < C; c += 1024) {
        const uint32_t n = counts[c];
        const double f = floor(quota(n));
        const uint32_t b = f <= 0.0 ? 0u : (f >= (double)n ? n : (uint32_t)f);
        kc[c] = b;
        nsum += n;
        bsum += b;
        cand += b < n;
    }
    const unsigned long long N = block_sum(nsum), base = block_sum(bsum), ncand = block_sum(cand);
    double x;
    {
#pragma clang fp contract(off)
        const double kn = keep * (double)N;
        x = floor(kn + 0.5);
    }
    const unsigned long long m = x <= 0.0 ? 0ull : (x >= (double)N ? N : (unsigned long long)x);
    unsigned long long rem = m > base ? m - base : 0ull;
    if (rem > ncand) rem = ncand;
    if (rem > 0) {
        // Radix select of the rem-th largest key among the candidates, ten bits at a time from the top. It ends early when
        // a bin is taken whole (then T is its lower bound and no class on it is left out): seldom more than three rounds.
        unsigned long long T = 0;
        uint32_t take = (uint32_t)rem;
        for (int shift = 54, bits = 10;;) {
            const unsigned long long mask = (1ull << bits) - 1;
            hist[t] = 0;
            __syncthreads();
            for (int c = t; c < C; c += 1024) {
                if (kc[c] >= counts[c]) continue;
                const unsigned long long key = frac_key(counts[c]);
                if (shift == 54 || (key >> (shift + bits)) == (T >> (shift + bits))) atomicAdd(&hist[(key >> shift) & mask], 1u);
            }
            __syncthreads();
            uint32_t digit, rest;
            pick_bin<1024, 1024>(hist, take, pw, digit, rest);
            const uint32_t full = hist[digit];
            T |= (unsigned long long)digit << shift;
            take = rest;
            __syncthreads();
            if (shift == 0) break;
            if (rest == full) {
                take = 0xFFFFFFFFu;  // every class at or above T gets a row
                break;
            }
            bits = shift < 10 ? shift : 10;  // (64 bits: six digits of ten and one of four)
            shift -= bits;
        }
        const bool whole = take == 0xFFFFFFFFu;
        // otherwise `take` of the classes exactly on the threshold still get a row, lowest class first
        // ordered count of the threshold classes: every thread owns a contiguous run of classes
        const int chunk = (C + 1023) / 1024;
        const int c0 = t * chunk, c1 = c0 + chunk < C ? c0 + chunk : C;
        unsigned long long eq = 0;
        for (int c = c0; c < c1; ++c) eq += (kc[c] < counts[c] && frac_key(counts[c]) == T);
        red[t] = eq;
        __syncthreads();
        for (int o = 1; o < 1024; o <<= 1) {  // Hillis-Steele inclusive scan
            const unsigned long long a = t >= o ? red[t - o] : 0ull;
            __syncthreads();
            red[t] += a;
            __syncthreads();
        }
        unsigned long long before = red[t] - eq;
        __syncthreads();
        for (int c = c0; c < c1; ++c) {
            if (kc[c] >= counts[c]) continue;
            const unsigned long long key = frac_key(counts[c]);
            if (key > T || (whole && key == T)) kc[c] += 1;
            else if (key == T) {
                if (before < take) kc[c] += 1;
                before += 1;
            }
        }
        __syncthreads();
    }
    unsigned long long tot = 0;
    for (int c = t; c < C; c += 1024) {
        tot += kc[c];
    }
    tot = block_sum(tot);
    if (t == 0) misc[0] = (uint32_t)tot;
    cb_starts(counts, C, start, cursor, red);
}

// The other budget rule: equal budgets. The m = floor(keep * N + 0.5) rows are dealt one at a time to the classes in
// turn, lowest class first, a full class being passed over. In closed form: with q the largest level for which
// sum_c min(N_c, q) <= m, class c gets min(N_c, q), and the m - sum_c min(N_c, q) rows left (fewer than there are
// classes larger than q) go one each to the lowest-numbered classes with N_c > q. Integer work throughout. One
// work-group of 1024 threads; also sets the places of the classes in the list and misc[0] = sum_c k_c, like cb_quota_kernel.
__global__ __launch_bounds__(1024) void cb_quota_equal_kernel(const uint32_t* __restrict__ counts, int C, double keep,
                                                              uint32_t* __restrict__ kc, uint32_t* __restrict__ start,
                                                              uint32_t* __restrict__ cursor, uint32_t* __restrict__ misc) {
#pragma clang fp contract(off)
    __shared__ unsigned long long red[1024];
    const int t = threadIdx.x;
    auto block_sum = [&](unsigned long long v) {
        for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
        if ((t & 63) == 0) red[t >> 6] = v;
        __syncthreads();
        unsigned long long r = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) r += red[w];
        __syncthreads();
        return r;
    };
    auto block_max = [&](unsigned long long v) {
        for (int o = 32; o >= 1; o >>= 1) {
            const unsigned long long x = __shfl_xor(v, o);
            v = v > x ? v : x;
        }
        if ((t & 63) == 0) red[t >> 6] = v;
        __syncthreads();
        unsigned long long r = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) r = r > red[w] ? r : red[w];
        __syncthreads();
        return r;
    };
    unsigned long long nsum = 0, nmax = 0;
    for (int c = t; c < C; c += 1024) {
        const unsigned long long n = counts[c];
        nsum += n;
        nmax = n > nmax ? n : nmax;
    }
    const unsigned long long N = block_sum(nsum), top = block_max(nmax);
    double x;
    {
#pragma clang fp contract(off)
        const double kn = keep * (double)N;
        x = floor(kn + 0.5);
    }
    const unsigned long long m = x <= 0.0 ? 0ull : (x >= (double)N ? N : (unsigned long long)x);
    auto dealt = [&](unsigned long long q) {  // sum_c min(N_c, q)
        unsigned long long s = 0;
        for (int c = t; c < C; c += 1024) {
            const unsigned long long n = counts[c];
            s += n < q ? n : q;
        }
        return block_sum(s);
    };
    unsigned long long lo = 0, hi = top;  // dealt(lo) <= m always (dealt(0) = 0); the answer is in [lo, hi]
    while (lo < hi) {                     // (every thread sees the same sums, so the loop is uniform)
        const unsigned long long mid = lo + (hi - lo + 1) / 2;
        if (dealt(mid) <= m) lo = mid;
        else hi = mid - 1;
    }
    const unsigned long long q = lo;
    const unsigned long long spare = m - dealt(q);  // < number of classes with N_c > q
    // ordered count of the classes that can take a spare row: every thread owns a contiguous run of classes
    const int chunk = (C + 1023) / 1024;
    const int c0 = t * chunk, c1 = c0 + chunk < C ? c0 + chunk : C;
    unsigned long long open = 0;
    for (int c = c0; c < c1; ++c) open += counts[c] > q;
    red[t] = open;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {  // Hillis-Steele inclusive scan
        const unsigned long long a = t >= o ? red[t - o] : 0ull;
        __syncthreads();
        red[t] += a;
        __syncthreads();
    }
    unsigned long long before = red[t] - open;
    __syncthreads();
    unsigned long long tot = 0;
    for (int c = c0; c < c1; ++c) {
        const unsigned long long n = counts[c];
        unsigned long long b = n < q ? n : q;
        if (n > q) {
            if (before < spare) b += 1;
            before += 1;
        }
        kc[c] = (uint32_t)b;
        tot += b;
    }
    tot = block_sum(tot);
    if (t == 0) misc[0] = (uint32_t)tot;
    cb_starts(counts, C, start, cursor, red);
}

// One work-group of T threads per class: which of its rows are kept. Up to 256 rows: by rank, a thread comparing its key
// with all of them from LDS (the square of the rows in LDS reads: 10 us at 256, which the select needs too). More: radix select of the k_c-th largest key (12 + 10 + 10 bits) and, if not all rows on the
// threshold can be kept, of the row index among those (10 + 10 + 12 bits).
template <int T>
__global__ __launch_bounds__(T) void cb_select_kernel(const uint32_t* __restrict__ skey, const uint32_t* __restrict__ ord,
                                                      const uint32_t* __restrict__ counts,
                                                      const uint32_t* __restrict__ start, const uint32_t* __restrict__ kc,
                                                      const uint32_t* __restrict__ misc, uint8_t* __restrict__ sel) {
    __shared__ uint32_t h[4096];
    __shared__ PickWork pw;
    if (misc[1]) return;
    const int c = blockIdx.x, t = threadIdx.x;
    const uint32_t n = counts[c], k = kc[c];
    if (n == 0) return;
    const uint32_t* key = skey + start[c];
    const uint32_t* row = ord + start[c];
    if (k == 0 || k >= n) {
        for (uint32_t i = t; i < n; i += T) sel[row[i]] = k != 0;
        return;
    }
    if (n <= 256) {
        uint2* kr = reinterpret_cast<uint2*>(h);
        const uint2 mine = (uint32_t)t < n ? make_uint2(key[t], row[t]) : make_uint2(0u, 0xFFFFFFFFu);
        if (t < 256) kr[t] = mine;
        __syncthreads();
        if ((uint32_t)t >= n) return;
        uint32_t rank = 0;
#pragma unroll 4
        for (uint32_t j = 0; j < n; ++j) {
            const uint2 o = kr[j];
            rank += o.x > mine.x || (o.x == mine.x && o.y < mine.y);
        }
        sel[mine.y] = rank < k;
        return;
    }
    // digit of the want-th largest among those that `digit_of` accepts (it returns the bin, or -1)
    auto pick = [&](auto bins, uint32_t want, auto digit_of, uint32_t& digit, uint32_t& rest) {
        constexpr int B = decltype(bins)::value;
        for (int b = t; b < B; b += T) h[b] = 0;
        __syncthreads();
        for (uint32_t i = t; i < n; i += T) {
            const int d = digit_of(i);
            if (d >= 0) atomicAdd(&h[d], 1u);
        }
        __syncthreads();
        pick_bin<T, B>(h, want, pw, digit, rest);
        const uint32_t whole = h[digit];
        __syncthreads();
        return whole;
    };
    using B12 = std::integral_constant<int, 4096>;
    using B10 = std::integral_constant<int, 1024>;
    uint32_t d1, d2, d3, rest;
    pick(B12{}, k, [&](uint32_t i) { return (int)(key[i] >> 20); }, d1, rest);
    pick(B10{}, rest, [&](uint32_t i) { return (key[i] >> 20) == d1 ? (int)((key[i] >> 10) & 1023u) : -1; }, d2, rest);
    const uint32_t p2 = (d1 << 10) | d2;
    const uint32_t ties =
        pick(B10{}, rest, [&](uint32_t i) { return (key[i] >> 10) == p2 ? (int)(key[i] & 1023u) : -1; }, d3, rest);
    const uint32_t thr = (p2 << 10) | d3;
    uint32_t lowest = 0;  // threshold on ~row: the `rest` lowest rows on the key threshold are kept
    if (rest < ties) {
        uint32_t e1, e2, e3;
        pick(B10{}, rest, [&](uint32_t i) { return key[i] == thr ? (int)(~row[i] >> 22) : -1; }, e1, rest);
        pick(B10{}, rest,
             [&](uint32_t i) { return key[i] == thr && (~row[i] >> 22) == e1 ? (int)((~row[i] >> 12) & 1023u) : -1; }, e2,
             rest);
        const uint32_t q2 = (e1 << 10) | e2;
        pick(B12{}, rest, [&](uint32_t i) { return key[i] == thr && (~row[i] >> 12) == q2 ? (int)(~row[i] & 4095u) : -1; },
             e3, rest);
        lowest = (q2 << 12) | e3;
    }
    for (uint32_t i = t; i < n; i += T) sel[row[i]] = key[i] > thr || (key[i] == thr && ~row[i] >= lowest);
}

constexpr int CB_T = 1024, CB_C = SELECT_BLOCK / CB_T;

// rows kept per block of SELECT_BLOCK
__global__ __launch_bounds__(CB_T) void cb_kept_kernel(const uint8_t* __restrict__ sel, int64_t N,
                                                       const uint32_t* __restrict__ misc, uint32_t* __restrict__ blk) {
    __shared__ uint32_t s;
    if (misc[1]) return;
    if (threadIdx.x == 0) s = 0;
    __syncthreads();
    uint32_t g = 0;
#pragma unroll
    for (int c = 0; c < CB_C; ++c) {
        const int64_t i = (int64_t)blockIdx.x * SELECT_BLOCK + c * CB_T + threadIdx.x;
        g += (uint32_t)__popcll(__ballot(i < N && sel[i]));
    }
    if ((threadIdx.x & 63) == 0) atomicAdd(&s, g);
    __syncthreads();
    if (threadIdx.x == 0) blk[blockIdx.x] = s;
}

// The kept rows, ascending; every work-group adds up the counts of the blocks before its own. Writes nothing if there is
// not room for all of them. report (host memory): {rows kept, a label was out of range}.
__global__ __launch_bounds__(CB_T) void cb_emit_kernel(const uint8_t* __restrict__ sel, int64_t N,
                                                       const uint32_t* __restrict__ misc, const uint32_t* __restrict__ blk,
                                                       int64_t cap, int64_t* __restrict__ out_idx,
                                                       uint32_t* __restrict__ report) {
    __shared__ uint32_t cnt[CB_C * (CB_T / 64)], tot[16], before;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        report[0] = misc[0];
        report[1] = misc[1];
    }
    if (misc[1] || (int64_t)misc[0] > cap || !out_idx) return;
    uint32_t key[CB_C];
#pragma unroll
    for (int c = 0; c < CB_C; ++c) {
        const int64_t i = (int64_t)blockIdx.x * SELECT_BLOCK + c * CB_T + threadIdx.x;
        key[c] = i < N && sel[i];
    }
    if (threadIdx.x == 0) before = 0;
    uint32_t g = 0;
    for (unsigned b = threadIdx.x; b < blockIdx.x; b += CB_T) g += blk[b];
    g = wave_scan(g);
    __syncthreads();
    if ((threadIdx.x & 63) == 63 && g) atomicAdd(&before, g);
    __syncthreads();
    emit_keys<CB_T, CB_C>(key, (int64_t)blockIdx.x * SELECT_BLOCK, 0u, 0u, before, 0u, cnt, tot, out_idx);
}

// sets the pointers (base may be null: only the size is wanted) and returns the bytes needed
static size_t cb_work_fill(CbWork& w, char* base, int C, int64_t N) {
    size_t at = 0;
    auto take = [&](auto*& p, size_t count) {
        p = (std::remove_reference_t<decltype(p)>)(base + at);
        at += (count * sizeof(*p) + 255) / 256 * 256;
    };
    const size_t rows = N > 0 ? (size_t)N : 1;
    take(w.sums, (size_t)C * 128);
    take(w.counts, (size_t)C);
    take(w.kc, (size_t)C);
    take(w.start, (size_t)C);
    take(w.cursor, (size_t)C);
    take(w.misc, 64);
    take(w.blk, (rows + SELECT_BLOCK - 1) / SELECT_BLOCK);
    take(w.ord, rows);
    take(w.skey, rows);
    take(w.sel, rows);
    return at;
}

size_t cb_work_bytes(int C, int64_t N) {
    CbWork w{};
    return cb_work_fill(w, nullptr, C, N);
}

CbWork cb_work_layout(void* base, int C, int64_t N) {
    CbWork w{};
    cb_work_fill(w, (char*)base, C, N);
    return w;
}

hipError_t launch_cb_select(const float* zhat, const int* labels, int64_t N, int k, int C, double keep, int rule,
                            float* alpha, int64_t cap, int64_t* out_idx, uint32_t* report, const CbWork& w, hipStream_t st) {
    hipLaunchKernelGGL(cb_zero_kernel, dim3((unsigned)(((int64_t)C * 128 + 255) / 256)), dim3(256), 0, st, w.counts, w.sums,
                       w.misc, C);
    int64_t cb = (N + 4095) / 4096;
    const unsigned nblk = (unsigned)(cb > 0 ? cb : 1);
    if (cb > 512) cb = 512;
    if (N > 0) hipLaunchKernelGGL(cb_count_kernel, dim3((unsigned)cb), dim3(1024), 0, st, labels, N, C, w.counts, w.misc);
    if (rule == SAGE_CB_EQUAL)
        hipLaunchKernelGGL(cb_quota_equal_kernel, dim3(1), dim3(1024), 0, st, w.counts, C, keep, w.kc, w.start, w.cursor,
                           w.misc);
    else
        hipLaunchKernelGGL(cb_quota_kernel, dim3(1), dim3(1024), 0, st, w.counts, C, keep, w.kc, w.start, w.cursor, w.misc);
    if (N > 0) {
        hipLaunchKernelGGL(cb_scatter_kernel, dim3(nblk), dim3(1024), 0, st, labels, N, C, w.cursor, w.ord, alpha);
        const unsigned runs = (unsigned)((N + 4 * CB_RUN - 1) / (4 * CB_RUN));
        hipLaunchKernelGGL(cb_sum_kernel, dim3(runs), dim3(256), 0, st, zhat, labels, w.ord, N, k, C, w.sums, w.misc);
        hipLaunchKernelGGL(cb_cosine_kernel, dim3(runs), dim3(256), 0, st, zhat, labels, w.ord, N, k, C, w.sums, w.misc, alpha,
                           w.skey);
        // the radix select of a large class wants the wider work-group, the ranks of a small one no more than 256 threads
        if (N / C > 256)
            hipLaunchKernelGGL(cb_select_kernel<1024>, dim3(C), dim3(1024), 0, st, w.skey, w.ord, w.counts, w.start, w.kc,
                               w.misc, w.sel);
        else
            hipLaunchKernelGGL(cb_select_kernel<256>, dim3(C), dim3(256), 0, st, w.skey, w.ord, w.counts, w.start, w.kc,
                               w.misc, w.sel);
        hipLaunchKernelGGL(cb_kept_kernel, dim3(nblk), dim3(CB_T), 0, st, w.sel, N, w.misc, w.blk);
    }
    hipLaunchKernelGGL(cb_emit_kernel, dim3(nblk), dim3(CB_T), 0, st, w.sel, N, w.misc, w.blk, cap, out_idx, report);
    return hipGetLastError();
}

}  // namespace sage
