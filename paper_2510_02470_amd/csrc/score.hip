// Scoring pass, first half (Algorithm 1, Phase II, first line; Method, "Two-pass scoring"):
//   z_i = V_k^T g_i  (fp32 matrix cores, split over D),  zhat_i = z_i / ||z_i||_2 (0 if z_i = 0),
//   consensus sum  s += sum_i zhat_i  (fixed-order reductions, fp64).
#include "score_ops.h"

namespace sage {

// load one 16-byte-wide piece (4 columns) of a batch row, widened to fp32; columns >= D read as 0
template <typename T, bool VEC>
__device__ __forceinline__ f32x4 load_piece(const T* __restrict__ row, int64_t d0, int64_t D) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if constexpr (VEC) {
        if (d0 < D) {  // D % 4 == 0 on this path
            if constexpr (sizeof(T) == 4) {
                v = *reinterpret_cast<const f32x4*>(row + d0);
            } else {
                uint2 u = *reinterpret_cast<const uint2*>(row + d0);
                v[0] = __uint_as_float(u.x << 16);
                v[1] = __uint_as_float(u.x & 0xffff0000u);
                v[2] = __uint_as_float(u.y << 16);
                v[3] = __uint_as_float(u.y & 0xffff0000u);
            }
        }
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float x = 0.f;
            if (d0 + c < D) {
                if constexpr (sizeof(T) == 4) x = row[d0 + c];
                else x = bf16_to_f32(row[d0 + c]);
            }
            v[c] = x;
        }
    }
    return v;
}

// Work-group tile: 128 batch rows x KP basis columns, a wave owns 32 rows. Split-K over D: block id ->
// (row tile, split) with the row tiles of one split adjacent on one XCD so that they share the basis slabs in L2.
// partial[split][row][KP] receives the fp32 partial projections.
template <int NT, typename T, bool VEC>  // NT = KP / 32
__global__ __launch_bounds__(256) void project_kernel(const T* __restrict__ G, int64_t R, const float* __restrict__ Vblk,
                                                      float* __restrict__ partial, int row_tiles, int64_t D,
                                                      int64_t slabs_total, int64_t slabs_per_split) {
    constexpr int KP = NT * 32;
    constexpr int GP = 128 * 4;       // batch pieces per stage
    constexpr int VP = KP * 4;        // basis pieces per stage
    constexpr int STAGE = GP + VP;
    constexpr int VPER = (VP + 255) / 256;
    __shared__ f32x4 lds[2 * STAGE];

    const int id = blockIdx.x;
    const int xcd = id & 7, y = id >> 3;
    const int rt = y % row_tiles;
    const int split = (y / row_tiles) * 8 + xcd;
    int64_t s0 = (int64_t)split * slabs_per_split;
    int64_t s1 = s0 + slabs_per_split;
    if (s1 > slabs_total) s1 = slabs_total;

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int l32 = lane & 31, h = lane >> 5;
    const int64_t row_base = (int64_t)rt * 128;

    f32x16 acc[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[n][i] = 0.f;

    // staging slots: batch piece slot ps -> (row ps/4, logical piece (ps%4)^((row/4)%4)); same for the basis
    int grow[2], gp[2];
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        int ps = it * 256 + tid;
        grow[it] = ps >> 2;
        gp[it] = (ps & 3) ^ ((grow[it] >> 2) & 3);
    }
    int vsrc[VPER];
#pragma unroll
    for (int it = 0; it < VPER; ++it) {
        int ps = it * 256 + tid;
        int row = ps >> 2;
        vsrc[it] = row * 4 + ((ps & 3) ^ ((row >> 2) & 3));
    }
    const f32x4* Vv = reinterpret_cast<const f32x4*>(Vblk);
    f32x4 gpre[2], vpre[VPER];

    auto fetch = [&](int64_t s) {
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            int64_t r = row_base + grow[it];
            gpre[it] = (r < R) ? load_piece<T, VEC>(G + r * D, s * DC + gp[it] * 4, D) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int it = 0; it < VPER; ++it)
            if (it * 256 + tid < VP) vpre[it] = Vv[s * VP + vsrc[it]];
    };
    auto stash = [&](int buf) {
        f32x4* dst = lds + buf * STAGE;
#pragma unroll
        for (int it = 0; it < 2; ++it) dst[it * 256 + tid] = gpre[it];
#pragma unroll
        for (int it = 0; it < VPER; ++it)
            if (it * 256 + tid < VP) dst[GP + it * 256 + tid] = vpre[it];
    };

    if (s0 < s1) {
        fetch(s0);
        stash(0);
    }
    __syncthreads();
    for (int64_t s = s0; s < s1; ++s) {
        const int cur = (int)((s - s0) & 1);
        const bool more = s + 1 < s1;
        if (more) fetch(s + 1);
        const f32x4* gs = lds + cur * STAGE;
        const f32x4* vs = gs + GP;
        f32x4 a[2];
        {
            int r = wave * 32 + l32;
#pragma unroll
            for (int j = 0; j < 2; ++j) a[j] = gs[r * 4 + ((2 * j + h) ^ ((r >> 2) & 3))];
        }
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            int r = n * 32 + l32;
            f32x4 b[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) b[j] = vs[r * 4 + ((2 * j + h) ^ ((r >> 2) & 3))];
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    acc[n] = mfma32(a[j][c], b[j][c], acc[n]);
        }
        if (more) stash(cur ^ 1);
        __syncthreads();
    }

    float* out = partial + (int64_t)split * R * KP;
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            int64_t r = row_base + wave * 32 + 8 * (i >> 2) + 4 * h + (i & 3);
            if (r < R) out[r * KP + n * 32 + l32] = acc[n][i];
        }
}

// Sum of the split-K partial projections, normalisation, consensus sum. A wave works on a row (WPR = 1) or a quarter of its
// splits (WPR = 4, many splits): KP / 4 lanes hold four coordinates each, the 64 / (KP / 4) groups of such lanes take the
// splits in turn. fp64 in a fixed order throughout: the result does not depend on timing.
// mode 0: zhat (R x k, fp32) and the consensus sum. mode 1: the consensus sum only (first scoring pass of a run that does not
// store zhat). mode 2: the second such pass: alpha_i = clamp(<zhat_i, u>, -1, 1) straight from the recomputed zhat_i, by the
// functions cosine_kernel uses, so that the scores are bit-equal to those of the run that stores zhat.
// The consensus sums of the work-groups go to memory past the L2 (device scope), and the work-group that comes last adds
// them up, in their order, to ssum: a kernel of its own for that was 5 to 10 us more. src_labels (may be null): the labels of
// the rows, kept in dst_labels.
template <int KP, int WPR>
__global__ __launch_bounds__(1024) void score_finalize_kernel(const float* __restrict__ partial, int64_t R, int k, int splits,
                                                              float* __restrict__ zhat, double* __restrict__ cons_partial,
                                                              unsigned* __restrict__ ticket, int mode, int first,
                                                              double* __restrict__ ssum, float* __restrict__ alpha,
                                                              const int* __restrict__ src_labels,
                                                              int* __restrict__ dst_labels) {
    constexpr int L = KP / 4, G = 64 / L, ROWS = 16 / WPR;
    __shared__ double red[WPR == 4 ? 16 : 1][KP];
    __shared__ double cs[ROWS][KP];
    __shared__ double part[8][128];
    __shared__ bool is_last;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int rr = wave / WPR, quarter = wave % WPR, g = lane / L, c0 = (lane % L) * 4;
    const int64_t r = (int64_t)blockIdx.x * ROWS + rr;
    double z[4] = {0.0, 0.0, 0.0, 0.0};
    if (r < R) {
        const int per = (splits + WPR - 1) / WPR;
        const int sa = quarter * per, sb = sa + per < splits ? sa + per : splits;
        const float4* p = reinterpret_cast<const float4*>(partial + r * KP + c0);
        const int64_t stride = R * KP / 4;
        constexpr int U = 16;
        for (int s0 = sa; s0 < sb; s0 += U * G) {
            float4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int ss = s0 + u * G + g;
                v[u] = p[(ss < sb ? ss : sb - 1) * stride];  // repeats are not added
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (s0 + u * G + g < sb) {
                    z[0] += (double)v[u].x;
                    z[1] += (double)v[u].y;
                    z[2] += (double)v[u].z;
                    z[3] += (double)v[u].w;
                }
        }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) z[c] = group_sum<L>(z[c]);
    if constexpr (WPR == 4) {
        if (g == 0) {
#pragma unroll
            for (int c = 0; c < 4; ++c) red[wave][c0 + c] = z[c];
        }
        __syncthreads();
        if (quarter == 0) {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                z[c] = ((red[wave][c0 + c] + red[wave + 1][c0 + c]) + red[wave + 2][c0 + c]) + red[wave + 3][c0 + c];
        }
    }
    if (quarter == 0) {
#pragma unroll
        for (int c = 0; c < 4; ++c) z[c] = c0 + c < k ? z[c] : 0.0;
        const double nrm = sqrt(row_dot<L>(z, z));
        float zh[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) zh[c] = r < R && nrm > 0.0 ? (float)(z[c] / nrm) : 0.f;
        if (r < R && g == 0) {
            if (mode == 0) {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (c0 + c < k) zhat[r * k + c0 + c] = zh[c];
            }
            if (dst_labels && lane == 0) dst_labels[r] = src_labels[r];
        }
        if (mode == 2) {
            double u[4], h[4];
            consensus_unit<L>(ssum, k, c0, u);
#pragma unroll
            for (int c = 0; c < 4; ++c) h[c] = (double)zh[c];
            const float f = clamp_score(row_dot<L>(h, u));
            if (r < R && lane == 0) alpha[r] = f;
        } else if (g == 0) {
#pragma unroll
            for (int c = 0; c < 4; ++c) cs[rr][c0 + c] = (double)zh[c];
        }
    }
    if (mode == 2) return;  // (uniform)
    __syncthreads();
    if (tid < KP) {
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < ROWS; ++q) s += cs[q][tid];
        __hip_atomic_store(cons_partial + (int64_t)blockIdx.x * 128 + tid, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the stores have reached memory
    __syncthreads();
    if (tid == 0) is_last = atomicAdd(ticket, 1u) == gridDim.x - 1;
    __syncthreads();
    if (!is_last) return;
    const int j = tid & 127, h = tid >> 7, nblocks = (int)gridDim.x;
    double s = 0.0;
    if (j < KP)
        for (int b = h; b < nblocks; b += 64) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                v[u] = b + 8 * u < nblocks ? __hip_atomic_load(cons_partial + (int64_t)(b + 8 * u) * 128 + j, __ATOMIC_RELAXED,
                                                               __HIP_MEMORY_SCOPE_AGENT)
                                           : 0.0;
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
    part[h][j] = s;
    __syncthreads();
    if (h == 0 && j < k) {
        double t = 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u) t += part[u][j];
        ssum[j] = first ? t : ssum[j] + t;
    }
    if (tid == 0) *ticket = 0;
}

ScorePlan score_plan(int64_t R, const Dims& d, int num_cu) {
    ScorePlan p;
    p.row_tiles = (int)((R + 127) / 128);
    int64_t want = ((int64_t)num_cu * 2 + p.row_tiles - 1) / p.row_tiles;
    int64_t s = (want + 7) / 8 * 8;
    int64_t smax = ((d.S + 3) / 4 + 7) / 8 * 8;  // at least ~4 slabs per split
    if (s > smax) s = smax;
    if (s < 8) s = 8;
    if (s > 512) s = 512;
    p.splits = (int)s;
    p.slabs_per_split = (d.S + s - 1) / s;
    return p;
}

template <int NT>
static hipError_t launch_project_nt(const void* G, int dtype, bool vec, int64_t R, const float* Vblk, float* partial,
                                    const ScorePlan& p, const Dims& d, hipStream_t st) {
    dim3 grid((unsigned)(p.row_tiles * p.splits));
#define SAGE_PROJ(TT, VV)                                                                                          \
    hipLaunchKernelGGL((project_kernel<NT, TT, VV>), grid, dim3(256), 0, st, (const TT*)G, R, Vblk, partial,       \
                       p.row_tiles, d.D, d.S, p.slabs_per_split)
    if (dtype == SAGE_BF16) {
        if (vec) SAGE_PROJ(uint16_t, true); else SAGE_PROJ(uint16_t, false);
    } else {
        if (vec) SAGE_PROJ(float, true); else SAGE_PROJ(float, false);
    }
#undef SAGE_PROJ
    return hipGetLastError();
}

hipError_t launch_project(const void* G, int dtype, int64_t R, const float* Vblk, int KP, float* partial,
                          const ScorePlan& p, const Dims& d, hipStream_t st) {
    size_t esz = dtype == SAGE_BF16 ? 2 : 4;
    bool vec = (d.D % 4 == 0) && (((uintptr_t)G) % (4 * esz) == 0);
    switch (KP / 32) {
        case 1: return launch_project_nt<1>(G, dtype, vec, R, Vblk, partial, p, d, st);
        case 2: return launch_project_nt<2>(G, dtype, vec, R, Vblk, partial, p, d, st);
        case 4: return launch_project_nt<4>(G, dtype, vec, R, Vblk, partial, p, d, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_score_finalize(const float* partial, int64_t R, int KP, int k, int splits, float* zhat_out,
                                 double* cons_partial, unsigned* ticket, double* ssum, int mode, bool first, float* alpha_out,
                                 const int* src_labels, int* dst_labels, hipStream_t st) {
    // four waves a row where a lane would add up more than 32 splits
    const int wpr = splits * KP / 256 > 32 ? 4 : 1;
    const unsigned blocks = (unsigned)((R * wpr + 15) / 16);
#define SAGE_FIN(K, W)                                                                                                  \
    hipLaunchKernelGGL((score_finalize_kernel<K, W>), dim3(blocks), dim3(1024), 0, st, partial, R, k, splits, zhat_out, \
                       cons_partial, ticket, mode, first ? 1 : 0, ssum, alpha_out, src_labels, dst_labels)
    switch (KP / 32) {
        case 1: if (wpr == 4) SAGE_FIN(32, 4); else SAGE_FIN(32, 1); break;
        case 2: if (wpr == 4) SAGE_FIN(64, 4); else SAGE_FIN(64, 1); break;
        case 4: if (wpr == 4) SAGE_FIN(128, 4); else SAGE_FIN(128, 1); break;
        default: return hipErrorInvalidValue;
    }
#undef SAGE_FIN
    return hipGetLastError();
}

}  // namespace sage
