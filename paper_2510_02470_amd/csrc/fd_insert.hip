// Row movement between the caller's row-major batches and the library's column-slab layout.
// Algorithm 1, Phase I, "S[r mod ell, :] <- g": a row is placed into a free (zero) buffer row.
#include "fd_rows.h"
#include "sage_internal.h"

namespace sage {

// A wave moves 16 rows x NS slabs: lane = (row, piece), so that a store is 16 consecutive rows of a slab, 1 KB without a
// gap, and the four waves of a work-group store 64 rows. (A thread per piece along a row stored 64-byte pieces 16 KB apart:
// 590 us for 256 fp32 rows of 1,048,576, 3.6 TB/s, and 1060 us for bf16 rows of 2,049,000.) The NS loads of a row are
// neighbours and in flight together. Columns >= D are written as zero so that padding never carries data.
// hole: see spare_unit_at.
template <int NS, typename Src>
__global__ __launch_bounds__(256) void insert_kernel(Src src, int rows, int row0, float* __restrict__ B, int NP, int64_t D,
                                                     int64_t S, int row_groups, int64_t units, const int* __restrict__ hole) {
    const int64_t unit = spare_unit_at(hole);
    if (unit < 0 || unit >= units) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = (int)((unsigned)unit % (unsigned)row_groups) * 64 + wave * 16 + (lane >> 2);
    if (r >= rows) return;
    const int64_t s0 = (int64_t)((unsigned)unit / (unsigned)row_groups) * NS;
    const int p = lane & 3;
    float4 v[NS];
    src.template load<NS>(r, s0 * DC + p * 4, D, v);
    float4* dst = reinterpret_cast<float4*>(B + (s0 * NP + row0 + r) * DC) + p;
#pragma unroll
    for (int i = 0; i < NS; ++i)
        if (s0 + i < S) dst[(int64_t)i * NP * (DC / 4)] = v[i];
}

// The same for a half kept in pieces of bf16: lane = (row, piece of four neighbours), so that a store is four runs of 16
// rows, 256 bytes each, and a work-group's are 1 KB.
template <int NS, typename Src>
__global__ __launch_bounds__(256) void insert16_kernel(Src src, int rows, int row0, u32x4* __restrict__ B, int LP, int64_t D,
                                                       int64_t Q, int row_groups, int64_t units, const int* __restrict__ hole) {
    const int64_t unit = spare_unit_at(hole);
    if (unit < 0 || unit >= units) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = (int)((unsigned)unit % (unsigned)row_groups) * 64 + wave * 16 + (lane & 15);
    if (r >= rows) return;
    const int64_t q0 = (int64_t)((unsigned)unit / (unsigned)row_groups) * (4 * NS) + (lane >> 4);
    u32x4 v[NS];
    src.template load16<NS>(r, q0 * 8, D, v);
    u32x4* dst = B + q0 * LP + row0 + r;
#pragma unroll
    for (int i = 0; i < NS; ++i)
        if (q0 + 4 * i < Q) dst[(int64_t)(4 * i) * LP] = v[i];
}

template <typename Src>
static hipError_t launch_insert_src(const Src& src, int64_t rows, int row0, float* half, int half_rows, const Dims& d,
                                    bool to16, const int* hole, hipStream_t st) {
    if (rows <= 0) return hipSuccess;
    const int row_groups = (int)((rows + 63) / 64);
    if constexpr (Src::BF16) {
        if (to16) {
            const int64_t Q = 2 * d.S, units = (Q + 31) / 32 * row_groups;  // 8 loads a lane, 512 bytes of a row
            hipLaunchKernelGGL((insert16_kernel<8, Src>), dim3((unsigned)spare_grid_at(units, hole)), dim3(256), 0, st, src, (int)rows,
                               row0, const_cast<u32x4*>(half16(half, half_rows, d.S)), half_rows, d.D, Q, row_groups, units, hole);
            return hipGetLastError();
        }
    }
    // 16 slabs a wave, 16 KB of fp32 stores; 4 where that would leave the chip short of waves
    const int64_t wide = (d.S + 15) / 16 * row_groups;
    const int64_t units = wide >= 1024 ? wide : (d.S + 3) / 4 * row_groups;
    const dim3 grid((unsigned)spare_grid_at(units, hole));
    if (wide >= 1024)
        hipLaunchKernelGGL((insert_kernel<16, Src>), grid, dim3(256), 0, st, src, (int)rows, row0, half, half_rows, d.D, d.S,
                           row_groups, units, hole);
    else
        hipLaunchKernelGGL((insert_kernel<4, Src>), grid, dim3(256), 0, st, src, (int)rows, row0, half, half_rows, d.D, d.S,
                           row_groups, units, hole);
    return hipGetLastError();
}

hipError_t launch_insert(const void* G, int dtype, int64_t rows, int row0, float* half, int half_rows, const Dims& d,
                         bool to16, const int* hole, hipStream_t st) {
    const bool vec = rows_start_on_four(G, dtype, d);
#define SAGE_INSERT(T, V) launch_insert_src(DenseRows<T, V>{(const T*)G}, rows, row0, half, half_rows, d, to16, hole, st)
    if (dtype == SAGE_BF16) return vec ? SAGE_INSERT(uint16_t, true) : SAGE_INSERT(uint16_t, false);
    return vec ? SAGE_INSERT(float, true) : SAGE_INSERT(float, false);
#undef SAGE_INSERT
}

// Pieces of bf16 to the fp32 half, in place: slab s goes to bytes [16 KB s ..) of LP = 256 rows, its pieces lie at half the
// memory plus 8 KB s. The first half of the slabs overwrites no pieces, the next quarter only such as are done with, and so
// on; the last slab overwrites its own, which its work-group has read by then.
__global__ __launch_bounds__(512) void widen_kernel(float* __restrict__ half, int LP, int64_t S, int64_t s0) {
    const int64_t s = s0 + blockIdx.x;
    const u32x4* src = half16(half, LP, S) + 2 * s * LP;
    u32x4 v[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int p = i * 512 + threadIdx.x;  // piece (column group p / LP, row p % LP)
        v[i] = p < 2 * LP ? src[p] : u32x4{0u, 0u, 0u, 0u};
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int p = i * 512 + threadIdx.x;
        if (p >= 2 * LP) continue;
        float4* dst = reinterpret_cast<float4*>(half + (s * LP + p % LP) * DC + (p / LP) * 8);
#pragma unroll
        for (int h = 0; h < 2; ++h)
            dst[h] = make_float4(__uint_as_float(v[i][2 * h] << 16), __uint_as_float(v[i][2 * h] & 0xffff0000u),
                                 __uint_as_float(v[i][2 * h + 1] << 16), __uint_as_float(v[i][2 * h + 1] & 0xffff0000u));
    }
}

hipError_t launch_widen(float* half, const Dims& d, hipStream_t st) {
    if (d.LP > 512) return hipErrorInvalidValue;
    for (int64_t lo = 0; lo < d.S;) {
        int64_t hi = (d.S + lo) / 2;
        if (hi == lo) hi = lo + 1;
        hipLaunchKernelGGL(widen_kernel, dim3((unsigned)(hi - lo)), dim3(512), 0, st, half, d.LP, d.S, lo);
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
        lo = hi;
    }
    return hipSuccess;
}

hipError_t launch_insert_outer(const void* E, const void* H, int dtype, int64_t C, int64_t dh, int64_t rows, int row0,
                               float* half, int half_rows, const Dims& d, bool to16, const int* hole, hipStream_t st) {
    if (dtype == SAGE_BF16)
        return launch_insert_src(OuterRows<uint16_t>{(const uint16_t*)E, (const uint16_t*)H, C, dh}, rows, row0, half,
                                 half_rows, d, to16, hole, st);
    return launch_insert_src(OuterRows<float>{(const float*)E, (const float*)H, C, dh}, rows, row0, half, half_rows, d, false,
                             hole, st);
}

// The same rows written out row-major in their own type (for shapes the factored projection does not take).
template <typename T>
__global__ __launch_bounds__(256) void expand_outer_kernel(const T* __restrict__ E, const T* __restrict__ H, int64_t C,
                                                           int64_t dh, T* __restrict__ out, int64_t D) {
    const int64_t col = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (col >= D) return;
    const int64_t r = blockIdx.y;
    const float x = outer_value(E + r * C, H + r * dh, col, C * dh, dh, D);
    if constexpr (sizeof(T) == 2) out[r * D + col] = (uint16_t)(__float_as_uint(x) >> 16);  // x is a bf16 value already
    else out[r * D + col] = x;
}

hipError_t launch_expand_outer(const void* E, const void* H, int dtype, int64_t C, int64_t dh, int64_t rows, void* out,
                               const Dims& d, hipStream_t st) {
    if (rows <= 0) return hipSuccess;
    dim3 grid((unsigned)((d.D + 255) / 256), (unsigned)rows);
    if (dtype == SAGE_BF16)
        hipLaunchKernelGGL(expand_outer_kernel<uint16_t>, grid, dim3(256), 0, st, (const uint16_t*)E, (const uint16_t*)H, C,
                           dh, (uint16_t*)out, d.D);
    else
        hipLaunchKernelGGL(expand_outer_kernel<float>, grid, dim3(256), 0, st, (const float*)E, (const float*)H, C, dh,
                           (float*)out, d.D);
    return hipGetLastError();
}

// slab layout (NPsrc rows) -> row-major nrows x D
__global__ __launch_bounds__(256) void export_kernel(const float* __restrict__ Bblk, int NPsrc, float* __restrict__ out,
                                                     int64_t D) {
    int64_t dcol = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (dcol >= D) return;
    int r = blockIdx.y;
    out[(int64_t)r * D + dcol] = Bblk[blk_off(dcol, r, NPsrc)];
}

hipError_t launch_export_rows(const float* Bblk, int NPsrc, int nrows, float* out, const Dims& d, hipStream_t st) {
    if (nrows <= 0) return hipSuccess;
    dim3 grid((unsigned)((d.D + 255) / 256), (unsigned)nrows);
    hipLaunchKernelGGL(export_kernel, grid, dim3(256), 0, st, Bblk, NPsrc, out, d.D);
    return hipGetLastError();
}

// row-major nrows x D -> slab layout with NPdst rows; rows nrows..NPdst-1 and columns >= D are zeroed.
__global__ __launch_bounds__(256) void import_kernel(const float* __restrict__ in, int nrows, float* __restrict__ Bblk,
                                                     int NPdst, int64_t D, int64_t Dp) {
    int64_t dcol = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (dcol >= Dp) return;
    int r = blockIdx.y;
    float v = (r < nrows && dcol < D) ? in[(int64_t)r * D + dcol] : 0.f;
    Bblk[blk_off(dcol, r, NPdst)] = v;
}

hipError_t launch_import_rows(const float* in, int nrows, float* Bblk, int NPdst, const Dims& d, hipStream_t st) {
    dim3 grid((unsigned)((d.Dp + 255) / 256), (unsigned)NPdst);
    hipLaunchKernelGGL(import_kernel, grid, dim3(256), 0, st, in, nrows, Bblk, NPdst, d.D, d.Dp);
    return hipGetLastError();
}

// out[r][c] = in[map(r)][both ? map(c) : c] with map = buffer-row order -> matrix index: r < ell -> r,
// ell <= r < 2 ell -> LP + r - ell, then the padding indices in ascending order.
__device__ __forceinline__ int probe_map(int r, int LP, int ell) {
    if (r < ell) return r;
    if (r < 2 * ell) return LP + r - ell;
    int k = r - 2 * ell;                    // k-th padding index
    return k < LP - ell ? ell + k : LP + ell + (k - (LP - ell));
}
__global__ __launch_bounds__(256) void probe_permute_kernel(const double* __restrict__ in, double* __restrict__ out, int NP,
                                                            int LP, int ell, int both) {
    int r = blockIdx.x;
    int mr = probe_map(r, LP, ell);
    for (int c = threadIdx.x; c < NP; c += 256) {
        int mc = both ? probe_map(c, LP, ell) : c;
        out[(int64_t)r * NP + c] = in[(int64_t)mr * NP + mc];
    }
}

hipError_t launch_probe_permute(const double* in, double* out, int NP, int LP, int ell, bool both, hipStream_t st) {
    hipLaunchKernelGGL(probe_permute_kernel, dim3(NP), dim3(256), 0, st, in, out, NP, LP, ell, both ? 1 : 0);
    return hipGetLastError();
}

// plain copy, 16 bytes per thread (harnesses time / count it to calibrate hardware counters)
__global__ __launch_bounds__(256) void plain_copy_kernel(const f32x4* __restrict__ src, f32x4* __restrict__ dst, int64_t n16) {
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n16) dst[i] = src[i];
}

hipError_t launch_plain_copy(const void* src, void* dst, int64_t bytes, hipStream_t st) {
    const int64_t n16 = bytes / 16;
    if (n16 <= 0) return hipSuccess;
    hipLaunchKernelGGL(plain_copy_kernel, dim3((unsigned)((n16 + 255) / 256)), dim3(256), 0, st, (const f32x4*)src,
                       (f32x4*)dst, n16);
    return hipGetLastError();
}

// Debug check of caller data: *count += the number of entries that are not finite (exponent bits all ones).
template <typename T>
__global__ __launch_bounds__(256) void count_nonfinite_kernel(const T* __restrict__ p, int64_t n, unsigned* __restrict__ count) {
    unsigned bad = 0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        if (sizeof(T) == 2) bad += (((unsigned)p[i]) & 0x7F80u) == 0x7F80u;
        else bad += (((unsigned)p[i]) & 0x7F800000u) == 0x7F800000u;
    }
    for (int o = 32; o >= 1; o >>= 1) bad += __shfl_xor(bad, o);
    if ((threadIdx.x & 63) == 0 && bad) atomicAdd(count, bad);
}

hipError_t launch_count_nonfinite(const void* p, int dtype, int64_t n, unsigned* count, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 2048) blocks = 2048;
    if (dtype == SAGE_BF16)
        hipLaunchKernelGGL(count_nonfinite_kernel<uint16_t>, dim3((unsigned)blocks), dim3(256), 0, st, (const uint16_t*)p, n, count);
    else
        hipLaunchKernelGGL(count_nonfinite_kernel<uint32_t>, dim3((unsigned)blocks), dim3(256), 0, st, (const uint32_t*)p, n, count);
    return hipGetLastError();
}

// zero buffer rows [r0, r1) in every slab
__global__ __launch_bounds__(256) void zero_rows_kernel(float* __restrict__ Bblk, int NP, int r0, int r1, int64_t S) {
    int per_slab = (r1 - r0) * 4;  // float4 pieces per slab
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= S * per_slab) return;
    int64_t s = i / per_slab;
    int rem = (int)(i % per_slab);
    float4* p = reinterpret_cast<float4*>(Bblk + (s * NP + r0) * DC) + rem;
    *p = make_float4(0.f, 0.f, 0.f, 0.f);
}

hipError_t launch_zero_rows(float* Bblk, int NP, int r0, int r1, const Dims& d, hipStream_t st) {
    if (r1 <= r0) return hipSuccess;
    int64_t total = d.S * (int64_t)(r1 - r0) * 4;
    hipLaunchKernelGGL(zero_rows_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, Bblk, NP, r0, r1, d.S);
    return hipGetLastError();
}

}  // namespace sage
