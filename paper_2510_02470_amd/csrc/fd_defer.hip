// Shrinks whose rows are not written at once.
//
// A shrink replaces [top; b] by M [top; b] (M = diag(w) Y^T, ell rows). The next eigensolve needs only the Gram matrix of those
// rows and the next block b': diag(known), b' b'^T and the rectangle b' [top; b]^T M^T. The products b' top^T and b' b^T do not
// depend on M, so they are formed beside the eigensolve that makes it, and what is left after it is an (ell x 2 ell) x (2 ell x ell)
// product in fp64. The rows themselves are written later (beside the next eigensolve, or once for several shrinks): after p
// of them they are W [top; b_1; ..; b_p] with W_1 = M_1, W_{p+1} = [M_top W_p, M_new]. W is kept in fp64, so p shrinks round the
// rows to fp32 once: the error of the sketch's covariance is 0.92 (p = 2) and 0.85 (p = 3) of that with a rebuild per shrink.
//
// Everything here is small (at most 256 x 1280 by 1280 x 256) and bound by latency: a 16 x 16 tile of a result per work-group, the
// contraction shared by its four waves.
#include <hip/hip_ext.h>

#include "fd_coeffs.h"
#include "sage_internal.h"

namespace sage {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

// Tile (i0, n0) of A B^T (B_ROWS: A B), A row-major: the sum over four waves in part[i][n].
template <bool B_ROWS>
__device__ __forceinline__ void gemm_tile(const double* __restrict__ A, int lda, const double* __restrict__ B, int ldb, int K, int i0,
                                          int n0, double (&part)[4][16][17]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, g = lane >> 4, per = K >> 2;
    // lane (r, g) supplies row r of either operand at k-slots 2 g, 2 g + 1 of every eight
    const double* a = A + (int64_t)(i0 + r) * lda + wave * per + 2 * g;
    const double* b = B_ROWS ? B + (int64_t)(wave * per + 2 * g) * ldb + n0 + r : B + (int64_t)(n0 + r) * ldb + wave * per + 2 * g;
    f64x4 acc0 = {0.0, 0.0, 0.0, 0.0}, acc1 = {0.0, 0.0, 0.0, 0.0};
    for (int k = 0; k < per; k += 8) {
        const f64x2 x = *reinterpret_cast<const f64x2*>(a + k);
        f64x2 y;
        if constexpr (B_ROWS) y = f64x2{b[(int64_t)k * ldb], b[(int64_t)(k + 1) * ldb]};
        else y = *reinterpret_cast<const f64x2*>(b + k);
        acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(x[0], y[0], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(x[1], y[1], acc1, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) part[wave][4 * v + g][r] = acc0[v] + acc1[v];
    __syncthreads();
}

// out[i][m] = sum_k K[i][k] W[m][k]
__global__ __launch_bounds__(256) void defer_fold_kernel(const double* __restrict__ K, int ldk, const double* __restrict__ W, int ldw,
                                                         int len, double* __restrict__ out, int ldo) {
    __shared__ double part[4][16][17];
    const int i0 = blockIdx.x * 16, m0 = blockIdx.y * 16;
    gemm_tile<false>(K, ldk, W, ldw, len, i0, m0, part);
    const int i = threadIdx.x >> 4, m = threadIdx.x & 15;
    out[(int64_t)(i0 + i) * ldo + m0 + m] = (part[0][i][m] + part[1][i][m]) + (part[2][i][m] + part[3][i][m]);
}

// The same into the new x top rectangle of C (both triangles); the top x top block becomes diag(known).
__global__ __launch_bounds__(256) void defer_cross_kernel(const double* __restrict__ K, int ldk, const double* __restrict__ W, int ldw,
                                                          int len, double* __restrict__ C, int NP, const double* __restrict__ known) {
    __shared__ double part[4][16][17];
    const int i0 = blockIdx.x * 16, m0 = blockIdx.y * 16, LP = NP >> 1;
    gemm_tile<false>(K, ldk, W, ldw, len, i0, m0, part);
    const int q = threadIdx.x >> 4, p = threadIdx.x & 15;
    C[(int64_t)(LP + i0 + q) * NP + m0 + p] = (part[0][q][p] + part[1][q][p]) + (part[2][q][p] + part[3][q][p]);
    C[(int64_t)(m0 + q) * NP + LP + i0 + p] = (part[0][p][q] + part[1][p][q]) + (part[2][p][q] + part[3][p][q]);
    C[(int64_t)(i0 + q) * NP + m0 + p] = i0 + q == m0 + p ? known[i0 + q] : 0.0;
}

// W' = [M_top W, M_new]: columns below `cols` by products, LP more copied.
__global__ __launch_bounds__(256) void defer_compose_kernel(const double* __restrict__ M, int NP, const double* __restrict__ W, int ldw,
                                                            int cols, double* __restrict__ out, int ldo) {
    __shared__ double part[4][16][17];
    const int m0 = blockIdx.x * 16, c0 = blockIdx.y * 16, LP = NP >> 1;
    const int m = threadIdx.x >> 4, c = threadIdx.x & 15;
    if (c0 >= cols) {
        out[(int64_t)(m0 + m) * ldo + c0 + c] = M[(int64_t)(m0 + m) * NP + LP + c0 - cols + c];
        return;
    }
    gemm_tile<true>(M, NP, W, ldw, LP, m0, c0, part);
    out[(int64_t)(m0 + m) * ldo + c0 + c] = (part[0][m][c] + part[1][m][c]) + (part[2][m][c] + part[3][m][c]);
}

// The rebuild's coefficients from W, `stages` stages of 16 buffer rows.
template <bool SPLIT>
__global__ __launch_bounds__(256) void defer_coeffs_kernel(const double* __restrict__ W, int ldw, int MP, int stages,
                                                           float* __restrict__ Mt, void* __restrict__ Mc3) {
    const int t = blockIdx.x * 256 + threadIdx.x, stg = (t >> 1) % stages, m = (t >> 1) / stages, h = t & 1;
    if (m >= MP) return;
    const double* w = W + (int64_t)m * ldw + stg * 16 + h;
    Coeffs8 v;
#pragma unroll
    for (int s = 0; s < 8; ++s) v.c[s] = (float)w[2 * s];
    store_coeffs<SPLIT>(Mt, Mc3, MP, stg, h, m, v);
}

// The partial tiles of the rectangles (new rows x the top rows of source s) summed over groups into K, source s from column
// col[s] on, and those of the new x new triangle into C. SEG threads share an element's groups, as in gram_reduce_kernel.
struct DeferReduce {
    const float* cross;
    int64_t stride;  // between the sources' partial tiles
    int sources, top_groups, cross_groups;  // groups of the first source, of the others
    int col[GRAM_TOPS];
    const float* fresh;  // the triangle's
    int fresh_tiles, fresh_groups;
};
template <int SEG>
__global__ __launch_bounds__(256) void defer_reduce_kernel(DeferReduce g, double* __restrict__ K, int ldk, double* __restrict__ C, int NP) {
    constexpr int EL = 256 / SEG;
    __shared__ double part[SEG][EL];
    const int q = NP / 128, LP = NP >> 1, t = blockIdx.x;
    const int el = threadIdx.x % EL, seg = threadIdx.x / EL, e = blockIdx.y * EL + el;
    const bool cross = t < g.sources * q * q;
    const int s = cross ? t / (q * q) : 0, idx = cross ? t - s * q * q : t - g.sources * q * q;
    const float* p0 = (cross ? g.cross + s * g.stride : g.fresh) + (int64_t)idx * 4096 + e;
    const int64_t gstride = (int64_t)(cross ? q * q : g.fresh_tiles) * 4096;
    const int groups = cross ? (s == 0 ? g.top_groups : g.cross_groups) : g.fresh_groups, per = (groups + SEG - 1) / SEG;
    int k = seg * per;
    const int k1 = k + per < groups ? k + per : groups;
    double sum = 0.0;
    for (; k + 8 <= k1; k += 8) {  // eight loads in flight, added in group order
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = p0[(k + u) * gstride];
#pragma unroll
        for (int u = 0; u < 8; ++u) sum += (double)v[u];
    }
    for (; k < k1; ++k) sum += (double)p0[k * gstride];
    part[seg][el] = sum;
    __syncthreads();
    if (seg > 0) return;
#pragma unroll
    for (int u = 1; u < SEG; ++u) sum += part[u][el];
    const int r = e >> 6, c = e & 63;
    if (cross) {
        K[(int64_t)(idx / q * 64 + r) * ldk + g.col[s] + idx % q * 64 + c] = sum;
        return;
    }
    int ti = 0;
    while ((ti + 1) * (ti + 2) / 2 <= idx) ++ti;
    const int tj = idx - ti * (ti + 1) / 2;
    if (ti == tj && c > r) return;  // the diagonal tiles hold both triangles; keep one
    const int64_t gr = LP + ti * 64 + r, gc = LP + tj * 64 + c;
    C[gr * NP + gc] = sum;
    C[gc * NP + gr] = sum;
}

hipError_t launch_defer_reduce(const float* cross, int64_t stride, int sources, const int* col, int top_groups, int groups, const float* fresh,
                               const GramPlan& pn, double* K, int ldk, double* C, const Dims& d, hipStream_t st) {
    DeferReduce g{cross, stride, sources, top_groups, groups, {}, fresh, pn.tiles, pn.groups};
    for (int s = 0; s < sources; ++s) g.col[s] = col[s];
    const int q = d.NP / 128, tiles = sources * q * q + q * (q + 1) / 2;
    if (groups >= 64)
        hipLaunchKernelGGL(defer_reduce_kernel<8>, dim3(tiles, 128), dim3(256), 0, st, g, K, ldk, C, d.NP);
    else
        hipLaunchKernelGGL(defer_reduce_kernel<1>, dim3(tiles, 16), dim3(256), 0, st, g, K, ldk, C, d.NP);
    return hipGetLastError();
}

hipError_t launch_defer_fold(const double* K, int ldk, const double* W, int ldw, int len, double* out, int ldo, const Dims& d,
                             hipStream_t st) {
    hipLaunchKernelGGL(defer_fold_kernel, dim3(d.LP / 16, d.LP / 16), dim3(256), 0, st, K, ldk, W, ldw, len, out, ldo);
    return hipGetLastError();
}

hipError_t launch_defer_cross(const double* K, int ldk, const double* W, int ldw, int len, double* C, const double* known,
                              const Dims& d, hipStream_t st, hipEvent_t done) {
    const dim3 grid(d.LP / 16, d.LP / 16);
    // (`done` rides on the launch's own completion, as in launch_gram_reduce)
    if (done)
        hipExtLaunchKernelGGL(defer_cross_kernel, grid, dim3(256), 0, st, nullptr, done, 0, K, ldk, W, ldw, len, C, d.NP, known);
    else
        hipLaunchKernelGGL(defer_cross_kernel, grid, dim3(256), 0, st, K, ldk, W, ldw, len, C, d.NP, known);
    return hipGetLastError();
}

hipError_t launch_defer_compose(const double* M, const double* W, int ldw, int cols, double* out, int ldo, const Dims& d,
                                hipStream_t st) {
    hipLaunchKernelGGL(defer_compose_kernel, dim3(d.LP / 16, (cols + d.LP) / 16), dim3(256), 0, st, M, d.NP, W, ldw, cols, out,
                       ldo);
    return hipGetLastError();
}

hipError_t launch_defer_coeffs(const double* W, int ldw, int rows, float* Mt, void* Mc3, const Dims& d, hipStream_t st) {
    const int stages = rows / 16;
    const dim3 grid((unsigned)((2 * stages * d.LP + 255) / 256));
    if (Mc3) hipLaunchKernelGGL(defer_coeffs_kernel<true>, grid, dim3(256), 0, st, W, ldw, d.LP, stages, Mt, Mc3);
    else hipLaunchKernelGGL(defer_coeffs_kernel<false>, grid, dim3(256), 0, st, W, ldw, d.LP, stages, Mt, Mc3);
    return hipGetLastError();
}

}  // namespace sage
