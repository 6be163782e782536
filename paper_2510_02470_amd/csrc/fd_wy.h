// Block reflectors of the back-transformation: eight Householder reflectors in one factor,
// H_0 H_1 .. H_7 = I - V T V^T with T upper triangular (R. Schreiber, C. Van Loan, SIAM J. Sci. Stat. Comput. 10, 1989).
#pragma once
#include "wave_ops.h"

namespace sage {

constexpr int WY = 8;  // reflectors per block

// T of block b (WY x WY, row-major, zeros below the diagonal) by one wave: V row k = reflector k (N = 64 J entries), only
// reflectors k <= n - 2 exist.
template <int J>
__device__ __forceinline__ void wy_factor(const double* __restrict__ V, const double* __restrict__ tauT, int b, int n, int lane,
                                          double* __restrict__ T) {
    constexpr int N = 64 * J;
    double v[WY][J], tau[WY];
#pragma unroll
    for (int i = 0; i < WY; ++i) {
        const int k = b * WY + i;
        tau[i] = k <= n - 2 ? tauT[k] : 0.0;
#pragma unroll
        for (int j = 0; j < J; ++j) v[i][j] = k <= n - 2 ? V[(int64_t)k * N + lane + 64 * j] : 0.0;
    }
    double t[WY][WY];
#pragma unroll
    for (int i = 0; i < WY; ++i) {
        double g[WY];
#pragma unroll
        for (int p = 0; p < i; ++p) {
            double s = 0.0;
#pragma unroll
            for (int j = 0; j < J; ++j) s = __builtin_fma(v[p][j], v[i][j], s);
            g[p] = lane_sum<64>(s);
        }
#pragma unroll
        for (int p = 0; p < i; ++p) {
            double s = 0.0;
#pragma unroll
            for (int q = p; q < i; ++q) s = __builtin_fma(t[p][q], g[q], s);
            t[p][i] = -tau[i] * s;
        }
        t[i][i] = tau[i];
#pragma unroll
        for (int p = i + 1; p < WY; ++p) t[p][i] = 0.0;
    }
    if (lane == 0) {
#pragma unroll
        for (int p = 0; p < WY; ++p)
#pragma unroll
            for (int i = 0; i < WY; ++i) T[b * WY * WY + p * WY + i] = t[p][i];
    }
}

}  // namespace sage
