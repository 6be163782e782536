// Rows of projections in a wave: L = KP / 4 lanes hold four coordinates each, the 64 / L groups of such lanes a copy each (or,
// before group_sum, a share of the sum each). Everything that two kernels must compute to the same bits is here.
#pragma once
#include "sage_internal.h"
#include "wave_ops.h"

namespace sage {

// sum over the groups: lanes l, l + L, l + 2 L, ...
template <int L>
__device__ __forceinline__ double group_sum(double v) {
    double a, b;
    if constexpr (L <= 8) v += dpp_move<0x128>(v);  // row_ror 8
    if constexpr (L <= 16) {
        swap_rows<16>(v, a, b);
        v = a + b;
    }
    swap_rows<32>(v, a, b);
    return a + b;
}

// <x, y> of one row, the same bits in every lane
template <int L>
__device__ __forceinline__ double row_dot(const double (&x)[4], const double (&y)[4]) {
    double v = x[0] * y[0];
#pragma unroll
    for (int c = 1; c < 4; ++c) v = __builtin_fma(x[c], y[c], v);
    v = lane_sum<8>(v);
    if constexpr (L >= 16) v += dpp_move<0x128>(v);  // row_ror 8
    if constexpr (L >= 32) {
        double a, b;
        swap_rows<16>(v, a, b);
        v = a + b;
    }
    return v;
}

// u = s / ||s||, 0 if s = 0: this lane's coordinates c0 .. c0 + 3
template <int L>
__device__ __forceinline__ void consensus_unit(const double* __restrict__ ssum, int k, int c0, double (&u)[4]) {
    double s[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) s[c] = c0 + c < k ? ssum[c0 + c] : 0.0;
    const double nrm = sqrt(row_dot<L>(s, s));
#pragma unroll
    for (int c = 0; c < 4; ++c) u[c] = nrm > 0.0 ? s[c] / nrm : 0.0;
}

__device__ __forceinline__ float clamp_score(double a) {
    if (a > 1.0) a = 1.0;
    if (a < -1.0) a = -1.0;
    float f = (float)a;
    if (f == 0.f) f = 0.f;  // -0 -> +0
    return f;
}

}  // namespace sage
