// fp64 helpers of the eigensolver kernels: sums over a wave by DPP (no LDS), reciprocals.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace sage {

template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
    const long long u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)u, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp((int)(u >> 32), CTRL, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
constexpr int DPP_XOR1 = 0xB1;         // quad_perm [1,0,3,2]
constexpr int DPP_XOR2 = 0x4E;         // quad_perm [2,3,0,1]
constexpr int DPP_HALF_MIRROR = 0x141; // lane l of 8 -> 7 - l: the other quad once quads are uniform
constexpr int DPP_MIRROR = 0x140;      // lane l of 16 -> 15 - l: the other half once halves are uniform

__device__ __forceinline__ double read_lane(double v, int lane) {
    const long long u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)u, lane);
    const int hi = __builtin_amdgcn_readlane((int)(u >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Partner of a lane 16 (32) lanes away: the swap instruction on two copies leaves one value of each pair in either result.
template <int D>
__device__ __forceinline__ void swap_rows(double v, double& a, double& b) {
    static_assert(D == 16 || D == 32, "rows of 16 or halves of 32 lanes");
    const long long u = __double_as_longlong(v);
    const unsigned lo = (unsigned)u, hi = (unsigned)(u >> 32);
    const auto l = D == 16 ? __builtin_amdgcn_permlane16_swap(lo, lo, false, false)
                           : __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto h = D == 16 ? __builtin_amdgcn_permlane16_swap(hi, hi, false, false)
                           : __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    a = __longlong_as_double(((long long)h[0] << 32) | l[0]);
    b = __longlong_as_double(((long long)h[1] << 32) | l[1]);
}

// Sum over groups of L lanes (L = 4, 8, 16 or 64), the same bits in every lane of the group.
template <int L>
__device__ __forceinline__ double lane_sum(double v) {
    v += dpp_move<DPP_XOR1>(v);
    v += dpp_move<DPP_XOR2>(v);
    if constexpr (L >= 8) v += dpp_move<DPP_HALF_MIRROR>(v);
    if constexpr (L >= 16) v += dpp_move<DPP_MIRROR>(v);
    if constexpr (L == 64) {
        double a, b;
        swap_rows<16>(v, a, b);
        v = a + b;
        swap_rows<32>(v, a, b);
        v = a + b;
    }
    return v;
}
// Three sums at once: their stages alternate, so that none waits for its own result.
template <int L>
__device__ __forceinline__ void lane_sum3(double& a, double& b, double& c) {
    auto stage = [&](auto ctrl) __attribute__((always_inline)) {
        constexpr int CTRL = decltype(ctrl)::value;
        const double x = dpp_move<CTRL>(a), y = dpp_move<CTRL>(b), z = dpp_move<CTRL>(c);
        a += x;
        b += y;
        c += z;
        __builtin_amdgcn_sched_barrier(0);
    };
    auto swap = [&](auto dist) __attribute__((always_inline)) {
        constexpr int D = decltype(dist)::value;
        double x0, x1, y0, y1, z0, z1;
        swap_rows<D>(a, x0, x1);
        swap_rows<D>(b, y0, y1);
        swap_rows<D>(c, z0, z1);
        a = x0 + x1;
        b = y0 + y1;
        c = z0 + z1;
        __builtin_amdgcn_sched_barrier(0);
    };
    stage(std::integral_constant<int, DPP_XOR1>{});
    stage(std::integral_constant<int, DPP_XOR2>{});
    if constexpr (L >= 8) stage(std::integral_constant<int, DPP_HALF_MIRROR>{});
    if constexpr (L >= 16) stage(std::integral_constant<int, DPP_MIRROR>{});
    if constexpr (L == 64) {
        swap(std::integral_constant<int, 16>{});
        swap(std::integral_constant<int, 32>{});
    }
}
template <int L>
__device__ __forceinline__ double lane_product(double v) {
    v *= dpp_move<DPP_XOR1>(v);
    v *= dpp_move<DPP_XOR2>(v);
    if constexpr (L >= 8) v *= dpp_move<DPP_HALF_MIRROR>(v);
    if constexpr (L >= 16) v *= dpp_move<DPP_MIRROR>(v);
    if constexpr (L == 64) {
        double a, b;
        swap_rows<16>(v, a, b);
        v = a * b;
        swap_rows<32>(v, a, b);
        v = a * b;
    }
    return v;
}
template <int CTRL>
__device__ __forceinline__ int dpp_move_i(int v) {
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, false);
}
template <int L>
__device__ __forceinline__ int lane_sum_i(int v) {
    v += dpp_move_i<DPP_XOR1>(v);
    v += dpp_move_i<DPP_XOR2>(v);
    if constexpr (L >= 8) v += dpp_move_i<DPP_HALF_MIRROR>(v);
    if constexpr (L >= 16) v += dpp_move_i<DPP_MIRROR>(v);
    if constexpr (L == 64)
        v = (__builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16)) +
            (__builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48));
    return v;
}

// 1 / x to about one unit in the last place for normal x: the hardware estimate y, good to 2^-22 or better, and one step of
// third order, y (1 + e + e^2) with e = 1 - x y.
__device__ __forceinline__ double rcp64(double x) {
    const double y = __builtin_amdgcn_rcp(x);
    const double e = __builtin_fma(-x, y, 1.0);
    return __builtin_fma(y, __builtin_fma(e, e, e), y);
}

}  // namespace sage
