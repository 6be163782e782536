// Where the rows that are stored come from: a caller's row-major batch or the two factors of last-layer gradient rows. load: NS
// float4, 16 columns apart; load16: NS pieces of eight bf16 values, 32 columns apart; both zero from column D on.
#pragma once
#include "sage_internal.h"

namespace sage {

// Every row of a batch starts on a multiple of four elements.
inline bool rows_start_on_four(const void* G, int dtype, const Dims& d) {
    return d.D % 4 == 0 && (uintptr_t)G % (dtype == SAGE_BF16 ? 8 : 16) == 0;
}

struct __attribute__((packed, aligned(2))) Eight {  // eight bf16 values at any element boundary
    u32x4 v;
};

// Rows of a row-major batch. VEC: every row starts on a multiple of four elements.
template <typename T, bool VEC>
struct DenseRows {
    static constexpr bool BF16 = sizeof(T) == 2;
    const T* G;
    // pieces of 8 columns, 32 columns apart, of a bf16 row (at any element boundary)
    template <int NS>
    __device__ __forceinline__ void load16(int r, int64_t d0, int64_t D, u32x4 (&v)[NS]) const {
        const T* g = G + r * D + d0;
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            const int64_t d = d0 + 32 * i;
            if (d + 8 <= D) {
                v[i] = reinterpret_cast<const Eight*>(g + 32 * i)->v;
            } else {
                T x[8];
#pragma unroll
                for (int c = 0; c < 8; ++c) x[c] = d + c < D ? g[32 * i + c] : (T)0;
                __builtin_memcpy(&v[i], x, sizeof(x) < 16 ? sizeof(x) : 16);
            }
        }
    }
    template <int NS>
    __device__ __forceinline__ void load(int r, int64_t d0, int64_t D, float4 (&v)[NS]) const {
        const T* g = G + r * D + d0;
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            const int64_t d = d0 + i * DC;
            float x[4] = {0.f, 0.f, 0.f, 0.f};
            if (VEC) {
                if (d < D) {  // (D is a multiple of four)
                    if constexpr (sizeof(T) == 2) {
                        const uint2 u = *reinterpret_cast<const uint2*>(g + i * DC);
                        x[0] = __uint_as_float(u.x << 16);
                        x[1] = __uint_as_float(u.x & 0xffff0000u);
                        x[2] = __uint_as_float(u.y << 16);
                        x[3] = __uint_as_float(u.y & 0xffff0000u);
                    } else {
                        const float4 u = *reinterpret_cast<const float4*>(g + i * DC);
                        x[0] = u.x, x[1] = u.y, x[2] = u.z, x[3] = u.w;
                    }
                }
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (d + c < D) {
                        if constexpr (sizeof(T) == 2) x[c] = bf16_to_f32(g[i * DC + c]);
                        else x[c] = g[i * DC + c];
                    }
            }
            v[i] = make_float4(x[0], x[1], x[2], x[3]);
        }
    }
};

// Factored rows (a linear last layer: column c*dh + t of row r is e_rc * h_rt, column C*dh + c is e_rc; Method,
// definition of g_i). The value a caller would have stored in a row of type T: the fp32 product, for bf16 rows
// rounded to nearest even (the product of two bf16 values is exact in fp32).
template <typename T>
__device__ __forceinline__ float outer_value(const T* __restrict__ e, const T* __restrict__ h, int64_t col, int64_t main,
                                             int64_t dh, int64_t D) {
    if (col >= D) return 0.f;
    if constexpr (sizeof(T) == 2) {
        if (col >= main) return bf16_to_f32(e[col - main]);
        const float x = bf16_to_f32(e[col / dh]) * bf16_to_f32(h[col % dh]);
        return (float)(__bf16)x;
    } else {
        if (col >= main) return e[col - main];
        return e[col / dh] * h[col % dh];
    }
}

// Four neighbouring values at any element boundary.
template <typename T>
struct __attribute__((packed, aligned(sizeof(T)))) Four {
    T v[4];
};

// Factored rows for insert_kernel. One division per thread, for the class and feature of its first column, then steps of
// sixteen columns with wrap-around; four columns of one class take one load of h and one of e.
template <typename T>
struct OuterRows {
    static constexpr bool BF16 = sizeof(T) == 2;
    const T* E;
    const T* H;
    int64_t C, dh;
    static __device__ __forceinline__ float value(T e, T h) {
        if constexpr (sizeof(T) == 2) return (float)(__bf16)(bf16_to_f32(e) * bf16_to_f32(h));
        else return e * h;
    }
    // pieces of 8 columns, 32 columns apart
    template <int NS>
    __device__ __forceinline__ void load16(int r, int64_t d0, int64_t D, u32x4 (&v)[NS]) const {
        const int64_t main = C * dh;
        const T* e = E + r * C;
        const T* h = H + r * dh;
        int64_t cls = d0 / dh, t = d0 - cls * dh;
        T ev[NS];
        bool fast[NS];
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            fast[i] = cls < C && t + 7 < dh;
            if (fast[i]) {
                ev[i] = e[cls];
                v[i] = reinterpret_cast<const Eight*>(h + t)->v;
            }
            t += 32;
            while (t >= dh) {
                t -= dh;
                ++cls;
            }
        }
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            if (fast[i]) {
                const float s = bf16_to_f32((uint16_t)ev[i]);
#pragma unroll
                for (int w = 0; w < 4; ++w)
                    v[i][w] = pack_bf16(s * __uint_as_float(v[i][w] << 16), s * __uint_as_float(v[i][w] & 0xffff0000u));
            }
        }
        // pieces across a class boundary or among the bias columns, by a loop that is not unrolled: with the divisions of 64
        // columns in line the kernel had 194 registers and too few waves in flight (853 us for 256 rows of 1000 x 2049)
        bool all = true;
#pragma unroll
        for (int i = 0; i < NS; ++i) all = all && fast[i];
        if (!all) {
#pragma unroll 1
            for (int i = 0; i < NS; ++i) {
                bool todo = false;
#pragma unroll
                for (int q = 0; q < NS; ++q) todo = q == i ? !fast[q] : todo;
                if (!todo) continue;
                unsigned w[4] = {0u, 0u, 0u, 0u};
#pragma unroll 1
                for (int c = 0; c < 8; ++c) {  // (outer_value's are bf16 values already)
                    const unsigned x = __float_as_uint(outer_value(e, h, d0 + 32 * i + c, main, dh, D)) >> 16;
#pragma unroll
                    for (int q = 0; q < 4; ++q) w[q] |= (c >> 1) == q ? x << (16 * (c & 1)) : 0u;
                }
#pragma unroll
                for (int q = 0; q < NS; ++q)
                    if (q == i) v[q] = u32x4{w[0], w[1], w[2], w[3]};
            }
        }
    }
    template <int NS>
    __device__ __forceinline__ void load(int r, int64_t d0, int64_t D, float4 (&v)[NS]) const {
        const int64_t main = C * dh;
        const T* e = E + r * C;
        const T* h = H + r * dh;
        int64_t cls = d0 / dh, t = d0 - cls * dh;
        T ev[NS];
        Four<T> hv[NS];
        bool fast[NS];
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            fast[i] = cls < C && t + 3 < dh;
            if (fast[i]) {
                ev[i] = e[cls];
                hv[i] = *reinterpret_cast<const Four<T>*>(h + t);
            }
            t += DC;
            while (t >= dh) {
                t -= dh;
                ++cls;
            }
        }
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            float x[4];
            if (fast[i]) {
#pragma unroll
                for (int c = 0; c < 4; ++c) x[c] = value(ev[i], hv[i].v[c]);
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) x[c] = outer_value(e, h, d0 + i * DC + c, main, dh, D);
            }
            v[i] = make_float4(x[0], x[1], x[2], x[3]);
        }
    }
};

}  // namespace sage
