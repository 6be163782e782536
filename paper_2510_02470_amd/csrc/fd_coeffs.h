// Coefficients of a rebuild in the orders its kernels stream them (fd_rebuild.hip).
#pragma once
#include "sage_internal.h"

namespace sage {

struct Coeffs8 {
    float c[8];
};
// The 8 coefficients (stage, k-half h, row m) that a matrix-core lane of the rebuild takes per stage of 16 buffer rows: buffer rows
// 16 * stage + 2 s + h, s < 8. SPLIT: as three bf16 parts in the order rebuild_split_kernel streams them; otherwise in
// coeff_offset order.
template <bool SPLIT>
__device__ __forceinline__ void store_coeffs(float* __restrict__ Mt, void* __restrict__ Mc3, int MP, int stg, int h, int m,
                                             const Coeffs8& v) {
    if constexpr (SPLIT) {
        u32x4 hi, mid, lo;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            unsigned a, b, c;
            split3_bf16(v.c[2 * e], v.c[2 * e + 1], a, b, c);
            hi[e] = a;
            mid[e] = b;
            lo[e] = c;
        }
        u32x4* dst = (u32x4*)Mc3 + (int64_t)stg * (3 * 2 * MP) + h * MP + m;
        dst[0] = hi;
        dst[2 * MP] = mid;
        dst[4 * MP] = lo;
    } else {
#pragma unroll
        for (int q = 0; q < 2; ++q)
            *reinterpret_cast<f32x4*>(Mt + coeff_offset(stg * 16 + h + 8 * q, m, MP)) =
                f32x4{v.c[4 * q], v.c[4 * q + 1], v.c[4 * q + 2], v.c[4 * q + 3]};
    }
}

}  // namespace sage
