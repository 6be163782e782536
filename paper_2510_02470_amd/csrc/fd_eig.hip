// The eigensolve C = Y Lambda Y^T of the (padded) Gram matrix in fp64, and the coefficient matrices built from it.
//
// The shrink step (Method, FD paragraph) needs sigma_j^2 = lambda_j and, for the rebuild, the left singular
// vectors y_j of the buffer:  sigma_j v_j^T = y_j^T B. The solve is direct: Householder reduction to a tridiagonal
// matrix (fd_tridiag.hip), divide and conquer on that (fd_dc.hip), and the reflectors applied to the eigenvectors that
// are needed (the leading ell of a shrink, the leading k of a basis). It is backward stable: residual and loss of
// orthogonality are a few n * 2^-52, whatever the spectrum, and its work does not depend on the data.
#include "sage_internal.h"
#include "wave_ops.h"

namespace sage {

// Coefficients of the rebuild, row m < count of diag(f) Y^T (zero rows above), for MP output rows.
//   mode 0, shrink (delta = sigma_ell^2, Sigma'_jj = sqrt(max(sigma_j^2 - delta, 0))): f_m = sqrt(max(lambda_m - delta, 0) /
//           lambda_m), so that row m is sqrt(sigma_m^2 - delta) v_m^T. Also records the Gram matrix of the rows the
//           rebuild is about to write, diag(max(lambda_m - delta, 0)), in `known`: the next cycle takes that block as
//           known instead of recomputing it.
//   mode 1, basis: f_m = 1 / sqrt(lambda_m), or 0 when lambda_m <= n 2^-23 lambda_1.
//   mode 2, weighted basis: f_m = sqrt(max(lambda_m - delta, 0) / lambda_m) under the same rank test, which makes the row the
//           m-th of the sketch a shrink of the buffer would write ("Two-pass scoring": z = S g).
// One thread makes the 8 coefficients (stage, k-half h, row m) that a matrix-core lane of the rebuild takes per stage of 16
// buffer rows: buffer rows 16 * stage + 2 s + h, s < 8. SPLIT: as three bf16 parts in the order rebuild_split_kernel
// streams them; otherwise fp32 in coeff_offset order.
template <bool SPLIT>
__global__ __launch_bounds__(256) void coeffs_kernel(const double* __restrict__ Yt, const double* __restrict__ dv,
                                                     const double* __restrict__ C, double* __restrict__ stat, int NP, int MP,
                                                     int count, int mode, int n, int ell, int ra0, int ra1, int rb0, int rb1,
                                                     float* __restrict__ Mt, u32x4* __restrict__ Mc3,
                                                     double* __restrict__ acc, double* __restrict__ known,
                                                     int* __restrict__ failed) {
    const int ex = (int)stat[0];
    auto lam = [&](int m) {  // m-th largest eigenvalue, clamped at 0
        const double v = dv[NP - 1 - m];
        return v > 0.0 ? __builtin_amdgcn_ldexp(v, ex) : 0.0;
    };
    const double delta = lam(ell - 1);
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < (NP / 16) * 2 * MP) {
        const int m = i % MP, h = (i / MP) & 1, stg = i / (2 * MP);
        float v[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) v[s] = 0.f;
        if (m < count) {
            const double lm = lam(m), keep = lm - delta;
            double f = 0.0;
            if (mode == 0) {
                f = keep > 0.0 ? sqrt(keep / lm) : 0.0;
            } else if (lm > (double)n * 1.1920928955078125e-07 * lam(0)) {
                f = mode == 1 ? 1.0 / sqrt(lm) : (keep > 0.0 ? sqrt(keep / lm) : 0.0);
            }
            const double* y = Yt + (int64_t)m * NP + stg * 16 + h;
#pragma unroll
            for (int s = 0; s < 8; ++s) v[s] = f > 0.0 ? (float)(f * y[2 * s]) : 0.f;
        }
        if constexpr (SPLIT) {
            u32x4 hi, mid, lo;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                unsigned a, b, c;
                split3_bf16(v[2 * e], v[2 * e + 1], a, b, c);
                hi[e] = a;
                mid[e] = b;
                lo[e] = c;
            }
            u32x4* dst = Mc3 + (int64_t)stg * (3 * 2 * MP) + h * MP + m;
            dst[0] = hi;
            dst[2 * MP] = mid;
            dst[4 * MP] = lo;
        } else {
#pragma unroll
            for (int q = 0; q < 2; ++q)
                *reinterpret_cast<f32x4*>(Mt + coeff_offset(stg * 16 + h + 8 * q, m, MP)) =
                    f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
        }
    }
    if (mode == 0 && i < NP / 2) known[i] = i < ell ? fmax(lam(i) - delta, 0.0) : 0.0;
    if (blockIdx.x == 0 && threadIdx.x < 64) {
        // rows not yet counted in ||A||_F^2: their squared norms are on the diagonal of C
        double f = 0.0;
        for (int r = ra0 + (int)threadIdx.x; r < ra1; r += 64) f += C[(int64_t)r * NP + r];
        for (int r = rb0 + (int)threadIdx.x; r < rb1; r += 64) f += C[(int64_t)r * NP + r];
        f = lane_sum<64>(f);
        if (threadIdx.x == 0) {
            acc[1] += f;
            if (mode == 0) {
                acc[0] += delta;
                acc[2] = delta;
            }
            if (stat[1] != 0.0) {  // the reduction gave up waiting: the host refuses the context from its next call on
                acc[4] += 1.0;
                stat[1] = 0.0;
                *(volatile int*)failed = 1;
            }
        }
    }
}

hipError_t launch_eig(const EigWork& w, int NP, int m0, int n, int count, hipStream_t st) {
    if (hipError_t e = launch_tridiag(w, NP, m0, n, st); e != hipSuccess) return e;
    if (hipError_t e = launch_dc(w, NP, n, st); e != hipSuccess) return e;
    return launch_tri_back(w, NP, m0, n, count, st);
}

hipError_t launch_coeffs(const EigWork& w, int NP, int MP, int count, int mode, int n, int ell, int ra0, int ra1, int rb0,
                         int rb1, float* Mt, void* Mc3, double* acc, int* failed, hipStream_t st) {
    const dim3 grid((unsigned)(((NP / 16) * 2 * MP + 255) / 256));
    const double* dv = w.dI[dc_result(NP)];
    if (Mc3)
        hipLaunchKernelGGL(coeffs_kernel<true>, grid, dim3(256), 0, st, w.Yt, dv, w.C, w.stat, NP, MP, count, mode, n, ell, ra0,
                           ra1, rb0, rb1, Mt, (u32x4*)Mc3, acc, w.known, failed);
    else
        hipLaunchKernelGGL(coeffs_kernel<false>, grid, dim3(256), 0, st, w.Yt, dv, w.C, w.stat, NP, MP, count, mode, n, ell, ra0,
                           ra1, rb0, rb1, Mt, (u32x4*)nullptr, acc, w.known, failed);
    return hipGetLastError();
}

// For the stage probes: eigenvectors in columns (ascending eigenvalues), eigenvalues at their columns.
__global__ __launch_bounds__(256) void eig_export_kernel(const double* __restrict__ Yt, const double* __restrict__ dv,
                                                         const double* __restrict__ stat, double* __restrict__ Y,
                                                         double* __restrict__ lam, const double* __restrict__ C,
                                                         double* __restrict__ record, int NP) {
    const int r = blockIdx.x, ex = (int)stat[0];
    if (record && r == 0 && threadIdx.x < 64) {  // 18 entries: trace, then zeros
        double t = 0.0;
        for (int c = threadIdx.x; c < NP; c += 64) t += C[(int64_t)c * NP + c];
        t = lane_sum<64>(t);
        if (threadIdx.x < 18) record[threadIdx.x] = threadIdx.x == 0 ? t : 0.0;
    }
    for (int c = threadIdx.x; c < NP; c += 256) {
        if (Y) Y[(int64_t)r * NP + c] = Yt[(int64_t)(NP - 1 - c) * NP + r];
        if (lam && r == 0) lam[c] = __builtin_amdgcn_ldexp(dv[c], ex);
    }
}

hipError_t launch_eig_export(const EigWork& w, int NP, double* Y, double* lam, double* record, hipStream_t st) {
    hipLaunchKernelGGL(eig_export_kernel, dim3(NP), dim3(256), 0, st, w.Yt, w.dI[dc_result(NP)], w.stat, Y, lam, w.C, record,
                       NP);
    return hipGetLastError();
}

}  // namespace sage
