// The eigensolve C = Y Lambda Y^T of the (padded) Gram matrix in fp64.
//
// The shrink step (Method, FD paragraph) needs sigma_j^2 = lambda_j and, for the rebuild, the left singular
// vectors y_j of the buffer:  sigma_j v_j^T = y_j^T B. The solve is direct: Householder reduction to a tridiagonal
// matrix (fd_tridiag.hip), divide and conquer on that (fd_dc.hip), and the reflectors applied to the eigenvectors that
// are needed (the leading ell of a shrink, the leading k of a basis), which become the rebuild's coefficients on the way. It is backward stable: residual and loss of
// orthogonality are a few n * 2^-52, whatever the spectrum, and its work does not depend on the data.
#include "sage_internal.h"
#include "wave_ops.h"

namespace sage {

hipError_t launch_eig(const EigWork& w, int NP, int m0, int n, int count, const CoeffArgs* cf, hipStream_t st, const RowJob* job) {
    if (hipError_t e = launch_tridiag(w, NP, m0, n, st, job); e != hipSuccess) return e;
    if (hipError_t e = launch_dc(w, NP, n, st); e != hipSuccess) return e;
    return launch_tri_back(w, NP, m0, n, count, cf, st);
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
