// First and last stage of the symmetric eigensolve C = Y Lambda Y^T of the Gram matrix (Method, FD paragraph: the SVD
// of the buffer): Householder reduction C = H T H^T to a tridiagonal T, and Y = H Z from the eigenvectors Z of T
// (fd_dc.hip). All in fp64.
//
// The reduction is a chain of n - 1 dependent steps (a matrix-vector product with the trailing matrix and a rank-2
// update of it, 2 flop per byte touched), so it is bound by the latency of a step, not by arithmetic. The matrix
// therefore never leaves the registers: the work-groups own columns of the (symmetric) matrix, a wave's lanes the rows
// lane, lane + 64, ..., and the rank-2 update of a step is applied in the same pass as the next step's product.
//   n = 64, 128:  one work-group of 4 waves; the only exchange of a step goes through LDS (tri_one_kernel).
//   n = 256, 512: n / 16 work-groups of 4 waves, one per CU of ONE XCD, which exchange two n-vectors per step through
//                 the L2 they share (tri_many_kernel).
// Every wave carries the vectors of the step (column, reflector, product) redundantly, so a step has one exchange and
// no other synchronisation.
#include "sage_internal.h"
#include "wave_ops.h"

namespace sage {

// Matrix index of active index i: the buffer's rows in use are 0 .. m0-1 (top half) and LP .. (new half).
__device__ __forceinline__ int active_index(int i, int m0, int LP) { return i < m0 ? i : LP + (i - m0); }

// 2^-e with 2^e >= max diag(C): the reduction and the eigensolve of T work on C * 2^-e (exact).
__device__ __forceinline__ int tri_exponent(double maxdiag) {
    return (maxdiag > 1e-280 && maxdiag < 1e280) ? __builtin_amdgcn_frexp_exp(maxdiag) : 0;
}
// max |diag(C)| over the padded matrix, by every wave
__device__ __forceinline__ double wave_max_diag(const double* __restrict__ C, int NP, int lane) {
    double m = 0.0;
    for (int i = lane; i < NP; i += 64) m = fmax(m, fabs(C[(int64_t)i * NP + i]));
    for (int o = 32; o >= 1; o >>= 1) m = fmax(m, __shfl_xor(m, o));
    return m;
}

// The Householder vector of a column: x = (alpha; rest), rest2 = |rest|^2. H x = beta e_1, H = I - tau v v^T,
// v = (1; scale * rest). A rest below 1e-30 of the matrix counts as zero (H = I, tau = 0): smaller ones, which a matrix of
// low rank leaves, would lose their digits to underflow in |rest|^2 and H its orthogonality.
constexpr double TRI_DROP2 = 1e-60;
__device__ __forceinline__ void householder(double alpha, double rest2, double& beta, double& tau, double& scale) {
    if (rest2 > TRI_DROP2) {
        const double nrm = __builtin_sqrt(__builtin_fma(alpha, alpha, rest2));
        beta = alpha >= 0.0 ? -nrm : nrm;
        tau = (beta - alpha) * rcp64(beta);
        scale = rcp64(alpha - beta);
    } else {
        beta = alpha;
        tau = 0.0;
        scale = 0.0;
    }
}

// ---- n = 64 J, J = 1, 2: one work-group ---------------------------------------------------------------------------
// Wave w owns the columns of the 8-column blocks w, w + 4, ... Step k (column k known to every wave as x):
// reflector v; own columns j > k: a_j -= v' w'_j + w' v'_j (primes: step k - 1), partial product sum_j a_j v_j; the
// owner of column k + 1 publishes it; one barrier; p = tau sum of the partials, w = p + alpha v, and
// x <- column k + 1 - v w_{k+1} - w v_{k+1} is the next column.
template <int J>
__global__ __launch_bounds__(256, 1) void tri_one_kernel(const double* __restrict__ C, int NP, int m0, int LP, int n,
                                                         double* __restrict__ dT, double* __restrict__ eT,
                                                         double* __restrict__ tauT, double* __restrict__ V,
                                                         double* __restrict__ stat) {
    constexpr int N = 64 * J, W = 4, NB = N / (8 * W);  // NB blocks of 8 columns per wave
    __shared__ double pbuf[2][W][N];                    // partial products
    __shared__ double cbuf[2][N];                       // next column
    __shared__ __attribute__((aligned(16))) double vs[W][2][N];  // each wave's own copies of v and w, by parity
    __shared__ __attribute__((aligned(16))) double ws[W][2][N];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    const double md = wave_max_diag(C, NP, lane);
    const int ex = tri_exponent(md);
    const double sc0 = __builtin_amdgcn_ldexp(1.0, -ex);
    if (tid == 0) stat[0] = (double)ex;

    double a[NB][8][J];
    int mrow[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int r = lane + 64 * j;
        mrow[j] = r < n ? active_index(r, m0, LP) : -1;
    }
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int col = 8 * (wave + W * b) + q;
            const double* src = C + (int64_t)active_index(col < n ? col : 0, m0, LP) * NP;
#pragma unroll
            for (int j = 0; j < J; ++j) a[b][q][j] = (col < n && mrow[j] >= 0) ? src[mrow[j]] * sc0 : 0.0;
        }
    double x[J], v[J], w[J];
    {
        const double* src = C + (int64_t)active_index(0, m0, LP) * NP;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            x[j] = mrow[j] >= 0 ? src[mrow[j]] * sc0 : 0.0;
            v[j] = 0.0;
            w[j] = 0.0;
        }
    }
    double xk = C[(int64_t)active_index(0, m0, LP) * NP + active_index(0, m0, LP)] * sc0;
    double xk1 = n > 1 ? C[(int64_t)active_index(0, m0, LP) * NP + active_index(1, m0, LP)] * sc0 : 0.0;

    for (int k = 0; k < n - 1; ++k) {
        const int par = k & 1;
        double r2 = 0.0;
#pragma unroll
        for (int j = 0; j < J; ++j) r2 = __builtin_fma(lane + 64 * j > k + 1 ? x[j] : 0.0, x[j], r2);
        r2 = lane_sum<64>(r2);
        double beta, tau, scale;
        householder(xk1, r2, beta, tau, scale);
        const double v1 = r2 > TRI_DROP2 ? 1.0 : 0.0;
        double vn[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int r = lane + 64 * j;
            vn[j] = r > k + 1 ? x[j] * scale : (r == k + 1 ? v1 : 0.0);
            vs[wave][par][r] = vn[j];
        }
        if (tid == 0) {
            dT[k] = xk;
            eT[k] = beta;
            tauT[k] = tau;
        }
        if (wave == (k & 3)) {
#pragma unroll
            for (int j = 0; j < J; ++j) V[(int64_t)k * N + lane + 64 * j] = vn[j];
        }
        asm volatile("" ::: "memory");
        double acc[J];
#pragma unroll
        for (int j = 0; j < J; ++j) acc[j] = 0.0;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int c0 = 8 * (wave + W * b);
            if (c0 + 7 > k && c0 < n) {
                double vj[8], vp[8], wp[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    vj[q] = vs[wave][par][c0 + q];
                    vp[q] = k > 0 ? vs[wave][par ^ 1][c0 + q] : 0.0;
                    wp[q] = k > 0 ? ws[wave][par ^ 1][c0 + q] : 0.0;
                }
#pragma unroll
                for (int q = 0; q < 8; ++q)
#pragma unroll
                    for (int j = 0; j < J; ++j) {
                        a[b][q][j] = __builtin_fma(-v[j], wp[q], __builtin_fma(-w[j], vp[q], a[b][q][j]));
                        acc[j] = __builtin_fma(a[b][q][j], vj[q], acc[j]);
                    }
                if (k + 1 >= c0 && k + 1 < c0 + 8) {
#pragma unroll
                    for (int q = 0; q < 8; ++q)
                        if (c0 + q == k + 1) {
#pragma unroll
                            for (int j = 0; j < J; ++j) cbuf[par][lane + 64 * j] = a[b][q][j];
                        }
                }
            }
        }
#pragma unroll
        for (int j = 0; j < J; ++j) pbuf[par][wave][lane + 64 * j] = acc[j];
        __syncthreads();
        double p[J], c[J];
        double dot = 0.0;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int r = lane + 64 * j;
            p[j] = tau * ((pbuf[par][0][r] + pbuf[par][1][r]) + (pbuf[par][2][r] + pbuf[par][3][r]));
            c[j] = cbuf[par][r];
            if (r <= k) p[j] = 0.0;
            dot = __builtin_fma(p[j], vn[j], dot);
        }
        const int r2i = k + 2 < n ? k + 2 : k + 1;
        const double p1 = tau * ((pbuf[par][0][k + 1] + pbuf[par][1][k + 1]) + (pbuf[par][2][k + 1] + pbuf[par][3][k + 1]));
        const double p2 = tau * ((pbuf[par][0][r2i] + pbuf[par][1][r2i]) + (pbuf[par][2][r2i] + pbuf[par][3][r2i]));
        const double c1 = cbuf[par][k + 1], c2 = cbuf[par][r2i], v2 = vs[wave][par][r2i];
        dot = lane_sum<64>(dot);
        const double al = -0.5 * tau * dot;
        const double w1 = __builtin_fma(al, v1, p1), w2 = __builtin_fma(al, v2, p2);
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int r = lane + 64 * j;
            v[j] = vn[j];
            w[j] = __builtin_fma(al, vn[j], p[j]);
            ws[wave][par][r] = w[j];
            x[j] = __builtin_fma(-v[j], w1, __builtin_fma(-w[j], v1, c[j]));
        }
        xk = __builtin_fma(-2.0 * v1, w1, c1);
        xk1 = __builtin_fma(-v2, w1, __builtin_fma(-w2, v1, c2));
    }
    if (tid == 0) {
        dT[n - 1] = xk;
        eT[n - 1] = 0.0;
        tauT[n - 1] = 0.0;
    }
    // the padding: decoupled, below every eigenvalue of a Gram matrix
    for (int i = n + tid; i < N; i += 256) {
        dT[i] = -1.0;
        eT[i] = 0.0;
        tauT[i] = 0.0;
    }
}

// ---- n = 64 J, J = 4, 8: n / 16 work-groups on one XCD ------------------------------------------------------------
// Exchange buffers: [3][2][N] doubles (ring slot, product p / next column c), every entry the EMPTY pattern before the
// launch. An entry is published by a relaxed agent-scope store and picked up by spinning on it with relaxed agent-scope
// loads until it is not EMPTY: no flags, no fences, an entry carries its own validity. Ring slot k % 3 serves step k.
// Once a work-group has all of step k it knows that everyone has finished reading step k - 1, so it sets its own
// entries of slot (k + 2) % 3 = (k - 1) % 3 back to EMPTY, waits for those stores before it publishes step k + 1, and
// nobody reads that slot before having all of step k + 1.
// A spin ends after SPIN_LIMIT polls (seconds; the partners are resident or about to be, whatever else the GPU runs
// ends by itself): the kernel then gives up, reports in stat[1], and every further wait returns at once.
constexpr long long EMPTY = -1LL;  // a NaN no arithmetic produces (published NaNs are replaced by the default one)
constexpr int SPIN_LIMIT = 1 << 23;

__device__ __forceinline__ void put(long long* p, double v) {
    long long u = __double_as_longlong(v);
    if (v != v) u = 0x7FF8000000000000LL;
    __hip_atomic_store(p, u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ long long get(const long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void wait_stores() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

template <int J>
__global__ __launch_bounds__(256, 1) void tri_many_kernel(const double* __restrict__ C, int NP, int m0, int LP, int n,
                                                          double* __restrict__ dT, double* __restrict__ eT,
                                                          double* __restrict__ tauT, double* __restrict__ V,
                                                          double* __restrict__ stat, long long* __restrict__ xch,
                                                          int xcd) {
    constexpr int N = 64 * J, NW = N / 4;  // NW waves in all, 4 columns each: gw, gw + NW, gw + 2 NW, gw + 3 NW
    constexpr int PT = N / 256;            // entries per thread and vector of the exchange
    if ((int)(blockIdx.x & 7) != xcd) return;  // consecutive work-groups go to consecutive XCDs
    __builtin_amdgcn_s_setprio(3);
    __shared__ double pb[2][N], cb[2][N];
    __shared__ double vs[4][N];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wg = blockIdx.x >> 3;
    const int gw = wg * 4 + wave;

    const double md = wave_max_diag(C, NP, lane);
    const int ex = tri_exponent(md);
    const double sc0 = __builtin_amdgcn_ldexp(1.0, -ex);
    if (wg == 0 && tid == 0) stat[0] = (double)ex;

    double a[4][J], x[J], v[J], w[J];
    double vcol[4], wcol[4];
    {
        int mrow[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int r = lane + 64 * j;
            mrow[j] = r < n ? active_index(r, m0, LP) : -1;
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int col = gw + NW * s;
            const double* src = C + (int64_t)active_index(col < n ? col : 0, m0, LP) * NP;
#pragma unroll
            for (int j = 0; j < J; ++j) a[s][j] = (col < n && mrow[j] >= 0) ? src[mrow[j]] * sc0 : 0.0;
            vcol[s] = 0.0;
            wcol[s] = 0.0;
        }
        const double* src = C + (int64_t)active_index(0, m0, LP) * NP;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            x[j] = mrow[j] >= 0 ? src[mrow[j]] * sc0 : 0.0;
            v[j] = 0.0;
            w[j] = 0.0;
        }
    }
    double xk = C[(int64_t)active_index(0, m0, LP) * NP + active_index(0, m0, LP)] * sc0;
    double xk1 = n > 1 ? C[(int64_t)active_index(0, m0, LP) * NP + active_index(1, m0, LP)] * sc0 : 0.0;
    int spins = SPIN_LIMIT;
    int slot = 0;

    for (int k = 0; k < n - 1; ++k) {
        const int par = k & 1;
        long long* const px = xch + (int64_t)slot * 2 * N;
        long long* const cx = px + N;
        double r2 = 0.0;
#pragma unroll
        for (int j = 0; j < J; ++j) r2 = __builtin_fma(lane + 64 * j > k + 1 ? x[j] : 0.0, x[j], r2);
        r2 = lane_sum<64>(r2);
        double beta, tau, scale;
        householder(xk1, r2, beta, tau, scale);
        const double v1 = r2 > TRI_DROP2 ? 1.0 : 0.0;
        double vn[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int r = lane + 64 * j;
            vn[j] = r > k + 1 ? x[j] * scale : (r == k + 1 ? v1 : 0.0);
            vs[wave][r] = vn[j];
        }
        wait_stores();  // last step's resets (long done)
        double acc[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            acc[s] = 0.0;
            const int col = gw + NW * s;
            if (col > k && col < n) {
#pragma unroll
                for (int j = 0; j < J; ++j)
                    if (64 * j + 63 > k) {
                        a[s][j] = __builtin_fma(-v[j], wcol[s], __builtin_fma(-w[j], vcol[s], a[s][j]));
                        acc[s] = __builtin_fma(a[s][j], vn[j], acc[s]);
                    }
                if (col == k + 1) {
#pragma unroll
                    for (int j = 0; j < J; ++j)
                        if (64 * j + 63 > k && lane + 64 * j > k && lane + 64 * j < n) put(cx + lane + 64 * j, a[s][j]);
                }
            }
        }
        // the four sums over the wave, two at a time per lane pair, then one per lane of a quad
        {
            const bool odd = lane & 1, hi = lane & 2;
            double t0 = odd ? acc[1] : acc[0], o0 = odd ? acc[0] : acc[1];
            double t1 = odd ? acc[3] : acc[2], o1 = odd ? acc[2] : acc[3];
            t0 += dpp_move<DPP_XOR1>(o0);   // lane parity q: column q
            t1 += dpp_move<DPP_XOR1>(o1);   // ... column 2 + q
            double t = hi ? t1 : t0, o = hi ? t0 : t1;
            t += dpp_move<DPP_XOR2>(o);     // lane & 3 = column; sums over quads so far
            t += dpp_move<0x124>(t);        // row_ror 4
            t += dpp_move<0x128>(t);        // row_ror 8: sums over rows of 16
            t += __shfl_xor(t, 16);
            t += __shfl_xor(t, 32);
            const int col = gw + NW * (lane & 3);
            if (lane < 4 && col > k && col < n) put(px + col, tau * t);
        }
        if (wg == (k & (N / 16 - 1))) {
            if (wave == 0) {
#pragma unroll
                for (int j = 0; j < J; ++j) V[(int64_t)k * N + lane + 64 * j] = vn[j];
            }
            if (tid == 64) {
                dT[k] = xk;
                eT[k] = beta;
                tauT[k] = tau;
            }
        }
        // pick up this thread's entries
        {
            long long up[PT], uc[PT];
            bool need[PT];
#pragma unroll
            for (int q = 0; q < PT; ++q) {
                const int i = tid + 256 * q;
                need[q] = i > k && i < n;
                up[q] = need[q] ? EMPTY : 0;
                uc[q] = need[q] ? EMPTY : 0;
            }
            bool more = true;
            while (more) {
#pragma unroll
                for (int q = 0; q < PT; ++q) {
                    if (need[q]) {
                        up[q] = get(px + tid + 256 * q);
                        uc[q] = get(cx + tid + 256 * q);
                    }
                }
                more = false;
#pragma unroll
                for (int q = 0; q < PT; ++q) more = more || up[q] == EMPTY || uc[q] == EMPTY;
                if (more && --spins <= 0) {
                    if (spins == 0) stat[1] = 1.0;
                    spins = -1000000;
                    more = false;
                }
            }
#pragma unroll
            for (int q = 0; q < PT; ++q) {
                pb[par][tid + 256 * q] = __longlong_as_double(up[q]);
                cb[par][tid + 256 * q] = __longlong_as_double(uc[q]);
            }
        }
        __syncthreads();
        {   // free the slot of step k - 1 for step k + 2
            const int old = slot == 0 ? 2 : slot - 1;
            const int col = gw + NW * (lane & 3);
            if (lane < 8 && col < n) {
                long long* const e = xch + (int64_t)old * 2 * N + (lane >> 2) * N + col;
                __hip_atomic_store(e, EMPTY, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        double p[J], c[J];
        double dot = 0.0;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            p[j] = pb[par][lane + 64 * j];
            c[j] = cb[par][lane + 64 * j];
            dot = __builtin_fma(p[j], vn[j], dot);
        }
        const int i2 = k + 2 < n ? k + 2 : k + 1;
        const double p1 = pb[par][k + 1], p2 = pb[par][i2], c1 = cb[par][k + 1], c2 = cb[par][i2], v2 = vs[wave][i2];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            vcol[s] = vs[wave][gw + NW * s];
            wcol[s] = pb[par][gw + NW * s];
        }
        dot = lane_sum<64>(dot);
        const double al = -0.5 * tau * dot;
        const double w1 = __builtin_fma(al, v1, p1), w2 = __builtin_fma(al, v2, p2);
#pragma unroll
        for (int s = 0; s < 4; ++s) wcol[s] = __builtin_fma(al, vcol[s], wcol[s]);
#pragma unroll
        for (int j = 0; j < J; ++j) {
            v[j] = vn[j];
            w[j] = __builtin_fma(al, vn[j], p[j]);
            x[j] = __builtin_fma(-v[j], w1, __builtin_fma(-w[j], v1, c[j]));
        }
        xk = __builtin_fma(-2.0 * v1, w1, c1);
        xk1 = __builtin_fma(-v2, w1, __builtin_fma(-w2, v1, c2));
        slot = slot == 2 ? 0 : slot + 1;
    }
    if (wg == 0 && tid == 0) {
        dT[n - 1] = xk;
        eT[n - 1] = 0.0;
        tauT[n - 1] = 0.0;
    }
    if (wg == 0)
        for (int i = n + tid; i < N; i += 256) {
            dT[i] = -1.0;
            eT[i] = 0.0;
            tauT[i] = 0.0;
        }
}

// ---- Y = H Z --------------------------------------------------------------------------------------------------------
// One wave per eigenvector: the vector in registers (rows lane, lane + 64, ...), the reflectors n - 3 .. 0 applied one
// after the other (they stream through L2 / L1; four requested ahead). Column `col` of Z (column-major, ascending
// eigenvalues) becomes row N - 1 - col of Yt (descending), in matrix indices; padding indices are zero.
template <int J>
__global__ __launch_bounds__(64) void tri_back_kernel(const double* __restrict__ Z, const double* __restrict__ V,
                                                      const double* __restrict__ tauT, int m0, int LP, int n,
                                                      double* __restrict__ Yt, int NP) {
    constexpr int N = 64 * J;
    const int lane = threadIdx.x;
    const int rank = blockIdx.x, col = N - 1 - rank;
    double z[J];
#pragma unroll
    for (int j = 0; j < J; ++j) z[j] = Z[(int64_t)col * N + lane + 64 * j];
    // pairs of reflectors: (I - t1 v1 v1^T)(I - t2 v2 v2^T) z with both products formed at once
    double va[2][J], vb[2][J];
    int k = n - 3;
    auto load = [&](int kk, double (&u)[J]) {
#pragma unroll
        for (int j = 0; j < J; ++j) u[j] = (kk >= 0 && 64 * j + 63 > kk) ? V[(int64_t)kk * N + lane + 64 * j] : 0.0;
    };
    load(k, vb[0]);
    load(k - 1, va[0]);
    load(k - 2, vb[1]);
    load(k - 3, va[1]);
    auto pair = [&](double (&ua)[J], double (&ub)[J], int kk) {  // reflectors kk (ub), then kk - 1 (ua)
        const double ta = kk >= 1 ? tauT[kk - 1] : 0.0, tb = tauT[kk];
        double sa = 0.0, sb = 0.0, sab = 0.0;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            sb = __builtin_fma(ub[j], z[j], sb);
            sa = __builtin_fma(ua[j], z[j], sa);
            sab = __builtin_fma(ua[j], ub[j], sab);
        }
        sb = lane_sum<64>(sb);
        sa = lane_sum<64>(sa);
        sab = lane_sum<64>(sab);
        const double fb = tb * sb, fa = ta * (sa - fb * sab);
#pragma unroll
        for (int j = 0; j < J; ++j) z[j] = __builtin_fma(-fa, ua[j], __builtin_fma(-fb, ub[j], z[j]));
        load(kk - 4, ub);
        load(kk - 5, ua);
    };
    for (; k >= 0; k -= 4) {
        pair(va[0], vb[0], k);
        if (k - 2 >= 0) pair(va[1], vb[1], k - 2);
    }
    // Padding indices (matrix indices outside the active ones): a padding eigenvector is its own unit vector.
    double* out = Yt + (int64_t)rank * NP;
    const int gap = LP - m0;  // padding indices m0 .. LP-1 come first
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int r = lane + 64 * j, q = r - n;
        out[r < n ? active_index(r, m0, LP) : (q < gap ? m0 + q : n - m0 + LP + q - gap)] = z[j];
    }
}

hipError_t launch_tridiag(const EigWork& w, int NP, int m0, int n, hipStream_t st) {
    const int LP = NP / 2;
    switch (NP / 64) {
        case 1:
            hipLaunchKernelGGL(tri_one_kernel<1>, dim3(1), dim3(256), 0, st, w.C, NP, m0, LP, n, w.dT, w.eT, w.tauT, w.V, w.stat);
            break;
        case 2:
            hipLaunchKernelGGL(tri_one_kernel<2>, dim3(1), dim3(256), 0, st, w.C, NP, m0, LP, n, w.dT, w.eT, w.tauT, w.V, w.stat);
            break;
        case 4:
            hipLaunchKernelGGL(tri_many_kernel<4>, dim3(8 * 16), dim3(256), 0, st, w.C, NP, m0, LP, n, w.dT, w.eT, w.tauT,
                               w.V, w.stat, w.xch, w.xcd);
            break;
        case 8:
            hipLaunchKernelGGL(tri_many_kernel<8>, dim3(8 * 32), dim3(256), 0, st, w.C, NP, m0, LP, n, w.dT, w.eT, w.tauT,
                               w.V, w.stat, w.xch, w.xcd);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_tri_back(const EigWork& w, int NP, int m0, int n, int count, hipStream_t st) {
    const int LP = NP / 2;
#define SAGE_BACK(J)                                                                                              \
    hipLaunchKernelGGL(tri_back_kernel<J>, dim3(count), dim3(64), 0, st, w.Z[dc_result(NP)], w.V, w.tauT, m0, LP, n, w.Yt, NP)
    switch (NP / 64) {
        case 1: SAGE_BACK(1); break;
        case 2: SAGE_BACK(2); break;
        case 4: SAGE_BACK(4); break;
        case 8: SAGE_BACK(8); break;
        default: return hipErrorInvalidValue;
    }
#undef SAGE_BACK
    return hipGetLastError();
}

}  // namespace sage
