// First and last stage of the symmetric eigensolve C = Y Lambda Y^T of the Gram matrix (Method, FD paragraph: the SVD
// of the buffer): Householder reduction C = H T H^T to a tridiagonal T, and Y = H Z from the eigenvectors Z of T
// (fd_dc.hip). All in fp64.
//
// The reduction is a chain of n - 1 dependent steps (a matrix-vector product with the trailing matrix and a rank-2
// update of it, 2 flop per byte touched), so it is bound by the latency of a step, not by arithmetic. The matrix
// therefore never leaves the registers: the work-groups own columns of the (symmetric) matrix, a wave's lanes the rows
// lane, lane + 64, ..., and the rank-2 update of a step is applied in the same pass as the next step's product.
//   n = 64:            one work-group; the exchanges of a step go through LDS (tri_one_kernel, 0.44 us a step).
//   n = 128, 256, 512: 16, 32, 32 work-groups, one per CU of ONE XCD, which exchange two n-vectors per step through the L2
//                      they share (tri_many_kernel, 0.77, 0.83, 1.02 us a step; every wave carries the vectors of the
//                      step redundantly, so a step has one exchange and no other synchronisation), until 64 rows are left;
//                      one of them goes on with those as if there were no others (n = 128: 98 -> 85 us, 256: 206 -> 205 to
//                      212, 512: 585 -> 545, the latter two beside the side stream's work).
// One work-group takes 92 us for the whole of 128 rows, which is what is done where work-groups cannot be placed on one XCD (XcdMap
// without a period); larger ones are then done as after a wait in vain (see tri_many_kernel).
#include <mutex>
#include <type_traits>

#include "sage_internal.h"
#include "fd_coeffs.h"
#include "fd_rows.h"
#include "fd_tri_plan.h"
#include "fd_wy.h"
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

// The reflector of a column (alpha; rest), rest2 = |rest|^2: H = I - tau v v^T, v = (v1; rest) takes it to (beta; 0). The
// vector is not normalised: the matrix-vector product of a step can then start from the column itself, while the norm
// is still being formed. A rest below 1e-30 of the matrix counts as zero (H = I): smaller ones, which a matrix of low
// rank leaves, would lose their digits to underflow in |rest|^2 and H its orthogonality.
constexpr double TRI_DROP2 = 1e-60;
__device__ __forceinline__ void householder(double alpha, double rest2, double& beta, double& tau, double& v1) {
    if (rest2 > TRI_DROP2) {
        const double s = __builtin_fma(alpha, alpha, rest2);
        double y = __builtin_amdgcn_rsq(s);
        y = __builtin_fma(y * 0.5, __builtin_fma(-s * y, y, 1.0), y);
        y = __builtin_fma(y * 0.5, __builtin_fma(-s * y, y, 1.0), y);
        double nrm = s * y;
        nrm = __builtin_fma(__builtin_fma(-nrm, nrm, s), 0.5 * y, nrm);
        const double m = fabs(alpha) + nrm;
        beta = alpha >= 0.0 ? -nrm : nrm;
        v1 = alpha >= 0.0 ? m : -m;
        tau = rcp64(nrm * m);
    } else {
        beta = alpha;
        tau = 0.0;
        v1 = 0.0;
    }
}
typedef double f64x2 __attribute__((ext_vector_type(2)));

// Loads before it are made where they stand: the compiler would move each to the place where its value is known to be wanted, behind
// a branch and with a wait of its own (16 elements of a matrix: 5 us).
__device__ __forceinline__ void loads_go_out() { asm volatile("" ::: "memory"); }

// Orders this wave's LDS traffic before the barrier and nothing else: __syncthreads() would also wait for the global
// stores in flight.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The reduction by one work-group of T threads, with the matrix in V (its rows become the reflectors) and the vectors of a step
// in LDS: every step reads and writes the trailing matrix once, through the L2. For solves that several work-groups could not
// do together: 0.5, 2.2 and 12.8 ms at 128, 256 and 512 rows, where they take 0.085, 0.21 and 0.55. vec: 4 N words.
template <int J, int T>
__device__ __forceinline__ void tri_alone(const double* __restrict__ C, int NP, int m0, int LP, int n, double* __restrict__ dT,
                                          double* __restrict__ eT, double* __restrict__ tauT, double* V, double sc0,
                                          double* vec) {
    constexpr int N = 64 * J;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int i = wave; i < n; i += T / 64)
        for (int j = lane; j < N; j += 64)
            V[(int64_t)i * N + j] = j < n ? C[(int64_t)active_index(i, m0, LP) * NP + active_index(j, m0, LP)] * sc0 : 0.0;
    for (int j = tid; j < 4 * N; j += T) vec[j] = 0.0;
    __syncthreads();
    for (int k = 0; k < n; ++k) {
        const double *v0 = vec + ((k + 1) & 1) * N, *w0 = v0 + 2 * N;  // of step k - 1 (v' and w' above)
        double *v = vec + (k & 1) * N, *w = v + 2 * N;
        // column k below the diagonal, with the update of step k - 1
        for (int j = tid; j < N; j += T) {
            const double a = V[(int64_t)k * N + j];
            const double x = __builtin_fma(-v0[j], w0[k], __builtin_fma(-w0[j], v0[k], a));
            v[j] = j > k && j < n ? x : 0.0;
            w[j] = 0.0;
            if (j == k) dT[k] = x;
        }
        __syncthreads();
        if (k == n - 1) break;
        double r2 = 0.0;
        for (int j = lane; j < n; j += 64) r2 = j > k + 1 ? __builtin_fma(v[j], v[j], r2) : r2;
        r2 = lane_sum<64>(r2);
        double beta, tau, v1;
        householder(v[k + 1], r2, beta, tau, v1);
        __syncthreads();
        for (int j = tid; j < N; j += T) {
            const double x = j == k + 1 ? v1 : v[j];
            if (j == k + 1) v[j] = x;
            V[(int64_t)k * N + j] = x;
        }
        if (tid == 0) {
            eT[k] = beta;
            tauT[k] = tau;
        }
        __syncthreads();
        const int c0 = (k + 1) & ~63;  // columns below are done with
        // (four rows of a wave at a time, for their loads to be in flight together)
        for (int i0 = k + 1 + wave; i0 < n; i0 += 4 * (T / 64)) {
            double vi[4], wi[4], s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = i0 + u * (T / 64);
                vi[u] = i < n ? v0[i] : 0.0;
                wi[u] = i < n ? w0[i] : 0.0;
            }
            for (int j = c0 + lane; j < n; j += 64) {
                const double vj = v0[j], wj = w0[j], xj = v[j];
                double a[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = i0 + u * (T / 64);
                    a[u] = i < n ? V[(int64_t)i * N + j] : 0.0;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = i0 + u * (T / 64);
                    a[u] = __builtin_fma(-vj, wi[u], __builtin_fma(-wj, vi[u], a[u]));
                    if (i < n) V[(int64_t)i * N + j] = a[u];
                    s[u] = __builtin_fma(a[u], xj, s[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = i0 + u * (T / 64);
                s[u] = lane_sum<64>(s[u]);
                if (lane == 0 && i < n) w[i] = tau * s[u];
            }
        }
        __syncthreads();
        double dot = 0.0;
        for (int j = lane; j < n; j += 64) dot = __builtin_fma(w[j], v[j], dot);
        dot = lane_sum<64>(dot);
        const double al = -0.5 * tau * dot;
        __syncthreads();
        for (int j = tid; j < N; j += T) w[j] = __builtin_fma(al, v[j], w[j]);
        __syncthreads();
    }
}

// What follows the last row in use of a reduction's results, by threads 0 .. step - 1. The rows of V that complete the last block of reflectors are zero; the
// padding of T is decoupled and below every eigenvalue of a Gram matrix.
template <int J>
__device__ __forceinline__ void tri_finish(int n, double* __restrict__ dT, double* __restrict__ eT, double* __restrict__ tauT,
                                           double* __restrict__ V, int tid, int step) {
    constexpr int N = 64 * J;
    for (int i = n - 1 + tid; i < N; i += step) {
        if (i >= n) dT[i] = -1.0;
        eT[i] = 0.0;
        tauT[i] = 0.0;
    }
    for (int k = n - 1; k % WY != 0; ++k)
        for (int i = tid; i < N; i += step) V[(int64_t)k * N + i] = 0.0;
}

// ---- n = 64 J, J = 1, 2: one work-group ---------------------------------------------------------------------------
// Waves 0 .. W - 1 hold the matrix, wave I its rows 16 I .. 16 I + 15: lane 16 g + r row 16 I + r of the columns 16 (g + 4 u) .. + 15, u < J.
// So the 16 lanes of a row of the register file hold, at their own places 16 g + r + 64 u, the 16 entries of a vector that go with
// its columns, and v_fmac_f64 with row_newbcast:c takes entry c for column c: the update and the product of a step are three
// instructions per element, without a broadcast and without sums over lanes but for the four groups g. Wave W forms the
// reflectors, wave W + 1 stores the results; all carry the vectors, each its own copy, so that a step has one barrier. Step k,
// with x = column k below row k + 1 and w' of step k - 1:
//   waves 0 .. W - 1: a -= v' w'^T + w' v'^T, q = a x, c = column k + 1, their part of x A x;
//   wave W meanwhile: the reflector (tau, v1) from |x|;                                                      barrier
//   all: v A v = x A x + 2 v1 q_{k+1} + v1^2 c_{k+1}, w = tau (q + v1 c) - tau^2/2 (v A v) v, next column c - v w_{k+1} - w v1.
// A step is a chain of latencies (LDS round trip 110 cycles, sum over a wave 120) and of instructions of four cycles each, dependent
// or not: 1,000 cycles where a SIMD has one of the waves, 2,050 where it has two (n = 128, first half: half the rows to a wave more, on
// four waves, took 2,430). Steps come in sixteens, written out, so that column k + 1 is a register; those beyond the last row change
// nothing. A wave whose rows are finished only keeps the barriers.
struct __attribute__((aligned(16))) Pair { double a, b; };

// a[c] += x(lane c of the row) s, c < 16. A DPP operand must not have been written by the two instructions before it, and the compiler
// does not look into these: hence the waits, at the end for what follows. (An instruction that needs the result of the one before it
// costs no more than another one, four cycles.)
__device__ __forceinline__ void row_update(double (&a)[16], double x, double s) {
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %16, %17 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %16, %17 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, %16, %17 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, %16, %17 row_newbcast:3 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %4, %16, %17 row_newbcast:4 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %5, %16, %17 row_newbcast:5 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %6, %16, %17 row_newbcast:6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %7, %16, %17 row_newbcast:7 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %8, %16, %17 row_newbcast:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %9, %16, %17 row_newbcast:9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %10, %16, %17 row_newbcast:10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %11, %16, %17 row_newbcast:11 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %12, %16, %17 row_newbcast:12 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %13, %16, %17 row_newbcast:13 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %14, %16, %17 row_newbcast:14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %15, %16, %17 row_newbcast:15 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1"
        : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]), "+v"(a[8]), "+v"(a[9]), "+v"(a[10]), "+v"(a[11]), "+v"(a[12]), "+v"(a[13]), "+v"(a[14]), "+v"(a[15])
        : "v"(x), "v"(s));
}
// q += the sum over c of x(lane c of the row) a[c]
__device__ __forceinline__ void row_product(double& q, double x, const double (&a)[16]) {
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %3 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %4 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %5 row_newbcast:3 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %6 row_newbcast:4 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %7 row_newbcast:5 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %8 row_newbcast:6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %9 row_newbcast:7 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %10 row_newbcast:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %11 row_newbcast:9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %12 row_newbcast:10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %13 row_newbcast:11 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %14 row_newbcast:12 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %15 row_newbcast:13 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %16 row_newbcast:14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %17 row_newbcast:15 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1"
        : "+v"(q)
        : "v"(x), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]), "v"(a[7]), "v"(a[8]), "v"(a[9]), "v"(a[10]), "v"(a[11]), "v"(a[12]), "v"(a[13]), "v"(a[14]), "v"(a[15]));
}
// the value of the given lane (4 * lane in `at`)
__device__ __forceinline__ double from_lane(double v, int at) {
    const long long u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_ds_bpermute(at, (int)u), hi = __builtin_amdgcn_ds_bpermute(at, (int)(u >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// The reduction by 4 J + 2 waves of rows off .. off + n - 1, the last of a solve of 64 JN buffer rows if JN > J. rest: what several
// work-groups leave of the matrix after `off` steps, 64 x 64 and scaled, with bad set if the diagonal has a NaN; null: it is C's.
template <int J, int JN>
__device__ __forceinline__ void tri_one(const double* __restrict__ C, int NP, int m0, int LP, int n, int off,
                                        const double* __restrict__ rest, double* __restrict__ dT, double* __restrict__ eT,
                                        double* __restrict__ tauT, double* __restrict__ V, double* __restrict__ stat, bool* bad) {
    constexpr int W = 4 * J, N = 64 * J, NV = 64 * JN;  // NV: columns of V
    constexpr bool TAIL = JN > J;
    __shared__ Pair qc[2][N + 64];  // {q, c} by step parity; what is not wanted goes beyond them
    __shared__ __attribute__((aligned(16))) double prm[2][2 * W];  // waves' sums of x A x, then tau, v1, off-diagonal element
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int blocks = (n + 15) >> 4, steps = 16 * blocks - 1;  // of all waves: one barrier each
    int ex = 0;
    double sc0 = 1.0;
    if (!TAIL || !rest) {
        ex = tri_exponent(wave_max_diag(C, NP, lane));
        sc0 = __builtin_amdgcn_ldexp(1.0, -ex);
    }
    auto inside = [&](int r, int c) __attribute__((always_inline)) { return r < n && c < n; };
    auto load = [&](int r, int c) __attribute__((always_inline)) {
        if (TAIL && rest) return __hip_atomic_load(rest + c * 64 + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // (past the L1)
        const bool in = inside(r, c);
        return C[(int64_t)(in ? active_index(c, m0, LP) : 0) * NP + (in ? active_index(r, m0, LP) : 0)];
    };
    double x[J], v[J], nw[J];  // column k below row k + 1; v and -w of the step before: rows lane + 64 j
#pragma unroll
    for (int j = 0; j < J; ++j) {
        x[j] = load(lane + 64 * j, 0);
        v[j] = nw[j] = 0.0;
    }
    double xk = load(0, 0), xk1 = load(1, 0);  // column k at rows k and k + 1, where it is wanted
    loads_go_out();
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int r = lane + 64 * j;
        x[j] = r > 1 && inside(r, 0) ? x[j] * sc0 : 0.0;
    }
    xk = inside(0, 0) ? xk * sc0 : 0.0;
    xk1 = inside(1, 0) ? xk1 * sc0 : 0.0;

    // what the waves do after the barrier of step k, whose column k + 1 is in registers J0 .. : v, -w and the next x. xn: the next column
    // with row k + 2, which x leaves out. (One read for all that is the same in all lanes: six waves' reads come at once.)
    struct Scal { double v1, w1, tau, c1, beta; };
    auto vectors = [&](auto uc, int k, double (&xn)[J]) __attribute__((always_inline)) {
        constexpr int J0 = decltype(uc)::value;
        const int par = k & 1;
        const double z = prm[par][lane & (2 * W - 1)];
        double q[J], c[J];
#pragma unroll
        for (int j = J0; j < J; ++j) {
            const Pair e = qc[par][lane + 64 * j];
            q[j] = e.a;
            c[j] = e.b;
        }
        const double tau = read_lane(z, W), v1 = read_lane(z, W + 1), beta = read_lane(z, W + 2);
        double s = read_lane(lane_sum<W>(z), 0);
        const double q1 = read_lane(q[J0], (k + 1) & 63), c1 = read_lane(c[J0], (k + 1) & 63);
        const double g1 = __builtin_fma(v1, c1, q1);                          // q + v1 c at k + 1
        s = __builtin_fma(v1, q1 + g1, s);                                    // v A v = x A x + 2 v1 q + v1^2 c
        const double nal = 0.5 * tau * (tau * s);
        const double w1 = __builtin_fma(-nal, v1, tau * g1);
#pragma unroll
        for (int j = J0; j < J; ++j) {
            const int r = lane + 64 * j;
            v[j] = r == k + 1 ? v1 : x[j];
            // (rows that are finished need no care: H leaves next to nothing of them, and x is zero there)
            nw[j] = __builtin_fma(nal, v[j], -tau * __builtin_fma(v1, c[j], q[j]));
            xn[j] = __builtin_fma(-v[j], w1, __builtin_fma(nw[j], v1, c[j]));
            x[j] = r > k + 2 ? xn[j] : 0.0;
        }
        return Scal{v1, w1, tau, c1, beta};
    };
    constexpr std::integral_constant<int, 0> first{};
    constexpr std::integral_constant<int, J - 1> second{};

    if (wave < W) {
        const int r16 = lane & 15, g = lane >> 4, row = 16 * wave + r16;
        double a[J][16];
#pragma unroll
        for (int u = 0; u < J; ++u)
#pragma unroll
            for (int c = 0; c < 16; ++c) a[u][c] = load(row, 16 * (g + 4 * u) + c);
        loads_go_out();
#pragma unroll
        for (int u = 0; u < J; ++u)
#pragma unroll
            for (int c = 0; c < 16; ++c) a[u][c] = inside(row, 16 * (g + 4 * u) + c) ? a[u][c] * sc0 : 0.0;
        // the vectors at this lane's row, which lane `row` of a register has
        const bool upper = J > 1 && wave >= 4;
        auto at_row = [&](const double (&y)[J]) __attribute__((always_inline)) { return from_lane(upper ? y[J - 1] : y[0], 4 * (row & 63)); };
        double vr = 0.0, nwr = 0.0, xr = at_row(x);
        if (lane < 2) prm[lane][wave] = 0.0;
        if (g < 2) qc[g][row] = Pair{0.0, 0.0};
        const int qat = g == 0 ? row : N + lane;
        lds_barrier();
        if (wave >= blocks) {  // no rows: what it would add is zero
            for (int k = 0; k < steps; ++k) lds_barrier();
            return;
        }
        const int mine = wave + 1;  // column blocks before this wave's rows are finished
        auto step = [&](auto uc, auto cc, int b, int cat) __attribute__((always_inline)) {
            constexpr int U = decltype(uc)::value, CC = decltype(cc)::value;
            const int k = 16 * b + CC - 1;
            constexpr int par = (CC + 1) & 1;  // of k
#pragma unroll
            for (int u = U; u < J; ++u) row_update(a[u], nw[u], vr);
#pragma unroll
            for (int u = U; u < J; ++u) row_update(a[u], v[u], nwr);
            qc[par][cat].b = a[U][CC];
            double q = 0.0, b0, b1;
#pragma unroll
            for (int u = U; u < J; ++u) row_product(q, x[u], a[u]);
            swap_rows<16>(q, b0, b1);
            q = b0 + b1;
            swap_rows<32>(q, b0, b1);
            q = b0 + b1;
            qc[par][qat].a = q;
            const double p = lane_sum<16>(q * xr);
            if (lane == 0) prm[par][wave] = p;
            lds_barrier();
            double xn[J];
            const Scal s = vectors(uc, k, xn);
            vr = row == k + 1 ? s.v1 : xr;
            xr = at_row(x);
            nwr = at_row(nw);
        };
        auto sixteen = [&](auto uc, int b) __attribute__((always_inline)) {
            constexpr int U = decltype(uc)::value;
            const int cat = g == b - 4 * U ? row : N + lane;
            if (b > 0) step(uc, std::integral_constant<int, 0>{}, b, cat);
            step(uc, std::integral_constant<int, 1>{}, b, cat);
            step(uc, std::integral_constant<int, 2>{}, b, cat);
            step(uc, std::integral_constant<int, 3>{}, b, cat);
            step(uc, std::integral_constant<int, 4>{}, b, cat);
            step(uc, std::integral_constant<int, 5>{}, b, cat);
            step(uc, std::integral_constant<int, 6>{}, b, cat);
            step(uc, std::integral_constant<int, 7>{}, b, cat);
            step(uc, std::integral_constant<int, 8>{}, b, cat);
            step(uc, std::integral_constant<int, 9>{}, b, cat);
            step(uc, std::integral_constant<int, 10>{}, b, cat);
            step(uc, std::integral_constant<int, 11>{}, b, cat);
            step(uc, std::integral_constant<int, 12>{}, b, cat);
            step(uc, std::integral_constant<int, 13>{}, b, cat);
            step(uc, std::integral_constant<int, 14>{}, b, cat);
            step(uc, std::integral_constant<int, 15>{}, b, cat);
        };
        int b = 0;
        for (; b < (mine < 4 ? mine : 4); ++b) sixteen(first, b);
        if constexpr (J == 2) {
            for (; b < mine; ++b) sixteen(second, b);
        }
        // Its rows are finished: x and so its part of x A x is zero from here on. (The sum of the step before last is still there.)
        if (lane == 0) prm[1][wave] = 0.0;
        for (int k = 16 * mine - 1; k < steps; ++k) lds_barrier();
        return;
    }

    if (wave > W) {  // stores the results
        if (lane == 0 && !(TAIL && rest)) stat[0] = (double)ex;
        lds_barrier();
        double* const Vo = V + (int64_t)off * NV;
        bool nan = xk != xk;
        auto steps_of = [&](auto uc, int k, int end) __attribute__((always_inline)) {
            constexpr int U = decltype(uc)::value;
            for (; k < end; ++k) {
                lds_barrier();
                double xn[J];
                const Scal s = vectors(uc, k, xn);
                double* const row = Vo + (int64_t)k * NV;
                if constexpr (TAIL) {  // (one register, its entries at columns off ..)
#pragma unroll
                    for (int j = 0; j < JN; ++j)
                        if (lane + 64 * j < off || lane + 64 * j >= off + 64) row[lane + 64 * j] = 0.0;
                    row[off + lane] = v[0];
                } else {
#pragma unroll
                    for (int j = 0; j < J; ++j) row[lane + 64 * j] = j >= U ? v[j] : 0.0;
                }
                if (lane < 3) (lane == 0 ? dT : lane == 1 ? eT : tauT)[off + k] = lane == 0 ? xk : lane == 1 ? s.beta : s.tau;
                xk = __builtin_fma(-2.0 * s.v1, s.w1, s.c1);
                nan = nan || xk != xk;
            }
            return k;
        };
        const int k63 = steps_of(first, 0, steps < 63 ? steps : 63);
        if constexpr (J == 2) steps_of(second, k63, steps);
        if (lane == 0 && steps == n - 1) dT[off + steps] = xk;
        // what follows the last row, with the steps beyond it (where there is a rest, that has been done)
        if (!(TAIL && rest)) tri_finish<JN>(n, dT, eT, tauT, V, lane, 64);
        if (TAIL && rest && lane == 0) *bad = nan;
        return;
    }
    // ---- the wave of the reflectors
    __builtin_amdgcn_s_setprio(3);
    auto reflect = [&](int k) __attribute__((always_inline)) {
        double r2 = 0.0, beta, tau, v1;
#pragma unroll
        for (int j = 0; j < J; ++j) r2 = __builtin_fma(x[j], x[j], r2);
        r2 = lane_sum<64>(r2);
        householder(xk1, r2, beta, tau, v1);
        if (lane == 0) {
            *reinterpret_cast<Pair*>(&prm[k & 1][W]) = Pair{tau, v1};
            prm[k & 1][W + 2] = beta;
        }
    };
    reflect(0);
    lds_barrier();
    auto steps_of = [&](auto uc, int k, int end) __attribute__((always_inline)) {
        constexpr int U = decltype(uc)::value;
        for (; k < end; ++k) {
            lds_barrier();
            double xn[J];
            vectors(uc, k, xn);
            xk1 = read_lane(k + 2 < 64 * (U + 1) || U + 1 >= J ? xn[U] : xn[U + 1 < J ? U + 1 : U], (k + 2) & 63);
            reflect(k + 1);
        }
        return k;
    };
    const int k63 = steps_of(first, 0, steps < 63 ? steps : 63);
    if constexpr (J == 2) steps_of(second, k63, steps);
}

// The whole reduction by T threads of one work-group, for solves that several could not do together, or where one of them found NaN. (If
// that is the matrix's, so is what comes of this, and it does no harm.)
template <int JN, int T>
__device__ __forceinline__ void tri_redo(const double* __restrict__ C, int NP, int m0, int LP, int n, double* __restrict__ dT,
                                         double* __restrict__ eT, double* __restrict__ tauT, double* __restrict__ V,
                                         double* __restrict__ stat, double* __restrict__ redone) {
    __shared__ double vec[4 * 64 * JN];
    const int tid = threadIdx.x;
    const int ex = tri_exponent(wave_max_diag(C, NP, tid & 63));
    if (tid == 0) {
        *redone += 1.0;
        stat[0] = (double)ex;
    }
    tri_alone<JN, T>(C, NP, m0, LP, n, dT, eT, tauT, V, __builtin_amdgcn_ldexp(1.0, -ex), vec);
    __syncthreads();
    tri_finish<JN>(n, dT, eT, tauT, V, tid, T);
}

// JN > J: no more than 64 J rows of a solve of 64 JN buffer rows; more of them, with `all`, are done as after a wait in vain.
template <int J, int JN>
__global__ __launch_bounds__(64 * (4 * J + 2), 1) void tri_one_kernel(const double* __restrict__ C, int NP, int m0, int LP, int n, bool all,
                                                                      double* __restrict__ dT, double* __restrict__ eT,
                                                                      double* __restrict__ tauT, double* __restrict__ V,
                                                                      double* __restrict__ stat, double* __restrict__ redone) {
    if constexpr (JN > J) {
        if (all) {
            tri_redo<JN, 64 * (4 * J + 2)>(C, NP, m0, LP, n, dT, eT, tauT, V, stat, redone);
            return;
        }
    }
    tri_one<J, JN>(C, NP, m0, LP, n, 0, nullptr, dT, eT, tauT, V, stat, nullptr);
}

// 64 rows, and beside them the next rows of a stream into another half (insert_kernel's work, 16 rows x 8 slabs a wave): as a launch
// of its own that took 4.7 us of a cycle of 85 (512 columns), and the chip is idle here but for one CU.
template <typename Src>
__global__ __launch_bounds__(384, 1) void tri_one_insert_kernel(const double* __restrict__ C, int m0, int n, double* __restrict__ dT,
                                                                double* __restrict__ eT, double* __restrict__ tauT,
                                                                double* __restrict__ V, double* __restrict__ stat, Src src, int rows,
                                                                float* __restrict__ half, int64_t D, int64_t S, int row_groups,
                                                                int64_t units) {
    constexpr int LP = 32, NS = 8;
    if (blockIdx.x == 0) {
        __builtin_amdgcn_s_setprio(3);
        tri_one<1, 1>(C, 2 * LP, m0, LP, n, 0, nullptr, dT, eT, tauT, V, stat, nullptr);
        return;
    }
    const int lane = threadIdx.x & 63;
    const int64_t unit = (int64_t)(blockIdx.x - 1) * 6 + (threadIdx.x >> 6);
    if (unit >= units) return;
    const int r = (int)((unsigned)unit % (unsigned)row_groups) * 16 + (lane >> 2), p = lane & 3;
    if (r >= rows) return;
    const int64_t s0 = (int64_t)((unsigned)unit / (unsigned)row_groups) * NS;
    float4 v[NS];
    src.template load<NS>(r, s0 * DC + p * 4, D, v);
    float4* dst = reinterpret_cast<float4*>(half + (s0 * LP + r) * DC) + p;
#pragma unroll
    for (int i = 0; i < NS; ++i)
        if (s0 + i < S) dst[(int64_t)i * LP * (DC / 4)] = v[i];
}
template <typename Src>
static void launch_tri_one_insert(const EigWork& w, int m0, int n, const Src& src, const RowJob& job, hipStream_t st) {
    const int row_groups = (job.rows + 15) / 16;
    const int64_t units = (job.d.S + 7) / 8 * row_groups;
    hipLaunchKernelGGL(tri_one_insert_kernel<Src>, dim3((unsigned)(1 + (units + 5) / 6)), dim3(384), 0, st, w.C, m0, n, w.dT, w.eT, w.tauT,
                       w.V, w.stat, src, job.rows, job.half, job.d.D, job.d.S, row_groups, units);
}
static void launch_tri_one_insert(const EigWork& w, int m0, int n, const RowJob& job, hipStream_t st) {
    const bool bf16 = job.dtype == SAGE_BF16;
    if (!job.G) {
        if (bf16) launch_tri_one_insert(w, m0, n, OuterRows<uint16_t>{(const uint16_t*)job.E, (const uint16_t*)job.H, job.C, job.dh}, job, st);
        else launch_tri_one_insert(w, m0, n, OuterRows<float>{(const float*)job.E, (const float*)job.H, job.C, job.dh}, job, st);
        return;
    }
    const bool vec = rows_start_on_four(job.G, job.dtype, job.d);
    if (bf16 && vec) launch_tri_one_insert(w, m0, n, DenseRows<uint16_t, true>{(const uint16_t*)job.G}, job, st);
    else if (bf16) launch_tri_one_insert(w, m0, n, DenseRows<uint16_t, false>{(const uint16_t*)job.G}, job, st);
    else if (vec) launch_tri_one_insert(w, m0, n, DenseRows<float, true>{(const float*)job.G}, job, st);
    else launch_tri_one_insert(w, m0, n, DenseRows<float, false>{(const float*)job.G}, job, st);
}

// ---- n = 64 J, J = 2, 4, 8: 16, 32, 32 work-groups on one XCD -----------------------------------------------------
// As above, but a wave owns 2 (n = 128, 256) or 4 whole columns, carries all vectors itself and sums its products over the
// lanes, and q and c go through the L2 the work-groups share. An exchanged value is its own 8 bytes: a slot holds a pattern that
// is no result until it is written, so there are no flags and no fences, and a reader polls, with loads that bypass its L1
// (sc1), until it sees anything else. Four slots by step; the work-group of the last column, which sees every step, empties them
// (fd_tri_plan.h). When 64 rows are left, their columns' owners store them and say so, a bit of a word for each column, and the
// work-group of the last one, which has the most to do with them, goes on alone (tri_one). A kernel of its own for that took 34 us
// where the chip was idle, but 49 to 73 at 512 rows and 57 at 96 beside the side stream's work: that keeps off the XCD of the solve only,
// and a launch's one work-group goes anywhere. The kernel after this one empties the slots and the word (dc_block_kernel), so that a solve needs no number of its own
// and a captured one can be replayed. (16-byte entries with a tag in each half, which need no emptying, moved twice the bytes and
// took two loads a thread at 512 rows: 830 us beside the look-ahead work instead of 595.)
// Stores: the L1 is write-through, so a plain store reaches the XCD's L2. Of the work-groups launched, one in `period` lands on
// the XCD of the solve and stays, in the role of its number (see TriClaim for what happens if none does).
// Waves 0..3 compute and publish, n / 64 more only poll and hand over through LDS, half of them q and half c: loads and stores of
// a wave retire in order, so one that did both would wait, with every poll, for its own stores.
// What a step costs (n = 256, cycles of 2.07 k): products and sums until q is out 600, until the last q is seen some 950 (a
// store's way to L2, half a poll's period, a poll of 550), handing over 150, w and the next column 350. A branch costs a
// wave 100 cycles, taken or not (an instruction about five), which is why the loop has as few as it has and
// is written out per 64 steps: 264 -> 212 us at 256 rows and 740 -> 520 at 512 together with the smaller entries.
// The work-groups must be resident together, which nothing guarantees: kernels of other streams and processes may hold the CUs
// of the XCD. So a thread polls at most `polls` times in vain in all and then goes on with NaN for what did not come. NaN
// goes into everything it publishes from then on, so the others lose no time waiting, and reaches the work-group of the
// last column or what is left of the matrix, where that one finds it. It then repeats the whole reduction alone (tri_redo): a
// solve never fails. A work-group that starts when the others have
// given up sees that in claim[1] and loses no time either.
// poll_limit: to wait for as long as the repetition takes, 1.9, 3.8 and 15 ms (0.23 us a poll), costs at most twice what the better
// of waiting and repeating would have. A reduction polls 500, 1100 and 3000 times in vain while it waits for its own steps.
constexpr int poll_limit(int J) { return J == 2 ? 1 << 13 : J == 4 ? 1 << 14 : 1 << 16; }

__device__ __forceinline__ void put_entry(double* p, double v) {
    *p = v;
    asm volatile("" ::: "memory");  // stays here
}

template <int J>
__global__ __launch_bounds__(TriPlan<J>::THREADS, 1) void tri_many_kernel(const double* __restrict__ C, int NP, int m0, int LP, int n,
                                                          double* __restrict__ dT, double* __restrict__ eT,
                                                          double* __restrict__ tauT, double* __restrict__ V,
                                                          double* __restrict__ stat, double* __restrict__ xch,
                                                          int xcd, int shift, int polls, double* __restrict__ rest,
                                                          unsigned* __restrict__ claim, double* __restrict__ redone) {
    using Plan = TriPlan<J>;
    constexpr int N = Plan::N, CW = Plan::CW, NW = Plan::NW, T = Plan::THREADS, T1 = 384;  // (T1: see tri_one)
    const int wg = blockIdx.x >> shift, last = n - 64;  // steps 0 .. last - 1
    const bool here = xcd_id() == xcd;
    const bool closes = Plan::closes(wg, n);  // this work-group stores what the solve's next stages read
    if (!here && !closes) return;
    __shared__ __attribute__((aligned(16))) double qc[4][N + 2];  // q by step parity, then c
    __shared__ __attribute__((aligned(16))) double vs[2][N];  // the closing work-group: the reflector, by step parity,
    __shared__ double sc[2][64];                              // and {diagonal, off-diagonal element, tau}
    __shared__ bool gave_up, bad;
    unsigned long long* const left = reinterpret_cast<unsigned long long*>(claim + 2);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (here) {  // waves that compute go before those that wait
        if (wave < 4) __builtin_amdgcn_s_setprio(3);
        else __builtin_amdgcn_s_setprio(1);
    }
    if (Plan::last_column(wg, n) < 0) return;
    const int steps = Plan::steps_until(wg, n, last), waits = Plan::waits_until(wg, n, last);  // waits >= steps - 1
    __shared__ TriClaim role;
    if (closes && tid == 256) {  // (a thread that waits anyway)
        const unsigned mine = claim_add(here);
        const unsigned word = mine + __hip_atomic_fetch_add(claim, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        role = claim_role(word, here, 1 << shift);
        if (claim_last(word, 1 << shift)) __hip_atomic_store(claim, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }

    auto wait_for_entries = [&]() __attribute__((always_inline)) {  // waves 4 ..: one half waits for q, the other for c
        const int t = tid - 256;
        const bool for_c = t >= N / 2;
        const int i0 = 2 * (for_c ? t - N / 2 : t);  // this thread's entries: i0, i0 + 1
        int spins = polls;
        if (__hip_atomic_load(claim + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) spins = 1;
        if (closes) tri_finish<J>(n, dT, eT, tauT, V, t, N);
        auto store_reflector = [&](int k) __attribute__((always_inline)) {
            *reinterpret_cast<Pair*>(V + (int64_t)k * N + i0) = *reinterpret_cast<const Pair*>(&vs[k & 1][i0]);
            if (i0 < 6) (i0 == 0 ? dT : i0 == 2 ? eT : tauT)[k] = sc[k & 1][i0 / 2];
        };
        for (int k = 0; k < steps; ++k) {
            double* const dst = &qc[(k & 1) + (for_c ? 2 : 0)][i0];
            if (closes) {
                if (for_c) {  // (it has time: c comes long before q)
                    if (k > 0) store_reflector(k - 1);
                } else {      // empty the slot of step k + 2 (TriPlan)
                    const u32x4 empty{~0u, ~0u, ~0u, ~0u};
                    double* const slot = xch + Plan::slot(k + 2) * 2 * N + i0;
                    *reinterpret_cast<u32x4*>(slot) = empty;
                    *reinterpret_cast<u32x4*>(slot + N) = empty;
                }
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // done before this step's barrier
            }
            // Both entries in one load; the thread is done with entries of rows <= k. What came goes to LDS before it is looked
            // at: if it is there, so is its copy. (In a last step that is not waited for, the waves that compute get zeros: nothing
            // comes of it.)
            const bool on0 = i0 > k && i0 < n, on1 = i0 + 1 > k && i0 + 1 < n;
            if ((on0 || on1) && k < waits) {
                const double* const src = xch + (Plan::slot(k) * 2 + (for_c ? 1 : 0)) * N + i0;
                bool more;
                do {
                    u32x4 e;
                    asm volatile(
                        "global_load_dwordx4 %0, %1, off sc1\n\t"
                        "s_waitcnt vmcnt(0)"
                        : "=&v"(e)
                        : "v"(src)
                        : "memory");
                    const bool empty0 = on0 && (e[0] & e[1]) == ~0u, empty1 = on1 && (e[2] & e[3]) == ~0u;
                    if (!on0) e[0] = e[1] = 0u;
                    if (!on1) e[2] = e[3] = 0u;
                    *reinterpret_cast<u32x4*>(dst) = e;
                    more = empty0 || empty1;
                    if (more && --spins <= 0) {
                        spins = 1;  // every further wait gives up after one round
                        more = false;
                        __hip_atomic_store(claim + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        const double nan = __longlong_as_double(0x7FF8000000000000ll);
                        if (empty0) dst[0] = nan;
                        if (empty1) dst[1] = nan;
                    }
                } while (more);
            } else {
                *reinterpret_cast<Pair*>(dst) = Pair{0.0, 0.0};
            }
            lds_barrier();
        }
        if (closes && for_c && steps > 0) store_reflector(steps - 1);
    };

    // Wave gw owns the columns of lane gw % 64: cl + 64 (H + s J / CW), s < CW, H = gw / 64 < J / CW. So the entries of v and w at
    // its own columns are in one lane of its own registers.
    const int gw = wg * 4 + wave, cl = gw & 63;
    auto reduce = [&](auto hc) __attribute__((always_inline)) {
        constexpr int H = decltype(hc)::value, ST = Plan::ST;  // register index of column s: H + ST * s
        double a[CW][J], x[J], v[J], w[J];
        const double md = wave_max_diag(C, NP, lane);
        const int ex = tri_exponent(md);
        const double sc0 = __builtin_amdgcn_ldexp(1.0, -ex);
        {
            int mrow[J];
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int r = lane + 64 * j;
                mrow[j] = r < n ? active_index(r, m0, LP) : -1;
            }
#pragma unroll
            for (int s = 0; s < CW; ++s) {
                const int col = cl + 64 * (H + ST * s);
                const double* src = C + (int64_t)active_index(col < n ? col : 0, m0, LP) * NP;
#pragma unroll
                for (int j = 0; j < J; ++j) a[s][j] = src[mrow[j] >= 0 ? mrow[j] : 0];
            }
            const double* src = C + (int64_t)active_index(0, m0, LP) * NP;
#pragma unroll
            for (int j = 0; j < J; ++j) x[j] = src[mrow[j] >= 0 ? mrow[j] : 0];
            loads_go_out();
#pragma unroll
            for (int s = 0; s < CW; ++s) {
                const int col = cl + 64 * (H + ST * s);
#pragma unroll
                for (int j = 0; j < J; ++j) a[s][j] = col < n && mrow[j] >= 0 ? a[s][j] * sc0 : 0.0;
            }
#pragma unroll
            for (int j = 0; j < J; ++j) {
                x[j] = mrow[j] >= 0 ? x[j] * sc0 : 0.0;
                v[j] = 0.0;
                w[j] = 0.0;
            }
        }
        double xk = C[(int64_t)active_index(0, m0, LP) * NP + active_index(0, m0, LP)] * sc0;
        double xk1 = n > 1 ? C[(int64_t)active_index(0, m0, LP) * NP + active_index(1, m0, LP)] * sc0 : 0.0;

        // The steps whose column k + 1 lies in [64 B, 64 B + 64): rows and columns below 64 B are done with, and left out at
        // compile time. A step is straight-line code but for the publishing of c: a branch costs a wave some 100 cycles, taken or
        // not, an instruction five.
        // Where the lane stores its column's sum; lanes beyond the wave's columns are out of the buffer's range, which the store
        // leaves out (an exec-masked store would cost a branch).
        const auto ring = __builtin_amdgcn_make_buffer_rsrc(xch, 0, Plan::SLOTS * 2 * N * 8, 0x00027000);
        const int qofs = lane < CW ? (cl + 64 * (H + ST * lane)) * 8 : 0x40000000;
        auto steps_of = [&](auto bc) __attribute__((always_inline)) {
            constexpr int B = decltype(bc)::value;
            constexpr int S0 = B > H ? (B - H + ST - 1) / ST : 0, NS = CW - S0;  // columns s < S0 are done with
            if constexpr (NS > 0) {
                const int end = 64 * B + 63 < steps ? 64 * B + 63 : steps;
                for (int k = B > 0 ? 64 * B - 1 : 0; k < end; ++k) {
                    double* const cx = xch + Plan::slot(k) * 2 * N + N;
                    x[B] = lane + 64 * B > k + 1 ? x[B] : 0.0;  // (in steps before the last of the rows, all beyond are)
                    double acc[CW];
                    {
                        double vcol[CW], wcol[CW];
#pragma unroll
                        for (int s = S0; s < CW; ++s) {
                            vcol[s] = read_lane(v[H + ST * s], cl);
                            wcol[s] = read_lane(w[H + ST * s], cl);
                        }
#pragma unroll
                        for (int s = S0; s < CW; ++s)
#pragma unroll
                            for (int j = B; j < J; ++j) a[s][j] = __builtin_fma(-w[j], vcol[s], a[s][j]);
#pragma unroll
                        for (int s = S0; s < CW; ++s)
#pragma unroll
                            for (int j = B; j < J; ++j) a[s][j] = __builtin_fma(-v[j], wcol[s], a[s][j]);
                    }
                    if constexpr ((B & (ST - 1)) == H) {  // column k + 1 may be this wave's
                        if (((k + 1) & 63) == cl) {
#pragma unroll
                            for (int j = B; j < J; ++j) put_entry(cx + lane + 64 * j, a[(B - H) / ST][j]);
                        }
                    }
#pragma unroll
                    for (int s = S0; s < CW; ++s) acc[s] = a[s][B] * x[B];
#pragma unroll
                    for (int j = B + 1; j < J; ++j)
#pragma unroll
                        for (int s = S0; s < CW; ++s) acc[s] = __builtin_fma(a[s][j], x[j], acc[s]);
                    // The sums over the wave, one column per lane of a quad (pair): two at a time per lane pair, then one. (What
                    // goes to finished columns is not read.)
                    double t;
                    if constexpr (CW == 4) {
                        const bool odd = lane & 1, hi = lane & 2;
                        constexpr int S1 = S0 > 1 ? S0 : 1;
                        const double a0 = acc[S0 > 0 ? S1 : 0], a1 = acc[S1], a2 = acc[S0 > 2 ? 3 : 2], a3 = acc[3];
                        double t1 = odd ? a3 : a2, o1 = odd ? a2 : a3;
                        t1 += dpp_move<DPP_XOR1>(o1);       // lane parity q: column 2 + q
                        if constexpr (S0 < 2) {
                            double t0 = odd ? a1 : a0, o0 = odd ? a0 : a1;
                            t0 += dpp_move<DPP_XOR1>(o0);   // ... column q
                            t = hi ? t1 : t0;
                            const double o = hi ? t0 : t1;
                            t += dpp_move<DPP_XOR2>(o);     // lane & 3 = column; sums over quads so far
                        } else {
                            t = t1 + dpp_move<DPP_XOR2>(t1);
                        }
                    } else {
                        const bool odd = lane & 1;
                        t = (odd ? acc[CW - 1] : acc[S0]) + dpp_move<DPP_XOR1>(odd ? acc[S0] : acc[CW - 1]);
                        t += dpp_move<DPP_XOR2>(t);
                    }
                    t += dpp_move<0x124>(t);  // row_ror 4
                    t += dpp_move<0x128>(t);  // row_ror 8: sums over rows of 16
                    double b0, b1;
                    swap_rows<16>(t, b0, b1);
                    t = b0 + b1;
                    swap_rows<32>(t, b0, b1);
                    t = b0 + b1;
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, t), ring, qofs, Plan::slot(k) * 2 * N * 8, 0);
                    asm volatile("" ::: "memory");  // stays here
                    // while the entries travel: the reflector
                    double r2 = 0.0;
#pragma unroll
                    for (int j = B; j < J; ++j) r2 = __builtin_fma(x[j], x[j], r2);
                    r2 = lane_sum<64>(r2);
                    double beta, tau, v1;
                    householder(xk1, r2, beta, tau, v1);
                    // (for the next step; after the last, nothing comes of it)
                    const double v2 = read_lane((k + 2) >> 6 == B ? x[B] : x[B + 1 < J ? B + 1 : B], (k + 2) & 63);
#pragma unroll
                    for (int j = B; j < J; ++j) v[j] = j == B && lane + 64 * j == k + 1 ? v1 : x[j];
                    if (closes) {
#pragma unroll
                        for (int g = 0; g < J; g += 4) {  // registers g + wave (the finished rows' are zero)
                            double z[4];
#pragma unroll
                            for (int i = 0; i < 4; ++i) z[i] = g + i < B || g + i >= J ? 0.0 : v[g + i < J ? g + i : 0];
                            const double lo = wave & 1 ? z[1] : z[0], up = wave & 1 ? z[3] : z[2];
                            vs[k & 1][lane + 64 * (g + (J >= 4 ? wave : wave & 1))] = J >= 4 && (wave & 2) ? up : lo;
                        }
                        if (wave == 0) sc[k & 1][lane] = lane == 1 ? beta : lane == 2 ? tau : xk;
                    }
                    lds_barrier();
                    const double *const ql = qc[k & 1], *const cl2 = qc[2 + (k & 1)];
                    const Pair e1{ql[k + 1], cl2[k + 1]}, e2{ql[k + 2], cl2[k + 2]};
                    double c[J], dot = 0.0, dot2 = 0.0;
#pragma unroll
                    for (int j = B; j < J; ++j) {
                        const Pair e{ql[lane + 64 * j], cl2[lane + 64 * j]};  // (entries of rows <= k are zero)
                        c[j] = e.b;
                        w[j] = tau * __builtin_fma(v1, e.b, e.a);
                        if ((j - B) & 1) dot2 = __builtin_fma(w[j], v[j], dot2);
                        else dot = __builtin_fma(w[j], v[j], dot);
                    }
                    dot = lane_sum<64>(dot + dot2);
                    const double al = -0.5 * tau * dot;
                    const double w1 = __builtin_fma(al, v1, tau * __builtin_fma(v1, e1.b, e1.a));
                    const double w2 = __builtin_fma(al, v2, tau * __builtin_fma(v1, e2.b, e2.a));
#pragma unroll
                    for (int j = B; j < J; ++j) {
                        w[j] = __builtin_fma(al, v[j], w[j]);
                        x[j] = __builtin_fma(-v[j], w1, __builtin_fma(-w[j], v1, c[j]));
                    }
                    xk = __builtin_fma(-2.0 * v1, w1, e1.b);
                    xk1 = __builtin_fma(-v2, w1, __builtin_fma(-w2, v1, e2.b));
                }
            }
        };
        steps_of(std::integral_constant<int, 0>{});
        steps_of(std::integral_constant<int, 1>{});
        if constexpr (J >= 4) {
            steps_of(std::integral_constant<int, 2>{});
            steps_of(std::integral_constant<int, 3>{});
        }
        if constexpr (J >= 8) {
            steps_of(std::integral_constant<int, 4>{});
            steps_of(std::integral_constant<int, 5>{});
            steps_of(std::integral_constant<int, 6>{});
            steps_of(std::integral_constant<int, 7>{});
        }
        // What is left of this wave's columns, with the update of the last step; NaN if anything of it did not come.
        if (waits == last) {
#pragma unroll
            for (int s = 0; s < CW; ++s) {
                const int col = cl + 64 * (H + ST * s);
                const double vcol = read_lane(v[H + ST * s], cl), wcol = read_lane(w[H + ST * s], cl);
                if (col >= last && col < n) {
#pragma unroll
                    for (int j = 0; j < J; ++j) {
                        const int r = lane + 64 * j;
                        const double e = __builtin_fma(-v[j], wcol, __builtin_fma(-w[j], vcol, a[s][j]));
                        if (r >= last && r < n) rest[(col - last) * 64 + r - last] = e;
                    }
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // there before the column counts as there
                    if (lane == 0) __hip_atomic_fetch_or(left, 1ull << (col - last), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
        if (closes && tid == 0) {  // (xk: of row `last`)
            stat[0] = (double)ex;
            gave_up = xk != xk;
        }
    };
    static_assert(NW == 64 || NW == 128, "one or two columns a lane");
    if (!here) gave_up = true;
    else if (wave >= 4) wait_for_entries();
    else if (NW == 64 || gw < 64) reduce(std::integral_constant<int, 0>{});
    else reduce(std::integral_constant<int, NW / 64 - 1>{});
    if (!closes) return;
    lds_barrier();
    if (role == CLAIM_LEAVE || wave >= T1 / 64) return;  // (barriers are those of the waves that are left)
    // ---- the rows that are left
    if (!gave_up) {
        __builtin_amdgcn_s_setprio(3);
        if (tid == 0) {
            int spins = polls;
            while (__hip_atomic_load(left, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != ~0ull && --spins > 0) {}
            bad = spins <= 0;
        }
        lds_barrier();
        const bool missing = bad;
        lds_barrier();
        if (!missing) {
            tri_one<1, J>(C, NP, m0, LP, 64, last, rest, dT, eT, tauT, V, stat, &bad);
            lds_barrier();
            if (!bad) return;
        }
    }
    __syncthreads();
    tri_redo<J, T1>(C, NP, m0, LP, n, dT, eT, tauT, V, stat, redone);
}

// ---- Y = H Z --------------------------------------------------------------------------------------------------------
// One wave per eigenvector, the vector in registers (rows lane, lane + 64, ...); the reflectors are applied eight at a time
// as I - V T V^T (T from wy_factor), last block first, the next block's V and T on their way meanwhile. A block is 8
// products summed over the wave together, an 8 x 8 triangle and 8 updates, so the latency of a sum over the wave is paid
// once per eight reflectors (one or two at a time it was the bound). Rows before a block's first are zero in V and left
// out in quarters, each a loop of its own: with the choice inside one loop the waits for the next block's loads came
// early. Column N - 1 - m of Z (column-major, ascending eigenvalues) is the eigenvector of the m-th largest eigenvalue.
//
// OUT_Y: the vectors are stored, row m of Yt, in matrix indices. Otherwise a wave goes on to the rebuild's coefficients made
// from its vector, row m < count of diag(f) Y^T (zero rows up to MP), which saves a launch and a trip through memory (4.5 us
// at n = 64, 7.5 at 512):
//   mode 0, shrink (delta = sigma_ell^2, Sigma'_jj = sqrt(max(sigma_j^2 - delta, 0))): f_m = sqrt(max(lambda_m - delta, 0) /
//           lambda_m), so that row m is sqrt(sigma_m^2 - delta) v_m^T. Also records the Gram matrix of the rows the
//           rebuild is about to write, diag(max(lambda_m - delta, 0)), in `known`: the next cycle takes that block as
//           known instead of recomputing it.
//   mode 1, basis: f_m = 1 / sqrt(lambda_m), or 0 when lambda_m <= n 2^-23 lambda_1.
//   mode 2, weighted basis: f_m = sqrt(max(lambda_m - delta, 0) / lambda_m) under the same rank test, which makes the row the
//           m-th of the sketch a shrink of the buffer would write ("Two-pass scoring": z = S g).
// OUT_SPLIT, OUT_F32: in the orders of the rebuild (fd_coeffs.h). OUT_M: in fp64, row m of M in matrix indices, for a rebuild that
// comes later (fd_defer.hip). The work-group after the last row does the scalars.
enum { OUT_Y, OUT_F32, OUT_SPLIT, OUT_M };

// Eigenvector `col` of the last merge of N = 64 J rows, rows 2 lane, 2 lane + 1 of each 128, by one wave: u_j = zh_j / (d_j - lambda),
// normalised, and the sum of u_j times the survivors' columns of Z, of which those of the left (right) half have rows in that half
// only. A kernel on the matrix cores for all of them, one launch more, took 10 us at N = 128 and 14 at 256, and formed those that
// nobody wants too; here they cost 6.5 and 8 (jobs of 128, 200 and 256 buffer rows: 10.62 -> 10.30, 8.93 -> 8.71 and 10.85 -> 10.67
// ms; at 512, where the side stream or the rebuild is what a cycle waits for, 29.4 as before).
template <int J>
__device__ __forceinline__ void merged_vector(const double* __restrict__ Z, const DcWork& dc, int col, int lane, double (&z)[J]) {
    constexpr int N = 64 * J, half = N / 2, PAIRS = J / 2, U = 16 / PAIRS;  // steps requested together
    static_assert(half % (2 * U) == 0, "two sets of steps at a time");
    __shared__ double us[N], lu[N];
    __shared__ int lc[N];  // survivors' columns and entries of u in the order they are taken
    const int q = dc.from[col] & (N - 1), K = dc.K[0], k1 = dc.k1[0];  // (an index whatever the input was)
    const bool dense = dc.dense[0] != 0;
    auto left_pair = [&](int p) { return N == 128 ? lane < 32 : p < PAIRS / 2; };
    if (q >= K) {  // deflated: a column as it is
        const int src = dc.col[q];
        const double* c = Z + (int64_t)src * N + 2 * lane;
#pragma unroll
        for (int p = 0; p < PAIRS; ++p) {
            const f64x2 x = *reinterpret_cast<const f64x2*>(c + 128 * p);
            const bool own = dense || (src < half) == left_pair(p);  // (what else is stored there is stale)
            z[2 * p] = own ? x[0] : 0.0;
            z[2 * p + 1] = own ? x[1] : 0.0;
        }
        return;
    }
    const double org = dc.org[q], tau = dc.tau[q];
    double u[J], nn = 0.0;
    int list[J];
#pragma unroll
    for (int e = 0; e < J; ++e) {
        const int j = lane + 64 * e;
        list[e] = j < K ? dc.half[j] : 0;
        u[e] = j < K ? dc.zh[j] * rcp64((dc.dk[j] - org) - tau) : 0.0;
        nn = __builtin_fma(u[e], u[e], nn);
        // fill: entries of zero with a column that is finite in its half
        lu[j] = 0.0;
        lc[j] = dense || j < half ? 0 : half;
    }
    nn = lane_sum<64>(nn);
    const double inv = nn > 0.0 ? rcp64(__builtin_sqrt(nn)) : 0.0;
#pragma unroll
    for (int e = 0; e < J; ++e) us[lane + 64 * e] = u[e] * inv;
    __syncthreads();
    // (not dense: at most `half` of either half, the left one's first)
#pragma unroll
    for (int e = 0; e < J; ++e) {
        const int s = lane + 64 * e;
        if (s < K) {
            const int to = dense || s < k1 ? s : half + s - k1;
            lu[to] = us[list[e]];
            lc[to] = dc.col[list[e]];
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < J; ++j) z[j] = 0.0;
    const double* const zl = Z + 2 * lane;
    if (dense) {
        for (int s = 0; s < K; ++s) {
            const double us_ = lu[s];
#pragma unroll
            for (int p = 0; p < PAIRS; ++p) {
                const f64x2 x = *reinterpret_cast<const f64x2*>(zl + (int64_t)lc[s] * N + 128 * p);
                z[2 * p] = __builtin_fma(us_, x[0], z[2 * p]);
                z[2 * p + 1] = __builtin_fma(us_, x[1], z[2 * p + 1]);
            }
        }
        return;
    }
    struct Steps {
        f64x2 x[U][PAIRS];
        double u[U][2];
    };
    auto fetch = [&](int s0, Steps& t) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int s = s0 + i;
            const int cl = lc[s], cr = lc[half + s];
            t.u[i][0] = lu[s];
            t.u[i][1] = lu[half + s];
#pragma unroll
            for (int p = 0; p < PAIRS; ++p)
                t.x[i][p] = *reinterpret_cast<const f64x2*>(zl + (left_pair(p) ? cl : cr) * N + 128 * p);
        }
    };
    auto add = [&](const Steps& t) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < U; ++i)
#pragma unroll
            for (int p = 0; p < PAIRS; ++p) {
                const double w = left_pair(p) ? t.u[i][0] : t.u[i][1];
                z[2 * p] = __builtin_fma(w, t.x[i][p][0], z[2 * p]);
                z[2 * p + 1] = __builtin_fma(w, t.x[i][p][1], z[2 * p + 1]);
            }
    };
    const int steps = max(k1, K - k1);  // <= half
    Steps ta, tb;
    fetch(0, ta);
    for (int s = 0; s < steps; s += 2 * U) {
        fetch(s + U, tb);  // (s + 2 U <= half)
        add(ta);
        fetch(s + 2 * U < half ? s + 2 * U : 0, ta);  // (beyond the end: repeated, not used)
        add(tb);
    }
}

template <int J, int OUT>
__global__ __launch_bounds__(64, 1) void tri_back_kernel(const double* __restrict__ Z, DcWork dc, const double* __restrict__ V,
                                                         const double* __restrict__ Tw, int m0, int LP, int n,
                                                         double* __restrict__ Yt, int NP, CoeffArgs cf,
                                                         const double* __restrict__ dv, const double* __restrict__ C,
                                                         double* __restrict__ stat, double* __restrict__ known) {
    constexpr int N = 64 * J, NQ = J >= 4 ? J / 2 : 1, QS = J / NQ, QB = N / WY / NQ;  // parts; registers, blocks of a part
    const int lane = threadIdx.x;
    const int rank = blockIdx.x, col = N - 1 - rank;
    double f = 0.0;
    if constexpr (OUT != OUT_Y) {
        const int ex = (int)stat[0];
        auto lam = [&](int m) {  // m-th largest eigenvalue, clamped at 0
            const double v = dv[N - 1 - m];
            return v > 0.0 ? __builtin_amdgcn_ldexp(v, ex) : 0.0;
        };
        const double delta = lam(cf.ell - 1);
        if (rank == cf.MP) {  // scalars
            if (cf.mode == 0)
                for (int i = lane; i < N / 2; i += 64) known[i] = i < cf.ell ? fmax(lam(i) - delta, 0.0) : 0.0;
            // rows not yet counted in ||A||_F^2: their squared norms are on the diagonal of C
            double q = 0.0;
            for (int r = cf.ra0 + lane; r < cf.ra1; r += 64) q += C[(int64_t)r * NP + r];
            for (int r = cf.rb0 + lane; r < cf.rb1; r += 64) q += C[(int64_t)r * NP + r];
            q = lane_sum<64>(q);
            if (lane == 0) {
                cf.acc[1] += q;
                if (cf.mode == 0) {
                    cf.acc[0] += delta;
                    cf.acc[2] = delta;
                }
            }
            return;
        }
        if (rank < cf.count) {
            const double lm = lam(rank), keep = lm - delta;
            if (cf.mode == 0) {
                f = keep > 0.0 ? sqrt(keep / lm) : 0.0;
            } else if (lm > (double)cf.n * 1.1920928955078125e-07 * lam(0)) {
                f = cf.mode == 1 ? 1.0 / sqrt(lm) : (keep > 0.0 ? sqrt(keep / lm) : 0.0);
            }
        }
        if (f == 0.0) {  // a zero row
            if constexpr (OUT == OUT_M) {
                for (int i = lane; i < N; i += 64) cf.M[(int64_t)rank * N + i] = 0.0;
            } else if (lane < 8 * J) {
                store_coeffs<OUT == OUT_SPLIT>(cf.Mt, cf.Mc3, cf.MP, lane >> 1, lane & 1, rank, {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f});
            }
            return;
        }
    }
    // Rows of a lane: 2 lane, 2 lane + 1 of each 128, so that it loads 16 bytes at a time (60 -> 52 us at n = 512, 20.1 -> 18.8 at
    // 256, 10.0 -> 9.3 at 128: every wave reads all reflectors through its CU's cache); lane, where there are 64.
    constexpr int JW = J >= 2 ? 2 : 1;
    auto row = [&](int j) { return JW * lane + j % JW + 64 * (j - j % JW); };
    auto load_rows = [](const double* src, double* dst, int j) __attribute__((always_inline)) {
        if constexpr (JW == 2) {
            const f64x2 x = *reinterpret_cast<const f64x2*>(src);
            dst[j] = x[0];
            dst[j + 1] = x[1];
        } else {
            dst[j] = *src;
        }
    };
    double z[J];
    if constexpr (J == 1) z[0] = Z[(int64_t)col * N + lane];
    else merged_vector<J>(Z, dc, col, lane, z);
    struct Block {
        double v[WY][J], t;  // t: entry (lane >> 3, lane & 7) of T
    };
    Block va, vb;
    const bool odd = lane & 1, hi = lane & 2;

    auto load = [&](auto qc, int b, Block& k) __attribute__((always_inline)) {
        constexpr int J0 = decltype(qc)::value * QS;
#pragma unroll
        for (int i = 0; i < WY; ++i)
#pragma unroll
            for (int j = J0; j < J; j += JW) load_rows(V + (int64_t)(b * WY + i) * N + JW * lane + 64 * j, k.v[i], j);
        k.t = Tw[b * WY * WY + lane];
    };
    auto apply = [&](auto qc, const Block& k) __attribute__((always_inline)) {
        constexpr int J0 = decltype(qc)::value * QS;
        double p[WY];
#pragma unroll
        for (int i = 0; i < WY; ++i) p[i] = k.v[i][J0] * z[J0];
#pragma unroll
        for (int j = J0 + 1; j < J; ++j)
#pragma unroll
            for (int i = 0; i < WY; ++i) p[i] = __builtin_fma(k.v[i][j], z[j], p[i]);
        // sums over the wave of the eight: lane & 3 tells four apart, two registers the halves
        double s2[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const double* q = p + 4 * g;
            double t0 = odd ? q[1] : q[0], o0 = odd ? q[0] : q[1];
            double t1 = odd ? q[3] : q[2], o1 = odd ? q[2] : q[3];
            t0 += dpp_move<DPP_XOR1>(o0);
            t1 += dpp_move<DPP_XOR1>(o1);
            double t = hi ? t1 : t0, o = hi ? t0 : t1;
            t += dpp_move<DPP_XOR2>(o);
            t += dpp_move<0x124>(t);  // row_ror 4
            t += dpp_move<0x128>(t);  // row_ror 8
            double a0, a1;
            swap_rows<16>(t, a0, a1);
            t = a0 + a1;
            swap_rows<32>(t, a0, a1);
            s2[g] = a0 + a1;
        }
        double y = k.t * (lane & 4 ? s2[1] : s2[0]);  // y_p = sum_q T_pq s_q, p = lane >> 3, q = lane & 7
        y = lane_sum<8>(y);
#pragma unroll
        for (int i = 0; i < WY; ++i) {
            const double yi = -read_lane(y, 8 * i);
#pragma unroll
            for (int j = J0; j < J; ++j) z[j] = __builtin_fma(yi, k.v[i][j], z[j]);
        }
    };
    // the blocks of part q, from b (in va already) down to the part's first; leaves the block below in va
    auto part = [&](auto qc, int b) __attribute__((always_inline)) {
        constexpr int Q = decltype(qc)::value;
        constexpr std::integral_constant<int, (Q > 0 ? Q - 1 : 0)> below{};
        if (((b - Q * QB) & 1) == 0) {  // odd number of blocks: one first
            load(below, max(b - 1, 0), vb);
            apply(qc, va);
            va = vb;
            --b;
        }
        for (; b > Q * QB + 1; b -= 2) {
            load(qc, b - 1, vb);
            apply(qc, va);
            load(qc, b - 2, va);
            apply(qc, vb);
        }
        if (b > Q * QB) {
            load(qc, b - 1, vb);
            apply(qc, va);
            load(below, max(b - 2, 0), va);
            apply(qc, vb);
        }
        return Q * QB - 1;
    };
    // (the reduction leaves zeros in the rows of V that complete its last block)
    if (n >= 2) {
        int b = (n - 2) / WY;
        load(std::integral_constant<int, 0>{}, b, va);
        if constexpr (NQ == 4) {
            if (b >= 3 * QB) b = part(std::integral_constant<int, 3>{}, b);
            if (b >= 2 * QB) b = part(std::integral_constant<int, 2>{}, b);
        }
        if constexpr (NQ >= 2) {
            if (b >= QB) b = part(std::integral_constant<int, 1>{}, b);
        }
        part(std::integral_constant<int, 0>{}, b);
    }
    // Padding indices (matrix indices outside the active ones): a padding eigenvector is its own unit vector.
    const int gap = LP - m0;  // padding indices m0 .. LP-1 come first
    auto place = [&](int r) {
        const int q = r - n;
        return r < n ? active_index(r, m0, LP) : (q < gap ? m0 + q : n - m0 + LP + q - gap);
    };
    if constexpr (OUT == OUT_Y) {
        double* out = Yt + (int64_t)rank * NP;
#pragma unroll
        for (int j = 0; j < J; ++j) out[place(row(j))] = z[j];
    } else if constexpr (OUT == OUT_M) {
        double* out = cf.M + (int64_t)rank * N;
#pragma unroll
        for (int j = 0; j < J; ++j) out[place(row(j))] = f * z[j];
    } else {
        __shared__ double y[N];
#pragma unroll
        for (int j = 0; j < J; ++j) y[place(row(j))] = z[j];
        __syncthreads();
        if (lane < 8 * J) {
            const int stg = lane >> 1, h = lane & 1;
            Coeffs8 v;
#pragma unroll
            for (int s = 0; s < 8; ++s) v.c[s] = (float)(f * y[stg * 16 + h + 2 * s]);
            store_coeffs<OUT == OUT_SPLIT>(cf.Mt, cf.Mc3, cf.MP, stg, h, rank, v);
        }
    }
}

__global__ void xcd_probe_kernel(int* __restrict__ out) {
    if (threadIdx.x == 0) out[blockIdx.x] = xcd_id();
}
// The place (spare_unit) of an XCD among the work-groups of the launches that follow on this stream.
__global__ void xcd_place_kernel(int xcd, int* __restrict__ place) {
    if (threadIdx.x == 0 && xcd_id() == xcd) *place = (int)blockIdx.x;
}
hipError_t launch_xcd_place(int xcd, int* place, hipStream_t st) {
    hipLaunchKernelGGL(xcd_place_kernel, dim3(8), dim3(64), 0, st, xcd, place);
    return hipGetLastError();
}
const XcdMap& xcd_map() {
    static std::mutex lock;
    static XcdMap known[64];
    static bool asked[64] = {false};
    static const XcdMap nothing{};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nothing;
    std::lock_guard<std::mutex> hold(lock);
    if (!asked[dev]) {
        constexpr int B = 512;
        int* d = nullptr;
        int h[B];
        bool ok = hipMalloc((void**)&d, sizeof(h)) == hipSuccess;
        if (ok) {
            hipStream_t st = nullptr;
            ok = hipStreamCreateWithFlags(&st, hipStreamNonBlocking) == hipSuccess;
            if (ok) {
                hipLaunchKernelGGL(xcd_probe_kernel, dim3(B), dim3(64), 0, st, d);
                ok = hipMemcpyAsync(h, d, sizeof(h), hipMemcpyDeviceToHost, st) == hipSuccess &&
                     hipStreamSynchronize(st) == hipSuccess;
                (void)hipStreamDestroy(st);
            }
            (void)hipFree(d);
        }
        if (ok) known[dev] = xcd_map_of(h, B);
        asked[dev] = true;
    }
    return known[dev];
}

hipError_t launch_tridiag(const EigWork& w, int NP, int m0, int n, hipStream_t st, const RowJob* job) {
    const int LP = NP / 2;
    if (job && NP != 64) return hipErrorInvalidValue;
    const bool alone = w.period == 0;
#define SAGE_TRI_ONE(J, JN, ALL)                                                                                       \
    hipLaunchKernelGGL((tri_one_kernel<J, JN>), dim3(1), dim3(64 * (4 * J + 2)), 0, st, w.C, NP, m0, LP, n, ALL, w.dT, w.eT, w.tauT, \
                       w.V, w.stat, w.redone)
#define SAGE_TRI_MANY(J)                                                                                           \
    do {                                                                                                           \
        if (n > 64 && !alone)                                                                                      \
            hipLaunchKernelGGL(tri_many_kernel<J>, dim3(w.period * TriPlan<J>::NWG), dim3(TriPlan<J>::THREADS), 0, st, w.C, NP, m0, LP, \
                               n, w.dT, w.eT, w.tauT, w.V, w.stat, w.xch, w.xcd, __builtin_ctz(w.period),           \
                               w.impatient ? 1 : poll_limit(J), w.Yt, w.claim, w.redone);                          \
        else                                                                                                       \
            SAGE_TRI_ONE(1, J, n > 64);                                                                            \
    } while (0)
    switch (NP / 64) {
        case 1:
            if (job) launch_tri_one_insert(w, m0, n, *job, st);
            else SAGE_TRI_ONE(1, 1, false);
            break;
        case 2:
            if (alone) SAGE_TRI_ONE(2, 2, false);
            else SAGE_TRI_MANY(2);
            break;
        case 4: SAGE_TRI_MANY(4); break;
        case 8: SAGE_TRI_MANY(8); break;
        default: return hipErrorInvalidValue;
    }
#undef SAGE_TRI_ONE
#undef SAGE_TRI_MANY
    return hipGetLastError();
}

hipError_t launch_tri_back(const EigWork& w, int NP, int m0, int n, int count, const CoeffArgs* cf, hipStream_t st) {
    const int LP = NP / 2;
    const double* dv = w.dI[dc_result(NP)];
    const CoeffArgs args = cf ? *cf : CoeffArgs{};
#define SAGE_BACK(J, OUT)                                                                                                 \
    hipLaunchKernelGGL((tri_back_kernel<J, OUT>), dim3(OUT == OUT_Y ? count : args.MP + 1), dim3(64), 0, st,               \
                       w.Z[NP == 64 ? 0 : dc_result(NP) ^ 1], w.dc, w.V, w.Tw, m0, LP, n, w.Yt, NP, args, dv, w.C, w.stat, w.known)
#define SAGE_BACK_J(J)                        \
    if (!cf) SAGE_BACK(J, OUT_Y);             \
    else if (args.M) SAGE_BACK(J, OUT_M);       \
    else if (args.Mc3) SAGE_BACK(J, OUT_SPLIT); \
    else SAGE_BACK(J, OUT_F32);               \
    break
    switch (NP / 64) {
        case 1: SAGE_BACK_J(1);
        case 2: SAGE_BACK_J(2);
        case 4: SAGE_BACK_J(4);
        case 8: SAGE_BACK_J(8);
        default: return hipErrorInvalidValue;
    }
#undef SAGE_BACK_J
#undef SAGE_BACK
    return hipGetLastError();
}

}  // namespace sage
