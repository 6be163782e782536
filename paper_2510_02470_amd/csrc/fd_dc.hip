// Eigen-decomposition T = Z D Z^T of the tridiagonal matrix fd_tridiag.hip leaves, by divide and conquer (J. Cuppen,
// Numer. Math. 36, 1981): T is torn into 1 x 1 pieces, T = diag(d) + sum of rank-one terms at the cuts, and the pieces
// are merged pairwise. A merge of two solved halves is the eigenproblem of diag(d) + rho z z^T with z made of the last
// row of the left half's eigenvectors and the first row of the right half's:
//   * entries with rho |z_i| below tol, and all but one of a group of equal poles (after a rotation of their columns),
//     are deflated: they are eigenpairs already;
//   * the other eigenvalues are the roots of the secular equation 1 + rho sum z_j^2 / (d_j - lambda) = 0, one in every
//     gap, each kept as (nearest pole, distance): rational interpolation of the two sums on either side of the gap
//     (J. Bunch, C. Nielsen, D. Sorensen, Numer. Math. 31, 1978), inside a bracket that is bisected when a step leaves it;
//   * z is recomputed from the roots (M. Gu, S. Eisenstat, SIAM J. Matrix Anal. Appl. 16, 1995), which makes the
//     eigenvectors z_j / (d_j - lambda_i) orthogonal to fp64 rounding however close the roots are.
// Merges up to 64 rows run inside one work-group per 64 x 64 block (everything in LDS); the merges above it are four
// kernels each: deflation, roots (a wave per root), z and the order of the new eigenvalues, and the products of the
// halves' eigenvectors with the merge's on the fp64 matrix cores.
// Every size, index and count derived here is clamped by construction (counts of comparisons between finite numbers), so
// non-finite input gives wrong numbers but no access out of bounds.
#include "sage_internal.h"
#include "wave_ops.h"

namespace sage {

constexpr double DC_EPS = 2.220446049250313e-16;

__device__ __forceinline__ double finite_or_zero(double v) { return fabs(v) < 1e300 ? v : 0.0; }

// max(|d|, |e|) of the whole T, by every wave; the deflation threshold is 4 eps of it
__device__ __forceinline__ double dc_tolerance(const double* __restrict__ dT, const double* __restrict__ eT, int N,
                                               int lane) {
    double m = 0.0;
    for (int i = lane; i < N; i += 64) {
        const double d = finite_or_zero(dT[i]), e = finite_or_zero(eT[i]);
        if (!(d == -1.0 && e == 0.0)) m = fmax(m, fmax(fabs(d), fabs(e)));  // -1: padding
    }
    for (int o = 32; o >= 1; o >>= 1) m = fmax(m, __shfl_xor(m, o));
    return 4.0 * DC_EPS * m;
}

// Root q of 1 + sum_j z_j / (d_j - lambda) (z_j = rho z_j^2 > 0, K poles ascending): lambda = org + tau with org the
// nearer of the poles around it. A group of L lanes works on a root; lane l holds the poles l + L e, e < 8 (z = 0 and
// d = 1e30 beyond K).
template <int L>
__device__ __forceinline__ void secular_root(int K, int q, int l, const double (&dj)[8], const double (&zj)[8],
                                             double dq, double dq1, double zsum, double& org, double& tau) {
    const bool last = q == K - 1;
    double lo, hi;
    org = dq;
    if (!last) {
        const double mid = 0.5 * (dq1 - dq);
        double f = 0.0;
#pragma unroll
        for (int e = 0; e < 8; ++e) f = __builtin_fma(zj[e], rcp64((dj[e] - dq) - mid), f);
        f = 1.0 + lane_sum<L>(f);
        if (f >= 0.0) {
            lo = 0.0;
            hi = mid;
        } else {
            org = dq1;
            lo = -mid;
            hi = 0.0;
        }
    } else {
        lo = 0.0;
        hi = zsum * (1.0 + 4.0 * DC_EPS);
    }
    double t = 0.5 * (lo + hi);
    double dl[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) dl[e] = dj[e] - org;
    const double dlq = dq - org, dlq1 = dq1 - org;
    for (int it = 0; it < 60; ++it) {
        double psi = 0.0, dpsi = 0.0, phi = 0.0, dphi = 0.0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const double inv = rcp64(dl[e] - t);
            const double r = zj[e] * inv, r2 = r * inv;
            const bool low = l + L * e <= q;
            psi += low ? r : 0.0;
            dpsi += low ? r2 : 0.0;
            phi += low ? 0.0 : r;
            dphi += low ? 0.0 : r2;
        }
        psi = lane_sum<L>(psi);
        dpsi = lane_sum<L>(dpsi);
        phi = lane_sum<L>(phi);
        dphi = lane_sum<L>(dphi);
        const double f = 1.0 + psi + phi;
        // psi < 0 < phi: phi - psi is the sum of the magnitudes
        if (!(fabs(f) > 0.5 * DC_EPS * K * (1.0 + (phi - psi)))) break;
        if (f < 0.0) lo = fmax(lo, t);
        else hi = fmin(hi, t);
        double x;
        const double di = dlq - t;
        if (!last) {
            const double dn = dlq1 - t;  // di < 0 < dn
            const double p = di * di * dpsi, g = dn * dn * dphi;
            const double c = 1.0 + (psi - di * dpsi) + (phi - dn * dphi);
            // c + p / (di - x) + g / (dn - x) = 0, the root between the poles
            const double b = -(c * (di + dn) + p + g), a0 = c * di * dn + p * dn + g * di;
            const double s = __builtin_sqrt(fmax(__builtin_fma(b, b, -4.0 * c * a0), 0.0));
            const double h = -0.5 * (b + __builtin_copysign(s, b));
            const double x1 = a0 / h, x2 = h / c;
            x = (x1 > di && x1 < dn) ? x1 : x2;
            if (!(x > di && x < dn)) x = __builtin_nan("");
        } else {
            const double s = 1.0 + (psi - di * dpsi);
            x = s > 0.0 ? di + di * di * dpsi / s : __builtin_nan("");
        }
        double tn = t + x;
        if (!(tn > lo && tn < hi)) tn = 0.5 * (lo + hi);
        if (tn == t || !(hi - lo > fabs(t) * DC_EPS)) break;
        t = tn;
    }
    tau = t;
}

// |z_j| of the rank-one problem whose eigenvalues are exactly the computed roots: the product over i != j of
// (lambda_i - d_j) / (d_i - d_j), times (lambda_j - d_j). Lane l holds roots l + L e.
template <int L>
__device__ __forceinline__ double secular_z(int K, int j, int l, double dj, const double (&di)[8], const double (&org)[8],
                                            const double (&tau)[8]) {
    double pr = 1.0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int i = l + L * e;
        if (i < K) {
            const double num = (org[e] - dj) + tau[e];
            pr *= i == j ? num : num * rcp64(di[e] - dj);
        }
    }
    pr = lane_product<L>(pr);
    return __builtin_sqrt(fabs(pr));
}

// Two neighbouring surviving poles (d0, z0), (d1, z1): is their coupling below tol after the rotation that zeroes z0?
__device__ __forceinline__ bool poles_equal(double d0, double z0, double d1, double z1, double tol) {
    const double t2 = z0 * z0 + z1 * z1;
    return fabs((d1 - d0) * z0 * z1) <= tol * t2;
}

// ---- merges of 2 .. 64 rows, one work-group per 64 x 64 diagonal block --------------------------------------------
// 512 threads: 8 lanes per index. All arrays of the block in LDS; Q column-major.
constexpr int DCB_LD = 65;
struct DcBlockLds {
    double Q[64 * DCB_LD], U[64 * DCB_LD];
    double d[64], e[64], z[64], ds[64], zs[64], dk[64], zk[64], org[64], tau[64], zh[64], val[64];
    double rc[64], rs[64];  // rotations
    int cs[64], sv[64], col[64], ra[64], rb[64];
    int K[64], nrot[64];    // per sub-problem (indexed by its base)
    int any;
};

__global__ __launch_bounds__(512, 1) void dc_block_kernel(const double* __restrict__ dT, const double* __restrict__ eT, int N,
                                                          double* __restrict__ dO, double* __restrict__ Z,
                                                          long long* __restrict__ xch) {
    // the exchange buffers of the reduction that has just ended, ready for the next one
    if (xch)
        for (int q = blockIdx.x * 512 + threadIdx.x; q < 6 * N; q += gridDim.x * 512) xch[q] = -1LL;
    extern __shared__ char dc_lds[];
    DcBlockLds& S = *reinterpret_cast<DcBlockLds*>(dc_lds);
    const int tid = threadIdx.x, i = tid >> 3, l = tid & 7;
    const int b0 = blockIdx.x * 64;
    const double tol = dc_tolerance(dT, eT, N, tid & 63);
    if (l == 0) {
        const int g = b0 + i;
        const double e0 = g > 0 ? fabs(finite_or_zero(eT[g - 1])) : 0.0;
        const double e1 = finite_or_zero(eT[g]);
        S.e[i] = e1;
        S.d[i] = finite_or_zero(dT[g]) - e0 - fabs(e1);  // every cut is torn: both its neighbours lose |e|
    }
    for (int r = l; r < 64; r += 8) S.Q[i * DCB_LD + r] = r == i ? 1.0 : 0.0;
    __syncthreads();

    for (int m = 2; m <= 64; m *= 2) {
        const int half = m >> 1, base = i & ~(m - 1), li = i & (m - 1);
        const double ec = S.e[base + half - 1], rho = fabs(ec);
        const double di = S.d[i];
        double zi;
        if (li < half) zi = S.Q[i * DCB_LD + base + half - 1];
        else zi = ec < 0.0 ? -S.Q[i * DCB_LD + base + half] : S.Q[i * DCB_LD + base + half];
        zi = finite_or_zero(zi);
        int cnt = 0;
        for (int j = l; j < m; j += 8) {
            const double x = S.d[base + j];
            cnt += (x < di || (x == di && j < li)) ? 1 : 0;
        }
        cnt = lane_sum_i<8>(cnt);
        if (l == 0) {
            S.ds[base + cnt] = di;
            S.zs[base + cnt] = zi;
            S.cs[base + cnt] = i;
        }
        if (tid == 0) S.any = 0;
        __syncthreads();
        // survivors in order, then the deflated
        bool live = rho * fabs(S.zs[i]) > tol;
        int before = 0, K = 0;
        for (int j = l; j < m; j += 8) {
            const int f = rho * fabs(S.zs[base + j]) > tol ? 1 : 0;
            K += f;
            before += j < li ? f : 0;
        }
        before = lane_sum_i<8>(before);
        K = lane_sum_i<8>(K);
        if (l == 0) {
            S.sv[base + (live ? before : K + li - before)] = i;
            if (li == 0) S.K[base] = K;
        }
        __syncthreads();
        if (l == 0 && li + 1 < K) {
            const int s0 = S.sv[i], s1 = S.sv[i + 1];
            if (poles_equal(S.ds[s0], S.zs[s0], S.ds[s1], S.zs[s1], tol)) S.any = 1;
        }
        __syncthreads();
        if (S.any) {  // rare: walk the survivors in order, rotate equal poles together
            if (tid < 64 && (tid & (m - 1)) == 0) {
                const int bb = tid, Kb = S.K[bb];
                int nk = 0, nr = 0, nd = 0, pj = -1;
                // (col is free here: survivors are collected there, the deflated in ra's tail via a second list)
                for (int q = 0; q < Kb; ++q) {
                    const int nj = S.sv[bb + q];
                    if (pj < 0) {
                        pj = nj;
                        continue;
                    }
                    const double z0 = S.zs[pj], z1 = S.zs[nj];
                    if (poles_equal(S.ds[pj], z0, S.ds[nj], z1, tol)) {
                        const double t = __builtin_sqrt(z0 * z0 + z1 * z1), c = z1 / t, s = -z0 / t;
                        const double d0 = S.ds[pj], d1 = S.ds[nj];
                        S.zs[nj] = t;
                        S.zs[pj] = 0.0;
                        S.ds[pj] = d0 * c * c + d1 * s * s;
                        S.ds[nj] = d0 * s * s + d1 * c * c;
                        S.ra[bb + nr] = S.cs[pj];
                        S.rb[bb + nr] = S.cs[nj];
                        S.rc[bb + nr] = c;
                        S.rs[bb + nr] = s;
                        ++nr;
                        S.col[bb + m - 1 - nd++] = pj;  // deflated, collected from the end
                        pj = nj;
                    } else {
                        S.col[bb + nk++] = pj;
                        pj = nj;
                    }
                }
                if (pj >= 0) S.col[bb + nk++] = pj;
                // nk + nd == Kb; entries Kb .. m-1 of sv stay deflated
                for (int q = 0; q < nk; ++q) S.sv[bb + q] = S.col[bb + q];
                for (int q = 0; q < nd; ++q) S.sv[bb + nk + q] = S.col[bb + m - 1 - q];
                S.K[bb] = nk;
                S.nrot[bb] = nr;
            }
            __syncthreads();
            if (l == 0) {
                const int nr = S.nrot[base];
                for (int q = 0; q < nr; ++q) {
                    double* A = S.Q + S.ra[base + q] * DCB_LD + i;
                    double* B = S.Q + S.rb[base + q] * DCB_LD + i;
                    const double a = *A, b = *B, c = S.rc[base + q], s = S.rs[base + q];
                    *A = c * a + s * b;
                    *B = c * b - s * a;
                }
            }
            K = S.K[base];
            __syncthreads();
        }
        // compact arrays in the order of sv
        const int sq = S.sv[i];
        if (l == 0) {
            S.dk[i] = S.ds[sq];
            S.zk[i] = S.zs[sq];
            S.col[i] = S.cs[sq];
        }
        __syncthreads();
        double dj[8], zj[8];
        double zsum = 0.0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int j = l + 8 * e;
            const bool on = j < K;
            dj[e] = on ? S.dk[base + j] : 1e30;
            const double z = on ? S.zk[base + j] : 0.0;
            zj[e] = rho * z * z;
            zsum += zj[e];
        }
        zsum = lane_sum<8>(zsum);
        double org = 0.0, tau = 0.0, val = S.dk[i];
        if (li < K) {
            secular_root<8>(K, li, l, dj, zj, S.dk[i], li + 1 < K ? S.dk[i + 1] : 0.0, zsum, org, tau);
            val = org + tau;
            val = finite_or_zero(val);
        }
        if (l == 0) {
            S.org[i] = org;
            S.tau[i] = tau;
            S.val[i] = val;
        }
        __syncthreads();
        double og[8], ta[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int j = l + 8 * e;
            og[e] = j < K ? S.org[base + j] : 0.0;
            ta[e] = j < K ? S.tau[base + j] : 0.0;
        }
        if (li < K) {
            const double zz = secular_z<8>(K, li, l, S.dk[i], dj, og, ta);
            if (l == 0) S.zh[i] = __builtin_copysign(zz, S.zk[i]);
        }
        int np = 0;
        for (int j = l; j < m; j += 8) {
            const double x = S.val[base + j];
            np += (x < val || (x == val && j < li)) ? 1 : 0;
        }
        np = lane_sum_i<8>(np);
        __syncthreads();
        if (li < K) {
            double u[8], nn = 0.0;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int j = l + 8 * e;
                u[e] = j < K ? S.zh[base + j] * rcp64((dj[e] - org) - tau) : 0.0;
                nn = __builtin_fma(u[e], u[e], nn);
            }
            nn = rcp64(__builtin_sqrt(lane_sum<8>(nn)));
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int j = l + 8 * e;
                if (j < K) S.U[i * DCB_LD + j] = u[e] * nn;
            }
        }
        __syncthreads();
        double out[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) out[r] = 0.0;
        const int nr8 = (m + 7) >> 3;
        if (li < K) {
            for (int j = 0; j < K; ++j) {
                const double u = S.U[i * DCB_LD + j];
                const double* qc = S.Q + S.col[base + j] * DCB_LD + base + l;
#pragma unroll
                for (int r = 0; r < 8; ++r)
                    if (r < nr8 && l + 8 * r < m) out[r] = __builtin_fma(qc[8 * r], u, out[r]);
            }
        } else {
            const double* qc = S.Q + S.col[i] * DCB_LD + base + l;
#pragma unroll
            for (int r = 0; r < 8; ++r)
                if (r < nr8 && l + 8 * r < m) out[r] = qc[8 * r];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 8; ++r)
            if (r < nr8 && l + 8 * r < m) S.Q[(base + np) * DCB_LD + base + l + 8 * r] = out[r];
        if (l == 0) S.d[base + np] = val;
        __syncthreads();
    }
    if (l == 0) dO[b0 + i] = S.d[i];
    for (int c = tid >> 6; c < 64; c += 8) Z[(int64_t)(b0 + c) * N + b0 + (tid & 63)] = S.Q[c * DCB_LD + (tid & 63)];
}

// ---- merges of m = 128, 256, 512 rows -----------------------------------------------------------------------------
// Work arrays (N each, sub-problem at its base): dk, zk (poles and z of the survivors, then the deflated), col (their
// columns of Z), half (indices of the survivors that live in the left half, then those in the right half), org, tau,
// zh, val, npos; per sub-problem: K, k1 (survivors in the left half), dense (rotations mixed the halves).
// One work-group of 512 threads per sub-problem: order the poles, deflate.
__global__ __launch_bounds__(512) void dc_deflate_kernel(const double* __restrict__ dT, const double* __restrict__ eT, int N,
                                                         int m, const double* __restrict__ dI, double* __restrict__ Z,
                                                         DcWork w) {
    __shared__ double d[512], ds[512], zs[512];
    __shared__ int cs[512], sv[512], col[512];
    __shared__ double rc[512], rs[512];
    __shared__ int ra[512], rb[512];
    __shared__ int sK, snr, sany;
    __shared__ int wsum[8], wsum2[8];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int base = blockIdx.x * m, half = m >> 1;
    const double tol = dc_tolerance(dT, eT, N, lane);
    const double ec = finite_or_zero(eT[base + half - 1]), rho = fabs(ec);
    const bool on = tid < m;
    double di = 0.0, zi = 0.0;
    if (on) {
        di = dI[base + tid];
        d[tid] = di;
        const double* zc = Z + (int64_t)(base + tid) * N;
        zi = finite_or_zero(tid < half ? zc[base + half - 1] : (ec < 0.0 ? -zc[base + half] : zc[base + half]));
    }
    if (tid == 0) sany = 0;
    __syncthreads();
    if (on) {
        // both halves are sorted: rank = own position + position in the other half
        const int o0 = tid < half ? half : 0;
        int a = 0, b = half;  // number of entries of the other half that go before this one
        while (a < b) {
            const int mid = (a + b) >> 1;
            const double x = d[o0 + mid];
            const bool pre = x < di || (x == di && o0 == 0);
            if (pre) a = mid + 1;
            else b = mid;
        }
        const int r = (tid < half ? tid : tid - half) + a;
        ds[r] = di;
        zs[r] = zi;
        cs[r] = tid;
    }
    __syncthreads();
    const bool live = on && rho * fabs(zs[tid]) > tol;
    {
        const unsigned long long mask = __ballot(live);
        const int pre = __popcll(mask & ((1ull << lane) - 1ull));
        if (lane == 0) wsum[wave] = __popcll(mask);
        __syncthreads();
        int off = 0, tot = 0;
        for (int q = 0; q < 8; ++q) {
            off += q < wave ? wsum[q] : 0;
            tot += wsum[q];
        }
        if (on) sv[live ? off + pre : tot + tid - (off + pre)] = tid;
        if (tid == 0) {
            sK = tot;
            snr = 0;
        }
    }
    __syncthreads();
    if (tid + 1 < sK) {
        const int s0 = sv[tid], s1 = sv[tid + 1];
        if (poles_equal(ds[s0], zs[s0], ds[s1], zs[s1], tol)) sany = 1;
    }
    __syncthreads();
    if (sany) {  // rare: walk the survivors in order, rotate equal poles together
        if (tid == 0) {
            const int Kb = sK;
            int nk = 0, nr = 0, nd = 0, pj = -1;
            for (int q = 0; q < Kb; ++q) {
                const int nj = sv[q];
                if (pj < 0) {
                    pj = nj;
                    continue;
                }
                const double z0 = zs[pj], z1 = zs[nj];
                if (poles_equal(ds[pj], z0, ds[nj], z1, tol)) {
                    const double t = __builtin_sqrt(z0 * z0 + z1 * z1), c = z1 / t, s = -z0 / t;
                    const double d0 = ds[pj], d1 = ds[nj];
                    zs[nj] = t;
                    zs[pj] = 0.0;
                    ds[pj] = d0 * c * c + d1 * s * s;
                    ds[nj] = d0 * s * s + d1 * c * c;
                    ra[nr] = cs[pj];
                    rb[nr] = cs[nj];
                    rc[nr] = c;
                    rs[nr] = s;
                    ++nr;
                    col[m - 1 - nd++] = pj;
                    pj = nj;
                } else {
                    col[nk++] = pj;
                    pj = nj;
                }
            }
            if (pj >= 0) col[nk++] = pj;
            for (int q = 0; q < nk; ++q) sv[q] = col[q];
            for (int q = 0; q < nd; ++q) sv[nk + q] = col[m - 1 - q];
            sK = nk;
            snr = nr;
        }
        __syncthreads();
        // the columns become dense: clear what was not stored of them, then rotate (a thread per row)
        if (on) {
            for (int c = 0; c < m; ++c)
                if ((c < half) != (tid < half)) Z[(int64_t)(base + c) * N + base + tid] = 0.0;
            const int nr = snr;
            for (int q = 0; q < nr; ++q) {
                double* A = Z + (int64_t)(base + ra[q]) * N + base + tid;
                double* B = Z + (int64_t)(base + rb[q]) * N + base + tid;
                const double a = *A, b = *B;
                *A = rc[q] * a + rs[q] * b;
                *B = rc[q] * b - rs[q] * a;
            }
        }
        __syncthreads();
    }
    const int K = sK;
    const bool dense = snr > 0;
    const int cq = on ? cs[sv[tid]] : 0;
    const bool inl = tid < K && !dense && cq < half, inr = tid < K && !dense && cq >= half;
    {
        const unsigned long long ml = __ballot(inl), mr = __ballot(inr);
        if (lane == 0) {
            wsum[wave] = __popcll(ml);
            wsum2[wave] = __popcll(mr);
        }
        __syncthreads();
        int ol = __popcll(ml & ((1ull << lane) - 1ull)), orr = __popcll(mr & ((1ull << lane) - 1ull)), tl = 0;
        for (int q = 0; q < 8; ++q) {
            ol += q < wave ? wsum[q] : 0;
            orr += q < wave ? wsum2[q] : 0;
            tl += wsum[q];
        }
        if (inl) w.half[base + ol] = tid;
        if (inr) w.half[base + tl + orr] = tid;
        if (dense && tid < K) w.half[base + tid] = tid;
        if (tid == 0) {
            w.K[blockIdx.x] = K;
            w.k1[blockIdx.x] = tl;
            w.dense[blockIdx.x] = dense ? 1 : 0;
        }
    }
    if (on) {
        w.dk[base + tid] = ds[sv[tid]];
        w.zk[base + tid] = zs[sv[tid]];
        w.col[base + tid] = base + cq;
    }
}

// one wave per root
__global__ __launch_bounds__(256) void dc_roots_kernel(const double* __restrict__ eT, int m, DcWork w) {
    const int lane = threadIdx.x & 63;
    const int q = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int base = blockIdx.y * m;
    const int K = w.K[blockIdx.y];
    double org = 0.0, tau = 0.0, val = w.dk[base + q];
    if (q < K) {
        const double rho = fabs(finite_or_zero(eT[base + (m >> 1) - 1]));
        double dj[8], zj[8], zsum = 0.0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int j = lane + 64 * e;
            const bool on = j < K;
            dj[e] = on ? w.dk[base + j] : 1e30;
            const double z = on ? w.zk[base + j] : 0.0;
            zj[e] = rho * z * z;
            zsum += zj[e];
        }
        zsum = lane_sum<64>(zsum);
        secular_root<64>(K, q, lane, dj, zj, w.dk[base + q], q + 1 < K ? w.dk[base + q + 1] : 0.0, zsum, org, tau);
        val = finite_or_zero(org + tau);
    }
    if (lane == 0) {
        w.org[base + q] = org;
        w.tau[base + q] = tau;
        w.val[base + q] = val;
    }
}

// one wave per index: z of the merge, and the place of its eigenvalue among all
__global__ __launch_bounds__(256) void dc_weights_kernel(int m, DcWork w, double* __restrict__ dO) {
    const int lane = threadIdx.x & 63;
    const int q = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int base = blockIdx.y * m;
    const int K = w.K[blockIdx.y];
    const double val = w.val[base + q];
    int np = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int j = lane + 64 * e;
        if (j < m) {
            const double x = w.val[base + j];
            np += (x < val || (x == val && j < q)) ? 1 : 0;
        }
    }
    np = lane_sum_i<64>(np);
    double zz = 0.0;
    if (q < K) {
        double di[8], og[8], ta[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int j = lane + 64 * e;
            di[e] = j < K ? w.dk[base + j] : 0.0;
            og[e] = j < K ? w.org[base + j] : 0.0;
            ta[e] = j < K ? w.tau[base + j] : 0.0;
        }
        zz = __builtin_copysign(secular_z<64>(K, q, lane, w.dk[base + q], di, og, ta), w.zk[base + q]);
    }
    if (lane == 0) {
        w.zh[base + q] = zz;
        w.npos[base + q] = np;
        dO[base + np] = val;
    }
}

typedef double f64x4 __attribute__((ext_vector_type(4)));
// fp64 matrix-core step acc(16x16) += a(16x4) b(4x16): lane l supplies a[l%16][l/16] and b[l/16][l%16];
// acc element v of lane l is row 4v + l/16, column l%16.
__device__ __forceinline__ f64x4 mfma64(double a, double b, f64x4 acc) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
}

// Z_out(:, npos_q) = Z_in(:, survivors) u_q, u_q(j) = zh_j / (d_j - lambda_q) normalised; deflated columns are copied.
// grid (m / 32 column tiles, m / 64 row tiles, sub-problems), 256 threads; a wave owns 16 rows x 32 columns. A row tile
// of the left (right) half only meets the survivors that live there.
__global__ __launch_bounds__(256) void dc_vectors_kernel(const double* __restrict__ Zin, double* __restrict__ Zout, int N,
                                                         int m, DcWork w) {
    constexpr int KT = 32, LDA = 72, LDB = 40;
    __shared__ double As[KT * LDA], Bs[KT * LDB];
    __shared__ double inv[32];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int base = blockIdx.z * m, half = m >> 1;
    const int q0 = blockIdx.x * 32, r0 = blockIdx.y * 64;
    const int K = w.K[blockIdx.z], k1 = w.k1[blockIdx.z];
    const bool dense = w.dense[blockIdx.z] != 0;
    const bool left = r0 < half;
    const int* list = w.half + base + (dense || left ? 0 : k1);
    const int len = dense ? K : (left ? k1 : K - k1);
    if (q0 < K) {
        {   // norms of the tile's vectors: 8 lanes per column
            const int c = tid >> 3, l = tid & 7, q = q0 + c;
            double nn = 0.0;
            if (q < K) {
                const double og = w.org[base + q], ta = w.tau[base + q];
                for (int j = l; j < K; j += 8) {
                    const double u = w.zh[base + j] * rcp64((w.dk[base + j] - og) - ta);
                    nn = __builtin_fma(u, u, nn);
                }
            }
            nn = lane_sum<8>(nn);
            if (l == 0) inv[c] = nn > 0.0 ? rcp64(__builtin_sqrt(nn)) : 0.0;
        }
        const int l16 = lane & 15, lk = lane >> 4;
        f64x4 acc[2] = {f64x4{0.0, 0.0, 0.0, 0.0}, f64x4{0.0, 0.0, 0.0, 0.0}};
        for (int k0 = 0; k0 < len; k0 += KT) {
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int kk = u * 4 + wave;
                As[kk * LDA + lane] = k0 + kk < len ? Zin[(int64_t)w.col[base + list[k0 + kk]] * N + base + r0 + lane] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int e = u * 256 + tid, kk = e >> 5, c = e & 31, q = q0 + c;
                double v = 0.0;
                if (k0 + kk < len && q < K) {
                    const int j = list[k0 + kk];
                    v = w.zh[base + j] * rcp64((w.dk[base + j] - w.org[base + q]) - w.tau[base + q]) * inv[c];
                }
                Bs[kk * LDB + c] = v;
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < KT; k += 4) {
                const double av = As[(k + lk) * LDA + wave * 16 + l16];
#pragma unroll
                for (int t = 0; t < 2; ++t) acc[t] = mfma64(av, Bs[(k + lk) * LDB + t * 16 + l16], acc[t]);
            }
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int q = q0 + t * 16 + l16;
            if (q < K) {
                double* o = Zout + (int64_t)(base + w.npos[base + q]) * N + base + r0 + wave * 16 + lk;
#pragma unroll
                for (int v = 0; v < 4; ++v) o[4 * v] = acc[t][v];
            }
        }
    }
    // deflated columns of this tile
    for (int c = wave; c < 32; c += 4) {
        const int q = q0 + c;
        if (q < K) continue;
        const int src = w.col[base + q] - base;
        const bool own = dense || ((src < half) == left);
        Zout[(int64_t)(base + w.npos[base + q]) * N + base + r0 + lane] =
            own ? Zin[(int64_t)(base + src) * N + base + r0 + lane] : 0.0;
    }
}

// T = Z D Z^T: eigenvalues ascending in dI, eigenvectors in the columns of Z (buffer dc_result(N) of either).
hipError_t launch_dc(const EigWork& w, int N, hipStream_t st) {
    if (hipError_t e = ensure_dynamic_lds((const void*)dc_block_kernel, (int)sizeof(DcBlockLds)); e != hipSuccess) return e;
    int cur = 0;
    hipLaunchKernelGGL(dc_block_kernel, dim3(N / 64), dim3(512), sizeof(DcBlockLds), st, w.dT, w.eT, N, w.dI[0], w.Z[0],
                       w.xch);
    for (int m = 128; m <= N; m *= 2) {
        const int S = N / m;
        hipLaunchKernelGGL(dc_deflate_kernel, dim3(S), dim3(512), 0, st, w.dT, w.eT, N, m, w.dI[cur], w.Z[cur], w.dc);
        hipLaunchKernelGGL(dc_roots_kernel, dim3(m / 4, S), dim3(256), 0, st, w.eT, m, w.dc);
        hipLaunchKernelGGL(dc_weights_kernel, dim3(m / 4, S), dim3(256), 0, st, m, w.dc, w.dI[cur ^ 1]);
        hipLaunchKernelGGL(dc_vectors_kernel, dim3(m / 32, m / 64, S), dim3(256), 0, st, w.Z[cur], w.Z[cur ^ 1], N, m, w.dc);
        cur ^= 1;
    }
    return hipGetLastError();
}

}  // namespace sage
