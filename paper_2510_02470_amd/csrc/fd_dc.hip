// Eigen-decomposition T = Z D Z^T of the tridiagonal matrix fd_tridiag.hip leaves, by divide and conquer (J. Cuppen,
// Numer. Math. 36, 1981): T is torn into 1 x 1 pieces, T = diag(d) + sum of rank-one terms at the cuts, and the pieces
// are merged pairwise. A merge of two solved halves is the eigenproblem of diag(d) + rho z z^T with z made of the last
// row of the left half's eigenvectors and the first row of the right half's:
//   * entries with rho |z_i| below tol, and all but one of a group of equal poles (after a rotation of their columns),
//     are deflated: they are eigenpairs already;
//   * the other eigenvalues are the roots of the secular equation 1 + rho sum z_j^2 / (d_j - lambda) = 0, one in every
//     gap, each kept as (nearest pole, distance): an interpolation with the gap's two poles and a constant that matches the
//     function and two derivatives (C. Borges, W. Gragg, Numerical Linear Algebra and Scientific Computing, de Gruyter 1993;
//     of two derivatives where J. Bunch, C. Nielsen, D. Sorensen, Numer. Math. 31, 1978, match one on either side of the gap),
//     inside a bracket that is bisected when a step leaves it;
//   * z is recomputed from the roots (M. Gu, S. Eisenstat, SIAM J. Matrix Anal. Appl. 16, 1995), which makes the
//     eigenvectors z_j / (d_j - lambda_i) orthogonal to fp64 rounding however close the roots are.
// Merges up to 64 rows run inside one work-group per 64 x 64 block (everything in LDS); the merges above it are three
// kernels each: deflation and roots (a wave per root), z and the order of the new eigenvalues, and the products of the
// halves' eigenvectors with the merge's on the fp64 matrix cores.
// Every size, index and count derived here is clamped by construction (counts of comparisons between finite numbers), so
// non-finite input gives wrong numbers but no access out of bounds.
#include "sage_internal.h"
#include "fd_wy.h"
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

// A root of f = 1 + sum_j z_j / (d_j - lambda) (z_j = rho z_j^2 > 0, K poles ascending), the one between the neighbouring poles pi and
// pn, of weights zi and zn, or (last) the one above pn, the last: lambda = org + tau with org the nearer of the poles around it. A
// group of L lanes works on a root; lane l holds the poles l + L e, e < E (z = 0 and d = 1e30 beyond K). on: this group has a
// root (all lanes take part in the loop). It starts from the root of the two poles and a constant that stands for the others, their
// sum at the middle of the bracket (R.-C. Li, LAPACK Working Note 89, 1993). The interpolation, which matches f, f' and f'' by two poles
// and a constant (Borges and Gragg), converges cubically: a step below 1e-7 of tau is the last one. About 2.8 evaluations a root,
// 4.8 for the slowest of 64 (started at a quarter of the gap and with one pole for the last root, which came in slowest most times,
// 3.6 and 7.5). An evaluation is a chain of some 700 cycles (reciprocal, sums over L, square root, reciprocal) and 11 fp64 instructions
// a pole; a branch costs 100 cycles, so there is none but the loop's. 64 rows in all: 32 -> 30 us.
template <int L, int E>
__device__ __forceinline__ void secular_root(bool on, bool last, int K, const double (&dj)[E], const double (&zj)[E], double pi, double pn,
                                             double zi, double zn, double zsum, double& org, double& tau) {
    // The root of c + p / (di - x) + g / (dn - x), di < dn: c x^2 - a x + b = 0. Its error shrinks with the step, which is below 1e-7
    // of t when it is the last, so a step needs few digits: the square root is the hardware's estimate with one correction, and so is
    // the quotient. (A fraction, num / den.)
    auto interpolate = [last](double c, double di, double dn, double p, double g, double& num, double& den) __attribute__((always_inline)) {
        const double a = __builtin_fma(c, di + dn, p + g), b = __builtin_fma(c * di, dn, __builtin_fma(p, dn, g * di));
        const double disc = fmax(__builtin_fma(a, a, -4.0 * c * b), 1e-280);
        const double ys = __builtin_amdgcn_rsq(disc), r = disc * ys;
        const double sq = __builtin_fma(__builtin_fma(-r, r, disc), 0.5 * ys, r);
        const double h = 0.5 * (a + __builtin_copysign(sq, a));
        const bool first = (a > 0.0) != last;  // of the two roots, the one between the poles or the one above them
        num = first ? b : h;
        den = first ? h : c;
    };
    auto inverse = [](double x) __attribute__((always_inline)) {
        const double y = __builtin_amdgcn_rcp(x);
        return __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
    };
    double num, den;
    const double gap = pn - pi, mid = 0.5 * (last ? zsum : gap), base = last ? pn : pi;
    double f0 = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) f0 = __builtin_fma(zj[e], rcp64((dj[e] - base) - mid), f0);
    f0 = 1.0 + lane_sum<L>(f0);
    const bool left = f0 >= 0.0;
    org = left ? base : pn;
    double lo = left ? 0.0 : (last ? mid : -mid);
    double hi = left ? mid : (last ? zsum * (1.0 + 4.0 * DC_EPS) : 0.0);
    const double dli = pi - org, dln = pn - org, tol = 0.0625 * DC_EPS * K;
    const double c0 = __builtin_fma(-zi, rcp64((pi - base) - mid), __builtin_fma(-zn, rcp64((pn - base) - mid), f0));
    interpolate(c0, dli, dln, zi, zn, num, den);
    const double t0 = num * inverse(den);
    double t = ((t0 > lo) & (t0 < hi)) ? t0 : 0.5 * (lo + hi);
    double dl[E];  // distance of the poles
#pragma unroll
    for (int e = 0; e < E; ++e) dl[e] = dj[e] - org;
    const double rgap = rcp64(gap);
    for (int it = 0; it < 60; ++it) {
        double f = 0.0, f1 = 0.0, f2 = 0.0;  // f - 1, f', f'' / 2
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const double inv = rcp64(dl[e] - t), u = zj[e] * inv, u1 = u * inv;
            f += u;
            f1 += u1;
            f2 = __builtin_fma(u1, inv, f2);
        }
        lane_sum3<L>(f, f1, f2);
        f += 1.0;
        lo = f < 0.0 ? t : lo;  // (t lies inside the bracket)
        hi = f < 0.0 ? hi : t;
        // c + P di^2 / (di - x) + G dn^2 / (dn - x) = 0 with P + G = f', P / di + G / dn = f'' / 2. The last root is above both poles,
        // where the difference of P and G leaves less of the digits: once f is small its steps are those of one pole, pn, x = dn +
        // f' dn^2 / (f - dn f') (last roots of 4 to 64 poles: mean error 0.76 ulp against 1.24, for 0.1 evaluations).
        const double di = dli - t, dn = dln - t;
        const double P = di * rgap * __builtin_fma(f2, dn, -f1), G = f1 - P;
        const double Pd = P * di, Gd = G * dn;
        interpolate(f - Pd - Gd, di, dn, Pd * di, Gd * dn, num, den);
        const double fd = f1 * dn;
        const bool one = last & !(fabs(f) > 0.01);
        num = one ? fd * dn : num;
        den = one ? f - fd : den;
        const double x = __builtin_fma(num, inverse(den), one ? dn : 0.0), step = t + x;
        // (false for NaN; the bracket lies between the poles. A small step that leaves it is rounding: t is the root.)
        const bool in = (step > lo) & (step < hi), small = fabs(x) <= 1e-7 * fabs(step);
        const double half = 0.5 * (lo + hi);
        const bool end = small | !(hi - lo > fabs(half) * DC_EPS);
        // f is rounding: an eighth of what its terms may leave, their magnitudes taken from the two poles of the interpolation (of
        // the last root's they sum up to 1)
        const bool there = !(fabs(f) > tol * (1.0 + (last ? 1.0 : fabs(Pd) + fabs(Gd))));
        double tn = (small | there) ? t : half;
        tn = in ? step : tn;
        t = on ? tn : t;
        on = on & !(end | there);
        if (!__any(on)) break;
    }
    tau = t;
}

// The lower one of the two poles next to root q of K: those around it, or the last two. (If there is one only, it is the upper one, with
// none of weight below it.)
__device__ __forceinline__ int lower_pole(int q, int K) { return max(min(q, K - 2), 0); }

// |z_j| of the rank-one problem whose eigenvalues are exactly the computed roots: the product over i != j of
// (lambda_i - d_j) / (d_i - d_j), times (lambda_j - d_j). Lane l holds roots l + L e.
template <int L, int E>
__device__ __forceinline__ double secular_z(int K, int j, int l, double dj, const double (&di)[E], const double (&org)[E],
                                            const double (&tau)[E]) {
    double pr = 1.0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = l + L * e;
        const double num = (org[e] - dj) + tau[e];
        const double f = i == j ? num : num * rcp64(di[e] - dj);
        pr *= i < K ? f : 1.0;
    }
    pr = lane_product<L>(pr);
    return __builtin_sqrt(fabs(pr));
}

// Two neighbouring surviving poles (d0, z0), (d1, z1): is their coupling below tol after the rotation that zeroes z0?
__device__ __forceinline__ bool poles_equal(double d0, double z0, double d1, double z1, double tol) {
    const double t2 = z0 * z0 + z1 * z1;
    return fabs((d1 - d0) * z0 * z1) <= tol * t2;
}

typedef double f64x4 __attribute__((ext_vector_type(4)));
// fp64 matrix-core step acc(16x16) += a(16x4) b(4x16): lane l supplies a[l%16][l/16] and b[l/16][l%16];
// acc element v of lane l is row 4v + l/16, column l%16.
__device__ __forceinline__ f64x4 mfma64(double a, double b, f64x4 acc) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
}

// ---- pairs in closed form and merges of 4 .. 64 rows, one work-group per 64 x 64 diagonal block ----------------------
// Merges up to 16 rows: 16 rows and four lanes per index to each of the first four waves, no barrier (dc_level_wave). Those of 32
// and 64: 512 threads, 8 lanes per index, a sub-problem of M rows per 8 M threads. All arrays of the block in LDS; Q column-major.
// A merge is a chain of short phases; half the time goes into the roots, which is why their loops are
// unrolled to what M needs, and the products of 16 rows and more run on the matrix cores (in scalar code, bound by LDS
// reads, the last product alone took 17 us). A merge of 4, 8, 16, 32, 64 rows takes 6.0, 6.7, 8.5, 13 and 15 thousand cycles (the first three
// with barriers between their phases: 8.3, 9.4 and 11.5). 28 us in all (38 with the roots' cases told apart by branches and quadratic
// steps; 30.7 with barriers in all merges), against 104 us for one loop over all sizes.
constexpr int DCB_LD = 65;   // columns of Q
constexpr int DCB_LDU = 68;  // columns of U: the 16 columns x 4 rows of a matrix-core operand fall on distinct banks
struct DcBlockLds {
    double Q[64 * DCB_LD], U[64 * DCB_LDU];
    double d[64], e[64], ds[64], zs[64], dk[64], zk[64], org[64], tau[64], zh[64], val[64];
    double rc[64], rs[64], td[64];  // rotations; poles they deflate
    int cs[64], col[64], np[64], ra[64], rb[64], tc[64];
    int K[64], nrot[64];            // per sub-problem (indexed by its base)
    int lst[64];                    // entries (in dk order) whose columns belong to the left half, then the others
    unsigned char mask[8], maskl[8];  // surviving entries, entries of the left half, in order
    int any;
};

// The K survivors of the sub-problem at bb, in order: equal poles are rotated together, one of each group stays. nrot rotations are left to be
// applied to the columns.
__device__ __forceinline__ void rotate_equal_poles(DcBlockLds& S, int bb, int K, double tol) {
    int nk = 0, nr = 0, pc = -1;
    double pd = 0.0, pz = 0.0;
    for (int q = 0; q < K; ++q) {
        double nd = S.dk[bb + q], nz = S.zk[bb + q];
        const int nc = S.col[bb + q];
        if (pc >= 0) {
            if (poles_equal(pd, pz, nd, nz, tol)) {
                const double t = __builtin_sqrt(pz * pz + nz * nz), c = nz / t, s = -pz / t;
                S.td[bb + nr] = pd * c * c + nd * s * s;
                S.tc[bb + nr] = pc;
                nd = pd * s * s + nd * c * c;
                nz = t;
                S.ra[bb + nr] = pc;
                S.rb[bb + nr] = nc;
                S.rc[bb + nr] = c;
                S.rs[bb + nr] = s;
                ++nr;
            } else {
                S.dk[bb + nk] = pd;
                S.zk[bb + nk] = pz;
                S.col[bb + nk] = pc;
                ++nk;
            }
        }
        pd = nd;
        pz = nz;
        pc = nc;
    }
    if (pc >= 0) {
        S.dk[bb + nk] = pd;
        S.zk[bb + nk] = pz;
        S.col[bb + nk] = pc;
        ++nk;
    }
    for (int q = 0; q < nr; ++q) {  // nk + nr == K
        S.dk[bb + nk + q] = S.td[bb + q];
        S.zk[bb + nk + q] = 0.0;
        S.col[bb + nk + q] = S.tc[bb + q];
    }
    S.K[bb] = nk;
    S.nrot[bb] = nr;
}
// ... and they are, in row i
__device__ __forceinline__ void rotate_columns(DcBlockLds& S, int bb, int i) {
    const int nr = S.nrot[bb];
    for (int q = 0; q < nr; ++q) {
        double* A = S.Q + S.ra[bb + q] * DCB_LD + i;
        double* B = S.Q + S.rb[bb + q] * DCB_LD + i;
        const double a = *A, b = *B, c = S.rc[bb + q], s = S.rs[bb + q];
        *A = c * a + s * b;
        *B = c * b - s * a;
    }
}

template <int M, bool WIDE>
__device__ __forceinline__ void dc_level(DcBlockLds& S, int tid, double tol) {
    static_assert(M == 32 || M == 64, "smaller ones: dc_level_wave");
    constexpr int H = M / 2, E = M / 8, EH = H / 8;
    const int i = tid >> 3, l = tid & 7;
    const int base = i & ~(M - 1), li = i & (M - 1);
    const double ec = S.e[base + H - 1], rho = fabs(ec);
    {
        const double di = S.d[i];
        double zi = li < H ? S.Q[i * DCB_LD + base + H - 1] : S.Q[i * DCB_LD + base + H];
        zi = finite_or_zero(li >= H && ec < 0.0 ? -zi : zi);
        // both halves are sorted: rank = own position + entries of the other half that go before
        const int o = base + (li < H ? H : 0);
        int cnt = 0;
#pragma unroll
        for (int e = 0; e < EH; ++e) {
            const int j = l + 8 * e;
            const double x = S.d[o + j];
            cnt += (x < di || (x == di && li >= H)) ? 1 : 0;
        }
        cnt = lane_sum_i<8>(cnt) + (li < H ? li : li - H);
        if (l == 0) {
            S.ds[base + cnt] = di;
            S.zs[base + cnt] = zi;
            S.cs[base + cnt] = i;
        }
    }
    if (tid == 0) S.any = 0;
    __syncthreads();
    // survivors in order, then the deflated
    const double dsi = S.ds[i], zsi = S.zs[i];
    const int csi = S.cs[i];
    const bool live = rho * fabs(zsi) > tol;
    {
        const unsigned long long b = __ballot(live) & 0x0101010101010101ull;  // bit 8 q: index 8 wave + q
        const unsigned long long c = __ballot((csi & (M - 1)) < H) & 0x0101010101010101ull;
        if ((tid & 63) == 0) {
            S.mask[tid >> 6] = (unsigned char)((b * 0x0102040810204080ull) >> 56);
            S.maskl[tid >> 6] = (unsigned char)((c * 0x0102040810204080ull) >> 56);
        }
    }
    __syncthreads();
    const unsigned long long all = *reinterpret_cast<const unsigned long long*>(S.mask);
    const unsigned long long sub = M == 64 ? all : (all >> base) & ((1ull << (M & 63)) - 1ull);
    int K = __popcll(sub);
    {
        const int before = __popcll(sub & ((1ull << li) - 1ull));
        const int pos = live ? before : K + li - before;
        if (l == 1) {
            const unsigned long long alll = *reinterpret_cast<const unsigned long long*>(S.maskl);
            const unsigned long long ones = M == 64 ? ~0ull : (1ull << (M & 63)) - 1ull, below = (1ull << li) - 1ull;
            const unsigned long long subl = (M == 64 ? alll : alll >> base) & ones;
            const bool left = (csi & (M - 1)) < H;
            const unsigned long long side = left ? subl : ~subl & ones;  // entries of this one's half
            const int r = live ? __popcll(side & sub & below) : __popcll(side & sub) + __popcll(side & ~sub & below);
            S.lst[base + (left ? r : H + r)] = pos;
        }
        if (l == 0) {
            S.dk[base + pos] = dsi;
            S.zk[base + pos] = zsi;
            S.col[base + pos] = csi;
            if (li == 0) S.K[base] = K;
            const unsigned long long after = li == 63 ? 0ull : sub >> (li + 1);
            if (live && after) {
                const int nx = base + li + 1 + __builtin_ctzll(after);
                if (poles_equal(dsi, zsi, S.ds[nx], S.zs[nx], tol)) S.any = 1;
            }
        }
    }
    __syncthreads();
    if (S.any) {  // rare: walk the survivors in order, rotate equal poles together
        if (tid < 64 && (tid & (M - 1)) == 0) rotate_equal_poles(S, tid, S.K[tid], tol);
        __syncthreads();
        if (l == 0) rotate_columns(S, base, i);
        K = S.K[base];
        __syncthreads();
    }
    const double dki = S.dk[i];
    // Four lanes a root: half the instructions of a step do not depend on the number of poles, and two waves per SIMD issue no
    // more of them than one. (64 rows: 9,850 cycles against 11,450 with eight lanes; those where registers are short.)
    constexpr int LR = M >= 64 && !WIDE ? 8 : 4, ER = M / LR;
    if (LR == 8 || tid < 256) {
        const int ir = tid / LR, lr = tid & (LR - 1), br = ir & ~(M - 1), lir = ir & (M - 1);
        const int Kr = LR == 8 ? K : S.K[br];
        const double dkr = S.dk[ir], rhor = fabs(S.e[br + H - 1]);
        double dj[ER], zj[ER], zsum = 0.0;
#pragma unroll
        for (int e = 0; e < ER; ++e) {
            const int j = lr + LR * e;
            const bool on = j < Kr;
            dj[e] = on ? S.dk[br + j] : 1e30;
            const double z = on ? S.zk[br + j] : 0.0;
            zj[e] = rhor * z * z;
            zsum += zj[e];
        }
        zsum = lane_sum<LR>(zsum);
        double org, tau;
        const bool has = lir < Kr;
        const int ip = br + lower_pole(lir, Kr);
        const double pn = S.dk[ip + (Kr > 1)], zi = S.zk[ip], zn = S.zk[ip + (Kr > 1)];
        secular_root<LR, ER>(has, lir >= Kr - 1, Kr, dj, zj, Kr > 1 ? S.dk[ip] : pn - 1.0, pn, Kr > 1 ? rhor * zi * zi : 0.0, rhor * zn * zn,
                             zsum, org, tau);
        const double val = has ? finite_or_zero(org + tau) : dkr;
        if (lr == 0) {
            S.org[ir] = org;
            S.tau[ir] = tau;
            S.val[ir] = val;
        }
    }
    __syncthreads();
    const double org = S.org[i], tau = S.tau[i], val = S.val[i];
    double dj[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int j = l + 8 * e;
        dj[e] = j < K ? S.dk[base + j] : 1e30;
    }
    {
        double og[E], ta[E];
        int np = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int j = l + 8 * e, jj = base + j;
            og[e] = S.org[jj];
            ta[e] = S.tau[jj];
            const double x = S.val[jj];
            np += x < val || (x == val && j < li) ? 1 : 0;
        }
        np = lane_sum_i<8>(np);
        const double zz = secular_z<8, E>(K, li, l, dki, dj, og, ta);
        if (l == 0) {
            S.zh[i] = __builtin_copysign(zz, S.zk[i]);
            S.np[i] = base + np;
            S.d[base + np] = val;
        }
    }
    __syncthreads();
    {
        double u[E], nn = 0.0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int j = l + 8 * e;
            u[e] = j < K ? S.zh[base + j] * rcp64((dj[e] - org) - tau) : 0.0;
            nn = __builtin_fma(u[e], u[e], nn);
        }
        nn = lane_sum<8>(nn);
        nn = rcp64(__builtin_sqrt(nn));
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int j = l + 8 * e;
            S.U[i * DCB_LDU + j] = li < K ? u[e] * nn : (j == li ? 1.0 : 0.0);
        }
    }
    __syncthreads();
    constexpr int T = M / 16, TILES = (64 / M) * T * T, PER = TILES > 8 ? TILES / 8 : 1;
    // The columns of Q are still those of the halves: a row tile meets the H of its own half, unless rotations mixed them.
    const bool dense = S.any != 0;
    const int wave = tid >> 6, lane = tid & 63, l16 = lane & 15, lk = lane >> 4;
    f64x4 acc[PER];
#pragma unroll
    for (int g = 0; g < PER; ++g) {
        acc[g] = f64x4{0.0, 0.0, 0.0, 0.0};
        const int t = wave + 8 * g;
        if (t < TILES) {
            const int sb = (t / (T * T)) * M, r0 = sb + ((t / T) % T) * 16, c0 = sb + (t % T) * 16;
            if (!dense) {
                const int half = (r0 - sb) & H;
#pragma unroll
                for (int k = 0; k < H; k += 4) {
                    const int j = S.lst[sb + half + k + lk];
                    const double av = S.Q[S.col[sb + j] * DCB_LD + r0 + l16];
                    acc[g] = mfma64(av, S.U[(c0 + l16) * DCB_LDU + j], acc[g]);
                }
            } else {
#pragma unroll 4
                for (int k = 0; k < M; k += 4) {
                    const double av = S.Q[S.col[sb + k + lk] * DCB_LD + r0 + l16];
                    acc[g] = mfma64(av, S.U[(c0 + l16) * DCB_LDU + k + lk], acc[g]);
                }
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < PER; ++g) {
        const int t = wave + 8 * g;
        if (t < TILES) {
            const int sb = (t / (T * T)) * M, r0 = sb + ((t / T) % T) * 16, c0 = sb + (t % T) * 16;
            double* o = S.Q + S.np[c0 + l16] * DCB_LD + r0 + lk;
#pragma unroll
            for (int v = 0; v < 4; ++v) o[4 * v] = acc[g][v];
        }
    }
    __syncthreads();
}

// A merge of 4, 8 or 16 rows by a wave, the first four waves 16 rows of the block each, four lanes an index: the steps of dc_level, but
// nothing goes from wave to wave, so there is no barrier. (The LDS takes a wave's instructions in their order.) Rotations are rare.
__device__ __forceinline__ void wave_order() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}
template <int M>
__device__ __forceinline__ void dc_level_wave(DcBlockLds& S, int tid, double tol) {
    static_assert(M == 4 || M == 8 || M == 16, "no more than a wave's rows");
    constexpr int H = M / 2, E = M / 4, EH = H > 4 ? H / 4 : 1;
    const int i = tid >> 2, l = tid & 3;
    const int base = i & ~(M - 1), li = i & (M - 1);
    const double ec = S.e[base + H - 1], rho = fabs(ec);
    {
        const double di = S.d[i];
        double zi = li < H ? S.Q[i * DCB_LD + base + H - 1] : S.Q[i * DCB_LD + base + H];
        zi = finite_or_zero(li >= H && ec < 0.0 ? -zi : zi);
        const int o = base + (li < H ? H : 0);
        int cnt = 0;
#pragma unroll
        for (int e = 0; e < EH; ++e) {
            const int j = l + 4 * e;
            const double x = S.d[o + (j & (H - 1))];
            cnt += j < H && (x < di || (x == di && li >= H)) ? 1 : 0;
        }
        cnt = lane_sum_i<4>(cnt) + (li < H ? li : li - H);
        if (l == 0) {
            S.ds[base + cnt] = di;
            S.zs[base + cnt] = zi;
            S.cs[base + cnt] = i;
        }
    }
    wave_order();
    const double dsi = S.ds[i], zsi = S.zs[i];
    const int csi = S.cs[i];
    const bool live = rho * fabs(zsi) > tol;
    const unsigned long long all = __ballot(live) & 0x1111111111111111ull;  // bit 4 q: index 16 wave + q
    const unsigned long long sub = M == 16 ? all : (all >> (4 * (base & 15))) & ((1ull << ((4 * M) & 63)) - 1ull);
    int K = __popcll(sub);
    bool equal = false;
    {
        const int before = __popcll(sub & ((1ull << (4 * li)) - 1ull));
        const int pos = live ? before : K + li - before;
        const unsigned long long after = li == 15 ? 0ull : sub >> (4 * (li + 1));
        if (live && after) {
            const int nx = base + li + 1 + (__builtin_ctzll(after) >> 2);
            equal = poles_equal(dsi, zsi, S.ds[nx], S.zs[nx], tol);
        }
        if (l == 0) {
            S.dk[base + pos] = dsi;
            S.zk[base + pos] = zsi;
            S.col[base + pos] = csi;
        }
    }
    wave_order();
    if (__any(equal)) {
        if (l == 0 && li == 0) rotate_equal_poles(S, base, K, tol);
        wave_order();
        if (l == 0) rotate_columns(S, base, i);
        K = S.K[base];
        wave_order();
    }
    double org, tau, val, dj[E];
    const double dki = S.dk[i];
    {
        double rj[E], zj[E], zsum = 0.0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int j = l + 4 * e;
            const bool on = j < K;
            dj[e] = rj[e] = on ? S.dk[base + j] : 1e30;
            const double z = on ? S.zk[base + j] : 0.0;
            zj[e] = rho * z * z;
            zsum += zj[e];
        }
        zsum = lane_sum<4>(zsum);
        const bool has = li < K;
        const int ip = base + lower_pole(li, K);
        const double pn = S.dk[ip + (K > 1)], zi = S.zk[ip], zn = S.zk[ip + (K > 1)];
        secular_root<4, E>(has, li >= K - 1, K, rj, zj, K > 1 ? S.dk[ip] : pn - 1.0, pn, K > 1 ? rho * zi * zi : 0.0, rho * zn * zn, zsum, org, tau);
        val = has ? finite_or_zero(org + tau) : dki;
        if (l == 0) {
            S.org[i] = org;
            S.tau[i] = tau;
            S.val[i] = val;
        }
    }
    wave_order();
    {
        double og[E], ta[E];
        int np = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int j = l + 4 * e;
            og[e] = S.org[base + j];
            ta[e] = S.tau[base + j];
            const double x = S.val[base + j];
            np += x < val || (x == val && j < li) ? 1 : 0;
        }
        np = lane_sum_i<4>(np);
        const double zz = secular_z<4, E>(K, li, l, dki, dj, og, ta);
        if (l == 0) {
            S.zh[i] = __builtin_copysign(zz, S.zk[i]);
            S.np[i] = base + np;
            S.d[base + np] = val;
        }
    }
    wave_order();
    {
        double u[E], nn = 0.0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int j = l + 4 * e;
            u[e] = j < K ? S.zh[base + j] * rcp64((dj[e] - org) - tau) : 0.0;
            nn = __builtin_fma(u[e], u[e], nn);
        }
        nn = lane_sum<4>(nn);
        nn = rcp64(__builtin_sqrt(nn));
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int j = l + 4 * e;
            S.U[i * DCB_LDU + j] = li < K ? u[e] * nn : (j == li ? 1.0 : 0.0);
        }
    }
    wave_order();
    if constexpr (M == 16) {
        const int lane = tid & 63, l16 = lane & 15, lk = lane >> 4;
        f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < M; k += 4) {
            const double av = S.Q[S.col[(tid >> 6) * 16 + k + lk] * DCB_LD + (tid >> 6) * 16 + l16];
            acc = mfma64(av, S.U[((tid >> 6) * 16 + l16) * DCB_LDU + k + lk], acc);
        }
        wave_order();
        double* o = S.Q + S.np[(tid >> 6) * 16 + l16] * DCB_LD + (tid >> 6) * 16 + lk;
#pragma unroll
        for (int v = 0; v < 4; ++v) o[4 * v] = acc[v];
    } else {
        double out[E];
#pragma unroll
        for (int e = 0; e < E; ++e) out[e] = 0.0;
#pragma unroll
        for (int j = 0; j < M; ++j) {
            const double uj = S.U[i * DCB_LDU + j];
            const double* q = S.Q + S.col[base + j] * DCB_LD + base + l;
#pragma unroll
            for (int e = 0; e < E; ++e) out[e] = __builtin_fma(q[4 * e], uj, out[e]);
        }
        wave_order();
        double* o = S.Q + S.np[i] * DCB_LD + base + l;
#pragma unroll
        for (int e = 0; e < E; ++e) o[4 * e] = out[e];
    }
    wave_order();
}

// A work-group per diagonal block of 64. WITH_WY (N = 64): the work-group after it forms the triangular factors of the
// reduction's blocks of reflectors meanwhile (a wave each; wy_factor), which the back-transformation needs; for larger N that
// is done beside the first merge's roots (dc_roots_kernel). Without it the kernel stays below 128 registers and fits on a
// CU beside a work-group of the Gram kernel that runs on the side stream (it waited 400 us for one to end otherwise).
template <bool WITH_WY>
__global__ __launch_bounds__(512, WITH_WY ? 1 : 4) void dc_block_kernel(const double* __restrict__ dT, const double* __restrict__ eT,
                                                          int N, double* __restrict__ dO, double* __restrict__ Z,
                                                          const double* __restrict__ V, const double* __restrict__ tauT,
                                                          int n, double* __restrict__ Tw, double* __restrict__ xch,
                                                          unsigned* __restrict__ claim) {
    if (!WITH_WY && blockIdx.x == 0) {  // the reduction before this is over: empty its exchange for the next
        for (int e = threadIdx.x; e < 4 * N; e += 512) reinterpret_cast<u32x4*>(xch)[e] = u32x4{~0u, ~0u, ~0u, ~0u};
        if (threadIdx.x >= 1 && threadIdx.x <= 3) claim[threadIdx.x] = 0u;
    }
    if (WITH_WY && blockIdx.x == 1) {
        const int b = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        if (b * WY <= n - 2) wy_factor<1>(V, tauT, b, n, threadIdx.x & 63, Tw);
        return;
    }
    __builtin_amdgcn_s_setprio(3);  // (96 rows beside a Gram launch of the side stream: 53 -> 43 us)
    extern __shared__ char dc_lds[];
    DcBlockLds& S = *reinterpret_cast<DcBlockLds*>(dc_lds);
    const int tid = threadIdx.x, i = tid >> 3, l = tid & 7;
    const int b0 = blockIdx.x * 64;
    const double tol = dc_tolerance(dT, eT, N, tid & 63);
    for (int r = l; r < 64; r += 8) S.Q[i * DCB_LD + r] = 0.0;
    __syncthreads();
    if (l == 0) {
        const int g = b0 + i, g0 = b0 + (i & ~1);
        S.e[i] = finite_or_zero(eT[g]);
        // every cut between pairs is torn: both its neighbours lose |e|; the pair itself is a 2 x 2 eigenproblem
        const double a = finite_or_zero(dT[g0]) - (g0 > 0 ? fabs(finite_or_zero(eT[g0 - 1])) : 0.0);
        const double c = finite_or_zero(dT[g0 + 1]) - fabs(finite_or_zero(eT[g0 + 1]));
        const double b = finite_or_zero(eT[g0]);
        double t = 0.0;
        if (b != 0.0) {
            const double z = (c - a) / (2.0 * b);
            t = __builtin_copysign(1.0, z) / (fabs(z) + __builtin_sqrt(1.0 + z * z));
        }
        const double cc = 1.0 / __builtin_sqrt(1.0 + t * t), ss = t * cc;
        const double l1 = a - t * b, l2 = c + t * b;  // vectors (cc, -ss) and (ss, cc)
        const bool first = ((i & 1) == 0) == (l1 <= l2);  // this index takes l1
        S.d[i] = first ? l1 : l2;
        S.Q[i * DCB_LD + (i & ~1)] = first ? cc : ss;
        S.Q[i * DCB_LD + (i | 1)] = first ? -ss : cc;
    }
    __syncthreads();
    if (tid < 256) {
        dc_level_wave<4>(S, tid, tol);
        dc_level_wave<8>(S, tid, tol);
        dc_level_wave<16>(S, tid, tol);
    }
    __syncthreads();
    dc_level<32, WITH_WY>(S, tid, tol);
    dc_level<64, WITH_WY>(S, tid, tol);
    if (l == 0) dO[b0 + i] = S.d[i];
    for (int c = tid >> 6; c < 64; c += 8) Z[(int64_t)(b0 + c) * N + b0 + (tid & 63)] = S.Q[c * DCB_LD + (tid & 63)];
}

// ---- merges of M = 128, 256, 512 rows -----------------------------------------------------------------------------
// Work arrays (N each, sub-problem at its base): dk, zk (poles and z of the survivors, then the deflated), col (their
// columns of Z), half (indices of the survivors that live in the left half, then those in the right half), org, tau,
// zh, val, npos (place of its eigenvalue), from (the inverse); ra, rb, rc, rs (rotations); per sub-problem: K, k1 (survivors in the left half), dense (rotations mixed the
// halves), nrot.

// Order of the poles, deflation, and one wave per root. Every work-group of a sub-problem orders and deflates for itself: a chain of
// some 2 us, whereas a launch that did it for all of them took 5 to 6, of which 3 to 4 pass before its first instruction. (Jobs of 128,
// 200 and 256 buffer rows: 10.84 -> 10.55, 9.21 -> 8.90 and 11.16 -> 10.79 ms, of 512: 29.44 -> 29.35.) The work-group after the
// last root's leaves the records for the kernels that follow. Columns that are rotated are rotated by dc_weights_kernel: here other work-groups still read them. WYJ > 0 (the first
// merge of N = 64 WYJ): the row of work-groups after the last sub-problem's forms the triangular factors of the
// reduction's blocks of reflectors, a wave each (wy_factor).
template <int M, int WYJ>
__global__ __launch_bounds__(256) void dc_roots_kernel(const double* __restrict__ dT, const double* __restrict__ eT, int N,
                                                       const double* __restrict__ dI, const double* __restrict__ Z, DcWork w,
                                                       const double* __restrict__ V, const double* __restrict__ tauT, int n,
                                                       double* __restrict__ Tw) {
    constexpr int E = M / 64, half = M / 2, P = M > 256 ? M / 256 : 1;  // entries a lane of a root's wave, a thread
    // (14.5 KB at 512 rows: it goes beside a Gram work-group of the side stream, of 144. With 18.5 KB it waited for that, 309 us.)
    __shared__ double d[M], ds[M], zs[M];
    __shared__ unsigned short cs[M], sv[M];
    __shared__ int sK, snr, sany;
    __shared__ int wsum[E], wsum2[E];  // per 64 entries
    int* const col = reinterpret_cast<int*>(d);  // (once the ranks are known)
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if constexpr (WYJ > 0) {
        static_assert(8 * WYJ <= M, "as many waves in a row of work-groups as blocks");
        if (blockIdx.y == gridDim.y - 1) {
            const int q = blockIdx.x * 4 + wave;
            if (q * WY <= n - 2) wy_factor<WYJ>(V, tauT, q, n, lane, Tw);
            return;
        }
    }
    const int base = blockIdx.y * M;
    const bool records = blockIdx.x == M / 4;
    const bool on = M >= 256 || tid < M;  // this thread has entries tid + 256 p
    const double ec = finite_or_zero(eT[base + half - 1]), rho = fabs(ec);
    double di[P], zi[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int t = tid + 256 * p;
        if (on) {
            const double* zc = Z + (int64_t)(base + t) * N;
            di[p] = dI[base + t];
            zi[p] = t < half ? zc[base + half - 1] : zc[base + half];
        }
    }
    const double tol = dc_tolerance(dT, eT, N, lane);
#pragma unroll
    for (int p = 0; p < P; ++p)
        if (on) {
            const int t = tid + 256 * p;
            d[t] = di[p];
            zi[p] = finite_or_zero(t >= half && ec < 0.0 ? -zi[p] : zi[p]);
        }
    if (tid == 0) {
        sany = 0;
        snr = 0;
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < P; ++p)
        if (on) {
            // both halves are sorted: rank = own position + position in the other half
            const int t = tid + 256 * p, o0 = t < half ? half : 0;
            int a = 0, b = half;  // number of entries of the other half that go before this one
            while (a < b) {
                const int mid = (a + b) >> 1;
                const double x = d[o0 + mid];
                const bool pre = x < di[p] || (x == di[p] && o0 == 0);
                if (pre) a = mid + 1;
                else b = mid;
            }
            const int r = (t < half ? t : t - half) + a;
            ds[r] = di[p];
            zs[r] = zi[p];
            cs[r] = (unsigned short)t;
        }
    __syncthreads();
    unsigned long long mask[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int t = tid + 256 * p;
        mask[p] = __ballot(on && rho * fabs(zs[t & (M - 1)]) > tol);
        if (on && lane == 0) wsum[t >> 6] = __popcll(mask[p]);
    }
    __syncthreads();
    int tot = 0;
#pragma unroll
    for (int g = 0; g < E; ++g) tot += wsum[g];
#pragma unroll
    for (int p = 0; p < P; ++p)
        if (on) {
            const int t = tid + 256 * p;
            int off = __popcll(mask[p] & ((1ull << lane) - 1ull));
#pragma unroll
            for (int g = 0; g < E; ++g) off += g < (t >> 6) ? wsum[g] : 0;
            sv[(mask[p] >> lane) & 1ull ? off : tot + t - off] = (unsigned short)t;
        }
    if (tid == 0) sK = tot;
    __syncthreads();
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int t = tid + 256 * p;
        if (on && t + 1 < tot) {
            const int s0 = sv[t], s1 = sv[t + 1];
            if (poles_equal(ds[s0], zs[s0], ds[s1], zs[s1], tol)) sany = 1;
        }
    }
    __syncthreads();
    if (sany) {  // rare: walk the survivors in order, rotate equal poles together
        if (tid == 0) {
            const int Kb = tot;
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
                    if (records) {
                        w.ra[base + nr] = cs[pj];
                        w.rb[base + nr] = cs[nj];
                        w.rc[base + nr] = c;
                        w.rs[base + nr] = s;
                    }
                    ++nr;
                    col[M - 1 - nd++] = pj;
                    pj = nj;
                } else {
                    col[nk++] = pj;
                    pj = nj;
                }
            }
            if (pj >= 0) col[nk++] = pj;
            for (int q = 0; q < nk; ++q) sv[q] = (unsigned short)col[q];
            for (int q = 0; q < nd; ++q) sv[nk + q] = (unsigned short)col[M - 1 - q];
            sK = nk;
            snr = nr;
        }
        __syncthreads();
    }
    const int K = sK;
    if (records) {
        const bool dense = snr > 0;
        int cq[P];
        unsigned long long ml[P], mr[P];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int t = tid + 256 * p;
            cq[p] = on ? cs[sv[t]] : 0;
            ml[p] = __ballot(on && t < K && !dense && cq[p] < half);
            mr[p] = __ballot(on && t < K && !dense && cq[p] >= half);
            if (on && lane == 0) {
                wsum[t >> 6] = __popcll(ml[p]);
                wsum2[t >> 6] = __popcll(mr[p]);
            }
        }
        __syncthreads();
        int tl = 0;
#pragma unroll
        for (int g = 0; g < E; ++g) tl += wsum[g];
#pragma unroll
        for (int p = 0; p < P; ++p)
            if (on) {
                const int t = tid + 256 * p;
                int ol = __popcll(ml[p] & ((1ull << lane) - 1ull)), orr = __popcll(mr[p] & ((1ull << lane) - 1ull));
#pragma unroll
                for (int g = 0; g < E; ++g) {
                    ol += g < (t >> 6) ? wsum[g] : 0;
                    orr += g < (t >> 6) ? wsum2[g] : 0;
                }
                if ((ml[p] >> lane) & 1ull) w.half[base + ol] = t;
                if ((mr[p] >> lane) & 1ull) w.half[base + tl + orr] = t;
                if (dense && t < K) w.half[base + t] = t;
                w.dk[base + t] = ds[sv[t]];
                w.zk[base + t] = zs[sv[t]];
                w.col[base + t] = base + cq[p];
            }
        if (tid == 0) {
            w.K[blockIdx.y] = K;
            w.k1[blockIdx.y] = tl;
            w.dense[blockIdx.y] = dense ? 1 : 0;
            w.nrot[blockIdx.y] = snr;
        }
        return;
    }
    const int q = blockIdx.x * 4 + wave;
    double org = 0.0, tau = 0.0, val = ds[sv[q]];
    if (q < K) {
        double dj[E], zj[E], zsum = 0.0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int j = lane + 64 * e, s = sv[j];
            const bool live = j < K;
            dj[e] = live ? ds[s] : 1e30;
            const double z = live ? zs[s] : 0.0;
            zj[e] = rho * z * z;
            zsum += zj[e];
        }
        zsum = lane_sum<64>(zsum);
        const int ip = lower_pole(q, K), si = sv[ip], sn = sv[ip + (K > 1)];
        const double pn = ds[sn], z0 = zs[si], z1 = zs[sn];
        secular_root<64, E>(true, q >= K - 1, K, dj, zj, K > 1 ? ds[si] : pn - 1.0, pn, K > 1 ? rho * z0 * z0 : 0.0, rho * z1 * z1, zsum, org,
                            tau);
        val = finite_or_zero(org + tau);
    }
    if (lane == 0) {
        w.org[base + q] = org;
        w.tau[base + q] = tau;
        w.val[base + q] = val;
    }
}

// one wave per index: z of the merge, and the place of its eigenvalue among all. The work-group after the last index's rotates
// columns of Z where that is called for.
template <int M>
__global__ __launch_bounds__(256) void dc_weights_kernel(DcWork w, double* __restrict__ dO, double* __restrict__ Z, int N) {
    constexpr int E = M / 64, m = M;
    const int lane = threadIdx.x & 63;
    const int q = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int base = blockIdx.y * m;
    if (blockIdx.x == M / 4) {
        const int nr = w.nrot[blockIdx.y];
        if (nr == 0) return;
        // the columns become dense: clear what was not stored of them, then rotate (a thread per row)
        for (int r = threadIdx.x; r < m; r += 256) {
            for (int c = 0; c < m; ++c)
                if ((c < m / 2) != (r < m / 2)) Z[(int64_t)(base + c) * N + base + r] = 0.0;
            for (int i = 0; i < nr; ++i) {
                double* A = Z + (int64_t)(base + w.ra[base + i]) * N + base + r;
                double* B = Z + (int64_t)(base + w.rb[base + i]) * N + base + r;
                const double a = *A, b = *B, c = w.rc[base + i], s = w.rs[base + i];
                *A = c * a + s * b;
                *B = c * b - s * a;
            }
        }
        return;
    }
    const int K = w.K[blockIdx.y];
    const double val = w.val[base + q];
    int np = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int j = lane + 64 * e;
        if (j < m) {
            const double x = w.val[base + j];
            np += (x < val || (x == val && j < q)) ? 1 : 0;
        }
    }
    np = lane_sum_i<64>(np);
    double zz = 0.0;
    if (q < K) {
        double di[E], og[E], ta[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int j = lane + 64 * e;
            di[e] = j < K ? w.dk[base + j] : 0.0;
            og[e] = j < K ? w.org[base + j] : 0.0;
            ta[e] = j < K ? w.tau[base + j] : 0.0;
        }
        zz = __builtin_copysign(secular_z<64, E>(K, q, lane, w.dk[base + q], di, og, ta), w.zk[base + q]);
    }
    if (lane == 0) {
        w.zh[base + q] = zz;
        w.npos[base + q] = np;
        w.from[base + np] = q;
        dO[base + np] = val;
    }
}

// Z_out(:, npos_q) = Z_in(:, survivors) u_q, u_q(j) = zh_j / (d_j - lambda_q) normalised; deflated columns are copied.
// grid (m / 32 column tiles, m / 64 row tiles, sub-problems), 256 threads; a wave owns 16 rows x 32 columns. A row tile
// of the left (right) half only meets the survivors that live there. Poles, weights and column numbers are brought to LDS
// once (chasing the column list through global memory in every step made the kernel 60 us at m = 512), the columns of
// Z_in are requested a step ahead, and the entries of u are formed on the way into LDS.
__global__ __launch_bounds__(256) void dc_vectors_kernel(const double* __restrict__ Zin, double* __restrict__ Zout, int N,
                                                         int m, DcWork w) {
    constexpr int KT = 32, LDA = 72, LDB = 40;
    __shared__ double As[KT * LDA], Bs[KT * LDB];
    __shared__ double inv[32], og[32], ta[32];
    __shared__ double dk[512], zh[512];
    __shared__ int lj[512], lc[512];  // survivors of this row tile's half: index, column
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int base = blockIdx.z * m, half = m >> 1;
    const int q0 = blockIdx.x * 32, r0 = blockIdx.y * 64;
    const int K = w.K[blockIdx.z], k1 = w.k1[blockIdx.z];
    const bool dense = w.dense[blockIdx.z] != 0;
    const bool left = r0 < half;
    const int* list = w.half + base + (dense || left ? 0 : k1);
    const int len = dense ? K : (left ? k1 : K - k1);
    if (q0 < K) {
        for (int j = tid; j < m; j += 256) {
            dk[j] = j < K ? w.dk[base + j] : 1e30;
            zh[j] = j < K ? w.zh[base + j] : 0.0;
            if (j < len) {
                const int q = list[j];
                lj[j] = q;
                lc[j] = w.col[base + q];
            }
        }
        if (tid < 32) {
            og[tid] = w.org[base + q0 + tid];
            ta[tid] = w.tau[base + q0 + tid];
        }
        __syncthreads();
        double av[8];
        auto fetch = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int kk = k0 + u * 4 + wave;
                av[u] = kk < len ? Zin[(int64_t)lc[kk] * N + base + r0 + lane] : 0.0;
            }
        };
        fetch(0);
        {   // norms of the tile's vectors: 8 lanes per column
            const int c = tid >> 3, l = tid & 7;
            const double o = og[c], t = ta[c];
            double n0 = 0.0, n1 = 0.0;
            for (int j = l; j < m; j += 16) {
                const double u0 = zh[j] * rcp64((dk[j] - o) - t), u1 = zh[j + 8] * rcp64((dk[j + 8] - o) - t);
                n0 = __builtin_fma(u0, u0, n0);
                n1 = __builtin_fma(u1, u1, n1);
            }
            const double nn = lane_sum<8>(n0 + n1);
            if (l == 0) inv[c] = nn > 0.0 ? rcp64(__builtin_sqrt(nn)) : 0.0;
        }
        const int l16 = lane & 15, lk = lane >> 4, bc = tid & 31;
        f64x4 acc[2] = {f64x4{0.0, 0.0, 0.0, 0.0}, f64x4{0.0, 0.0, 0.0, 0.0}};
        for (int k0 = 0; k0 < len; k0 += KT) {
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 8; ++u) As[(u * 4 + wave) * LDA + lane] = av[u];
            fetch(k0 + KT);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int kk = u * 8 + (tid >> 5);
                double v = 0.0;
                if (k0 + kk < len && q0 + bc < K) {
                    const int j = lj[k0 + kk];
                    v = zh[j] * rcp64((dk[j] - og[bc]) - ta[bc]) * inv[bc];
                }
                Bs[kk * LDB + bc] = v;
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < KT; k += 4) {
                const double a = As[(k + lk) * LDA + wave * 16 + l16];
#pragma unroll
                for (int t = 0; t < 2; ++t) acc[t] = mfma64(a, Bs[(k + lk) * LDB + t * 16 + l16], acc[t]);
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

// T = Z D Z^T: eigenvalues ascending in dI[dc_result(N)], the triangular factors of the reflectors in Tw. The eigenvectors are the
// columns of Z[0] (N = 64), or what the last merge makes of those of Z[dc_result(N) ^ 1] by `dc`. n: rows in use.
hipError_t launch_dc(const EigWork& w, int N, int n, hipStream_t st) {
    if (N != 64 && N != 128 && N != 256 && N != 512) return hipErrorInvalidValue;
    const void* block = N == 64 ? (const void*)dc_block_kernel<true> : (const void*)dc_block_kernel<false>;
    if (hipError_t e = ensure_dynamic_lds(block, (int)sizeof(DcBlockLds)); e != hipSuccess) return e;
    if (N == 64)
        hipLaunchKernelGGL(dc_block_kernel<true>, dim3(2), dim3(512), sizeof(DcBlockLds), st, w.dT, w.eT, N, w.dI[0], w.Z[0],
                           w.V, w.tauT, n, w.Tw, w.xch, w.claim);
    else
        hipLaunchKernelGGL(dc_block_kernel<false>, dim3(N / 64), dim3(512), sizeof(DcBlockLds), st, w.dT, w.eT, N, w.dI[0],
                           w.Z[0], w.V, w.tauT, n, w.Tw, w.xch, w.claim);
    int cur = 0;
    for (int m = 128; m <= N; m *= 2) {
        const int S = N / m;
#define SAGE_ROOTS(M, WYJ)                                                                                               \
    do {                                                                                                                \
        hipLaunchKernelGGL((dc_roots_kernel<M, WYJ>), dim3(M / 4 + 1, WYJ > 0 ? S + 1 : S), dim3(256), 0, st, w.dT, w.eT, N, w.dI[cur], \
                           w.Z[cur], w.dc, w.V, w.tauT, n, w.Tw);                                                       \
        hipLaunchKernelGGL(dc_weights_kernel<M>, dim3(M / 4 + 1, S), dim3(256), 0, st, w.dc, w.dI[cur ^ 1], w.Z[cur], N); \
    } while (0)
        if (m == 512) SAGE_ROOTS(512, 0);
        else if (m == 256) SAGE_ROOTS(256, 0);
        else if (N == 128) SAGE_ROOTS(128, 2);
        else if (N == 256) SAGE_ROOTS(128, 4);
        else SAGE_ROOTS(128, 8);
#undef SAGE_ROOTS
        if (m == N) break;  // (the last merge's vectors are formed where they are used: tri_back_kernel)
        hipLaunchKernelGGL(dc_vectors_kernel, dim3(m / 32, m / 64, S), dim3(256), 0, st, w.Z[cur], w.Z[cur ^ 1], N, m, w.dc);
        cur ^= 1;
    }
    return hipGetLastError();
}

}  // namespace sage
