// Gram matrix of the sketch buffer, C = B B^T, on the fp32 matrix cores.
//
// The shrink step needs the SVD of the buffer (Method, FD paragraph: "compute a thin SVD S = U Sigma V^T");
// it is taken through the eigen-decomposition of this Gram matrix. Only the lower triangle is computed, in
// 64x64 tiles. The long dimension (D) is split over work-group "groups"; each group writes fp32 partial tiles
// that gram_reduce adds in a fixed order in fp64.
#include <type_traits>

#include <hip/hip_ext.h>

#include "fd_rows.h"
#include "sage_internal.h"

namespace sage {

__device__ __forceinline__ void tile_coords(int t, int& ti, int& tj) {
    // row-major enumeration of the lower triangle: t = ti*(ti+1)/2 + tj, tj <= ti
    int i = 0;
    while ((i + 1) * (i + 2) / 2 <= t) ++i;
    ti = i;
    tj = t - i * (i + 1) / 2;
}

// Rows not in use are loaded like the others and dropped by a select: a predicate on the load is a branch, of which a wave paid one
// per 16 bytes (cross block of 256 bf16 rows of 2,049,000: 716 us with it, 673 without; jobs of 128 and of 100 fp32 rows, 1,081,576
// and 1,562,728 columns: 19.5 -> 18.6 and 26.1 -> 24.6 ms). What is loaded in their place is the last row in use, which is there anyway.
__device__ __forceinline__ int row_in_use(int row, int rows) { return row < rows ? row : (rows > 0 ? rows - 1 : 0); }

// P = NP / 64 row panels. Tiles t0 .. t0 + tiles - 1 of the row-major lower-triangle enumeration are computed (t0 > 0
// leaves out the leading panels whose Gram block the caller already knows). 256 threads = 4 waves; the unit of work is half a tile (32 rows x 64 columns, two
// 32x32 accumulators); a wave owns up to 3 units, a work-group 12 (6 tiles), and two work-groups share a CU so
// that one's LDS reads and barrier waits hide under the other's matrix-core work.
// Dynamic LDS: 2 stages x NP rows x 64 B, 16-byte pieces XOR-swizzled by (row/4)%4 so that the 16 rows read
// by a quarter wave fall in distinct banks.
// The buffer is two half buffers of LP = NP/2 rows each (same slab layout): `top` holds matrix rows 0 .. LP-1, `nw`
// matrix rows LP .. NP-1, of which only the first nfill hold data (the rest are taken as zero, whatever they hold).
// mode 0: tiles t0 .. t0+tiles-1 of the triangle; mode 1: the rectangle (new rows) x (top rows), tiles row-major;
// mode 2: the triangle of (new rows) x (new rows).
__device__ __forceinline__ void gram_tile(int mode, int P, int t0, int idx, int& ti, int& tj) {
    const int q = P >> 1;
    if (mode == 0) {
        tile_coords(t0 + idx, ti, tj);
    } else if (mode == 1) {
        ti = q + idx / q;
        tj = idx % q;
    } else {
        tile_coords(idx, ti, tj);
        ti += q;
        tj += q;
    }
}

// The launch's row of work-groups y takes tops.p[y] for the top half and has its partial tiles y * stride floats further on.
// FRESH: mode 2, which needs no top rows.
template <int P, bool FRESH>
__global__ __launch_bounds__(256, 2) void gram_kernel(GramTops tops, const float* __restrict__ nw,
                                                      int nfill, float* __restrict__ partial, int mode, int t0,
                                                      int tiles, int wg_per_group, int64_t slabs_total,
                                                      int64_t slabs_per_group, int wgs,
                                                      const int* __restrict__ hole) {
    const float* __restrict__ top = tops.p[blockIdx.y];
    partial += blockIdx.y * tops.stride;
    constexpr int NP = P * 64;
    constexpr int STAGE = NP * 4;  // 16-byte pieces per stage
    extern __shared__ f32x4 lds[];

    const int id = (int)spare_unit_at(hole);
    if (id < 0 || id >= wgs) return;
    const int xcd = id & 7;  // consecutive block ids go to consecutive XCDs: keep a group on one XCD (shared L2)
    const int y = id >> 3;
    const int w = y % wg_per_group;
    const int group = (y / wg_per_group) * 8 + xcd;
    int64_t s0 = (int64_t)group * slabs_per_group;
    int64_t s1 = s0 + slabs_per_group;
    if (s1 > slabs_total) s1 = slabs_total;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int l32 = lane & 31, h = lane >> 5;

    // unit u = 2 * tile + row half; dealt to the waves in turn, so that few units are spread evenly
    int arow[3], brow[3];
    bool on[3];
    const int ubase = w * 12 + wave;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        int u = ubase + 4 * q;
        on[q] = u < 2 * tiles;
        int ti = 0, tj = 0;
        if (on[q]) gram_tile(mode, P, t0, u >> 1, ti, tj);
        arow[q] = ti * 64 + (u & 1) * 32 + l32;
        brow[q] = tj * 64 + l32;
    }

    f32x16 acc[3][2];
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[q][b][i] = 0.f;

    // staging map: slot ps = it*256 + tid holds (row = ps/4, logical piece = (ps%4) ^ ((row/4)%4)); the row comes from
    // the top half, the new half, or is zero
    constexpr int LP = NP / 2;
    constexpr int HALF4 = LP * 4;  // 16-byte pieces of one half buffer per slab
    int src[P];                    // piece index inside the half's slab
    bool isnew[P], used[P];        // (see row_in_use)
#pragma unroll
    for (int it = 0; it < P; ++it) {
        int ps = it * 256 + tid;
        int row = ps >> 2;
        int p = (ps & 3) ^ ((row >> 2) & 3);
        isnew[it] = row >= LP;
        int hr = isnew[it] ? row - LP : row;
        const int rows = isnew[it] ? nfill : tops.rows;
        src[it] = row_in_use(hr, rows) * 4 + p;
        used[it] = hr < rows && (isnew[it] || !FRESH);
    }
    constexpr int IT0 = FRESH ? P / 2 : 0;  // the first with new rows, where the others are not needed
    const f32x4* Tv = reinterpret_cast<const f32x4*>(top);
    const f32x4* Nv = reinterpret_cast<const f32x4*>(nw);
    // Slabs are requested two stages before they are used: one set of registers goes to LDS while the other fills (with P = 8
    // there are registers for one set only: one stage).
    constexpr bool TWO = P < 8;
    f32x4 pre0[P], pre1[P];
    auto fetch = [&](int64_t sl, f32x4 (&pre)[P]) __attribute__((always_inline)) {
        const int64_t sc = sl < s1 ? sl : s1 - 1;  // beyond the end: repeat (never used)
#pragma unroll
        for (int it = IT0; it < P; ++it) pre[it] = ((isnew[it] ? Nv : Tv) + sc * HALF4)[src[it]];
    };
    auto store = [&](const f32x4 (&pre)[P], f32x4* dst) __attribute__((always_inline)) {
#pragma unroll
        for (int it = IT0; it < P; ++it) dst[it * 256 + tid] = used[it] ? pre[it] : f32x4{0.f, 0.f, 0.f, 0.f};
    };

    if (s0 < s1) {
        fetch(s0, pre0);
        if constexpr (TWO) fetch(s0 + 1, pre1);
        store(pre0, lds);
    }
    __syncthreads();

    auto step = [&](int64_t s, int cur, f32x4 (&next)[P], f32x4 (&far)[P]) __attribute__((always_inline)) {
        fetch(TWO ? s + 2 : s + 1, far);
        const f32x4* st = lds + cur * STAGE;
        // operands of the whole stage are fetched up front, first the pieces of k-half 0 for every unit, then those of
        // k-half 1, which land while the matrix cores work on half 0; one straight-line block per number of units
        auto products = [&](auto nq) __attribute__((always_inline)) {
            constexpr int NQ = decltype(nq)::value;
            f32x4 a[2][NQ], b[2][NQ][2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int p = 2 * j + h;
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    const int ra = arow[q];
                    a[j][q] = st[ra * 4 + (p ^ ((ra >> 2) & 3))];
#pragma unroll
                    for (int cb = 0; cb < 2; ++cb) {
                        const int rb = brow[q] + cb * 32;
                        b[j][q][cb] = st[rb * 4 + (p ^ ((rb >> 2) & 3))];
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);  // keep the LDS reads above: the scheduler would sink each next to its use
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int q = 0; q < NQ; ++q)
#pragma unroll
                        for (int cb = 0; cb < 2; ++cb) acc[q][cb] = mfma32(a[j][q][c], b[j][q][cb][c], acc[q][cb]);
            __builtin_amdgcn_sched_barrier(0);
        };
        // (wave-uniform; a work-group of a small triangle has no third, second or any unit for some of its waves: carried
        // along they cost 48 matrix-core instructions a slab where 16 are needed)
        if (on[2]) products(std::integral_constant<int, 3>{});
        else if (on[1]) products(std::integral_constant<int, 2>{});
        else if (on[0]) products(std::integral_constant<int, 1>{});
        store(next, lds + (cur ^ 1) * STAGE);
        // a bare barrier after the LDS traffic: __syncthreads() would also wait for the loads of the slab after next
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    for (int64_t s = s0; s < s1; s += 2) {
        if constexpr (TWO) {
            step(s, 0, pre1, pre0);
            if (s + 1 < s1) step(s + 1, 1, pre0, pre1);
        } else {
            step(s, 0, pre0, pre0);
            if (s + 1 < s1) step(s + 1, 1, pre0, pre0);
        }
    }

    // partial[group][tile - t0][64 x 64]; unit u covers rows (u & 1) * 32 .. + 32 of tile t0 + u / 2
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        if (!on[q]) continue;
        const int u = ubase + 4 * q;
        float* out = partial + ((int64_t)group * tiles + (u >> 1)) * 4096 + (u & 1) * 2048;
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                int r = 8 * (i >> 2) + 4 * h + (i & 3);
                int c = cb * 32 + l32;
                out[r * 64 + c] = acc[q][cb][i];
            }
    }
}

// The (new rows) x (top rows) rectangle for NP = 512, with wider wave tiles than gram_kernel's: a wave owns 128 new rows
// x 64 top rows (8 accumulator tiles), so the 256 x 256 rectangle is exactly 8 wave tiles = 2 work-groups per column
// range -- no idle wave slots, a third less staging traffic than 3 work-groups, and 12 operand reads per 64
// matrix-core instructions instead of 18 per 48. Same staging, LDS layout and partial-tile output as gram_kernel
// in mode 1 (tile index (ti - 4) * 4 + tj).
__global__ __launch_bounds__(256, 2) void gram_cross8_kernel(const float* __restrict__ top, const float* __restrict__ nw,
                                                             int nfill, float* __restrict__ partial,
                                                             int64_t slabs_total, int64_t slabs_per_group) {
    constexpr int P = 8, NP = 512, LP = 256;
    constexpr int STAGE = NP * 4;
    constexpr int HALF4 = LP * 4;
    extern __shared__ f32x4 lds[];

    const int id = blockIdx.x;
    const int xcd = id & 7;
    const int y = id >> 3;
    const int w = y & 1;  // 2 work-groups per group
    const int group = (y >> 1) * 8 + xcd;
    int64_t s0 = (int64_t)group * slabs_per_group;
    int64_t s1 = s0 + slabs_per_group;
    if (s1 > slabs_total) s1 = slabs_total;

    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int l32 = lane & 31, h = lane >> 5;
    const int wt = w * 4 + wave;          // wave tile 0..7
    const int ag = wt >> 2, bg = wt & 3;  // new rows 128*ag .. + 128, top rows 64*bg .. + 64
    const int arow = LP + ag * 128 + l32; // + 32 * i, i < 4 (matrix row index: new half starts at LP)
    const int brow = bg * 64 + l32;       // + 32 * cb

    f32x16 acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][b][e] = 0.f;

    int src[P];
#pragma unroll
    for (int it = 0; it < P; ++it) {
        int ps = it * 256 + tid;
        int row = ps >> 2;
        int p = (ps & 3) ^ ((row >> 2) & 3);
        int hr = row >= LP ? row - LP : row;
        src[it] = (row >= LP && hr >= nfill) ? -1 : hr * 4 + p;
    }
    const f32x4* Tv = reinterpret_cast<const f32x4*>(top);
    const f32x4* Nv = reinterpret_cast<const f32x4*>(nw);
    f32x4 pre[P];
    auto fetch = [&](int64_t sl) {
#pragma unroll
        for (int it = 0; it < P; ++it) {
            const f32x4* base = (it >= P / 2 ? Nv : Tv) + sl * HALF4;  // rows it*64 .. : the new half from it = 4 on
            pre[it] = src[it] >= 0 ? base[src[it]] : f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };
    if (s0 < s1) {
        fetch(s0);
#pragma unroll
        for (int it = 0; it < P; ++it) lds[it * 256 + tid] = pre[it];
    }
    __syncthreads();

    for (int64_t s = s0; s < s1; ++s) {
        const int cur = (int)((s - s0) & 1);
        const bool more = (s + 1 < s1);
        if (more) fetch(s + 1);
        const f32x4* st = lds + cur * STAGE;
        f32x4 a[2][4], b[2][2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int p = 2 * j + h;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int ra = arow + 32 * i;
                a[j][i] = st[ra * 4 + (p ^ ((ra >> 2) & 3))];
            }
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                const int rb = brow + 32 * cb;
                b[j][cb] = st[rb * 4 + (p ^ ((rb >> 2) & 3))];
            }
        }
        __builtin_amdgcn_sched_barrier(0);  // keep the LDS reads above: the scheduler would sink each next to its use
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int cb = 0; cb < 2; ++cb) acc[i][cb] = mfma32(a[j][i][c], b[j][cb][c], acc[i][cb]);
        __builtin_amdgcn_sched_barrier(0);
        if (more) {
            f32x4* nx = lds + (cur ^ 1) * STAGE;
#pragma unroll
            for (int it = 0; it < P; ++it) nx[it * 256 + tid] = pre[it];
        }
        __syncthreads();
    }

    // tiles (ti - 4, tj) = (2*ag + i/2, bg); rows (i & 1) * 32 .. + 32 of the tile
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int tidx = (2 * ag + (i >> 1)) * 4 + bg;
        float* out = partial + ((int64_t)group * 16 + tidx) * 4096 + (i & 1) * 2048;
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                int r = 8 * (e >> 2) + 4 * h + (e & 3);
                int c = cb * 32 + l32;
                out[r * 64 + c] = acc[i][cb][e];
            }
    }
}

// The same rectangle on the bf16 matrix cores: every fp32 value is written as three bf16 parts (24 significant bits)
// and the six products that matter (hi*hi, hi*mid, mid*hi, hi*lo, lo*hi, mid*mid) are accumulated in fp32 -- the
// fp32 result to a few 2^-24 per term, 6 x 32 cycles per 32 x 32 x 16 block instead of 8 x 64 on the fp32 matrix
// cores. One slab (16 columns) is exactly one k-step. The values are split when they are staged, once per
// work-group, so one work-group of 8 waves owns all 8 wave tiles of a column range (staging traffic is half of
// gram_cross8_kernel's, where two work-groups stage the same slabs). LDS holds a slab as [part][k-half][row] pieces
// of 16 bytes (8 bf16: the k-half of a row), 48 KB, double buffered; the 32 rows a matrix-core operand reads are
// 512 contiguous bytes. The next slab is split and stored piece by piece between the six groups of matrix-core
// instructions (all waves of a work-group run in step: conversions done in one block would leave the matrix cores
// idle), from registers that were loaded a stage earlier and are reloaded, for the slab after next, as soon as they
// have been consumed.
// NEW1: the new half is kept in pieces of bf16 (half16): its mid and lo parts are zero, so only one part is staged, as it
// is, and only the three products with it are issued. The three left out would add exact
// zeros: the result has the same bits either way.
template <bool NEW1>
__global__ __launch_bounds__(512, 1) void gram_cross8_split_kernel(GramTops tops,
                                                                   const float* __restrict__ nw, int nfill,
                                                                   float* __restrict__ partial, int64_t slabs_total,
                                                                   int64_t slabs_per_group, int groups,
                                                                   const int* __restrict__ hole) {
    constexpr int NP = 512, LP = 256;
    constexpr int HALF4 = LP * 4;        // 16-byte pieces of a half buffer per slab
    constexpr int HREG = NP + 8;         // pieces per k-half region: the rows plus 128 bytes, so that the two regions a
                                         // staging store touches fall on different banks
    constexpr int PART16 = 2 * HREG;     // pieces per part: [k-half][row]
    constexpr int STAGE16 = 3 * PART16;  // 48.4 KB
    extern __shared__ u32x4 ldsx[];      // 2 * STAGE16

    const int group = (int)spare_unit_at(hole);
    if (group < 0 || group >= groups) return;
    const float* __restrict__ top = tops.p[blockIdx.y];
    partial += blockIdx.y * tops.stride;
    const int64_t s0 = (int64_t)group * slabs_per_group;
    int64_t s1 = s0 + slabs_per_group;
    if (s1 > slabs_total) s1 = slabs_total;

    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int l32 = lane & 31, h = lane >> 5;
    const int ag = wave >> 2, bg = wave & 3;  // new rows 128*ag .. + 128, top rows 64*bg .. + 64
    const int arow = LP + ag * 128 + l32;     // + 32 * i, i < 4
    const int brow = bg * 64 + l32;           // + 32 * cb

    f32x16 acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][b][e] = 0.f;

    // staging: piece ps = it * 512 + tid is columns 4p .. 4p+3 of row ps >> 2 (rows >= LP: the new half)
    // (NEW1: the new rows' pieces are those of half16: piece tid is k-half tid >> 8 of row tid & 255)
    const f32x4* Tv = reinterpret_cast<const f32x4*>(top);
    const f32x4* Nv = reinterpret_cast<const f32x4*>(nw);
    const u32x4* N16 = half16(nw, LP, slabs_total);
    constexpr int IT = NEW1 ? 3 : 4;
    int src[4], dst8[4];  // source piece in the half buffer, LDS offset in 8-byte units
    bool used[4];         // (see row_in_use)
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int ps = it * 512 + tid, row = ps >> 2, p = ps & 3;
        const int hr = row & (LP - 1);
        const int rows = it >= 2 ? nfill : tops.rows;
        src[it] = row_in_use(hr, rows) * 4 + p;
        used[it] = hr < rows;
        dst8[it] = (((p >> 1) * HREG + row) << 1) + (p & 1);
    }
    const bool used16 = (tid & 255) < nfill;
    const int src16 = (tid & 256) + row_in_use(tid & 255, nfill);
    const int dst16 = (tid >> 8) * HREG + LP + (tid & 255);
    f32x4 pre[4];
    u32x4 pre16;
    auto fetch1 = [&](int it, int64_t sl) __attribute__((always_inline)) {
        const int64_t sc = sl < s1 ? sl : s1 - 1;  // beyond the end: repeat (never used)
        if (NEW1 && it == 2) {
            pre16 = N16[sc * 512 + src16];
            return;
        }
        pre[it] = ((it >= 2 ? Nv : Tv) + sc * HALF4)[src[it]];
    };
    auto store1 = [&](int it, int buf) __attribute__((always_inline)) {
        if (NEW1 && it == 2) {
            ldsx[buf * STAGE16 + dst16] = used16 ? pre16 : u32x4{0u, 0u, 0u, 0u};
            return;
        }
        uint2* d = reinterpret_cast<uint2*>(ldsx + buf * STAGE16) + dst8[it];
        unsigned a0, a1, a2, b0, b1, b2;
        if (!used[it]) pre[it] = f32x4{0.f, 0.f, 0.f, 0.f};
        split3_bf16(pre[it][0], pre[it][1], a0, a1, a2);
        split3_bf16(pre[it][2], pre[it][3], b0, b1, b2);
        d[0] = make_uint2(a0, b0);
        d[2 * PART16] = make_uint2(a1, b1);
        d[4 * PART16] = make_uint2(a2, b2);
    };
    if (s0 < s1) {
#pragma unroll
        for (int it = 0; it < IT; ++it) fetch1(it, s0);
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            store1(it, 0);
            fetch1(it, s0 + 1);
        }
    }
    __syncthreads();

    constexpr int AP = NEW1 ? 1 : 3;  // parts of a new row
    constexpr int NQ = NEW1 ? 3 : 6;  // products
    for (int64_t s = s0; s < s1; ++s) {
        const int cur = (int)((s - s0) & 1);
        const u32x4* st = ldsx + cur * STAGE16 + h * HREG;
        u32x4 a[4][AP], b[2][3];
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            if (p < AP) {
#pragma unroll
                for (int i = 0; i < 4; ++i) a[i][p] = st[p * PART16 + arow + 32 * i];
            }
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) b[cb][p] = st[p * PART16 + brow + 32 * cb];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {  // in the order the parts were read: the first group needs the hi parts only
            constexpr int PA[6] = {0, 0, 1, 1, 0, 2}, PB[6] = {0, 1, 0, 1, 2, 0};
            const int pa = NEW1 ? 0 : PA[q], pb = NEW1 ? q : PB[q];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) acc[i][cb] = mfma_bf16(a[i][pa], b[cb][pb], acc[i][cb]);
            // slab s + 1 into the other buffer, slab s + 2 on its way
            if (!NEW1 && q < 4) {
                store1(q, cur ^ 1);
                fetch1(q, s + 2);
            }
            if (NEW1) {
                store1(q, cur ^ 1);
                fetch1(q, s + 2);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // the LDS stores above must be visible, the reads of this stage are consumed; the loads for slab s + 2 stay
        // in flight (a bare barrier: __syncthreads() would wait for them)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }

    // tiles (ti - 4, tj) = (2*ag + i/2, bg); rows (i & 1) * 32 .. + 32 of the tile
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int tidx = (2 * ag + (i >> 1)) * 4 + bg;
        float* out = partial + ((int64_t)group * 16 + tidx) * 4096 + (i & 1) * 2048;
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                int r = 8 * (e >> 2) + 4 * h + (e & 3);
                int c = cb * 32 + l32;
                out[r * 64 + c] = acc[i][cb][e];
            }
    }
}

// The same rectangle of two blocks kept in pieces of bf16 (half16), the top rows being an earlier block's: one part each, one
// product (the bits of the kernel above, whose other products add exact zeros), nothing to convert. Bound by memory: the pieces
// go straight to LDS, two slabs (32 KB) at a time into a ring of three, two of them on their way. (With three slabs at a time, 144 KB of
// a CU's 160, the merges of the eigensolve beside it waited for it, 230 us.) Several earlier blocks: the new rows of a range come from
// the L2 for all but one of them (three blocks of 256 rows of 2,049,000: 1100 us, 1270 one block after the other).
__global__ __launch_bounds__(512, 1) void gram_cross8_half_kernel(GramTops tops, const float* __restrict__ nw, int nfill,
                                                                  float* __restrict__ partial, int64_t slabs_total,
                                                                  int64_t slabs_per_group, int groups, int count,
                                                                  const int* __restrict__ hole) {
    constexpr int LP = 256, SL = 2, SLAB = 2 * 2 * LP, STAGE = SL * SLAB, ML = STAGE / 512;  // SLAB: [top, new][k-half][row]
    extern __shared__ u32x4 ldsc[];  // 3 * STAGE
    const int at = hole ? *hole : -1, unit = (int)spare_unit(blockIdx.x, at);
    if (unit < 0) return;
    const int group = range_unit(unit, count, at).range, block = range_unit(unit, count, at).part;
    if (group >= groups) return;
    partial += block * tops.stride;
    const int64_t s0 = (int64_t)group * slabs_per_group;
    int64_t s1 = s0 + slabs_per_group;
    if (s1 > slabs_total) s1 = slabs_total;
    const u32x4* T16 = half16(tops.p[block], LP, slabs_total);
    const u32x4* N16 = half16(nw, LP, slabs_total);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, h = lane >> 5;
    const int ag = wave >> 2, bg = wave & 3;  // new rows 128*ag .. + 128, top rows 64*bg .. + 64

    const int trow = (tid & 256) + row_in_use(tid & 255, tops.rows), nrow = (tid & 256) + row_in_use(tid & 255, nfill);

    f32x16 acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][b][e] = 0.f;

    auto stage = [&](int64_t sl, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < ML; ++q) {  // 512 pieces of a slab's top rows, then of its new rows
            const int64_t s = sl + q / 2;
            const int64_t sc = s < s1 ? s : s1 - 1;  // beyond the end: repeat (never used)
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void*)((q & 1 ? N16 + nrow : T16 + trow) + sc * (2 * LP)),
                (__attribute__((address_space(3))) void*)(ldsc + buf * STAGE + q * 512 + wave * 64), 16, 0, 0);
        }
    };
    if (s0 < s1) {
        stage(s0, 0);
        stage(s0 + SL, 1);
    }
    int buf = 0;
    for (int64_t s = s0; s < s1; s += SL) {
        // all but the last stage's loads have landed; everyone is done with the buffer of the stage before
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0F70 | ML);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        stage(s + 2 * SL, buf == 0 ? 2 : buf - 1);
        const u32x4* st = ldsc + buf * STAGE + h * LP + l32;
#pragma unroll
        for (int u = 0; u < SL; ++u) {
            if (s + u >= s1) break;  // (uniform)
            u32x4 a[4], b[2];
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                const int r = bg * 64 + 32 * cb;
                b[cb] = st[u * SLAB + r];
                if (r + l32 >= tops.rows) b[cb] = u32x4{0u, 0u, 0u, 0u};
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = ag * 128 + 32 * i;
                a[i] = st[u * SLAB + 2 * LP + r];
                if (r + l32 >= nfill) a[i] = u32x4{0u, 0u, 0u, 0u};
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) acc[i][cb] = mfma_bf16(a[i], b[cb], acc[i][cb]);
        }
        buf = buf == 2 ? 0 : buf + 1;
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): nothing on its way to LDS when the work-group ends

#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int tidx = (2 * ag + (i >> 1)) * 4 + bg;
        float* out = partial + ((int64_t)group * 16 + tidx) * 4096 + (i & 1) * 2048;
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int e = 0; e < 16; ++e) out[(8 * (e >> 2) + 4 * h + (e & 3)) * 64 + cb * 32 + l32] = acc[i][cb][e];
    }
}

// The (new rows) x (new rows) triangle for NP = 512: 256 rows, i.e. 8 row blocks of 32 and 36 blocks (bi >= bj) of
// 32 x 32. Only the new rows are staged (16 KB per slab). The 36 blocks are dealt to the 4 waves, 9 each, so that a
// wave needs at most 6 operand rows-blocks per k-step: three 3 x 3 rectangles
//   rows {5,6,7} x {0,1,2},   rows {5,6,7} x {3,4,5},   rows {2,3,4} x {0,1,2},
// and the three 2 x 2 triangles on the diagonal that are left, {0,1}, {3,4}, {6,7} (on a diagonal block both
// operands are the same registers). No idle accumulators, 12 LDS reads per 72 matrix-core instructions. One
// work-group per column range; partial tiles in the layout of gram_kernel's mode 2 (the upper 32 x 32 block of a
// diagonal tile is not written and never read).
template <int W>
struct New8Map;
template <>
struct New8Map<0> {
    static constexpr int rows[6] = {5, 6, 7, 0, 1, 2};
    static constexpr int pa[9] = {0, 0, 0, 1, 1, 1, 2, 2, 2}, pb[9] = {3, 4, 5, 3, 4, 5, 3, 4, 5};
};
template <>
struct New8Map<1> {
    static constexpr int rows[6] = {5, 6, 7, 3, 4, 4};
    static constexpr int pa[9] = {0, 0, 0, 1, 1, 1, 2, 2, 2}, pb[9] = {3, 4, 0, 3, 4, 0, 3, 4, 0};
};
template <>
struct New8Map<2> {
    static constexpr int rows[6] = {2, 3, 4, 0, 1, 1};
    static constexpr int pa[9] = {0, 0, 0, 1, 1, 1, 2, 2, 2}, pb[9] = {3, 4, 0, 3, 4, 0, 3, 4, 0};
};
template <>
struct New8Map<3> {
    static constexpr int rows[6] = {0, 1, 3, 4, 6, 7};
    static constexpr int pa[9] = {0, 1, 1, 2, 3, 3, 4, 5, 5}, pb[9] = {0, 0, 1, 2, 2, 3, 4, 4, 5};
};

template <int W>
__device__ __forceinline__ void gram_new8_wave(const f32x4* __restrict__ Nv, int nfill, float* __restrict__ partial,
                                               int group, int64_t s0, int64_t s1, int64_t trips, f32x4* lds) {
    using M = New8Map<W>;
    constexpr int LP = 256, STAGE = LP * 4;
    const int tid = threadIdx.x & 255, lane = tid & 63;
    const int l32 = lane & 31, h = lane >> 5;

    f32x16 acc[9];
#pragma unroll
    for (int q = 0; q < 9; ++q)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[q][e] = 0.f;

    int src[4];
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int ps = it * 256 + tid;
        const int row = ps >> 2;
        const int p = (ps & 3) ^ ((row >> 2) & 3);
        src[it] = row >= nfill ? -1 : row * 4 + p;
    }
    f32x4 pre[4];
    auto fetch = [&](int64_t sl) {  // a slab beyond the range reads as zero
        const f32x4* base = Nv + sl * STAGE;
#pragma unroll
        for (int it = 0; it < 4; ++it) pre[it] = (src[it] >= 0 && sl < s1) ? base[src[it]] : f32x4{0.f, 0.f, 0.f, 0.f};
    };
    fetch(s0);
#pragma unroll
    for (int it = 0; it < 4; ++it) lds[it * 256 + tid] = pre[it];
    __syncthreads();

    for (int64_t t = 0; t < trips; ++t) {
        const int cur = (int)(t & 1);
        const bool more = (t + 1 < trips);
        if (more) fetch(s0 + t + 1);
        const f32x4* st = lds + cur * STAGE;
        f32x4 op[2][6];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int p = 2 * j + h;
#pragma unroll
            for (int o = 0; o < 6; ++o) {
                const int r = M::rows[o] * 32 + l32;
                op[j][o] = st[r * 4 + (p ^ ((r >> 2) & 3))];
            }
        }
        __builtin_amdgcn_sched_barrier(0);  // keep the LDS reads above: the scheduler would sink each next to its use
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int q = 0; q < 9; ++q) acc[q] = mfma32(op[j][M::pa[q]][c], op[j][M::pb[q]][c], acc[q]);
        __builtin_amdgcn_sched_barrier(0);
        if (more) {
            f32x4* nx = lds + (cur ^ 1) * STAGE;
#pragma unroll
            for (int it = 0; it < 4; ++it) nx[it * 256 + tid] = pre[it];
        }
        __syncthreads();
    }

#pragma unroll
    for (int q = 0; q < 9; ++q) {
        const int bi = M::rows[M::pa[q]], bj = M::rows[M::pb[q]];
        const int ti = bi >> 1, tj = bj >> 1;
        float* out = partial + ((int64_t)group * 10 + ti * (ti + 1) / 2 + tj) * 4096 + (bi & 1) * 2048 + (bj & 1) * 32;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int r = 8 * (e >> 2) + 4 * h + (e & 3);
            out[r * 64 + l32] = acc[q][e];
        }
    }
}

// One work-group (4 waves, 32 KB of LDS) per column range, two per CU. Used when the launch has the chip to itself.
__global__ __launch_bounds__(256, 2) void gram_new8_kernel(const float* __restrict__ nw, int nfill,
                                                           float* __restrict__ partial, int64_t slabs_total,
                                                           int64_t slabs_per_group) {
    extern __shared__ f32x4 lds[];
    const int group = blockIdx.x;
    int64_t s0 = (int64_t)group * slabs_per_group;
    int64_t s1 = s0 + slabs_per_group;
    if (s1 > slabs_total) s1 = slabs_total;
    if (s0 > s1) s0 = s1;
    const f32x4* Nv = reinterpret_cast<const f32x4*>(nw);
    switch (threadIdx.x >> 6) {  // wave-uniform
        case 0: gram_new8_wave<0>(Nv, nfill, partial, group, s0, s1, s1 - s0, lds); break;
        case 1: gram_new8_wave<1>(Nv, nfill, partial, group, s0, s1, s1 - s0, lds); break;
        case 2: gram_new8_wave<2>(Nv, nfill, partial, group, s0, s1, s1 - s0, lds); break;
        default: gram_new8_wave<3>(Nv, nfill, partial, group, s0, s1, s1 - s0, lds); break;
    }
}

// The same triangle on the bf16 matrix cores with three-way split values (see gram_cross8_split_kernel): the new rows
// of a slab are split when they are staged ([part][k-half][row] pieces, 24 KB per stage), a wave's six operand row
// blocks are 18 LDS reads per 54 matrix-core instructions, and the next slab is split and stored between the six
// groups of matrix-core instructions.
template <int W>
__device__ __forceinline__ void gram_new8_split_wave(const f32x4* __restrict__ Nv, int nfill, float* __restrict__ partial,
                                                     int group, int64_t s0, int64_t s1, u32x4* lds) {
    using M = New8Map<W>;
    constexpr int LP = 256, HALF4 = LP * 4;
    constexpr int HREG = LP + 8;         // pieces per k-half region (padded, see gram_cross8_split_kernel)
    constexpr int PART16 = 2 * HREG;     // pieces per part: [k-half][row]
    constexpr int STAGE16 = 3 * PART16;  // 24.4 KB
    const int tid = threadIdx.x & 255, lane = tid & 63;
    const int l32 = lane & 31, h = lane >> 5;

    f32x16 acc[9];
#pragma unroll
    for (int q = 0; q < 9; ++q)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[q][e] = 0.f;

    int src[4], dst8[4];
    bool used[4];  // (see row_in_use)
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int ps = it * 256 + tid, row = ps >> 2, p = ps & 3;
        src[it] = row_in_use(row, nfill) * 4 + p;
        used[it] = row < nfill;
        dst8[it] = (((p >> 1) * HREG + row) << 1) + (p & 1);
    }
    f32x4 pre[4];
    auto fetch1 = [&](int it, int64_t sl) __attribute__((always_inline)) {
        const int64_t sc = sl < s1 ? sl : s1 - 1;  // beyond the end: repeat (never used)
        pre[it] = Nv[sc * HALF4 + src[it]];
    };
    auto store1 = [&](int it, int buf) __attribute__((always_inline)) {
        uint2* d = reinterpret_cast<uint2*>(lds + buf * STAGE16) + dst8[it];
        unsigned a0, a1, a2, b0, b1, b2;
        if (!used[it]) pre[it] = f32x4{0.f, 0.f, 0.f, 0.f};
        split3_bf16(pre[it][0], pre[it][1], a0, a1, a2);
        split3_bf16(pre[it][2], pre[it][3], b0, b1, b2);
        d[0] = make_uint2(a0, b0);
        d[2 * PART16] = make_uint2(a1, b1);
        d[4 * PART16] = make_uint2(a2, b2);
    };
    if (s0 < s1) {
#pragma unroll
        for (int it = 0; it < 4; ++it) fetch1(it, s0);
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            store1(it, 0);
            fetch1(it, s0 + 1);
        }
    }
    __syncthreads();

    for (int64_t s = s0; s < s1; ++s) {
        const int cur = (int)((s - s0) & 1);
        const u32x4* st = lds + cur * STAGE16 + h * HREG + l32;
        constexpr int NP3 = 3, NQ = 6;
        u32x4 op[6][NP3];
#pragma unroll
        for (int p = 0; p < NP3; ++p)
#pragma unroll
            for (int o = 0; o < 6; ++o) op[o][p] = st[p * PART16 + M::rows[o] * 32];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < NQ; ++k) {  // in the order the parts were read
            constexpr int PA[6] = {0, 0, 1, 1, 0, 2}, PB[6] = {0, 1, 0, 1, 2, 0};
#pragma unroll
            for (int q = 0; q < 9; ++q) acc[q] = mfma_bf16(op[M::pa[q]][PA[k]], op[M::pb[q]][PB[k]], acc[q]);
            if (k < 4) {
                store1(k, cur ^ 1);
                fetch1(k, s + 2);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the LDS stores; the loads for slab s + 2 stay in flight
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }

#pragma unroll
    for (int q = 0; q < 9; ++q) {
        const int bi = M::rows[M::pa[q]], bj = M::rows[M::pb[q]];
        const int ti = bi >> 1, tj = bj >> 1;
        float* out = partial + ((int64_t)group * 10 + ti * (ti + 1) / 2 + tj) * 4096 + (bi & 1) * 2048 + (bj & 1) * 32;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int r = 8 * (e >> 2) + 4 * h + (e & 3);
            out[r * 64 + l32] = acc[q][e];
        }
    }
}

__global__ __launch_bounds__(256, 2) void gram_new8_split_kernel(const float* __restrict__ nw, int nfill,
                                                                 float* __restrict__ partial, int64_t slabs_total,
                                                                 int64_t slabs_per_group, int groups,
                                                                 const int* __restrict__ hole) {
    extern __shared__ u32x4 ldsn[];
    const int group = (int)spare_unit_at(hole);
    if (group < 0 || group >= groups) return;
    int64_t s0 = (int64_t)group * slabs_per_group;
    int64_t s1 = s0 + slabs_per_group;
    if (s1 > slabs_total) s1 = slabs_total;
    if (s0 > s1) s0 = s1;
    const f32x4* Nv = reinterpret_cast<const f32x4*>(nw);
    switch (threadIdx.x >> 6) {  // wave-uniform
        case 0: gram_new8_split_wave<0>(Nv, nfill, partial, group, s0, s1, ldsn); break;
        case 1: gram_new8_split_wave<1>(Nv, nfill, partial, group, s0, s1, ldsn); break;
        case 2: gram_new8_split_wave<2>(Nv, nfill, partial, group, s0, s1, ldsn); break;
        default: gram_new8_split_wave<3>(Nv, nfill, partial, group, s0, s1, ldsn); break;
    }
}

// The triangle of a new half kept in pieces of bf16 (half16): one part, one product, and nothing to convert, so the pieces go
// straight to LDS, three slabs (24 KB) at a time into a ring of three: a barrier per three slabs, two stages on their way.
// (By way of registers and fp32, a slab at a time, the kernel took 590 us beside the eigensolve at D = 2,049,000.)
// FULL: all 256 rows are in use; otherwise the rows beyond nfill are taken as zero.
template <int W, bool FULL>
__device__ __forceinline__ void gram_new8_half_wave(const u32x4* __restrict__ N16, int nfill, float* __restrict__ partial,
                                                    int group, int64_t s0, int64_t s1, u32x4* lds) {
    using M = New8Map<W>;
    constexpr int LP = 256, SL = 3, STAGE = SL * 2 * LP, ML = STAGE / 256;
    const int tid = threadIdx.x & 255, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, h = lane >> 5;

    const int row = FULL ? tid : row_in_use(tid, nfill);

    f32x16 acc[9];
#pragma unroll
    for (int q = 0; q < 9; ++q)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[q][e] = 0.f;

    auto stage = [&](int64_t sl, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < ML; ++q) {
            const int64_t s = sl + q / 2;  // (512 pieces a slab, two loads of 256)
            const int64_t sc = s < s1 ? s : s1 - 1;  // beyond the end: repeat (never used)
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void*)(N16 + sc * (2 * LP) + (q & 1) * 256 + row),
                (__attribute__((address_space(3))) void*)(lds + buf * STAGE + q * 256 + wave * 64), 16, 0, 0);
        }
    };
    if (s0 < s1) {
        stage(s0, 0);
        stage(s0 + SL, 1);
    }
    int buf = 0;
    for (int64_t s = s0; s < s1; s += SL) {
        // all but the last stage's loads have landed; everyone is done with the buffer of the stage before
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0F70 | ML);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        stage(s + 2 * SL, buf == 0 ? 2 : buf - 1);
        const u32x4* st = lds + buf * STAGE + h * LP + l32;
#pragma unroll
        for (int u = 0; u < SL; ++u) {
            if (s + u >= s1) break;  // (uniform)
            u32x4 op[6];
#pragma unroll
            for (int o = 0; o < 6; ++o) {
                op[o] = st[u * 2 * LP + M::rows[o] * 32];
                if (!FULL && M::rows[o] * 32 + l32 >= nfill) op[o] = u32x4{0u, 0u, 0u, 0u};
            }
#pragma unroll
            for (int q = 0; q < 9; ++q) acc[q] = mfma_bf16(op[M::pa[q]], op[M::pb[q]], acc[q]);
        }
        buf = buf == 2 ? 0 : buf + 1;
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): nothing on its way to LDS when the work-group ends

#pragma unroll
    for (int q = 0; q < 9; ++q) {
        const int bi = M::rows[M::pa[q]], bj = M::rows[M::pb[q]];
        const int ti = bi >> 1, tj = bj >> 1;
        float* out = partial + ((int64_t)group * 10 + ti * (ti + 1) / 2 + tj) * 4096 + (bi & 1) * 2048 + (bj & 1) * 32;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int r = 8 * (e >> 2) + 4 * h + (e & 3);
            out[r * 64 + l32] = acc[q][e];
        }
    }
}

template <bool FULL>
__global__ __launch_bounds__(256, 2) void gram_new8_half_kernel(const float* __restrict__ nw, int nfill,
                                                                float* __restrict__ partial, int64_t slabs_total,
                                                                int64_t slabs_per_group, int groups,
                                                                const int* __restrict__ hole) {
    extern __shared__ u32x4 ldsh[];
    const int group = (int)spare_unit_at(hole);
    if (group < 0 || group >= groups) return;
    int64_t s0 = (int64_t)group * slabs_per_group;
    int64_t s1 = s0 + slabs_per_group;
    if (s1 > slabs_total) s1 = slabs_total;
    if (s0 > s1) s0 = s1;
    const u32x4* N16 = half16(nw, 256, slabs_total);
    switch (threadIdx.x >> 6) {  // wave-uniform
        case 0: gram_new8_half_wave<0, FULL>(N16, nfill, partial, group, s0, s1, ldsh); break;
        case 1: gram_new8_half_wave<1, FULL>(N16, nfill, partial, group, s0, s1, ldsh); break;
        case 2: gram_new8_half_wave<2, FULL>(N16, nfill, partial, group, s0, s1, ldsh); break;
        default: gram_new8_half_wave<3, FULL>(N16, nfill, partial, group, s0, s1, ldsh); break;
    }
}

// ... of rows on their way from the caller's batch into the half, which saves reading them a second time: a stage is four slabs, 128 bytes of every row, loaded as insert16_kernel
// does (lane = (row, piece of four neighbours), the two halves of a line one after the other), two stages ahead, and goes from the
// registers to LDS and to the half. 256 rows of 2,049,000 beside an eigensolve: 490 us (4.3 TB/s), stored and multiplied by a kernel each
// 480 + 240. (Fp32 rows, six products a pair and no registers for a second slab ahead, took 1090 us where two kernels take 1010.)
template <int W>
__device__ __forceinline__ void gram_new8_rows16_wave(u32x4* __restrict__ N16, const uint16_t* __restrict__ G, int64_t D, int nfill,
                                                      float* __restrict__ partial, int group, int64_t s0, int64_t s1, u32x4* lds) {
    using M = New8Map<W>;
    constexpr int LP = 256, SL = 4, STAGE = SL * 2 * LP, KC = SL * DC;  // KC: columns of a stage
    const int lane = threadIdx.x & 63;
    const int l32 = lane & 31, h = lane >> 5;
    const int row = W * 64 + (lane & 15), piece = lane >> 4;  // (wave W loads rows 64 W .. + 63)

    f32x16 acc[9];
#pragma unroll
    for (int q = 0; q < 9; ++q)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[q][e] = 0.f;
    unsigned src[4];  // bytes from the first column of a stage in row 0
#pragma unroll
    for (int g = 0; g < 4; ++g) src[g] = (unsigned)row_in_use(row + 16 * g, nfill) * (unsigned)D * 2u + 16u * piece;

    // (a stage that ends beyond the range of the work-group reads columns of the next one's, or none)
    auto fetch = [&](int64_t sl, u32x4 (&v)[8]) __attribute__((always_inline)) {
        const int64_t c = (sl < s1 ? sl : s1 - 1) * DC;
        const char* g0 = reinterpret_cast<const char*>(G + c);
        if (c + KC <= D) {  // (uniform)
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = reinterpret_cast<const Eight*>(g0 + src[q >> 1] + 64 * (q & 1))->v;
        } else {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int left = (int)(D - c) - 8 * piece - 32 * (q & 1);
                const uint16_t* g = reinterpret_cast<const uint16_t*>(g0 + src[q >> 1] + 64 * (q & 1));
                u32x4 x = {0u, 0u, 0u, 0u};
                if (left >= 8) {
                    x = reinterpret_cast<const Eight*>(g)->v;
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) x[e >> 1] |= e < left ? (unsigned)g[e] << (16 * (e & 1)) : 0u;
                }
                v[q] = x;
            }
        }
    };
    auto store = [&](int64_t sl, int buf, const u32x4 (&v)[8]) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int at = (4 * (q & 1) + piece) * LP + row + 16 * (q >> 1);
            lds[buf * STAGE + at] = v[q];
            if (sl + 2 * (q & 1) + (piece >> 1) < s1) N16[sl * (2 * LP) + at] = v[q];
        }
    };
    u32x4 va[8], vb[8];
    if (s0 < s1) {
        fetch(s0, va);
        fetch(s0 + SL, vb);
    }
    auto step = [&](int64_t s, int buf, u32x4 (&v)[8]) __attribute__((always_inline)) {
        if (s >= s1) return;  // (uniform)
        store(s, buf, v);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0); the loads stay in flight
        __builtin_amdgcn_s_barrier();        // (whoever stores into this buffer next has been past the other one's barrier)
        asm volatile("" ::: "memory");
        fetch(s + 2 * SL, v);
        const u32x4* st = lds + buf * STAGE + h * LP + l32;
#pragma unroll
        for (int u = 0; u < SL; ++u) {
            if (s + u >= s1) break;  // (uniform)
            u32x4 op[6];
#pragma unroll
            for (int o = 0; o < 6; ++o) {
                op[o] = st[u * 2 * LP + M::rows[o] * 32];
                if (M::rows[o] * 32 + l32 >= nfill) op[o] = u32x4{0u, 0u, 0u, 0u};
            }
#pragma unroll
            for (int q = 0; q < 9; ++q) acc[q] = mfma_bf16(op[M::pa[q]], op[M::pb[q]], acc[q]);
        }
    };
    for (int64_t s = s0; s < s1; s += 2 * SL) {
        step(s, 0, va);
        step(s + SL, 1, vb);
    }

#pragma unroll
    for (int q = 0; q < 9; ++q) {
        const int bi = M::rows[M::pa[q]], bj = M::rows[M::pb[q]];
        const int ti = bi >> 1, tj = bj >> 1;
        float* out = partial + ((int64_t)group * 10 + ti * (ti + 1) / 2 + tj) * 4096 + (bi & 1) * 2048 + (bj & 1) * 32;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int r = 8 * (e >> 2) + 4 * h + (e & 3);
            out[r * 64 + l32] = acc[q][e];
        }
    }
}

__global__ __launch_bounds__(256, 2) void gram_new8_rows16_kernel(float* __restrict__ nw, const uint16_t* __restrict__ G, int64_t D,
                                                                  int nfill, float* __restrict__ partial, int64_t slabs_total,
                                                                  int64_t slabs_per_group, int groups,
                                                                  const int* __restrict__ hole) {
    extern __shared__ u32x4 ldsr[];
    const int group = (int)spare_unit_at(hole);
    if (group < 0 || group >= groups) return;
    int64_t s0 = (int64_t)group * slabs_per_group;
    int64_t s1 = s0 + slabs_per_group;
    if (s1 > slabs_total) s1 = slabs_total;
    if (s0 > s1) s0 = s1;
    u32x4* N16 = const_cast<u32x4*>(half16(nw, 256, slabs_total));
    switch (threadIdx.x >> 6) {  // wave-uniform
        case 0: gram_new8_rows16_wave<0>(N16, G, D, nfill, partial, group, s0, s1, ldsr); break;
        case 1: gram_new8_rows16_wave<1>(N16, G, D, nfill, partial, group, s0, s1, ldsr); break;
        case 2: gram_new8_rows16_wave<2>(N16, G, D, nfill, partial, group, s0, s1, ldsr); break;
        default: gram_new8_rows16_wave<3>(N16, G, D, nfill, partial, group, s0, s1, ldsr); break;
    }
}

// C (NP x NP, fp64, both triangles) = sum over groups of the partial tiles, in group order. With q = P/2:
// known_top: tiles with ti < q are not summed, their block is diag(known) (the top rows are the rows the last shrink
// wrote, whose Gram matrix it recorded). Otherwise tile (ti, tj) comes from the first of the sources whose mode covers it
// (launches of different modes write separate partial buffers; mode 3: the mode-2 kernel given the top rows).
struct GramSrc {
    const float* partial;
    int mode, t0, tiles, groups;
};
__device__ __forceinline__ int gram_src_index(const GramSrc& g, int P, int t, int ti, int tj) {
    const int q = P >> 1;
    if (g.mode == 0) return (t >= g.t0 && t < g.t0 + g.tiles) ? t - g.t0 : -1;
    if (g.mode == 1) return (ti >= q && tj < q) ? (ti - q) * q + tj : -1;
    if (g.mode == 3) return ti < q ? t : -1;
    return (ti >= q && tj >= q) ? (ti - q) * (ti - q + 1) / 2 + (tj - q) : -1;
}
// SEG threads share an element's groups (in runs, added in order afterwards): with one thread each, a loop over hundreds of
// groups with eight loads in flight, the kernel took 22 to 25 us after the launches that fill the chip.
template <int SEG>
__global__ __launch_bounds__(256) void gram_reduce_kernel(GramSrc a, GramSrc b, GramSrc top, double* __restrict__ C, int NP,
                                                          int known_top, const double* __restrict__ known) {
    constexpr int EL = 256 / SEG;  // elements of a work-group
    __shared__ double part[SEG > 1 ? SEG : 1][EL];
    const int P = NP / 64;
    const int t = blockIdx.x;
    const int el = threadIdx.x % EL, seg = threadIdx.x / EL;
    const int e = blockIdx.y * EL + el;  // 0..4095
    int ti, tj;
    tile_coords(t, ti, tj);
    const int r = e >> 6, c = e & 63;
    const int gr = ti * 64 + r, gc = tj * 64 + c;
    const bool diag = known_top && ti < (P >> 1);
    double s = 0.0;
    if (!diag) {
        const int ia = gram_src_index(a, P, t, ti, tj);
        const int ib = gram_src_index(b, P, t, ti, tj);
        const GramSrc& g = ia >= 0 ? a : (ib >= 0 ? b : top);
        const int idx = ia >= 0 ? ia : (ib >= 0 ? ib : gram_src_index(top, P, t, ti, tj));
        if (idx >= 0) {
            const float* p0 = g.partial + (int64_t)idx * 4096 + e;
            const int64_t gstride = (int64_t)g.tiles * 4096;
            const int per = (g.groups + SEG - 1) / SEG;
            int k = seg * per;
            const int k1 = k + per < g.groups ? k + per : g.groups;
            for (; k + 8 <= k1; k += 8) {  // eight loads in flight, added in group order
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = p0[(k + u) * gstride];
#pragma unroll
                for (int u = 0; u < 8; ++u) s += (double)v[u];
            }
            for (; k < k1; ++k) s += (double)p0[k * gstride];
        }
    }
    if constexpr (SEG > 1) {
        part[seg][el] = s;
        __syncthreads();
        if (seg > 0) return;
#pragma unroll
        for (int q = 1; q < SEG; ++q) s += part[q][el];
    }
    if (ti == tj && c > r) return;  // the diagonal tiles hold both triangles; keep one
    if (diag) s = gr == gc ? known[gr] : 0.0;
    C[(int64_t)gr * NP + gc] = s;
    C[(int64_t)gc * NP + gr] = s;
}

// ---- 64 buffer rows: the Gram matrix, and with it the rebuild of the shrink before ---------------------------------
// top x top, new x top and new x new of [top; next], or (REBUILD, where the next block's rows are in the other half already: the
// reduction's launch has stored them) of [M [top; nw]; next], whose first rows are formed and stored on the way: the wave that forms the
// new top rows of 32 columns multiplies them there and then. Their product is formed transposed, which leaves a lane row l % 32 of the
// result at the columns 8 q + 4 h + j, q, j < 4: four stores of 16 bytes, and, one column of either h a step, the operand that a contraction
// over the columns takes; rows that are loaded come in the same order. No LDS but for the sums at the end, the coefficients stay in
// registers, and a wave goes through its units with the next one's rows on their way. The bits of the Gram matrix are the same
// either way. HS: stages of 16 rows of a half in use.
// Bound by memory where rows are long: with the rebuild 1.05 GB at 2,049,000 columns in 215 to 235 us by the card, where a kernel for each took 130 and (all
// four blocks, through LDS) 190; by the launch where they are short (512 columns: 6.2 us, were 5.2 and 4.9). In between the two are
// even (51,300: a unit for each wave, 12.8 us for 7.5 and 6.3). An update of 17 blocks of 32 rows: 9.5 -> 6.0 ms at 2,049,000, 3.31 -> 2.36 at
// 524,288; a job of 64 blocks of 512 columns: 5.39 -> 5.24.
template <int HS, bool REBUILD>
__global__ __launch_bounds__(256, 2) void gram64_kernel(std::conditional_t<REBUILD, float, const float>* top, int top_rows,
                                                        const float* __restrict__ nw, const float* __restrict__ next, int rows,
                                                        const float* __restrict__ Mc, float* __restrict__ partial, int64_t S, int64_t units) {
    constexpr int LP = 32, K = REBUILD ? 8 * HS : 1;  // steps of two rows of a half
    __shared__ float sums[4][48][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, h = lane >> 5;
    f32x4 m[2][HS][2];  // coefficients of the top's and of the block's stages for row c of the result (see coeff_offset)
    if constexpr (REBUILD) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int g = 0; g < HS; ++g)
#pragma unroll
                for (int p = 0; p < 2; ++p)
                    m[b][g][p] = reinterpret_cast<const f32x4*>(Mc)[(2 * b + g) * (16 * LP / 4) + (h * LP + c) * 2 + (p ^ ((c >> 3) & 1))];
    }
    struct Rows {
        float t[K], b[K];  // REBUILD: rows 2 s + h of column c of the unit: top, block;
        f32x4 o[4];        // otherwise row c of the top at columns 8 q + 4 h ..
        f32x4 n[4];        // row c of the next block there
    };
    const int nrow = row_in_use(c, rows), trow = row_in_use(c, top_rows);
    auto fetch = [&](int64_t u, Rows& r) __attribute__((always_inline)) {
        const int64_t s0 = 2 * (u < units ? u : units - 1), s1 = s0 + 1 < S ? s0 + 1 : s0;  // (beyond the end: repeated, not used)
        if constexpr (REBUILD) {
            const int64_t col = ((c < 16 ? s0 : s1) * LP + h) * DC + (c & 15);
#pragma unroll
            for (int s = 0; s < K; ++s) r.t[s] = top[col + 2 * s * DC];
#pragma unroll
            for (int s = 0; s < K; ++s) r.b[s] = nw[col + 2 * s * DC];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t at = (q < 2 ? s0 : s1) * LP * DC + 8 * (q & 1) + 4 * h;
            if constexpr (!REBUILD) r.o[q] = *reinterpret_cast<const f32x4*>(top + at + trow * DC);
            r.n[q] = *reinterpret_cast<const f32x4*>(next + at + nrow * DC);
        }
    };
    f32x16 tt, nt, nn;
#pragma unroll
    for (int i = 0; i < 16; ++i) tt[i] = nt[i] = nn[i] = 0.f;
    auto unit = [&](int64_t u, Rows& r) __attribute__((always_inline)) {
        const bool both = 2 * u + 1 < S;  // (wave-uniform) the second slab is there
        f32x16 acc;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = REBUILD || c >= top_rows ? 0.f : r.o[i >> 2][i & 3];
        if constexpr (REBUILD) {
#pragma unroll
            for (int s = 0; s < K; ++s) acc = mfma32(r.t[s], m[0][s >> 3][s >> 2 & 1][s & 3], acc);
#pragma unroll
            for (int s = 0; s < K; ++s) acc = mfma32(2 * s + h < rows ? r.b[s] : 0.f, m[1][s >> 3][s >> 2 & 1][s & 3], acc);
        }
        float x[16];  // of the next block
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const bool there = i < 8 || both;
            x[i] = there && c < rows ? r.n[i >> 2][i & 3] : 0.f;
            acc[i] = there ? acc[i] : 0.f;
        }
        if constexpr (REBUILD) {
            if (c < 16 * HS) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (q < 2 || both)
                        *reinterpret_cast<f32x4*>(top + ((2 * u + (q >> 1)) * LP + c) * DC + 8 * (q & 1) + 4 * h) =
                            f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
            }
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            nn = mfma32(x[i], x[i], nn);
            nt = mfma32(x[i], acc[i], nt);
            tt = mfma32(acc[i], acc[i], tt);
        }
    };
    const int64_t stride = (int64_t)gridDim.x * 4, u0 = (int64_t)blockIdx.x * 4 + wave;
    if (u0 < units) {
        Rows ra, rb;
        fetch(u0, ra);
        for (int64_t u = u0; u < units; u += 2 * stride) {
            fetch(u + stride, rb);
            unit(u, ra);
            if (u + stride >= units) break;
            fetch(u + 2 * stride, ra);
            unit(u + stride, rb);
        }
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        sums[wave][i][lane] = tt[i];
        sums[wave][16 + i][lane] = nt[i];
        sums[wave][32 + i][lane] = nn[i];
    }
    __syncthreads();
    float* const out = partial + (int64_t)blockIdx.x * 4096;  // a 64 x 64 tile, of which the reduction reads the lower triangle
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        const int i = 4 * k + wave, e = i & 15;
        const float s = (float)(((double)sums[0][i][lane] + (double)sums[1][i][lane]) +
                                ((double)sums[2][i][lane] + (double)sums[3][i][lane]));  // (rounded once)
        const int row = 8 * (e >> 2) + 4 * h + (e & 3) + (i < 16 ? 0 : LP), col = c + (i < 32 ? 0 : LP);
        out[row * 64 + col] = s;
    }
}

hipError_t launch_rebuild_gram(float* top, const float* nw, const float* next, const float* Mc, float* partial, const GramPlan& p,
                               const Dims& d, hipStream_t st) {
    if (d.NP != 64 || p.mode != 0 || p.t0 != 0) return hipErrorInvalidValue;
    const auto kern = d.ell <= 16 ? gram64_kernel<1, true> : gram64_kernel<2, true>;
    hipLaunchKernelGGL(kern, dim3(p.groups), dim3(256), 0, st, top, d.LP, nw, next, d.ell, Mc, partial, d.S, (d.S + 1) / 2);
    return hipGetLastError();
}

// wg_per_cu = 2 fills the chip. wg_per_cu = 1 is for the launch that shares the chip with the eigensolve (side stream): it
// leaves an eighth of the CUs, an XCD, to the eigensolve's reduction (see spare_unit_at).
GramPlan gram_plan(const Dims& d, int num_cu, int mode, bool skip_top, int wg_per_cu) {
    GramPlan p;
    const bool side = wg_per_cu == 1;
    const int P = d.NP / 64, q = P / 2;
    p.mode = mode;
    p.t0 = 0;
    if (mode == 0) {
        p.t0 = skip_top ? q * (q + 1) / 2 : 0;
        p.tiles = P * (P + 1) / 2 - p.t0;
    } else if (mode == 1) {
        p.tiles = (P - q) * q;
    } else {
        p.tiles = (P - q) * (P - q + 1) / 2;
    }
    p.wg_per_group = (p.tiles + 5) / 6;
    if (mode == 1 && P == 8) p.wg_per_group = 2;  // gram_cross8_kernel: 8 wave tiles of 128 x 64
    // gram_new8_kernel (the whole triangle in one work-group) when the launch has the chip to itself
    if (mode == 2 && P == 8 && !side) p.wg_per_group = 1;
    const int cus = side && num_cu > 32 ? num_cu / 8 * 7 : num_cu;
    int g;
    if (P == 1) {  // gram64_kernel: a wave takes units of two slabs
        const int64_t wgs = ((d.S + 1) / 2 + 3) / 4;
        g = wgs < (int64_t)wg_per_cu * num_cu ? (int)wgs : wg_per_cu * num_cu;
    } else {
        g = (wg_per_cu * cus / p.wg_per_group) / 8 * 8;
        if (g < 8) g = 8;
        // At least 4 slabs per group so that small problems do not drown in partial tiles; 2 where there are few slabs: as fast (us a
        // cycle, 2 / 4: ell = 64, 159.4 / 160.4 at 512 columns, 162.6 / 161.2 at 4096; 100, 256.0 / 254.9 and 262.6 / 260.5; 128, 304.6 / 303.1
        // and 309.9 / 308.6; 256, 682.6 / 681.0 and 684.8 / 683.7; runs of a side differ by 1%) and half as long sums in fp32.
        const int64_t least = d.S <= 256 ? 2 : 4;
        int64_t gmax = ((d.S + least - 1) / least + 7) / 8 * 8;
        if (gmax < 8) gmax = 8;
        if (g > gmax) g = (int)gmax;
    }
    p.groups = g;
    p.slabs_per_group = (d.S + g - 1) / g;
    p.partial_floats = (size_t)g * p.tiles * 4096;
    return p;
}

GramPlan gram_plan_split(const GramPlan& base, const Dims& d, int groups) {
    GramPlan p = base;
    const bool ok = d.NP == 512 && ((base.mode == 1 && base.tiles == 16) || (base.mode == 2 && base.tiles == 10));
    if (!ok) {
        p.tiles = 0;  // not available
        return p;
    }
    p.wg_per_group = 1;
    p.split = true;
    if (groups > 0) {
        int64_t gmax = ((d.S + 3) / 4 + 7) / 8 * 8;
        if (gmax < 8) gmax = 8;
        p.groups = groups > gmax ? (int)gmax : groups;
        p.slabs_per_group = (d.S + p.groups - 1) / p.groups;
        p.partial_floats = (size_t)p.groups * p.tiles * 4096;
    }
    return p;
}

// Lane offsets are 32-bit, over 256 rows.
bool gram_rows_ok(const GramPlan& p, const Dims& d) {
    return p.mode == 2 && p.split && d.NP == 512 && d.D * 2 * 256 + 256 < ((int64_t)1 << 32);
}
hipError_t launch_gram_rows16(const void* G, int rows, float* nw, float* partial, const GramPlan& p, const Dims& d, const int* hole,
                              hipStream_t st) {
    constexpr int LDS = 2 * 4 * 2 * 256 * 16;  // two stages of four slabs
    if (hipError_t ea = ensure_dynamic_lds((const void*)gram_new8_rows16_kernel, LDS); ea != hipSuccess) return ea;
    hipLaunchKernelGGL(gram_new8_rows16_kernel, dim3((unsigned)spare_grid_at(p.groups, hole)), dim3(256), LDS, st, nw,
                       (const uint16_t*)G, d.D, rows, partial, d.S, p.slabs_per_group, p.groups, hole);
    return hipGetLastError();
}

hipError_t launch_gram(const float* top, const float* nw, int nfill, float* partial, const GramPlan& p, const Dims& d,
                       hipStream_t st, bool new_one, const int* hole) {
    return launch_gram_tops(GramTops{{top}, 0, d.LP}, 1, nw, nfill, partial, p, d, st, new_one, hole);
}

hipError_t launch_gram_blocks(const GramTops& tops, int count, const float* nw, int nfill, float* partial, const GramPlan& p,
                              const Dims& d, hipStream_t st, const int* hole) {
    constexpr int LDS = 3 * 2 * 2 * 2 * 256 * 16;  // three stages of two slabs
    if (count <= 0) return hipSuccess;
    if (hipError_t ea = ensure_dynamic_lds((const void*)gram_cross8_half_kernel, LDS); ea != hipSuccess) return ea;
    hipLaunchKernelGGL(gram_cross8_half_kernel, dim3((unsigned)spare_grid_at(range_units(p.groups, count, hole ? 0 : -1), hole)), dim3(512), LDS, st, tops, nw, nfill,
                       partial, d.S, p.slabs_per_group, p.groups, count, hole);
    return hipGetLastError();
}

hipError_t launch_gram_tops(const GramTops& tops, int count, const float* nw, int nfill, float* partial, const GramPlan& p,
                            const Dims& d, hipStream_t st, bool new_one, const int* hole) {
    if (p.tiles <= 0 || count <= 0) return hipSuccess;
    const float* const top = tops.p[0];
    dim3 grid((unsigned)(p.groups * p.wg_per_group));
    size_t lds = (size_t)2 * d.NP * 64;
    if (p.mode == 1 && d.NP == 512 && p.split) {
        constexpr int LDS_SPLIT = 2 * 3 * 2 * (512 + 8) * 16;  // two stages of [part][k-half][row + pad] pieces
        const void* kern = new_one ? (const void*)gram_cross8_split_kernel<true> : (const void*)gram_cross8_split_kernel<false>;
        if (hipError_t ea = ensure_dynamic_lds(kern, LDS_SPLIT); ea != hipSuccess) return ea;
        const dim3 wgs((unsigned)spare_grid_at(p.groups, hole), count);
        if (new_one)
            hipLaunchKernelGGL(gram_cross8_split_kernel<true>, wgs, dim3(512), LDS_SPLIT, st, tops, nw, nfill, partial, d.S,
                               p.slabs_per_group, p.groups, hole);
        else
            hipLaunchKernelGGL(gram_cross8_split_kernel<false>, wgs, dim3(512), LDS_SPLIT, st, tops, nw, nfill, partial,
                               d.S, p.slabs_per_group, p.groups, hole);
        return hipGetLastError();
    }
    if (p.mode == 1 && d.NP == 512) {
        if (hipError_t ea = ensure_dynamic_lds((const void*)gram_cross8_kernel, 65536); ea != hipSuccess) return ea;
        hipLaunchKernelGGL(gram_cross8_kernel, grid, dim3(256), lds, st, top, nw, nfill, partial, d.S, p.slabs_per_group);
        return hipGetLastError();
    }
    if (p.mode == 2 && d.NP == 512 && p.split) {
        const dim3 wgs((unsigned)spare_grid_at(p.groups, hole));
        if (new_one) {
            constexpr int LDS = 3 * 3 * 2 * 256 * 16;  // three stages of three slabs
            const bool full = nfill >= 256;
            const void* kern = full ? (const void*)gram_new8_half_kernel<true> : (const void*)gram_new8_half_kernel<false>;
            if (hipError_t ea = ensure_dynamic_lds(kern, LDS); ea != hipSuccess) return ea;
            if (full)
                hipLaunchKernelGGL(gram_new8_half_kernel<true>, wgs, dim3(256), LDS, st, nw, nfill, partial, d.S,
                                   p.slabs_per_group, p.groups, hole);
            else
                hipLaunchKernelGGL(gram_new8_half_kernel<false>, wgs, dim3(256), LDS, st, nw, nfill, partial, d.S,
                                   p.slabs_per_group, p.groups, hole);
        } else {
            constexpr int LDS = 2 * 3 * 2 * (256 + 8) * 16;  // two stages
            hipLaunchKernelGGL(gram_new8_split_kernel, wgs, dim3(256), LDS, st, nw, nfill, partial, d.S, p.slabs_per_group,
                               p.groups, hole);
        }
        return hipGetLastError();
    }
    if (p.mode == 2 && d.NP == 512 && p.wg_per_group == 1) {
        if (hipError_t ea = ensure_dynamic_lds((const void*)gram_new8_kernel, 65536); ea != hipSuccess) return ea;
        hipLaunchKernelGGL(gram_new8_kernel, grid, dim3(256), 32768, st, nw, nfill, partial, d.S, p.slabs_per_group);
        return hipGetLastError();
    }
    if (d.NP == 64) {
        if (p.mode != 0 || count != 1 || hole) return hipErrorInvalidValue;
        hipLaunchKernelGGL((gram64_kernel<2, false>), grid, dim3(256), 0, st, top, tops.rows, nullptr, nw, nfill, nullptr, partial, d.S,
                           (d.S + 1) / 2);
        return hipGetLastError();
    }
    switch (d.NP / 64) {
#define SAGE_GRAM_CASE(PP)                                                                                          \
    case PP: {                                                                                                      \
        const auto kern = p.mode == 2 ? gram_kernel<PP, true> : gram_kernel<PP, false>;                             \
        if (hipError_t ea = ensure_dynamic_lds((const void*)kern, 65536); ea != hipSuccess) return ea;              \
        hipLaunchKernelGGL(kern, dim3((unsigned)spare_grid_at(grid.x, hole), count), dim3(256), lds, st, tops, nw, nfill,   \
                           partial, p.mode, p.t0, p.tiles, p.wg_per_group, d.S, p.slabs_per_group, (int)grid.x, hole);  \
    } break;
        SAGE_GRAM_CASE(2)
        SAGE_GRAM_CASE(4)
        SAGE_GRAM_CASE(8)
#undef SAGE_GRAM_CASE
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// a, b: the launches whose partial tiles make up C (b may be null); known: LP doubles, read when known_top.
// partial_top, top: a mode-2 launch that was given the top rows in place of the new ones (may be null)
hipError_t launch_gram_reduce(const float* partial_a, const GramPlan& a, const float* partial_b, const GramPlan* b,
                              double* C, bool known_top, const double* known, const Dims& d, hipStream_t st,
                              const float* partial_top, const GramPlan* top, hipEvent_t done) {
    const int P = d.NP / 64;
    GramSrc sa{partial_a, a.mode, a.t0, a.tiles, a.groups};
    GramSrc sb{partial_b, b ? b->mode : 0, b ? b->t0 : 0, b ? b->tiles : 0, b ? b->groups : 0};
    GramSrc stop{partial_top, top ? 3 : 0, 0, top ? top->tiles : 0, top ? top->groups : 0};
    void (*const kern)(GramSrc, GramSrc, GramSrc, double*, int, int, const double*) =
        sa.groups >= 64 ? gram_reduce_kernel<8> : gram_reduce_kernel<1>;
    const dim3 grid(P * (P + 1) / 2, sa.groups >= 64 ? 128 : 16);
    // `done` rides on the launch's own completion: recorded after it, it is a packet of its own, and the reduction that follows
    // started 6.7 us later (4096 rows of 5130 at sketch size 64: 12.88 ms with the packet, 12.70 without).
    if (done)
        hipExtLaunchKernelGGL(kern, grid, dim3(256), 0, st, nullptr, done, 0, sa, sb, stop, C, d.NP, known_top ? 1 : 0, known);
    else
        hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, sa, sb, stop, C, d.NP, known_top ? 1 : 0, known);
    return hipGetLastError();
}

}  // namespace sage
