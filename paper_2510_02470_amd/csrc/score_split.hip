// Scoring pass projection on the bf16 matrix cores with a split basis (Algorithm 1, Phase II, first line:
// z_i = V_k^T g_i; Method, "Two-pass scoring").
//
// At k = 128 the projection does 2k/e = 64..128 flop per byte of input row, far above what the fp32 matrix
// cores sustain per byte of HBM traffic, so the fp32 kernel in score.hip is compute-bound at a small fraction of
// the memory bandwidth. Here every fp32 basis entry is written as v = hi + lo with hi = bf16(v), lo = bf16(v - hi)
// (|v - hi - lo| <= 2^-17 |v|), bf16 rows are used as they are (exact), fp32 rows are split the same way in
// registers, and the products g*hi, g*lo (and glo*hi for fp32 rows) are accumulated in fp32 by
// v_mfma_f32_32x32x16_bf16. The error against an fp32 product is a few 2^-17 relative per term, below the fp32
// accumulation error over D ~ 1e6 terms.
//
// Work-group = 512 threads = 8 waves, one work-group per CU. A wave owns 64 batch rows x KP basis columns (2 x KP/32
// accumulator tiles). Its rows are loaded whole memory lines at a time and turned to the matrix cores' order through LDS of
// the wave's own (nobody else needs them); the basis operand is shared by the waves and is streamed through LDS with direct
// global->LDS loads. The basis is kept in HBM as "images": for each chunk of KC columns exactly the bytes LDS will hold,
// so staging is a linear copy.
#include <type_traits>

#include "sage_internal.h"

namespace sage {

// ---- basis images -----------------------------------------------------------------------------------------
// Chunk c covers columns c*KC .. c*KC + KC - 1 (KC = 64 for bf16 rows, 32 for fp32 rows: 128 bytes of a row).
// Its image has 2*KP rows of KC bf16: image row cc < KP is hi(v_cc), image row KP + cc is lo(v_cc). A row is cut
// into 16-byte pieces (8 columns); piece p of image row cc is stored at position swz(cc, p) of that row so that the
// lanes of a matrix-core operand read (32 consecutive image rows, one piece each) spread over all LDS banks. A
// 16-byte read is served 16 lanes at a time from 64 banks of 4 bytes (256 bytes), so the 16 pieces that 16
// consecutive image rows ask for must fall on 16 different 16-byte columns modulo 256 bytes:
//   KC = 64 (8 pieces, 128 B rows: even and odd rows are 128 bytes apart): swz = p ^ ((cc >> 1) & 7);
//   KC = 32 (4 pieces,  64 B rows: four rows span 256 bytes):              swz = p ^ ((cc >> 2) & 3).
// (With swz = p ^ (cc & 7), conflict-free for 8 lanes over 32 banks, the hardware counters showed one conflict
// cycle for every useful cycle of the operand reads.)
template <int KC>
__device__ __forceinline__ int img_piece(int cc, int p) {
    if constexpr (KC == 64) return cc * 8 + (p ^ ((cc >> 1) & 7));
    else return cc * 4 + (p ^ ((cc >> 2) & 3));
}

// (Images of three parts, for project_any_kernel, have KP rows more: hi, mid, lo.)
//
// One thread takes 8 columns of one basis row and writes the 16-byte piece of each part (a thread per piece read the basis once
// per part: 414 us for 128 rows of 2,049,000, now 384, 5.5 TB/s read and written). Vblk is the fp32 column-slab basis
// (KP rows); columns >= D are zero there and columns >= Dp are written as zero here.
template <int KC, int PARTS>
__global__ __launch_bounds__(256) void basis_split_kernel(const float* __restrict__ Vblk, int KP, int64_t Dp,
                                                          int64_t chunks, u32x4* __restrict__ img) {
    constexpr int PPR = KC / 8;
    const int64_t per_chunk = (int64_t)KP * PPR;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= chunks * per_chunk) return;
    const int64_t c = i / per_chunk;
    const int rem = (int)(i % per_chunk);
    const int cc = rem / PPR, p = rem % PPR;
    const int64_t d0 = c * KC + p * 8;
    f32x4 v[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    if (d0 < Dp) {  // 8 | DC: the piece lies inside one slab
        const f32x4* src = reinterpret_cast<const f32x4*>(Vblk + blk_off(d0, cc, KP));
        v[0] = src[0];
        v[1] = src[1];
    }
    u32x4 out[PARTS];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float x = v[e >> 1][2 * (e & 1)], y = v[e >> 1][2 * (e & 1) + 1];
        if constexpr (PARTS == 3) {
            unsigned a, b, l;
            split3_bf16(x, y, a, b, l);
            out[0][e] = a;
            out[1][e] = b;
            out[2][e] = l;
        } else {
            const unsigned hi = pack_bf16(x, y);
            out[0][e] = hi;
            out[1][e] = pack_bf16(x - __uint_as_float(hi << 16), y - __uint_as_float(hi & 0xffff0000u));
        }
    }
#pragma unroll
    for (int q = 0; q < PARTS; ++q) img[c * (PARTS * per_chunk) + img_piece<KC>(q * KP + cc, p)] = out[q];
}

hipError_t launch_basis_split(const float* Vblk, int KP, int dtype, int parts, void* img, const Dims& d, hipStream_t st) {
    const int KC = dtype == SAGE_BF16 ? 64 : 32;
    const int64_t chunks = (d.D + KC - 1) / KC;
    const int64_t total = chunks * KP * (KC / 8);
    dim3 grid((unsigned)((total + 255) / 256));
#define SAGE_IMG(K, P) \
    hipLaunchKernelGGL((basis_split_kernel<K, P>), grid, dim3(256), 0, st, Vblk, KP, d.Dp, chunks, (u32x4*)img)
    if (KC == 64 && parts == 2) SAGE_IMG(64, 2);
    else if (KC == 64) SAGE_IMG(64, 3);
    else if (parts == 2) SAGE_IMG(32, 2);
    else SAGE_IMG(32, 3);
#undef SAGE_IMG
    return hipGetLastError();
}

size_t basis_image_bytes(int KP, int dtype, int parts, const Dims& d) {
    const int KC = dtype == SAGE_BF16 ? 64 : 32;
    const int64_t chunks = (d.D + KC - 1) / KC;
    return (size_t)chunks * parts * KP * KC * 2;
}

// ---- projection -------------------------------------------------------------------------------------------
// fp32 pieces (8 values in two u32x4) -> bf16 hi and lo operands
__device__ __forceinline__ void split8(const u32x4& x0, const u32x4& x1, u32x4& hi, u32x4& lo) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const u32x4& s = e < 2 ? x0 : x1;
        float x = __uint_as_float(s[(2 * e) & 3]), y = __uint_as_float(s[(2 * e + 1) & 3]);
        unsigned hh = pack_bf16(x, y);
        hi[e] = hh;
        lo[e] = pack_bf16(x - __uint_as_float(hh << 16), y - __uint_as_float(hh & 0xffff0000u));
    }
}

// Rows of a batch are D * sizeof(T) bytes apart, which in general is not a multiple of the 128-byte memory line, so a
// row's k-th 128 bytes straddle two lines and a kernel that walks every row in steps of 128 bytes from the row
// start fetches most lines twice. Here a wave only holds rows whose start addresses are congruent modulo 128 (rows
// w, w + 8, w + 16, ... of the work-group's 512: 8 * pitch is a multiple of 128 because the pitch is a multiple of 16)
// and walks them in line-aligned windows: with phi = (row address mod 128) / (bytes of 8 columns), window m of the
// wave is the 128 bytes that start 8*phi columns before column m*KC. Its basis operand is then the last phi pieces
// of image m-1 followed by the first PPR-phi pieces of image m, so LDS keeps a ring of four images: m-1 and m in
// use, m+1 and m+2 on their way in (an image requested only one window ahead arrived late: with the memory system
// saturated a load takes about two windows). The first and the last window of a split reach into the neighbouring
// splits; those pieces of the row operand are zeroed.
//
// Work-group = 512 threads = 8 waves (two per SIMD), one per CU, 512 batch rows x KP basis columns; a wave owns 64
// rows (2 accumulator row tiles) x KP columns. The rows of window m+2 are requested into registers during window m and
// turned at the start of window m+2; images are streamed with direct global->LDS loads, also two windows ahead.
template <typename T>
struct RowOp {
    u32x4 v[4];  // bf16 rows: v[j] = k-step j; fp32 rows: v[2j], v[2j+1] = k-step j
};
// Rows are loaded eight lanes to the 128 bytes of a row, and turned to the matrix cores' order through LDS, 32 rows (4 KB) at a
// time in memory of the wave's own. (Loaded in that order, a row a lane and 16 bytes at a time, a line was asked for in
// four instructions while it was still on its way, which the vector cache waits for: it stalled 71% of the cycles at fp32
// rows of 1,048,576 columns and 35% at bf16 rows of 2,049,000, and half of the former's lines were fetched from L2 twice. 512
// such fp32 rows with 128 vectors: 945 us, now 629; 1024 such bf16 rows: 1073, now 1026, where the matrix cores' rate, as far
// as the clock holds under this load, is the bound: 1.07 PFLOP.)
struct RowRaw {
    u32x4 v[4];  // v[x]: piece lane % 8 of row 8 x + lane / 8
};
// Piece p of row r lies at r * 8 + (p ^ (r / 2) % 8): the 16 lanes that are served together fall on all banks, both ways. The
// addresses of a lane's accesses differ by constants (added, or xored in), so that only three are kept.
struct TurnAt {
    unsigned w0, w1, r;  // bytes: stores of even and odd x, loads
};
template <typename T>
__device__ __forceinline__ TurnAt turn_at(int piece0, int lane) {
    const int row = lane >> 3, s = lane & 7, n = lane & 31, h = lane >> 5;
    TurnAt at;
    at.w0 = (unsigned)(piece0 + row * 8 + (s ^ (row >> 1))) * 16;
    at.w1 = (unsigned)(piece0 + row * 8 + (s ^ (4 + (row >> 1)))) * 16;
    at.r = (unsigned)(piece0 + n * 8 + ((sizeof(T) == 2 ? h : 2 * h) ^ ((n >> 1) & 7))) * 16;
    return at;
}
template <int TILES, int LX, typename T>
__device__ __forceinline__ void turn_rows(u32x4* lds, TurnAt at, const RowRaw (&raw)[TILES], RowOp<T> (&a)[TILES]) {
    char* const m = reinterpret_cast<char*>(lds);
    asm volatile("" : "+v"(at.r));  // (the loads' addresses are formed here, not kept)
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
#pragma unroll
        for (int x = 0; x < LX; ++x) *reinterpret_cast<u32x4*>(m + (x & 1 ? at.w1 : at.w0) + x * 1024) = raw[t].v[x];
        asm volatile("" ::: "memory");  // (a wave's LDS accesses keep their order)
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const unsigned p = sizeof(T) == 2 ? 2 * x : 4 * (x >> 1) + (x & 1);
            a[t].v[x] = *reinterpret_cast<const u32x4*>(m + (at.r ^ (p * 16)));
        }
        asm volatile("" ::: "memory");
    }
}
template <int NT, typename T, int NL>  // NT = KP / 32; NL: see loads_of
__global__ __launch_bounds__(512, 1) void project_split_kernel(const T* __restrict__ G, int64_t R,
                                                               const u32x4* __restrict__ img,
                                                               float* __restrict__ partial, int row_tiles, int64_t D,
                                                               int64_t chunks_total, int64_t chunks_per_split) {
    constexpr int KP = NT * 32;
    constexpr int TILES = NL > 4 ? 2 : 1, LX = NL > 4 ? 4 : NL;  // row tiles of a wave, row loads of a tile and window
    constexpr int KC = 128 / (int)sizeof(T);
    constexpr int PPR = KC / 8;        // pieces (8 columns) per window
    constexpr int PB = 8 * (int)sizeof(T);  // bytes of a piece in a row: 16 or 32
    constexpr int IMG = 2 * KP * PPR;  // 16-byte pieces per image
    constexpr int KS = KC / 16;        // matrix-core k-steps per window
    extern __shared__ u32x4 lds[];     // 4 * IMG, then 256 pieces of each wave

    const int id = blockIdx.x;
    const int xcd = id & 7, y = id >> 3;
    const int rt = y % row_tiles;
    const int split = (y / row_tiles) * 8 + xcd;
    const int64_t c0 = (int64_t)split * chunks_per_split;
    int64_t c1 = c0 + chunks_per_split;
    if (c1 > chunks_total) c1 = chunks_total;
    const int64_t nc = c1 - c0;
    const int64_t nv = nc > 0 ? nc + 1 : 0;  // windows c0 .. c1

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, h = lane >> 5;
    const int64_t S = D * (int64_t)sizeof(T);  // row pitch in bytes
    const int64_t row0 = (int64_t)rt * 512;
    // phase of this wave's rows, in pieces
    const int phi = (int)(((reinterpret_cast<uintptr_t>(G) + (uintptr_t)((row0 + wave) * S)) & 127) / PB);

    // A load takes eight rows, eight lanes the 128 bytes of each (load x of row tile t: rows 32 t + 8 x + lane / 8). Lane
    // offsets are taken from gbase = (first row of the work-group) - 128 bytes, so that they are never negative; every offset is
    // clamped to its own row, so no lane reads outside the batch (pieces outside the row meet zeros of the image or are
    // zeroed below). Rows >= R repeat row R-1; their results are not written.
    const char* gbase = reinterpret_cast<const char*>(G) + row0 * S - 128;
    const int64_t last = R - 1 - row0 < 511 ? R - 1 - row0 : 511;
    const unsigned lrow = (unsigned)((wave + 8 * (lane >> 3)) * S), last_row = (unsigned)(last * S);
    const unsigned lofs = 128u + 16u * (unsigned)(lane & 7) - (unsigned)(PB * phi);
    auto load_rows = [&](RowRaw& a, int t, int64_t m) __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < LX; ++x) {
            unsigned r = lrow + (unsigned)((t * 32 + 8 * x) * 8) * (unsigned)S;
            r = r > last_row ? last_row : r;
            const unsigned lo = r + 128u, hi = lo + (unsigned)S - 16u;
            unsigned o = r + lofs + (unsigned)(m * 128);
            o = o < lo ? lo : o;
            o = o > hi ? hi : o;
            a.v[x] = *reinterpret_cast<const u32x4*>(gbase + o);
        }
    };
    const TurnAt turn = turn_at<T>(4 * IMG + wave * 256, lane);
    f32x16 acc[TILES][NT];
#pragma unroll
    for (int t = 0; t < TILES; ++t)
#pragma unroll
        for (int ct = 0; ct < NT; ++ct)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[t][ct][i] = 0.f;

    auto image_of = [&](int64_t c) {  // images outside the matrix repeat the nearest one (finite data, never counted)
        return c < 0 ? (int64_t)0 : (c > chunks_total - 1 ? chunks_total - 1 : c);
    };
    auto stage = [&](int64_t c, int slot) __attribute__((always_inline)) {
        const u32x4* src = img + image_of(c) * IMG + tid;
#pragma unroll
        for (int q = 0; q < IMG / 512; ++q)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + q * 512),
                                             (__attribute__((address_space(3))) void*)(lds + slot * IMG + q * 512 + wave * 64),
                                             16, 0, 0);
        if constexpr (IMG % 512 != 0) {  // IMG = 256 (KP = 32, fp32 rows): half a round; waves 4..7 repeat it, so that
                                         // every wave has the same number of loads in flight (the wait below counts)
            const u32x4* src2 = img + image_of(c) * IMG + (tid & 255);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src2),
                                             (__attribute__((address_space(3))) void*)(lds + slot * IMG + (wave & 3) * 64), 16,
                                             0, 0);
        }
    };
    constexpr int VL = (IMG + 511) / 512;  // image loads per wave and window

    // One window. Step s = (k-step j, column tile ct) in order; the basis operand of step s + 1 is fetched from LDS
    // before the matrix-core instructions of step s are issued, and the scheduler may not move anything across a
    // step (left alone it hoists a whole window of LDS reads and spills). The ring has four slots, image c in slot
    // c mod 4: m-1 and m are read, m+1 has landed or is landing, m+2 is requested now. raw: the rows of this window as they
    // were loaded; it receives those of window m+2.
    auto visit = [&](RowRaw (&raw)[TILES], int64_t m) __attribute__((always_inline)) {
        const int sp = (int)((m - 1) & 3), sc = (int)(m & 3);
        RowOp<T> a[TILES];
        turn_rows<TILES, LX, T>(lds, turn, raw, a);
        stage(m + 2, (int)((m + 2) & 3));
        // The row loads of window m+2 go out in two bursts, row tile 0 a quarter through the window, when the registers of
        // the first operands are free again (the loads of this window's rows and accumulators fill the file otherwise: spills,
        // whose reloads the count below would not know), row tile 1 half way.
        const int64_t m2 = m + 2 > c1 ? c1 : m + 2;  // beyond the last window: repeat it (never used)
        if (m == c0 || m == c1) {
            const bool first = m == c0, last = m == c1;
#pragma unroll
            for (int t = 0; t < TILES; ++t)
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const int q = 2 * (sizeof(T) == 2 ? x : (x >> 1)) + h;
                    if ((first && q < phi) || (last && q >= phi)) a[t].v[x] = u32x4{0u, 0u, 0u, 0u};
                }
        }
        // LDS piece (column tile 0) of this lane's basis operand for k-step j, which may lie in the previous image. Formed when
        // it is needed: registers are short.
        int hq = h;
        asm volatile("" : "+v"(hq));
        auto operand_at = [&](int j) __attribute__((always_inline)) {
            const int q = 2 * j + hq;
            return img_piece<KC>(n, (q - phi) & (PPR - 1)) + (q < phi ? sp : sc) * IMG;
        };
        constexpr int STEPS = KS * 2 * NT;
        u32x4 b[2];
        int at = operand_at(0);
        b[0] = lds[at];
        u32x4 ahi[TILES], alo[TILES];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            const int j = s / (2 * NT), ct = s % (2 * NT);
            if (ct == 0) {
                if constexpr (sizeof(T) == 2) {
#pragma unroll
                    for (int t = 0; t < TILES; ++t) ahi[t] = a[t].v[j];
                } else {
#pragma unroll
                    for (int t = 0; t < TILES; ++t) split8(a[t].v[2 * j], a[t].v[2 * j + 1], ahi[t], alo[t]);
                }
            }
            if (s + 1 < STEPS) {
                const int j2 = (s + 1) / (2 * NT), ct2 = (s + 1) % (2 * NT);
                if (ct2 == 0) at = operand_at(j2);
                b[(s + 1) % 2] = lds[at + ct2 * 32 * PPR];
            }
            if (s == STEPS / 4) load_rows(raw[0], 0, m2);
            if (s == STEPS / 2 && TILES == 2) load_rows(raw[TILES - 1], 1, m2);
            const u32x4 bb = b[s % 2];
#pragma unroll
            for (int t = 0; t < TILES; ++t) acc[t][ct % NT] = mfma_bf16(ahi[t], bb, acc[t][ct % NT]);
            if constexpr (sizeof(T) == 4) {
                if (ct < NT) {
#pragma unroll
                    for (int t = 0; t < TILES; ++t) acc[t][ct] = mfma_bf16(alo[t], bb, acc[t][ct]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // This window requested VL image loads (image m+2) and NL row loads (window m+2): once at most NL + VL loads are
        // outstanding, image m+1 and the rows of window m+1 (and every older load) have landed; both were requested a
        // whole window earlier. A bare barrier: __syncthreads() carries a release fence, which on this target drains
        // every outstanding load and would throw the prefetch distance away. The LDS reads of this window have all
        // been consumed by matrix-core instructions above.
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0F70 | (NL + VL));  // vmcnt(NL + VL); expcnt, lgkmcnt not waited for
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    // The windows of a split are walked from a start that differs from split to split and wrap around: work-groups
    // that all start at the first window of their split march over memory in lock step, a regular pattern that left
    // some memory channels idle (5.1 TB/s for the row stream alone against 6.2 TB/s with rotated starts). The two row
    // tiles of a split keep the same start, so that they still share the basis images through L2. A run of
    // consecutive windows needs the ring primed with the images around its first window, so the walk is two runs.
    RowRaw a0[TILES], a1[TILES];
    if (nv > 0) {
        const int64_t rot = nv >= 8 ? (int64_t)(((unsigned)split * 37u) % (unsigned)(nv - 4)) + 2 : 0;  // 2 .. nv - 3
        int64_t ms = c0 + rot, me = c0 + nv;
#pragma unroll 1
        for (;;) {  // (one copy of the loop for both runs)
            stage(ms - 1, (int)((ms - 1) & 3));
            stage(ms, (int)(ms & 3));
            stage(ms + 1, (int)((ms + 1) & 3));
#pragma unroll
            for (int t = 0; t < TILES; ++t) {
                load_rows(a0[t], t, ms);
                load_rows(a1[t], t, ms + 1 > c1 ? c1 : ms + 1);
            }
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
#pragma unroll 1
            for (int64_t m = ms; m < me; m += 2) {  // two windows per trip: the row buffers return to their roles
                visit(a0, m);
                if (m + 1 < me) visit(a1, m + 1);
            }
            if (ms == c0) break;
            ms = c0;
            me = c0 + rot;
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): nothing on its way to LDS when the work-group ends
    }

    float* out = partial + (int64_t)split * R * KP;
#pragma unroll
    for (int t = 0; t < TILES; ++t)
#pragma unroll
        for (int ct = 0; ct < NT; ++ct)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int64_t r = row0 + wave + 8 * (t * 32 + 8 * (i >> 2) + 4 * h + (i & 3));
                if (r < R) out[r * KP + ct * 32 + n] = acc[t][ct][i];
            }
}

// ---- projection of rows of any width and alignment ---------------------------------------------------------------
// Where rows do not start on a multiple of 8 columns' bytes, windows are counted from the row's first column, wherever that
// lies in a memory line, and a piece is loaded at any element boundary. Such rows went through the fp32 matrix cores
// before (157 us for 2048 rows of 51,300 with 64 vectors), so here the basis has three bf16 parts (24 bits) and fp32 rows
// are split the same way: six products (three for bf16 rows, which are exact), the fp32 result to a few 2^-24 per term.
//
// Shapes as in project_split_kernel: 512 threads, a wave owns 64 rows x KP columns, rows are loaded eight lanes to 128 bytes, two
// windows ahead, and turned through LDS. Every window is a whole image, so the ring has three slots (two where three do not
// fit, four column tiles of bf16 rows: a window is long there, an image requested at its start lands within it). The last,
// partial window of the row is taken after the others, by the split that owns it.
//
// With rows loaded in the matrix cores' order (the vector cache stalled four fifths of the time), and turned: 2048 rows of
// 51,300 fp32, 64 vectors 121 and 113 us; 512 rows of 1,000,001 fp32, 128 vectors 965 and 825; 1024 such rows of bf16 1100 and
// 715. The rows' loads remain the bound of the first: each takes two lines (103 us where rows start on a line), and with one
// product instead of six it takes 104.
template <typename T>
struct __attribute__((packed, aligned(sizeof(T)))) AnyPiece {
    u32x4 v;
};

template <int NT, typename T>
struct AnyShape {
    static constexpr int IMG = 3 * NT * 32 * (16 / (int)sizeof(T));  // 16-byte pieces of an image
    static constexpr int SLOTS = sizeof(T) == 2 && NT == 4 ? 2 : 3;
    static constexpr int LDS = (SLOTS * IMG + 8 * 256) * 16;
    static_assert(LDS <= 160 * 1024, "of one CU");
};

template <int NT, typename T, int NL>
__global__ __launch_bounds__(512, 1) void project_any_kernel(const T* __restrict__ G, int64_t R,
                                                             const u32x4* __restrict__ img, float* __restrict__ partial,
                                                             int row_tiles, int64_t D, int64_t chunks_total,
                                                             int64_t chunks_per_split) {
    constexpr int KP = NT * 32;
    constexpr int TILES = NL > 4 ? 2 : 1, LX = NL > 4 ? 4 : NL;
    constexpr int KC = 128 / (int)sizeof(T);
    constexpr int PPR = KC / 8;
    constexpr int IMG = AnyShape<NT, T>::IMG, SLOTS = AnyShape<NT, T>::SLOTS;
    constexpr int KS = KC / 16;
    extern __shared__ u32x4 lds[];  // SLOTS * IMG, then 256 pieces of each wave

    const int id = blockIdx.x;
    const int xcd = id & 7, y = id >> 3;
    const int rt = y % row_tiles;
    const int split = (y / row_tiles) * 8 + xcd;
    const int64_t full = D / KC;  // whole windows of a row
    const int64_t c0 = (int64_t)split * chunks_per_split;
    int64_t c1 = c0 + chunks_per_split;
    if (c1 > chunks_total) c1 = chunks_total;
    const bool tail = c0 < c1 && c1 > full;
    if (c1 > full) c1 = full;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, h = lane >> 5;
    const int64_t S = D * (int64_t)sizeof(T);
    const int64_t row0 = (int64_t)rt * 512;
    const char* gbase = reinterpret_cast<const char*>(G) + row0 * S;
    // rows >= R repeat row R - 1; their results are not written
    const int64_t last = R - 1 - row0 < 511 ? R - 1 - row0 : 511;
    const unsigned lrow = (unsigned)((wave + 8 * (lane >> 3)) * S), last_row = (unsigned)(last * S);
    auto load_rows = [&](RowRaw& a, int t, int64_t m) __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < LX; ++x) {
            unsigned r = lrow + (unsigned)((t * 32 + 8 * x) * 8) * (unsigned)S;
            r = r > last_row ? last_row : r;
            a.v[x] = reinterpret_cast<const AnyPiece<T>*>(gbase + (r + 16u * (unsigned)(lane & 7) + (unsigned)(m * 128)))->v;
        }
    };
    const TurnAt turn = turn_at<T>(SLOTS * IMG + wave * 256, lane);
    f32x16 acc[TILES][NT];
#pragma unroll
    for (int t = 0; t < TILES; ++t)
#pragma unroll
        for (int ct = 0; ct < NT; ++ct)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[t][ct][i] = 0.f;

    constexpr int VL = (IMG + 511) / 512;
    auto stage = [&](int64_t c, int slot) __attribute__((always_inline)) {
        if (c > chunks_total - 1) c = chunks_total - 1;  // beyond the end: repeat (never used)
        const u32x4* src = img + c * IMG;
#pragma unroll
        for (int q = 0; q < VL; ++q) {
            // (where IMG is no multiple of 512 the waves left over repeat its start: every wave has VL loads in flight)
            const int at = (q * 512 + wave * 64) % IMG;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + at + lane),
                                             (__attribute__((address_space(3))) void*)(lds + slot * IMG + at), 16, 0, 0);
        }
    };

    static_assert(NL + VL <= 15, "the low field of the count");
    int sc = 0;  // slot of the present window's image
    // the products of one window: row operands a
    auto multiply = [&](const RowOp<T> (&a)[TILES], auto&& between) __attribute__((always_inline)) {
        constexpr int STEPS = KS * 3 * NT;  // (k-step, part of the basis, column tile)
        int hq = h;
        asm volatile("" : "+v"(hq));  // (addresses are formed when they are needed: registers are short)
        auto addr = [&](int s) {
            const int j = s / (3 * NT), pt = (s / NT) % 3, ct = s % NT;
            return img_piece<KC>(n, 2 * j + hq) + sc * IMG + (pt * KP + ct * 32) * PPR;
        };
        u32x4 b[2];
        b[0] = lds[addr(0)];
        u32x4 ap[TILES][3];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            const int j = s / (3 * NT), pt = (s / NT) % 3, ct = s % NT;
            if (s % (3 * NT) == 0) {
#pragma unroll
                for (int t = 0; t < TILES; ++t) {
                    if constexpr (sizeof(T) == 2) {
                        ap[t][0] = a[t].v[j];
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const u32x4& x = a[t].v[2 * j + (e >> 1)];
                            unsigned p0, p1, p2;
                            split3_bf16(__uint_as_float(x[(2 * e) & 3]), __uint_as_float(x[(2 * e + 1) & 3]), p0, p1, p2);
                            ap[t][0][e] = p0;
                            ap[t][1][e] = p1;
                            ap[t][2][e] = p2;
                        }
                    }
                }
            }
            if (s + 1 < STEPS) b[(s + 1) % 2] = lds[addr(s + 1)];
            if (s == STEPS / 4) between(0);
            if (s == STEPS / 2 && TILES == 2) between(1);
            const u32x4 bb = b[s % 2];
            constexpr int QS = sizeof(T) == 2 ? 1 : 3;
#pragma unroll
            for (int q = 0; q < QS; ++q)
                if (q + pt <= 2) {
#pragma unroll
                    for (int t = 0; t < TILES; ++t) acc[t][ct] = mfma_bf16(ap[t][q], bb, acc[t][ct]);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // One window: its image is in slot sc, its rows in raw as they were loaded, which receives the rows of window m + 2. The image
    // requested is that of m + SLOTS - 1. more: false where the split has two windows at most, as those of small projections
    // have, and nothing beyond them is requested (333 rows of 25,447 bf16: 22.2 us with such requests, 19.5
    // without; 20.5 before rows were turned).
    auto visit = [&](RowRaw (&raw)[TILES], int64_t m, auto more) __attribute__((always_inline)) {
        constexpr bool MORE = decltype(more)::value;
        const int64_t m2 = m + 2 > c1 - 1 ? c1 - 1 : m + 2;  // beyond the last window: repeat it (never used)
        RowOp<T> a[TILES];
        turn_rows<TILES, LX, T>(lds, turn, raw, a);
        if (MORE || SLOTS == 2) stage(m + SLOTS - 1, sc == 0 ? SLOTS - 1 : sc - 1);
        multiply(a, [&](int t) __attribute__((always_inline)) {
            if constexpr (MORE) load_rows(raw[t], t, m2);
        });
        // at most this window's row loads, with three slots its image loads too, stay outstanding: image m + 1 and rows m + 1
        // have landed
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0F70 | (MORE ? NL + (SLOTS == 3 ? VL : 0) : 0));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        sc = sc == SLOTS - 1 ? 0 : sc + 1;
    };
    constexpr std::true_type MORE{};
    constexpr std::false_type LAST{};

    const int64_t len = c1 - c0;
    auto begin = [&](RowRaw (&a0)[TILES], RowRaw (&a1)[TILES]) __attribute__((always_inline)) {
        stage(c0, 0);
        if (SLOTS == 3) stage(c0 + 1, 1);
        const int64_t m1 = len > 1 ? c0 + 1 : c0;
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
            load_rows(a0[t], t, c0);
            load_rows(a1[t], t, m1);
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
    };
    if (len > 2) {
        RowRaw a0[TILES], a1[TILES];
        begin(a0, a1);
#pragma unroll 1
        for (int64_t m = c0; m < c1; m += 2) {  // two windows per trip: the row buffers return to their roles
            visit(a0, m, MORE);
            if (m + 1 < c1) visit(a1, m + 1, MORE);
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): nothing on its way to LDS any more
    }
    if (len == 1 || len == 2) {
        RowRaw a0[TILES], a1[TILES];
        begin(a0, a1);
        visit(a0, c0, LAST);
        if (len == 2) visit(a1, c0 + 1, LAST);
    }
    if (tail) {  // work-group uniform
        __syncthreads();
        stage(full, 0);
        // The last 128 bytes of every row are loaded, and the columns beyond the whole windows picked out of them in LDS.
        const int left = (int)(D - full * KC);
        RowRaw raw[TILES];
#pragma unroll
        for (int t = 0; t < TILES; ++t)
#pragma unroll
            for (int x = 0; x < LX; ++x) {
                unsigned r = lrow + (unsigned)((t * 32 + 8 * x) * 8) * (unsigned)S;
                r = r > last_row ? last_row : r;
                raw[t].v[x] = reinterpret_cast<const AnyPiece<T>*>(gbase + (r + (unsigned)S - 128u + 16u * (unsigned)(lane & 7)))->v;
            }
        RowOp<T> a[TILES];
        char* const l = reinterpret_cast<char*>(lds);
        const unsigned line = (unsigned)(SLOTS * IMG + wave * 256 + n * 8) * 16u, swz = (unsigned)((n >> 1) & 7) * 16u;
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
#pragma unroll
            for (int x = 0; x < LX; ++x) *reinterpret_cast<u32x4*>(l + (x & 1 ? turn.w1 : turn.w0) + x * 1024) = raw[t].v[x];
            asm volatile("" ::: "memory");  // (a wave's LDS accesses keep their order)
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                constexpr int E = 16 / (int)sizeof(T);
                const int at = (sizeof(T) == 2 ? 16 * x : 16 * (x >> 1) + 4 * (x & 1)) + 8 * h;
                T v[E];
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int c = at + e < left ? KC - left + at + e : 0;  // column of the 128 bytes
                    const T w = *reinterpret_cast<const T*>(l + line + (((unsigned)c * (unsigned)sizeof(T)) ^ swz));
                    v[e] = at + e < left ? w : (T)0;
                }
                __builtin_memcpy(&a[t].v[x], v, 16);
            }
            asm volatile("" ::: "memory");
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        sc = 0;
        multiply(a, [](int) {});
    }

    float* out = partial + (int64_t)split * R * KP;
#pragma unroll
    for (int t = 0; t < TILES; ++t)
#pragma unroll
        for (int ct = 0; ct < NT; ++ct)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int64_t r = row0 + wave + 8 * (t * 32 + 8 * (i >> 2) + 4 * h + (i & 3));
                if (r < R) out[r * KP + ct * 32 + n] = acc[t][ct][i];
            }
}

// Any row start that is a multiple of the element, a row of at least one window, lane offsets of 32 bits.
bool any_path_ok(const void* G, int dtype, const Dims& d) {
    const int64_t esz = dtype == SAGE_BF16 ? 2 : 4;
    return d.D >= 128 / esz && d.D * esz * 513 + 256 < ((int64_t)1 << 32) && ((uintptr_t)G) % esz == 0;
}

// Every row must start on a multiple of the bytes of 8 columns (16 for bf16, 32 for fp32 rows), hold at least one
// chunk, and 512 rows plus a line must span < 4 GiB (lane offsets are 32-bit).
bool split_path_ok(const void* G, int dtype, const Dims& d) {
    const int64_t esz = dtype == SAGE_BF16 ? 2 : 4;
    const int64_t KC = 128 / esz;
    return d.D % 8 == 0 && d.D >= KC && d.D * esz * 513 + 256 < ((int64_t)1 << 32) && ((uintptr_t)G) % (8 * esz) == 0;
}

ScorePlan score_split_plan(int64_t R, int dtype, const Dims& d, int num_cu) {
    ScorePlan p;
    const int KC = dtype == SAGE_BF16 ? 64 : 32;
    const int64_t chunks = (d.D + KC - 1) / KC;
    p.row_tiles = (int)((R + 511) / 512);
    int64_t want = ((int64_t)num_cu + p.row_tiles - 1) / p.row_tiles;  // one work-group per CU
    int64_t s = (want + 7) / 8 * 8;
    // At least ~2 chunks per split: a small projection is a chain of loads, 1 us per chunk and more (1024 rows of 5136 fp32:
    // 25.7 us at 8 chunks, 16.2 at 2, with the finish of the more numerous partial sums as fast)
    int64_t smax = ((chunks + 1) / 2 + 7) / 8 * 8;
    if (s > smax) s = smax;
    if (s < 8) s = 8;
    if (s > 512) s = 512;
    p.splits = (int)s;
    p.slabs_per_split = (chunks + s - 1) / s;  // chunks per split on this path
    return p;
}

// Row loads of a wave and window (eight rows each; the waves take the rows of a work-group in turn): as few as hold the batch.
// (Eight whatever the batch: of 64 rows most loads ask for the last row again, a line that is on its way. 64 fp32 rows of 977,864
// with 8 vectors: 183 us with eight, 101 with one; 128 bf16 rows of 200,001 with 100 vectors 67 and 41.)
int loads_of(int64_t R) { return R > 256 ? 8 : R > 128 ? 4 : R > 64 ? 2 : 1; }

template <int NT, typename T, int NL>
static hipError_t launch_split_nl(const T* G, int64_t R, int parts, const void* img, float* partial, const ScorePlan& p,
                                  const Dims& d, hipStream_t st) {
    constexpr int KC = 128 / (int)sizeof(T);
    const int lds = parts == 3 ? AnyShape<NT, T>::LDS : 4 * 2 * NT * 32 * (KC / 8) * 16 + 8 * 256 * 16;
    void (*const kern)(const T*, int64_t, const u32x4*, float*, int, int64_t, int64_t, int64_t) =
        parts == 3 ? project_any_kernel<NT, T, NL> : project_split_kernel<NT, T, NL>;
    if (hipError_t ea = ensure_dynamic_lds((const void*)kern, lds); ea != hipSuccess) return ea;
    hipLaunchKernelGGL(kern, dim3((unsigned)(p.row_tiles * p.splits)), dim3(512), lds, st, G, R, (const u32x4*)img, partial,
                       p.row_tiles, d.D, (d.D + KC - 1) / KC, p.slabs_per_split);
    return hipGetLastError();
}
template <int NT, typename T>
static hipError_t launch_split_t(const T* G, int64_t R, int parts, const void* img, float* partial, const ScorePlan& p,
                                 const Dims& d, hipStream_t st) {
    switch (loads_of(R)) {
        case 1: return launch_split_nl<NT, T, 1>(G, R, parts, img, partial, p, d, st);
        case 2: return launch_split_nl<NT, T, 2>(G, R, parts, img, partial, p, d, st);
        case 4: return launch_split_nl<NT, T, 4>(G, R, parts, img, partial, p, d, st);
        default: return launch_split_nl<NT, T, 8>(G, R, parts, img, partial, p, d, st);
    }
}

template <int NT>
static hipError_t launch_split_nt(const void* G, int dtype, int64_t R, int parts, const void* img, float* partial,
                                  const ScorePlan& p, const Dims& d, hipStream_t st) {
    if (dtype == SAGE_BF16) return launch_split_t<NT, uint16_t>((const uint16_t*)G, R, parts, img, partial, p, d, st);
    return launch_split_t<NT, float>((const float*)G, R, parts, img, partial, p, d, st);
}

hipError_t launch_project_split(const void* G, int dtype, int64_t R, int parts, const void* img, int KP, float* partial,
                                const ScorePlan& p, const Dims& d, hipStream_t st) {
    switch (KP / 32) {
        case 1: return launch_split_nt<1>(G, dtype, R, parts, img, partial, p, d, st);
        case 2: return launch_split_nt<2>(G, dtype, R, parts, img, partial, p, d, st);
        case 4: return launch_split_nt<4>(G, dtype, R, parts, img, partial, p, d, st);
        default: return hipErrorInvalidValue;
    }
}


// ---- projection of factored rows ----------------------------------------------------------------------------
// A per-example gradient of a linear last layer (weights C x dh, bias C) under a loss on the logits is the outer
// product of the logit error e_i (C values) with [h_i; 1] (dh features and a one): column c*dh + t of row i is
// e_ic * h_it, column C*dh + c is e_ic (Method, definition of g_i, for that layer). The row is never stored: the
// kernel below forms the row operand of a window (KC columns of class c starting at feature tw*KC) from 128 bytes of
// h_i and the value e_ic, rounds it as a stored row of the context's type would have been rounded (bf16: nearest
// even; fp32: the fp32 product, then split as above) and multiplies it with the same basis images. The C bias
// columns are added by project_bias_kernel into a partial slot of their own.
//
// A split is a block of classes x feature windows and is walked feature window by feature window, classes inside:
// the 128 bytes of h_i stay in registers for all classes of the split, and per window only the image and one value of
// e per row are fetched (e comes from a transposed copy, so that the 32 rows of a tile read 32 neighbouring values).
// From HBM the kernel reads little more than the images, once. (Walking the columns in their order instead re-reads
// the feature rows for every class; they do not stay in L2 beside the image stream, and that variant ran at the
// speed of the row-major kernel.)
//
// Work-group and wave shapes as in project_split_kernel (512 threads, 512 rows; a wave owns rows 64w .. 64w+63).
// Every window is a whole image, so the ring has three slots: the window's image in use, the next landed or landing,
// the one after requested.
struct OuterGeom {
    int C, dh;
    int class_groups, classes_per_group;  // split -> (class group, window group): split % class_groups, split / ...
    int window_groups, windows_per_group;
    int64_t et_pitch;                     // elements between classes in the transposed error matrix
};

template <int NT, typename T>
__global__ __launch_bounds__(512, 1) void project_outer_kernel(const T* __restrict__ Et, const T* __restrict__ H,
                                                               int64_t R, OuterGeom g, const u32x4* __restrict__ img,
                                                               float* __restrict__ partial, int row_tiles) {
    constexpr int KP = NT * 32;
    constexpr int KC = 128 / (int)sizeof(T);
    constexpr int PPR = KC / 8;
    constexpr int PB = 8 * (int)sizeof(T);
    constexpr int IMG = 2 * KP * PPR;
    constexpr int KS = KC / 16;
    extern __shared__ u32x4 lds[];  // 3 * IMG

    const int id = blockIdx.x;
    const int xcd = id & 7, y = id >> 3;
    const int rt = y % row_tiles;
    const int split = (y / row_tiles) * 8 + xcd;
    const int cpc = g.dh / KC;  // windows per class
    const int kg = split % g.class_groups, tg = split / g.class_groups;
    const int k0 = kg * g.classes_per_group;
    int k1 = k0 + g.classes_per_group;
    if (k1 > g.C) k1 = g.C;
    int t0 = tg * g.windows_per_group, t1 = t0 + g.windows_per_group;
    if (t1 > cpc) t1 = cpc;
    if (tg >= g.window_groups) t1 = t0;  // padding splits: nothing to do, their slot is zero
    const int nk = k1 > k0 ? k1 - k0 : 0;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, h = lane >> 5;
    const int64_t row0 = (int64_t)rt * 512;
    // Rows >= R repeat row R-1 for the features; the transposed errors are padded to whole row tiles. Results of such
    // rows are not written.
    const char* hrow[2];
    const T* ecol[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int64_t rr = row0 + wave * 64 + t * 32 + n;
        const int64_t r = rr > R - 1 ? R - 1 : rr;
        hrow[t] = reinterpret_cast<const char*>(H + r * g.dh) + PB * h;
        ecol[t] = Et + rr;
    }
    int boff[KS];
#pragma unroll
    for (int j = 0; j < KS; ++j) boff[j] = img_piece<KC>(n, (2 * j + h) & (PPR - 1));

    f32x16 acc[2][NT];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int ct = 0; ct < NT; ++ct)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[t][ct][i] = 0.f;

    const int64_t n_img = (int64_t)g.C * cpc;
    auto stage = [&](int cls, int tw, int slot) __attribute__((always_inline)) {
        int64_t ci = (int64_t)cls * cpc + tw;
        if (ci > n_img - 1) ci = n_img - 1;  // beyond the end: repeat (never used)
        const u32x4* src = img + ci * IMG + tid;
#pragma unroll
        for (int q = 0; q < IMG / 512; ++q)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + q * 512),
                                             (__attribute__((address_space(3))) void*)(lds + slot * IMG + q * 512 + wave * 64),
                                             16, 0, 0);
        if constexpr (IMG % 512 != 0) {  // IMG = 256: waves 4..7 repeat the half round (equal load counts per wave)
            const u32x4* src2 = img + ci * IMG + (tid & 255);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src2),
                                             (__attribute__((address_space(3))) void*)(lds + slot * IMG + (wave & 3) * 64), 16,
                                             0, 0);
        }
    };
    constexpr int VL = (IMG + 511) / 512;

    u32x4 hv[2][4];  // this lane's pieces of the feature rows, current feature window
    // the row operand of k-step j: e * h, rounded to the row type
    auto operand = [&](int t, T eraw, int j, u32x4& hi, u32x4& lo) __attribute__((always_inline)) {
        if constexpr (sizeof(T) == 2) {
            const float e = bf16_to_f32(eraw);
            const u32x4 raw = hv[t][j];
#pragma unroll
            for (int w = 0; w < 4; ++w)
                hi[w] = pack_bf16(__uint_as_float(raw[w] << 16) * e, __uint_as_float(raw[w] & 0xffff0000u) * e);
        } else {
            u32x4 x0, x1;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                x0[w] = __float_as_uint(__uint_as_float(hv[t][2 * j][w]) * eraw);
                x1[w] = __float_as_uint(__uint_as_float(hv[t][2 * j + 1][w]) * eraw);
            }
            split8(x0, x1, hi, lo);
        }
    };
    auto load_e = [&](T (&e)[2], int cls) __attribute__((always_inline)) {
        const int cc = cls > g.C - 1 ? g.C - 1 : cls;
#pragma unroll
        for (int t = 0; t < 2; ++t) e[t] = ecol[t][(int64_t)cc * g.et_pitch];
    };

    // One window: class cls of feature window tw, its image in slot sc; the image and the errors of class cls + 2 are
    // requested.
    auto visit = [&](const T (&e)[2], T (&efar)[2], int cls, int tw, int sc) __attribute__((always_inline)) {
        stage(cls + 2, tw, sc == 0 ? 2 : sc - 1);
        load_e(efar, cls + 2);
        int baddr[KS];
#pragma unroll
        for (int j = 0; j < KS; ++j) baddr[j] = boff[j] + sc * IMG;
        constexpr int STEPS = KS * 2 * NT;
        u32x4 b[2];
        b[0] = lds[baddr[0]];
        u32x4 ahi[2], alo[2];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            const int j = s / (2 * NT), ct = s % (2 * NT);
            if (ct == 0) {
                operand(0, e[0], j, ahi[0], alo[0]);
                operand(1, e[1], j, ahi[1], alo[1]);
            }
            if (s + 1 < STEPS) {
                const int j2 = (s + 1) / (2 * NT), ct2 = (s + 1) % (2 * NT);
                b[(s + 1) % 2] = lds[baddr[j2] + ct2 * 32 * PPR];
            }
            const u32x4 bb = b[s % 2];
#pragma unroll
            for (int t = 0; t < 2; ++t) acc[t][ct % NT] = mfma_bf16(ahi[t], bb, acc[t][ct % NT]);
            if constexpr (sizeof(T) == 4) {
                if (ct < NT) {
#pragma unroll
                    for (int t = 0; t < 2; ++t) acc[t][ct] = mfma_bf16(alo[t], bb, acc[t][ct]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // This window issued VL image loads and 2 error loads, all for class cls + 2: with at most that many
        // outstanding, the image and the errors of class cls + 1 have landed. Bare barrier as above.
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0F70 | (2 + VL));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    T e0[2], e1[2], e2[2];
    if (nk > 0) {
        for (int tw = t0; tw < t1; ++tw) {
            stage(k0, tw, 0);
            stage(k0 + 1, tw, 1);
            load_e(e0, k0);
            load_e(e1, k0 + 1);
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const int xoff = sizeof(T) == 2 ? 32 * x : 64 * (x >> 1) + 16 * (x & 1);
                    hv[t][x] = *reinterpret_cast<const u32x4*>(hrow[t] + tw * 128 + xoff);
                }
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            int i = 0;
            for (; i + 2 < nk; i += 3) {
                visit(e0, e2, k0 + i, tw, 0);
                visit(e1, e0, k0 + i + 1, tw, 1);
                visit(e2, e1, k0 + i + 2, tw, 2);
            }
            if (i < nk) visit(e0, e2, k0 + i, tw, 0);
            if (i + 1 < nk) visit(e1, e0, k0 + i + 1, tw, 1);
            // every wave has passed the last window's barrier: the ring may be primed again
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): nothing on its way to LDS when the work-group ends
    }

    float* out = partial + (int64_t)split * R * KP;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int ct = 0; ct < NT; ++ct)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int64_t r = row0 + wave * 64 + t * 32 + 8 * (i >> 2) + 4 * h + (i & 3);
                if (r < R) out[r * KP + ct * 32 + n] = acc[t][ct][i];
            }
}

// Et[c][r] = E[min(r, R-1)][c] for r < Rp (Rp: R rounded up to whole row tiles). 64 x 64 tiles through LDS.
template <typename T>
__global__ __launch_bounds__(256) void transpose_errors_kernel(const T* __restrict__ E, int64_t R, int C, int64_t Rp,
                                                               T* __restrict__ Et) {
    __shared__ T tile[64][65];
    const int64_t r0 = (int64_t)blockIdx.x * 64;
    const int c0 = blockIdx.y * 64;
    const int a = threadIdx.x & 63, b = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int rr = b + 4 * i;
        int64_t r = r0 + rr;
        if (r > R - 1) r = R - 1;
        tile[rr][a] = c0 + a < C ? E[r * C + c0 + a] : (T)0;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int cc = b + 4 * i;
        if (c0 + cc < C && r0 + a < Rp) Et[(int64_t)(c0 + cc) * Rp + r0 + a] = tile[a][cc];
    }
}

// The bias columns: out[r][j] = sum_c e_rc * V[j][C*dh + c] in fp32 (e is a stored value of the row type, so no
// rounding is involved). 256 threads, 8 rows x KP outputs per work-group, 16 columns of the basis at a time in LDS;
// blockIdx.y takes the classes [y * cps, (y + 1) * cps) and writes partial slot y (cps a multiple of 16).
template <typename T>
__global__ __launch_bounds__(256) void project_bias_kernel(const T* __restrict__ E, int64_t R, int C, int cps,
                                                           int64_t col0, const float* __restrict__ Vblk, int KP,
                                                           float* __restrict__ out) {
    __shared__ float Vs[128][17];
    __shared__ float Es[8][16];
    const int tid = threadIdx.x;
    const int64_t r0 = (int64_t)blockIdx.x * 8;
    const int per = KP / 32;  // outputs per thread: (8 * KP) / 256
    const int cb0 = blockIdx.y * cps;
    int cb1 = cb0 + cps;
    if (cb1 > C) cb1 = C;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int cb = cb0; cb < cb1; cb += 16) {
        for (int i = tid; i < KP * 16; i += 256) {
            const int j = i >> 4, cc = i & 15;
            Vs[j][cc] = cb + cc < cb1 ? Vblk[blk_off(col0 + cb + cc, j, KP)] : 0.f;
        }
        if (tid < 128) {
            const int rr = tid >> 4, cc = tid & 15;
            const int64_t r = r0 + rr;
            float e = 0.f;
            if (r < R && cb + cc < cb1) {
                if constexpr (sizeof(T) == 2) e = bf16_to_f32(E[r * C + cb + cc]);
                else e = E[r * C + cb + cc];
            }
            Es[rr][cc] = e;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (q < per) {
                const int o = tid + 256 * q, rr = o / KP, j = o % KP;
#pragma unroll
                for (int cc = 0; cc < 16; ++cc) acc[q] = fmaf(Es[rr][cc], Vs[j][cc], acc[q]);
            }
        }
        __syncthreads();
    }
    float* dst = out + (int64_t)blockIdx.y * R * KP;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (q < per) {
            const int o = tid + 256 * q, rr = o / KP, j = o % KP;
            if (r0 + rr < R) dst[(r0 + rr) * KP + j] = acc[q];
        }
    }
}

// Work space of launch_project_outer: the transposed errors, C x (row tiles * 512) values.
size_t outer_work_bytes(int64_t R, int dtype, int64_t C) {
    return (size_t)C * (size_t)((R + 511) / 512 * 512) * (dtype == SAGE_BF16 ? 2 : 4);
}

// The factored projection needs whole windows inside a class and 16-byte aligned feature rows.
bool outer_path_ok(const void* E, const void* H, int dtype, int64_t C, int64_t dh) {
    const int64_t esz = dtype == SAGE_BF16 ? 2 : 4;
    const int64_t KC = 128 / esz;
    return dh >= KC && dh % KC == 0 && C < ((int64_t)1 << 24) && dh < ((int64_t)1 << 24) && ((uintptr_t)H) % 16 == 0 &&
           ((uintptr_t)E) % esz == 0;
}

// splits counts the slots of the main columns (a grid of class groups x window groups, padded to a multiple of 8);
// the bias columns go to the bias_slots slots after them, classes_per_bias_slot classes each. Window groups are kept as small as the split count
// allows, classes per split as many: the feature rows are read once per window of a split.
ScorePlan score_outer_plan(int64_t R, int dtype, int64_t C, int64_t dh, int num_cu) {
    ScorePlan p;
    const int KC = dtype == SAGE_BF16 ? 64 : 32;
    const int64_t cpc = dh / KC;
    p.row_tiles = (int)((R + 511) / 512);
    int64_t target = (((int64_t)num_cu + p.row_tiles - 1) / p.row_tiles + 7) / 8 * 8;
    if (target < 8) target = 8;
    if (target > 512) target = 512;
    int64_t wg = cpc < target ? cpc : target;
    int64_t cg = target / wg;
    if (cg < 1) cg = 1;
    if (cg > C) cg = C;
    p.windows_per_group = (int)((cpc + wg - 1) / wg);
    p.window_groups = (int)((cpc + p.windows_per_group - 1) / p.windows_per_group);
    p.classes_per_group = (int)((C + cg - 1) / cg);
    p.class_groups = (int)((C + p.classes_per_group - 1) / p.classes_per_group);
    p.splits = (p.class_groups * p.window_groups + 7) / 8 * 8;
    p.slabs_per_split = (int64_t)p.classes_per_group * p.windows_per_group;
    p.classes_per_bias_slot = (int)(((C + 7) / 8 + 15) / 16 * 16);  // up to 8 slots
    p.bias_slots = (int)((C + p.classes_per_bias_slot - 1) / p.classes_per_bias_slot);
    return p;
}

template <int NT, typename T>
static hipError_t launch_outer_t(const T* E, const T* H, int64_t R, int64_t C, int64_t dh, void* work, const void* img,
                                 const float* Vblk, float* partial, const ScorePlan& p, hipStream_t st) {
    constexpr int KC = 128 / (int)sizeof(T);
    constexpr size_t LDS = (size_t)3 * 2 * NT * 32 * (KC / 8) * 16;
    if (hipError_t ea = ensure_dynamic_lds((const void*)project_outer_kernel<NT, T>, (int)LDS); ea != hipSuccess) return ea;
    const int64_t Rp = (int64_t)p.row_tiles * 512;
    hipLaunchKernelGGL(transpose_errors_kernel<T>, dim3((unsigned)(Rp / 64), (unsigned)((C + 63) / 64)), dim3(256), 0, st, E,
                       R, (int)C, Rp, (T*)work);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    OuterGeom g;
    g.C = (int)C;
    g.dh = (int)dh;
    g.class_groups = p.class_groups;
    g.classes_per_group = p.classes_per_group;
    g.window_groups = p.window_groups;
    g.windows_per_group = p.windows_per_group;
    g.et_pitch = Rp;
    dim3 grid((unsigned)(p.row_tiles * p.splits));
    hipLaunchKernelGGL((project_outer_kernel<NT, T>), grid, dim3(512), LDS, st, (const T*)work, H, R, g, (const u32x4*)img,
                       partial, p.row_tiles);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(project_bias_kernel<T>, dim3((unsigned)((R + 7) / 8), (unsigned)p.bias_slots), dim3(256), 0, st, E, R,
                       (int)C, p.classes_per_bias_slot, C * dh, Vblk, NT * 32, partial + (size_t)p.splits * R * (NT * 32));
    return hipGetLastError();
}

template <int NT>
static hipError_t launch_outer_nt(const void* E, const void* H, int dtype, int64_t R, int64_t C, int64_t dh, void* work,
                                  const void* img, const float* Vblk, float* partial, const ScorePlan& p, hipStream_t st) {
    if (dtype == SAGE_BF16)
        return launch_outer_t<NT, uint16_t>((const uint16_t*)E, (const uint16_t*)H, R, C, dh, work, img, Vblk, partial, p,
                                            st);
    return launch_outer_t<NT, float>((const float*)E, (const float*)H, R, C, dh, work, img, Vblk, partial, p, st);
}

hipError_t launch_project_outer(const void* E, const void* H, int dtype, int64_t R, int64_t C, int64_t dh, void* work,
                                const void* img, const float* Vblk, int KP, float* partial, const ScorePlan& p,
                                hipStream_t st) {
    switch (KP / 32) {
        case 1: return launch_outer_nt<1>(E, H, dtype, R, C, dh, work, img, Vblk, partial, p, st);
        case 2: return launch_outer_nt<2>(E, H, dtype, R, C, dh, work, img, Vblk, partial, p, st);
        case 4: return launch_outer_nt<4>(E, H, dtype, R, C, dh, work, img, Vblk, partial, p, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace sage
