// Internal declarations shared by the translation units of the SAGE HIP library (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sage.h"
#include "select_plan.h"
#include "xcd_map.h"

namespace sage {

// ---- sketch / basis layout --------------------------------------------------------------------------------
// The 2*ell x D buffer is kept as column slabs: element (row r, column d) lives at
//     ((d / DC) * NP + r) * DC + d % DC
// with DC = 16 floats (64 B) per row per slab and NP = padded row count. One slab (NP x 16 floats) is one
// contiguous block, so the Gram kernel stages a slab with linear 1 KB wave loads, and the rebuild / basis
// kernels read a 128 B line per buffer-row pair. Columns D..Dp-1 and rows beyond 2*ell are always zero.
constexpr int DC = 16;

struct Dims {
    int ell;      // sketch size
    int n;        // 2*ell buffer rows
    int LP;       // ell padded to 32 * 2^j (32, 64, 128, 256)
    int NP;       // 2*LP padded buffer rows (64 .. 512)
    int64_t D;    // columns
    int64_t S;    // slabs = ceil(D / DC)
    int64_t Dp;   // S * DC
};

__host__ __device__ inline int64_t blk_off(int64_t d, int r, int NP) {
    return ((d / DC) * NP + r) * (int64_t)DC + (d % DC);
}

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));  // indexable 16-byte piece

// fp32 matrix-core step: acc(32x32) += a(32x2) * b(2x32). Lane l supplies a[l%32][l/32] and b[l/32][l%32];
// acc element i of lane l is row 8*(i/4) + 4*(l/32) + i%4, column l%32.
__device__ __forceinline__ f32x16 mfma32(float a, float b, f32x16 acc) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0);
}

__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// v_mfma_f32_32x32x16_bf16: acc(32x32) += a(32x16) b(16x32). Lane l supplies a[l%32][8*(l/32) .. +8] and
// b[8*(l/32) .. +8][l%32]; acc element i of lane l is row 8*(i/4) + 4*(l/32) + i%4, column l%32.
__device__ __forceinline__ f32x16 mfma_bf16(u32x4 a, u32x4 b, f32x16 acc) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0,
                                                   0, 0);
}

__device__ __forceinline__ unsigned pack_bf16(float x, float y) {
    bf16x2 h = {(__bf16)x, (__bf16)y};  // round to nearest even (v_cvt_pk_bf16_f32)
    return __builtin_bit_cast(unsigned, h);
}

// An fp32 pair as three bf16 pairs hi + mid + lo (each the nearest bf16 of what the previous ones left): the three
// parts carry 24 significant bits, |x - hi - mid - lo| <= 2^-26 |x|.
__device__ __forceinline__ void split3_bf16(float x, float y, unsigned& hi, unsigned& mid, unsigned& lo) {
    hi = pack_bf16(x, y);
    const float rx = x - __uint_as_float(hi << 16), ry = y - __uint_as_float(hi & 0xffff0000u);
    mid = pack_bf16(rx, ry);
    lo = pack_bf16(rx - __uint_as_float(mid << 16), ry - __uint_as_float(mid & 0xffff0000u));
}

// The upper halves of an fp32 pair as a bf16 pair: exact when both are bf16 values (rows of a bf16 stream kept as fp32).
__device__ __forceinline__ unsigned hi_bf16(float x, float y) {
    return __builtin_amdgcn_perm(__float_as_uint(y), __float_as_uint(x), 0x07060302u);
}

// The new half of a bf16 stream at the largest size (256 rows) is kept in bf16: pieces of 8 columns (16 bytes), those of
// column group q and row r at (q * LP + r), in the upper half of the memory of the fp32 half (so that it can be widened in
// place). Half the bytes, and a piece is what a matrix-core lane of the Gram kernels takes.
__host__ __device__ inline const u32x4* half16(const float* half, int LP, int64_t S) {
    return reinterpret_cast<const u32x4*>(half + S * LP * (DC / 2));
}

// ---- kernel launchers (each enqueues on `st` and returns hipGetLastError()) ---------------------------------
// launch_util.hip: raise a kernel's dynamic LDS limit, once per (device, kernel); thread-safe
hipError_t ensure_dynamic_lds(const void* kernel, int bytes);
// The XCD this work-group runs on, 0..7.
__device__ __forceinline__ int xcd_id() {
    int id;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(id));
    return id & 7;
}
// Work that runs beside an eigensolve keeps off the XCD that the reduction has to itself: *hole is the place left out (spare_unit), set
// by launch_xcd_place before it on the same stream; null: none is.
__device__ __forceinline__ int64_t spare_unit_at(const int* __restrict__ hole) {
    return spare_unit(blockIdx.x, hole ? *hole : -1);
}
inline int64_t spare_grid_at(int64_t units, const int* hole) { return spare_grid(units, hole ? 0 : -1); }
// fd_insert.hip
// copy `rows` batch rows into rows row0.. of a half buffer (half_rows rows per slab)
// (to16: in pieces of bf16, see half16; rows of bf16 only)
hipError_t launch_insert(const void* G, int dtype, int64_t rows, int row0, float* half, int half_rows, const Dims& d,
                         bool to16, const int* hole, hipStream_t st);
// factored rows (E: rows x C logit errors, H: rows x dh features, both of the row type): column c*dh + t = e_c * h_t
// rounded as a stored row would be, column C*dh + c = e_c; requires D = C * (dh + 1)
hipError_t launch_insert_outer(const void* E, const void* H, int dtype, int64_t C, int64_t dh, int64_t rows, int row0,
                               float* half, int half_rows, const Dims& d, bool to16, const int* hole, hipStream_t st);
hipError_t launch_widen(float* half, const Dims& d, hipStream_t st);  // pieces of bf16 -> the fp32 half
// ... written out row-major (rows x D of the row type)
hipError_t launch_expand_outer(const void* E, const void* H, int dtype, int64_t C, int64_t dh, int64_t rows, void* out,
                               const Dims& d, hipStream_t st);
hipError_t launch_plain_copy(const void* src, void* dst, int64_t bytes, hipStream_t st);
// *count += entries of p (n values of the row type) that are not finite
hipError_t launch_count_nonfinite(const void* p, int dtype, int64_t n, unsigned* count, hipStream_t st);
hipError_t launch_probe_permute(const double* in, double* out, int NP, int LP, int ell, bool both, hipStream_t st);
hipError_t launch_export_rows(const float* Bblk, int NPsrc, int nrows, float* out, const Dims& d, hipStream_t st);
hipError_t launch_import_rows(const float* in, int nrows, float* Bblk, int NPdst, const Dims& d, hipStream_t st);
hipError_t launch_zero_rows(float* Bblk, int NP, int r0, int r1, const Dims& d, hipStream_t st);

// fd_gram.hip
// The buffer is two half buffers (top: matrix rows 0 .. LP-1, new: matrix rows LP .. NP-1, the first nfill in use).
struct GramPlan {
    int mode;         // 0: tiles t0.. of the lower triangle; 1: new rows x top rows; 2: new rows x new rows (triangle)
    int t0;           // mode 0: first tile computed (the top x top block before it is known to the caller)
    int tiles;        // 64x64 tiles computed
    int wg_per_group; // ceil(tiles / 6): a work-group computes 12 half-tiles
    int groups;       // split-K groups (multiple of 8)
    int64_t slabs_per_group;
    size_t partial_floats; // groups * tiles * 4096
    bool split = false;    // modes 1 and 2, NP = 512 only: the kernels on the bf16 matrix cores (three-way split values)
};
// The plan of the same block (mode 1 or 2) for the split-arithmetic kernels: one work-group per group, same partial
// tiles; groups > 0 overrides the group count (tiles = 0 in the result: not available for this sketch size).
GramPlan gram_plan_split(const GramPlan& base, const Dims& d, int groups);
GramPlan gram_plan(const Dims& d, int num_cu, int mode, bool skip_top, int wg_per_cu);
// new_one (split-arithmetic kernels): the new half is kept in pieces of bf16 (half16): one part instead of three, the result
// has the same bits
hipError_t launch_gram(const float* top, const float* nw, int nfill, float* partial, const GramPlan& p, const Dims& d,
                       hipStream_t st, bool new_one = false, const int* hole = nullptr);
// Mode 2 of row-major bf16 rows that are stored into the half `nw`, in pieces of bf16, on the way (from its row 0 on).
bool gram_rows_ok(const GramPlan& p, const Dims& d);
hipError_t launch_gram_rows16(const void* G, int rows, float* nw, float* partial, const GramPlan& p, const Dims& d, const int* hole,
                              hipStream_t st);
// Mode 1 with several half buffers for the top rows: the partial tiles of p[j] are `stride` floats after those of p[j - 1]. (NP <= 256
// or a split plan.)
constexpr int GRAM_TOPS = 6;
struct GramTops {
    const float* p[GRAM_TOPS];
    int64_t stride;
    int rows;  // of each; what a half holds beyond counts as zero
};
hipError_t launch_gram_tops(const GramTops& tops, int count, const float* nw, int nfill, float* partial, const GramPlan& p,
                            const Dims& d, hipStream_t st, bool new_one, const int* hole);
// ... all of them and the new half kept in pieces of bf16 (half16; NP = 512, a split plan)
hipError_t launch_gram_blocks(const GramTops& tops, int count, const float* nw, int nfill, float* partial, const GramPlan& p,
                              const Dims& d, hipStream_t st, const int* hole);
// C = sum of the partial tiles of launch a and (if given) launch b; known_top: the top x top block is diag(known)
// (the Gram matrix of the rows the last shrink wrote, see EigWork::known). done: recorded when C is complete (may be null; not
// on a stream that is captured)
hipError_t launch_gram_reduce(const float* partial_a, const GramPlan& a, const float* partial_b, const GramPlan* b,
                              double* C, bool known_top, const double* known, const Dims& d, hipStream_t st,
                              const float* partial_top = nullptr, const GramPlan* top = nullptr, hipEvent_t done = nullptr);

// NP = 64: top <- M [top; nw], and the partial tiles of the Gram matrix of [top; next], ell rows each, by the plan of the whole triangle.
hipError_t launch_rebuild_gram(float* top, const float* nw, const float* next, const float* Mc, float* partial, const GramPlan& p,
                               const Dims& d, hipStream_t st);

// Rows to be stored into a half, from its row 0 on, as fp32, by a launch of the eigensolve (NP = 64): a row-major batch G, or factors.
struct RowJob {
    const void *G, *E, *H;
    int64_t C, dh;
    int dtype, rows;
    float* half;
    Dims d;
};
// fd_tridiag.hip, fd_dc.hip, fd_eig.hip: the eigensolve
struct DcWork {  // work arrays of the merges above 64 rows (see fd_dc.hip)
    double *dk, *zk, *org, *tau, *val, *zh, *rc, *rs;  // NP each
    int *col, *half, *npos, *from, *ra, *rb;           // NP each
    int *K, *k1, *dense, *nrot;                        // per sub-problem
};
struct EigWork {
    double* C;      // NP x NP Gram matrix, left untouched
    double* Yt;     // NP x NP: row m = eigenvector of the m-th largest eigenvalue
    double* V;      // NP x NP Householder vectors (row k: the reflector of step k)
    double* Tw;     // 8 NP: triangular factors of the blocks of eight reflectors (fd_wy.h)
    double* Z[2];   // NP x NP, column-major: eigenvectors of T, ping-pong between the merges
    double* dT;     // NP: diagonal, sub-diagonal and reflector factors of the reduction
    double* eT;
    double* tauT;
    double* dI[2];  // NP: eigenvalues, ascending, in units of 2^stat[0]
    double* stat;   // [0] exponent of the scaling
    double* redone; // solves whose reduction one work-group repeated because the others were not there in time
    unsigned* claim; // [0] zero before and after a reduction (TriClaim), [1] set when the solve is given up, [2], [3] bits of the
                     // columns that are left of it (zero before it)
    bool impatient; // test hook: its work-groups wait for each other for one poll only
    double* known;  // LP: Gram matrix of the rows the last shrink wrote (diagonal): max(lambda_j - delta, 0)
    double* xch;    // exchange of the reduction (NP = 128, 256, 512): 4 slots of q and c, NP each; empty (all ones) before it
    int xcd;        // the XCD the reduction runs on (NP = 128, 256, 512)
    int period;     // of the work-groups of a launch over the XCDs (XcdMap), 0: not known
    DcWork dc;
};
// which of dI / Z the last merge of a solve of size NP writes
inline int dc_result(int NP) { return (NP == 128 || NP == 512) ? 1 : 0; }
// Matrix indices in use: 0 .. m0-1 and LP .. LP + (n - m0) - 1, n in all (the others are zero rows and columns); the count
// leading eigenvectors are formed.
hipError_t launch_xcd_place(int xcd, int* place, hipStream_t st);  // *place: 0 .. 7, device memory
const XcdMap& xcd_map();  // of the launches on some stream of the current device; asked once per device
hipError_t launch_tridiag(const EigWork& w, int NP, int m0, int n, hipStream_t st, const RowJob* job = nullptr);  // (job: NP = 64)
hipError_t launch_dc(const EigWork& w, int NP, int n, hipStream_t st);
// Coefficients of a shrink (mode 0), a basis (1) or a weighted basis (2), MP rows of which `count` are not zero; into M if given, else into
// Mc3 (split parts) if given, else into Mt. Scalars on device: acc[0] sum_delta, acc[1] frob2 (+= diag(C) over matrix indices [ra0, ra1)
// and [rb0, rb1), the rows not yet counted), acc[2] last_delta. (acc[4]: EigWork::redone)
struct CoeffArgs {
    int MP, count, mode, n, ell, ra0, ra1, rb0, rb1;
    float* Mt;
    void* Mc3;
    double* acc;
    double* M = nullptr;  // given: the coefficients go here in fp64, MP x NP in matrix indices, and to neither of the above
};
// the `count` leading eigenvectors into Yt, or (cf given) only the coefficients made from them
hipError_t launch_tri_back(const EigWork& w, int NP, int m0, int n, int count, const CoeffArgs* cf, hipStream_t st);
hipError_t launch_eig(const EigWork& w, int NP, int m0, int n, int count, const CoeffArgs* cf, hipStream_t st, const RowJob* job = nullptr);
hipError_t launch_eig_export(const EigWork& w, int NP, double* Y, double* lam, double* record, hipStream_t st);

// fd_defer.hip: shrinks whose rows are written later. LP = 64, 128, 256; all in fp64.
// Partial tiles of `sources` rectangles (launch_gram_tops with plan pc, `stride` floats apart) into K, source s from column col[s]
// on, and of the new x new triangle (plan pn) into C.
hipError_t launch_defer_reduce(const float* cross, int64_t stride, int sources, const int* col, int top_groups, int groups, const float* fresh,
                               const GramPlan& pn, double* K, int ldk, double* C, const Dims& d, hipStream_t st);
// out (LP x LP) = K W^T over `len` columns
hipError_t launch_defer_fold(const double* K, int ldk, const double* W, int ldw, int len, double* out, int ldo, const Dims& d,
                             hipStream_t st);
// ... into the new x top rectangle of C; its top x top block becomes diag(known)
hipError_t launch_defer_cross(const double* K, int ldk, const double* W, int ldw, int len, double* C, const double* known,
                              const Dims& d, hipStream_t st, hipEvent_t done);
// out = [M_top W, M_new], W of `cols` columns
hipError_t launch_defer_compose(const double* M, const double* W, int ldw, int cols, double* out, int ldo, const Dims& d,
                                hipStream_t st);
// the rebuild's coefficients of W's first `rows` columns, into Mc3 if given, else into Mt
hipError_t launch_defer_coeffs(const double* W, int ldw, int rows, float* Mt, void* Mc3, const Dims& d, hipStream_t st);

// Where the coefficient M[m][i] (output row m < MP, buffer row i < NP) is stored for the rebuild kernel: chunks of
// 16 buffer rows; inside a chunk [i & 1][m][(i & 15) >> 1], i.e. the 8 values a matrix-core lane needs are
// contiguous, and the two 16-byte halves of those 32 bytes are swapped when (m >> 3) is odd so that a quarter wave
// reading one half touches every LDS bank once.
__host__ __device__ inline int64_t coeff_offset(int i, int m, int MP) {
    const int s = (i & 15) >> 1, h = i & 1;
    const int piece = (s >> 2) ^ ((m >> 3) & 1);
    return (int64_t)(i >> 4) * 16 * MP + ((h * MP + m) * 2 + piece) * 4 + (s & 3);
}

// Blocks of new rows that lie in one ring of half buffers: block b is slot (slots >> 4 b) & 15 of it.
struct NewBlocks {
    const float* ring = nullptr;
    int64_t stride = 0;  // floats
    unsigned slots = 0;
    int count = 0;
    __host__ __device__ __forceinline__ int64_t offset(int b) const { return (int64_t)(slots >> (4 * b) & 15u) * stride; }
    __host__ __device__ __forceinline__ const float* at(int b) const { return ring + offset(b); }
};
// fd_rebuild.hip: out[0:MP] = M * B over every column, B = [top; the blocks, the first nfill rows of each in use]; Mc holds the
// coefficients, LP (1 + blocks) x MP, in coeff_offset order; out has out_NP rows per slab and may be `top` itself (in place).
hipError_t launch_rebuild(const float* top, const NewBlocks& nw, int nfill, const float* Mc, float* out, int out_NP, int MP,
                          const Dims& d, hipStream_t st, const int* hole = nullptr);
// The same product on the bf16 matrix cores with both factors split into three bf16 parts (six products: 24-bit
// accuracy at 2.7 times the fp32 matrix-core rate). Mc3: the split coefficients of `rows` buffer rows, rebuild_split_bytes(rows, MP)
// bytes. Only for MP = 128 or 256 (rebuild_split_ok).
bool rebuild_split_ok(int MP);
size_t rebuild_split_bytes(int rows, int MP);
// new_one: every new row in use holds bf16 values (three products instead of six for the blocks, the same bits); at NP = 512
// the blocks are then kept in pieces of bf16.
hipError_t launch_rebuild_split(const float* top, const NewBlocks& nw, int nfill, const void* Mc3, float* out, int out_NP, int MP,
                                const Dims& d, hipStream_t st, bool new_one = false, const int* hole = nullptr);
// KP rows of a basis (mode: CoeffArgs) from those that the last shrink wrote, nothing else being in the buffer
hipError_t launch_basis_rows(const float* top, const double* known, int k, int mode, float* out, int KP, const Dims& d, hipStream_t st);

// score.hip
struct ScorePlan {
    int row_tiles;    // ceil(R / 128)
    int splits;       // split-K over D
    int64_t slabs_per_split;
    // factored rows only: the splits form a grid of class groups x feature-window groups
    int class_groups = 0, classes_per_group = 0, window_groups = 0, windows_per_group = 0;
    int bias_slots = 0, classes_per_bias_slot = 0;  // ... followed by the slots of the bias columns
};
ScorePlan score_plan(int64_t R, const Dims& d, int num_cu);
hipError_t launch_project(const void* G, int dtype, int64_t R, const float* Vblk, int KP, float* partial,
                          const ScorePlan& p, const Dims& d, hipStream_t st);
// first: ssum is set, not added to. ticket: one word, zero, and zero again afterwards. src_labels (may be null): labels of the
// rows, copied to dst_labels.
hipError_t launch_score_finalize(const float* partial, int64_t R, int KP, int k, int splits, float* zhat_out,
                                 double* cons_partial, unsigned* ticket, double* ssum, int mode, bool first, float* alpha_out,
                                 const int* src_labels, int* dst_labels, hipStream_t st);

// score_split.hip: the same projection on the bf16 matrix cores with the basis split as hi + lo (bf16 each).
// The basis is kept as per-chunk LDS images built once per basis by launch_basis_split (from the fp32 slabs).
// Usable when every row starts on a 16-byte boundary (split_path_ok); ScorePlan::slabs_per_split then counts
// chunks of 128 row bytes.
bool split_path_ok(const void* G, int dtype, const Dims& d);
// ... or, with a basis of three parts (fp32 accuracy), for rows of any alignment.
bool any_path_ok(const void* G, int dtype, const Dims& d);
size_t basis_image_bytes(int KP, int dtype, int parts, const Dims& d);
hipError_t launch_basis_split(const float* Vblk, int KP, int dtype, int parts, void* img, const Dims& d, hipStream_t st);
ScorePlan score_split_plan(int64_t R, int dtype, const Dims& d, int num_cu);
hipError_t launch_project_split(const void* G, int dtype, int64_t R, int parts, const void* img, int KP, float* partial,
                                const ScorePlan& p, const Dims& d, hipStream_t st);

// The projection of factored rows (see launch_insert_outer) without storing them. Needs the images and the fp32 slabs
// of the basis; writes p.splits + p.bias_slots partial slots (the last ones hold the bias columns).
bool outer_path_ok(const void* E, const void* H, int dtype, int64_t C, int64_t dh);
ScorePlan score_outer_plan(int64_t R, int dtype, int64_t C, int64_t dh, int num_cu);
// work: outer_work_bytes(R, dtype, C) bytes (receives the transposed errors)
size_t outer_work_bytes(int64_t R, int dtype, int64_t C);
hipError_t launch_project_outer(const void* E, const void* H, int dtype, int64_t R, int64_t C, int64_t dh, void* work,
                                const void* img, const float* Vblk, int KP, float* partial, const ScorePlan& p,
                                hipStream_t st);

// select.hip
hipError_t launch_cosine(const float* zhat, int64_t N, int k, const double* ssum, float* alpha, hipStream_t st);
struct SelectWork {
    uint32_t* hist;      // TOPM_HIST_WORDS: one histogram per digit
    uint32_t* state;     // 4: {digits found, count left} after the first and the second digit
    uint32_t* blk_gt;    // per block: keys above all that share the first two digits
    uint32_t* blk_in;    // per block: keys that share them
    uint16_t* table;     // per block, 1024: those with a third digit of at least the index
    int64_t nblk_cap;
};
// a work space of topm_work_words(blocks) words at p
inline SelectWork select_work_at(uint32_t* p, int64_t blocks) {
    SelectWork w{};
    w.hist = p;
    w.state = w.hist + TOPM_HIST_WORDS;
    w.blk_gt = w.state + SELECT_STATE_WORDS;
    w.blk_in = w.blk_gt + blocks;
    w.table = (uint16_t*)(w.blk_in + blocks);
    w.nblk_cap = blocks;
    return w;
}
bool topm_needs_work(int64_t N);    // false: launch_topm uses no work space
// A word of pinned host memory that the last kernel of a call sets to `token` once the call's results are in memory, for a
// host that spins on it: 6.5 us from launch to answer where hipStreamSynchronize takes 11.5. null: no signal.
struct HostSignal {
    unsigned* word = nullptr;
    unsigned token = 0;
};
bool topm_signals(int64_t N, int64_t m);  // launch_topm sets the word
// clear: the histograms of w are zero, as every run leaves them; otherwise one launch more makes them so.
hipError_t launch_topm(const float* alpha, int64_t N, int64_t m, int64_t* out_idx, const SelectWork& w, bool clear,
                       hipStream_t st, HostSignal done = HostSignal{});
constexpr int COPY_SIGNAL_MAX = 32768;  // floats: 32 a thread of the one work-group; more is the copy engine's work
hipError_t launch_copy_signal(const float* src, int n, float* dst, HostSignal done, hipStream_t st);

// select_cb.hip: class-balanced selection (per-class centroid, cosine to it, top k_c of every class)
struct CbWork {
    long long* sums;   // C x 128 fixed-point class sums of zhat
    uint32_t* counts;  // rows per class
    uint32_t* kc;      // rows kept per class
    uint32_t* start;   // first place of the class in ord
    uint32_t* cursor;  // ... next free one
    uint32_t* misc;    // [0] total kept, [1] a label was out of range
    uint32_t* blk;     // per block of SELECT_BLOCK rows: rows kept
    uint32_t* ord;     // the rows, class after class
    uint32_t* skey;    // their score keys, in that order
    uint8_t* sel;      // per row: kept
};
size_t cb_work_bytes(int C, int64_t N);
CbWork cb_work_layout(void* base, int C, int64_t N);
// rule: sage_cb_rule (how the subset size is shared out among the classes). Scores to alpha; the kept rows, ascending, to
// out_idx if there are at most cap; report (host memory the device can write): {rows kept, a label was out of range}.
hipError_t launch_cb_select(const float* zhat, const int* labels, int64_t N, int k, int C, double keep, int rule,
                            float* alpha, int64_t cap, int64_t* out_idx, uint32_t* report, const CbWork& w, hipStream_t st);

}  // namespace sage
