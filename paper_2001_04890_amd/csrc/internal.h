// Device-side data structures shared by the host driver (host.cpp) and the HIP kernels
// (kernels.hip). Plain structs, no HIP types, so host-only builds can include it.
//
// Padded layouts. Every operator block in the pool is stored row-major with its rows padded to a
// multiple of 16 and its leading dimension (columns) padded to a multiple of 32, zero-filled.
// Before each H.psi the input vector is packed into the same kind of layout (rows and columns of
// every psi block padded to multiples of 32). MFMA tiles therefore never need bounds masks.
#pragma once
#include <stdint.h>

namespace dmrg {

constexpr int kRowPad = 16;    // row padding of pool blocks (MFMA tile height)
constexpr int kLd = 32;        // leading-dimension padding of pool blocks and packed psi blocks
inline int32_t ld_of(int32_t m) { return (m + kLd - 1) / kLd * kLd; }
inline int32_t rows_of(int32_t m) { return (m + kRowPad - 1) / kRowPad * kRowPad; }
// Bytes allocated behind the arrays whose operands hpsi_rs64.hip and hpsi_lds.hip read with a scalar offset in
// the buffer load (the operand pools and the packed X^T). A kernel class made for longer operands asks up to 15
// column groups of 128 rows (120 KB) past the end of a short one. The card's range check stops these loads, but
// the compiler's intrinsic leaves the scalar offset out of the check that it promises; with the slack they would
// stay inside the allocation without it.
constexpr int kOperandSlack = 15 * 32 * 256;

// One sector-GEMM contribution to an output psi block (Eq. dgemm, Section 2.2.1):
//   Y_target += f * A . X_source . B^T
// A (m_a' x m_a) and B (m_d' x m_d) live in the operator pool (padded layout); a_off / b_off < 0
// mean identity. X is read from the packed input (pa x pd, row-major, ld = pd; and for the split
// path also its transpose, ld = pa).
struct Task {
    int64_t x_off;   // element offset of the packed source block
    int64_t a_off;   // pool offset of A, or -1
    int64_t b_off;   // pool offset of B, or -1
    double  f;
    int32_t pa;      // source rows padded to 32 (leading dimension of A and of the packed X^T)
    int32_t pd;      // source cols padded to 32 (leading dimension of B and of the packed X)
    int32_t ka;      // source rows padded to 16 (FP64 reduction bound over m_a)
    int32_t kd;      // source cols padded to 16 (FP64 reduction bound over m_d)
};

// One wavefront's work: a contiguous range of the tasks writing one output tile of a target block
// (rows [r0, r0 + 16*TP) x cols [c0, c0 + 16*TQ)). slot < 0: the item owns the whole tile and stores
// it into y; otherwise it stores a partial tile into partial slot `slot` and a reduction item adds
// the slots of the tile in a fixed order (deterministic, no atomics).
struct Item {
    int64_t y_off;
    int64_t part_off;        // < 0: store into y; else offset of this item's partial tile (tm x tn)
    int32_t m_ap, m_dp;
    int32_t r0, c0;
    int32_t t_begin, t_end;
    int32_t part = 0;        // merged problem of the target (dmrg_hop_combine), see kPartActive
    int32_t pad = 0;
};
constexpr int kTileRows = 32;                  // max rows of a tile (TP <= 2)
constexpr int kPartialVecs = 4;                // vectors per launch

struct Reduce {
    int64_t y_off;
    int64_t part_off;        // first partial tile; the tile's n_parts partials follow contiguously
    int32_t m_ap, m_dp;
    int32_t r0, c0;
    int32_t tm, tn;          // tile extent
    int32_t n_parts;
    int32_t part;            // merged problem of the target
};
// Part mask of a merged handle: launchers take an optional device array with one entry per merged
// problem; the records (items, reductions, pass-1 groups) of a problem whose entry is not
// kPartActive are skipped, which leaves its part of y unspecified. A null mask runs every record.
constexpr int32_t kPartActive = 1;

// ---------------------------------------------------------------- tiled split-BF16 operands
// Split-BF16 operands of the sector-GEMM kernels are stored pre-tiled in MFMA fragment
// order: a matrix with R rows (padded to 16) and K columns (padded to 32) is cut into 16 x 32 tiles,
// tile (rt, kt) at ((rt * K/32) + kt) * kTileU16 elements, row-major over tiles. Inside a tile the
// 64 lanes' 8-element fragments are contiguous (hi: lane * 8 + u, lo: 512 + lane * 8 + u) with lane
// l = (row % 16) + 16 * ((col % 32) / 8), u = col % 8 -- the operand layout of
// v_mfma_f32_16x16x32_bf16. A pool block of rows_of(R) x ld_of(K) doubles at pool offset o occupies
// exactly the u16 range [2 o, 2 o + 2 rows_of(R) ld_of(K)) of the tiled array.
constexpr int kTileU16 = 1024;
struct PoolBlock { int64_t off; int32_t r16, k32, rows, cols; };   // rows, cols: before padding

// Task of the split row-mode and task-mode kernels: Y_tile += f * A . X . B^T with every factor present (identity
// factors point at tiled identity blocks). Offsets are u16 offsets into the tiled arrays.
struct LTask {
    int64_t x_off;   // tiled X^T of the source block (see k_pack_xt)
    int64_t a_off;   // tiled A block (rows = target rows, K = source rows)
    int64_t b_off;   // tiled B block (rows = target cols, K = source cols)
    float   f;
    int16_t pa32;    // source rows padded to 32, in units of 32
    int16_t pd32;    // source cols padded to 32, in units of 32
};

// Packing of one psi block into the padded input layout.
struct PackBlock {
    int64_t src_off;         // offset in the caller's x (m_a x m_d, row-major)
    int64_t dst_off;         // offset in the packed buffers
    int32_t m_a, m_d;
    int32_t pa, pd;
};

// Pre-summed / transposed operator block (Section 2.2.3): out = sum_k coeff_k * src_k (or src_k^T).
struct PresumBlock {
    int64_t out_off;
    int32_t rows, cols;
    int32_t t_begin, t_end;
};
struct PresumTerm {
    int64_t src_off;
    int32_t src_ld;
    int32_t trans;
    double  coeff;
};

// Diagonal contribution of a task that maps a block onto itself: D += f diag(A) diag(B)^T.
struct DiagTask {
    int64_t a_off, b_off;   // -1 for identity
    double  f;
};
struct DiagBlock {
    int64_t off;
    int32_t m_a, m_d;
    int32_t t_begin, t_end;
};

}  // namespace dmrg

#ifndef DMRG_HOST_ONLY
#include <hip/hip_runtime.h>
namespace dmrg {
// H.psi launch plan. Work items are grouped by phase (a subset of the operator combinations whose
// operators fit in the last-level cache) and, inside a phase, by tile class
// c = (TP - 1) * 8 + (TQ - 1), TP in 1..2, TQ in 1..8. y is zeroed first; every item and every
// reduction then adds its tile into y (each tile has one owner per phase, phases run in order).
constexpr int kClasses = 16;
struct HpsiLaunch { int cls, item_begin, item_count; };
struct HpsiPhase { int launch_begin, launch_end, reduce_begin, reduce_end; };
struct HpsiPlan {
    const Item* items;            // device
    const Reduce* reduces;        // device
    const Task* tasks;            // device
    double* partial;              // device, partial_size * kPartialVecs doubles
    int64_t partial_size;         // elements of the partial tiles of one vector (largest phase)
    const HpsiLaunch* launches;   // host
    const HpsiPhase* phases;      // host
    int n_phases;
    const PackBlock* packs;       // device
    int n_packs;
    int64_t packed_size;          // elements of one packed vector
    double* xp;                   // packed FP64 input, kPartialVecs vectors
    uint16_t* xr_hi;              // packed BF16 split input, row-major
    uint16_t* xr_lo;
    uint16_t* xt_hi;              // packed BF16 split input, transposed
    uint16_t* xt_lo;
};

// Launch plan of the split row-mode and task-mode kernels (hpsi_lds.hip). Row-mode items (internal.h Item)
// cover whole targets; class (S, NW): S = largest padded dimension (64 or 96), NW = wavefronts of two row
// tiles each; each class is one launch.
// Tasks whose source is a single 32 x 32 tile run in the task-mode kernel (one wavefront per target
// block of NR row tiles and at most NQ column tiles), classes (NR, NQ) = (1,2) (2,2) (1,4), launched
// after the row-mode classes; items[small_begin[c] .. small_begin[c+1]).
// Row-mode classes (64,2) (64,3) (96,2) (96,3): a target's tasks whose source and columns are within 64
// run in the S = 64 classes, the other big-source tasks in the S = 96 classes; targets of up to kLdsRows row
// tiles have two wavefronts, the others three. The FP64 sums in LDS bound the wavefronts of a CU: 16 KB each
// at S = 64, so 10 (two a workgroup) or 9 (three), 24 KB at S = 96, so 6; the registers would allow 12 and 8.
constexpr int kLdsRows = 4;
constexpr int kLdsClasses = 4;
constexpr int kSmallClasses = 3;
constexpr int kReduceKinds = 3;         // partial tiles of S = 64 runs, S = 96 runs, task-mode runs
struct LdsPlan {
    const Item* items = nullptr;        // device
    const LTask* tasks = nullptr;       // device
    const Reduce* reduces = nullptr;    // device, grouped by kind; one reduction launch per kind
                                        // (records of one kind cover disjoint parts of y)
    int red_begin[kReduceKinds + 1] = {0, 0, 0, 0};
    int red_chunks[kReduceKinds] = {1, 1, 1};   // 256-element chunks of the largest tile per kind
    int cls_begin[kLdsClasses + 1] = {0, 0, 0, 0, 0};   // item ranges per class
    int small_begin[kSmallClasses + 1] = {0, 0, 0, 0};
    double* partial = nullptr;          // device, partial_size * kPartialVecs doubles
    int64_t partial_size = 0;
    const PackBlock* packs = nullptr;   // device (same packing geometry as HpsiPlan)
    int n_packs = 0;
    int64_t xt_size = 0;                // u16 elements of one tiled X^T vector (2 * packed_size)
    uint16_t* xt = nullptr;             // device, xt_size * kPartialVecs
};

// ---------------------------------------------------------------- FP64 operands of the MFMA kernels
// Operand form of the FP64 kernels (hpsi_rs64.hip, hpsi_big64.hip): a matrix of R rows and K columns (K
// the reduction index) is padded to R4 = ceil(R / 4) groups of 4 rows and ceil(K / 8) groups of 8
// columns, zero-filled, and stored by column group p, inside it by 16-row tile, inside that as [g][li][u]
// with element M[16 rt + li][8 p + 4 u + g], g < 4, li < the tile's rows, u < 2. So a lane (li, g) of
// v_mfma_f64_16x16x4f64 reads its operands of two k steps as 16 contiguous bytes, a full tile's column
// group is 1 KB in lane order, and a small block takes little more than its elements: 8 x 8 states are
// 512 B where whole 16 x 16 tiles of a 32-padded matrix are 4 KB.
inline int32_t k4_of(int32_t m) { return (m + 3) / 4; }
inline int64_t op64_size(int32_t rows, int32_t cols) { return (int64_t)k4_of(rows) * ((cols + 7) / 8) * 32; }
struct OpBlock64 { int64_t src, dst; int32_t ld, rows, cols, pad; };   // pool block -> operand form

// Launch plan of the register-streamed FP64 kernel (hpsi_rs64.hip). Items (internal.h Item) are
// wavefronts: r0 = 16 x the row tile, c0 = the class 8 k + q, with k an index into kRsK (source rows in
// 16-wide tiles; 0: source rows and columns both within 8) and q one into kRsQ (target columns).
// begin[g] .. begin[g + 1]: the items of launch group g (register budgets, see the kernel).
constexpr int kRsWaves = 4;             // wavefronts (items) per workgroup (1: 3% slower at 1024 states, 1% faster at 333)
constexpr int kRsGroups = 5;
constexpr int kRsK[7] = {0, 1, 2, 3, 4, 6, 8};
constexpr int kRsQ[6] = {1, 2, 3, 4, 6, 8};
constexpr int kRsMaxTiles = 8;          // target rows are any; target columns, source rows and columns
inline int rs_kclass(int ka4, int kd4) {
    if (ka4 <= 2 && kd4 <= 2) return 0;
    int c = 1;
    while (4 * kRsK[c] < ka4) ++c;
    return c;
}
inline int rs_qclass(int tiles) { int c = 0; while (kRsQ[c] < tiles) ++c; return c; }
// Launch group of a class: the accumulators (8 registers a column tile), the A row tile (8 a source tile),
// the two rings and what the compiler takes besides (16 .. 30) within 64, 96, 128, 168 or 256 registers, i.e.
// 8, 5, 4, 3 or 2 wavefronts per SIMD.
constexpr int rs_group(int k, int q) {
    const int kp = k == 0 ? 1 : 2 * kRsK[k], qt = kRsQ[q], jp = k == 0 ? 1 : 2;
    const int rx = kp == 16 ? 8 : kp, rb = qt == 8 ? 4 : qt;
    const int regs = 8 * qt + 4 * (kp + rx + rb * jp) + (qt == 8 ? 30 : qt == 6 ? 20 : qt == 4 ? 18 : 16);
    return regs <= 64 ? 0 : regs <= 96 ? 1 : regs < 128 ? 2 : regs <= 168 ? 3 : 4;
}
struct LTask64 {
    int64_t x_off, a_off, b_off;        // doubles: X^T of the source in xt, A and B in the operand pool
    double  f;
    int32_t ka4, kd4;                   // source rows / columns in 4-wide k steps
};
struct RsPlan64 {
    const Item* items = nullptr;        // device
    const LTask64* tasks = nullptr;     // device
    const Reduce* reduces = nullptr;    // device; one record per target cut into several items
    int n_reduces = 0;
    int red_chunks = 1;                 // 256-element chunks of the largest partial tile
    int begin[kRsGroups + 1] = {0, 0, 0, 0, 0, 0};
    double* partial = nullptr;          // device, partial tiles of one vector
    int64_t partial_size = 0;
    int n_items = 0;                    // task ranges (each runs as one wavefront per row tile of its target)
};
// y (one vector) += the plan's targets of f A X B^T; xt = that vector's X^T in operand form
hipError_t launch_hpsi_rs64(const RsPlan64& P, const double* ops, const double* xt, double* y, hipStream_t s,
                            const int32_t* active = nullptr);
// operand form of the pool's blocks, and of X^T of every psi block (hpsi_big64.hip); y (if given) = 0
hipError_t launch_op64(const double* pool, const OpBlock64* blocks, int n_blocks, double* ops, hipStream_t s);
hipError_t launch_pack_xt64(const PackBlock* packs, int n_packs, const double* x, double* xt, double* y, hipStream_t s);
// y (one vector) += the partial tiles of each record, in order (hpsi_lds.hip)
hipError_t launch_reduce_partials(const Reduce* reduces, int n, int chunks, const double* partial, double* y,
                                  hipStream_t s, const int32_t* active = nullptr);

// Two-pass large-block path, split (hpsi_big.hip) or FP64 (hpsi_big64.hip). Targets are grouped into chunks;
// per chunk, pass 1 writes T = f A X of every task into a buffer of tiles in the A-operand layout of pass 2
// (tile (rt, jt) of a task's T is its tile rt * pd + jt), pass 2 accumulates Y += sum_tasks T B^T.
// Split form: offsets in u16, T in tiles of 16 x 32 (hi and lo, kTileU16). FP64 form: offsets in doubles, A, B
// and X^T in the FP64 operand form, T in tiles of 16 x 16 (256 doubles).
struct BigT {              // one wavefront's part of a task's T; ka = 0: none
    int64_t xt, a, t;
    double f;
    int32_t ka;            // source rows: in 32-wide k tiles (split), in 4-wide k steps (FP64)
    int32_t kd, ra;        // FP64 form: source columns and target rows in 4-wide groups
    int32_t pd;            // T tiles along the source columns
    int16_t rb, nr, jb, nj;   // row tiles [rb, rb + nr) and T tile columns [jb, jb + nj)
    int32_t part;          // merged problem of the target
    int32_t pad;
};
// n tiles are cut into equal parts of at most `most`, the longer ones first: length of the one at tile t
constexpr int part_len(int n, int t, int most) {
    const int parts = (n + most - 1) / most, len = n / parts, more = n % parts;
    return t < more * (len + 1) ? len + 1 : len;
}
struct BigT2 {             // pass-2 task: T of the task and its B block
    int64_t t, b;
    int32_t pd32;
    int32_t kd;            // FP64 form: 4-wide k steps holding data
};
// Chunk c: pass-1 work [t1_begin, t1_end), pass-2 items [item_begin, item_end) (one wavefront each),
// reductions [red_begin, red_end).
struct BigChunk { int t1_begin, t1_end, item_begin, item_end, red_begin, red_end; };
struct BigPlan {
    const BigT* t1 = nullptr;       // device
    const BigT2* t2 = nullptr;      // device
    const Item* items = nullptr;    // device: pass-2 items (r0 = 16 rb, c0 = 16 qb, task range in t2)
    const Reduce* reduces = nullptr;
    const BigChunk* chunks = nullptr;   // host
    int n_chunks = 0;
    int red_chunks = 1;             // 256-element chunks of the largest partial tile
    uint16_t* tbuf = nullptr;       // device, largest chunk's T (one vector at a time; doubles in the FP64 form)
    double* partial = nullptr;      // device, partial tiles of the largest chunk
    int64_t partial_size = 0;
};

// Launchers (kernels.hip). All asynchronous on `s`.
hipError_t launch_presum(const PresumBlock* blocks, int n_blocks, const PresumTerm* terms,
                         double* pool, hipStream_t s);
hipError_t launch_split(const double* pool, int64_t n, uint16_t* hi, uint16_t* lo, hipStream_t s);
hipError_t launch_hpsi_f64(const HpsiPlan& plan, const double* pool, const double* x, double* y,
                           int64_t n_coeff, int nvec, hipStream_t s, const int32_t* active = nullptr);
hipError_t launch_hpsi_split(const HpsiPlan& plan, const uint16_t* hi, const uint16_t* lo, const double* x,
                             double* y, int64_t n_coeff, int nvec, hipStream_t s, const int32_t* active = nullptr);
hipError_t launch_diag(const DiagBlock* blocks, int n_blocks, const DiagTask* tasks,
                       const double* pool, double* d, hipStream_t s);
// Davidson vector kernels (FP64).
hipError_t launch_multidot(const double* V, int nv, int64_t n, const double* w, double* partial,
                           int n_part, double* out, hipStream_t s);
constexpr int kMaxCombine = 72;
struct Coefs { double c[kMaxCombine]; };
hipError_t launch_combine(const double* V, int nv, int64_t n, const Coefs& coef, double* out,
                          double beta, hipStream_t s);
hipError_t launch_precond(const double* r, const double* d, double theta, double* t, int64_t n,
                          hipStream_t s);
hipError_t launch_scale(double* x, double a, int64_t n, hipStream_t s);
int multidot_parts(int64_t n);
// out -= sum_j c[j] V[j], c in device memory; x *= 1 / sqrt(*nrm2) with *nrm2 in device memory.
// x -= sum_j (V[j] . x) V[j] (sums: room for nv doubles); x /= |x| with |x|^2 left in *nrm2
hipError_t launch_orthogonalize(const double* V, int nv, int64_t n, double* x, double* partial, int n_part, double* sums,
                                hipStream_t s);
hipError_t launch_normalize(double* x, int64_t n, double* partial, int n_part, double* nrm2, hipStream_t s);

// Reduced density matrix of the enlarged left block (Section 2.1), one item per (sector, row group,
// row group): rho[rho_off + l * ld + l2] = sum over the sector's n_cd column groups k of
// sum_r X_{g,k}[l][r] X_{g2,k}[l2][r], with X_{g,k} the psi block at gblk[g + k] (row-major, m_d =
// cdmd[cd + k] columns), l < ma, l2 < ma2. Every element of rho is written by exactly one item.
struct RdmItem {
    int64_t rho_off;
    int32_t ld, ma, ma2, g, g2, cd, n_cd, pad;
};
// units: the 32 x 32 tiles of every item (row-major tile index). right: rho^R = psi^T psi with the same
// items: ma, ma2 are then the column counts of the two psi blocks of each term (their m_d), cdmd[cd + k]
// the k-th row count (m_a), and the sum runs over rows.
struct RdmUnit { int32_t item, tile; };
hipError_t launch_rdm(bool right, const RdmItem* items, const RdmUnit* units, int n_units, const int64_t* gblk,
                      const int32_t* cdmd, const double* psi, double* rho, hipStream_t s);

// Eq. renorm_mat per sector block, out = O_out^T A O_in (renorm.hip). A is rows x cols (= O_out rows x
// O_in rows), row-major; O matrices are row-major (rows x k). The first n_large items have a workgroup or
// more each, max_in / max_out: most columns of O_in / O_out of one of them; the n_small others, for which
// renorm_small holds, a wavefront.
struct RenormItem {
    int64_t a_off, out_off, oo_off, oi_off;
    int32_t rows, cols, k_out, k_in;
};
inline bool renorm_small(const RenormItem& it) { return it.rows <= 32 && it.k_in <= 32; }
hipError_t launch_renormalize(const RenormItem* items, int n_large, int n_small, int max_in, int max_out, const double* A,
                              const double* O, double* out, hipStream_t s);
// Tiled split-BF16 kernels (hpsi_lds.hip).
hipError_t launch_split_tiled(const double* pool, const PoolBlock* blocks, int n_blocks, uint16_t* tiled, hipStream_t s);
// y (+)= H x over the LDS plan's targets; zero_y: clear y first (else accumulate into it).
hipError_t launch_hpsi_lds(const LdsPlan& plan, const uint16_t* pool_t, const double* x, double* y, int64_t n_coeff,
                           int nvec, bool zero_y, hipStream_t s, const int32_t* active = nullptr);
// Large-block split path (hpsi_big.hip) for one vector: y += the large targets' part of H x;
// xt = that vector's tiled X^T (packed by launch_hpsi_lds).
hipError_t launch_hpsi_big(const BigPlan& plan, const uint16_t* pool_t, const uint16_t* xt, double* y,
                           hipStream_t s, const int32_t* active = nullptr);
// FP64 large-block path (hpsi_big64.hip) for one vector: y += the large targets' part of H x, over the
// FP64 operand pool and that vector's X^T in operand form (launch_pack_xt64).
hipError_t launch_hpsi_big64(const BigPlan& plan, const double* ops, const double* xt, double* y, hipStream_t s,
                             const int32_t* active = nullptr);
// Old-kernel split path over a plan without clearing y first.
hipError_t launch_hpsi_split_acc(const HpsiPlan& plan, const uint16_t* hi, const uint16_t* lo, const double* x,
                                 double* y, int64_t n_coeff, int nvec, hipStream_t s,
                                 const int32_t* active = nullptr);
}  // namespace dmrg
#endif
