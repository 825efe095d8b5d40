// Internal declarations shared by the host-side translation units of the
// library (launchers, polar driver, server).  Not part of the ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/la.h"
#include "polar_host.h"

struct la_context {
    int device;
    int num_cus;
    void *scratch;   // this device's static polar workspace (la_polar_noalloc)
};

namespace la {

// One GEMM-shaped launch: out = alpha * op(A) op(B) + beta * E + gamma * I.
//   op(A) (M x K): a_kcontig ? A[i * lda + k] : A[k * lda + i]
//   op(B) (K x N): b_kcontig ? B[j * ldb + k] : B[k * ldb + j]
//   out  (M x N): C[i * ldc + j]
//   E: optional addend (may equal C for beta * C), E[i * lde + j]
//   gram: output is symmetric (M == N): only tiles on or above the diagonal
//         are computed; element (i, j), i <= j, is written to (i, j) and
//         (j, i), so the result is exactly symmetric.
//   partials: optional, one FP64 per output tile: sum over the tile of
//         (out - E)^2, for the step norm ||X' - X||_F; requires E.
struct GemmDesc {
    const float *A;
    const float *B;
    float *C;
    const float *E;
    double *partials;
    int64_t lda, ldb, ldc, lde;
    int64_t M, N, K;
    float alpha, beta, gamma;
    int a_kcontig, b_kcontig;
    int gram;
    int gram_upper;    // gram: write only the upper triangle (no mirror)
    int vec_a, vec_b;  // the operand's leading dimension suits the loader's 32-bit offsets
    int tiles_m, tiles_n;
    int num_tiles;     // tiles launched (upper triangle only for gram)
    int small;         // tile class (chosen from the problem's own shape)
    int quarters;      // small tiles covering large Gram tiles tail_first.. (4 per tile)
    int tail_first;
    // split-K slices in one launch: slice y takes k in [y slice_k, min(K,
    // (y + 1) slice_k)) and writes C + y slice_stride (slice_k a multiple of
    // 32, so every slice but the last is whole K stages; any on the direct classes)
    int slices;
    int64_t slice_k, slice_stride;
    // (what every launch reads ends here, in three lines of kernel arguments: each
    // further line a kernel touches late is a read it waits for)
    // PREC_F16X3: powers of two op(A) and op(B) are multiplied by before their
    // split (the caller divides alpha by their product: gemm_f16_scales)
    float scale_a, scale_b;
    // PREC_F16X3 on operands packed row by row (launch_pack's rmax): the bits of
    // the largest magnitude of each row of op(A) and each column of op(B), or
    // null; out_max: optional, takes the maximum with each output column's
    const uint32_t *row_max, *col_max;
    uint32_t *out_max;
    int ptile;         // packed operands: tile side, 256, 192 or 128 (gemm_set_packed)
    // direct classes and packed operands: optional device word; while it is not 0 the
    // launch leaves its outputs as they are (a step queued past the iteration's stop, a
    // product of an input too uneven for its arithmetic)
    const int *stop;
    // direct classes, two-term precisions: the output is also (or, with C null, only)
    // written as packed operands of arithmetic pack_prec (factor pack_scale): pack_row with the
    // output's rows as rows and its columns as k, pack_col the other way round
    // (either may be null; a Gram's are one matrix: pack_row only).  pack_pairs:
    // rows in the order the 64 x 64 class gives a row-contiguous operand.
    char *pack_row, *pack_col;
    float pack_scale;
    int pack_prec, pack_pairs;
    int b_pairs;       // packed operands: op(B)'s rows are in that order
    int prec, packed;  // launch_gemm_mixed: arithmetic; packed operands
};

// Tile classes.  Large (256 x 256) and small (128 x 128) tiles (gemm_tile.h) use
// the same K stages and product order, so the choice between these two never
// changes a result.  The direct classes (gemm_direct.h: 64 x 64 and 32 x 32
// tiles whose waves split K) each add in an order of their own, the same on
// packed operands.  The class follows from the problem's own shape, whatever the
// leading dimensions, so a problem's result does not depend on what it is launched
// with or where its operands lie.
constexpr int kClassLarge = 0, kClassSmall = 1, kClassDirect64 = 2, kClassDirect32 = 3;
inline bool is_direct(int cls) { return cls >= kClassDirect64; }

// Tile geometry of each precision and tile class.
int tile_m(int prec, int cls = 0);
int tile_n(int prec, int cls = 0);

// Fills the derived fields (tile class, vec flags, tile counts) of d.
void gemm_finalize(GemmDesc &d, int prec);
// Sets d's tile class and the tile counts that follow from it.
void gemm_set_class(GemmDesc &d, int prec, int cls);
// Sets d up for packed operands (launch_gemm_packed): a direct class as it is,
// else the tile side and the counts that follow from it.
void gemm_set_packed(GemmDesc &d);
// Partials of a step norm that a workspace has room for, of an M x N iterate: one per
// 128 x 128 tile.  The region of the norm partials (sumsq_num_partials) follows it and
// is free during the steps, so a launch of smaller tiles may write its partials over both
// (step_room); a launch with more of them (a long side beside one below 128, and a few
// sizes at FP32) leaves its partials out, and launch_diff_sumsq writes others.
size_t step_partials(int64_t M, int64_t N);
inline bool step_room(int64_t count, const double *tiles, const double *sumsq, int sumsq_count)
{
    return count <= (sumsq - tiles) + sumsq_count;
}

// Sets the factors of a PREC_F16X3 product (powers of two sa, sb with |sa a| and
// |sb b| below the fp16 range for every entry of its operands) and takes them
// out of alpha again; other precisions are left as they are.
inline void gemm_f16_scales(GemmDesc &d, int prec, float sa, float sb)
{
    if (prec == PREC_F16X3) {
        d.scale_a = sa;
        d.scale_b = sb;
        d.alpha /= sa * sb;
    }
}

hipError_t launch_gemm(int prec, const GemmDesc &d, hipStream_t s);

// MI355X dispatches consecutive workgroups round-robin over its 8 XCDs.
constexpr int kXcds = 8;

// Grouped launch: every item is one output tile of one problem; all problems
// share precision, operand layouts and tile class.  probs / items live in
// device memory.  One workgroup per item, item b on workgroup b, hence on XCD
// b % kXcds.  An item with prob < 0 is empty (padding of a list laid out for
// the XCDs).  hipErrorInvalidValue for an op(B) with k contiguous, and for the direct
// classes at another arithmetic than FP32.
struct GroupItem {
    int prob;
    int tile;   // linear tile index within the problem
};
hipError_t launch_gemm_grouped(int prec, int a_kcontig, int b_kcontig, int cls,
                               const GemmDesc *probs_dev,
                               const GroupItem *items_dev, int num_items, hipStream_t s);
// The same over problems of the direct classes of several arithmetics (not FP32)
// and classes, each with its own (d.prec, d.small) and on FP32 or packed operands
// (d.packed).  update: op(A) k contiguous, op(B) row-contiguous or packed in pair
// order; else both row-contiguous or packed in order.
hipError_t launch_gemm_mixed(int update, const GemmDesc *probs_dev, const GroupItem *items_dev,
                             int num_items, hipStream_t s);

// Packed operands of two 16-bit terms (gemm_x3.hip: 3xBF16, gemm_f16x3.hip:
// F16X3, whose entries are multiplied by sc before the split, or, with rmax, each
// row by the power of two that brings its largest entry to [2^14, 2^15); with skip, nothing
// is done while *skip is not 0): op(X) (rows x k; kc: k contiguous,
// X[r * ld + k], else X[k * ld + r]) split into bf16 hi/lo terms and laid out
// in the GEMM's LDS fragment order, zero-padded to 256 rows and 16 k.
size_t packed_x3_bytes(int64_t rows, int64_t k);
// A matrix is too uneven for PREC_F16X3 if more than a quarter of the entries of some row
// or column are smaller than what two scaled fp16 terms hold with 23 bits (zeros too).  A
// product with one operand that is even has an error floor below the rounding of its
// accumulation, whatever the other holds: every column of the other meets entries of
// the size of the first one's largest.  A pack with rmax and counts (rows + k words of
// zeros) looks for entries below 2^-17 of their row's largest (a row of zeros has none)
// and sets bit in *flag if op(X) is uneven.
struct PackCheck {
    uint32_t *counts = nullptr;
    int *flag = nullptr;
    int bit = 0;
};
hipError_t launch_pack(int prec, const float *X, int64_t ld, int kc, int64_t rows, int64_t k,
                       float sc, void *out, hipStream_t s, const uint32_t *rmax = nullptr,
                       const int *skip = nullptr, const PackCheck &check = PackCheck());
// GEMM on packed operands: d.A and d.B point at packed op(A) (M x K) and
// packed op(B)^T (N x K), set up by gemm_set_packed.
// Computes the same products in the same order as launch_gemm's kernel of that precision.
hipError_t launch_gemm_packed(int prec, const GemmDesc &d, hipStream_t s);

// C (rows x cols, ldc) <- C - Y Z with Y (rows x K, k contiguous, ldy) and
// Z (K x cols, ldz), K <= 128 (qr_update.hip): the short-K update of
// Algorithm caqr, every element as launch_gemm computes alpha Y Z + beta C
// with alpha = -1, beta = 1 on the 128 x 128 tile class.
hipError_t launch_short_update(int prec, const float *Y, int64_t ldy, const float *Z, int64_t ldz,
                               float *C, int64_t ldc, int64_t rows, int64_t cols, int K,
                               hipStream_t s);

// Auxiliary kernels (aux_kernels.hip).
// Sum of squares of an m x n strided matrix into nparts FP64 partials.
int sumsq_num_partials();
hipError_t launch_sumsq(const float *X, int64_t m, int64_t n, int64_t ld,
                        double *partials, hipStream_t s);
// The same of X - E.
hipError_t launch_diff_sumsq(const float *X, int64_t ldx, const float *E, int64_t lde, int64_t m,
                             int64_t n, double *partials, hipStream_t s);
// out[0] = sum of parts[0..count) in a fixed order (deterministic).
hipError_t launch_reduce_fixed(const double *parts, int64_t count, double *out,
                               hipStream_t s);
// Y = X / nrm, element-wise in FP64 then rounded to FP32 (so scaling A by a
// power of two leaves Y bitwise unchanged).
hipError_t launch_scale(const float *X, int64_t ldx, float *Y, int64_t ldy,
                        int64_t m, int64_t n, double nrm, hipStream_t s);
// The same with nrm = sqrt(*nrm2) read on the device (no host round trip); Y
// stays as it is if stop is given and *stop is not 0.
hipError_t launch_scale_by_norm(const float *X, int64_t ldx, float *Y, int64_t ldy,
                                int64_t m, int64_t n, const double *nrm2, hipStream_t s,
                                const int *stop = nullptr);
// State of an iteration whose steps are queued ahead of their stop test, in
// device memory.  launch_norm_state: norm2 = the sum of the partials; stop = 1
// (reason 3) unless sqrt(norm2) is positive and finite.  launch_step_state,
// after a step: nothing once stopped, else steps += 1, delta = scale *
// sqrt(sum of the partials) and the driver's stop test in FP64: not finite
// (reason 3); delta <= the tolerance, tol, or tol 2^steps if tol_doubles
// (reason 0); delta < stag_below and delta > half the one before (reason 1;
// stag_below <= 0: off); steps = max_steps (reason 2).
struct StepState {
    double norm2, delta, prev, pad0;
    int stop, steps, reason, pad1;
};
struct StepTest {
    double scale, tol, stag_below;
    int tol_doubles, max_steps;
};
// StepState::reason of an input too uneven for the arithmetic of the steps queued
constexpr int kReasonUneven = 4;
hipError_t launch_norm_state(const double *parts, int64_t count, StepState *st, hipStream_t s);
hipError_t launch_clear_state(StepState *st, hipStream_t s);
hipError_t launch_step_state(const double *parts, int64_t count, StepState *st,
                             const StepTest &test, hipStream_t s);
// X = A^T / a (FP64 division, rounded once); A is n x m, X is m x n.
hipError_t launch_transpose_scale(const float *A, int64_t lda, float *X, int64_t ldx,
                                  int64_t n, int64_t m, double a, hipStream_t s);
// out[i] = bits of the largest magnitude in row i (by_row) or column i of the m x n
// X (the largest of any NaN's bits if there is one).  launch_zero: count words.
hipError_t launch_absmax(const float *X, int64_t ldx, int64_t m, int64_t n, int by_row,
                         uint32_t *out, hipStream_t s);
hipError_t launch_zero(uint32_t *out, int64_t count, hipStream_t s);
// Y (may be X) = X with each row times the power of two that takes its largest magnitude
// (mx: launch_absmax by row) to [2^14, 2^15), or divided by it (unscale).
hipError_t launch_scale_rows(const float *X, int64_t ldx, float *Y, int64_t ldy, int64_t m,
                             int64_t n, const uint32_t *mx, int unscale, hipStream_t s);
// Whether the m x n X (m, n >= 1, ||X||_F^2 in *nrm2) is too uneven (see PackCheck) for
// operands scaled by their norm: with entries below 2^-18 ||X||_F for the small ones.  If
// so *flag (may be null) becomes 1, and *st (may be null; unless stopped) stops for
// kReasonUneven; else both stay as they are.  counts: m + n words of zeros.
hipError_t launch_uneven(const float *X, int64_t ldx, int64_t m, int64_t n, const double *nrm2,
                         uint32_t *counts, int *flag, StepState *st, hipStream_t s);
// Y = s A + t I for an n x n A (FP64 per element, rounded once).
hipError_t launch_affine(const float *A, int64_t lda, float *Y, int64_t ldy, int64_t n,
                         double sc, double t, hipStream_t s);
// Y = X (strided copy).
hipError_t launch_copy(const float *X, int64_t ldx, float *Y, int64_t ldy,
                       int64_t m, int64_t n, hipStream_t s);
// In place H <- (H + H^T) / 2 for an n x n matrix.
hipError_t launch_symmetrize(float *H, int64_t ldh, int64_t n, hipStream_t s);
// Split-K reduction for a symmetric (gram) output: out(i, j) =
// alpha * sum_s part_s(i, j) + gamma * [i == j], summed over s in order in
// FP64 and rounded once; parts are `splits` exactly symmetric n x n slices
// (row-major, ld n).
// Slice s is at parts + s * stride (elements; any distance within one
// allocation).
hipError_t launch_splitk_sym_reduce(const float *parts, int64_t stride, int splits, int64_t n,
                                    double alpha, double gamma, float *out,
                                    int64_t ldo, hipStream_t s);
// Split-K reduction of an m x n product: out = alpha * sum_s part_s + beta * E
// (FP64, rounded once; E may be null), parts m x n row-major (ld n).  If step
// is not null, FP64 partial sums of (out - E)^2 go to
// step[0 .. splitk_update_num_partials()).
int splitk_update_num_partials();
hipError_t launch_splitk_update_reduce(const float *parts, int splits, int64_t m, int64_t n,
                                       double alpha, double beta, const float *E, int64_t lde,
                                       float *out, int64_t ldo, double *step, hipStream_t s);

// Grouped fixed-order FP64 reduction: one workgroup per item,
// out[0] = sum of parts[0..count) (same order as launch_reduce_fixed).
struct ReduceItem {
    const double *parts;
    int64_t count;
    double *out;
};
hipError_t launch_reduce_grouped(const ReduceItem *items_dev, int n, hipStream_t s);

// Polar building blocks shared by la_polar and the server (PolarPlan,
// polar_plan and the stop test are in polar_host.h).
// Number of split-K slices the Gram of an m x n iterate uses, and the number
// needed to keep an inner dimension K within the FP32 accumulation depth.
int gram_splits(int64_t m, int64_t n, int prec, int64_t max_acc);
int acc_splits(int64_t K, int64_t max_acc);
size_t polar_workspace_bytes(const PolarPlan &p);

// Packed copies that the products of a polar iteration on the direct classes
// hand on: each writes its result both as FP32 and split into the terms that the
// next product reads (X_i as rows for the update, as columns for the Gram, P_i for
// the update), so no operand is split again by every tile that reads it.  Every
// product is the same bits as on FP32 operands (and its partial sums too), so a
// caller without room for them runs unpacked with the same result.
struct PolarChain {
    char *row[2];   // X (m x n) with its rows as rows, for X in either buffer
    char *col;      // X with its columns as rows
    char *P;        // P (n x n)
    int pairs;      // P's rows in pair order: the update is of the 64 x 64 class
};
// Bytes of a chain for p, 0 where its products don't take one: a product that is
// not two-term or not of a direct class, or, for la_polar, a split update, a split
// Gram or n < kChainMinN.  served: the server's rule.
size_t polar_chain_bytes(const PolarPlan &p, bool served = false);
PolarChain polar_chain_carve(const PolarPlan &p, char *base);


// Argument helpers shared by the ABI entry points (la_api.hip).
la_status dev_fail(hipError_t e, const char *where);   // sets the error, LA_ERR_DEVICE
bool overlaps(const void *a, size_t abytes, const void *b, size_t bbytes);
size_t extent_bytes(int64_t rows, int64_t cols, int64_t ld);   // bytes spanned by a matrix
int resolve_prec(int p, int dflt);                      // AUTO -> dflt
bool valid_prec(int p);
size_t align_up256(size_t x);

#define LA_HIP(call, where)                        \
    do {                                           \
        hipError_t e_ = (call);                    \
        if (e_ != hipSuccess)                      \
            return ::la::dev_fail(e_, where);      \
    } while (0)

}  // namespace la
