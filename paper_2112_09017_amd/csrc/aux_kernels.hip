// Auxiliary kernels of the polar, inversion and matrix-function drivers: FP64
// norm reductions (the scaling ||A||_F and the step norm ||U' - U||_F of
// Algorithm NS_Polar, section III.D), scaling, transpose-scaling, the affine
// map s A + t I, copies, symmetrisation of H, split-K reduction, and the
// precision dispatch of the GEMM launchers.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "la_internal.h"

namespace la {

hipError_t launch_gemm_fp32(const GemmDesc &d, hipStream_t s);
hipError_t launch_gemm_x3(const GemmDesc &d, hipStream_t s);
hipError_t launch_gemm_x6(const GemmDesc &d, hipStream_t s);
hipError_t launch_gemm_f16(const GemmDesc &d, hipStream_t s);
hipError_t launch_grouped_f16(int, int, int, const GemmDesc *, const GroupItem *, int,
                              hipStream_t);
hipError_t launch_pack_x3(const float *, int64_t, int, int64_t, int64_t, void *, hipStream_t);
hipError_t launch_pack_f16(const float *, int64_t, int, int64_t, int64_t, float, const uint32_t *,
                           void *, const int *, const PackCheck &, hipStream_t);
hipError_t launch_gemm_packed_x3(const GemmDesc &d, hipStream_t s);
hipError_t launch_gemm_packed_f16(const GemmDesc &d, hipStream_t s);
hipError_t launch_grouped_fp32(int, int, int, const GemmDesc *, const GroupItem *, int,
                               hipStream_t);
hipError_t launch_grouped_x3(int, int, int, const GemmDesc *, const GroupItem *, int,
                             hipStream_t);
hipError_t launch_grouped_x6(int, int, int, const GemmDesc *, const GroupItem *, int,
                             hipStream_t);

int tile_m(int, int cls)
{
    return cls == kClassLarge ? 256 : cls == kClassSmall ? 128 : cls == kClassDirect64 ? 64 : 32;
}
int tile_n(int prec, int cls) { return tile_m(prec, cls); }

static bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Tile class of a product, by its shape alone.  Measured (ns per unit of K,
// 3xBF16 / 6xBF16 / FP32; the last round of workgroups counts as a whole one):
//   direct64, up to 512 tiles 28 / 35 / 59, 1024 47 / 56 / 107, 1536 62 / 71 /
//     131, 2048 79 / 93 / 156, 2560 96 / 118 / 203;
//   small, up to 256 tiles 43 / 52 / 84, 512 57 / 85 / 160, 768 91 / 127 / 234;
//   large, up to 256 tiles 92 / 135 / 271.
// n^3 products (us, 3xBF16): 256 direct32 9 (the host's launch rate), direct64
// 10, small 17; 640 11, 14, 31; 768 19, 17, 36; 1000 26, 20, 65; 1536 84, 63, 69;
// 2048 166, 97, 90; 3000: small 274, large 277.
// So: 32 x 32 tiles while one round of workgroups holds them, 64 x 64 tiles up
// to 2.5 rounds of one per CU and, for FP32, whose small tiles do not gain from
// a second workgroup per CU, from 4 to 6 rounds; large tiles once they give
// half the CUs one; small tiles between.  A matrix with a side below
// 128 is all edge to the staged classes and always direct, and large tiles
// need both sides to hold one.
static int gemm_class(const GemmDesc &d, int prec)
{
    auto tiles = [&](int64_t t) {
        const int64_t tm = (d.M + t - 1) / t, tn = (d.N + t - 1) / t;
        return d.gram ? tn * (tn + 1) / 2 : tm * tn;
    };
    constexpr int64_t kCus = 256;
    const int64_t side = std::min(d.M, d.N);
    if (side >= 256 && tiles(256) >= kCus / 2)
        return kClassLarge;
    if (tiles(32) <= kCus || side < 2)
        return kClassDirect32;
    const int64_t t64 = tiles(64);
    const bool one_deep = prec == PREC_FP32;
    if (side < 128 || 2 * t64 <= 5 * kCus || (one_deep && t64 > 4 * kCus && t64 <= 6 * kCus))
        return kClassDirect64;
    return kClassSmall;
}

void gemm_finalize(GemmDesc &d, int prec)
{
    // The unguarded loader keeps 32-bit element offsets of up to 255 rows (or 24
    // k rows) from a 64-bit stage base; an operand with a longer leading
    // dimension takes the guarded loader, which indexes in 64 bits.
    constexpr int64_t kMaxFastLd = (int64_t)1 << 23;
    d.vec_a = d.lda < kMaxFastLd;
    d.vec_b = d.ldb < kMaxFastLd;
    gemm_set_class(d, prec, gemm_class(d, prec));
}

void gemm_set_class(GemmDesc &d, int prec, int cls)
{
    d.small = cls;
    const int bm = tile_m(prec, cls), bn = tile_n(prec, cls);
    d.tiles_m = (int)((d.M + bm - 1) / bm);
    d.tiles_n = (int)((d.N + bn - 1) / bn);
    if (d.gram)
        d.num_tiles = d.tiles_n * (d.tiles_n + 1) / 2;
    else
        d.num_tiles = d.tiles_m * d.tiles_n;
    if (d.M == 0 || d.N == 0)
        d.num_tiles = 0;
}

// Tile side of a product on packed operands, from the rounds of workgroups its
// tiles take.  Measured, ns per unit of K (n^3 products): 256 x 256 tiles (one
// workgroup per CU) 70-80 per round of 256; 192 x 192 48-51 per round of 256; 128
// x 128 (two per CU) 28 up to 256 tiles, 38 / 40 / 44 at 324 / 400 / 484, 63 / 77
// / 85 at 576 / 784 / 1024, 120 / 187 / 260 / 339 at 1369 / 2209 / 3025 / 4096.
// (3000^3: 256 tiles 206 us, 192 153, 128 188; 7000^3: 2071, 1995, 1820; 8192^3:
// 2539, 3216, 2774.)  The larger tile unless a smaller one is 3% better: it
// reads its operands less often.  A product of the small class keeps its 128 x
// 128 tiles, so that its step norm is summed the same way without a pack.
static int packed_tile(const GemmDesc &d, int cls)
{
    if (cls == kClassSmall)
        return 128;
    auto count = [&](int64_t t) {
        const int64_t tm = (d.M + t - 1) / t, tn = (d.N + t - 1) / t;
        return (d.gram ? tn * (tn + 1) / 2 : tm * tn) * std::max(d.slices, 1);
    };
    auto rounds = [](int64_t t) { return (double)((t + 255) / 256); };
    const int64_t t128 = count(128), rem = t128 % 512;
    const double c256 = 73.0 * rounds(count(256)), c192 = 49.0 * rounds(count(192));
    const double c128 = 43.5 * (double)(t128 / 512) +
                        (rem == 0 ? 0.0 : 28.5 + 15.0 * (double)std::max<int64_t>(0, rem - 256) / 256.0);
    int side = 256;
    double best = c256;
    if (c192 < 0.97 * best) {
        side = 192;
        best = c192;
    }
    return c128 < 0.97 * best ? 128 : side;
}

void gemm_set_packed(GemmDesc &d)
{
    if (is_direct(d.small))
        return;
    d.ptile = packed_tile(d, d.small);
    d.small = kClassLarge;
    d.tiles_m = (int)((d.M + d.ptile - 1) / d.ptile);
    d.tiles_n = (int)((d.N + d.ptile - 1) / d.ptile);
    d.num_tiles = d.gram ? d.tiles_n * (d.tiles_n + 1) / 2 : d.tiles_m * d.tiles_n;
}

size_t step_partials(int64_t M, int64_t N)
{
    return (size_t)((M + 127) / 128) * (size_t)((N + 127) / 128);
}

hipError_t launch_gemm(int prec, const GemmDesc &d, hipStream_t s)
{
    switch (prec) {
    case PREC_FP32: return launch_gemm_fp32(d, s);
    case PREC_BF16X3: return launch_gemm_x3(d, s);
    case PREC_BF16X6: return launch_gemm_x6(d, s);
    case PREC_F16X3: return launch_gemm_f16(d, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_gemm_grouped(int prec, int akc, int bkc, int cls, const GemmDesc *probs,
                               const GroupItem *items, int num_items, hipStream_t s)
{
    switch (prec) {
    case PREC_FP32:
        return launch_grouped_fp32(akc, bkc, cls, probs, items, num_items, s);
    case PREC_BF16X3:
        return launch_grouped_x3(akc, bkc, cls, probs, items, num_items, s);
    case PREC_BF16X6:
        return launch_grouped_x6(akc, bkc, cls, probs, items, num_items, s);
    case PREC_F16X3:
        return launch_grouped_f16(akc, bkc, cls, probs, items, num_items, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_pack(int prec, const float *X, int64_t ld, int kc, int64_t rows, int64_t k,
                       float sc, void *out, hipStream_t s, const uint32_t *rmax, const int *skip,
                       const PackCheck &check)
{
    switch (prec) {
    case PREC_BF16X3: return launch_pack_x3(X, ld, kc, rows, k, out, s);
    case PREC_F16X3: return launch_pack_f16(X, ld, kc, rows, k, sc, rmax, out, skip, check, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_gemm_packed(int prec, const GemmDesc &d, hipStream_t s)
{
    switch (prec) {
    case PREC_BF16X3: return launch_gemm_packed_x3(d, s);
    case PREC_F16X3: return launch_gemm_packed_f16(d, s);
    default: return hipErrorInvalidValue;
    }
}

// ------------------------------------------------------------------ norms

namespace {

constexpr int kSumsqBlocks = 1024;
constexpr int kThreads = 256;

// Block-wide FP64 sum in a fixed order: wave64 butterfly, then wave 0.
__device__ double block_sum(double v, double *sh)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        v += __shfl_xor(v, off, 64);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0)
        sh[w] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int k = 0; k < (int)(blockDim.x >> 6); ++k)
            s += sh[k];
    return s;
}

// Block b sums the squares of rows b, b + grid, ... ; thread t takes columns
// t, t + 256, ...  Each square is formed and accumulated in FP64.
__global__ void __launch_bounds__(kThreads) sumsq_kernel(const float *__restrict__ X, int64_t m,
                                                         int64_t n, int64_t ld,
                                                         double *__restrict__ parts)
{
    __shared__ double sh[kThreads / 64];
    double acc = 0.0;
    for (int64_t r = blockIdx.x; r < m; r += gridDim.x) {
        const float *row = X + r * ld;
        for (int64_t c = threadIdx.x; c < n; c += kThreads) {
            const double x = (double)row[c];
            acc += x * x;
        }
    }
    const double s = block_sum(acc, sh);
    if (threadIdx.x == 0)
        parts[blockIdx.x] = s;
}

// The same of the differences to E: a step norm whose partials per tile have no room.
// Bound by reading both (1000000 x 64, 512 MB: 150 us).
__global__ void __launch_bounds__(kThreads) diff_sumsq_kernel(const float *__restrict__ X,
                                                              int64_t ldx,
                                                              const float *__restrict__ E,
                                                              int64_t lde, int64_t m, int64_t n,
                                                              double *__restrict__ parts)
{
    __shared__ double sh[kThreads / 64];
    double acc = 0.0;
    const int64_t total = m * n, step = (int64_t)gridDim.x * kThreads;
    int64_t r = ((int64_t)blockIdx.x * kThreads + threadIdx.x) / n;
    int64_t c = (int64_t)blockIdx.x * kThreads + threadIdx.x - r * n;
    const int64_t dr = step / n, dc = step - dr * n;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < total; i += step) {
        const double df = (double)X[r * ldx + c] - (double)E[r * lde + c];
        acc += df * df;
        r += dr;
        c += dc;
        if (c >= n) {
            c -= n;
            ++r;
        }
    }
    const double s = block_sum(acc, sh);
    if (threadIdx.x == 0)
        parts[blockIdx.x] = s;
}

// One block: thread t sums parts t, t + 256, ... in order; then block_sum.
__global__ void __launch_bounds__(kThreads) reduce_fixed_kernel(const double *__restrict__ parts,
                                                                int64_t count,
                                                                double *__restrict__ out)
{
    __shared__ double sh[kThreads / 64];
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < count; i += kThreads)
        acc += parts[i];
    const double s = block_sum(acc, sh);
    if (threadIdx.x == 0)
        out[0] = s;
}

// reduce_fixed_kernel's sum, then the state of an iteration (see StepState).
__device__ double fixed_sum(const double *parts, int64_t count, double *sh)
{
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < count; i += kThreads)
        acc += parts[i];
    return block_sum(acc, sh);
}

__device__ void reset_state(StepState *st, double norm2, bool ok)
{
    st->norm2 = norm2;
    st->delta = INFINITY;
    st->prev = INFINITY;
    st->stop = ok ? 0 : 1;
    st->steps = 0;
    st->reason = ok ? 2 : 3;
}

__global__ void __launch_bounds__(kThreads) norm_state_kernel(const double *__restrict__ parts,
                                                              int64_t count, StepState *st)
{
    __shared__ double sh[kThreads / 64];
    const double s = fixed_sum(parts, count, sh);
    if (threadIdx.x == 0) {
        const double nrm = sqrt(s);
        reset_state(st, s, nrm > 0.0 && isfinite(nrm));
    }
}

__global__ void clear_state_kernel(StepState *st) { reset_state(st, 0.0, true); }

__global__ void __launch_bounds__(kThreads) step_state_kernel(const double *__restrict__ parts,
                                                              int64_t count, StepState *st,
                                                              StepTest t)
{
    __shared__ double sh[kThreads / 64];
    if (st->stop)
        return;
    const double s = fixed_sum(parts, count, sh);
    if (threadIdx.x == 0) {
        const double delta = t.scale * sqrt(s);
        const int steps = st->steps + 1;
        int stop = 1, reason = 2;
        if (!isfinite(delta))
            reason = 3;
        else if (delta <= (t.tol_doubles ? ldexp(t.tol, steps) : t.tol))
            reason = 0;
        else if (delta < t.stag_below && delta > 0.5 * st->prev)
            reason = 1;
        else
            stop = steps >= t.max_steps;
        st->prev = delta;
        st->delta = delta;
        st->steps = steps;
        st->reason = reason;
        st->stop = stop;
    }
}

__global__ void __launch_bounds__(kThreads) reduce_grouped_kernel(const ReduceItem *__restrict__ items)
{
    __shared__ double sh[kThreads / 64];
    const ReduceItem it = items[blockIdx.x];
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < it.count; i += kThreads)
        acc += it.parts[i];
    const double s = block_sum(acc, sh);
    if (threadIdx.x == 0)
        it.out[0] = s;
}

__global__ void scale_kernel(const float *__restrict__ X, int64_t ldx, float *__restrict__ Y,
                             int64_t ldy, int64_t m, int64_t n, double nrm)
{
    for (int64_t r = blockIdx.y; r < m; r += gridDim.y)
        for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < n;
             c += (int64_t)gridDim.x * blockDim.x)
            Y[r * ldy + c] = (float)((double)X[r * ldx + c] / nrm);
}

// scale_kernel with nrm = sqrt(*nrm2) taken on the device (FP64, correctly
// rounded as on the host).
__global__ void scale_by_norm_kernel(const float *__restrict__ X, int64_t ldx,
                                     float *__restrict__ Y, int64_t ldy, int64_t m, int64_t n,
                                     const double *__restrict__ nrm2,
                                     const int *__restrict__ stop)
{
    if (stop && *stop)
        return;
    const double nrm = sqrt(*nrm2);
    for (int64_t r = blockIdx.y; r < m; r += gridDim.y)
        for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < n;
             c += (int64_t)gridDim.x * blockDim.x)
            Y[r * ldy + c] = (float)((double)X[r * ldx + c] / nrm);
}

// X = A^T / a for an n x m A (X is m x n): 32 x 32 tiles staged through LDS
// (padded rows) so that both the read of A and the write of X are coalesced.
// The division is done in FP64 and rounded once, as in scale_kernel.
__global__ void transpose_scale_kernel(const float *__restrict__ A, int64_t lda,
                                       float *__restrict__ X, int64_t ldx, int64_t n,
                                       int64_t m, double a)
{
    __shared__ float t[32][33];
    const int64_t tiles_m = (m + 31) / 32;
    for (int64_t bm = blockIdx.y; bm < tiles_m; bm += gridDim.y) {
        const int64_t i0 = (int64_t)blockIdx.x * 32;   // rows of A = columns of X
        const int64_t j0 = bm * 32;                     // columns of A = rows of X
        for (int r = threadIdx.y; r < 32; r += 8) {
            const int64_t i = i0 + r, j = j0 + threadIdx.x;
            t[r][threadIdx.x] = (i < n && j < m) ? A[i * lda + j] : 0.0f;
        }
        __syncthreads();
        for (int r = threadIdx.y; r < 32; r += 8) {
            const int64_t row = j0 + r, col = i0 + threadIdx.x;
            if (row < m && col < n)
                X[row * ldx + col] = (float)((double)t[threadIdx.x][r] / a);
        }
        __syncthreads();
    }
}

__global__ void zero_kernel(uint32_t *out, int64_t count)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        out[i] = 0;
}

// One wave per row: the maximum of the magnitudes' bits over its columns.
__global__ void __launch_bounds__(kThreads) row_absmax_kernel(const float *__restrict__ X,
                                                              int64_t ldx, int64_t m, int64_t n,
                                                              uint32_t *__restrict__ out)
{
    const int lane = threadIdx.x & 63;
    for (int64_t r = blockIdx.x * (int64_t)(kThreads / 64) + (threadIdx.x >> 6); r < m;
         r += (int64_t)gridDim.x * (kThreads / 64)) {
        uint32_t v = 0;
        for (int64_t c = lane; c < n; c += 64)
            v = max(v, __float_as_uint(X[r * ldx + c]) & 0x7fffffffu);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1)
            v = max(v, (uint32_t)__shfl_xor((int)v, off, 64));
        if (lane == 0)
            out[r] = v;
    }
}

// One thread per column of a strip of rows; the strips meet by atomic maximum.
constexpr int kMaxStrip = 64;
__global__ void __launch_bounds__(kThreads) col_absmax_kernel(const float *__restrict__ X,
                                                              int64_t ldx, int64_t m, int64_t n,
                                                              uint32_t *__restrict__ out)
{
    const int64_t c = blockIdx.x * (int64_t)kThreads + threadIdx.x;
    if (c >= n)
        return;
    for (int64_t r0 = blockIdx.y * (int64_t)kMaxStrip; r0 < m;
         r0 += (int64_t)gridDim.y * kMaxStrip) {
        const int64_t r1 = r0 + kMaxStrip < m ? r0 + kMaxStrip : m;
        uint32_t v = 0;
        for (int64_t r = r0; r < r1; ++r)
            v = max(v, __float_as_uint(X[r * ldx + c]) & 0x7fffffffu);
        atomicMax(out + c, v);
    }
}

// Entries too small for all bits of two scaled fp16 terms, below 2^-18 sqrt(*nrm2),
// counted per row and per column in one pass; whoever takes a count past its quarter
// decides.  A wave takes 16 rows of 128 columns: a lane counts its two columns in
// registers, and lane i the ballots of row i, so an even operand takes no atomics to
// speak of.  Bound by reading X.  (Polars with this pass / without: 320^2 389 / 385 us,
// 400^2 413 / 407, 1000^2 856 / 861, 16384^2 0.874 / 0.876 s.)
constexpr int kEvenRows = 16, kEvenGroups = 2;
__global__ void __launch_bounds__(kThreads)
    small_count_kernel(const float *__restrict__ X, int64_t ldx, int64_t m, int64_t n,
                       const double *__restrict__ nrm2, uint32_t *counts, int *flag, StepState *st)
{
    const int lane = threadIdx.x & 63;
    bool bad = false;
    const int64_t c0 =
        (blockIdx.x * (int64_t)(kThreads / 64) + (threadIdx.x >> 6)) * (64 * kEvenGroups) + lane;
    const float t = (float)(sqrt(*nrm2) * 0x1p-18);
    uint32_t cc[kEvenGroups] = {};
    for (int64_t r0 = blockIdx.y * (int64_t)kEvenRows; r0 < m;
         r0 += gridDim.y * (int64_t)kEvenRows) {
        uint32_t rc = 0;
#pragma unroll
        for (int i = 0; i < kEvenRows; ++i) {
            const int64_t r = r0 + i < m ? r0 + i : m - 1;
            uint32_t count = 0;
#pragma unroll
            for (int g = 0; g < kEvenGroups; ++g) {
                const int64_t c = c0 + 64 * g;
                const float v = X[r * ldx + (c < n ? c : n - 1)];
                const bool small = fabsf(v) < t && c < n && r0 + i < m;
                cc[g] += small;
                count += (uint32_t)__popcll(__ballot(small));
            }
            rc = lane == i ? count : rc;
        }
        if (lane < kEvenRows && rc)
            bad |= 4 * (int64_t)(atomicAdd(counts + r0 + lane, rc) + rc) > n;
    }
#pragma unroll
    for (int g = 0; g < kEvenGroups; ++g)
        if (cc[g])
            bad |= 4 * (int64_t)(atomicAdd(counts + m + c0 + 64 * g, cc[g]) + cc[g]) > m;
    if (!bad)
        return;
    if (flag)
        *flag = 1;
    if (st && atomicCAS(&st->stop, 0, 1) == 0)
        st->reason = kReasonUneven;
}

// Y = X with row r times 2^s (unscale: 2^-s), s taking mx[r] (bits) to [2^14, 2^15), 0 for a
// row of zeros or one that is not finite.
__global__ void __launch_bounds__(kThreads)
    scale_rows_kernel(const float *X, int64_t ldx, float *Y, int64_t ldy, int64_t m, int64_t n,
                      const uint32_t *__restrict__ mx, int unscale)
{
    for (int64_t r = blockIdx.y; r < m; r += gridDim.y) {
        const uint32_t b = mx[r];
        const int s = b == 0 || b >= 0x7f800000u ? 0 : 141 - (int)(b >> 23);
        for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < n;
             c += (int64_t)gridDim.x * blockDim.x)
            Y[r * ldy + c] = ldexpf(X[r * ldx + c], unscale ? -s : s);
    }
}

// Y = s A + t I for an n x n A, in FP64 per element, rounded once (A is not
// read when s == 0).
__global__ void affine_kernel(const float *__restrict__ A, int64_t lda, float *__restrict__ Y,
                              int64_t ldy, int64_t n, double sc, double t)
{
    for (int64_t r = blockIdx.y; r < n; r += gridDim.y)
        for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < n;
             c += (int64_t)gridDim.x * blockDim.x)
            Y[r * ldy + c] =
                (float)((sc != 0.0 ? sc * (double)A[r * lda + c] : 0.0) + (r == c ? t : 0.0));
}

__global__ void copy_kernel(const float *__restrict__ X, int64_t ldx, float *__restrict__ Y,
                            int64_t ldy, int64_t m, int64_t n)
{
    for (int64_t r = blockIdx.y; r < m; r += gridDim.y)
        for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < n;
             c += (int64_t)gridDim.x * blockDim.x)
            Y[r * ldy + c] = X[r * ldx + c];
}

// 32 x 32 blocks on or above the diagonal; each (i < j) pair is owned by one
// thread, so the in-place update is race free.
__global__ void symmetrize_kernel(float *H, int64_t ldh, int64_t n)
{
    const int64_t bi = blockIdx.y, bj = blockIdx.x;
    if (bj < bi)
        return;
    const int64_t i = bi * 32 + threadIdx.y, j = bj * 32 + threadIdx.x;
    if (i >= n || j >= n || j <= i)
        return;
    const float a = H[i * ldh + j], b = H[j * ldh + i];
    const float h = 0.5f * (a + b);
    H[i * ldh + j] = h;
    H[j * ldh + i] = h;
}

// Split-K sums of a symmetric product: the slices hold only their upper
// triangles (i <= j; what lies below is not read).  Block (bj, bi), bj >= bi,
// adds the 64 x 64 tile (bi, bj) of the slices in FP64 in slice order,
// applies the epilogue in FP64, rounds once, writes the tile and, through
// LDS, its transpose at (bj, bi), so out is exactly symmetric and both
// writes are coalesced.  VEC (n, ldo and the slice stride multiples of 4,
// 16-byte aligned bases): each thread moves 4 x 4 elements as float4 rows.
constexpr int kSymTile = 64;

template <bool VEC>
__global__ void __launch_bounds__(256) splitk_sym_reduce_kernel(
    const float *__restrict__ parts, int64_t stride, int splits, int64_t n, double alpha,
    double gamma, float *__restrict__ out, int64_t ldo)
{
    const int64_t bi = blockIdx.y, bj = blockIdx.x;
    if (bj < bi)
        return;
    __shared__ float t[kSymTile][kSymTile + 1];
    const bool diag = bi == bj;
    if constexpr (VEC) {
        const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;   // float4 column, row phase
        const int64_t j0 = bj * kSymTile + 4 * tx;
        for (int r = ty; r < kSymTile; r += 16) {
            const int64_t i = bi * kSymTile + r;
            if (i >= n || j0 >= n)
                continue;
            double acc[4] = {0.0, 0.0, 0.0, 0.0};
            for (int sl = 0; sl < splits; ++sl) {
                const float4 v =
                    *reinterpret_cast<const float4 *>(parts + sl * stride + i * n + j0);
                acc[0] += (double)v.x;
                acc[1] += (double)v.y;
                acc[2] += (double)v.z;
                acc[3] += (double)v.w;
            }
            float f[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                double v = alpha * acc[q];
                if (i == j0 + q)
                    v += gamma;
                f[q] = (float)v;
                t[r][4 * tx + q] = f[q];
            }
            if (!diag) {
                *reinterpret_cast<float4 *>(out + i * ldo + j0) = make_float4(f[0], f[1], f[2], f[3]);
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (i <= j0 + q)
                        out[i * ldo + j0 + q] = f[q];
            }
        }
        __syncthreads();
        // out(j, i) for i < j: row j of the (bj, bi) tile, columns i0 .. i0 + 3
        const int64_t i0 = bi * kSymTile + 4 * tx;
        for (int r = ty; r < kSymTile; r += 16) {
            const int64_t j = bj * kSymTile + r;
            if (j >= n || i0 >= n)
                continue;
            float f[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                f[q] = t[4 * tx + q][r];
            if (!diag) {
                *reinterpret_cast<float4 *>(out + j * ldo + i0) = make_float4(f[0], f[1], f[2], f[3]);
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (i0 + q < j)
                        out[j * ldo + i0 + q] = f[q];
            }
        }
    } else {
        const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
        for (int r = ty; r < kSymTile; r += 4) {
            const int64_t i = bi * kSymTile + r, j = bj * kSymTile + tx;
            if (i < n && j < n && i <= j) {
                double acc = 0.0;
                for (int sl = 0; sl < splits; ++sl)
                    acc += (double)parts[sl * stride + i * n + j];
                double v = alpha * acc;
                if (i == j)
                    v += gamma;
                const float f = (float)v;
                out[i * ldo + j] = f;
                t[r][tx] = f;
            }
        }
        __syncthreads();
        for (int r = ty; r < kSymTile; r += 4) {
            const int64_t j = bj * kSymTile + r, i = bi * kSymTile + tx;   // out(j, i), i < j
            if (i < n && j < n && i < j)
                out[j * ldo + i] = t[tx][r];
        }
    }
}

// out = alpha sum_s part_s + beta E for an m x n product whose slices are
// m x n row-major (ld n), with the FP64 partial sum of (out - E)^2 of block b
// in step[b] (step may be null).  Every thread visits its elements in a fixed
// order and the block sum is a fixed tree, so the partials are reproducible.
// VEC (n, lde, ldo multiples of 4, 16-byte aligned bases): four consecutive
// columns per thread and step, as float4 loads and stores.
template <bool VEC>
__global__ void __launch_bounds__(kThreads) splitk_update_reduce_kernel(
    const float *__restrict__ parts, int splits, int64_t m, int64_t n, double alpha, double beta,
    const float *__restrict__ E, int64_t lde, float *__restrict__ out, int64_t ldo,
    double *__restrict__ step)
{
    __shared__ double sh[kThreads / 64];
    const int64_t mn = m * n;
    double ss = 0.0;
    if constexpr (VEC) {
        for (int64_t r = blockIdx.x; r < m; r += gridDim.x)
            for (int64_t c = 4 * (int64_t)threadIdx.x; c < n; c += 4 * kThreads) {
                double acc[4] = {0.0, 0.0, 0.0, 0.0};
                for (int sl = 0; sl < splits; ++sl) {
                    const float4 v = *reinterpret_cast<const float4 *>(parts + sl * mn + r * n + c);
                    acc[0] += (double)v.x;
                    acc[1] += (double)v.y;
                    acc[2] += (double)v.z;
                    acc[3] += (double)v.w;
                }
                float4 e = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                if (E)
                    e = *reinterpret_cast<const float4 *>(E + r * lde + c);
                const double ev[4] = {(double)e.x, (double)e.y, (double)e.z, (double)e.w};
                float o[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    o[q] = (float)(alpha * acc[q] + beta * ev[q]);
                    const double df = (double)o[q] - ev[q];
                    ss += df * df;
                }
                *reinterpret_cast<float4 *>(out + r * ldo + c) = make_float4(o[0], o[1], o[2], o[3]);
            }
    } else {
        for (int64_t r = blockIdx.x; r < m; r += gridDim.x)
            for (int64_t c = threadIdx.x; c < n; c += kThreads) {
                double acc = 0.0;
                for (int sl = 0; sl < splits; ++sl)
                    acc += (double)parts[sl * mn + r * n + c];
                const double e = E ? (double)E[r * lde + c] : 0.0;
                const float v = (float)(alpha * acc + beta * e);
                out[r * ldo + c] = v;
                const double df = (double)v - e;
                ss += df * df;
            }
    }
    if (step) {
        const double t = block_sum(ss, sh);
        if (threadIdx.x == 0)
            step[blockIdx.x] = t;
    }
}

dim3 grid2d(int64_t m, int64_t n)
{
    int64_t gx = (n + kThreads - 1) / kThreads;
    if (gx > 64)
        gx = 64;
    int64_t gy = m < 4096 ? m : 4096;
    if (gx < 1) gx = 1;
    if (gy < 1) gy = 1;
    return dim3((unsigned)gx, (unsigned)gy);
}

}  // namespace

int sumsq_num_partials() { return kSumsqBlocks; }

hipError_t launch_sumsq(const float *X, int64_t m, int64_t n, int64_t ld, double *partials,
                        hipStream_t s)
{
    hipLaunchKernelGGL(sumsq_kernel, dim3(kSumsqBlocks), dim3(kThreads), 0, s, X, m, n, ld,
                       partials);
    return hipGetLastError();
}

hipError_t launch_diff_sumsq(const float *X, int64_t ldx, const float *E, int64_t lde, int64_t m,
                             int64_t n, double *partials, hipStream_t s)
{
    hipLaunchKernelGGL(diff_sumsq_kernel, dim3(kSumsqBlocks), dim3(kThreads), 0, s, X, ldx, E, lde,
                       m, n, partials);
    return hipGetLastError();
}

hipError_t launch_reduce_fixed(const double *parts, int64_t count, double *out, hipStream_t s)
{
    hipLaunchKernelGGL(reduce_fixed_kernel, dim3(1), dim3(kThreads), 0, s, parts, count, out);
    return hipGetLastError();
}

hipError_t launch_norm_state(const double *parts, int64_t count, StepState *st, hipStream_t s)
{
    hipLaunchKernelGGL(norm_state_kernel, dim3(1), dim3(kThreads), 0, s, parts, count, st);
    return hipGetLastError();
}

hipError_t launch_clear_state(StepState *st, hipStream_t s)
{
    hipLaunchKernelGGL(clear_state_kernel, dim3(1), dim3(1), 0, s, st);
    return hipGetLastError();
}

hipError_t launch_step_state(const double *parts, int64_t count, StepState *st,
                             const StepTest &test, hipStream_t s)
{
    hipLaunchKernelGGL(step_state_kernel, dim3(1), dim3(kThreads), 0, s, parts, count, st, test);
    return hipGetLastError();
}

hipError_t launch_reduce_grouped(const ReduceItem *items, int n, hipStream_t s)
{
    if (n <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(reduce_grouped_kernel, dim3(n), dim3(kThreads), 0, s, items);
    return hipGetLastError();
}

hipError_t launch_scale(const float *X, int64_t ldx, float *Y, int64_t ldy, int64_t m, int64_t n,
                        double nrm, hipStream_t s)
{
    if (m == 0 || n == 0)
        return hipSuccess;
    hipLaunchKernelGGL(scale_kernel, grid2d(m, n), dim3(kThreads), 0, s, X, ldx, Y, ldy, m, n,
                       nrm);
    return hipGetLastError();
}

hipError_t launch_scale_by_norm(const float *X, int64_t ldx, float *Y, int64_t ldy, int64_t m,
                                int64_t n, const double *nrm2, hipStream_t s, const int *stop)
{
    if (m == 0 || n == 0)
        return hipSuccess;
    hipLaunchKernelGGL(scale_by_norm_kernel, grid2d(m, n), dim3(kThreads), 0, s, X, ldx, Y, ldy,
                       m, n, nrm2, stop);
    return hipGetLastError();
}

hipError_t launch_transpose_scale(const float *A, int64_t lda, float *X, int64_t ldx, int64_t n,
                                  int64_t m, double a, hipStream_t s)
{
    if (m == 0 || n == 0)
        return hipSuccess;
    const int64_t tn = (n + 31) / 32, tm = (m + 31) / 32;
    if (tn > 0x7fffffff)
        return hipErrorInvalidValue;
    const unsigned gy = (unsigned)std::min<int64_t>(tm, 65535);
    hipLaunchKernelGGL(transpose_scale_kernel, dim3((unsigned)tn, gy), dim3(32, 8), 0, s, A, lda,
                       X, ldx, n, m, a);
    return hipGetLastError();
}

hipError_t launch_zero(uint32_t *out, int64_t count, hipStream_t s)
{
    if (count <= 0)
        return hipSuccess;
    const int64_t g = std::min<int64_t>((count + kThreads - 1) / kThreads, 1024);
    hipLaunchKernelGGL(zero_kernel, dim3((unsigned)g), dim3(kThreads), 0, s, out, count);
    return hipGetLastError();
}

hipError_t launch_absmax(const float *X, int64_t ldx, int64_t m, int64_t n, int by_row,
                         uint32_t *out, hipStream_t s)
{
    if (m == 0 || n == 0)
        return launch_zero(out, by_row ? m : n, s);
    if (by_row) {
        const int64_t g = std::min<int64_t>((m + 3) / 4, 65535);
        hipLaunchKernelGGL(row_absmax_kernel, dim3((unsigned)g), dim3(kThreads), 0, s, X, ldx, m,
                           n, out);
        return hipGetLastError();
    }
    const hipError_t e = launch_zero(out, n, s);
    if (e != hipSuccess)
        return e;
    const int64_t gx = (n + kThreads - 1) / kThreads;
    if (gx > 0x7fffffff)
        return hipErrorInvalidValue;
    const int64_t gy = std::min<int64_t>((m + kMaxStrip - 1) / kMaxStrip, 65535);
    hipLaunchKernelGGL(col_absmax_kernel, dim3((unsigned)gx, (unsigned)gy), dim3(kThreads), 0, s,
                       X, ldx, m, n, out);
    return hipGetLastError();
}

hipError_t launch_scale_rows(const float *X, int64_t ldx, float *Y, int64_t ldy, int64_t m,
                             int64_t n, const uint32_t *mx, int unscale, hipStream_t s)
{
    if (m == 0 || n == 0)
        return hipSuccess;
    hipLaunchKernelGGL(scale_rows_kernel, grid2d(m, n), dim3(kThreads), 0, s, X, ldx, Y, ldy, m, n,
                       mx, unscale);
    return hipGetLastError();
}

hipError_t launch_uneven(const float *X, int64_t ldx, int64_t m, int64_t n, const double *nrm2,
                         uint32_t *counts, int *flag, StepState *st, hipStream_t s)
{
    const int64_t gx = (n + kThreads * kEvenGroups - 1) / (kThreads * kEvenGroups);
    if (gx > 0x7fffffff)
        return hipErrorInvalidValue;
    const int64_t strips = (m + kEvenRows - 1) / kEvenRows;
    const int64_t gy = std::min<int64_t>(strips, std::max<int64_t>(1, 2048 / gx));
    hipLaunchKernelGGL(small_count_kernel, dim3((unsigned)gx, (unsigned)gy), dim3(kThreads), 0, s,
                       X, ldx, m, n, nrm2, counts, flag, st);
    return hipGetLastError();
}

hipError_t launch_affine(const float *A, int64_t lda, float *Y, int64_t ldy, int64_t n,
                         double sc, double t, hipStream_t s)
{
    if (n == 0)
        return hipSuccess;
    hipLaunchKernelGGL(affine_kernel, grid2d(n, n), dim3(kThreads), 0, s, A, lda, Y, ldy, n, sc,
                       t);
    return hipGetLastError();
}

hipError_t launch_copy(const float *X, int64_t ldx, float *Y, int64_t ldy, int64_t m, int64_t n,
                       hipStream_t s)
{
    if (m == 0 || n == 0)
        return hipSuccess;
    hipLaunchKernelGGL(copy_kernel, grid2d(m, n), dim3(kThreads), 0, s, X, ldx, Y, ldy, m, n);
    return hipGetLastError();
}

hipError_t launch_symmetrize(float *H, int64_t ldh, int64_t n, hipStream_t s)
{
    if (n <= 1)
        return hipSuccess;
    const int64_t nb = (n + 31) / 32;
    hipLaunchKernelGGL(symmetrize_kernel, dim3((unsigned)nb, (unsigned)nb), dim3(32, 32), 0, s,
                       H, ldh, n);
    return hipGetLastError();
}

int splitk_update_num_partials() { return kSumsqBlocks; }

hipError_t launch_splitk_update_reduce(const float *parts, int splits, int64_t m, int64_t n,
                                       double alpha, double beta, const float *E, int64_t lde,
                                       float *out, int64_t ldo, double *step, hipStream_t s)
{
    if (m == 0 || n == 0)
        return hipSuccess;
    const bool vec = n % 4 == 0 && aligned16(parts) && aligned16(out) && ldo % 4 == 0 &&
                     (!E || (aligned16(E) && lde % 4 == 0));
    if (vec)
        hipLaunchKernelGGL(splitk_update_reduce_kernel<true>, dim3(kSumsqBlocks), dim3(kThreads),
                           0, s, parts, splits, m, n, alpha, beta, E, lde, out, ldo, step);
    else
        hipLaunchKernelGGL(splitk_update_reduce_kernel<false>, dim3(kSumsqBlocks), dim3(kThreads),
                           0, s, parts, splits, m, n, alpha, beta, E, lde, out, ldo, step);
    return hipGetLastError();
}

hipError_t launch_splitk_sym_reduce(const float *parts, int64_t stride, int splits, int64_t n,
                                    double alpha, double gamma, float *out, int64_t ldo,
                                    hipStream_t s)
{
    if (n == 0)
        return hipSuccess;
    const int64_t nb = (n + kSymTile - 1) / kSymTile;
    if (nb > 65535)
        return hipErrorInvalidValue;
    const bool vec = n % 4 == 0 && stride % 4 == 0 && ldo % 4 == 0 && aligned16(parts) &&
                     aligned16(out);
    if (vec)
        hipLaunchKernelGGL(splitk_sym_reduce_kernel<true>, dim3((unsigned)nb, (unsigned)nb),
                           dim3(256), 0, s, parts, stride, splits, n, alpha, gamma, out, ldo);
    else
        hipLaunchKernelGGL(splitk_sym_reduce_kernel<false>, dim3((unsigned)nb, (unsigned)nb),
                           dim3(256), 0, s, parts, stride, splits, n, alpha, gamma, out, ldo);
    return hipGetLastError();
}

}  // namespace la
