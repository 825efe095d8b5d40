// QR factorisation (section III.B of arXiv 2112.09017) on one GPU.
//
// la_tsqr -- Algorithm tsqr for an m x n panel, n <= 128.  The rows are cut
//            into blocks of at most 256 rows (each with at least n rows).
//            One workgroup factors one block by Householder reflections with
//            the block resident in registers (each wave owns whole columns),
//            writes its R and forms its Q in place.
//            The R factors are stacked and factored again the same way (a
//            256-row block holds 256 / n of them, so the tree reduces by that
//            factor per level rather than pairwise) until one R remains.  The
//            Q factors are then multiplied down the tree: every row of a
//            level's Q times the n x n slice of the level above that belongs
//            to its block.
// la_wy   -- eq. (Yamamoto): W = Q - [I; 0] and Y = W (I - Q_1)^-1, the
//            inverse by Gauss-Jordan elimination with partial pivoting in FP64
//            in one workgroup, then one row-parallel product.
// la_caqr -- Algorithm caqr (right-looking): per panel of b columns, la_tsqr,
//            la_wy, A_l <- [R; 0] and A_r <- A_r - Y (W^T A_r) as two GEMM
//            launches (the first split along its long K = rows dimension),
//            with one panel of look-ahead: the next panel's columns are
//            updated on the caller's stream and the rest on a second stream
//            (the update is the short-K kernel of qr_update.hip); optionally
//            Q = Q_f(0) ... Q_f(last) [I; 0] afterwards.  AUTO runs
//            the products as 6xBF16: the update's K is only the panel width,
//            too short for the 3xBF16 products' per-term error (about 2^-16
//            relative) to average out.
#include <hip/hip_runtime.h>

#include <math.h>
#include <string.h>

#include <algorithm>
#include <type_traits>

#include "la_internal.h"

namespace la {
namespace {

constexpr int kRows = 256;        // rows of one local factorisation
constexpr int kMaxPanel = 128;
constexpr int kRowmulRows = 128;   // rows of a block per workgroup of rowmul_kernel
constexpr int kMaxLevels = 40;
constexpr int kMaxSplits = 16;
// The next panel's product W^T A_next (b x b output, K = the panel's rows) is
// on the critical path of every panel: it takes up to 64 slices of at least
// 256 rows, so its launch is short, where the other split products (wide
// outputs) keep slices of at least 1024 rows.
constexpr int kMaxSplitsNext = 64;
constexpr int64_t kMinSliceNext = 256;
constexpr int64_t kMinSlice = 1024;
// A Gauss-Jordan pivot of I - Q_1 below this magnitude is reported as the
// breakdown of eq. (Yamamoto): Y would carry errors of order u / pivot.
constexpr double kPivotFloor = 1.0 / 65536.0;

// Row partition of a tall matrix into blocks of 256 rows.  When the last
// block would hold fewer than nc rows, the last two blocks share their rows
// evenly (at least 128 >= nc each), so every block has at least nc rows.
struct Part {
    int64_t rows;
    int64_t last_start;
    int nb;
};

__host__ __device__ inline Part make_part(int64_t rows, int nc)
{
    Part p;
    p.rows = rows;
    const int64_t nb = (rows + kRows - 1) / kRows;
    p.nb = (int)nb;
    const int64_t rem = rows - kRows * (nb - 1);
    p.last_start = (nb > 1 && rem < nc) ? kRows * (nb - 2) + (kRows + rem) / 2 : kRows * (nb - 1);
    return p;
}

__host__ __device__ inline int64_t part_start(const Part &p, int64_t i)
{
    if (i >= p.nb)
        return p.rows;
    return i == p.nb - 1 ? p.last_start : kRows * i;
}

// ---------------------------------------------------------------- kernels

// Sum over the L consecutive lanes of an aligned lane group (L = 4 or 8),
// returned in every lane of the group, by DPP moves within the group
// (lane ^ 1, lane ^ 2, then the mirror of each half-row of 8).
template <int CTRL>
__device__ inline float dpp_f32(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ inline double dpp_f64(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}
template <int L, typename T>
__device__ inline T group_sum(T v)
{
    static_assert(L == 4 || L == 8, "lane groups of 4 or 8");
    if constexpr (sizeof(T) == 4) {
        v += dpp_f32<0xB1>(v);        // quad_perm [1, 0, 3, 2]
        v += dpp_f32<0x4E>(v);        // quad_perm [2, 3, 0, 1]
        if constexpr (L == 8)
            v += dpp_f32<0x141>(v);   // row_half_mirror
    } else {
        v += dpp_f64<0xB1>(v);
        v += dpp_f64<0x4E>(v);
        if constexpr (L == 8)
            v += dpp_f64<0x141>(v);
    }
    return v;
}

// Sum over the 64 lanes of a wave, returned as a wave-uniform value: DPP
// within rows of 16 lanes (lane ^ 1, lane ^ 2, half-row and row mirrors),
// then row 0 into row 1 and row 2 into row 3 (row_bcast:15), rows 0 + 1 into
// rows 2 and 3 (row_bcast:31); lane 63 ends with the total.
template <int CTRL, int ROWS>
__device__ inline float bcast_f32(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xF, false));
}
template <int CTRL, int ROWS>
__device__ inline double bcast_f64(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xF, false);
    return __hiloint2double(hi, lo);
}
__device__ inline float wave_sum(float v)
{
    v += dpp_f32<0xB1>(v);
    v += dpp_f32<0x4E>(v);
    v += dpp_f32<0x141>(v);          // row_half_mirror
    v += dpp_f32<0x140>(v);          // row_mirror: each row of 16 holds its sum
    v += bcast_f32<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
    v += bcast_f32<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
// Maximum over the 64 lanes of a wave of an unsigned key, wave-uniform: the
// DPP steps of wave_sum with max in place of the sum (keys are >= 0, so the
// zeros that the masked broadcast rows read change nothing).
__device__ inline unsigned wave_max(unsigned v)
{
    auto mx = [](unsigned a, unsigned b) { return a > b ? a : b; };
    v = mx(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true));
    v = mx(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true));
    v = mx(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true));
    v = mx(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true));
    v = mx(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, true));
    v = mx(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, true));
    return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}

// Sums over the 64 lanes of a wave of N values per lane, halving the number of
// values held at each of the first steps: v_permlane32_swap_b32 and
// v_permlane16_swap_b32 put the halves of two values that belong together side by
// side, so one add serves both (a value without a partner is paired with itself).
// N = 8 takes 21 instructions against the 48 adds of eight wave_sum.  On return
// out[i] is the wave-uniform total of v[i] times scale.
template <int N>
__device__ __forceinline__ void wave_sums(const float (&v)[N], float scale, float (&out)[N])
{
    constexpr int N1 = (N + 1) / 2, N2 = (N1 + 1) / 2;
    static_assert(N >= 1 && N2 <= 2, "at most eight values");
    float a[N1], b[N2];
#pragma unroll
    for (int i = 0; i < N1; ++i) {
        const int lo = 2 * i, hi = 2 * i + 1 < N ? 2 * i + 1 : lo;
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[lo]),
                                                        __float_as_uint(v[hi]), false, false);
        a[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
#pragma unroll
    for (int i = 0; i < N2; ++i) {
        const int lo = 2 * i, hi = 2 * i + 1 < N1 ? 2 * i + 1 : lo;
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a[lo]),
                                                        __float_as_uint(a[hi]), false, false);
        b[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    float c = b[0];
    if constexpr (N2 == 1) {
        c += dpp_f32<0x128>(c);          // row_ror:8
    } else {
        const bool up = threadIdx.x & 8;   // this half of the row takes b[1]
        const float keep = up ? b[1] : b[0], send = up ? b[0] : b[1];
        c = keep + dpp_f32<0x128>(send);
    }
    c += dpp_f32<0xB1>(c);
    c += dpp_f32<0x4E>(c);
    c += dpp_f32<0x141>(c);              // row_half_mirror
    c *= scale;
#pragma unroll
    for (int i = 0; i < N; ++i)
        out[i] = __int_as_float(__builtin_amdgcn_readlane(
            __float_as_int(c), 32 * (i & 1) + 16 * ((i >> 1) & 1) + 8 * ((i >> 2) & 1)));
}
__device__ inline double wave_sum(double v)
{
    v += dpp_f64<0xB1>(v);
    v += dpp_f64<0x4E>(v);
    v += dpp_f64<0x141>(v);
    v += dpp_f64<0x140>(v);
    v += bcast_f64<0x142, 0xA>(v);
    v += bcast_f64<0x143, 0xC>(v);
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
    return __hiloint2double(hi, lo);
}

// Q = H_0 ... H_{nc-1} [I; 0] of a block's 64-column reflector set, in
// compact WY form: H_0 ... H_{nc-1} = I - U T U^T with U = [u_0 ... u_{nc-1}]
// (u_j zero above row j) and T upper triangular, T^-1 = diag(1/kappa) +
// N, N the strict upper part of S = U^T U; T = (I + diag(kappa) N)^-1
// diag(kappa) needs no division (a column without a reflection, kappa = 0,
// gives a zero row and column of T).  So Q = [I; 0] - U Z with Z = T U_top^T
// (U_top: the first 64 rows of U).  With T in 32 x 32 blocks, T_LH =
// -T_LL N_LH T_HH (two reflector sets joined).
//   1. each lane writes its 32 entries of U (zero above the diagonal, u_j on
//      it, the stored x below) to LDS, row r at r * 64, column j at slot
//      j ^ (r & 31), so both a row and a column of 32 are conflict-free;
//   2. three waves form the blocks (0,0), (0,1), (1,1) of S on the matrix
//      cores (v_mfma_f32_32x32x2f32, K = the block's rows) and write S
//      transposed (S[i][k] at k * 64 + i);
//   3. wave 0 forms T_LL and T_HH (lane = column), 32 steps each, side by
//      side in the two halves of the wave;
//   4. wave 1 forms T_LH on the matrix cores;
//   5. four waves form Z = T U_top^T on the matrix cores;
//   6. all eight waves form [I; 0] - U Z, 16 blocks of 32 x 32, on the matrix
//      cores and write it to Q (rows of this block; ldq).
// write_u(Us): stores this thread's entries of U (step 1), given the values it
// read before the call (the LDS space is reused); s_kap: kappa_j (read before the
// reuse); lds: the kernel's 80 KiB buffer.
template <class WriteU>
__device__ __forceinline__ void form_q64(WriteU write_u, int nc, int lane, int w, int rows,
                                         const float *s_kap, float *lds, float *Qb, int64_t ldq)
{
    typedef float f32x16_t __attribute__((ext_vector_type(16)));
    const float kapl = lane < nc ? s_kap[lane] : 0.0f;
    __syncthreads();   // every wave is past the reflections and has its u_j / kappa
    float *Us = lds;
    float *SZ = lds + kRows * 64;
    write_u(Us);
    __syncthreads();
    const int li = lane & 31, hk = lane >> 5;
    if (w < 3) {
        const int bi = w == 2 ? 1 : 0, bj = w == 0 ? 0 : 1;
        f32x16_t acc = {};
        // 16 rows per step, the loads ahead of the products (U is zero below
        // the block's rows, so the padding adds exact zeros)
        const int kend = (rows + 15) & ~15;
        for (int k0 = 0; k0 < kend; k0 += 16) {
            float a[8], b[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int r = k0 + 2 * q + hk;
                a[q] = Us[r * 64 + ((bi * 32 + li) ^ (r & 31))];
                b[q] = Us[r * 64 + ((bj * 32 + li) ^ (r & 31))];
            }
#pragma unroll
            for (int q = 0; q < 8; ++q)
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q], b[q], acc, 0, 0, 0);
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int i = bi * 32 + 8 * (e >> 2) + 4 * hk + (e & 3), j = bj * 32 + li;
            SZ[j * 64 + i] = acc[e];
        }
    }
    __syncthreads();
    // 3. T_LL and T_HH, the diagonal 32 x 32 blocks of T, in one wave: lane
    // c of half h solves (I + diag(kappa_h) N_hh) t = kappa_c e_c from the
    // last row up without a division (t_k *= kappa_k once final, then
    // t_i -= N[i][k] t_k for i < k), then stores row-major, column slot
    // c ^ r, over the S block it has read
    if (w == 0) {
        const int hf = lane >> 5, c = lane & 31;
        float *sb = SZ + hf * (32 * 64 + 32);   // S[32 hf + i][32 hf + k] at sb[k * 64 + i]
        float z[32];
#pragma unroll
        for (int i = 0; i < 32; ++i)
            z[i] = i == c ? 1.0f : 0.0f;
#pragma unroll
        for (int k = 31; k >= 0; --k) {
            const float klo = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(kapl), k));
            const float khi =
                __int_as_float(__builtin_amdgcn_readlane(__float_as_int(kapl), 32 + k));
            z[k] *= hf ? khi : klo;
            const float *sk = sb + k * 64;
#pragma unroll
            for (int i = 0; i < (k & ~3); i += 4) {
                const float4 sv = *reinterpret_cast<const float4 *>(sk + i);
                z[i] = fmaf(-sv.x, z[k], z[i]);
                z[i + 1] = fmaf(-sv.y, z[k], z[i + 1]);
                z[i + 2] = fmaf(-sv.z, z[k], z[i + 2]);
                z[i + 3] = fmaf(-sv.w, z[k], z[i + 3]);
            }
#pragma unroll
            for (int i = k & ~3; i < k; ++i)
                z[i] = fmaf(-sk[i], z[k], z[i]);
        }
        // every lane's reads of the block before any lane's stores over it
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
#pragma unroll
        for (int r = 0; r < 32; ++r)
            sb[r * 64 + (c ^ r)] = z[r];           // T_hh[r][c]
    }
    __syncthreads();
    // 4. T_LH = -T_LL (N_LH T_HH) in one wave on the matrix cores: P =
    // N_LH T_HH into the unused lower-left block (P[i][j] at i * 64 + 32 + j),
    // then -T_LL P over N_LH (T_LH[i][j] at (32 + j) * 64 + i)
    if (w == 1) {
        f32x16_t acc = {};
#pragma unroll
        for (int k0 = 0; k0 < 32; k0 += 16) {
            float a[8], b[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int kk = k0 + 2 * q + hk;
                a[q] = SZ[(32 + kk) * 64 + li];                 // N_LH[li][kk]
                b[q] = SZ[(32 + kk) * 64 + 32 + (li ^ kk)];     // T_HH[kk][li]
            }
#pragma unroll
            for (int q = 0; q < 8; ++q)
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q], b[q], acc, 0, 0, 0);
        }
#pragma unroll
        for (int e = 0; e < 16; ++e)
            SZ[(8 * (e >> 2) + 4 * hk + (e & 3)) * 64 + 32 + li] = acc[e];
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        f32x16_t acc2 = {};
#pragma unroll
        for (int k0 = 0; k0 < 32; k0 += 16) {
            float a[8], b[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int kk = k0 + 2 * q + hk;
                a[q] = SZ[li * 64 + (kk ^ li)];                 // T_LL[li][kk]
                b[q] = SZ[kk * 64 + 32 + li];                   // P[kk][li]
            }
#pragma unroll
            for (int q = 0; q < 8; ++q)
                acc2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q], b[q], acc2, 0, 0, 0);
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
#pragma unroll
        for (int e = 0; e < 16; ++e)
            SZ[(32 + li) * 64 + 8 * (e >> 2) + 4 * hk + (e & 3)] = -acc2[e];
    }
    __syncthreads();
    // 5. Z = T U_top^T, four 32 x 32 blocks on four waves (T_HL = 0), then Z
    // row-major over T
    f32x16_t zacc = {};
    if (w < 4) {
        const int bi = w >> 1, col = (w & 1) * 32 + li;
#pragma unroll
        for (int k0 = 0; k0 < 64; k0 += 16) {
            if (k0 < 32 * bi)
                continue;
            float a[8], b[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int kk = k0 + 2 * q + hk;
                if (bi == 1)
                    a[q] = SZ[(32 + li) * 64 + 32 + ((kk - 32) ^ li)];   // T_HH[li][kk - 32]
                else if (k0 < 32)
                    a[q] = SZ[li * 64 + (kk ^ li)];                       // T_LL[li][kk]
                else
                    a[q] = SZ[kk * 64 + li];                              // T_LH[li][kk - 32]
                b[q] = Us[col * 64 + (kk ^ (col & 31))];                  // U[col][kk]
            }
#pragma unroll
            for (int q = 0; q < 8; ++q)
                zacc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q], b[q], zacc, 0, 0, 0);
        }
    }
    __syncthreads();
    if (w < 4) {
        const int bi = w >> 1, col = (w & 1) * 32 + li;
#pragma unroll
        for (int e = 0; e < 16; ++e)
            SZ[(32 * bi + 8 * (e >> 2) + 4 * hk + (e & 3)) * 64 + col] = zacc[e];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int bid = 2 * w + q, br = bid >> 1, bc = bid & 1;
        if (br * 32 >= rows)
            continue;
        f32x16_t acc = {};
        // 16 columns of U per step, the loads ahead of the products (U's
        // columns and Z's rows from nc on are zero)
        const int kend = (nc + 15) & ~15;
        for (int k0 = 0; k0 < kend; k0 += 16) {
            float a[8], b[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int kk = k0 + 2 * q + hk, r = br * 32 + li;
                a[q] = Us[r * 64 + (kk ^ (r & 31))];
                b[q] = SZ[kk * 64 + bc * 32 + li];
            }
#pragma unroll
            for (int q = 0; q < 8; ++q)
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q], b[q], acc, 0, 0, 0);
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int rr = br * 32 + 8 * (e >> 2) + 4 * hk + (e & 3), cc = bc * 32 + li;
            if (rr < rows && cc < nc)
                Qb[(int64_t)rr * ldq + cc] = (rr == cc ? 1.0f : 0.0f) - acc[e];
        }
    }
}

// Householder QR of one row block (rows x nc, rows <= 256, nc <= NC) per
// workgroup of NC / 8 waves, the block in registers with the rows across the
// lanes: lane l holds rows 4 l .. 4 l + 3 of its wave's 8 columns (wave w:
// columns 8 w .. 8 w + 7).  A column vector such as u_j is then spread over
// the lanes of every wave alike, so the wave that forms a reflection keeps
// u_j in registers and a column dot product is a sum over the wave
// (wave_sum: DPP and one readlane).
//
// Reflection j uses u = x - beta e_j (x = column j from row j down,
// beta = -sign(x_j) ||x||) unscaled, H_j = I - kappa u u^T,
// kappa = 1 / (beta (beta - x_j)); ||x||^2, beta and kappa in FP32, or in
// FP64 (squares exact for FP32 entries) when the FP32 sum of squares leaves
// [2^-96, 2^96] (zero or non-finite included).  Each wave applies the
// reflections in order: those of the waves to its left as they are
// published (u_j from LDS, then u_j^T x_c and x_c -= kappa (u^T x_c) u for its
// 8 columns), then its own, each formed from its column, published and
// applied at once to the wave's later columns.  A reflection is published
// by a workgroup-scope release store of the count of published reflections
// after u_j, kappa_j and beta_j are in LDS; a wave waits for reflection j
// with acquire loads of that count.  No barrier until all reflections are
// done: a wave starts its own columns once it has applied the last
// reflection of the wave to its left.  Every wait is for a reflection that a
// wave to its left publishes without waiting on this one; it is bounded all
// the same, and a wait that runs out marks the block's R with NaN instead of
// hanging.  Column j keeps x below the diagonal and the pivot x_j on it.
// The chain of 64 reflections bounds it (256 x 64: 44 us with a wave_sum per
// column, the library's sqrt and divide and one poll per reflection, 36 us now;
// leaves of 131072 rows, two blocks per CU, 49 -> 40 us).
// R (row block blk of R, ld ldr) is then written from the registers, and
// Q = H_0 ... H_{nc-1} [I; 0] is formed in compact WY form (form_q64) and
// written to Q (ldq); X may equal Q.  SPLIT: instead the reflectors U go to Q
// and their kappa to kap (64 per block), for qr_form64_kernel: the next level of
// the TSQR tree needs R only, so the forming of Q (22 of a block's 59 us) leaves
// the chain of levels.  NC = 128 (64 < nc) is always split, for qr_form128_kernel,
// and has its kappa in U's zero upper triangle: kappa_c at (0, c), kappa_0 at (1, 2).
template <int NC, bool SPLIT>
__global__ __launch_bounds__(NC * 8) void qr_block_kernel(const float *X, int64_t ldx, Part part,
                                                         int nc, float *Q, int64_t ldq, float *R,
                                                         int64_t ldr, float *kap)
{
    constexpr int CPW = 8;              // columns per wave
    constexpr int RPL = kRows / 64;     // rows per lane
    // LDS: u_j of every reflection (each stays until every wave has applied
    // it), u_j's pivot entry, kappa, beta and the count of published
    // reflections; the same space then holds U and S / Z of the compact WY
    // form (80 KiB in all, so two workgroups share a CU)
    constexpr int kLdsF = SPLIT ? NC * kRows + 3 * NC + 4 : kRows * 64 + 64 * 64;
    static_assert(NC == 64 || SPLIT, "more than 64 columns: qr_form128_kernel forms Q");
    static_assert(NC * kRows + 3 * NC + 1 <= kLdsF, "reflection buffers fit the WY space");
    __shared__ __attribute__((aligned(16))) float lds[kLdsF];
    float(*ubuf)[kRows] = reinterpret_cast<float(*)[kRows]>(lds);
    float *s_u0 = lds + NC * kRows, *s_kap = s_u0 + NC, *s_beta = s_kap + NC;
    int *s_pub = reinterpret_cast<int *>(s_beta + NC);

    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int rlo = lane * RPL;
    const int64_t blk = blockIdx.x;
    const int64_t r0 = part_start(part, blk);
    const int rows = (int)(part_start(part, blk + 1) - r0);
    nc = __builtin_amdgcn_readfirstlane(nc);
    const int own = __builtin_amdgcn_readfirstlane(w * CPW);   // the wave's first column

    float f[CPW][RPL];
    const bool vec = own + CPW <= nc && (ldx & 3) == 0 && ((uintptr_t)X & 15) == 0;
#pragma unroll
    for (int i = 0; i < RPL; ++i) {
        const int r = rlo + i;
        if (vec) {
            float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f), b = a;
            if (r < rows) {
                const float *xr = X + (r0 + r) * ldx + own;
                a = *(const float4 *)xr;
                b = *(const float4 *)(xr + 4);
            }
            f[0][i] = a.x, f[1][i] = a.y, f[2][i] = a.z, f[3][i] = a.w;
            f[4][i] = b.x, f[5][i] = b.y, f[6][i] = b.z, f[7][i] = b.w;
        } else {
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc)
                f[cc][i] = (own + cc < nc && r < rows) ? X[(r0 + r) * ldx + own + cc] : 0.0f;
        }
    }

    // x_c -= kappa (u^T x_c) u for the wave's columns FIRST .. CPW - 1
    auto apply = [&](auto first, const float (&u)[RPL], float kap, auto &&between) {
        constexpr int F = decltype(first)::value;
        if constexpr (F < CPW) {
            float d[CPW - F], sc[CPW - F];
#pragma unroll
            for (int c = 0; c < CPW - F; ++c) {
                d[c] = 0.0f;
#pragma unroll
                for (int i = 0; i < RPL; ++i)
                    d[c] = fmaf(u[i], f[F + c][i], d[c]);
            }
            wave_sums(d, kap, sc);
            between();
#pragma unroll
            for (int c = 0; c < CPW - F; ++c)
#pragma unroll
                for (int i = 0; i < RPL; ++i)
                    f[F + c][i] = fmaf(-sc[c], u[i], f[F + c][i]);
        } else {
            between();
        }
    };

    if (t == 0)
        *s_pub = 0;
    __syncthreads();
    bool timed_out = false;
    if (own < nc) {
        // the reflections of the waves to the left, as they are published; the
        // next one is read ahead where it is already there.  The wave whose
        // turn is next goes ahead of the others on its SIMD.
        int have = 0;
        float4 uv, un;
        float kv, kn;
        bool ahead = false;
        for (int jv = 0; jv < own; ++jv) {
            const int j = __builtin_amdgcn_readfirstlane(jv);
            if (j == own - CPW)
                __builtin_amdgcn_s_setprio(2);
            if (!ahead) {
                int spins = 0;
                while ((have = __builtin_amdgcn_readfirstlane(__hip_atomic_load(
                            s_pub, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP))) <= j) {
                    if (j < own - CPW)
                        __builtin_amdgcn_s_sleep(1);
                    if (++spins > (1 << 22)) {
                        timed_out = true;
                        break;
                    }
                }
                uv = *(const float4 *)&ubuf[j][rlo];
                kv = s_kap[j];
            }
            ahead = j + 1 < own && j + 1 < have;
            if (ahead) {
                un = *(const float4 *)&ubuf[j + 1][rlo];
                kn = s_kap[j + 1];
            }
            const float u[RPL] = {uv.x, uv.y, uv.z, uv.w};
            apply(std::integral_constant<int, 0>{}, u, kv, [] {});
            uv = un;
            kv = kn;
        }
        __builtin_amdgcn_s_setprio(3);
        // this wave's reflections
        auto reflection = [&](auto cjc) {
            constexpr int cj = decltype(cjc)::value;
            const int j = own + cj;
            if (j >= nc)
                return;
            float o[RPL], s4 = 0.0f;
#pragma unroll
            for (int i = 0; i < RPL; ++i) {
                o[i] = rlo + i < j ? 0.0f : f[cj][i];
                s4 = fmaf(o[i], o[i], s4);
            }
            const float ss = wave_sum(s4);
            // x_j: row j is entry j % 4 (= cj % 4) of lane j / 4
            const float x0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(f[cj][cj & 3]),
                                                                      j >> 2));
            float u0 = 0.0f, kap = 0.0f, beta = 0.0f;   // a zero column needs no reflection
            if (ss >= 0x1p-96f && ss <= 0x1p96f) {
                // sqrt and 1 / x by one Newton step from the hardware's estimates
                // (within one ulp): well inside the normal range here, and a
                // third of the chain of the library's
                const float y = __builtin_amdgcn_rsqf(ss), g = ss * y;
                const float nrm = fmaf(0.5f * y, fmaf(-g, g, ss), g);
                beta = x0 >= 0.0f ? -nrm : nrm;
                u0 = x0 - beta;
                const float q = -beta * u0, r = __builtin_amdgcn_rcpf(q);
                kap = fmaf(r, fmaf(-q, r, 1.0f), r);
            } else {
                double sd = 0.0;
#pragma unroll
                for (int i = 0; i < RPL; ++i)
                    sd = fma((double)o[i], (double)o[i], sd);
                const double nrm = sqrt(wave_sum(sd));
                if (nrm > 0.0) {
                    const double bt = x0 >= 0.0f ? -nrm : nrm;
                    u0 = (float)((double)x0 - bt);
                    kap = (float)(1.0 / (bt * (bt - (double)x0)));
                    beta = (float)bt;
                }
            }
            if (rlo + (cj & 3) == j)
                o[cj & 3] = u0;
            *(float4 *)&ubuf[j][rlo] = make_float4(o[0], o[1], o[2], o[3]);
            if (lane == 0) {
                s_u0[j] = u0;
                s_kap[j] = kap;
                s_beta[j] = beta;
            }
            // published once the sums are under way: the stores have then landed
            apply(std::integral_constant<int, cj + 1>{}, o, kap, [&] {
                __hip_atomic_store(s_pub, j + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
            });
        };
        static_assert(CPW == 8, "one call per column");
        reflection(std::integral_constant<int, 0>{});
        reflection(std::integral_constant<int, 1>{});
        reflection(std::integral_constant<int, 2>{});
        reflection(std::integral_constant<int, 3>{});
        reflection(std::integral_constant<int, 4>{});
        reflection(std::integral_constant<int, 5>{});
        reflection(std::integral_constant<int, 6>{});
        reflection(std::integral_constant<int, 7>{});
        __builtin_amdgcn_s_setprio(0);
    }
    __syncthreads();
    if (timed_out)
        f[0][0] = NAN;

    float *Rb = R + blk * nc * ldr;
#pragma unroll
    for (int cc = 0; cc < CPW; ++cc) {
        const int c = own + cc;
#pragma unroll
        for (int i = 0; i < RPL; ++i) {
            const int rr = rlo + i;
            if (c < nc && rr < nc)
                Rb[(int64_t)rr * ldr + c] = c > rr ? f[cc][i] : (c == rr ? s_beta[rr] : 0.0f);
        }
    }

    float u0c[CPW];
#pragma unroll
    for (int cc = 0; cc < CPW; ++cc)
        u0c[cc] = own + cc < nc ? s_u0[own + cc] : 0.0f;
    if constexpr (SPLIT) {
        if (NC == 64 && t < nc)
            kap[blk * 64 + t] = s_kap[t];
        const bool vecq = own + CPW <= nc && (ldq & 3) == 0 && ((uintptr_t)Q & 15) == 0;
#pragma unroll
        for (int i = 0; i < RPL; ++i) {
            const int r = rlo + i;
            if (r >= rows)
                continue;
            float v[CPW];
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc) {
                const int c = own + cc;
                v[cc] = r < c ? 0.0f : (r == c ? u0c[cc] : f[cc][i]);
                if (NC == 128 && c < nc) {
                    if (r == 0 && c > 0)
                        v[cc] = s_kap[c];
                    if (r == 1 && c == 2)
                        v[cc] = s_kap[0];
                }
            }
            float *qr = Q + (r0 + r) * ldq + own;
            if (vecq) {
                *(float4 *)qr = make_float4(v[0], v[1], v[2], v[3]);
                *(float4 *)(qr + 4) = make_float4(v[4], v[5], v[6], v[7]);
            } else {
#pragma unroll
                for (int cc = 0; cc < CPW; ++cc)
                    if (own + cc < nc)
                        qr[cc] = v[cc];
            }
        }
    } else {
        form_q64(
            [&](float *Us) {
#pragma unroll
                for (int cc = 0; cc < CPW; ++cc) {
                    const int c = own + cc;
#pragma unroll
                    for (int i = 0; i < RPL; ++i) {
                        const int r = rlo + i;
                        const float v = (c >= nc || r < c) ? 0.0f : (r == c ? u0c[cc] : f[cc][i]);
                        Us[r * 64 + (c ^ (r & 31))] = v;
                    }
                }
            },
            nc, lane, w, rows, s_kap, lds, Q + r0 * ldq, ldq);
    }
}

// Q of the blocks of several levels of a TSQR tree, in place of the reflectors
// that qr_block_kernel<64, true> left: one workgroup per block, every level's in one
// launch (the same products as the unsplit kernel's, bit for bit).
constexpr int kFormLevels = 24;
struct FormArgs {
    int levels, nc;
    int first[kFormLevels + 1];   // first workgroup of each level
    float *Q[kFormLevels];
    const float *kap[kFormLevels];
    int64_t ldq[kFormLevels];
    Part part[kFormLevels];
};
__global__ __launch_bounds__(512) void qr_form64_kernel(FormArgs a)
{
    constexpr int CPW = 8, RPL = kRows / 64;
    __shared__ __attribute__((aligned(16))) float lds[kRows * 64 + 64 * 64];
    int l = 0;
    while (l + 1 < a.levels && (int)blockIdx.x >= a.first[l + 1])
        ++l;
    const int64_t blk = (int)blockIdx.x - a.first[l];
    const int64_t ldq = a.ldq[l];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int rlo = lane * RPL;
    const int64_t r0 = part_start(a.part[l], blk);
    const int rows = (int)(part_start(a.part[l], blk + 1) - r0);
    const int nc = a.nc;
    const int own = __builtin_amdgcn_readfirstlane(w * CPW);
    float *Qb = a.Q[l] + r0 * ldq;
    float f[CPW][RPL];
    const bool vec = own + CPW <= nc && (ldq & 3) == 0 && ((uintptr_t)a.Q[l] & 15) == 0;
#pragma unroll
    for (int i = 0; i < RPL; ++i) {
        const int r = rlo + i;
        const float *qr = Qb + (int64_t)r * ldq + own;
        if (vec) {
            float4 x = make_float4(0.0f, 0.0f, 0.0f, 0.0f), y = x;
            if (r < rows) {
                x = *(const float4 *)qr;
                y = *(const float4 *)(qr + 4);
            }
            f[0][i] = x.x, f[1][i] = x.y, f[2][i] = x.z, f[3][i] = x.w;
            f[4][i] = y.x, f[5][i] = y.y, f[6][i] = y.z, f[7][i] = y.w;
        } else {
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc)
                f[cc][i] = (own + cc < nc && r < rows) ? qr[cc] : 0.0f;
        }
    }
    form_q64(
        [&](float *Us) {
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc)
#pragma unroll
                for (int i = 0; i < RPL; ++i) {
                    const int r = rlo + i;
                    Us[r * 64 + ((own + cc) ^ (r & 31))] = f[cc][i];
                }
        },
        nc, lane, w, rows, a.kap[l] + blk * 64, lds, Qb, ldq);
}

// The same for 64 < nc <= 128, in place of the U and kappa that
// qr_block_kernel<128, true> left: Q = H_0 ... H_{nc-1} [I; 0], last reflection
// first (column j becomes H_j e_j once the columns to its right hold
// H_{j+1} ... e_c), one barrier per reflection.  1024 threads; wave w owns columns
// 8 w .. 8 w + 7, a column is held by L = 8 consecutive lanes with RPL = 32
// consecutive rows each, and its dot products reduce inside the wave.  Off the
// chain of levels it costs its throughput only, one workgroup per CU (131072 x 128:
// 5.0 -> 1.8 ms, 236482 x 76 3.0 -> 1.4, against one kernel that factored and
// formed a block in 300 us a level).
__global__ __launch_bounds__(1024) void qr_form128_kernel(FormArgs a)
{
    constexpr int B = 128;
    constexpr int CPW = 8;              // columns per wave
    constexpr int L = 64 / CPW;         // lanes per column
    constexpr int RPL = kRows / L;      // rows per lane
    // the two u buffers (alternating reflections) and kappa
    __shared__ __attribute__((aligned(16))) float ubuf[2][kRows];
    __shared__ float s_kap[B];
    int l = 0;
    while (l + 1 < a.levels && (int)blockIdx.x >= a.first[l + 1])
        ++l;
    const int64_t blk = (int)blockIdx.x - a.first[l];
    const int64_t ldq = a.ldq[l];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int c = w * CPW + lane / L;
    const int rlo = (lane % L) * RPL;
    const int64_t r0 = part_start(a.part[l], blk);
    const int rows = (int)(part_start(a.part[l], blk + 1) - r0);
    const int nc = __builtin_amdgcn_readfirstlane(a.nc);
    const bool col = c < nc;
    float *Qb = a.Q[l] + r0 * ldq;

    // column c of U, zero above its diagonal (where the kappa are)
    float f[RPL], u[RPL];
#pragma unroll
    for (int i = 0; i < RPL; ++i) {
        const int r = rlo + i;
        f[i] = (col && r < rows && r >= c) ? Qb[(int64_t)r * ldq + c] : 0.0f;
    }
    if (t < nc)
        s_kap[t] = t ? Qb[t] : Qb[ldq + 2];

    // owners of column jn: its reflector to ubuf[jn & 1]
    auto publish = [&](int jn) {
        float *ub = ubuf[jn & 1];
#pragma unroll
        for (int i = 0; i < RPL; i += 4)
            *(float4 *)&ub[rlo + i] = make_float4(f[i], f[i + 1], f[i + 2], f[i + 3]);
    };
    auto axpy_u = [&](float sc) {
#pragma unroll
        for (int i = 0; i < RPL; ++i)
            f[i] = fmaf(-sc, u[i], f[i]);
    };
    if (c == nc - 1)
        publish(nc - 1);
    __syncthreads();
    for (int jv = nc - 1; jv >= 0; --jv) {
        const int j = __builtin_amdgcn_readfirstlane(jv);
        const float *ub = ubuf[j & 1];
        const float kap = s_kap[j], u0 = ub[j];
        float d4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int i = 0; i < RPL; i += 4) {
            const float4 uv = *(const float4 *)&ub[rlo + i];
            const float ua[4] = {uv.x, uv.y, uv.z, uv.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                u[i + e] = ua[e];
                d4[e] = fmaf(ua[e], f[i + e], d4[e]);
            }
        }
        const float d = group_sum<L>((d4[0] + d4[1]) + (d4[2] + d4[3]));
        if (col && c > j) {
            axpy_u(kap * d);
        } else if (c == j) {
            // column j = H_j e_j = e_j - kappa u_j u (u is zero above row j)
            const float s2 = kap * u0;
#pragma unroll
            for (int i = 0; i < RPL; ++i)
                f[i] = rlo + i == j ? 1.0f : 0.0f;
            axpy_u(s2);
        }
        if (c == j - 1)
            publish(j - 1);
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < RPL; ++i)
        if (col && rlo + i < rows)
            Qb[(int64_t)(rlo + i) * ldq + c] = f[i];
}

// out[r, :] = (in[r, :] - sub [r < nc] e_r^T) M_b for every row r < part.rows,
// with M_b = Mb + b * nc * nc (nc x nc, ld nc) for the partition block b
// holding row r, or M_0 for every row when single; wout (optional) receives
// in[r, :] - sub e_r^T.  Workgroup (b, y) takes rows 128 y .. 128 y + 127 of
// block b, each wave 32 of them on the matrix cores (v_mfma_f32_32x32x2f32): lane
// l holds half of row l & 31 (k from B / 2 (l >> 5) on; step q takes k = q and
// B / 2 + q, in four sums, at B = 128 two, that shorten the chain of
// roundings: with one, A - Q R came out 1.5% larger than from the vector units); M_b
// is in LDS.  Latency bound on the tree's upper levels and in
// CAQR's panels, HBM bound on the leaves (64 columns, 131072 rows, tree of six
// levels: 20 us a level on the vector units with an index division per element,
// 8.7 us now; CAQR's panels of 6144 rows 12 -> 7.3 us); at most 32 columns take
// B = 32, whose rows are not padded to 64 (la_wy of 1000000 x 32:
// 334 -> 133 us).  out may equal in: a
// wave reads its rows whole before it writes any.
template <int B>
__global__ __launch_bounds__(256) void rowmul_kernel(const float *in, int64_t ldi, Part part,
                                                     int single, int nc,
                                                     const float *__restrict__ Mb, float *out,
                                                     int64_t ldo, float *wout, int64_t ldw,
                                                     int sub)
{
    typedef float f32x16_t __attribute__((ext_vector_type(16)));
    constexpr int HK = B / 2, NJ = B / 32;
    __shared__ __attribute__((aligned(16))) float ms[B * B];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, li = lane & 31, h = lane >> 5;
    const int64_t b = blockIdx.x;
    const int64_t rbase = part_start(part, b) + (int64_t)blockIdx.y * kRowmulRows + 32 * w;
    const int64_t rend = part_start(part, b + 1);
    if (rbase - 32 * w >= rend)
        return;   // the whole workgroup
    const int64_t row = rbase + li;
    float x[HK];
    const bool vec = (nc & 3) == 0 && (ldi & 3) == 0 && ((uintptr_t)in & 15) == 0;
    const float *xr = in + row * ldi + h * HK;
    if (vec && nc == B && row < rend) {
#pragma unroll
        for (int q = 0; q < HK; q += 4) {
            const float4 v = *(const float4 *)(xr + q);
            x[q] = v.x, x[q + 1] = v.y, x[q + 2] = v.z, x[q + 3] = v.w;
        }
    } else if (B == 32 && vec && row < rend) {
#pragma unroll
        for (int q = 0; q < HK; q += 4) {
            float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (h * HK + q < nc)
                v = *(const float4 *)(xr + q);
            x[q] = v.x, x[q + 1] = v.y, x[q + 2] = v.z, x[q + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int q = 0; q < HK; ++q)
            x[q] = row < rend && h * HK + q < nc ? xr[q] : 0.0f;
    }
    const float *M = Mb + (single ? 0 : b * nc * nc);
    if (nc == B && ((uintptr_t)M & 15) == 0) {
        constexpr int NV = B * B / 1024;   // 16-byte pieces per thread
        constexpr int VS = NV < 4 ? NV : 4;
#pragma unroll
        for (int v0 = 0; v0 < NV; v0 += VS) {
            float4 mv[VS];
#pragma unroll
            for (int v = 0; v < VS; ++v)
                mv[v] = ((const float4 *)M)[(v0 + v) * 256 + t];
#pragma unroll
            for (int v = 0; v < VS; ++v)
                ((float4 *)ms)[(v0 + v) * 256 + t] = mv[v];
        }
    } else {
        for (int r = w; r < B; r += 4)
#pragma unroll
            for (int c = lane; c < B; c += 64)   // (B = 32: half of the wave)
                ms[r * B + c] = r < nc && c < nc ? M[r * nc + c] : 0.0f;
    }
    if (sub) {
#pragma unroll
        for (int q = 0; q < HK; ++q)
            if (row == h * HK + q && row < nc)
                x[q] -= 1.0f;
    }
    if (wout && row < rend) {
        float *wr = wout + row * ldw + h * HK;
        const bool vecw = (nc & 3) == 0 && (ldw & 3) == 0 && ((uintptr_t)wout & 15) == 0;
        if (vecw && nc == B) {
#pragma unroll
            for (int q = 0; q < HK; q += 4)
                *(float4 *)(wr + q) = make_float4(x[q], x[q + 1], x[q + 2], x[q + 3]);
        } else if (B == 32 && vecw) {
#pragma unroll
            for (int q = 0; q < HK; q += 4)
                if (h * HK + q < nc)
                    *(float4 *)(wr + q) = make_float4(x[q], x[q + 1], x[q + 2], x[q + 3]);
        } else {
#pragma unroll
            for (int q = 0; q < HK; ++q)
                if (h * HK + q < nc)
                    wr[q] = x[q];
        }
    }
    __syncthreads();
    constexpr int NS = B == 128 ? 2 : 4;
    f32x16_t acc[NS][NJ] = {};
#pragma unroll
    for (int q = 0; q < HK / NS; ++q)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int p = 0; p < NS; ++p) {
                const int k = q + HK / NS * p;
                acc[p][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                    x[k], ms[(h * HK + k) * B + 32 * j + li], acc[p][j], 0, 0, 0);
            }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        if constexpr (NS == 4) {
            acc[0][j] += acc[2][j];
            acc[1][j] += acc[3][j];
        }
        acc[0][j] += acc[1][j];
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int64_t r = rbase + 8 * (e >> 2) + 4 * h + (e & 3);
            if (r < rend && 32 * j + li < nc)
                out[r * ldo + 32 * j + li] = acc[0][j][e];
        }
}

// Minv = (I - Q_1)^-1 for the top nc x nc block Q_1 of Q (ld ldq), by
// Gauss-Jordan elimination with partial pivoting in FP64 in LDS (512
// threads; thread (i0, c) owns column c of rows i0, i0 + 512 / B, ...), eight
// columns at a time: the elimination is a chain of nc pivots, and with two
// barriers and a pass over the whole array per pivot it took 64 us at nc = 64; 36
// now.
// Rows are not moved: step k pivots on the unused row p_k with the largest
// |M[p_k][k]| (compared in FP32, ties to the lower row), scales row p_k and
// eliminates column k from the other rows.  Wave 0 does this to the eight
// columns in its registers (lane = row); what they then hold is the matrix G of
// the eight eliminations together, and every other column becomes
// x_i <- (i a pivot of these eight ? 0 : x_i) + sum_j G_ij x_{p_j} with the x before,
// by all waves.  The array ends as (P M)^-1 in pivot order, and
// Minv[k][p_c] = B[p_k][c].  Rounded to FP32 (nc x nc, ld nc).  flag[0] = 1
// if a pivot is below kPivotFloor in magnitude or not finite.
template <int B>
__global__ __launch_bounds__(512) void wy_inverse_kernel(const float *__restrict__ Q, int64_t ldq,
                                                         int nc, float *__restrict__ Minv,
                                                         int *flag)
{
    constexpr int LD = B + 1;
    constexpr int RP = 512 / B;   // row phases: thread (i0, c) takes rows i0 + RP q
    constexpr int RO = B / RP;    // rows owned per thread
    constexpr int RL = B / 64;    // rows per lane in wave 0's columns
    constexpr int NB = 8;         // columns per panel
    __shared__ double M[B * LD];
    __shared__ __attribute__((aligned(16))) double G[B * NB];
    __shared__ int piv[B];
    __shared__ int panel_of[B];   // panel in which a row was the pivot, or -1
    const int t = threadIdx.x, lane = t & 63;
    const int cc = t % B, i0 = t / B;
    nc = __builtin_amdgcn_readfirstlane(nc);
    const bool ccol = cc < nc;
    for (int i = i0; i < nc; i += RP)
        if (ccol)
            M[i * LD + cc] = (i == cc ? 1.0 : 0.0) - (double)Q[(int64_t)i * ldq + cc];
    if (t < B)
        panel_of[t] = -1;
    bool used[RL];
#pragma unroll
    for (int q = 0; q < RL; ++q)
        used[q] = false;
    __syncthreads();
    for (int k0 = 0, pn = 0; k0 < nc; k0 += NB, ++pn) {
        if (t < 64) {
            double a[RL][NB];
#pragma unroll
            for (int q = 0; q < RL; ++q)
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    const int r = lane + 64 * q;
                    a[q][j] = r < nc && k0 + j < nc ? M[r * LD + k0 + j] : 0.0;
                }
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                if (k0 + j >= nc)
                    break;
                // key = FP32 magnitude bits (low 7 mantissa bits dropped) | (127 - row)
                unsigned key = 0;
#pragma unroll
                for (int q = 0; q < RL; ++q) {
                    const int r = lane + 64 * q;
                    if (r < nc && !used[q]) {
                        const unsigned kk =
                            ((unsigned)__float_as_int((float)fabs(a[q][j])) & ~0x7Fu) |
                            (unsigned)(127 - r);
                        key = kk > key ? kk : key;
                    }
                }
                key = wave_max(key);
                const int p = __builtin_amdgcn_readfirstlane(127 - (int)(key & 0x7Fu));
                double pr[NB];   // the pivot row's eight entries, uniform
#pragma unroll
                for (int jj = 0; jj < NB; ++jj) {
                    double v = a[0][jj];
                    if (RL > 1 && p >= 64)
                        v = a[RL - 1][jj];
                    pr[jj] = __hiloint2double(
                        __builtin_amdgcn_readlane(__double2hiint(v), p & 63),
                        __builtin_amdgcn_readlane(__double2loint(v), p & 63));
                }
                const double pv = pr[j], inv = 1.0 / pv;
#pragma unroll
                for (int q = 0; q < RL; ++q) {
                    const bool isp = lane + 64 * q == p;
                    const double fi = -a[q][j] * inv;
#pragma unroll
                    for (int jj = 0; jj < NB; ++jj)
                        if (jj != j)
                            a[q][jj] = isp ? pr[jj] * inv : fma(fi, pr[jj], a[q][jj]);
                    a[q][j] = isp ? inv : fi;
                    if (isp)
                        used[q] = true;
                }
                if (lane == 0) {
                    piv[k0 + j] = p;
                    panel_of[p] = pn;
                    if (!(fabs(pv) >= kPivotFloor && isfinite(pv)))
                        flag[0] = 1;
                }
            }
#pragma unroll
            for (int q = 0; q < RL; ++q)
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    G[(lane + 64 * q) * NB + j] = a[q][j];
        }
        __syncthreads();
        const int nb = nc - k0 < NB ? nc - k0 : NB;
        double xp[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j)
            xp[j] = j < nb && ccol ? M[piv[k0 + j] * LD + cc] : 0.0;
        __syncthreads();
        if (ccol) {
            const int own = cc - k0;   // 0 .. nb - 1: a column of the panel itself
#pragma unroll
            for (int q = 0; q < RO; ++q) {
                const int i = i0 + RP * q;
                if (i >= nc)
                    continue;
                const double *g = G + i * NB;
                double v = panel_of[i] == pn ? 0.0 : M[i * LD + cc];
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    v = fma(g[j], xp[j], v);
                if (own >= 0 && own < nb)
                    v = g[own];
                M[i * LD + cc] = v;
            }
        }
        __syncthreads();
    }
    for (int k = i0; k < nc; k += RP)
        if (ccol)
            Minv[(int64_t)k * nc + piv[cc]] = (float)M[piv[k] * LD + cc];
}

// A (ml x nc, lda) <- [R; 0] with R upper triangular (nc x nc, ldr).
__global__ void place_r_kernel(float *A, int64_t lda, int64_t ml, int nc, const float *R,
                               int64_t ldr)
{
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= ml * nc)
        return;
    const int64_t i = idx / nc;
    const int j = (int)(idx % nc);
    A[i * lda + j] = (i < nc && j >= i) ? R[i * ldr + j] : 0.0f;
}

// Q (m x n, ldq) <- [I_n; 0].
__global__ void eye_kernel(float *Q, int64_t ldq, int64_t m, int64_t n)
{
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= m * n)
        return;
    const int64_t i = idx / n, j = idx % n;
    Q[i * ldq + j] = i == j ? 1.0f : 0.0f;
}

__global__ void clear_flag_kernel(int *flag) { flag[threadIdx.x] = 0; }

// out (rows x cols, ldo) = sum over s of parts[s] (rows x cols, ld cols), in order.
__global__ void sum_slices_kernel(const float *__restrict__ parts, int splits, int64_t rows,
                                  int64_t cols, float *__restrict__ out, int64_t ldo)
{
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= rows * cols)
        return;
    float acc = 0.0f;
    for (int s = 0; s < splits; ++s)
        acc += parts[(int64_t)s * rows * cols + idx];
    out[(idx / cols) * ldo + idx % cols] = acc;
}

unsigned grid1d(int64_t count) { return (unsigned)((count + 255) / 256); }

// ----------------------------------------------------------------- planning

size_t al(size_t b) { return align_up256(b); }

// Levels of the TSQR tree for an m x nc panel: level 0 factors the rows of
// A, level l >= 1 factors the stacked R factors of level l - 1
// (rows[l] = nb[l - 1] * nc rows, held in buffer l of the workspace, which
// then receives that level's Q in place).  The top level has one block.
struct TsqrPlan {
    int levels;                 // index of the top level
    int64_t rows[kMaxLevels];
    int nb[kMaxLevels];
    size_t off[kMaxLevels];     // byte offset of buffer l (l >= 1)
    size_t bytes;
    // kappa of every level's blocks, after the buffers, for a tree of several
    // levels of at most 64 columns; a workspace without them factors and forms Q
    // block by block (the same result)
    size_t kap[kMaxLevels], kap_bytes;
};

TsqrPlan tsqr_plan(int64_t m, int nc)
{
    TsqrPlan p;
    memset(&p, 0, sizeof p);
    p.rows[0] = m;
    p.nb[0] = make_part(m, nc).nb;
    int l = 0;
    size_t b = 0;
    while (p.nb[l] > 1 && l + 1 < kMaxLevels) {
        ++l;
        p.rows[l] = (int64_t)p.nb[l - 1] * nc;
        p.nb[l] = make_part(p.rows[l], nc).nb;
        p.off[l] = b;
        b += al((size_t)p.rows[l] * nc * sizeof(float));
    }
    p.levels = l;
    p.bytes = b;
    if (nc <= 64 && l >= 1 && l < kFormLevels) {
        size_t k = 0;
        for (int i = 0; i <= l; ++i) {
            p.kap[i] = k;
            k += al((size_t)p.nb[i] * 64 * sizeof(float));
        }
        p.kap_bytes = k;
    }
    return p;
}

hipError_t launch_rowmul(const float *in, int64_t ldi, const Part &part, int single, int nc,
                         const float *Mb, float *out, int64_t ldo, float *wout, int64_t ldw,
                         int sub, hipStream_t s)
{
    const dim3 grid(part.nb, kRows / kRowmulRows), block(256);
    auto *k = nc <= 32 ? rowmul_kernel<32> : nc <= 64 ? rowmul_kernel<64> : rowmul_kernel<128>;
    hipLaunchKernelGGL(k, grid, block, 0, s, in, ldi, part, single, nc, Mb, out, ldo, wout, ldw,
                       sub);
    return hipGetLastError();
}

template <int B>
hipError_t tsqr_run_b(const float *A, int64_t lda, int nc, float *Q, int64_t ldq, float *R,
                      int64_t ldr, char *ws, const TsqrPlan &tp, char *kap, hipStream_t s)
{
    const int L = tp.levels;
    auto buf = [&](int l) { return (float *)(ws + tp.off[l]); };
    FormArgs fa;
    fa.levels = L + 1;
    fa.nc = nc;
    fa.first[0] = 0;
    const bool split = B == 64 && kap && tp.kap_bytes;
    for (int l = 0; l <= L; ++l) {
        const Part pl = make_part(tp.rows[l], nc);
        const float *in = l == 0 ? A : buf(l);
        const int64_t ldi = l == 0 ? lda : nc;
        float *qo = l == 0 ? Q : buf(l);
        const int64_t ldo = l == 0 ? ldq : nc;
        float *ro = l == L ? R : buf(l + 1);
        const int64_t ldro = l == L ? ldr : nc;
        if constexpr (B == 64) {
            if (split) {
                float *kl = (float *)(kap + tp.kap[l]);
                hipLaunchKernelGGL((qr_block_kernel<64, true>), dim3(pl.nb), dim3(512), 0, s, in, ldi,
                                   pl, nc, qo, ldo, ro, ldro, kl);
                fa.Q[l] = qo;
                fa.ldq[l] = ldo;
                fa.part[l] = pl;
                fa.kap[l] = kl;
                fa.first[l + 1] = fa.first[l] + pl.nb;
            } else {
                hipLaunchKernelGGL((qr_block_kernel<64, false>), dim3(pl.nb), dim3(512), 0, s, in, ldi,
                                   pl, nc, qo, ldo, ro, ldro, (float *)nullptr);
            }
        } else {
            hipLaunchKernelGGL((qr_block_kernel<B, true>), dim3(pl.nb), dim3(8 * B), 0, s, in, ldi,
                               pl, nc, qo, ldo, ro, ldro, (float *)nullptr);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    if constexpr (B == 128) {
        // every level's Q, kFormLevels levels at a time
        for (int l0 = 0; l0 <= L; l0 += kFormLevels) {
            fa.levels = std::min(kFormLevels, L + 1 - l0);
            for (int i = 0; i < fa.levels; ++i) {
                const int l = l0 + i;
                fa.part[i] = make_part(tp.rows[l], nc);
                fa.Q[i] = l == 0 ? Q : buf(l);
                fa.ldq[i] = l == 0 ? ldq : nc;
                fa.first[i + 1] = fa.first[i] + fa.part[i].nb;
            }
            hipLaunchKernelGGL(qr_form128_kernel, dim3(fa.first[fa.levels]), dim3(1024), 0, s, fa);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess)
                return e;
        }
    }
    if (split) {
        hipLaunchKernelGGL(qr_form64_kernel, dim3(fa.first[L + 1]), dim3(512), 0, s, fa);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    for (int l = L - 1; l >= 0; --l) {
        const Part pl = make_part(tp.rows[l], nc);
        float *io = l == 0 ? Q : buf(l);
        const int64_t ld = l == 0 ? ldq : nc;
        hipError_t e = launch_rowmul(io, ld, pl, 0, nc, buf(l + 1), io, ld, nullptr, 0, 0, s);
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

hipError_t tsqr_run(const float *A, int64_t lda, int nc, float *Q, int64_t ldq, float *R,
                    int64_t ldr, char *ws, const TsqrPlan &tp, char *kap, hipStream_t s)
{
    if (nc <= 64)
        return tsqr_run_b<64>(A, lda, nc, Q, ldq, R, ldr, ws, tp, kap, s);
    return tsqr_run_b<128>(A, lda, nc, Q, ldq, R, ldr, ws, tp, kap, s);
}

// W = Q - [I; 0], Y = W (I - Q_1)^-1 for an m x nc Q; Minv: nc x nc scratch.
template <int B>
hipError_t wy_run_b(int64_t m, int nc, const float *Q, int64_t ldq, float *W, int64_t ldw,
                    float *Y, int64_t ldy, float *Minv, int *flag, hipStream_t s)
{
    hipLaunchKernelGGL(wy_inverse_kernel<B>, dim3(1), dim3(512), 0, s, Q, ldq, nc, Minv, flag);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    const Part p = make_part(m, nc);
    return launch_rowmul(Q, ldq, p, 1, nc, Minv, Y, ldy, W, ldw, 1, s);
}

hipError_t wy_run(int64_t m, int nc, const float *Q, int64_t ldq, float *W, int64_t ldw, float *Y,
                  int64_t ldy, float *Minv, int *flag, hipStream_t s)
{
    if (nc <= 64)
        return wy_run_b<64>(m, nc, Q, ldq, W, ldw, Y, ldy, Minv, flag, s);
    return wy_run_b<128>(m, nc, Q, ldq, W, ldw, Y, ldy, Minv, flag, s);
}

size_t wy_bytes(int nc) { return al((size_t)nc * nc * sizeof(float)) + 256; }

// Tile class of a split product X^T V, rows x cols with K slices: direct, so
// that a panel of 64 columns has no idle half tile and each workgroup's share
// of K is a few steps per wave.  32 x 32 tiles while they cover the output in
// four (the next panel's product: the slices give the chip enough workgroups
// and the launch is on the critical path), 64 x 64 tiles else.
int split_class(const GemmDesc &d)
{
    return (d.M <= 64 && d.N <= 64) || d.M < 2 || d.N < 2 ? kClassDirect32 : kClassDirect64;
}

// Split count for a GEMM whose output (rows x cols) is small beside its K:
// enough slices to give every compute unit about two tiles, each slice at
// least min_slice deep, at most max_splits.
int splits_for(int64_t tiles, int64_t K, int num_cus, int max_splits, int64_t min_slice)
{
    tiles = std::max<int64_t>(1, tiles);
    int64_t sp = (2 * num_cus + tiles - 1) / tiles;
    sp = std::min<int64_t>(sp, std::max<int64_t>(1, K / min_slice));
    return (int)std::max<int64_t>(1, std::min<int64_t>(sp, max_splits));
}

// Split-K GEMM Z (rows x cols, ld cols) = X^T V with X (K x rows, ldx) and V
// (K x cols, ldv) in one launch: each slice of K writes its own part (max_splits x
// rows x cols scratch), and the parts are summed in slice order.
hipError_t run_split(int prec, const float *X, int64_t ldx, const float *V, int64_t ldv,
                     int64_t rows, int64_t cols, int64_t K, float *Z, float *parts, int num_cus,
                     int max_splits, int64_t min_slice, hipStream_t s)
{
    GemmDesc d;
    memset(&d, 0, sizeof d);
    d.A = X;
    d.lda = ldx;
    d.a_kcontig = 0;
    d.B = V;
    d.ldb = ldv;
    d.b_kcontig = 0;
    d.ldc = cols;
    d.M = rows;
    d.N = cols;
    d.K = K;
    d.alpha = 1.0f;
    gemm_set_class(d, prec, split_class(d));
    d.slices = splits_for(d.num_tiles, K, num_cus, max_splits, min_slice);
    d.slice_k = (K + d.slices - 1) / d.slices;
    d.slice_stride = rows * cols;
    d.C = d.slices == 1 ? Z : parts;
    const hipError_t e = launch_gemm(prec, d, s);
    if (e != hipSuccess || d.slices == 1)
        return e;
    hipLaunchKernelGGL(sum_slices_kernel, dim3(grid1d(rows * cols)), dim3(256), 0, s,
                       (const float *)parts, d.slices, rows, cols, Z, cols);
    return hipGetLastError();
}

// C (rows x cols, ldc) -= X Z with X (rows x K, ldx) and Z (K x cols, ld cols):
// K is the panel width, so the short-K kernel streams C once with its reads
// issued ahead of the products.
hipError_t gemm_sub(int prec, const float *X, int64_t ldx, const float *Z, int64_t rows,
                    int64_t cols, int64_t K, float *C, int64_t ldc, hipStream_t s)
{
    return launch_short_update(prec, X, ldx, Z, cols, C, ldc, rows, cols, (int)K, s);
}

// Workspace of la_caqr, in order: Qr (m x b), Rr (b x b), the TSQR tree of an
// m x b panel, Minv + flag, W and Y (m x n each with Q; without Q two m x b
// buffers each, alternating between panels), then for the critical stream Z0
// (b x b) and its split-K parts, and for the trailing stream Z1 (b x n) and its
// parts.
struct CaqrWs {
    size_t qr, rr, tree, wy, w, y, z0, parts0, z1, parts1, bytes;
    size_t kap_bytes;   // after them: the TSQR tree's kappa (optional, as la_tsqr's)
};

CaqrWs caqr_ws(int64_t m, int64_t n, int b, int want_q)
{
    CaqrWs w;
    size_t o = 0;
    w.qr = o;
    o += al((size_t)m * b * sizeof(float));
    w.rr = o;
    o += al((size_t)b * b * sizeof(float));
    w.tree = o;
    o += tsqr_plan(m, b).bytes;
    w.wy = o;
    o += wy_bytes(b);
    const size_t wyb = al((size_t)m * (want_q ? n : 2 * b) * sizeof(float));
    w.w = o;
    o += wyb;
    w.y = o;
    o += wyb;
    w.z0 = o;
    o += al((size_t)b * b * sizeof(float));
    // a split product's K is at most m, so it takes at most m / min_slice slices
    const size_t sp_next = (size_t)std::min<int64_t>(kMaxSplitsNext,
                                                     std::max<int64_t>(1, m / kMinSliceNext));
    const size_t sp_wide = (size_t)std::min<int64_t>(kMaxSplits,
                                                     std::max<int64_t>(1, m / kMinSlice));
    w.parts0 = o;
    o += al(sp_next * b * b * sizeof(float));
    w.z1 = o;
    o += al((size_t)b * n * sizeof(float));
    w.parts1 = o;
    o += al(sp_wide * b * n * sizeof(float));
    w.bytes = o;
    w.kap_bytes = tsqr_plan(m, b).kap_bytes;
    return w;
}

// The second stream and the two events of one la_caqr call.
struct LookAhead {
    hipStream_t s1 = nullptr;
    hipEvent_t wy_ready = nullptr, trail_done = nullptr;
    ~LookAhead()
    {
        if (wy_ready)
            (void)hipEventDestroy(wy_ready);
        if (trail_done)
            (void)hipEventDestroy(trail_done);
        if (s1)
            (void)hipStreamDestroy(s1);
    }
};

la_status read_flag(const int *flag, hipStream_t s, const char *who)
{
    int h = 0;
    LA_HIP(hipMemcpyAsync(&h, flag, sizeof h, hipMemcpyDeviceToHost, s), who);
    LA_HIP(hipStreamSynchronize(s), who);
    if (h) {
        set_error("%s: I - Q_1 is singular or nearly so (a pivot below 2^-16): the WY form of "
                  "eq. (Yamamoto) breaks down", who);
        return LA_ERR_BREAKDOWN;
    }
    return LA_OK;
}

la_status check_ws(void *ws, size_t ws_bytes, size_t need, const char *who)
{
    if (need > 0 && !ws) {
        set_error("%s: NULL workspace", who);
        return LA_ERR_INVALID_ARG;
    }
    if (((uintptr_t)ws & 255u) != 0) {
        set_error("%s: workspace must be 256-byte aligned", who);
        return LA_ERR_INVALID_ARG;
    }
    if (ws_bytes < need) {
        set_error("%s: workspace %zu bytes, need %zu", who, ws_bytes, need);
        return LA_ERR_OUT_OF_MEMORY;
    }
    return LA_OK;
}

}  // namespace
}  // namespace la

using namespace la;

extern "C" {

size_t la_tsqr_workspace_size(int64_t m, int64_t n)
{
    if (n < 1 || n > kMaxPanel || m < n)
        return 0;
    const TsqrPlan tp = tsqr_plan(m, (int)n);
    return std::max<size_t>(256, tp.bytes + tp.kap_bytes);
}

la_status la_tsqr(la_context *ctx, int64_t m, int64_t n, const float *A, int64_t lda, float *Q,
                  int64_t ldq, float *R, int64_t ldr, void *workspace, size_t ws_bytes,
                  void *hip_stream)
{
    static const char *who = "la_tsqr";
    set_error("%s", "");
    if (n < 1 || n > kMaxPanel || m < n || lda < n || ldq < n || ldr < n) {
        set_error("%s: bad shape (m %lld, n %lld (1..128, <= m), lda %lld, ldq %lld, ldr %lld)",
                  who, (long long)m, (long long)n, (long long)lda, (long long)ldq,
                  (long long)ldr);
        return LA_ERR_SHAPE;
    }
    if (!ctx || !A || !Q || !R) {
        set_error("%s: NULL argument", who);
        return LA_ERR_INVALID_ARG;
    }
    const TsqrPlan tp = tsqr_plan(m, (int)n);
    la_status st = check_ws(workspace, ws_bytes, tp.bytes, who);
    if (st != LA_OK)
        return st;
    const size_t ab = extent_bytes(m, n, lda), qb = extent_bytes(m, n, ldq),
                 rb = extent_bytes(n, n, ldr);
    if (overlaps(Q, qb, A, ab) || overlaps(R, rb, A, ab) || overlaps(Q, qb, R, rb) ||
        overlaps(A, ab, workspace, tp.bytes) || overlaps(Q, qb, workspace, tp.bytes) ||
        overlaps(R, rb, workspace, tp.bytes)) {
        set_error("%s: A, Q, R and the workspace must not overlap", who);
        return LA_ERR_INVALID_ARG;
    }
    LA_HIP(hipSetDevice(ctx->device), "la_tsqr: hipSetDevice");
    hipStream_t s = (hipStream_t)hip_stream;
    // the optional region after the required one is used only where it is free
    const size_t full = tp.bytes + tp.kap_bytes;
    const bool room = tp.kap_bytes && ws_bytes >= full && !overlaps(A, ab, workspace, full) &&
                      !overlaps(Q, qb, workspace, full) && !overlaps(R, rb, workspace, full);
    LA_HIP(tsqr_run(A, lda, (int)n, Q, ldq, R, ldr, (char *)workspace, tp,
                    room ? (char *)workspace + tp.bytes : nullptr, s),
           "la_tsqr: launch");
    LA_HIP(hipStreamSynchronize(s), "la_tsqr: sync");
    return LA_OK;
}

size_t la_wy_workspace_size(int64_t n)
{
    if (n < 1 || n > kMaxPanel)
        return 0;
    return wy_bytes((int)n);
}

la_status la_wy(la_context *ctx, int64_t m, int64_t n, const float *Q, int64_t ldq, float *W,
                int64_t ldw, float *Y, int64_t ldy, void *workspace, size_t ws_bytes,
                void *hip_stream)
{
    static const char *who = "la_wy";
    set_error("%s", "");
    if (n < 1 || n > kMaxPanel || m < n || ldq < n || ldw < n || ldy < n) {
        set_error("%s: bad shape (m %lld, n %lld (1..128, <= m), ldq %lld, ldw %lld, ldy %lld)",
                  who, (long long)m, (long long)n, (long long)ldq, (long long)ldw,
                  (long long)ldy);
        return LA_ERR_SHAPE;
    }
    if (!ctx || !Q || !W || !Y) {
        set_error("%s: NULL argument", who);
        return LA_ERR_INVALID_ARG;
    }
    const size_t need = wy_bytes((int)n);
    la_status st = check_ws(workspace, ws_bytes, need, who);
    if (st != LA_OK)
        return st;
    const size_t qb = extent_bytes(m, n, ldq), wb = extent_bytes(m, n, ldw),
                 yb = extent_bytes(m, n, ldy);
    if (overlaps(W, wb, Q, qb) || overlaps(Y, yb, Q, qb) || overlaps(W, wb, Y, yb) ||
        overlaps(Q, qb, workspace, need) || overlaps(W, wb, workspace, need) ||
        overlaps(Y, yb, workspace, need)) {
        set_error("%s: Q, W, Y and the workspace must not overlap", who);
        return LA_ERR_INVALID_ARG;
    }
    LA_HIP(hipSetDevice(ctx->device), "la_wy: hipSetDevice");
    hipStream_t s = (hipStream_t)hip_stream;
    float *Minv = (float *)workspace;
    int *flag = (int *)((char *)workspace + al((size_t)n * n * sizeof(float)));
    hipLaunchKernelGGL(clear_flag_kernel, dim3(1), dim3(1), 0, s, flag);
    LA_HIP(hipGetLastError(), "la_wy: clear");
    LA_HIP(wy_run(m, (int)n, Q, ldq, W, ldw, Y, ldy, Minv, flag, s), "la_wy: launch");
    return read_flag(flag, s, who);
}

size_t la_caqr_workspace_size(int64_t m, int64_t n, int panel, int want_q)
{
    if (n < 1 || m < n || panel < 1 || panel > kMaxPanel)
        return 0;
    const CaqrWs cw = caqr_ws(m, n, (int)std::min<int64_t>(panel, n), want_q);
    return cw.bytes + cw.kap_bytes;
}

la_status la_caqr(la_context *ctx, int64_t m, int64_t n, float *A, int64_t lda, float *Q,
                  int64_t ldq, int panel, void *workspace, size_t ws_bytes, la_precision prec,
                  void *hip_stream)
{
    static const char *who = "la_caqr";
    set_error("%s", "");
    if (n < 1 || m < n || lda < n || (Q && ldq < n) || panel < 1 || panel > kMaxPanel) {
        set_error("%s: bad shape (m %lld, n %lld, lda %lld, ldq %lld, panel %d (1..128))", who,
                  (long long)m, (long long)n, (long long)lda, (long long)ldq, panel);
        return LA_ERR_SHAPE;
    }
    if (!valid_prec(prec)) {
        set_error("%s: unknown precision %d", who, (int)prec);
        return LA_ERR_INVALID_ARG;
    }
    if (!ctx || !A) {
        set_error("%s: NULL argument", who);
        return LA_ERR_INVALID_ARG;
    }
    const int b = (int)std::min<int64_t>(panel, n);
    const CaqrWs cw = caqr_ws(m, n, b, Q != nullptr);
    la_status st = check_ws(workspace, ws_bytes, cw.bytes, who);
    if (st != LA_OK)
        return st;
    const size_t ab = extent_bytes(m, n, lda);
    if (overlaps(A, ab, workspace, cw.bytes) ||
        (Q && (overlaps(Q, extent_bytes(m, n, ldq), A, ab) ||
               overlaps(Q, extent_bytes(m, n, ldq), workspace, cw.bytes)))) {
        set_error("%s: A, Q and the workspace must not overlap", who);
        return LA_ERR_INVALID_ARG;
    }
    const size_t full = cw.bytes + cw.kap_bytes;
    const size_t kap_room =
        ws_bytes >= full && !overlaps(A, ab, workspace, full) &&
                !(Q && overlaps(Q, extent_bytes(m, n, ldq), workspace, full))
            ? cw.kap_bytes
            : 0;
    const int pr = resolve_prec(prec, PREC_BF16X6);
    LA_HIP(hipSetDevice(ctx->device), "la_caqr: hipSetDevice");
    hipStream_t s = (hipStream_t)hip_stream;
    char *ws = (char *)workspace;
    float *Qr = (float *)(ws + cw.qr), *Rr = (float *)(ws + cw.rr);
    float *Minv = (float *)(ws + cw.wy);
    int *flag = (int *)(ws + cw.wy + al((size_t)b * b * sizeof(float)));
    float *Wb = (float *)(ws + cw.w), *Yb = (float *)(ws + cw.y);
    float *Z0 = (float *)(ws + cw.z0), *P0 = (float *)(ws + cw.parts0);
    float *Z1 = (float *)(ws + cw.z1), *P1 = (float *)(ws + cw.parts1);
    const int64_t ldwy = Q ? n : b;
    const int64_t np = (n + b - 1) / b;
    auto wpan = [&](int64_t jp) { return Q ? Wb + jp * b * (n + 1) : Wb + (jp & 1) * m * b; };
    auto ypan = [&](int64_t jp) { return Q ? Yb + jp * b * (n + 1) : Yb + (jp & 1) * m * b; };

    // Look-ahead: panel j's reflector is applied first to panel j + 1's
    // columns on the caller's stream (the critical path: the next panel is
    // factored right after), and to the columns beyond on a second stream,
    // where it overlaps the next panels' factorisations.  The next-panel
    // update of panel j waits for the trailing update of panel j - 1 (which
    // covers those columns); a trailing update waits for its panel's W and Y.
    LookAhead la;
    LA_HIP(hipStreamCreateWithFlags(&la.s1, hipStreamNonBlocking), "la_caqr: stream");
    LA_HIP(hipEventCreateWithFlags(&la.wy_ready, hipEventDisableTiming), "la_caqr: event");
    LA_HIP(hipEventCreateWithFlags(&la.trail_done, hipEventDisableTiming), "la_caqr: event");
    // the second stream starts after everything already queued on the caller's
    LA_HIP(hipEventRecord(la.wy_ready, s), "la_caqr: record");
    LA_HIP(hipStreamWaitEvent(la.s1, la.wy_ready, 0), "la_caqr: wait");

    hipLaunchKernelGGL(clear_flag_kernel, dim3(1), dim3(1), 0, s, flag);
    LA_HIP(hipGetLastError(), "la_caqr: clear");
    bool trail_pending = false;   // a trailing update was queued since the last wait on it
    for (int64_t jp = 0; jp < np; ++jp) {
        const int64_t c = jp * b, ml = m - c;
        const int nc = (int)std::min<int64_t>(b, n - c);
        const int64_t nx = c + nc, nc2 = std::min<int64_t>(b, n - nx), rest = nx + nc2;
        float *Ap = A + c * lda + c;
        float *W = wpan(jp), *Y = ypan(jp);
        const TsqrPlan tp = tsqr_plan(ml, nc);
        // (a later panel's tree has no more blocks than the first's)
        LA_HIP(tsqr_run(Ap, lda, nc, Qr, b, Rr, b, ws + cw.tree, tp,
                        tp.kap_bytes <= kap_room ? ws + cw.bytes : nullptr, s),
               "la_caqr: tsqr");
        LA_HIP(wy_run(ml, nc, Qr, b, W, ldwy, Y, ldwy, Minv, flag, s), "la_caqr: wy");
        hipLaunchKernelGGL(place_r_kernel, dim3(grid1d(ml * nc)), dim3(256), 0, s, Ap, lda, ml,
                           nc, (const float *)Rr, (int64_t)b);
        LA_HIP(hipGetLastError(), "la_caqr: place R");
        if (rest < n)
            LA_HIP(hipEventRecord(la.wy_ready, s), "la_caqr: record");
        if (nc2 > 0) {
            if (trail_pending) {
                LA_HIP(hipStreamWaitEvent(s, la.trail_done, 0), "la_caqr: wait");
                trail_pending = false;
            }
            // next panel's columns <- Q_f^T (...) = (...) - Y (W^T (...))
            LA_HIP(run_split(pr, W, ldwy, A + c * lda + nx, lda, nc, nc2, ml, Z0, P0, ctx->num_cus,
                             kMaxSplitsNext, kMinSliceNext, s),
                   "la_caqr: W^T A_next");
            LA_HIP(gemm_sub(pr, Y, ldwy, Z0, ml, nc2, nc, A + c * lda + nx, lda, s),
                   "la_caqr: next-panel update");
        }
        if (rest < n) {
            LA_HIP(hipStreamWaitEvent(la.s1, la.wy_ready, 0), "la_caqr: wait");
            LA_HIP(run_split(pr, W, ldwy, A + c * lda + rest, lda, nc, n - rest, ml, Z1, P1,
                             ctx->num_cus, kMaxSplits, kMinSlice, la.s1),
                   "la_caqr: W^T A_rest");
            LA_HIP(gemm_sub(pr, Y, ldwy, Z1, ml, n - rest, nc, A + c * lda + rest, lda, la.s1),
                   "la_caqr: trailing update");
            LA_HIP(hipEventRecord(la.trail_done, la.s1), "la_caqr: record");
            trail_pending = true;
        }
    }
    // join: the caller's stream continues after the last trailing update
    LA_HIP(hipEventRecord(la.trail_done, la.s1), "la_caqr: record");
    LA_HIP(hipStreamWaitEvent(s, la.trail_done, 0), "la_caqr: wait");
    if (Q) {
        hipLaunchKernelGGL(eye_kernel, dim3(grid1d(m * n)), dim3(256), 0, s, Q, ldq, m, n);
        LA_HIP(hipGetLastError(), "la_caqr: eye");
        for (int64_t jp = np - 1; jp >= 0; --jp) {
            const int64_t c = jp * b, ml = m - c;
            const int nc = (int)std::min<int64_t>(b, n - c);
            float *Qc = Q + c * ldq + c;
            // Q[c:, c:] <- Q_f Q[c:, c:] = Q[c:, c:] - W (Y^T Q[c:, c:])
            LA_HIP(run_split(pr, ypan(jp), n, Qc, ldq, nc, n - c, ml, Z1, P1, ctx->num_cus,
                             kMaxSplits, kMinSlice, s),
                   "la_caqr: Y^T Q");
            LA_HIP(gemm_sub(pr, wpan(jp), n, Z1, ml, n - c, nc, Qc, ldq, s), "la_caqr: Q");
        }
    }
    return read_flag(flag, s, who);
}

}  // extern "C"
