// gemm_direct.h -- small-product GEMM for gfx950: operands go from memory
// straight into MFMA fragments, without LDS, and the waves of a workgroup
// share one tile by splitting K.  Included by the per-precision translation
// units next to gemm_tile.h.
//
// What bounds a product too small to give every CU a 128 x 128 tile is not
// arithmetic but the serial chain of K stages (load, split, LDS write,
// barrier, MFMA) on the few CUs that have a tile: 18 us for 256^3 at 3xBF16,
// of which the MFMAs are 1 us.  Here
//   * the tile is 64 x 64 (KW = 4 waves) or 32 x 32 (KW = 8), so 4 to 16 times
//     as many CUs have one;
//   * wave w takes the 16-k steps w, w + KW, ..., so the chain is KW times
//     shorter, no operand is needed by two waves (hence no LDS staging
//     and no barrier in the loop), and each wave keeps D steps of loads in
//     flight in registers;
//   * the partial sums meet once, in LDS, and every wave finishes its share of
//     the tile's elements.
// Operand rows past the edge are clamped (their products land in elements that
// are not stored), loads need 4-byte alignment only, and the one partial step
// of a K that is no multiple of 16 is loaded element by element and computed
// first by the wave whose turn it is: no tile takes a slower loop for its
// edges, sizes or alignment.
#pragma once

#include "gemm_tile.h"

namespace la {
namespace dev {

// Tile classes (GemmDesc::small), KW waves each.  WPE: waves per SIMD the
// registers are shared by (64 x 64: 64 accumulators and 32 values per step in
// flight and lane, so two workgroups of four waves; eight waves on one 64 x 64
// tile measured the same up to n = 1000 and 10% slower beyond).
template <int CLS> struct DirectCfg;
template <> struct DirectCfg<kClassDirect64> {
    static constexpr int FM = 2, FN = 2, KW = 4, WPE = 2;
};
template <> struct DirectCfg<kClassDirect32> {
    static constexpr int FM = 1, FN = 1, KW = 8, WPE = 4;
};

typedef const __attribute__((address_space(1))) char gchar;

// op(X) rows of a wave's F 32-row blocks and one 16-k step: lane l holds, for
// each block, the 8 k of half l >> 5 of one row.  KC (k contiguous): lane l,
// block b is row r0 + 32 b + (l & 31), two 16-byte loads.  Row-contiguous: lane
// l's F rows are neighbours, r0 + F (l & 31) + b, one F-float load per k (256
// consecutive bytes per k over the lanes for F = 2); a start past R - F is
// moved back to it, so the last lane of an odd R repeats a row instead of
// reading past the matrix.  row() gives the op(X) row of block b, index i, or
// -1 where it is past the edge or such a repeat.  (Offsets are 64-bit a lane: any
// leading dimension; the loop's addresses were 64-bit sums already, so 32-bit ones
// saved three registers and no instruction of it.)
template <bool KC, int F> struct DirectOperand {
    gchar *base;
    uint64_t off[KC ? F : 1];
    int64_t ld;

    __device__ __forceinline__ void init(const float *X, int64_t ld_, int64_t R, int64_t r0,
                                         int lane)
    {
        ld = ld_;
        const int i = lane & 31, h = lane >> 5;
        base = (gchar *)X;
        if constexpr (KC) {
#pragma unroll
            for (int b = 0; b < F; ++b) {
                const int64_t r = r0 + 32 * b + i;
                off[b] = (uint64_t)(((r < R ? r : R - 1) * ld + 8 * h) * 4);
            }
        } else {
            const int64_t r = r0 + F * i;
            off[0] = (uint64_t)(((r < R - F ? r : R - F) + 8 * h * ld) * 4);
        }
    }
    // the step's values; k0 (uniform) + 16 <= K
    __device__ __forceinline__ void load(float (&v)[F][8], int64_t k0) const
    {
        if constexpr (KC) {
            gchar *p = base + k0 * 4;
#pragma unroll
            for (int b = 0; b < F; ++b) {
                const f32x4u x = *(gf32x4u *)(p + off[b]), y = *(gf32x4u *)(p + off[b] + 16);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    v[b][j] = x[j];
                    v[b][4 + j] = y[j];
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                gchar *p = base + (k0 + j) * ld * 4;
                if constexpr (F == 2) {
                    const f32x2u x = *(gf32x2u *)(p + off[0]);
                    v[0][j] = x[0];
                    v[1][j] = x[1];
                } else {
                    v[0][j] = *(const __attribute__((address_space(1))) float *)(p + off[0]);
                }
            }
        }
    }
    // a partial step: k0 + i for i < kn (< 16), zero beyond
    __device__ __forceinline__ void load_tail(float (&v)[F][8], int64_t k0, int kn, int lane) const
    {
        const int h = lane >> 5;
#pragma unroll
        for (int b = 0; b < F; ++b)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                gchar *p = KC ? base + (k0 + j) * 4 + off[b]
                              : base + (k0 + j) * ld * 4 + off[0] + 4 * b;
                v[b][j] = 8 * h + j < kn ? *(const __attribute__((address_space(1))) float *)p : 0.0f;
            }
    }
    __device__ __forceinline__ static int64_t row(int64_t R, int64_t r0, int b, int i)
    {
        if constexpr (KC) {
            const int64_t r = r0 + 32 * b + i;
            return r < R ? r : -1;
        } else {
            const int64_t s = r0 + F * i, c = s < R - F ? s : R - F;
            return s < R && c + b >= s ? c + b : -1;
        }
    }
};

// The same fragments of a packed operand (pack_x3_kernel's layout): lane l's 16
// bytes of each chunk are its fragment of one term.
template <int F> struct DirectPacked {
    gchar *base;
    int64_t kstride;

    __device__ __forceinline__ void init(const void *X, int64_t rbt, int64_t r0, int lane)
    {
        kstride = packed_kstride(rbt);
        base = (gchar *)X + ((r0 / 32) << 11) + lane * 16;
    }
    __device__ __forceinline__ void load(bf16x8 (&v)[F][2], int64_t kb) const
    {
#pragma unroll
        for (int b = 0; b < F; ++b)
#pragma unroll
            for (int t = 0; t < 2; ++t)
                v[b][t] = *(const __attribute__((address_space(1))) bf16x8 *)(
                    base + kb * kstride + (b << 11) + (t << 10));
    }
};

template <int PREC, int FM, int FN>
__device__ __forceinline__ void direct_mfma(const bf16x8 (&a)[FM][Cfg<PREC>::terms],
                                            const bf16x8 (&b)[FN][Cfg<PREC>::terms],
                                            f32x16 (&acc)[FM][FN])
{
    using P = Products<PREC>;
#pragma unroll
    for (int p = 0; p < P::n; ++p)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
                acc[i][j] = mfma16<PREC>(a[i][P::a[p]], b[j][P::b[p]], acc[i][j]);
}

// One 16-k step from FP32 values: split into the precision's terms in
// registers, then the MFMAs, smallest products first.
template <int PREC, int FM, int FN>
__device__ __forceinline__ void direct_step(const float (&va)[FM][8], const float (&vb)[FN][8],
                                            float sa, float sb, f32x16 (&acc)[FM][FN])
{
    if constexpr (PREC == PREC_FP32) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(va[i][e], vb[j][e], acc[i][j],
                                                                    0, 0, 0);
    } else {
        constexpr int T = Cfg<PREC>::terms;
        bf16x8 a[FM][T], b[FN][T];
        u32x4 parts[T];
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            Split<PREC>::run(va[i], parts, sa);
#pragma unroll
            for (int t = 0; t < T; ++t)
                a[i][t] = __builtin_bit_cast(bf16x8, parts[t]);
        }
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            Split<PREC>::run(vb[j], parts, sb);
#pragma unroll
            for (int t = 0; t < T; ++t)
                b[j][t] = __builtin_bit_cast(bf16x8, parts[t]);
        }
        direct_mfma<PREC, FM, FN>(a, b, acc);
    }
}

// A T x T tile of values (LDS, row stride T + 1) as part of a packed operand of
// R rows and K k: rows r0 .. and k0 .. of it (trans: the tile's columns are the
// rows).  A thread takes 8 k of one row, so both terms go out as 16-byte stores,
// consecutive over the rows.  The last block of k is filled with zeros; rows past
// R are left, since what they hold reaches only elements that are not stored.
// pairs: DirectOperand<false, 2>'s order, where row 2 i + b of a block of 64 is
// index i of block b, and a last row on its own the second of its pair.
template <int T, int NT>
__device__ __forceinline__ void direct_pack_out(const float *tile, char *out, int64_t R, int64_t K,
                                                int64_t r0, int64_t k0, bool trans, bool pairs,
                                                int prec, float sc)
{
    const int64_t kstride = packed_kstride(packed_row_blocks(R));
    for (int e = threadIdx.x; e < T * T / 8; e += NT) {
        const int r = e % T, g = e / T;
        const int64_t row = r0 + r, k = k0 + 8 * g;
        if (row >= R || k >= ((K + 15) & ~(int64_t)15))
            continue;
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float x = trans ? tile[(8 * g + j) * (T + 1) + r] : tile[r * (T + 1) + 8 * g + j];
            v[j] = k + j < K ? x : 0.0f;
        }
        u32x4 parts[2];
        if (prec == PREC_F16X3)
            Split<PREC_F16X3>::run(v, parts, sc);
        else
            Split<PREC_BF16X3>::run(v, parts);
        const int64_t q = pairs ? (row & ~(int64_t)63) + 32 * ((row & 1) | (row == R - 1)) +
                                      ((row & 63) >> 1)
                                : row;
        auto *o = (__attribute__((address_space(1))) char *)(out + (k >> 4) * kstride +
                                                              ((q >> 5) << 11)) +
                  ((int)(q & 31) + 32 * (int)((k >> 3) & 1)) * 16;
        *(__attribute__((address_space(1))) u32x4 *)o = parts[0];
        *(__attribute__((address_space(1))) u32x4 *)(o + 1024) = parts[1];
    }
}

// Sum of the waves' partial tiles in LDS (a fixed order, so reproducible), then
// this wave's share of the elements through the common epilogue: out = alpha
// acc + beta E + gamma I, mirrored for a full Gram, with the FP64 sum of
// (out - E)^2, and the packed copies of out.  A workgroup has KW / V waves, each
// in the place of V of the KW (w, w + KW / V, ...: acc[v] and the elements of each).
template <int PREC, class OA, class OB, int FM, int FN, int KW, int V>
__device__ __forceinline__ void direct_epilogue(const GemmDesc &d, f32x16 (&acc)[V][FM][FN],
                                                int64_t row0, int64_t col0, int tm, int tn, int w,
                                                int lane, float *red, double *red8)
{
    constexpr int NE = FM * FN * 16, EPT = NE / KW, EPW = EPT * V, HW = KW / 2, PW = KW / V;
    static_assert(V == 1 || PW == HW, "a wave is one of the KW or a pair of them");
    auto at = [&](int v, int el) -> float & { return red[(v * NE + el) * 64 + lane]; };
    // element q of this thread, of the place w + PW (q / EPT)
    auto element = [&](int q) { return (w + PW * (q / EPT)) * EPT + q % EPT; };
    // place w < HW takes in place w + HW's sums, then those are added in order:
    // half the LDS of KW partial tiles
    if constexpr (V == 1) {
        if (w >= HW)
#pragma unroll
            for (int el = 0; el < NE; ++el)
                at(w - HW, el) = acc[0][el / (16 * FN)][el / 16 % FN][el % 16];
        __syncthreads();
        if (w < HW)
#pragma unroll
            for (int el = 0; el < NE; ++el)
                at(w, el) = acc[0][el / (16 * FN)][el / 16 % FN][el % 16] + at(w, el);
    } else {
#pragma unroll
        for (int el = 0; el < NE; ++el)
            at(w, el) = acc[0][el / (16 * FN)][el / 16 % FN][el % 16] +
                        acc[V - 1][el / (16 * FN)][el / 16 % FN][el % 16];
    }
    __syncthreads();
    float out[EPW];
#pragma unroll
    for (int q = 0; q < EPW; ++q) {
        float s = at(0, element(q));
#pragma unroll
        for (int v = 1; v < HW; ++v)
            s += at(v, element(q));
        out[q] = s;
    }
    const bool want_ss = d.partials != nullptr;
    double ss[V] = {};
    float ev[EPW];
    int64_t rows[EPW], cols[EPW];
#pragma unroll
    for (int q = 0; q < EPW; ++q) {
        const int el = element(q), blk = el >> 4, e = el & 15;
        rows[q] = OA::row(d.M, row0, blk / FN, 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3));
        cols[q] = OB::row(d.N, col0, blk % FN, lane & 31);
        if (d.E) {
            // past the edge element (0, 0) is read and not used
            const int64_t r = rows[q] < 0 ? 0 : rows[q], c = cols[q] < 0 ? 0 : cols[q];
            ev[q] = gmem(d.E)[r * d.lde + c];
        }
    }
    if (d.E)
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
    constexpr int T = 32 * FM;
    static_assert(FM == FN && T * (T + 1) <= HW * NE * 64, "the tile fits the sums' space");
    const bool pack = Cfg<PREC>::terms == 2 && (d.pack_row || d.pack_col);
    if (pack)
        __syncthreads();   // every wave has read its sums
#pragma unroll
    for (int q = 0; q < EPW; ++q) {
        const int64_t row = rows[q], col = cols[q];
        if (row < 0 || col < 0 || (d.gram && row > col))
            continue;
        float val = d.alpha * out[q];
        float evv = 0.0f;
        if (d.E) {
            evv = ev[q];
            val = val + d.beta * evv;
        }
        if (row == col)
            val = val + d.gamma;
        if (d.C) {
            gmem(d.C)[row * d.ldc + col] = val;
            if (d.gram && !d.gram_upper && row != col)
                gmem(d.C)[col * d.ldc + row] = val;
        }
        if (pack) {
            const int lr = (int)(row - row0), lc = (int)(col - col0);
            red[lr * (T + 1) + lc] = val;
            if (d.gram && tm == tn)
                red[lc * (T + 1) + lr] = val;
        }
        if (want_ss) {
            const double df = (double)val - (double)evv;
            ss[q / EPT] += df * df;
        }
    }
    if (want_ss) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1)
                ss[v] += __shfl_xor(ss[v], off, 64);
            if (lane == 0)
                red8[w + PW * v] = ss[v];
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            double s = 0.0;
            for (int k = 0; k < KW; ++k)
                s += red8[k];
            gmem(d.partials)[(int64_t)tm * d.tiles_n + tn] = s;
        }
    }
    if constexpr (Cfg<PREC>::terms == 2) {
        if (!pack)
            return;
        __syncthreads();
        const bool pairs = d.pack_pairs;
        if (d.pack_row)
            direct_pack_out<T, PW * 64>(red, d.pack_row, d.M, d.N, row0, col0, false, pairs,
                                        d.pack_prec, d.pack_scale);
        if (d.gram && tm != tn)
            direct_pack_out<T, PW * 64>(red, d.pack_row, d.M, d.N, col0, row0, true, pairs,
                                        d.pack_prec, d.pack_scale);
        if (d.pack_col)
            direct_pack_out<T, PW * 64>(red, d.pack_col, d.N, d.M, col0, row0, true, false,
                                        d.pack_prec, d.pack_scale);
    }
}

// The sums of place w of the KW that share a tile, k in [kb, ke) of the operands (left
// undone with stop, looked at once the first loads are on their way).
template <int PREC, bool AKC, bool BKC, int CLS>
__device__ __forceinline__ void
direct_sums(const GemmDesc &d, int64_t row0, int64_t col0, int64_t kb, int64_t ke, int w, int lane,
            int stop, f32x16 (&acc)[DirectCfg<CLS>::FM][DirectCfg<CLS>::FN])
{
    using G = DirectCfg<CLS>;
    constexpr int FM = G::FM, FN = G::FN, KW = G::KW;
    // steps of loads in flight per wave: what the registers of WPE waves per
    // SIMD leave beside the accumulators and the split terms
    constexpr int D = CLS == kClassDirect32 ? 3 : (PREC == PREC_BF16X6 ? 2 : 3);
    DirectOperand<AKC, FM> oa;
    DirectOperand<BKC, FN> ob;
    oa.init(d.A, d.lda, d.M, row0, lane);
    ob.init(d.B, d.ldb, d.N, col0, lane);

#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
            acc[i][j] = f32x16{};

    const int nfull = (int)((ke - kb) >> 4), kn = (int)((ke - kb) & 15);
    const int cnt = w < nfull ? (nfull - w + KW - 1) / KW : 0;
    float va[D][FM][8], vb[D][FN][8];
    auto fetch = [&](int slot, int i) {
        const int64_t k0 = kb + 16 * (int64_t)(w + KW * i);
        oa.load(va[slot], k0);
        ob.load(vb[slot], k0);
    };
    if (cnt > 0) {
        // past the last step the loads repeat it: no branch in the loop
#pragma unroll
        for (int s = 0; s < D; ++s)
            fetch(s, min(s, cnt - 1));
    }
    if (stop)
        return;
    if (kn && w == nfull % KW) {
        float ta[FM][8], tb[FN][8];
        oa.load_tail(ta, kb + 16 * (int64_t)nfull, kn, lane);
        ob.load_tail(tb, kb + 16 * (int64_t)nfull, kn, lane);
        direct_step<PREC, FM, FN>(ta, tb, d.scale_a, d.scale_b, acc);
    }
    int i = 0;
    for (; i + D <= cnt; i += D) {
#pragma unroll
        for (int s = 0; s < D; ++s) {
            direct_step<PREC, FM, FN>(va[s], vb[s], d.scale_a, d.scale_b, acc);
            fetch(s, min(i + s + D, cnt - 1));
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int s = 0; s < D - 1; ++s)
        if (i + s < cnt)
            direct_step<PREC, FM, FN>(va[s], vb[s], d.scale_a, d.scale_b, acc);
}

// One tile by KW / V waves.
template <int PREC, bool AKC, bool BKC, int CLS, int V = 1>
__device__ __forceinline__ void direct_tile(const GemmDesc &d, int tm, int tn, int64_t kb,
                                            int64_t ke, float *red, double *red8)
{
    using G = DirectCfg<CLS>;
    constexpr int FM = G::FM, FN = G::FN, KW = G::KW;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t row0 = (int64_t)tm * (32 * FM), col0 = (int64_t)tn * (32 * FN);
    const int stop = d.stop ? *gmem(d.stop) : 0;
    f32x16 acc[V][FM][FN];
#pragma unroll
    for (int v = 0; v < V; ++v)
        direct_sums<PREC, AKC, BKC, CLS>(d, row0, col0, kb, ke, w + KW / V * v, lane, stop, acc[v]);
    if (stop)
        return;   // uniform over the launch
    direct_epilogue<PREC, DirectOperand<AKC, FM>, DirectOperand<BKC, FN>, FM, FN, KW, V>(
        d, acc, row0, col0, tm, tn, w, lane, red, red8);
}

template <int CLS> constexpr int direct_red_floats()
{
    return DirectCfg<CLS>::KW / 2 * DirectCfg<CLS>::FM * DirectCfg<CLS>::FN * 16 * 64;
}

// One workgroup per tile; with d.slices, grid row y takes the K slice
// [y slice_k, min(K, (y + 1) slice_k)) and writes C + y slice_stride.
template <int PREC, bool AKC, bool BKC, int CLS>
__global__ void __launch_bounds__(DirectCfg<CLS>::KW * 64, DirectCfg<CLS>::WPE)
    gemm_direct_kernel(GemmDesc d)
{
    __shared__ float red[direct_red_floats<CLS>()];
    __shared__ double red8[DirectCfg<CLS>::KW];
    int64_t kb = 0, ke = d.K;
    if (d.slices > 1) {
        kb = (int64_t)blockIdx.y * d.slice_k;
        ke = kb + d.slice_k < d.K ? kb + d.slice_k : d.K;
        if (ke < kb)
            ke = kb;
        d.C += (int64_t)blockIdx.y * d.slice_stride;
    }
    int tm, tn;
    tile_coords(d, xcd_remap(blockIdx.x, d.num_tiles), tm, tn);
    direct_tile<PREC, AKC, BKC, CLS>(d, tm, tn, kb, ke, red, red8);
}

// The same for the items of a grouped launch (one workgroup per item).
template <int PREC, bool AKC, bool BKC, int CLS>
__global__ void __launch_bounds__(DirectCfg<CLS>::KW * 64, DirectCfg<CLS>::WPE)
    gemm_direct_items_kernel(const GemmDesc *__restrict__ probs,
                             const GroupItem *__restrict__ items, int num_items)
{
    __shared__ float red[direct_red_floats<CLS>()];
    __shared__ double red8[DirectCfg<CLS>::KW];
    const int it = blockIdx.x;
    if (it >= num_items)
        return;
    const GroupItem gi = items[it];
    if (gi.prob < 0)
        return;   // empty item
    const GemmDesc d = probs[gi.prob];
    int tm, tn;
    tile_coords(d, gi.tile, tm, tn);
    direct_tile<PREC, AKC, BKC, CLS>(d, tm, tn, 0, d.K, red, red8);
}

// Packed operands, for la_gemm_packed's small shapes and for iterations whose
// products write their results packed for the next (pack_row, pack_col): every
// element is the same sums in the same order as gemm_direct_kernel's (a partial
// step first, the waves' steps interleaved), and with PAIRS its place in the wave
// too.  The unpacked kernel spends most of a step splitting operand values that
// every tile in their row or column splits again; here a step is its loads and
// MFMAs (3xBF16, n^3 in one graph: 256 4.5 -> 3.5 us, 512 6.3 -> 4.3, 1000 19.4
// -> 11.6, 1600 60 -> 35).  Inside an iteration the operands come from the other
// XCDs' writes and the launch is bound by fetching them: two, three and four
// steps in flight measured the same (polar 1000^2 856, 861, 858 us).
template <int PREC, int CLS, bool PAIRS, int V = 1>
__device__ __forceinline__ void direct_packed_tile(const GemmDesc &d, int tm, int tn, float *red,
                                                   double *red8)
{
    using G = DirectCfg<CLS>;
    constexpr int FM = G::FM, FN = G::FN, KW = G::KW, D = 2;
    const int lane = threadIdx.x & 63;
    const int w0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t row0 = (int64_t)tm * (32 * FM), col0 = (int64_t)tn * (32 * FN);
    const int stop = d.stop ? *gmem(d.stop) : 0;
    DirectPacked<FM> oa;
    DirectPacked<FN> ob;
    oa.init(d.A, packed_row_blocks(d.M), row0, lane);
    ob.init(d.B, packed_row_blocks(d.N), col0, lane);
    f32x16 acc[V][FM][FN];
    const int nfull = (int)(d.K >> 4), kn = (int)(d.K & 15);
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int w = w0 + KW / V * v;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
                acc[v][i][j] = f32x16{};
        const int cnt = w < nfull ? (nfull - w + KW - 1) / KW : 0;
        bf16x8 a[D][FM][2], b[D][FN][2];
        if (kn && w == nfull % KW) {
            oa.load(a[0], nfull);
            ob.load(b[0], nfull);
            direct_mfma<PREC, FM, FN>(a[0], b[0], acc[v]);
        }
        auto fetch = [&](int s, int i) {
            oa.load(a[s], w + KW * (int64_t)i);
            ob.load(b[s], w + KW * (int64_t)i);
        };
        if (cnt > 0) {
#pragma unroll
            for (int s = 0; s < D; ++s)
                fetch(s, min(s, cnt - 1));
        }
        if (stop)
            return;   // uniform over the launch
        int i = 0;
        for (; i + D <= cnt; i += D) {
#pragma unroll
            for (int s = 0; s < D; ++s) {
                direct_mfma<PREC, FM, FN>(a[s], b[s], acc[v]);
                fetch(s, min(i + s + D, cnt - 1));
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int s = 0; s < D - 1; ++s)
            if (i + s < cnt)
                direct_mfma<PREC, FM, FN>(a[s], b[s], acc[v]);
    }
    direct_epilogue<PREC, DirectOperand<true, FM>, DirectOperand<!PAIRS, FN>, FM, FN, KW, V>(
        d, acc, row0, col0, tm, tn, w0, lane, red, red8);
}

template <int PREC, int CLS, bool PAIRS>
__global__ void __launch_bounds__(DirectCfg<CLS>::KW * 64, DirectCfg<CLS>::WPE)
    gemm_direct_packed_kernel(GemmDesc d)
{
    __shared__ float red[direct_red_floats<CLS>()];
    __shared__ double red8[DirectCfg<CLS>::KW];
    int tm, tn;
    tile_coords(d, xcd_remap(blockIdx.x, d.num_tiles), tm, tn);
    direct_packed_tile<PREC, CLS, PAIRS>(d, tm, tn, red, red8);
}

// ---------------------------------------------------------------- launchers

template <int PREC, int CLS>
hipError_t launch_direct(const GemmDesc &d, hipStream_t s)
{
    const int sl = d.slices > 1 ? d.slices : 1;
    if (sl > 1 && (d.slice_k <= 0 || sl > 65535))
        return hipErrorInvalidValue;
    // a row-contiguous operand is read FM (FN) rows at a time
    if (d.M < DirectCfg<CLS>::FM || d.N < DirectCfg<CLS>::FN)
        return hipErrorInvalidValue;
    const dim3 grid(d.num_tiles, sl), block(DirectCfg<CLS>::KW * 64);
    if (d.a_kcontig && d.b_kcontig)
        hipLaunchKernelGGL((gemm_direct_kernel<PREC, true, true, CLS>), grid, block, 0, s, d);
    else if (d.a_kcontig)
        hipLaunchKernelGGL((gemm_direct_kernel<PREC, true, false, CLS>), grid, block, 0, s, d);
    else if (d.b_kcontig)
        hipLaunchKernelGGL((gemm_direct_kernel<PREC, false, true, CLS>), grid, block, 0, s, d);
    else
        hipLaunchKernelGGL((gemm_direct_kernel<PREC, false, false, CLS>), grid, block, 0, s, d);
    return hipGetLastError();
}

// launch_t with the direct classes
template <int PREC>
hipError_t launch_any(const GemmDesc &d, hipStream_t s)
{
    if (d.num_tiles <= 0)
        return hipSuccess;
    if (d.small == kClassDirect64)
        return launch_direct<PREC, kClassDirect64>(d, s);
    if (d.small == kClassDirect32)
        return launch_direct<PREC, kClassDirect32>(d, s);
    return launch_t<PREC>(d, s);
}

// (op(B) is row-contiguous: launch_grouped_any)
template <int PREC, int CLS>
hipError_t launch_direct_items(int akc, const GemmDesc *probs, const GroupItem *items,
                               int num_items, hipStream_t s)
{
    const dim3 grid(num_items), block(DirectCfg<CLS>::KW * 64);
    if (akc)
        hipLaunchKernelGGL((gemm_direct_items_kernel<PREC, true, false, CLS>), grid, block, 0, s,
                           probs, items, num_items);
    else
        hipLaunchKernelGGL((gemm_direct_items_kernel<PREC, false, false, CLS>), grid, block, 0, s,
                           probs, items, num_items);
    return hipGetLastError();
}

// A grouped launch of one class.  Every caller's op(B) is row-contiguous, and the direct
// classes come here at FP32 only (launch_gemm_mixed takes the others): nothing else is
// built.
template <int PREC>
hipError_t launch_grouped_any(int akc, int bkc, int small, const GemmDesc *probs,
                              const GroupItem *items, int num_items, hipStream_t s)
{
    if (num_items <= 0)
        return hipSuccess;
    if (bkc)
        return hipErrorInvalidValue;
    if (!is_direct(small))
        return launch_grouped_t<PREC>(akc, small, probs, items, num_items, s);
    if constexpr (PREC == PREC_FP32)
        return small == kClassDirect64
                   ? launch_direct_items<PREC, kClassDirect64>(akc, probs, items, num_items, s)
                   : launch_direct_items<PREC, kClassDirect32>(akc, probs, items, num_items, s);
    return hipErrorInvalidValue;
}

template <int PREC, int CLS> hipError_t launch_direct_packed(const GemmDesc &d, hipStream_t s)
{
    const dim3 grid(d.num_tiles), block(DirectCfg<CLS>::KW * 64);
    if (d.b_pairs)
        hipLaunchKernelGGL((gemm_direct_packed_kernel<PREC, CLS, true>), grid, block, 0, s, d);
    else
        hipLaunchKernelGGL((gemm_direct_packed_kernel<PREC, CLS, false>), grid, block, 0, s, d);
    return hipGetLastError();
}

// Packed operands on the tile class of d.
template <int PREC>
hipError_t launch_packed_any(const GemmDesc &d, hipStream_t s)
{
    if (d.num_tiles <= 0)
        return hipSuccess;
    if (d.small == kClassDirect64)
        return launch_direct_packed<PREC, kClassDirect64>(d, s);
    if (d.small == kClassDirect32)
        return launch_direct_packed<PREC, kClassDirect32>(d, s);
    return launch_packed_x3<PREC>(d, s);
}

}  // namespace dev
}  // namespace la
