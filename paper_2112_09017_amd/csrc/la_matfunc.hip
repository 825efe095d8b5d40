// Polynomial matrix functions (section III.D of arXiv 2112.09017).
//
// la_matfunc_odd: an odd polynomial acting on the singular values
// (eqs. MatFunc, odd_power, OddPoly):
//   F = sum_j c_j A (A^T A)^j = A p(G),  G = A^T A,  p(x) = sum_j c_j x^j,
// evaluated as one symmetric Gram launch, Horner's rule in G (one GEMM per
// coefficient beyond the second, c_j I added in the epilogue), and F = A P.
//
// la_matfunc_cheb: a Chebyshev series acting on the eigenvalues
// (eqs. MatFuncEig, any_power, EigenvaluePolynomial):
//   F = sum_k c_k T_k(B),  B = (2A - (lo + hi) I) / (hi - lo),
// evaluated by Clenshaw's recurrence b_k = 2 B b_{k+1} - b_{k+2} + c_k I,
// F = B b_1 - b_2 + c_0 I: d - 1 GEMM launches for degree d >= 2, each with
// the -b_{k+2} + c_k I update in its epilogue (written in place over b_{k+2}).
#include <hip/hip_runtime.h>

#include <math.h>
#include <string.h>

#include <algorithm>

#include "la_internal.h"

namespace la {
namespace {

size_t matfunc_bytes(int64_t n) { return 3 * align_up256((size_t)n * n * sizeof(float)); }

// AUTO's products as three products of two scaled fp16 terms (PREC_F16X3) on
// packed operands, in place of 6xBF16, where the fixed operand is even: half the
// matrix-core work and half the FP32 accumulation roundings (degree 16 at 4096^2:
// 9.6 -> 6.4 ms; 3000^2 6.4 -> 3.1 ms).  Each row of op(A) and each column of op(B) is
// scaled by the power of two of its own largest entry, so rows and columns of very
// different size keep their accuracy.  An element far below its row's largest keeps
// an absolute error of 2^-39 of that only, which a sum sees where the other operand is
// large there (B = D S D^-1, D from 1 to 2^20, degree 8 at 2048^2: error 3.1e-7 against
// 1.6e-7 with the similarity undone; odd series of columns from 1 to 2^-30: 5e-3 against
// 4.3e-7 in the worst), so an uneven fixed operand (PackCheck) keeps 6xBF16.
// The answer stays on the device, where it turns the packs and products
// queued behind it into nothing; the host reads it after the last of them and queues
// them again at 6xBF16.  The largest entries come from one pass over a fixed operand
// and, for the recurrence's iterates, from the epilogue that writes them.  The packs
// live after the three matrices, where the workspace has room.
struct F16 {
    bool on = false;
    char *pa = nullptr, *pb = nullptr;            // packed op(A), op(B)^T
    uint32_t *ra = nullptr, *cb[2] = {};          // their rows' and columns' maxima
    int *uneven = nullptr;   // answers: [0] for the recurrence (kUneven*), [1] for F = A P
    uint32_t *counts[3] = {};   // of the Gram's A, of Horner's G or the series' B, of A's rows
};
constexpr int kUnevenA = 1, kUnevenG = 2;
constexpr size_t kFlagWords = 64;

// Words of the answers and the counts after them.
size_t f16_count_words(int64_t m, int64_t n) { return kFlagWords + 2 * (size_t)(m + 2 * n); }

// Whether an M x N x K product of the recurrence runs as F16X3: on tiles that the
// packed kernel has (the direct ones are bound by reading their operands, not by
// multiplying them), with K deep enough to repay the packs, and for the
// accumulation roundings to outweigh the one bit less per operand.  (4096^2
// product: 640 us at 6xBF16, 355 and 24 for the pack; errors of whole calls,
// F16X3 / 6xBF16: degree 16 at 1700 1.51e-7 / 1.68e-7, 4096 2.23e-7 / 2.40e-7, odd
// series of 6 terms at 4096 7.7e-7 / 8.4e-7; with K = 300 2.59e-7 / 2.48e-7 and no
// gain in time.)
bool f16_class(int64_t M, int64_t N, int64_t K, int gram)
{
    GemmDesc d;
    memset(&d, 0, sizeof d);
    d.M = M;
    d.N = N;
    d.K = K;
    d.lda = gram ? N : K;
    d.ldb = N;
    d.a_kcontig = gram ? 0 : 1;
    d.gram = gram;
    gemm_finalize(d, PREC_F16X3);
    return !is_direct(d.small) && std::min(M, N) >= 256 && K >= 1024;
}

size_t f16_bytes(int64_t m, int64_t n)
{
    size_t pa = 0, pb = 0;
    if (f16_class(n, n, m, 1))
        pa = std::max(pa, packed_x3_bytes(n, m));
    if (f16_class(n, n, n, 0))
        pa = std::max(pa, packed_x3_bytes(n, n));
    if (f16_class(m, n, n, 0))
        pa = std::max(pa, packed_x3_bytes(m, n));
    if (!pa)
        return 0;
    pb = packed_x3_bytes(n, n);
    return align_up256(pa) + align_up256(pb) +
           align_up256((size_t)std::max(m, n) * sizeof(uint32_t)) +
           2 * align_up256((size_t)n * sizeof(uint32_t)) +
           align_up256(f16_count_words(m, n) * sizeof(uint32_t));
}

F16 f16_carve(int64_t m, int64_t n, void *workspace)
{
    F16 f;
    f.on = true;
    char *b = (char *)workspace + matfunc_bytes(n) + f16_bytes(m, n) -
              align_up256(f16_count_words(m, n) * sizeof(uint32_t));
    f.uneven = (int *)b;
    f.counts[0] = (uint32_t *)b + kFlagWords;
    f.counts[1] = f.counts[0] + m + n;
    f.counts[2] = f.counts[1] + 2 * n;
    for (uint32_t *&c : f.cb) {
        b -= align_up256((size_t)n * sizeof(uint32_t));
        c = (uint32_t *)b;
    }
    b -= align_up256((size_t)std::max(m, n) * sizeof(uint32_t));
    f.ra = (uint32_t *)b;
    b -= align_up256(packed_x3_bytes(n, n));
    f.pb = b;
    f.pa = (char *)workspace + matfunc_bytes(n);
    return f;
}

// Packs op(A) = X (M x K, kc) or X^T (M columns, K rows, !kc) into f.pa, rows scaled
// by their own largest entries; an uneven X sets bit in f.uneven[w].
hipError_t f16_pack_a(const F16 &f, const float *X, int64_t ldx, int kc, int64_t M, int64_t K,
                      int w, int bit, uint32_t *counts, hipStream_t s)
{
    hipError_t e = launch_absmax(X, ldx, kc ? M : K, kc ? K : M, kc, f.ra, s);
    if (e == hipSuccess)
        e = launch_pack(PREC_F16X3, X, ldx, kc, M, K, 1.0f, f.pa, s, f.ra, nullptr,
                        PackCheck{counts, f.uneven + w, bit});
    return e;
}

// out = alpha op(A) Y + beta E + gamma I with op(A) (M x K) in f.pa and Y (K x N,
// columns' maxima in f.cb[c]); the columns' maxima of out go to f.cb[c ^ 1].  Nothing is
// done where f.uneven[w].
hipError_t f16_product(const F16 &f, int w, int c, const float *Y, int64_t ldy, float *out,
                       int64_t ldo, int64_t M, int64_t N, int64_t K, float alpha, float beta, const float *E,
                       int64_t lde, float gamma, hipStream_t s)
{
    GemmDesc d;
    memset(&d, 0, sizeof d);
    d.C = out;
    d.ldc = ldo;
    d.M = M;
    d.N = N;
    d.K = K;
    d.alpha = alpha;
    d.gamma = gamma;
    if (E) {
        d.E = E;
        d.lde = lde;
        d.beta = beta;
    }
    d.stop = f.uneven + w;
    hipError_t e = launch_pack(PREC_F16X3, Y, ldy, 0, N, K, 1.0f, f.pb, s, f.cb[c], d.stop);
    if (e == hipSuccess)
        e = launch_zero(f.cb[c ^ 1], N, s);
    if (e != hipSuccess)
        return e;
    d.A = (const float *)f.pa;
    d.B = (const float *)f.pb;
    d.row_max = f.ra;
    d.col_max = f.cb[c];
    d.out_max = f.cb[c ^ 1];
    gemm_set_packed(d);
    return launch_gemm_packed(PREC_F16X3, d, s);
}

la_status check_coef(const double *coef, int ncoef, const char *who)
{
    if (!coef || ncoef < 1) {
        set_error("%s: need at least one coefficient", who);
        return LA_ERR_INVALID_ARG;
    }
    for (int i = 0; i < ncoef; ++i)
        if (!isfinite(coef[i])) {
            set_error("%s: coefficient %d is not finite", who, i);
            return LA_ERR_INVALID_ARG;
        }
    return LA_OK;
}

// The F16X3 packs of a call, on where prec is AUTO, some product takes them and
// the workspace has a free region for them after the three matrices (a smaller
// workspace runs every product at 6xBF16).
F16 use_f16(int prec, int64_t m, int64_t n, void *workspace, size_t ws_bytes, const float *A,
            size_t ab, const float *F, size_t fb)
{
    const size_t full = matfunc_bytes(n) + f16_bytes(m, n);
    if (prec != LA_PREC_AUTO || full == matfunc_bytes(n) || ws_bytes < full ||
        overlaps(workspace, full, A, ab) || overlaps(workspace, full, F, fb))
        return F16{};
    return f16_carve(m, n, workspace);
}

// out = alpha X Y + beta E + gamma I, X (M x K) and Y (K x N) row-major.
hipError_t product(int prec, const float *X, int64_t ldx, const float *Y, int64_t ldy, float *out,
                   int64_t ldo, int64_t M, int64_t N, int64_t K, float alpha, float beta,
                   const float *E, int64_t lde, float gamma, hipStream_t s)
{
    GemmDesc d;
    memset(&d, 0, sizeof d);
    d.A = X;
    d.lda = ldx;
    d.a_kcontig = 1;
    d.B = Y;
    d.ldb = ldy;
    d.b_kcontig = 0;
    d.C = out;
    d.ldc = ldo;
    d.M = M;
    d.N = N;
    d.K = K;
    d.alpha = alpha;
    d.gamma = gamma;
    if (E) {
        d.E = E;
        d.lde = lde;
        d.beta = beta;
    }
    gemm_finalize(d, prec);
    return launch_gemm(prec, d, s);
}

}  // namespace
}  // namespace la

using namespace la;

extern "C" {

size_t la_matfunc_workspace_size(int64_t m, int64_t n)
{
    if (m < 1 || n < 1)
        return 0;
    return matfunc_bytes(n) + f16_bytes(m, n);
}

la_status la_matfunc_odd(la_context *ctx, int64_t m, int64_t n, const float *A, int64_t lda,
                         const double *coef, int ncoef, float *F, int64_t ldf, void *workspace,
                         size_t ws_bytes, la_precision prec, void *hip_stream)
{
    static const char *who = "la_matfunc_odd";
    set_error("%s", "");
    if (m < 1 || n < 1 || lda < n || ldf < n) {
        set_error("%s: bad shape (m %lld, n %lld, lda %lld, ldf %lld)", who, (long long)m,
                  (long long)n, (long long)lda, (long long)ldf);
        return LA_ERR_SHAPE;
    }
    la_status st = check_coef(coef, ncoef, who);
    if (st != LA_OK)
        return st;
    if (!valid_prec(prec)) {
        set_error("%s: unknown precision %d", who, (int)prec);
        return LA_ERR_INVALID_ARG;
    }
    if (!ctx || !A || !F || !workspace) {
        set_error("%s: NULL argument", who);
        return LA_ERR_INVALID_ARG;
    }
    if (((uintptr_t)workspace & 255u) != 0) {
        set_error("%s: workspace must be 256-byte aligned", who);
        return LA_ERR_INVALID_ARG;
    }
    const size_t need = matfunc_bytes(n);
    if (ws_bytes < need) {
        set_error("%s: workspace %zu bytes, need %zu", who, ws_bytes, need);
        return LA_ERR_OUT_OF_MEMORY;
    }
    const size_t fb = extent_bytes(m, n, ldf);
    if (overlaps(F, fb, A, extent_bytes(m, n, lda)) || overlaps(F, fb, workspace, need)) {
        set_error("%s: F overlaps A or the workspace", who);
        return LA_ERR_INVALID_ARG;
    }
    const int pr = resolve_prec(prec, PREC_BF16X6);
    const F16 f = use_f16(prec, m, n, workspace, ws_bytes, A, extent_bytes(m, n, lda), F, fb);
    LA_HIP(hipSetDevice(ctx->device), "la_matfunc_odd: hipSetDevice");
    hipStream_t s = (hipStream_t)hip_stream;
    const int d = ncoef - 1;
    if (d == 0) {
        // F = c_0 A (FP64 per element: A / (1 / c_0), and 0 for c_0 = 0)
        LA_HIP(launch_scale(A, lda, F, ldf, m, n, 1.0 / coef[0], s), "la_matfunc_odd: scale");
        LA_HIP(hipStreamSynchronize(s), "la_matfunc_odd: sync");
        return LA_OK;
    }
    const size_t nb = align_up256((size_t)n * n * sizeof(float));
    float *G = (float *)workspace;
    float *P[2] = {(float *)((char *)workspace + nb), (float *)((char *)workspace + 2 * nb)};

    // A is the fixed operand of the Gram and of F = A P, G of Horner's products
    bool f_gram = f.on && f16_class(n, n, m, 1), f_final = f.on && f16_class(m, n, n, 0);
    bool f_horner = f.on && d >= 2 && f16_class(n, n, n, 0);
    const bool scaled = f_final;
    // G = A^T A (symmetric tiles only, mirror-written)
    auto gram = [&]() {
        GemmDesc g;
        memset(&g, 0, sizeof g);
        g.A = A;
        g.B = A;
        g.lda = lda;
        g.ldb = lda;
        g.a_kcontig = 0;
        g.b_kcontig = 0;
        g.C = G;
        g.ldc = n;
        g.M = n;
        g.N = n;
        g.K = m;
        g.alpha = 1.0f;
        g.gram = 1;
        if (!f_gram) {
            gemm_finalize(g, pr);
            LA_HIP(launch_gemm(pr, g, s), "la_matfunc_odd: gram");
            return LA_OK;
        }
        LA_HIP(f16_pack_a(f, A, lda, 0, n, m, 0, kUnevenA, f.counts[0], s), "la_matfunc_odd: pack");
        g.A = (const float *)f.pa;
        g.B = (const float *)f.pa;
        g.row_max = f.ra;
        g.col_max = f.ra;
        g.stop = f.uneven;
        gemm_finalize(g, PREC_F16X3);
        gemm_set_packed(g);
        LA_HIP(launch_gemm_packed(PREC_F16X3, g, s), "la_matfunc_odd: gram");
        return LA_OK;
    };
    // Horner in G: P = c_d G + c_{d-1} I, then P <- G P + c_j I for j = d-2 .. 0
    int cur = 0;
    auto horner = [&]() {
        cur = 0;
        LA_HIP(launch_affine(G, n, P[0], n, n, coef[d], coef[d - 1], s), "la_matfunc_odd: affine");
        if (f_horner) {
            LA_HIP(f16_pack_a(f, G, n, 1, n, n, 0, kUnevenG, f.counts[1], s),
                   "la_matfunc_odd: pack");
            LA_HIP(launch_absmax(P[0], n, n, n, 0, f.cb[0], s), "la_matfunc_odd: pack");
        }
        for (int j = d - 2; j >= 0; --j) {
            if (f_horner)
                LA_HIP(f16_product(f, 0, cur, P[cur], n, P[cur ^ 1], n, n, n, n, 1.0f, 0.0f,
                                   nullptr, 0, (float)coef[j], s),
                       "la_matfunc_odd: horner");
            else
                LA_HIP(product(pr, G, n, P[cur], n, P[cur ^ 1], n, n, n, n, 1.0f, 0.0f, nullptr, 0,
                               (float)coef[j], s),
                       "la_matfunc_odd: horner");
            cur ^= 1;
        }
        return LA_OK;
    };
    // F = A P
    auto last = [&]() {
        if (f_final) {
            if (!f_horner)
                LA_HIP(launch_absmax(P[cur], n, n, n, 0, f.cb[cur], s), "la_matfunc_odd: pack");
            LA_HIP(f16_pack_a(f, A, lda, 1, m, n, 1, 1, f.counts[2], s), "la_matfunc_odd: pack");
            LA_HIP(f16_product(f, 1, cur, P[cur], n, F, ldf, m, n, n, 1.0f, 0.0f, nullptr, 0, 0.0f,
                               s),
                   "la_matfunc_odd: final product");
        } else if (scaled) {
            // an uneven A, at 6xBF16: its rows scaled all the same, so that the third
            // term of a small row's entries stays in range
            float *As = (float *)f.pa;
            LA_HIP(launch_absmax(A, lda, m, n, 1, f.ra, s), "la_matfunc_odd: rows");
            LA_HIP(launch_scale_rows(A, lda, As, n, m, n, f.ra, 0, s), "la_matfunc_odd: rows");
            LA_HIP(product(pr, As, n, P[cur], n, F, ldf, m, n, n, 1.0f, 0.0f, nullptr, 0, 0.0f, s),
                   "la_matfunc_odd: final product");
            LA_HIP(launch_scale_rows(F, ldf, F, ldf, m, n, f.ra, 1, s), "la_matfunc_odd: rows");
        } else {
            LA_HIP(product(pr, A, lda, P[cur], n, F, ldf, m, n, n, 1.0f, 0.0f, nullptr, 0, 0.0f, s),
                   "la_matfunc_odd: final product");
        }
        return LA_OK;
    };
    // from the first phase on; what an uneven operand turned into nothing is queued again
    for (int phase = 0; phase < 3;) {
        if (f.on)
            LA_HIP(launch_zero((uint32_t *)f.uneven, f16_count_words(m, n), s),
                   "la_matfunc_odd: unevenness");
        if (phase == 0 && (st = gram()) != LA_OK)
            return st;
        if (phase <= 1 && (st = horner()) != LA_OK)
            return st;
        if ((st = last()) != LA_OK)
            return st;
        int uneven[2] = {0, 0};
        if (f.on)
            LA_HIP(hipMemcpyAsync(uneven, f.uneven, sizeof uneven, hipMemcpyDeviceToHost, s),
                   "la_matfunc_odd: readback");
        LA_HIP(hipStreamSynchronize(s), "la_matfunc_odd: sync");
        if (uneven[1])
            f_final = false;
        if (uneven[0] & kUnevenA) {
            f_gram = false;
            phase = 0;
        } else if (uneven[0]) {
            f_horner = false;
            phase = 1;
        } else {
            phase = uneven[1] ? 2 : 3;
        }
    }
    return LA_OK;
}

la_status la_matfunc_cheb(la_context *ctx, int64_t n, const float *A, int64_t lda, double lo,
                          double hi, const double *coef, int ncoef, float *F, int64_t ldf,
                          void *workspace, size_t ws_bytes, la_precision prec, void *hip_stream)
{
    static const char *who = "la_matfunc_cheb";
    set_error("%s", "");
    if (n < 1 || lda < n || ldf < n) {
        set_error("%s: bad shape (n %lld, lda %lld, ldf %lld)", who, (long long)n,
                  (long long)lda, (long long)ldf);
        return LA_ERR_SHAPE;
    }
    la_status st = check_coef(coef, ncoef, who);
    if (st != LA_OK)
        return st;
    if (!isfinite(lo) || !isfinite(hi) || !(hi > lo)) {
        set_error("%s: need finite lo < hi", who);
        return LA_ERR_INVALID_ARG;
    }
    if (!valid_prec(prec)) {
        set_error("%s: unknown precision %d", who, (int)prec);
        return LA_ERR_INVALID_ARG;
    }
    if (!ctx || !A || !F || !workspace) {
        set_error("%s: NULL argument", who);
        return LA_ERR_INVALID_ARG;
    }
    if (((uintptr_t)workspace & 255u) != 0) {
        set_error("%s: workspace must be 256-byte aligned", who);
        return LA_ERR_INVALID_ARG;
    }
    const size_t need = matfunc_bytes(n);
    if (ws_bytes < need) {
        set_error("%s: workspace %zu bytes, need %zu", who, ws_bytes, need);
        return LA_ERR_OUT_OF_MEMORY;
    }
    const size_t fb = extent_bytes(n, n, ldf);
    if (overlaps(F, fb, A, extent_bytes(n, n, lda)) || overlaps(F, fb, workspace, need)) {
        set_error("%s: F overlaps A or the workspace", who);
        return LA_ERR_INVALID_ARG;
    }
    const int pr = resolve_prec(prec, PREC_BF16X6);
    F16 f = use_f16(prec, n, n, workspace, ws_bytes, A, extent_bytes(n, n, lda), F, fb);
    f.on = f.on && f16_class(n, n, n, 0);
    LA_HIP(hipSetDevice(ctx->device), "la_matfunc_cheb: hipSetDevice");
    hipStream_t s = (hipStream_t)hip_stream;
    // B = sc A + t I maps [lo, hi] onto [-1, 1]
    const double sc = 2.0 / (hi - lo), t = -(hi + lo) / (hi - lo);
    const int d = ncoef - 1;
    const double *c = coef;
    if (d <= 1) {
        // c_0 I  or  c_0 I + c_1 B
        const double c1 = d == 1 ? c[1] : 0.0;
        LA_HIP(launch_affine(A, lda, F, ldf, n, c1 * sc, c1 * t + c[0], s),
               "la_matfunc_cheb: affine");
        LA_HIP(hipStreamSynchronize(s), "la_matfunc_cheb: sync");
        return LA_OK;
    }
    const size_t nb = align_up256((size_t)n * n * sizeof(float));
    float *B = (float *)workspace;
    float *P[2] = {(float *)((char *)workspace + nb), (float *)((char *)workspace + 2 * nb)};
    LA_HIP(launch_affine(A, lda, B, n, n, sc, t, s), "la_matfunc_cheb: B");
    // b_{d-1} = 2 c_d B + c_{d-1} I (b_d = c_d I, b_{d+1} = 0)
    LA_HIP(launch_affine(A, lda, P[0], n, n, 2.0 * c[d] * sc, 2.0 * c[d] * t + c[d - 1], s),
           "la_matfunc_cheb: b_{d-1}");
    // op(A) is B throughout; the iterate in P[i] has its columns' maxima in cb[i]
    auto times_b = [&](int c, float *out, int64_t ldo, float alpha, float beta, const float *E,
                       float gamma) {
        if (f.on)
            return f16_product(f, 0, c, P[c], n, out, ldo, n, n, n, alpha, beta, E, n, gamma, s);
        return product(pr, B, n, P[c], n, out, ldo, n, n, n, alpha, beta, E, n, gamma, s);
    };
    // from b_{d-1} on; where B is uneven, nothing has been written and the loop runs again
    for (int uneven = 1; uneven;) {
        uneven = 0;
        if (f.on) {
            LA_HIP(launch_zero((uint32_t *)f.uneven, f16_count_words(n, n), s),
                   "la_matfunc_cheb: unevenness");
            LA_HIP(f16_pack_a(f, B, n, 1, n, n, 0, 1, f.counts[1], s), "la_matfunc_cheb: pack");
            LA_HIP(launch_absmax(P[0], n, n, n, 0, f.cb[0], s), "la_matfunc_cheb: pack");
        }
        if (d == 2) {
            // F = B b_1 - b_2 + c_0 I with b_2 = c_2 I
            LA_HIP(times_b(0, F, ldf, 1.0f, 0.0f, nullptr, (float)(c[0] - c[2])),
                   "la_matfunc_cheb: final product");
        } else {
            // b_{d-2} = 2 B b_{d-1} - c_d I + c_{d-2} I
            LA_HIP(times_b(0, P[1], n, 2.0f, 0.0f, nullptr, (float)(c[d - 2] - c[d])),
                   "la_matfunc_cheb: clenshaw");
            int cur = 1;   // P[cur] = b_{k+1}, P[cur ^ 1] = b_{k+2}
            for (int k = d - 3; k >= 1; --k) {
                // b_k = 2 B b_{k+1} - b_{k+2} + c_k I, written over b_{k+2}
                float *prev = P[cur ^ 1];
                LA_HIP(times_b(cur, prev, n, 2.0f, -1.0f, prev, (float)c[k]),
                       "la_matfunc_cheb: clenshaw");
                cur ^= 1;
            }
            // F = B b_1 - b_2 + c_0 I
            LA_HIP(times_b(cur, F, ldf, 1.0f, -1.0f, P[cur ^ 1], (float)c[0]),
                   "la_matfunc_cheb: final product");
        }
        if (f.on)
            LA_HIP(hipMemcpyAsync(&uneven, f.uneven, sizeof uneven, hipMemcpyDeviceToHost, s),
                   "la_matfunc_cheb: readback");
        LA_HIP(hipStreamSynchronize(s), "la_matfunc_cheb: sync");
        f.on = f.on && !uneven;
    }
    return LA_OK;
}

}  // extern "C"
