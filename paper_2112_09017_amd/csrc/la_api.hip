// C ABI: context, error reporting, la_gemm, the la_polar driver and the
// la_inverse driver (Algorithm NS_Inverse, at the end of this file).
//
// la_polar follows Algorithm NS_Polar (section III.D of arXiv 2112.09017):
//   U <- A / ||A||_F                                   (FP64 norm on the GPU)
//   k_pre steps  U <- a U (I - (4/27) a^2 U^T U)       (eqs. a_def, RogueMatrix)
//     with k_pre from the scalar recurrence of eq. (RogueScalar) on the host
//   Newton-Schulz U' <- U (3I - U^T U) / 2 until ||U' - U||_F <= max(M,N) eps
//     (eq. NewtonSchulz), evaluated as U' = U + U (I - U^T U) / 2, which is the
//     same polynomial written so the small correction is formed separately
//   H <- (U^T A + A^T U) / 2
// Each step is two launches: the symmetric Gram (only upper tiles, the
// polynomial coefficients applied in its epilogue) and the product with the
// update applied in the epilogue.  The only host synchronisation per step is
// the 8-byte readback of ||U' - U||_F^2 for the data-dependent stop test; small
// problems queue their steps in batches instead, with the test on the device.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <mutex>

#include "la_internal.h"

namespace la {

static thread_local char g_err[512];

// The one statically allocated device buffer of the library: the workspace of
// la_polar_noalloc, for callers that cannot allocate device memory.  Each GPU
// the library runs on holds its own copy until the process ends; its address
// on a device comes from hipGetSymbolAddress, taken once per device when the
// first context on that device is created.
constexpr size_t kScratchBytes = LA_POLAR_NOALLOC_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void *g_scratch_ptr[kMaxDevices];

// Device address of `scratch` on `device` (the caller has made it current).
static hipError_t scratch_address(int device, void **out)
{
    std::lock_guard<std::mutex> g(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess)
            return e;
        g_scratch_ptr[device] = p;
    }
    *out = g_scratch_ptr[device];
    return hipSuccess;
}

void set_error(const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
}

la_status dev_fail(hipError_t e, const char *where)
{
    set_error("%s: %s", where, hipGetErrorString(e));
    return LA_ERR_DEVICE;
}

bool overlaps(const void *a, size_t abytes, const void *b, size_t bbytes)
{
    if (!a || !b || abytes == 0 || bbytes == 0)
        return false;
    const uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
    return a0 < b0 + bbytes && b0 < a0 + abytes;
}

size_t extent_bytes(int64_t rows, int64_t cols, int64_t ld)
{
    if (rows <= 0 || cols <= 0)
        return 0;
    return (size_t)((rows - 1) * ld + cols) * sizeof(float);
}

int resolve_prec(int p, int dflt)
{
    return p == LA_PREC_AUTO ? dflt : p;
}

bool valid_prec(int p)
{
    return p == LA_PREC_AUTO || p == LA_PREC_FP32 || p == LA_PREC_BF16X3 ||
           p == LA_PREC_BF16X6;
}

// ------------------------------------------------------------------ polar plan

// (polar_plan, the FP32 accumulation depth kMaxAccK and the stop test are in
// polar_host.h)

int acc_splits(int64_t K, int64_t max_acc)
{
    const int64_t a = max_acc > 0 ? max_acc : kMaxAccK;
    return K > a ? (int)std::min<int64_t>(65535, (K + a - 1) / a) : 1;
}

// Slices of K for a requested count: the slice length is a multiple of 32 (whole
// K stages of every kernel), so the count that results may be smaller.
static int slice_plan(int64_t K, int want, int64_t *slice_k)
{
    int64_t sk = (K + want - 1) / want;
    sk = (sk + 31) / 32 * 32;
    *slice_k = sk;
    return (int)((K + sk - 1) / sk);
}

// Split-K slices of a Gram: enough to keep each slice's FP32 accumulation
// within kMaxAccK, and, when the tiles cannot fill the 256 CUs, enough to
// fill them (the slices run in one launch; each keeps at least 2048 of the
// K = m rows).
int gram_splits(int64_t m, int64_t n, int prec, int64_t max_acc)
{
    const int64_t nb = (n + tile_n(prec) - 1) / tile_n(prec);
    const int64_t tiles = nb * (nb + 1) / 2;
    int fill = 1;
    const int64_t cap = std::max<int64_t>(1, std::min<int64_t>(16, m / 2048));
    if (tiles >= 256) {
        fill = 1;
    } else if (tiles >= 128) {
        // large tiles, one per CU: take the count whose rounds of 256 tiles
        // cost least per unit of K (N = 4096: 136 tiles x 15 slices = 2040,
        // 8 rounds of K / 15, against 3 rounds of K / 4 with 4 slices)
        int64_t best = 1, best_rounds = 1;
        for (int64_t sp = 2; sp <= cap; ++sp) {
            const int64_t rounds = (tiles * sp + 255) / 256;
            if (rounds * best < best_rounds * sp) {
                best = sp;
                best_rounds = rounds;
            }
        }
        fill = (int)best;
    } else {
        // small tiles: about two tiles per CU
        const int64_t sp = (512 + tiles - 1) / tiles;
        fill = (int)std::max<int64_t>(1, std::min<int64_t>(sp, cap));
    }
    int64_t sk = 0;
    return slice_plan(m, std::max(fill, acc_splits(m, max_acc)), &sk);
}

size_t align_up256(size_t x) { return (x + 255) & ~(size_t)255; }
static size_t align256(size_t x) { return align_up256(x); }

// A region for packed operands; a product whose packs don't fit it runs unpacked,
// with the same result.
struct PackBuf {
    char *p;        // null: none
    size_t bytes;
};

struct PolarWs {
    float *X;        // m x n, ld n: the iterate's second buffer
    float *P;        // n x n: I - c U^T U or I - U^T U
    float *parts;    // split-K slices of a Gram, an update or H (may be null)
    double *tiles;   // per-tile (or per-block) step-norm partials
    double *sumsq;   // norm partials, then the rest of the step-norm partials
    double *scal;    // [0] ||A||_F^2, [1] ||U' - U||_F^2
    PackBuf pk;      // packed copies of U and P for the update, or of U^T for the Gram
    PolarChain chain;   // where col is not null
    size_t parts_floats;
};

static bool two_term(int prec) { return prec == PREC_BF16X3 || prec == PREC_F16X3; }

// Whether an M x N x K product on large tiles (at least 128 of 256 x 256) takes
// the packed-operand kernel: two 16-bit terms and K >= 256, as in la_gemm_ws.
// The packed kernel computes every product exactly as the unpacked one, so the
// choice never changes a result.
static bool packs(int prec, int64_t M, int64_t N, int64_t K)
{
    return two_term(prec) && K >= 256 && ((M + 255) / 256) * ((N + 255) / 256) >= 128;
}

// Whether a product of the small class takes it too where there is room for its
// packs: the 128 x 128 packed tiles run at 28 to 44 ns per unit of K against 43
// to 57 unpacked, the packs cost about 8 us each (2048^3: 59 + 16 us against
// 86).
static bool packs_small(int prec, const GemmDesc &d)
{
    return two_term(prec) && d.small == kClassSmall && std::min(d.M, d.N) >= 256 && d.K >= 1024;
}

// Bytes of the packed op(A) and op(B)^T of a product that packs (0 otherwise).
static size_t pack_bytes(int prec, int64_t M, int64_t N, int64_t K)
{
    if (!packs(prec, M, N, K))
        return 0;
    return align_up256(packed_x3_bytes(M, K)) + align_up256(packed_x3_bytes(N, K));
}

// The same for a product of the small class.
static size_t pack_small_bytes(int prec, int64_t M, int64_t N, int64_t K)
{
    GemmDesc d;
    memset(&d, 0, sizeof d);
    d.M = M;
    d.N = N;
    d.K = K;
    gemm_finalize(d, prec);
    if (!packs_small(prec, d))
        return 0;
    return align_up256(packed_x3_bytes(M, K)) + align_up256(packed_x3_bytes(N, K));
}

// Launch d, through the packed-operand kernel when it qualifies and its packs fit
// pk: op(A) and op(B)^T are packed into pk first,
// unless an operand packed earlier is passed (pre_a / pre_b).  K-slices of d
// (d.slices > 1) run on whichever kernel is chosen; d's tile counts are those of
// the launch.
static hipError_t gemm_packed_or_plain(int prec, GemmDesc &d, PackBuf pk, hipStream_t s,
                                       const char *pre_a = nullptr, const char *pre_b = nullptr)
{
    const size_t ab = align_up256(packed_x3_bytes(d.M, d.K));
    if (pk.p && !d.gram && ab + align_up256(packed_x3_bytes(d.N, d.K)) <= pk.bytes &&
        ((!d.small && packs(prec, d.M, d.N, d.K)) || packs_small(prec, d))) {
        char *pa = pk.p, *pb = pk.p + ab;
        hipError_t e = hipSuccess;
        if (!pre_a)
            e = launch_pack(prec, d.A, d.lda, d.a_kcontig, d.M, d.K, d.scale_a, pa, s);
        if (e == hipSuccess && !pre_b)
            e = launch_pack(prec, d.B, d.ldb, d.b_kcontig, d.N, d.K, d.scale_b, pb, s);
        if (e != hipSuccess)
            return e;
        d.A = (const float *)(pre_a ? pre_a : pa);
        d.B = (const float *)(pre_b ? pre_b : pb);
        gemm_set_packed(d);
        return launch_gemm_packed(prec, d, s);
    }
    return launch_gemm(prec, d, s);
}

// Whether a Gram X^T X (n x n, K = m) at prec runs on the packed-operand
// kernel: two 16-bit terms with at least 128 upper 256 x 256 tiles and K >= 256.
// X^T is packed once and serves as both operands.
static bool gram_packs(int prec, int64_t m, int64_t n)
{
    const int64_t nb = (n + 255) / 256;
    return two_term(prec) && m >= 256 && nb * (nb + 1) / 2 >= 128;
}

// Packed copies the iteration keeps: X and P for a packed update, or X^T for
// a packed Gram (the Gram's pack is consumed before the update packs).  Steps
// at 3xBF16 size the region; F16X3 steps (the same bytes) use it where it is
// there and run unpacked otherwise, with the same result.
static size_t packed_update_bytes(const PolarPlan &p)
{
    size_t b = 0;
    for (int pr : {p.prec_pre, p.prec_ns}) {
        if (pr != PREC_BF16X3)
            continue;
        b = std::max(b, pack_bytes(pr, p.m, p.n, p.n));
        if (gram_packs(pr, p.m, p.n))
            b = std::max(b, align_up256(packed_x3_bytes(p.n, p.m)));
    }
    return b;
}

// Bytes by which that region has to grow for the products of the small class that
// pack.  It is part of what la_polar_workspace_size asks for, but a
// workspace without it is taken, and gives the same result on unpacked operands.
static size_t packed_small_bytes(const PolarPlan &p)
{
    size_t b = 0;
    for (int pr : {p.prec_pre, p.prec_ns}) {
        if (!two_term(pr))
            continue;
        b = std::max(b, pack_small_bytes(pr, p.m, p.n, p.n));
        GemmDesc g;
        memset(&g, 0, sizeof g);
        g.M = p.n;
        g.N = p.n;
        g.K = p.m;
        g.lda = p.n;
        g.ldb = p.n;
        g.gram = 1;
        gemm_finalize(g, pr);
        if (packs_small(pr, g))
            b = std::max(b, align_up256(packed_x3_bytes(p.n, p.m)));
    }
    const size_t have = packed_update_bytes(p);
    return b > have ? b - have : 0;
}

// Slices of the update X P (K = n) and of each half of H (K = m).
static int update_splits(const PolarPlan &p)
{
    int64_t sk = 0;
    return slice_plan(p.n, acc_splits(p.n, p.max_acc), &sk);
}

static int h_splits(const PolarPlan &p)
{
    int64_t sk = 0;
    return slice_plan(p.m, acc_splits(p.m, p.max_acc), &sk);
}

// Floats of split-K slices the iteration and H need at most: a Gram's
// slices (n x n each), an update's (m x n each, when its K = n is split),
// and H's two sets of n x n slices (U^T A and A^T U).
static size_t parts_floats(const PolarPlan &p)
{
    size_t f = 0;
    for (int pr : {p.prec_pre, p.prec_ns, (int)PREC_BF16X6}) {
        const int g = gram_splits(p.m, p.n, pr, p.max_acc);
        if (g > 1)
            f = std::max(f, (size_t)g * p.n * p.n);
    }
    const int u = update_splits(p);
    if (u > 1)
        f = std::max(f, (size_t)u * p.m * p.n);
    f = std::max(f, (size_t)2 * h_splits(p) * p.n * p.n);
    return f;
}

static size_t max_update_tiles(const PolarPlan &p)
{
    return std::max((size_t)splitk_update_num_partials(), step_partials(p.m, p.n));
}

size_t polar_workspace_bytes(const PolarPlan &p)
{
    size_t b = 0;
    b += align256((size_t)p.m * p.n * sizeof(float));
    b += align256((size_t)p.n * p.n * sizeof(float));
    b += align256(parts_floats(p) * sizeof(float));
    b += align256(max_update_tiles(p) * sizeof(double));
    b += align256((size_t)sumsq_num_partials() * sizeof(double));
    b += align256(8 * sizeof(double));
    b += packed_update_bytes(p);
    return b;
}

// Smallest n of a polar on packed copies: below, writing them costs what reading
// them saves (polar of n^2 without / with them: 256 358 / 365 us, 384 430 / 396,
// 700 756 / 648, 1000 1104 / 857, 1600 2620 / 1780).  (The server's launches hold
// many requests and are bound by their operands at any n.)
constexpr int64_t kChainMinN = 320;

// The shape of the update X P (its tile class at the two-term arithmetics is the same).
static GemmDesc update_shape(const PolarPlan &p, int prec)
{
    GemmDesc d;
    memset(&d, 0, sizeof d);
    d.M = p.m;
    d.N = p.n;
    d.K = p.n;
    gemm_finalize(d, prec);
    return d;
}

size_t polar_chain_bytes(const PolarPlan &p, bool served)
{
    if (!two_term(p.prec_pre) || !two_term(p.prec_ns))
        return 0;
    if (!served && (p.n < kChainMinN || update_splits(p) > 1))
        return 0;
    for (int pr : {p.prec_pre, p.prec_ns}) {
        if (!served && gram_splits(p.m, p.n, pr, p.max_acc) > 1)
            return 0;
        GemmDesc d = update_shape(p, pr);
        if (!is_direct(d.small))
            return 0;
        d.M = p.n;
        d.K = p.m;
        d.gram = 1;
        gemm_finalize(d, pr);
        if (!is_direct(d.small))
            return 0;
    }
    return 2 * align_up256(packed_x3_bytes(p.m, p.n)) + align_up256(packed_x3_bytes(p.n, p.m)) +
           align_up256(packed_x3_bytes(p.n, p.n));
}

PolarChain polar_chain_carve(const PolarPlan &p, char *base)
{
    PolarChain c;
    const size_t row = align_up256(packed_x3_bytes(p.m, p.n));
    c.row[0] = base;
    c.row[1] = base + row;
    c.col = base + 2 * row;
    c.P = c.col + align_up256(packed_x3_bytes(p.n, p.m));
    c.pairs = update_shape(p, p.prec_ns).small == kClassDirect64;
    return c;
}

static PolarWs carve(const PolarPlan &p, void *ws, bool room, bool chain)
{
    PolarWs w;
    char *b = (char *)ws;
    w.X = (float *)b;
    b += align256((size_t)p.m * p.n * sizeof(float));
    w.P = (float *)b;
    b += align256((size_t)p.n * p.n * sizeof(float));
    w.parts_floats = parts_floats(p);
    w.parts = (float *)b;
    b += align256(w.parts_floats * sizeof(float));
    w.tiles = (double *)b;
    b += align256(max_update_tiles(p) * sizeof(double));
    w.sumsq = (double *)b;
    b += align256((size_t)sumsq_num_partials() * sizeof(double));
    w.scal = (double *)b;
    b += align256(8 * sizeof(double));
    w.pk.bytes = packed_update_bytes(p) + (room ? packed_small_bytes(p) : 0);
    w.pk.p = w.pk.bytes ? b : nullptr;
    memset(&w.chain, 0, sizeof w.chain);
    if (chain) {
        w.chain = polar_chain_carve(p, b);
        w.pk = PackBuf{};
    }
    return w;
}

// Launch the Gram-mode product d (k-major operands).  Where both operands are
// one matrix, it qualifies and X^T fits pk, X^T is packed once into pk and read as
// both; the packed kernel computes every product exactly as the unpacked one.
static hipError_t gram_packed_or_plain(int prec, GemmDesc &d, PackBuf pk, hipStream_t s)
{
    if (pk.p && d.A == d.B && d.lda == d.ldb && packed_x3_bytes(d.N, d.K) <= pk.bytes &&
        ((!d.small && gram_packs(prec, d.K, d.N)) || packs_small(prec, d))) {
        hipError_t e = launch_pack(prec, d.A, d.lda, 0, d.N, d.K, d.scale_a, pk.p, s);
        if (e != hipSuccess)
            return e;
        d.A = (const float *)pk.p;
        d.B = (const float *)pk.p;
        gemm_set_packed(d);
        return launch_gemm_packed(prec, d, s);
    }
    return launch_gemm(prec, d, s);
}

// X1^T X2 for K x n operands X1, X2 (row-major, leading dimensions ld1, ld2)
// as about `want` K-slices in one Gram-mode launch: slice y writes the upper
// triangle (i <= j) of its n x n part, the sum over its k range, at
// parts + y n^2.  *count receives the number of slices.  sc1, sc2: the
// operands' factors where prec is F16X3.
static hipError_t gram_slices(int prec, const float *X1, int64_t ld1, float sc1,
                              const float *X2, int64_t ld2, float sc2, int64_t K, int64_t n,
                              int want, float *parts, int *count, hipStream_t s,
                              PackBuf pk = PackBuf{})
{
    GemmDesc d;
    memset(&d, 0, sizeof d);
    d.A = X1;
    d.B = X2;
    d.a_kcontig = 0;
    d.b_kcontig = 0;
    d.lda = ld1;
    d.ldb = ld2;
    d.M = n;
    d.N = n;
    d.K = K;
    d.gram = 1;
    d.gram_upper = 1;
    d.C = parts;
    d.ldc = n;
    d.alpha = 1.0f;
    gemm_f16_scales(d, prec, sc1, sc2);
    gemm_finalize(d, prec);
    d.slices = slice_plan(K, want, &d.slice_k);
    d.slice_stride = n * n;
    *count = d.slices;
    return gram_packed_or_plain(prec, d, pk, s);
}

// P <- alpha X^T X + gamma I (exactly symmetric), X m x n with leading dim ldx.
// chained: X's packed columns are there, and P is written packed too.
static hipError_t gram_step(const PolarPlan &p, int prec, const float *X, int64_t ldx,
                            double alpha, double gamma, float *P, const PolarWs &w,
                            hipStream_t s, bool chained = false, const int *stop = nullptr)
{
    const int64_t m = p.m, n = p.n;
    const int splits = gram_splits(m, n, prec, p.max_acc);
    if (splits <= 1 || (size_t)splits * n * n > w.parts_floats) {
        GemmDesc d;
        memset(&d, 0, sizeof d);
        d.a_kcontig = 0;
        d.b_kcontig = 0;
        d.lda = ldx;
        d.ldb = ldx;
        d.M = n;
        d.N = n;
        d.gram = 1;
        d.A = X;
        d.B = X;
        d.C = P;
        d.ldc = n;
        d.K = m;
        d.alpha = (float)alpha;
        d.gamma = (float)gamma;
        d.stop = stop;
        gemm_f16_scales(d, prec, kIterScale, kIterScale);
        gemm_finalize(d, prec);
        if (chained) {
            d.A = d.B = (const float *)w.chain.col;
            d.C = nullptr;   // only the update reads P
            d.pack_row = w.chain.P;
            d.pack_prec = prec;
            d.pack_scale = kIterScale;
            d.pack_pairs = w.chain.pairs;
            return launch_gemm_packed(prec, d, s);
        }
        return gram_packed_or_plain(prec, d, w.pk, s);
    }
    // the slices run in one launch; slice y sums k in [y ks, (y + 1) ks) into
    // the upper triangle of its own n x n part, and the parts are added in
    // slice order in FP64
    int count = 0;
    hipError_t e = gram_slices(prec, X, ldx, kIterScale, X, ldx, kIterScale, m, n, splits, w.parts,
                               &count, s, w.pk);
    if (e != hipSuccess)
        return e;
    return launch_splitk_sym_reduce(w.parts, n * n, count, n, alpha, gamma, P, n, s);
}

// A chained update: whether X and P are there packed (X in buffer cur), and the
// arithmetic that the next step reads Xn in.
struct ChainStep {
    bool packed;
    int cur, next_prec;
    bool only;   // nothing but the next step's products reads Xn
};

// Partials of a step norm (Xn - X)^2, where they ended up.
struct StepNorm {
    const double *parts;
    int64_t count;
};

// The Gram's slices have been added before the update, so their region is free for its
// partials (polar of 1000000 x 64 20.2 ms with the pass behind the update, 19.0 without).
static double *spare_region(const PolarWs &w, int64_t count)
{
    return 2 * (size_t)count <= w.parts_floats ? (double *)w.parts : nullptr;
}

// Where the partials of a launch of tiles_m x tiles_n tiles go; without room for them
// the launch has none and step_norm_after writes others behind it.
template <class Ws>
static double *step_norm_room(const GemmDesc &d, const Ws &w, StepNorm *norm)
{
    norm->count = (int64_t)d.tiles_m * d.tiles_n;
    double *to = step_room(norm->count, w.tiles, w.sumsq, sumsq_num_partials())
                     ? w.tiles
                     : spare_region(w, norm->count);
    norm->parts = to;
    return to;
}

template <class Ws>
static hipError_t step_norm_after(const GemmDesc &d, const Ws &w, StepNorm *norm, hipStream_t s)
{
    if (norm->parts) {
        norm->count = (int64_t)d.tiles_m * d.tiles_n;   // (packed operands: other tiles)
        return hipSuccess;
    }
    norm->parts = w.sumsq;
    norm->count = sumsq_num_partials();
    return launch_diff_sumsq(d.C, d.ldc, d.E, d.lde, d.M, d.N, w.sumsq, s);
}

// Xn <- alpha X P + beta X, with the partials of (Xn - X)^2 if norm is not null.
static hipError_t update_step(const PolarPlan &p, int prec, const float *X, int64_t ldx,
                              const float *P, double alpha, double beta, float *Xn, int64_t ldxn,
                              StepNorm *norm, const PolarWs &w, hipStream_t s,
                              const int *stop = nullptr, const ChainStep *cs = nullptr)
{
    const int64_t m = p.m, n = p.n;
    GemmDesc d;
    memset(&d, 0, sizeof d);
    d.A = X;
    d.lda = ldx;
    d.a_kcontig = 1;
    d.B = P;
    d.ldb = n;
    d.b_kcontig = 0;
    d.M = m;
    d.N = n;
    d.K = n;
    const int splits = update_splits(p);
    if (splits > 1 && (size_t)splits * m * n <= w.parts_floats) {
        // K-slices into m x n parts, added in FP64 with the update applied
        d.C = w.parts;
        d.ldc = n;
        d.alpha = 1.0f;
        gemm_f16_scales(d, prec, kIterScale, kIterScale);
        gemm_finalize(d, prec);
        d.slices = slice_plan(n, splits, &d.slice_k);
        d.slice_stride = m * n;
        hipError_t e = gemm_packed_or_plain(prec, d, w.pk, s);
        if (e != hipSuccess)
            return e;
        if (norm)
            *norm = StepNorm{w.tiles, splitk_update_num_partials()};
        return launch_splitk_update_reduce(w.parts, d.slices, m, n, alpha, beta,
                                           beta != 0.0 ? X : nullptr, ldx, Xn, ldxn,
                                           norm ? w.tiles : nullptr, s);
    }
    d.C = Xn;
    d.ldc = ldxn;
    d.alpha = (float)alpha;
    if (beta != 0.0) {
        d.E = X;
        d.lde = ldx;
        d.beta = (float)beta;
    }
    d.stop = stop;
    gemm_f16_scales(d, prec, kIterScale, kIterScale);
    gemm_finalize(d, prec);
    if (norm)
        d.partials = step_norm_room(d, w, norm);
    if (cs) {
        d.pack_row = w.chain.row[cs->cur ^ 1];
        d.pack_col = w.chain.col;
        d.pack_prec = cs->next_prec;
        d.pack_scale = kIterScale;
        if (cs->only)
            d.C = nullptr;
        if (cs->packed) {
            d.A = (const float *)w.chain.row[cs->cur];
            d.B = (const float *)w.chain.P;
            d.b_pairs = 1;
        }
    }
    const hipError_t e = cs && cs->packed ? launch_gemm_packed(prec, d, s)
                                          : gemm_packed_or_plain(prec, d, w.pk, s);
    return e == hipSuccess && norm ? step_norm_after(d, w, norm, s) : e;
}

// Newton-Schulz (inversion) steps queued before the first look at the stop test, and
// between later ones: well-conditioned inputs stop within the first batch.
constexpr int kFirstBatch = 10, kNextBatch = 4;
constexpr int kFirstInvBatch = 16;

// Whether every step of p runs on the direct kernels: launches short enough that
// the host's turn between steps would take longer, so the steps are queued ahead of
// their stop test.  (With polish the step after the stop differs, so those wait.)
static bool queues_ahead(const PolarPlan &p)
{
    return !p.polish && update_splits(p) <= 1 && is_direct(update_shape(p, p.prec_pre).small) &&
           is_direct(update_shape(p, p.prec_ns).small);
}

// H = (U^T A + A^T U) / 2 in one symmetric pass: the upper triangle of U^T A
// and of A^T U = (U^T A)^T are accumulated as Gram-mode slices (each of at most
// kMaxAccK rows of the K = m sum), and the 2 s slices are added in FP64 with
// the factor 1/2 and written to both triangles, so H is exactly symmetric.
static hipError_t h_step(const PolarPlan &p, const float *U, int64_t ldu, const float *A,
                         int64_t lda, double fro, float *H, int64_t ldh, const PolarWs &w,
                         hipStream_t s)
{
    const int64_t n = p.n;
    const int want = h_splits(p);
    float sc = 1.0f;
    const int prec = h_prec(p.prec_h, fro, &sc);
    int c1 = 0, c2 = 0;
    hipError_t e = gram_slices(prec, U, ldu, kIterScale, A, lda, sc, p.m, n, want, w.parts, &c1, s);
    if (e != hipSuccess)
        return e;
    e = gram_slices(prec, A, lda, sc, U, ldu, kIterScale, p.m, n, want,
                    w.parts + (size_t)c1 * n * n, &c2, s);
    if (e != hipSuccess)
        return e;
    return launch_splitk_sym_reduce(w.parts, n * n, c1 + c2, n, 0.5, 0.0, H, ldh, s);
}

// ------------------------------------------------------------------ inverse

// Algorithm NS_Inverse (section III.D) for an n x m A: X0 = A^T / ||A A^T||_F,
// X' = X (2I - A X) = (2I - X A) X.  The step forms the smaller product:
// A X (n x n) when n <= m, X A (m x m) when n > m.
struct InvPlan {
    int64_t n, m;
    int64_t r;       // side of the formed product
    int wide;        // 1: n <= m (forms A X); 0: n > m (forms X A)
    double eps;
    int max_iter, polish, literal, f16_polish;
    int prec;
};

static la_status inverse_plan(int64_t n, int64_t m, const la_inverse_opts *opts, InvPlan *out)
{
    if (n < 1 || m < 1) {
        set_error("la_inverse: sizes must be positive (n %lld, m %lld)", (long long)n,
                  (long long)m);
        return LA_ERR_SHAPE;
    }
    la_inverse_opts o;
    memset(&o, 0, sizeof o);
    if (opts)
        o = *opts;
    if (!valid_prec(o.prec)) {
        set_error("la_inverse: unknown precision %d", o.prec);
        return LA_ERR_INVALID_ARG;
    }
    if (!(o.eps >= 0.0) || !isfinite(o.eps) || o.max_iter < 0) {
        set_error("la_inverse: bad eps or max_iter");
        return LA_ERR_INVALID_ARG;
    }
    InvPlan p;
    p.n = n;
    p.m = m;
    p.wide = n <= m;
    p.r = p.wide ? n : m;
    p.eps = o.eps > 0.0 ? o.eps : ldexp(1.0, -24);
    p.max_iter = o.max_iter > 0 ? o.max_iter : 100;
    // AUTO: 3xBF16 steps, then one at FP32 level (6xBF16, or F16X3 on the larger
    // sizes: polish_f16).  Forming I - A X near the fixed point cancels to O(1) from
    // terms of size ~cond(A), so the dropped lo*lo products of 3xBF16 (2^-18
    // relative) limit its accuracy; the iteration converges quadratically, so one
    // such step restores FP32-level accuracy.
    p.polish = o.polish != 0 || o.prec == LA_PREC_AUTO;
    p.f16_polish = o.prec == LA_PREC_AUTO;
    p.literal = o.literal_delta != 0;
    p.prec = resolve_prec(o.prec, PREC_BF16X3);
    *out = p;
    return LA_OK;
}

struct InvWs {
    float *X;        // m x n, ld n: the iterate's second buffer
    float *R;        // r x r: the Gram A A^T (or A^T A), then I - A X (or I - X A)
    double *tiles;   // per-tile step-norm partials
    double *sumsq;   // norm partials, then the rest of the step-norm partials
    double *scal;    // [0] ||A A^T||_F^2, [1] ||X' - X||_F^2
    PackBuf pk;      // packed operands of the step's products
    char *pka;       // A packed once for the first product (may be null)
    // F16X3 polish: maxima of a product's rows and columns (may be null: 6xBF16); answer
    // and counts of unevenness (A's, then X's)
    uint32_t *mx, *counts;
    int *uneven;
};
constexpr size_t kFlagWords = 64;
static double *spare_region(const InvWs &, int64_t) { return nullptr; }

// Packed operands of the larger of the two products of a step: R = A X
// (r x r, K = m) or X A (K = n), then X R (m x n, K = n) or R X (K = m);
// and A itself, packed once, as op(A) of A X or op(B)^T of X A (r rows, K = m
// or n).
static size_t inverse_step_pack_bytes(const InvPlan &p)
{
    const int64_t k1 = p.wide ? p.m : p.n, k2 = p.wide ? p.n : p.m;
    return std::max(pack_bytes(p.prec, p.r, p.r, k1), pack_bytes(p.prec, p.m, p.n, k2));
}

static size_t inverse_a_pack_bytes(const InvPlan &p)
{
    const int64_t k1 = p.wide ? p.m : p.n;
    return packs(p.prec, p.r, p.r, k1) ? align_up256(packed_x3_bytes(p.r, k1)) : 0;
}

static size_t inverse_pack_bytes(const InvPlan &p)
{
    return inverse_step_pack_bytes(p) + inverse_a_pack_bytes(p);
}

// The same regions with products of the small class too, where those need more (used
// where the workspace has room, as la_polar's).
static size_t inverse_small_step_bytes(const InvPlan &p)
{
    const int64_t k1 = p.wide ? p.m : p.n, k2 = p.wide ? p.n : p.m;
    const size_t have = inverse_step_pack_bytes(p);
    const size_t b = std::max(have, std::max(pack_small_bytes(p.prec, p.r, p.r, k1),
                                             pack_small_bytes(p.prec, p.m, p.n, k2)));
    return b > have ? b : 0;
}

static size_t inverse_small_a_bytes(const InvPlan &p)
{
    const int64_t k1 = p.wide ? p.m : p.n;
    return pack_small_bytes(p.prec, p.r, p.r, k1) ? align_up256(packed_x3_bytes(p.r, k1)) : 0;
}

static size_t inverse_small_pack_bytes(const InvPlan &p)
{
    return inverse_small_step_bytes(p) + inverse_small_a_bytes(p);
}

// Whether an M x N x K product of AUTO's polish step runs as F16X3, each row of
// op(A) and column of op(B) scaled by its own largest entry, instead of 6xBF16:
// where the step's products pack (pk) and K is deep enough, as for the matrix
// functions, that its fewer accumulation roundings outweigh one bit less per
// operand.  (3000^2: a product 438 us at 6xBF16, 160 and 70 for the maxima and packs,
// the inverse 7.72 -> 7.21 ms; its error at cond 10 1.17e-6 -> 8.9e-7, cond 30 2.27e-6
// -> 1.66e-6.)  A and X, one of which is in each product, have to be even for it
// (PackCheck); an input where they are not is polished once more, at 6xBF16.
static bool polish_f16(const InvPlan &p, const GemmDesc &d)
{
    return p.f16_polish && d.K >= 1024 &&
           ((!d.small && packs(PREC_F16X3, d.M, d.N, d.K)) || packs_small(PREC_F16X3, d));
}

// Bytes of the maxima those products need (part of the size asked for; a workspace
// without them polishes at 6xBF16).
static size_t inverse_max_bytes(const InvPlan &p)
{
    return p.f16_polish && (inverse_step_pack_bytes(p) || inverse_small_step_bytes(p))
               ? 2 * align_up256((size_t)std::max(p.m, p.n) * sizeof(uint32_t)) +
                     align_up256((kFlagWords + 2 * (size_t)(p.m + p.n)) * sizeof(uint32_t))
               : 0;
}

static size_t inverse_workspace_bytes(const InvPlan &p)
{
    size_t b = 0;
    b += align256((size_t)p.m * p.n * sizeof(float));
    b += align256((size_t)p.r * p.r * sizeof(float));
    b += align256(step_partials(p.m, p.n) * sizeof(double));
    b += align256((size_t)sumsq_num_partials() * sizeof(double));
    b += align256(8 * sizeof(double));
    b += inverse_pack_bytes(p);
    return b;
}

static InvWs inverse_carve(const InvPlan &p, void *ws, bool room, bool max_room)
{
    InvWs w;
    char *b = (char *)ws;
    char *mb = b + inverse_workspace_bytes(p) + inverse_small_pack_bytes(p);
    w.mx = max_room ? (uint32_t *)mb : nullptr;
    mb += 2 * align_up256((size_t)std::max(p.m, p.n) * sizeof(uint32_t));
    w.uneven = (int *)mb;
    w.counts = (uint32_t *)mb + kFlagWords;
    w.X = (float *)b;
    b += align256((size_t)p.m * p.n * sizeof(float));
    w.R = (float *)b;
    b += align256((size_t)p.r * p.r * sizeof(float));
    w.tiles = (double *)b;
    b += align256(step_partials(p.m, p.n) * sizeof(double));
    w.sumsq = (double *)b;
    b += align256((size_t)sumsq_num_partials() * sizeof(double));
    w.scal = (double *)b;
    b += align256(8 * sizeof(double));
    w.pk.bytes = inverse_step_pack_bytes(p);
    w.pk.p = w.pk.bytes ? b : nullptr;
    b += w.pk.bytes;
    w.pka = inverse_a_pack_bytes(p) ? b : nullptr;
    b += inverse_a_pack_bytes(p);
    if (room && inverse_small_step_bytes(p)) {
        w.pk.p = b;
        w.pk.bytes = inverse_small_step_bytes(p);
    }
    if (room && inverse_small_a_bytes(p))
        w.pka = b + inverse_small_step_bytes(p);
    return w;
}

// Whether the steps' updates run on the direct kernels, so that they are queued
// ahead of their stop test as la_polar's are.
static bool queues_ahead(const InvPlan &p)
{
    GemmDesc u;
    memset(&u, 0, sizeof u);
    u.M = p.m;
    u.N = p.n;
    u.K = p.wide ? p.n : p.m;
    gemm_finalize(u, p.prec);
    return is_direct(u.small);
}

// A product of the polish step (op(A) k contiguous, op(B) row-contiguous) as F16X3,
// packed into w.pk, unless *w.uneven; A or X is op(A) (p.wide) or op(B).
static hipError_t polish_product(const InvPlan &p, GemmDesc &d, const InvWs &w, uint32_t *counts,
                                 hipStream_t s)
{
    uint32_t *ra = w.mx, *cb = w.mx + align_up256((size_t)std::max(p.m, p.n) * 4) / 4;
    char *pa = w.pk.p, *pb = w.pk.p + align_up256(packed_x3_bytes(d.M, d.K));
    hipError_t e = launch_absmax(d.A, d.lda, d.M, d.K, 1, ra, s);
    if (e == hipSuccess)
        e = launch_absmax(d.B, d.ldb, d.K, d.N, 0, cb, s);
    const PackCheck check{counts, w.uneven, 1};
    if (e == hipSuccess)
        e = launch_pack(PREC_F16X3, d.A, d.lda, 1, d.M, d.K, 1.0f, pa, s, ra, nullptr,
                        p.wide ? check : PackCheck());
    if (e == hipSuccess)
        e = launch_pack(PREC_F16X3, d.B, d.ldb, 0, d.N, d.K, 1.0f, pb, s, cb, nullptr,
                        p.wide ? PackCheck() : check);
    if (e != hipSuccess)
        return e;
    d.stop = w.uneven;
    d.A = (const float *)pa;
    d.B = (const float *)pb;
    d.row_max = ra;
    d.col_max = cb;
    gemm_set_packed(d);
    return launch_gemm_packed(PREC_F16X3, d, s);
}

// One step X' = X + X (I - A X)  (wide / square)  or  X + (I - X A) X  (tall),
// with FP64 partials of (X' - X)^2.
static hipError_t inverse_step(const InvPlan &p, int prec, const float *A, int64_t lda,
                               const float *X, int64_t ldx, float *Xn, int64_t ldxn,
                               const InvWs &w, StepNorm *norm, hipStream_t s,
                               const int *stop = nullptr)
{
    GemmDesc d;
    memset(&d, 0, sizeof d);
    d.C = w.R;
    d.ldc = p.r;
    d.M = p.r;
    d.N = p.r;
    d.alpha = -1.0f;
    d.gamma = 1.0f;
    if (p.wide) {               // R = I - A X: A (n x m) . X (m x n)
        d.A = A;
        d.lda = lda;
        d.a_kcontig = 1;
        d.B = X;
        d.ldb = ldx;
        d.b_kcontig = 0;
        d.K = p.m;
    } else {                    // R = I - X A: X (m x n) . A (n x m)
        d.A = X;
        d.lda = ldx;
        d.a_kcontig = 1;
        d.B = A;
        d.ldb = lda;
        d.b_kcontig = 0;
        d.K = p.n;
    }
    d.stop = stop;
    gemm_finalize(d, prec);
    // A was packed once for the step precision (the polish step packs its own)
    const char *pre = prec == p.prec ? w.pka : nullptr;
    auto f16 = [&](GemmDesc &g) {
        if (prec != PREC_BF16X6 || !w.mx ||
            align_up256(packed_x3_bytes(g.M, g.K)) + align_up256(packed_x3_bytes(g.N, g.K)) >
                w.pk.bytes)
            return false;
        GemmDesc t = g;
        gemm_finalize(t, PREC_F16X3);
        if (!polish_f16(p, t))
            return false;
        g = t;
        return true;
    };
    hipError_t e = f16(d) ? polish_product(p, d, w, w.counts, s)
                          : gemm_packed_or_plain(prec, d, w.pk, s, p.wide ? pre : nullptr,
                                                 p.wide ? nullptr : pre);
    if (e != hipSuccess)
        return e;

    GemmDesc u;
    memset(&u, 0, sizeof u);
    u.C = Xn;
    u.ldc = ldxn;
    u.M = p.m;
    u.N = p.n;
    u.alpha = 1.0f;
    u.beta = 1.0f;
    u.E = X;
    u.lde = ldx;
    if (p.wide) {               // X' = X + X R: X (m x n) . R (n x n)
        u.A = X;
        u.lda = ldx;
        u.a_kcontig = 1;
        u.B = w.R;
        u.ldb = p.r;
        u.b_kcontig = 0;
        u.K = p.n;
    } else {                    // X' = X + R X: R (m x m) . X (m x n)
        u.A = w.R;
        u.lda = p.r;
        u.a_kcontig = 1;
        u.B = X;
        u.ldb = ldx;
        u.b_kcontig = 0;
        u.K = p.m;
    }
    u.stop = stop;
    gemm_finalize(u, prec);
    const bool fp16 = f16(u);
    u.partials = step_norm_room(u, w, norm);
    e = fp16 ? polish_product(p, u, w, w.counts + p.m + p.n, s)
             : gemm_packed_or_plain(prec, u, w.pk, s);
    return e == hipSuccess ? step_norm_after(u, w, norm, s) : e;
}

// Tile class of a caller's product whose 64 x 64 tiles take a third (FP32: also a fifth
// or sixth) round of workgroups, one per CU each: 128 x 128 tiles instead unless K is
// long enough to repay that round.  (us, direct / small, NN where not named: 1500^2 x 64
// 3xBF16 17.0 / 12.8, x 256 22.9 / 18.9, x 640 31.5 / 31.2, x 2000 67 / 82, NT 76 / 82;
// 6xBF16 x 256 24.1 / 22.3, x 600 36 / 39, x 2000 84 / 99, 1536^2 x 2048 NT 98 / 84; FP32
// 529 tiles x 256 30.0 / 29.2, x 600 55 / 58, 576 tiles x 600 71 / 58, x 2000 163 / 168,
// 1521 tiles x 256 58 / 52, x 1200 195 / 200.)  3xBF16 has one line for all layouts,
// since la_gemm_packed gives the same bits for each.  The steps of the iterations keep
// the direct class there, which lets them be queued ahead of their stop test.
static void gemm_last_round(GemmDesc &d, int prec)
{
    constexpr int64_t kCus = 256;
    const int64_t tiles = (int64_t)d.tiles_m * d.tiles_n;
    if (d.small != kClassDirect64 || std::min(d.M, d.N) < 128 || tiles <= 2 * kCus)
        return;
    const bool nt = d.a_kcontig && d.b_kcontig, tn = !d.a_kcontig && !d.b_kcontig;
    int64_t min_k;
    if (prec != PREC_FP32)
        min_k = prec != PREC_BF16X6 ? 640 : nt ? INT64_MAX : 320;
    else if (2 * tiles <= 5 * kCus)
        min_k = 256 + (nt ? 8 : tn ? 10 : 16) * std::max<int64_t>(0, tiles - 520);
    else
        min_k = 256 + 2 * std::max<int64_t>(0, tiles - 1089);
    if (d.K < min_k)
        gemm_set_class(d, prec, kClassSmall);
}

// Tile class of a product of packed operands: the direct class that la_gemm takes
// for the shape (the same sums), else the tile side of gemm_set_packed.
static void gemm_packed_class(GemmDesc &d)
{
    gemm_finalize(d, PREC_BF16X3);
    gemm_last_round(d, PREC_BF16X3);
    gemm_set_packed(d);
}

// Tile class of an unpacked product that qualifies for 256 x 256 tiles: 128 x 128 ones
// (the same sums) where their rounds, two workgroups per CU, come out cheaper.  A
// round of the large ones starts and ends with nothing beside it on its CU, 33 us
// that a short K does not repay.  Microseconds a round, measured from K = 64 to 1600
// on five shapes (3xBF16, large / small: 3392 x 4672 x 91 53 / 32 us, 8000^2 x 400 246 / 219,
// 2900 x 12000 x 800 280 / 219, 8000^2 x 800 370 / 383, x 1600 642 / 712).
static void gemm_pick_tiles(GemmDesc &d, int prec)
{
    if (d.small != kClassLarge || d.gram)
        return;
    double l0 = 33.5, lk = 0.0788, s0 = 8.3, sk = 0.0575;   // 3xBF16
    if (prec == PREC_FP32)
        l0 = 40.0, lk = 0.2535, s0 = 9.5, sk = 0.146;
    else if (prec == PREC_BF16X6)
        l0 = 32.5, lk = 0.1207, s0 = 6.0, sk = 0.0826;
    auto tiles = [&](int64_t t) { return ((d.M + t - 1) / t) * ((d.N + t - 1) / t); };
    // (the small ones start as others end, so a last partial round counts in part)
    const double rl = (double)((tiles(256) + 255) / 256), rs = std::max(1.0, tiles(128) / 512.0);
    if (rs * (s0 + sk * d.K) < 0.97 * rl * (l0 + lk * d.K))
        gemm_set_class(d, prec, kClassSmall);
}

// Validation and descriptor of a la_gemm-style call.  *empty: nothing to do
// (m or n is 0) after successful validation.
static la_status gemm_prepare(const char *who, la_context *ctx, int trans_a, int trans_b,
                              int64_t m, int64_t n, int64_t k, float alpha, const float *A,
                              int64_t lda, const float *B, int64_t ldb, float beta, float *C,
                              int64_t ldc, int prec, GemmDesc *out, int *prec_out, bool *empty)
{
    *empty = false;
    if (!valid_prec(prec)) {
        set_error("%s: invalid precision %d", who, prec);
        return LA_ERR_INVALID_ARG;
    }
    if (m < 0 || n < 0 || k < 0) {
        set_error("%s: negative size", who);
        return LA_ERR_SHAPE;
    }
    const int64_t a_cols = trans_a ? m : k, a_rows = trans_a ? k : m;
    const int64_t b_cols = trans_b ? k : n, b_rows = trans_b ? n : k;
    if (lda < std::max<int64_t>(a_cols, 1) || ldb < std::max<int64_t>(b_cols, 1) ||
        ldc < std::max<int64_t>(n, 1)) {
        set_error("%s: leading dimension smaller than the row length", who);
        return LA_ERR_SHAPE;
    }
    if (!ctx) {
        set_error("%s: ctx is NULL", who);
        return LA_ERR_INVALID_ARG;
    }
    if (m == 0 || n == 0) {
        *empty = true;
        return LA_OK;
    }
    if (!C || (k > 0 && (!A || !B))) {
        set_error("%s: NULL matrix pointer", who);
        return LA_ERR_INVALID_ARG;
    }
    const size_t cb = extent_bytes(m, n, ldc);
    if (k > 0 && (overlaps(C, cb, A, extent_bytes(a_rows, a_cols, lda)) ||
                  overlaps(C, cb, B, extent_bytes(b_rows, b_cols, ldb)))) {
        set_error("%s: C overlaps A or B", who);
        return LA_ERR_INVALID_ARG;
    }
    LA_HIP(hipSetDevice(ctx->device), "la_gemm: hipSetDevice");
    const int p = resolve_prec(prec, PREC_BF16X3);
    GemmDesc d;
    memset(&d, 0, sizeof d);
    d.A = A;
    d.lda = lda;
    d.a_kcontig = trans_a ? 0 : 1;
    d.B = B;
    d.ldb = ldb;
    d.b_kcontig = trans_b ? 1 : 0;
    d.C = C;
    d.ldc = ldc;
    d.M = m;
    d.N = n;
    d.K = k;
    d.alpha = alpha;
    if (beta != 0.0f) {
        d.E = C;
        d.lde = ldc;
        d.beta = beta;
    }
    gemm_finalize(d, p);
    gemm_last_round(d, p);
    *out = d;
    *prec_out = p;
    return LA_OK;
}

}  // namespace la

using namespace la;

extern "C" {

const char *la_status_string(la_status s)
{
    switch (s) {
    case LA_OK: return "LA_OK";
    case LA_ERR_INVALID_ARG: return "LA_ERR_INVALID_ARG";
    case LA_ERR_SHAPE: return "LA_ERR_SHAPE";
    case LA_ERR_NONFINITE: return "LA_ERR_NONFINITE";
    case LA_ERR_NOT_CONVERGED: return "LA_ERR_NOT_CONVERGED";
    case LA_ERR_OUT_OF_MEMORY: return "LA_ERR_OUT_OF_MEMORY";
    case LA_ERR_DEVICE: return "LA_ERR_DEVICE";
    case LA_ERR_QUEUE_FULL: return "LA_ERR_QUEUE_FULL";
    case LA_ERR_TOO_LARGE: return "LA_ERR_TOO_LARGE";
    case LA_ERR_NOT_READY: return "LA_ERR_NOT_READY";
    case LA_ERR_UNKNOWN_REQUEST: return "LA_ERR_UNKNOWN_REQUEST";
    case LA_ERR_BREAKDOWN: return "LA_ERR_BREAKDOWN";
    }
    return "LA_ERR_UNKNOWN_STATUS";
}

const char *la_last_error(void) { return g_err; }

la_status la_create(int device, la_context **out)
{
    g_err[0] = 0;
    if (!out) {
        set_error("la_create: out is NULL");
        return LA_ERR_INVALID_ARG;
    }
    int count = 0;
    hipError_t e = hipGetDeviceCount(&count);
    if (e != hipSuccess || count == 0) {
        set_error("la_create: no HIP device (%s)", hipGetErrorString(e));
        return LA_ERR_DEVICE;
    }
    if (device < 0 || device >= count) {
        set_error("la_create: device %d out of range [0, %d)", device, count);
        return LA_ERR_INVALID_ARG;
    }
    hipDeviceProp_t prop;
    e = hipGetDeviceProperties(&prop, device);
    if (e != hipSuccess)
        return dev_fail(e, "la_create: hipGetDeviceProperties");
    if (strncmp(prop.gcnArchName, "gfx950", 6) != 0) {
        set_error("la_create: device %d is %s; this library is built for gfx950 only", device,
                  prop.gcnArchName);
        return LA_ERR_DEVICE;
    }
    if (device >= kMaxDevices) {
        set_error("la_create: device %d beyond the %d this library tracks", device, kMaxDevices);
        return LA_ERR_INVALID_ARG;
    }
    // the static workspace's address on this device, with the device current
    // (the caller's current device is restored)
    int prev = -1;
    e = hipGetDevice(&prev);
    if (e != hipSuccess)
        return dev_fail(e, "la_create: hipGetDevice");
    e = hipSetDevice(device);
    if (e != hipSuccess)
        return dev_fail(e, "la_create: hipSetDevice");
    void *sp = nullptr;
    e = scratch_address(device, &sp);
    const hipError_t e2 = hipSetDevice(prev);
    if (e != hipSuccess)
        return dev_fail(e, "la_create: hipGetSymbolAddress(scratch)");
    if (e2 != hipSuccess)
        return dev_fail(e2, "la_create: restoring the current device");
    la_context *c = new (std::nothrow) la_context;
    if (!c) {
        set_error("la_create: out of host memory");
        return LA_ERR_OUT_OF_MEMORY;
    }
    c->device = device;
    c->num_cus = prop.multiProcessorCount;
    c->scratch = sp;
    *out = c;
    return LA_OK;
}

la_status la_destroy(la_context *ctx)
{
    delete ctx;
    return LA_OK;
}

la_status la_gemm(la_context *ctx, int trans_a, int trans_b, int64_t m, int64_t n, int64_t k,
                  float alpha, const float *A, int64_t lda, const float *B, int64_t ldb,
                  float beta, float *C, int64_t ldc, la_precision prec, void *hip_stream)
{
    g_err[0] = 0;
    GemmDesc d;
    int p = 0;
    bool empty = false;
    la_status st = gemm_prepare("la_gemm", ctx, trans_a, trans_b, m, n, k, alpha, A, lda, B, ldb,
                                beta, C, ldc, prec, &d, &p, &empty);
    if (st != LA_OK || empty)
        return st;
    gemm_pick_tiles(d, p);
    LA_HIP(launch_gemm(p, d, (hipStream_t)hip_stream), "la_gemm: launch");
    return LA_OK;
}

size_t la_pack_size(int64_t rows, int64_t k)
{
    if (rows < 0 || k < 0)
        return 0;
    return packed_x3_bytes(rows, k);
}

la_status la_pack_bf16x3(la_context *ctx, int kc, int64_t rows, int64_t k, const float *X,
                         int64_t ld, void *packed, size_t packed_bytes, void *hip_stream)
{
    g_err[0] = 0;
    if (rows < 0 || k < 0 || ld < std::max<int64_t>(kc ? k : rows, 1)) {
        set_error("la_pack_bf16x3: bad shape (rows %lld, k %lld, ld %lld)", (long long)rows,
                  (long long)k, (long long)ld);
        return LA_ERR_SHAPE;
    }
    if (!ctx || (rows > 0 && k > 0 && (!X || !packed))) {
        set_error("la_pack_bf16x3: NULL argument");
        return LA_ERR_INVALID_ARG;
    }
    const size_t need = packed_x3_bytes(rows, k);
    if (packed_bytes < need) {
        set_error("la_pack_bf16x3: buffer %zu bytes, need %zu", packed_bytes, need);
        return LA_ERR_OUT_OF_MEMORY;
    }
    if (need == 0)
        return LA_OK;
    if (overlaps(packed, need, X, extent_bytes(kc ? rows : k, kc ? k : rows, ld))) {
        set_error("la_pack_bf16x3: output overlaps X");
        return LA_ERR_INVALID_ARG;
    }
    LA_HIP(hipSetDevice(ctx->device), "la_pack_bf16x3: hipSetDevice");
    LA_HIP(launch_pack(PREC_BF16X3, X, ld, kc ? 1 : 0, rows, k, 1.0f, packed,
                       (hipStream_t)hip_stream),
           "la_pack_bf16x3: launch");
    return LA_OK;
}

la_status la_gemm_packed(la_context *ctx, int64_t m, int64_t n, int64_t k, float alpha,
                         const void *Ap, const void *Bp, float beta, float *C, int64_t ldc,
                         void *hip_stream)
{
    g_err[0] = 0;
    if (m < 0 || n < 0 || k < 0 || ldc < std::max<int64_t>(n, 1)) {
        set_error("la_gemm_packed: bad shape");
        return LA_ERR_SHAPE;
    }
    if (!ctx) {
        set_error("la_gemm_packed: ctx is NULL");
        return LA_ERR_INVALID_ARG;
    }
    if (m == 0 || n == 0)
        return LA_OK;
    if (!C || (k > 0 && (!Ap || !Bp))) {
        set_error("la_gemm_packed: NULL argument");
        return LA_ERR_INVALID_ARG;
    }
    const size_t cb = extent_bytes(m, n, ldc);
    if (k > 0 && (overlaps(C, cb, Ap, packed_x3_bytes(m, k)) ||
                  overlaps(C, cb, Bp, packed_x3_bytes(n, k)))) {
        set_error("la_gemm_packed: C overlaps a packed operand");
        return LA_ERR_INVALID_ARG;
    }
    LA_HIP(hipSetDevice(ctx->device), "la_gemm_packed: hipSetDevice");
    GemmDesc d;
    memset(&d, 0, sizeof d);
    d.A = (const float *)Ap;
    d.B = (const float *)Bp;
    d.C = C;
    d.ldc = ldc;
    d.M = m;
    d.N = n;
    d.K = k;
    d.alpha = alpha;
    if (beta != 0.0f) {
        d.E = C;
        d.lde = ldc;
        d.beta = beta;
    }
    // the class la_gemm takes for this shape, so that the sums are the same; the
    // 128 x 128 class adds as the large tiles do
    gemm_packed_class(d);
    LA_HIP(launch_gemm_packed(PREC_BF16X3, d, (hipStream_t)hip_stream), "la_gemm_packed: launch");
    return LA_OK;
}

size_t la_gemm_workspace_size(int64_t m, int64_t n, int64_t k)
{
    if (m < 0 || n < 0 || k < 0)
        return 0;
    return align256(packed_x3_bytes(m, k)) + align256(packed_x3_bytes(n, k));
}

la_status la_gemm_ws(la_context *ctx, int trans_a, int trans_b, int64_t m, int64_t n, int64_t k,
                     float alpha, const float *A, int64_t lda, const float *B, int64_t ldb,
                     float beta, float *C, int64_t ldc, la_precision prec, void *workspace,
                     size_t ws_bytes, void *hip_stream)
{
    g_err[0] = 0;
    GemmDesc d;
    int p = 0;
    bool empty = false;
    la_status st = gemm_prepare("la_gemm_ws", ctx, trans_a, trans_b, m, n, k, alpha, A, lda, B,
                                ldb, beta, C, ldc, prec, &d, &p, &empty);
    if (st != LA_OK || empty)
        return st;
    hipStream_t s = (hipStream_t)hip_stream;
    // packed path: 3xBF16 on large tiles with enough K to repay the pack pass (the
    // workspace is asked for whatever the smaller side, though one below 256 packs nothing)
    const bool plain = p != PREC_BF16X3 || d.small || k < 256;
    if (plain && !packs(p, m, n, k)) {
        gemm_pick_tiles(d, p);
        LA_HIP(launch_gemm(p, d, s), "la_gemm_ws: launch");
        return LA_OK;
    }
    const size_t pa = align256(packed_x3_bytes(m, k)), need = pa + align256(packed_x3_bytes(n, k));
    if (!workspace || ((uintptr_t)workspace & 255u) != 0) {
        set_error("la_gemm_ws: workspace must be non-NULL and 256-byte aligned");
        return LA_ERR_INVALID_ARG;
    }
    if (ws_bytes < need) {
        set_error("la_gemm_ws: workspace %zu bytes, need %zu", ws_bytes, need);
        return LA_ERR_OUT_OF_MEMORY;
    }
    const int64_t a_cols = trans_a ? m : k, a_rows = trans_a ? k : m;
    const int64_t b_cols = trans_b ? k : n, b_rows = trans_b ? n : k;
    if (overlaps(workspace, need, A, extent_bytes(a_rows, a_cols, lda)) ||
        overlaps(workspace, need, B, extent_bytes(b_rows, b_cols, ldb)) ||
        overlaps(workspace, need, C, extent_bytes(m, n, ldc))) {
        set_error("la_gemm_ws: workspace overlaps A, B or C");
        return LA_ERR_INVALID_ARG;
    }
    if (plain) {
        LA_HIP(launch_gemm(p, d, s), "la_gemm_ws: launch");
        return LA_OK;
    }
    char *wa = (char *)workspace, *wb = wa + pa;
    // op(A) rows are the output rows; op(B)^T rows are the output columns
    LA_HIP(launch_pack(PREC_BF16X3, A, lda, trans_a ? 0 : 1, m, k, 1.0f, wa, s), "la_gemm_ws: pack A");
    LA_HIP(launch_pack(PREC_BF16X3, B, ldb, trans_b ? 1 : 0, n, k, 1.0f, wb, s), "la_gemm_ws: pack B");
    d.A = (const float *)wa;
    d.B = (const float *)wb;
    gemm_set_packed(d);
    LA_HIP(launch_gemm_packed(PREC_BF16X3, d, s), "la_gemm_ws: launch");
    return LA_OK;
}

size_t la_polar_workspace_size(int64_t m, int64_t n, const la_polar_opts *opts)
{
    PolarPlan p;
    if (polar_plan(m, n, opts, &p) != LA_OK)
        return 0;
    return polar_workspace_bytes(p) +
           std::max(packed_small_bytes(p), polar_chain_bytes(p));
}

}  // extern "C"

namespace la {

static la_status polar_impl(la_context *ctx, const PolarPlan &p, const float *A, int64_t lda,
                            float *U, int64_t ldu, float *H, int64_t ldh, void *workspace,
                            size_t ws_bytes, la_polar_info *info, void *hip_stream);

}  // namespace la

extern "C" {

la_status la_polar(la_context *ctx, int64_t m, int64_t n, const float *A, int64_t lda, float *U,
                   int64_t ldu, float *H, int64_t ldh, void *workspace, size_t ws_bytes,
                   const la_polar_opts *opts, la_polar_info *info, void *hip_stream)
{
    g_err[0] = 0;
    PolarPlan p;
    la_status st = polar_plan(m, n, opts, &p);
    if (st != LA_OK)
        return st;
    return polar_impl(ctx, p, A, lda, U, ldu, H, ldh, workspace, ws_bytes, info, hip_stream);
}

la_status la_polar_noalloc(la_context *ctx, int64_t m, int64_t n, const float *A, int64_t lda,
                           float *U, int64_t ldu, float *H, int64_t ldh,
                           const la_polar_opts *opts, la_polar_info *info, void *hip_stream)
{
    g_err[0] = 0;
    PolarPlan p;
    la_status st = polar_plan(m, n, opts, &p);
    if (st != LA_OK)
        return st;
    if (!ctx) {
        set_error("la_polar_noalloc: ctx is NULL");
        return LA_ERR_INVALID_ARG;
    }
    const size_t need = polar_workspace_bytes(p);
    if (need > kScratchBytes) {
        set_error("la_polar_noalloc: a %lld x %lld polar needs %zu bytes of workspace; the "
                  "static buffer holds %zu (use la_polar with a workspace)",
                  (long long)m, (long long)n, need, kScratchBytes);
        return LA_ERR_TOO_LARGE;
    }
    return polar_impl(ctx, p, A, lda, U, ldu, H, ldh, ctx->scratch, kScratchBytes, info,
                      hip_stream);
}

}  // extern "C"

namespace la {

static la_status polar_impl(la_context *ctx, const PolarPlan &plan, const float *A, int64_t lda,
                            float *U, int64_t ldu, float *H, int64_t ldh, void *workspace,
                            size_t ws_bytes, la_polar_info *info, void *hip_stream)
{
    PolarPlan p = plan;
    const int64_t m = p.m, n = p.n;
    if (lda < n || ldu < n || (H && ldh < n)) {
        set_error("la_polar: leading dimension smaller than n");
        return LA_ERR_SHAPE;
    }
    if (!ctx || !A || !U || !workspace) {
        set_error("la_polar: NULL argument");
        return LA_ERR_INVALID_ARG;
    }
    if (((uintptr_t)workspace & 255u) != 0) {
        set_error("la_polar: workspace must be 256-byte aligned");
        return LA_ERR_INVALID_ARG;
    }
    const size_t need = polar_workspace_bytes(p);
    if (ws_bytes < need) {
        set_error("la_polar: workspace %zu bytes, need %zu", ws_bytes, need);
        return LA_ERR_OUT_OF_MEMORY;
    }
    const size_t ab = extent_bytes(m, n, lda), ub = extent_bytes(m, n, ldu);
    const size_t hb = H ? extent_bytes(n, n, ldh) : 0;
    if (overlaps(U, ub, A, ab) || overlaps(U, ub, workspace, need) ||
        (H && (overlaps(H, hb, A, ab) || overlaps(H, hb, U, ub) ||
               overlaps(H, hb, workspace, need)))) {
        set_error("la_polar: U / H overlap A, each other or the workspace");
        return LA_ERR_INVALID_ARG;
    }
    LA_HIP(hipSetDevice(ctx->device), "la_polar: hipSetDevice");
    hipStream_t s = (hipStream_t)hip_stream;
    // the optional region after the required one is used only where it is free
    auto room = [&](size_t extra) {
        const size_t full = need + extra;
        return ws_bytes >= full && !overlaps(workspace, full, A, ab) &&
               !overlaps(workspace, full, U, ub) && !overlaps(workspace, full, H, hb);
    };
    const size_t chain_bytes = polar_chain_bytes(p);
    bool chain = chain_bytes && room(chain_bytes);
    PolarWs w = carve(p, workspace, room(packed_small_bytes(p)), chain);

    la_polar_info inf;
    memset(&inf, 0, sizeof inf);
    inf.prec_precond = public_prec(p.prec_pre);
    inf.prec_ns = public_prec(p.prec_ns);
    inf.prec_h = public_prec(p.prec_h);
    inf.last_delta = INFINITY;
    inf.stop_reason = 2;

    // ping-pong between U (ld ldu) and the workspace copy (ld n)
    float *buf[2] = {U, w.X};
    int64_t ld[2] = {ldu, n};
    int cur = 0;
    double h2[2];
    double fro = 0.0;
    StopState stop;
    bool converged = false, finite = true;

    const bool ahead = queues_ahead(p);
    StepState *st = (StepState *)w.scal;
    StepState h;
    const int *dev_stop = ahead ? &st->stop : nullptr;
    // (a short Gram past the stop costs less than the look at it in every other: P is
    // scratch.  256^2 374 us with the look, 367 without)
    const int *gram_stop = m >= 512 ? dev_stop : nullptr;
    auto bad_norm = [&]() {
        if (info)
            *info = inf;
        set_error("la_polar: ||A||_F = %g (zero or not finite)", fro);
        return LA_ERR_NONFINITE;
    };
    // The norm; an A without one, or one too uneven for the F16X3 phases (the counts are
    // in the second iterate's buffer), stops every later write of queued steps.  Steps
    // that wait for the host take what they need from the readback of the norm.
    auto begin = [&]() {
        LA_HIP(launch_sumsq(A, m, n, lda, w.sumsq, s), "la_polar: norm");
        LA_HIP(launch_norm_state(w.sumsq, sumsq_num_partials(), st, s), "la_polar: norm");
        if (ahead)
            LA_HIP(launch_scale_by_norm(A, lda, buf[0], ld[0], m, n, &st->norm2, s, dev_stop),
                   "la_polar: scale");
        if (uses_f16(p, H != nullptr)) {
            LA_HIP(launch_zero((uint32_t *)w.X, m + n, s), "la_polar: unevenness");
            LA_HIP(launch_uneven(A, lda, m, n, &st->norm2, (uint32_t *)w.X, nullptr, st, s),
                   "la_polar: unevenness");
        }
        return LA_OK;
    };
    auto read_state = [&]() {
        LA_HIP(hipMemcpyAsync(&h, st, sizeof h, hipMemcpyDeviceToHost, s), "la_polar: readback");
        LA_HIP(hipStreamSynchronize(s), "la_polar: sync");
        return LA_OK;
    };
    auto fall_back = [&]() {
        without_f16(p);
        chain = chain && two_term(p.prec_pre);
    };
    la_status rc = begin();
    if (rc != LA_OK)
        return rc;
    if (!ahead) {
        rc = read_state();
        if (rc != LA_OK)
            return rc;
        fro = sqrt(h.norm2);
        inf.fro_norm_a = fro;
        if (!(fro > 0.0) || !isfinite(fro))
            return bad_norm();
        if (h.reason == kReasonUneven)
            fall_back();
        LA_HIP(launch_scale(A, lda, buf[cur], ld[cur], m, n, fro, s), "la_polar: scale");
    }

    // preconditioning: U <- a U (I - c U^T U), c = (4/27) a^2
    // (chained from the second step on: X0 is not there packed)
    ChainStep cs{false, 0, 0, false};
    const ChainStep *csp = nullptr;
    // (an uneven input of queued steps goes through a second time)
    for (bool again = true; again;) {
        cs.packed = false;
        csp = chain ? &cs : nullptr;
        inf.iters_precond = 0;
        for (int i = 0; i < p.k_pre; ++i) {
            cs.cur = cur;
            cs.only = i + 1 < p.k_pre;
            cs.next_prec = cs.only ? p.prec_pre : p.prec_ns;
            LA_HIP(gram_step(p, p.prec_pre, buf[cur], ld[cur], -p.c, 1.0, w.P, w, s, cs.packed,
                             gram_stop),
                   "la_polar: precondition gram");
            LA_HIP(update_step(p, p.prec_pre, buf[cur], ld[cur], w.P, p.a, 0.0, buf[cur ^ 1],
                               ld[cur ^ 1], nullptr, w, s, dev_stop, csp),
                   "la_polar: precondition update");
            cs.packed = chain;
            cur ^= 1;
            inf.iters_precond++;
        }
        cs.next_prec = p.prec_ns;
        cs.only = false;

        // Newton-Schulz: U' = U + U (I - U^T U) / 2, delta = ||U' - U||_F, until the
        // stop test (polar_host.h); a polish step runs at BF16X6
        if (ahead) {
            // Steps are queued in batches; the device applies the stop test after
            // each, and from the stop on leaves the iterates alone.  256^2: 20 us
            // of readback and wait per step saved, 540 -> 360 us for the polar
            // (9 steps), at three launches that leave, 12 us, per step queued in
            // vain (1000^2, where one that runs takes 33 us: 12 too).
            StepTest t;
            t.scale = 1.0;
            t.tol = (double)std::max(m, n) * p.eps;
            t.tol_doubles = 0;
            t.stag_below = p.stagnation ? 1e-2 * sqrt((double)n) : 0.0;
            t.max_steps = p.max_iter;
            const int start = cur;
            int queued = 0, batch = kFirstBatch;
            do {
                for (const int to = std::min(queued + batch, p.max_iter); queued < to; ++queued) {
                    StepNorm norm;
                    cs.cur = cur;
                    LA_HIP(gram_step(p, p.prec_ns, buf[cur], ld[cur], -1.0, 1.0, w.P, w, s,
                                     cs.packed, gram_stop),
                           "la_polar: NS gram");
                    LA_HIP(update_step(p, p.prec_ns, buf[cur], ld[cur], w.P, 0.5, 1.0, buf[cur ^ 1],
                                       ld[cur ^ 1], &norm, w, s, dev_stop, csp),
                           "la_polar: NS update");
                    cs.packed = chain;
                    LA_HIP(launch_step_state(norm.parts, norm.count, st, t, s),
                           "la_polar: delta");
                    cur ^= 1;
                }
                batch = kNextBatch;
                rc = read_state();
                if (rc != LA_OK)
                    return rc;
            } while (!h.stop);
            if (h.reason == kReasonUneven) {
                // nothing after X0 was written: once more from there
                fall_back();
                cur = 0;
                rc = begin();
                if (rc != LA_OK)
                    return rc;
                continue;
            }
            fro = sqrt(h.norm2);
            inf.fro_norm_a = fro;
            if (!(fro > 0.0) || !isfinite(fro)) {
                inf.iters_precond = 0;
                return bad_norm();
            }
            cur = (start + h.steps) & 1;
            inf.iters_ns = h.steps;
            inf.last_delta = h.delta;
            finite = h.reason != 3;
            converged = h.reason < 2;
            if (finite)
                inf.stop_reason = h.reason;
        }
        again = false;
    }
    while (!ahead) {
        const int prec = stop.stopped ? PREC_BF16X6 : p.prec_ns;
        StepNorm norm;
        const bool last = stop.stopped;   // the polish step, from FP32
        cs.cur = cur;
        LA_HIP(gram_step(p, prec, buf[cur], ld[cur], -1.0, 1.0, w.P, w, s, cs.packed && !last),
               "la_polar: NS gram");
        LA_HIP(update_step(p, prec, buf[cur], ld[cur], w.P, 0.5, 1.0, buf[cur ^ 1], ld[cur ^ 1],
                           &norm, w, s, nullptr, last ? nullptr : csp),
               "la_polar: NS update");
        cs.packed = chain;
        LA_HIP(launch_reduce_fixed(norm.parts, norm.count, w.scal + 1, s), "la_polar: delta");
        LA_HIP(hipMemcpyAsync(h2 + 1, w.scal + 1, sizeof(double), hipMemcpyDeviceToHost, s),
               "la_polar: readback");
        LA_HIP(hipStreamSynchronize(s), "la_polar: sync");
        cur ^= 1;
        inf.iters_ns++;
        const double delta = sqrt(h2[1]);
        inf.last_delta = delta;
        if (!isfinite(delta)) {
            finite = false;
            break;
        }
        const StopDecision d = stop_test(p, m, n, delta, stop, inf.iters_ns);
        inf.stop_reason = stop.reason;
        if (d == STOP_DONE) {
            converged = true;
            break;
        }
        if (d == STOP_CAP)
            break;
    }
    if (!finite) {
        if (info)
            *info = inf;
        set_error("la_polar: step norm is not finite");
        return LA_ERR_NONFINITE;
    }
    if (cur != 0)
        LA_HIP(launch_copy(buf[cur], ld[cur], U, ldu, m, n, s), "la_polar: copy");

    if (H)
        LA_HIP(h_step(p, U, ldu, A, lda, fro, H, ldh, w, s), "la_polar: H");
    LA_HIP(hipStreamSynchronize(s), "la_polar: final sync");
    if (info)
        *info = inf;
    if (!converged) {
        set_error("la_polar: no convergence after %d Newton-Schulz steps (delta %g)",
                  inf.iters_ns, inf.last_delta);
        return LA_ERR_NOT_CONVERGED;
    }
    return LA_OK;
}

}  // namespace la

extern "C" {

size_t la_inverse_workspace_size(int64_t n, int64_t m, const la_inverse_opts *opts)
{
    InvPlan p;
    if (inverse_plan(n, m, opts, &p) != LA_OK)
        return 0;
    return inverse_workspace_bytes(p) + inverse_small_pack_bytes(p) + inverse_max_bytes(p);
}

la_status la_inverse(la_context *ctx, int64_t n, int64_t m, const float *A, int64_t lda,
                     float *X, int64_t ldx, void *workspace, size_t ws_bytes,
                     const la_inverse_opts *opts, la_inverse_info *info, void *hip_stream)
{
    g_err[0] = 0;
    InvPlan p;
    la_status st = inverse_plan(n, m, opts, &p);
    if (st != LA_OK)
        return st;
    if (lda < m || ldx < n) {
        set_error("la_inverse: leading dimension too small (lda %lld < m or ldx %lld < n)",
                  (long long)lda, (long long)ldx);
        return LA_ERR_SHAPE;
    }
    if (!ctx || !A || !X || !workspace) {
        set_error("la_inverse: NULL argument");
        return LA_ERR_INVALID_ARG;
    }
    if (((uintptr_t)workspace & 255u) != 0) {
        set_error("la_inverse: workspace must be 256-byte aligned");
        return LA_ERR_INVALID_ARG;
    }
    const size_t need = inverse_workspace_bytes(p);
    if (ws_bytes < need) {
        set_error("la_inverse: workspace %zu bytes, need %zu", ws_bytes, need);
        return LA_ERR_OUT_OF_MEMORY;
    }
    const size_t ab = extent_bytes(n, m, lda), xb = extent_bytes(m, n, ldx);
    if (overlaps(X, xb, A, ab) || overlaps(X, xb, workspace, need)) {
        set_error("la_inverse: X overlaps A or the workspace");
        return LA_ERR_INVALID_ARG;
    }
    LA_HIP(hipSetDevice(ctx->device), "la_inverse: hipSetDevice");
    hipStream_t s = (hipStream_t)hip_stream;
    auto room = [&](size_t extra) {
        return ws_bytes >= need + extra && !overlaps(workspace, need + extra, A, ab) &&
               !overlaps(workspace, need + extra, X, xb);
    };
    const size_t packs_b = inverse_small_pack_bytes(p), max_b = inverse_max_bytes(p);
    InvWs w = inverse_carve(p, workspace, room(packs_b), max_b && room(packs_b + max_b));

    la_inverse_info inf;
    memset(&inf, 0, sizeof inf);
    inf.product_side = p.wide;
    inf.prec = p.prec;
    inf.last_delta = INFINITY;
    inf.stop_reason = 2;

    // a = ||A A^T||_F = ||A^T A||_F, from the smaller symmetric Gram (FP64 norm)
    {
        GemmDesc g;
        memset(&g, 0, sizeof g);
        g.A = A;
        g.B = A;
        g.lda = lda;
        g.ldb = lda;
        g.C = w.R;
        g.ldc = p.r;
        g.M = p.r;
        g.N = p.r;
        g.alpha = 1.0f;
        g.gram = 1;
        if (p.wide) {           // A A^T: op(A)(i, k) = A[i][k], op(B)(k, j) = A[j][k]
            g.a_kcontig = 1;
            g.b_kcontig = 1;
            g.K = p.m;
        } else {                // A^T A: op(A)(i, k) = A[k][i], op(B)(k, j) = A[k][j]
            g.a_kcontig = 0;
            g.b_kcontig = 0;
            g.K = p.n;
        }
        gemm_finalize(g, p.prec);
        LA_HIP(launch_gemm(p.prec, g, s), "la_inverse: gram");
    }
    double h2[2];
    LA_HIP(launch_sumsq(w.R, p.r, p.r, p.r, w.sumsq, s), "la_inverse: norm");
    LA_HIP(launch_reduce_fixed(w.sumsq, sumsq_num_partials(), w.scal, s), "la_inverse: norm");
    LA_HIP(hipMemcpyAsync(h2, w.scal, sizeof(double), hipMemcpyDeviceToHost, s),
           "la_inverse: readback");
    LA_HIP(hipStreamSynchronize(s), "la_inverse: sync");
    const double a = sqrt(h2[0]);
    inf.gram_norm = a;
    if (!(a > 0.0) || !isfinite(a)) {
        if (info)
            *info = inf;
        set_error("la_inverse: ||A A^T||_F = %g (zero or not finite)", a);
        return LA_ERR_NONFINITE;
    }

    // X0 = A^T / a; ping-pong between X (ld ldx) and the workspace copy (ld n)
    float *buf[2] = {X, w.X};
    int64_t ld[2] = {ldx, n};
    int cur = 0;
    LA_HIP(launch_transpose_scale(A, lda, buf[cur], ld[cur], n, m, a, s), "la_inverse: X0");
    if (w.pka)   // A as op(A) of A X (k contiguous) or as op(B)^T of X A (k-major)
        LA_HIP(launch_pack(p.prec, A, lda, p.wide ? 1 : 0, p.r, p.wide ? p.m : p.n, 1.0f, w.pka, s),
               "la_inverse: pack A");

    const double scale = p.literal ? 1.0 : sqrt(a);
    double eps = p.eps;
    const int total = p.max_iter + (p.polish ? 1 : 0);
    bool stopped = false, finite = true;
    int it = 0;
    if (queues_ahead(p)) {
        // steps queued in batches, the stop test on the device (as in la_polar)
        StepTest t;
        t.scale = scale;
        t.tol = p.eps;
        t.tol_doubles = 1;
        t.stag_below = 0.0;
        t.max_steps = p.max_iter;
        StepState *st = (StepState *)w.scal;
        StepState h;
        LA_HIP(launch_clear_state(st, s), "la_inverse: state");
        int queued = 0, batch = kFirstInvBatch;
        do {
            for (const int to = std::min(queued + batch, p.max_iter); queued < to; ++queued) {
                StepNorm norm;
                const int from = queued & 1;
                LA_HIP(inverse_step(p, p.prec, A, lda, buf[from], ld[from], buf[from ^ 1],
                                    ld[from ^ 1], w, &norm, s, &st->stop),
                       "la_inverse: step");
                LA_HIP(launch_step_state(norm.parts, norm.count, st, t, s), "la_inverse: delta");
            }
            batch = kNextBatch;
            LA_HIP(hipMemcpyAsync(&h, st, sizeof h, hipMemcpyDeviceToHost, s),
                   "la_inverse: readback");
            LA_HIP(hipStreamSynchronize(s), "la_inverse: sync");
        } while (!h.stop);
        cur = h.steps & 1;
        inf.iters = h.steps;
        finite = h.reason != 3;
        stopped = h.reason == 0;
        if (finite) {
            inf.last_delta = h.delta;
            inf.last_tol = ldexp(p.eps, h.steps);
            inf.stop_reason = h.reason;
        }
        it = stopped && p.polish ? h.steps : total;   // what is left: the polish step
    }
    for (; it < total && finite; ++it) {
        const bool polishing = stopped;
        const int prec = polishing ? PREC_BF16X6 : p.prec;
        int uneven = 0;
        StepNorm norm;
        if (polishing && w.mx)
            LA_HIP(launch_zero((uint32_t *)w.uneven, kFlagWords + 2 * (p.m + p.n), s),
                   "la_inverse: unevenness");
        LA_HIP(inverse_step(p, prec, A, lda, buf[cur], ld[cur], buf[cur ^ 1], ld[cur ^ 1], w,
                            &norm, s),
               "la_inverse: step");
        if (polishing && w.mx)
            LA_HIP(hipMemcpyAsync(&uneven, w.uneven, sizeof uneven, hipMemcpyDeviceToHost, s),
                   "la_inverse: readback");
        LA_HIP(launch_reduce_fixed(norm.parts, norm.count, w.scal + 1, s), "la_inverse: delta");
        LA_HIP(hipMemcpyAsync(h2 + 1, w.scal + 1, sizeof(double), hipMemcpyDeviceToHost, s),
               "la_inverse: readback");
        LA_HIP(hipStreamSynchronize(s), "la_inverse: sync");
        if (uneven) {
            w.mx = nullptr;
            --it;
            continue;
        }
        cur ^= 1;
        inf.iters++;
        const double delta = scale * sqrt(h2[1]);
        if (!isfinite(delta)) {
            finite = false;
            break;
        }
        if (polishing)
            break;
        eps *= 2.0;                 // the tolerance grows after every step
        inf.last_delta = delta;
        inf.last_tol = eps;
        if (!(delta > eps)) {
            inf.stop_reason = 0;
            stopped = true;
        }
        if (stopped && !p.polish)
            break;
        if (!stopped && it + 1 >= p.max_iter)
            break;
    }
    if (!finite) {
        if (info)
            *info = inf;
        set_error("la_inverse: step norm is not finite");
        return LA_ERR_NONFINITE;
    }
    if (cur != 0)
        LA_HIP(launch_copy(buf[cur], ld[cur], X, ldx, m, n, s), "la_inverse: copy");
    LA_HIP(hipStreamSynchronize(s), "la_inverse: final sync");
    if (info)
        *info = inf;
    if (!stopped) {
        set_error("la_inverse: tolerance not met after %d steps (delta %g, tol %g)", inf.iters,
                  inf.last_delta, inf.last_tol);
        return LA_ERR_NOT_CONVERGED;
    }
    return LA_OK;
}

}  // extern "C"
