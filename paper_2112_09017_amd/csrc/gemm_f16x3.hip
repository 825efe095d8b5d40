// Instantiates the GEMM kernels (gemm_tile.h, gemm_direct.h) for F16X3 (two scaled fp16 terms per
// operand, three products), all tile classes and the packed operands; kept in
// its own translation unit so the precisions compile in parallel.
#include "gemm_direct.h"

namespace la {

hipError_t launch_gemm_f16(const GemmDesc &d, hipStream_t s)
{
    return dev::launch_any<PREC_F16X3>(d, s);
}

hipError_t launch_grouped_f16(int akc, int bkc, int cls, const GemmDesc *probs,
                              const GroupItem *items, int num_items, hipStream_t s)
{
    return dev::launch_grouped_any<PREC_F16X3>(akc, bkc, cls, probs, items, num_items, s);
}

hipError_t launch_pack_f16(const float *X, int64_t ld, int kc, int64_t rows, int64_t k, float sc,
                           const uint32_t *rmax, void *out, const int *skip,
                           const PackCheck &check, hipStream_t s)
{
    return dev::launch_pack_x3<PREC_F16X3>(X, ld, kc, rows, k, sc, rmax, static_cast<char *>(out),
                                           skip, check, s);
}

hipError_t launch_gemm_packed_f16(const GemmDesc &d, hipStream_t s)
{
    return dev::launch_packed_any<PREC_F16X3>(d, s);
}

}  // namespace la
