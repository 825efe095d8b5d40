// Instantiates the GEMM kernels (gemm_tile.h, gemm_direct.h) for one precision, all tile
// classes; kept in its own translation unit so the precisions compile in
// parallel.
#include "gemm_direct.h"

namespace la {

hipError_t launch_gemm_x3(const GemmDesc &d, hipStream_t s)
{
    return dev::launch_any<PREC_BF16X3>(d, s);
}

hipError_t launch_grouped_x3(int akc, int bkc, int cls, const GemmDesc *probs,
                             const GroupItem *items, int num_items, hipStream_t s)
{
    return dev::launch_grouped_any<PREC_BF16X3>(akc, bkc, cls, probs, items, num_items, s);
}

size_t packed_x3_bytes(int64_t rows, int64_t k) { return dev::packed_bytes(rows, k); }

hipError_t launch_pack_x3(const float *X, int64_t ld, int kc, int64_t rows, int64_t k, void *out,
                          hipStream_t s)
{
    return dev::launch_pack_x3<PREC_BF16X3>(X, ld, kc, rows, k, 1.0f, nullptr,
                                            static_cast<char *>(out), nullptr, PackCheck(), s);
}

hipError_t launch_gemm_packed_x3(const GemmDesc &d, hipStream_t s)
{
    return dev::launch_packed_any<PREC_BF16X3>(d, s);
}

}  // namespace la
