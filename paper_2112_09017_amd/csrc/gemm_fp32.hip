// Instantiates the GEMM kernels (gemm_tile.h, gemm_direct.h) for one precision, all tile
// classes; kept in its own translation unit so the precisions compile in
// parallel.
#include "gemm_direct.h"

namespace la {

hipError_t launch_gemm_fp32(const GemmDesc &d, hipStream_t s)
{
    return dev::launch_any<PREC_FP32>(d, s);
}

hipError_t launch_grouped_fp32(int akc, int bkc, int cls, const GemmDesc *probs,
                             const GroupItem *items, int num_items, hipStream_t s)
{
    return dev::launch_grouped_any<PREC_FP32>(akc, bkc, cls, probs, items, num_items, s);
}

}  // namespace la
