// A grouped launch over problems of the direct classes, whatever their arithmetic
// (two-term or 6xBF16), tile class and operands (FP32 or packed): the server's Gram
// and update of a tick.  Kept in its own translation unit so it compiles beside
// the others.
//
// One launch per arithmetic, class and kind of operand left each of them a part of
// the device and a tail of its own, and joining them on side streams cost the host
// more than the products took (twelve requests of 128^2 to 1536^2: four to six
// launches a phase, 11.6 ms a pass; in one launch 9.3 ms).  Here a
// workgroup of four waves takes any item; a 32 x 32 tile, which eight waves share
// in the launches of one class, has each wave do the work of two in turn, with the
// same sums in the same order.
#include "gemm_direct.h"

namespace la {
namespace dev {

template <int PREC, bool UPDATE, int CLS>
__device__ __forceinline__ void mixed_tile(const GemmDesc &d, int tm, int tn, float *red,
                                           double *red8)
{
    constexpr int V = DirectCfg<CLS>::KW / 4;
    if constexpr (Cfg<PREC>::terms == 2) {
        if (d.packed) {
            direct_packed_tile<PREC, CLS, UPDATE, V>(d, tm, tn, red, red8);
            return;
        }
    }
    direct_tile<PREC, UPDATE, false, CLS, V>(d, tm, tn, 0, d.K, red, red8);
}

// UPDATE: op(A) k contiguous, op(B) row-contiguous (packed: in pair order); else
// both are row-contiguous (packed: in order).  Every branch below is uniform over
// the workgroup.
template <bool UPDATE>
__global__ void __launch_bounds__(256, 2)
    gemm_mixed_kernel(const GemmDesc *__restrict__ probs, const GroupItem *__restrict__ items,
                      int num_items)
{
    __shared__ float red[direct_red_floats<kClassDirect64>()];
    __shared__ double red8[DirectCfg<kClassDirect32>::KW];
    static_assert(direct_red_floats<kClassDirect32>() <= direct_red_floats<kClassDirect64>(), "");
    const int it = blockIdx.x;
    if (it >= num_items)
        return;
    const GroupItem gi = items[it];
    if (gi.prob < 0)
        return;   // empty item
    const GemmDesc d = probs[gi.prob];
    int tm, tn;
    tile_coords(d, gi.tile, tm, tn);
    const bool c64 = d.small == kClassDirect64;
    switch (d.prec) {
    case PREC_F16X3:
        c64 ? mixed_tile<PREC_F16X3, UPDATE, kClassDirect64>(d, tm, tn, red, red8)
            : mixed_tile<PREC_F16X3, UPDATE, kClassDirect32>(d, tm, tn, red, red8);
        break;
    case PREC_BF16X3:
        c64 ? mixed_tile<PREC_BF16X3, UPDATE, kClassDirect64>(d, tm, tn, red, red8)
            : mixed_tile<PREC_BF16X3, UPDATE, kClassDirect32>(d, tm, tn, red, red8);
        break;
    case PREC_BF16X6:
        c64 ? mixed_tile<PREC_BF16X6, UPDATE, kClassDirect64>(d, tm, tn, red, red8)
            : mixed_tile<PREC_BF16X6, UPDATE, kClassDirect32>(d, tm, tn, red, red8);
        break;
    }
}

}  // namespace dev

hipError_t launch_gemm_mixed(int update, const GemmDesc *probs, const GroupItem *items,
                             int num_items, hipStream_t s)
{
    if (num_items <= 0)
        return hipSuccess;
    const dim3 grid(num_items), block(256);
    if (update)
        hipLaunchKernelGGL(dev::gemm_mixed_kernel<true>, grid, block, 0, s, probs, items, num_items);
    else
        hipLaunchKernelGGL(dev::gemm_mixed_kernel<false>, grid, block, 0, s, probs, items,
                           num_items);
    return hipGetLastError();
}

}  // namespace la
