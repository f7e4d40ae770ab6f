// Small tiles on the fp32 matrix pipe (ukst_small_kernel.h): instances of one kind and operand type.
#include "ukst_small_kernel.h"

namespace ukst {
namespace small {

template <>
hipError_t launch_kind<kInputGrad, uint16_t>(const SmallArgs& a, int n, int s, int mt, int wv, const Epilogue& ep, const void* x,
                                const void* w, void* y, hipStream_t st)
{
    return launch_kind_impl<kInputGrad, uint16_t>(a, n, s, mt, wv, ep, x, w, y, st);
}

}  // namespace small
}  // namespace ukst
