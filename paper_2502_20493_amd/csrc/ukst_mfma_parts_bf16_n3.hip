// Instances of the matrix-core kernel on bf16 parts for n = 3, bf16 operands (one translation unit per kernel side).
#include "ukst_mfma_parts_kernel.h"

namespace ukst {
namespace parts {
template <>
hipError_t launch_side<3, uint16_t>(const PartsArgs& a, const Config& c, const Epilogue& ep, const void* x, const void* w,
                                void* y, bool out16, hipStream_t st)
{
    return launch_side_impl<3, uint16_t>(a, c, ep, x, w, y, out16, st);
}
}  // namespace parts
}  // namespace ukst
