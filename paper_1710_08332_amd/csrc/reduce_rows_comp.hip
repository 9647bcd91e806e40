// Kernels and launches of contiguous lanes, ROWS to a wavefront.
#include "reduce.h"

namespace dpia {

template hipError_t launch_rows<KahanDotF32, kFinalKahan32>(const Plan&, const KahanDotF32&, const ReduceArgs&, int,
                                              hipStream_t);
template hipError_t launch_rows<KahanDotF32, kFinalKahan64>(const Plan&, const KahanDotF32&, const ReduceArgs&, int,
                                              hipStream_t);
template hipError_t launch_rows<Sum2DotF32, kFinalSum2_32>(const Plan&, const Sum2DotF32&, const ReduceArgs&, int,
                                              hipStream_t);
template hipError_t launch_rows<Sum2DotF32, kFinalSum2_64>(const Plan&, const Sum2DotF32&, const ReduceArgs&, int,
                                              hipStream_t);

}  // namespace dpia
