// Kernels and launches of contiguous lanes, ROWS to a wavefront.
#include "reduce.h"

namespace dpia {

template hipError_t launch_rows<DotF32, kFinalPlain>(const Plan&, const DotF32&, const ReduceArgs&, int,
                                              hipStream_t);
template hipError_t launch_rows<AsumF32, kFinalPlain>(const Plan&, const AsumF32&, const ReduceArgs&, int,
                                              hipStream_t);

}  // namespace dpia
