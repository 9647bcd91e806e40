// Kernels and launches of dots fed by loader wavefronts.
#include "reduce.h"

namespace dpia {

template hipError_t launch_fed<DotF32, kFinalPlain>(const Plan&, const DotF32&, const ReduceArgs&, int,
                                             hipStream_t);

}  // namespace dpia
