// Kernels and launches of asums fed by loader wavefronts.
#include "reduce.h"

namespace dpia {

template hipError_t launch_fed<AsumF32, kFinalPlain>(const Plan&, const AsumF32&, const ReduceArgs&, int,
                                             hipStream_t);

}  // namespace dpia
