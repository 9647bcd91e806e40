// Kernels and launches of binary32 rows fed by loader wavefronts.
#include "gemv.h"

namespace dpia {

template hipError_t launch_gemv_fed<GemvF32>(const Plan&, const GemvF32&, int64_t, int64_t, int,
                                             hipStream_t);

}  // namespace dpia
