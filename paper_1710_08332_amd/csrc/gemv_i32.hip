// Kernels and launches of one matrix type (built apart from the others, so
// that they build in parallel).
#include "gemv.h"

namespace dpia {

template hipError_t launch_gemv<GemvU32, 4>(const Plan&, const GemvU32&, int64_t, int64_t,
                                              hipStream_t);

}  // namespace dpia
