// Kernels and launches of one matrix type (built apart from the others, so
// that they build in parallel).
#include "gemv.h"

namespace dpia {

template hipError_t launch_gemv<GemvBF16, 8>(const Plan&, const GemvBF16&, int64_t, int64_t,
                                              hipStream_t);

}  // namespace dpia
