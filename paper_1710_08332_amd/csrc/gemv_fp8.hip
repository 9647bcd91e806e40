// Kernels and launches of one matrix type (built apart from the others, so
// that they build in parallel).
#include "gemv.h"

namespace dpia {

template hipError_t launch_gemv<GemvFP8, 16>(const Plan&, const GemvFP8&, int64_t, int64_t,
                                              hipStream_t);
template hipError_t launch_gemv<GemvFP8Deep, 16>(const Plan&, const GemvFP8Deep&, int64_t, int64_t,
                                              hipStream_t);

}  // namespace dpia
