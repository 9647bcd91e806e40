// Row-blocked kernels of one matrix type (built apart from the others, so
// that they build in parallel).
#include "gemv.h"

namespace dpia {

template hipError_t launch_gemv_block<GemvBF16, 4>(const Plan&, const GemvBF16&, int64_t, int64_t,
                                                 hipStream_t);
template hipError_t launch_gemv_block<GemvBF16, 2>(const Plan&, const GemvBF16&, int64_t, int64_t,
                                                 hipStream_t);
template hipError_t launch_gemv_block<GemvBF16Deep, 1>(const Plan&, const GemvBF16Deep&, int64_t, int64_t,
                                                 hipStream_t);

}  // namespace dpia
