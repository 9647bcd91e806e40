// Kernels and launches of binary32 rows: contiguous lanes ROWS to a wavefront,
// few strided lanes one to a thread, and long strided rows in half batches.
#include "gemv.h"

namespace dpia {

template hipError_t launch_gemv_rows<GemvF32>(const Plan&, const GemvF32&, int64_t, int64_t, int,
                                              hipStream_t);
template hipError_t launch_gemv_block<GemvF32, 1>(const Plan&, const GemvF32&, int64_t, int64_t,
                                                  hipStream_t);
template hipError_t launch_gemv_thin<GemvF32Deep>(const Plan&, const GemvF32Deep&, int64_t, int64_t,
                                                  hipStream_t);

}  // namespace dpia
