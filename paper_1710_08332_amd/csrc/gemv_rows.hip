// Kernels and launches of binary32 rows: contiguous lanes ROWS to a wavefront,
// and few strided lanes one to a thread.
#include "gemv.h"

namespace dpia {

template hipError_t launch_gemv_rows<GemvF32>(const Plan&, const GemvF32&, int64_t, int64_t, int,
                                              hipStream_t);
template hipError_t launch_gemv<GemvF32Deep, 4>(const Plan&, const GemvF32Deep&, int64_t, int64_t,
                                                hipStream_t);

}  // namespace dpia
