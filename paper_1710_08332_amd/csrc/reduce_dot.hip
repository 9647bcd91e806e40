// Kernels and launches of one family of reductions (built apart from the
// others, so that they build in parallel).
#include "reduce.h"

namespace dpia {

template hipError_t launch_reduce<DotF32, kFinalPlain>(const Plan&, const DotF32&, void*, int, void*,
                                                void*, hipStream_t, void*);
template hipError_t launch_chunks<DotF32, kFinalPlain>(const Plan&, const DotF32&, const ReduceArgs&,
                                                hipStream_t);
template hipError_t launch_fold<DotF32, kFinalPlain>(int64_t, const void*, void*, int, hipStream_t);

}  // namespace dpia
