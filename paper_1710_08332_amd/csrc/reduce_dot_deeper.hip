// Kernels and launches of one family of reductions (built apart from the
// others, so that they build in parallel).
#include "reduce.h"

namespace dpia {

extern template hipError_t launch_rows<DotF32, kFinalPlain>(const Plan&, const DotF32&, const ReduceArgs&, int,
                                              hipStream_t);
// (fed kernels: reduce_dot_fed.hip)
extern template hipError_t launch_fed<DotF32, kFinalPlain>(const Plan&, const DotF32&, const ReduceArgs&, int,
                                             hipStream_t);

template hipError_t launch_reduce<DotF32Deeper, kFinalPlain>(const Plan&, const DotF32Deeper&, void*, int, void*,
                                                void*, hipStream_t, void*);
template hipError_t launch_chunks<DotF32Deeper, kFinalPlain>(const Plan&, const DotF32Deeper&, const ReduceArgs&,
                                                hipStream_t);
template hipError_t launch_fold<DotF32Deeper, kFinalPlain>(int64_t, const void*, void*, int, hipStream_t);
template hipError_t launch_reduce<Deep<DotF32>, kFinalPlain>(const Plan&, const Deep<DotF32>&, void*, int,
                                                void*, void*, hipStream_t, void*);
template hipError_t launch_chunks<Deep<DotF32>, kFinalPlain>(const Plan&, const Deep<DotF32>&,
                                                const ReduceArgs&, hipStream_t);
template hipError_t launch_fold<Deep<DotF32>, kFinalPlain>(int64_t, const void*, void*, int, hipStream_t);

}  // namespace dpia
