// Kernels and launches of one family of reductions (built apart from the
// others, so that they build in parallel).
#include "reduce.h"

namespace dpia {

template hipError_t launch_reduce<DotU32, kFinalPlain>(const Plan&, const DotU32&, void*, int, void*,
                                                void*, hipStream_t, void*);
template hipError_t launch_chunks<DotU32, kFinalPlain>(const Plan&, const DotU32&, const ReduceArgs&,
                                                hipStream_t);
template hipError_t launch_fold<DotU32, kFinalPlain>(int64_t, const void*, void*, int, hipStream_t);
template hipError_t launch_reduce<Deep<DotU32>, kFinalPlain>(const Plan&, const Deep<DotU32>&, void*, int, void*,
                                                void*, hipStream_t, void*);
template hipError_t launch_chunks<Deep<DotU32>, kFinalPlain>(const Plan&, const Deep<DotU32>&, const ReduceArgs&,
                                                hipStream_t);
template hipError_t launch_fold<Deep<DotU32>, kFinalPlain>(int64_t, const void*, void*, int, hipStream_t);

}  // namespace dpia
