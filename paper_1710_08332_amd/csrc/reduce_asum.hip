// Kernels and launches of one family of reductions (built apart from the
// others, so that they build in parallel).
#include "reduce.h"

namespace dpia {

extern template hipError_t launch_rows<AsumF32, kFinalPlain>(const Plan&, const AsumF32&, const ReduceArgs&, int,
                                              hipStream_t);
// (fed kernels: reduce_asum_fed.hip)
extern template hipError_t launch_fed<AsumF32, kFinalPlain>(const Plan&, const AsumF32&, const ReduceArgs&, int,
                                             hipStream_t);

template hipError_t launch_reduce<AsumF32, kFinalPlain>(const Plan&, const AsumF32&, void*, int, void*,
                                                void*, hipStream_t, void*);
template hipError_t launch_chunks<AsumF32, kFinalPlain>(const Plan&, const AsumF32&, const ReduceArgs&,
                                                hipStream_t);
template hipError_t launch_fold<AsumF32, kFinalPlain>(int64_t, const void*, void*, int, hipStream_t);

}  // namespace dpia
