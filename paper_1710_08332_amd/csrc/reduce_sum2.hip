// Kernels and launches of one family of reductions (built apart from the
// others, so that they build in parallel).
#include "reduce.h"

namespace dpia {

extern template hipError_t launch_rows<Sum2DotF32, kFinalSum2_64>(const Plan&, const Sum2DotF32&, const ReduceArgs&, int,
                                              hipStream_t);
extern template hipError_t launch_rows<Sum2DotF32, kFinalSum2_32>(const Plan&, const Sum2DotF32&, const ReduceArgs&, int,
                                              hipStream_t);
template hipError_t launch_reduce<Sum2DotF32, kFinalSum2_32>(const Plan&, const Sum2DotF32&, void*, int, void*,
                                                void*, hipStream_t, void*);
template hipError_t launch_chunks<Sum2DotF32, kFinalSum2_32>(const Plan&, const Sum2DotF32&, const ReduceArgs&,
                                                hipStream_t);
template hipError_t launch_fold<Sum2DotF32, kFinalSum2_32>(int64_t, const void*, void*, int, hipStream_t);
template hipError_t launch_reduce<Sum2DotF32, kFinalSum2_64>(const Plan&, const Sum2DotF32&, void*, int, void*,
                                                void*, hipStream_t, void*);
template hipError_t launch_chunks<Sum2DotF32, kFinalSum2_64>(const Plan&, const Sum2DotF32&, const ReduceArgs&,
                                                hipStream_t);
template hipError_t launch_fold<Sum2DotF32, kFinalSum2_64>(int64_t, const void*, void*, int, hipStream_t);
template hipError_t launch_reduce<Deep<Sum2DotF32>, kFinalSum2_32>(const Plan&, const Deep<Sum2DotF32>&, void*, int, void*,
                                                void*, hipStream_t, void*);
template hipError_t launch_chunks<Deep<Sum2DotF32>, kFinalSum2_32>(const Plan&, const Deep<Sum2DotF32>&, const ReduceArgs&,
                                                hipStream_t);
template hipError_t launch_fold<Deep<Sum2DotF32>, kFinalSum2_32>(int64_t, const void*, void*, int, hipStream_t);
template hipError_t launch_reduce<Deep<Sum2DotF32>, kFinalSum2_64>(const Plan&, const Deep<Sum2DotF32>&, void*, int, void*,
                                                void*, hipStream_t, void*);
template hipError_t launch_chunks<Deep<Sum2DotF32>, kFinalSum2_64>(const Plan&, const Deep<Sum2DotF32>&, const ReduceArgs&,
                                                hipStream_t);
template hipError_t launch_fold<Deep<Sum2DotF32>, kFinalSum2_64>(int64_t, const void*, void*, int, hipStream_t);

}  // namespace dpia
