// Kernels and launches of one family of reductions (built apart from the
// others, so that they build in parallel).
#include "reduce.h"

namespace dpia {

extern template hipError_t launch_rows<KahanDotF32, kFinalKahan64>(const Plan&, const KahanDotF32&, const ReduceArgs&, int,
                                              hipStream_t);
extern template hipError_t launch_rows<KahanDotF32, kFinalKahan32>(const Plan&, const KahanDotF32&, const ReduceArgs&, int,
                                              hipStream_t);
template hipError_t launch_reduce<KahanDotF32, kFinalKahan32>(const Plan&, const KahanDotF32&, void*, int, void*,
                                                void*, hipStream_t, void*);
template hipError_t launch_chunks<KahanDotF32, kFinalKahan32>(const Plan&, const KahanDotF32&, const ReduceArgs&,
                                                hipStream_t);
template hipError_t launch_fold<KahanDotF32, kFinalKahan32>(int64_t, const void*, void*, int, hipStream_t);
template hipError_t launch_reduce<KahanDotF32, kFinalKahan64>(const Plan&, const KahanDotF32&, void*, int, void*,
                                                void*, hipStream_t, void*);
template hipError_t launch_chunks<KahanDotF32, kFinalKahan64>(const Plan&, const KahanDotF32&, const ReduceArgs&,
                                                hipStream_t);
template hipError_t launch_fold<KahanDotF32, kFinalKahan64>(int64_t, const void*, void*, int, hipStream_t);
template hipError_t launch_reduce<Deep<KahanDotF32>, kFinalKahan32>(const Plan&, const Deep<KahanDotF32>&, void*, int, void*,
                                                void*, hipStream_t, void*);
template hipError_t launch_chunks<Deep<KahanDotF32>, kFinalKahan32>(const Plan&, const Deep<KahanDotF32>&, const ReduceArgs&,
                                                hipStream_t);
template hipError_t launch_fold<Deep<KahanDotF32>, kFinalKahan32>(int64_t, const void*, void*, int, hipStream_t);
template hipError_t launch_reduce<Deep<KahanDotF32>, kFinalKahan64>(const Plan&, const Deep<KahanDotF32>&, void*, int, void*,
                                                void*, hipStream_t, void*);
template hipError_t launch_chunks<Deep<KahanDotF32>, kFinalKahan64>(const Plan&, const Deep<KahanDotF32>&, const ReduceArgs&,
                                                hipStream_t);
template hipError_t launch_fold<Deep<KahanDotF32>, kFinalKahan64>(int64_t, const void*, void*, int, hipStream_t);

}  // namespace dpia
