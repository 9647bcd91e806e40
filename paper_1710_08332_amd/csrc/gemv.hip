// Entry points of gemv: validation, and the launch that a plan calls for
// (gemv.h; each matrix type's kernels are built in a file of their own).
#include "gemv.h"

namespace dpia {

extern template hipError_t launch_gemv<GemvF32, 4>(const Plan&, const GemvF32&, int64_t, int64_t,
                                              hipStream_t, int);
extern template hipError_t launch_gemv<GemvF32Cached, 4>(const Plan&, const GemvF32Cached&, int64_t, int64_t,
                                              hipStream_t, int);
extern template hipError_t launch_gemv<GemvBF16, 8>(const Plan&, const GemvBF16&, int64_t, int64_t,
                                              hipStream_t, int);
extern template hipError_t launch_gemv<GemvFP8, 16>(const Plan&, const GemvFP8&, int64_t, int64_t,
                                              hipStream_t, int);
extern template hipError_t launch_gemv<GemvFP8Long, 16>(const Plan&, const GemvFP8Long&, int64_t, int64_t,
                                              hipStream_t, int);
extern template hipError_t launch_gemv<GemvU32, 4>(const Plan&, const GemvU32&, int64_t, int64_t,
                                              hipStream_t, int);
extern template hipError_t launch_gemv_fed<GemvF32>(const Plan&, const GemvF32&, int64_t, int64_t, int,
                                             hipStream_t);

}  // namespace dpia

using namespace dpia;

#ifndef DPIA_ROW_BLOCK
#define DPIA_ROW_BLOCK 2
#endif
// Rows one team reduces at once for bf16 / fp8 matrices (1 = no blocking):
// with narrow A elements the x operand, reloaded per row, would otherwise
// dominate the traffic through the vector caches.
static constexpr int kRowBlock = DPIA_ROW_BLOCK;

// fp8 rows: 4 rows per team where that still gives one or two work-groups
// per compute unit, else 2.  Measured at 16384^2 (cache evicted), 4 rows
// per team: C=64 L=256 66.0 -> 52.8 us, C=32 L=512 68.4 -> 58.8 us (256
// and 512 work-groups); slower where it leaves 128 work-groups (C=128
// L=128: 57.4 -> 67.9 us) or 1024 (C=16 L=1024: 58.6 -> 68.5 us).
static int fp8_row_block(const Plan& p, int64_t m) {
  const int64_t wgs4 = (m + int64_t(p.teams_per_wg) * 4 - 1) / (int64_t(p.teams_per_wg) * 4);
  const int64_t cus = device_cus();
  return (wgs4 >= cus && wgs4 <= 2 * cus) ? 4 : kRowBlock;
}

namespace {

// Shared body of dpia_gemv (blas = false) and dpia_gemv_blas.
dpia_status gemv_impl(const char* name, const dpia_strategy* s, dpia_dtype a_dt, int64_t m,
                      int64_t k, int64_t lda, const void* A, const float* row_scale, bool blas,
                      float alpha, const void* x, float beta, void* y, dpia_stream_t stream) {
  Plan p;
  std::string detail;
  dpia_status st = make_plan(s, DPIA_OP_GEMV, a_dt, m, k, &p, &detail);
  if (st != DPIA_OK) return bad(st, detail);
  if (lda < k) return bad(DPIA_ERR_SHAPE, "lda must be >= k");
  if (lda % p.nv)
    return bad(DPIA_ERR_SHAPE, "lda must keep every row aligned for the strategy's vector loads");
  if (a_dt == DPIA_FP8_E4M3 && !row_scale && m > 0)
    return bad(DPIA_ERR_NULL, "an FP8 matrix needs row_scale");
  if (a_dt != DPIA_FP8_E4M3 && row_scale)
    return bad(DPIA_ERR_DTYPE, "row_scale applies to FP8 matrices only");
  if (blas && a_dt == DPIA_I32)
    return bad(DPIA_ERR_DTYPE, "the alpha / beta form takes F32, BF16 or FP8 matrices");
  if (m == 0) {
    clear_detail();
    return DPIA_OK;
  }
  if (!A || !x || !y) return bad(DPIA_ERR_NULL, "A, x and y must be non-NULL");
  if (!aligned16(A) || !aligned16(x))
    return bad(DPIA_ERR_SHAPE, "A and x must be 16-byte aligned");
  hipStream_t hs = reinterpret_cast<hipStream_t>(stream);
  hipError_t e = hipErrorInvalidValue;
  auto with_epilogue = [&](auto op) {
    op.blas = blas;
    op.alpha = alpha;
    op.beta = beta;
    op.beta_zero = beta == 0.0f;
    return op;
  };
  switch (a_dt) {
    case DPIA_F32:
      if (const int rows = fed_gemv_rows(p, m, lda))
        e = launch_gemv_fed(
            p, with_epilogue(GemvF32{static_cast<const float*>(A), static_cast<const float*>(x),
                                     nullptr, static_cast<float*>(y)}),
            m, lda, rows, hs);
      else if (p.order == DPIA_ORDER_STRIDED && p.team < 4)
        e = launch_gemv<GemvF32Cached, 4>(
            p, with_epilogue(GemvF32Cached{static_cast<const float*>(A),
                                           static_cast<const float*>(x), nullptr,
                                           static_cast<float*>(y)}),
            m, lda, hs);
      else
        e = launch_gemv<GemvF32, 4>(
            p, with_epilogue(GemvF32{static_cast<const float*>(A), static_cast<const float*>(x),
                                     nullptr, static_cast<float*>(y)}),
            m, lda, hs);
      break;
    case DPIA_BF16:
      e = launch_gemv<GemvBF16, 8>(
          p, with_epilogue(GemvBF16{static_cast<const uint16_t*>(A),
                                    static_cast<const float*>(x), nullptr,
                                    static_cast<float*>(y)}),
          m, lda, hs, kRowBlock);
      break;
    case DPIA_FP8_E4M3:
      if (p.C >= 64)
        e = launch_gemv<GemvFP8Long, 16>(
            p, with_epilogue(GemvFP8Long{static_cast<const uint8_t*>(A),
                                         static_cast<const float*>(x), row_scale,
                                         static_cast<float*>(y)}),
            m, lda, hs, fp8_row_block(p, m));
      else
        e = launch_gemv<GemvFP8, 16>(
            p, with_epilogue(GemvFP8{static_cast<const uint8_t*>(A),
                                     static_cast<const float*>(x), row_scale,
                                     static_cast<float*>(y)}),
            m, lda, hs, fp8_row_block(p, m));
      break;
    case DPIA_I32:
      e = launch_gemv<GemvU32, 4>(
          p, GemvU32{static_cast<const uint32_t*>(A), static_cast<const uint32_t*>(x), nullptr,
                     static_cast<uint32_t*>(y)},
          m, lda, hs);
      break;
    default:
      return bad(DPIA_ERR_DTYPE, "unsupported matrix type");
  }
  if (e != hipSuccess) return hip_fail(e, name);
  clear_detail();
  return DPIA_OK;
}

}  // namespace

extern "C" dpia_status dpia_gemv(const dpia_strategy* s, dpia_dtype a_dt, int64_t m, int64_t k,
                                 int64_t lda, const void* A, const float* row_scale,
                                 const void* x, void* y, void* ws, size_t ws_bytes,
                                 dpia_stream_t stream) {
  (void)ws;
  (void)ws_bytes;
  return gemv_impl("dpia_gemv launch", s, a_dt, m, k, lda, A, row_scale, false, 1.0f, x, 0.0f,
                   y, stream);
}

extern "C" dpia_status dpia_gemv_blas(const dpia_strategy* s, dpia_dtype a_dt, int64_t m,
                                      int64_t k, int64_t lda, float alpha, const void* A,
                                      const float* row_scale, const float* x, float beta,
                                      float* y, dpia_stream_t stream) {
  return gemv_impl("dpia_gemv_blas launch", s, a_dt, m, k, lda, A, row_scale, true, alpha, x,
                   beta, y, stream);
}
