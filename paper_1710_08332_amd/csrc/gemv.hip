// Entry points of gemv: validation, and the launch that a plan calls for
// (gemv.h; each matrix type's kernels are built in a file of their own).
#include "gemv.h"

namespace dpia {

extern template hipError_t launch_gemv<GemvF32, 4>(const Plan&, const GemvF32&, int64_t, int64_t,
                                              hipStream_t);
extern template hipError_t launch_gemv<GemvF32Cached, 4>(const Plan&, const GemvF32Cached&, int64_t, int64_t,
                                              hipStream_t);
extern template hipError_t launch_gemv<GemvBF16, 8>(const Plan&, const GemvBF16&, int64_t, int64_t,
                                              hipStream_t);
extern template hipError_t launch_gemv<GemvFP8, 16>(const Plan&, const GemvFP8&, int64_t, int64_t,
                                              hipStream_t);
extern template hipError_t launch_gemv<GemvFP8Deep, 16>(const Plan&, const GemvFP8Deep&, int64_t, int64_t,
                                              hipStream_t);
extern template hipError_t launch_gemv_thin<GemvF32Deep>(const Plan&, const GemvF32Deep&, int64_t, int64_t,
                                              hipStream_t);
extern template hipError_t launch_gemv_block<GemvF32, 1>(const Plan&, const GemvF32&, int64_t,
                                                         int64_t, hipStream_t);
extern template hipError_t launch_gemv_rows<GemvF32>(const Plan&, const GemvF32&, int64_t, int64_t, int,
                                              hipStream_t);
extern template hipError_t launch_gemv<GemvU32, 4>(const Plan&, const GemvU32&, int64_t, int64_t,
                                              hipStream_t);
extern template hipError_t launch_gemv_block<GemvBF16, 4>(const Plan&, const GemvBF16&, int64_t, int64_t,
                                                 hipStream_t);
extern template hipError_t launch_gemv_block<GemvBF16, 2>(const Plan&, const GemvBF16&, int64_t, int64_t,
                                                 hipStream_t);
extern template hipError_t launch_gemv_block<GemvBF16Deep, 1>(const Plan&, const GemvBF16Deep&, int64_t, int64_t,
                                                 hipStream_t);
extern template hipError_t launch_gemv_block<GemvFP8, 4>(const Plan&, const GemvFP8&, int64_t, int64_t,
                                                 hipStream_t);
extern template hipError_t launch_gemv_block<GemvFP8Deep, 4>(const Plan&, const GemvFP8Deep&, int64_t, int64_t,
                                                 hipStream_t);
extern template hipError_t launch_gemv_block<GemvFP8Deep, 2>(const Plan&, const GemvFP8Deep&, int64_t, int64_t,
                                                 hipStream_t);
extern template hipError_t launch_gemv_block<GemvFP8Deep, 1>(const Plan&, const GemvFP8Deep&, int64_t, int64_t,
                                                 hipStream_t);
extern template hipError_t launch_gemv_fed<GemvF32>(const Plan&, const GemvF32&, int64_t, int64_t, int,
                                             hipStream_t);

}  // namespace dpia

using namespace dpia;

namespace {

// Strided binary32 rows over 64 or 128 long lanes, in launches with wavefronts
// enough: the row-blocked kernel with one row per team, whose batch is two
// halves, one in flight while the other is folded.  A wavefront holds 4 or 2
// such rows, so its loads cover 256 or 512 bytes of each, and gemv_kernel's
// whole batches leave it without loads while it folds (us, before and now:
// 8192^2 C=64 L=128 49.8, 42.4, C=128 L=64 46.7, 43.9; 16384^2 C=128 L=128
// 168.6, 154.9, C=256 L=64 168.1, 162.7; but 8192^2 C=32 L=256 42.7, 44.2,
// 16384^2 C=512 L=32 160.5, 166.6).  16 wavefronts are resident per compute
// unit; with fewer the one row of each is too little, most of all where they
// begin on another wavefront per SIMD (speed against gemv_kernel, C=64 L=128 and
// C=128 L=64: 2300 wavefronts 0.89 0.99, 2560 0.87 0.98, 3584 0.96 1.00, 3900
// 1.00 1.03, 4096 1.09 1.22, 9000 1.09 1.15, 16384 1.05 1.13).
bool gemv_halves(const Plan& p, int64_t m) {
  return gemv_blocks<GemvF32>(p) && (p.L == 64 || p.L == 128) && p.C >= 64 &&
         m * p.team >= 15 * kWave * static_cast<int64_t>(device_cus()) &&
         !grid_is_bound(p, m * p.team / kWave);
}

// Row-blocked bf16 / fp8 rows.  More rows per team share each load of x;
// fewer, with deeper batches, keep the memory busy when there are few
// wavefronts.  `waves`: wavefronts of the launch with one row per team.
// Measured with 64-thread work-groups (us; rows per team x elements per batch):
//  bf16  L=256 C=16   2048 waves   1x64 11.7  2x16 11.9     3000  19.8  13.5
//              C=64   2048         27.1  31.0               3000  43.0  35.6
//        L=16  C=3, two parts 300 waves 5.5 4.6
//        L=512 C=32   1024         11.7  15.4  2048  18.9  17.6  3000  32.2  21.0
//              C=32   8000         66.5  50.5  4x16 49.4   16384  131  96.5  96.5
//  fp8   L=512 C=32   1400 waves   1x64 20.6  2x64 17.2  4x64 24.0  4x16 33.6
//                     2000         26.3  18.8  25.7  35.3
//                     3000         45.5  34.5  28.2  37.1
//                     4600         --    37.5  39.9  34.8
//                     9000         --    63.0  61.8  69.7
//              C=16   4600         --    23.2  23.5  20.2
//        L=256 C=64   4000         81.1  61.3  55.9  72.6   8000  --  120  108  125
//        L=64  C=16   12000        --    50.7  47.9  59.6
// and with many wavefronts (S: work-groups of 256 threads, 2 rows x 16):
//  bf16  L=256 C=32   16500 waves  S 93.3  2x16 82.3  4x16 91.7   33000  S 182  158  166
//        L=512 C=8    20480        S 29.3  27.3  28.7             50000  S 68.3  62.3  61.3
//        L=512 C=32   16384        S 91.6  85.0  83.4             16500  S 92.9  85.3  90.3
//              C=16   21000        S 54.9  56.5  55.4             50000  S 136   130   120
//  fp8   L=512 C=24   9000 waves   S 54.5  4x64 49.3  4x16 60.7   13000  S 81.1  65.4  69.8
//              C=24   16384        S 90.1  79.0  79.1             17000  S 88.7  84.1  98.2
//              C=33   11000        S 75.0  68.8  78.1             13000  S 101   88.7  82.5
//              C=33   16384        S 111   101   89.2             30000  S 208   181   169
//        L=64  C=5    5000         S 33.2  31.8  26.4             8000   S 39.1  37.0  44.8
//        L=128 C=16   10000        S 36.5  35.8  38.3             16384  S 57.8  54.7  47.0
// Hence: bf16 1x64 up to 8 wavefronts per compute unit (6 with 64 threads to a
// team; 1 where lanes of fewer than 8 elements have no deep batch), then 2x16; 4x16 for teams of 64 threads with lanes of 13 and more, from
// 80 on, and at 64, where the launch is one round of what is resident.  fp8 1x64
// up to 6, 2x64 up to 8, 4x64 up to 16, then 4x16; but 4x64 for narrow teams of
// long lanes, and where 4x16 would just begin on another wavefront per SIMD (32
// to 44 or 48, 64 to 72).  (With 256-thread work-groups, 2 rows and 16 elements, the
// bf16 launches of 2048 and 3000 wavefronts above took 12.3, 13.7, 32.2, 39.2,
// 18.7 and 21.2 us; the fp8 ones, of 2 or 4 rows, 34.6, 36.0, 40.0, 37.9, 65.5,
// 20.2, 82.7, 155 and 51.3.)
// (a bounded grid: 2 bf16 rows instead of 4, 2 fp8 rows instead of 1, as the
// work-groups of launch_gemv_block are large then)
int64_t block_waves(const Plan& p, int64_t m) { return (m * p.team + kWave - 1) / kWave; }

hipError_t launch_bf16(const Plan& p, const GemvBF16& op, int64_t m, int64_t lda, hipStream_t s) {
  if (!gemv_blocks<GemvBF16>(p)) return launch_gemv<GemvBF16, 8>(p, op, m, lda, s);
  const int64_t waves = block_waves(p, m), cus = device_cus();
  const bool whole = waves > 62 * cus && waves <= 64 * cus;   // one round of 4 rows
  if (p.team >= kWave && p.C >= 13 && (waves >= 80 * cus || whole) && !grid_is_bound(p, waves / 4))
    return launch_gemv_block<GemvBF16, 4>(p, op, m, lda, s);
  if (waves > (p.C < 8 ? 1 : (p.team >= kWave ? 6 : 8)) * cus)
    return launch_gemv_block<GemvBF16, 2>(p, op, m, lda, s);
  const GemvBF16Deep deep{op.A, op.x, op.scale, op.y, op.blas, op.beta_zero, op.alpha, op.beta};
  return launch_gemv_block<GemvBF16Deep, 1>(p, deep, m, lda, s);
}

hipError_t launch_fp8(const Plan& p, const GemvFP8& op, int64_t m, int64_t lda, hipStream_t s) {
  const GemvFP8Deep deep{op.A, op.x, op.scale, op.y, op.blas, op.beta_zero, op.alpha, op.beta};
  if (!gemv_blocks<GemvFP8>(p)) {
    if (p.C >= 64) return launch_gemv<GemvFP8Deep, 16>(p, deep, m, lda, s);
    return launch_gemv<GemvFP8, 16>(p, op, m, lda, s);
  }
  const int64_t waves = block_waves(p, m), cus = device_cus();
  if (waves > 8 * cus) {
    const bool many = waves > 32 * cus, narrow = p.team <= 16;
    const bool deep4 = waves <= 16 * cus || (p.C >= 64 && narrow) ||
                       (p.team <= 4 && (p.C >= 16 || waves > 24 * cus)) ||
                       (many && p.C >= 32 && (narrow || waves <= 48 * cus)) ||
                       (many && p.C >= 16 && p.team <= 32 && waves <= (p.C >= 18 ? 48 : 44) * cus) ||
                       (p.C >= 18 && waves > 64 * cus && waves <= 72 * cus);
    if (deep4) return launch_gemv_block<GemvFP8Deep, 4>(p, deep, m, lda, s);
    return launch_gemv_block<GemvFP8, 4>(p, op, m, lda, s);
  }
  if (waves > 6 * cus || grid_is_bound(p, waves))
    return launch_gemv_block<GemvFP8Deep, 2>(p, deep, m, lda, s);
  return launch_gemv_block<GemvFP8Deep, 1>(p, deep, m, lda, s);
}

}  // namespace

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
      else if (const int per_wave = gemv_rows_per_wave(p, m))
        e = launch_gemv_rows(
            p, with_epilogue(GemvF32{static_cast<const float*>(A), static_cast<const float*>(x),
                                     nullptr, static_cast<float*>(y)}),
            m, lda, per_wave, hs);
      else if (gemv_thin(p, m))
        e = launch_gemv_thin<GemvF32Deep>(
            gemv_thin_plan(p, m),
            with_epilogue(GemvF32Deep{static_cast<const float*>(A), static_cast<const float*>(x),
                                      nullptr, static_cast<float*>(y)}),
            m, lda, hs);
      else if (gemv_halves(p, m))
        e = launch_gemv_block<GemvF32, 1>(
            p, with_epilogue(GemvF32{static_cast<const float*>(A), static_cast<const float*>(x),
                                     nullptr, static_cast<float*>(y)}),
            m, lda, hs);
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
      e = launch_bf16(p,
                      with_epilogue(GemvBF16{static_cast<const uint16_t*>(A),
                                             static_cast<const float*>(x), nullptr,
                                             static_cast<float*>(y)}),
                      m, lda, hs);
      break;
    case DPIA_FP8_E4M3:
      e = launch_fp8(p,
                     with_epilogue(GemvFP8{static_cast<const uint8_t*>(A),
                                           static_cast<const float*>(x), row_scale,
                                           static_cast<float*>(y)}),
                     m, lda, hs);
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
