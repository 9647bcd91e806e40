// scal: y[i] = alpha * x[i] (the scal benchmark of Sec. 7.1), under the same
// strategy descriptor as the reductions.  A map has no association: whichever
// work-item makes an element, it is one binary32 product, so the chunks and
// lanes of a strategy put no constraint on the hardware's placement.  y may be
// x (in place): each element is read and written by the same thread.
//
// Bound by HBM, half reads and half writes.  One 16-byte piece per thread and
// a work-group for every 4 KiB in address order, so that the launch sweeps
// both arrays as a whole: measured at 2^26 (512 MiB moved, three pairs of
// arrays in turn) 81 us, 6.6 TB/s; 8 pieces per thread 83-88 us, and 83-98 us
// with resident work-groups that stride over the arrays or own a range each.
// Non-temporal loads and stores 81 us, cached ones 88 us.  With the strategy's
// chunks on work-groups and its lanes on threads (staged through LDS where
// contiguous) a call of 2^26 elements took 93-101 us, now 83; 9,854,077
// elements 18-87 us, now 13.7; 1,000,003 8-80 us, now 4.4.
#include "device.h"
#include "host.h"
#include "plan.h"

namespace dpia {

constexpr int kMapThreads = 256;

__global__ void __launch_bounds__(kMapThreads) scal_kernel(float alpha, const float* x, float* y,
                                                           int64_t n) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * (kMapThreads * 4);
  for (int64_t i = (static_cast<int64_t>(blockIdx.x) * kMapThreads + threadIdx.x) * 4; i < n;
       i += stride) {
    if (i + 4 <= n) {
      f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(x + i));
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = alpha * v[j];
      __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(y + i));
    } else {
      for (int64_t j = i; j < n; ++j) y[j] = alpha * x[j];
    }
  }
}

// The same where the strategy bounds the grid and a work-group makes many
// pieces: 8 of each thread in flight (2^26 elements, bounds of 64 / 256 / 512:
// one piece 541, 168, 102 us, 8 pieces 184, 87, 89).
__global__ void __launch_bounds__(kMapThreads) scal_bound_kernel(float alpha, const float* x,
                                                                 float* y, int64_t n) {
  constexpr int U = 8;
  constexpr int64_t kPer = kMapThreads * 4 * U;
  for (int64_t base = static_cast<int64_t>(blockIdx.x) * kPer; base < n;
       base += static_cast<int64_t>(gridDim.x) * kPer) {
    const int64_t first = base + static_cast<int64_t>(threadIdx.x) * 4;
    if (base + kPer <= n) {
      f32x4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        v[u] = __builtin_nontemporal_load(
            reinterpret_cast<const f32x4*>(x + first + u * (kMapThreads * 4)));
      __builtin_amdgcn_sched_barrier(0);   // issue all loads first
#pragma unroll
      for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[u][j] = alpha * v[u][j];
        __builtin_nontemporal_store(
            v[u], reinterpret_cast<f32x4*>(y + first + u * (kMapThreads * 4)));
      }
    } else {
      for (int u = 0; u < U; ++u) {
        const int64_t i = first + u * (kMapThreads * 4);
        for (int64_t j = i; j < i + 4 && j < n; ++j) y[j] = alpha * x[j];
      }
    }
  }
}

}  // namespace dpia

using namespace dpia;

extern "C" dpia_status dpia_scal(const dpia_strategy* s, dpia_dtype dt, int64_t n, float alpha,
                                 const void* x, void* y, dpia_stream_t stream) {
  Plan p;
  std::string detail;
  dpia_status st = make_plan(s, DPIA_OP_SCAL, dt, 0, n, &p, &detail);
  if (st != DPIA_OK) return bad(st, detail);
  if (n > 0 && (!x || !y)) return bad(DPIA_ERR_NULL, "x and y must be non-NULL");
  if (n > 0 && (!aligned16(x) || !aligned16(y)))
    return bad(DPIA_ERR_SHAPE, "x and y must be 16-byte aligned");
  if (p.items == 0) {
    clear_detail();
    return DPIA_OK;
  }
  // one work-group per 1,024 elements, or the strategy's bound on them
  constexpr int64_t kPer = kMapThreads * 4;
  const int64_t need = (p.n + kPer - 1) / kPer;
  auto kern = grid_is_bound(p, need) ? scal_bound_kernel : scal_kernel;
  const int64_t grid = bounded_grid(need, p.max_grid, kMapThreads);
  const float* xp = static_cast<const float*>(x);
  float* yp = static_cast<float*>(y);
  void* args[] = {&alpha, &xp, &yp, &p.n};
  hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(kern), dim3(grid),
                                 dim3(kMapThreads), args, 0, reinterpret_cast<hipStream_t>(stream));
  if (e != hipSuccess) return hip_fail(e, "dpia_scal launch");
  clear_detail();
  return DPIA_OK;
}
