// Entry points of dot and asum: validation, and the launch that a plan calls
// for (reduce.h; each family of kernels is built in a file of its own).
#include <mutex>

#include "reduce.h"

namespace dpia {

// Kernels and launches of an operation (built in the files of its family).
#define DPIA_EXTERN(OP, FINAL)                                                                  \
  extern template hipError_t launch_reduce<OP, FINAL>(const Plan&, const OP&, void*, int, void*, \
                                                      void*, hipStream_t, void*);               \
  extern template hipError_t launch_chunks<OP, FINAL>(const Plan&, const OP&, const ReduceArgs&, \
                                                      hipStream_t);                             \
  extern template hipError_t launch_fold<OP, FINAL>(int64_t, const void*, void*, int, hipStream_t)
DPIA_EXTERN(DotF32, kFinalPlain);
DPIA_EXTERN(DotF32Deep, kFinalPlain);
DPIA_EXTERN(DotF32Deeper, kFinalPlain);
DPIA_EXTERN(DotU32, kFinalPlain);
DPIA_EXTERN(AsumF32, kFinalPlain);
DPIA_EXTERN(KahanDotF32, kFinalKahan32);
DPIA_EXTERN(KahanDotF32, kFinalKahan64);
DPIA_EXTERN(Sum2DotF32, kFinalSum2_32);
DPIA_EXTERN(Sum2DotF32, kFinalSum2_64);
DPIA_EXTERN(Deep<DotF32>, kFinalPlain);
DPIA_EXTERN(Deep<DotU32>, kFinalPlain);
DPIA_EXTERN(Deep<AsumF32>, kFinalPlain);
DPIA_EXTERN(Deep<KahanDotF32>, kFinalKahan32);
DPIA_EXTERN(Deep<KahanDotF32>, kFinalKahan64);
DPIA_EXTERN(Deep<Sum2DotF32>, kFinalSum2_32);
DPIA_EXTERN(Deep<Sum2DotF32>, kFinalSum2_64);
#undef DPIA_EXTERN

#ifndef DPIA_DEEPER_DOT
#define DPIA_DEEPER_DOT 1
#endif

// The load batch of a plain binary32 dot that is not thin (thin_plan): strided
// lanes in teams narrower than 1024 lanes use DotF32Deep, or DotF32Deeper when
// the whole launch has fewer than two wavefronts per compute unit.  Contiguous
// dots staged through LDS whose launch has fewer wavefronts than compute units
// use DotF32Deeper too (two staged tiles in flight); unstaged contiguous
// dots keep the default batch (a deeper one would need 128 registers of
// loads in flight).
inline int dot_depth(const Plan& p) {
  const int64_t waves = p.items * ((p.team + 63) / 64);
  const int64_t cus = device_cus();
  if (p.order != DPIA_ORDER_STRIDED)
    return (DPIA_DEEPER_DOT && p.stage && waves < cus) ? 2 : 0;
  if (p.L >= 1024) return 0;
  return (DPIA_DEEPER_DOT && waves < 2 * cus) ? 2 : 1;
}

// Calls f(op, final-kind constant) for the operation, accumulation and load
// batch of a plan.
template <class F>
hipError_t with_reduction(const Plan& p, const void* x, const void* y, F&& f) {
  const float* xf = static_cast<const float*>(x);
  const float* yf = static_cast<const float*>(y);
  const bool thin = thin_lanes(p);
  // `op`, or the same with deep batches
  auto at_depth = [&](auto op, auto fin) {
    using Op = decltype(op);
    if (thin) return f(Deep<Op>{op}, fin);
    return f(op, fin);
  };
  if (p.op == DPIA_OP_ASUM) return at_depth(AsumF32{xf}, ic<kFinalPlain>{});
  if (p.dt == DPIA_I32)
    return at_depth(DotU32{static_cast<const uint32_t*>(x), static_cast<const uint32_t*>(y)},
                    ic<kFinalPlain>{});
  if (p.accum == DPIA_ACCUM_KAHAN) {
    if (p.final_f64) return at_depth(KahanDotF32{xf, yf}, ic<kFinalKahan64>{});
    return at_depth(KahanDotF32{xf, yf}, ic<kFinalKahan32>{});
  }
  if (p.accum == DPIA_ACCUM_SUM2) {
    if (p.final_f64) return at_depth(Sum2DotF32{xf, yf}, ic<kFinalSum2_64>{});
    return at_depth(Sum2DotF32{xf, yf}, ic<kFinalSum2_32>{});
  }
  if (thin) return f(Deep<DotF32>{{xf, yf}}, ic<kFinalPlain>{});
  const int depth = dot_depth(p);
  if (depth == 2) return f(DotF32Deeper{{xf, yf}}, ic<kFinalPlain>{});
  if (depth == 1) return f(DotF32Deep{{xf, yf}}, ic<kFinalPlain>{});
  return f(DotF32{xf, yf}, ic<kFinalPlain>{});
}

namespace {

dpia_status check_ws(const Plan& p, void* ws, size_t ws_bytes) {
  if (ws_bytes < p.ws_bytes) {
    return bad(DPIA_ERR_WORKSPACE, "workspace of " + std::to_string(ws_bytes) +
                                       " bytes is smaller than the required " +
                                       std::to_string(p.ws_bytes));
  }
  if (p.ws_bytes && !ws) return bad(DPIA_ERR_WORKSPACE, "workspace is NULL");
  if (ws && (reinterpret_cast<uintptr_t>(ws) % kWsAlign))
    return bad(DPIA_ERR_SHAPE, "workspace must be 256-byte aligned");
  return DPIA_OK;
}

}  // namespace
}  // namespace dpia

using namespace dpia;

namespace {

// Shared body of dpia_dot and dpia_dot_noalloc after validation: the launches
// of a dot with its chunk values in `partials` and the 1-pass arrival
// counter at `counter`.
dpia_status dot_launch(const Plan& p, const void* x, const void* y, void* out,
                       dpia_dtype out_dt, void* partials, void* counter, hipStream_t hs,
                       const char* name, void* split = nullptr) {
  const int f64 = out_dt == DPIA_F64;
  const Plan q = thin_plan(p);
  hipError_t e = with_reduction(p, x, y, [&](auto op, auto fin) {
    return launch_reduce<decltype(op), decltype(fin)::value>(q, op, out, f64, partials, counter, hs,
                                                             split);
  });
  if (e != hipSuccess) return hip_fail(e, name);
  clear_detail();
  return DPIA_OK;
}

// Everything dpia_dot checks apart from the workspace.
dpia_status dot_validate(const dpia_strategy* s, dpia_dtype dt, int64_t n, const void* x,
                         const void* y, const void* out, dpia_dtype out_dt, Plan* p) {
  std::string detail;
  dpia_status st = make_plan(s, DPIA_OP_DOT, dt, 0, n, p, &detail);
  if (st != DPIA_OK) return bad(st, detail);
  if (!out || (n > 0 && (!x || !y))) return bad(DPIA_ERR_NULL, "x, y and out must be non-NULL");
  if (n > 0 && (!aligned16(x) || !aligned16(y)))
    return bad(DPIA_ERR_SHAPE, "x and y must be 16-byte aligned");
  if (dt == DPIA_I32) {
    if (out_dt != DPIA_I32) return bad(DPIA_ERR_DTYPE, "an I32 dot writes an I32 result");
  } else if (p->accum == DPIA_ACCUM_KAHAN || p->accum == DPIA_ACCUM_SUM2) {
    if (out_dt != DPIA_F32 && !(out_dt == DPIA_F64 && p->final_f64))
      return bad(DPIA_ERR_DTYPE, "a compensated dot writes F32, or F64 with final_f64");
  } else if (out_dt != DPIA_F32) {
    return bad(DPIA_ERR_DTYPE, "an F32 dot writes an F32 result");
  }
  return DPIA_OK;
}

}  // namespace

extern "C" dpia_status dpia_dot(const dpia_strategy* s, dpia_dtype dt, int64_t n, const void* x,
                                const void* y, void* out, dpia_dtype out_dt, void* ws,
                                size_t ws_bytes, dpia_stream_t stream) {
  Plan p;
  dpia_status st = dot_validate(s, dt, n, x, y, out, out_dt, &p);
  if (st != DPIA_OK) return st;
  st = check_ws(p, ws, ws_bytes);
  if (st != DPIA_OK) return st;
  void* split = p.split_off ? static_cast<char*>(ws) + p.split_off : nullptr;
  return dot_launch(p, x, y, out, out_dt, ws, static_cast<char*>(ws) + p.partial_bytes,
                    reinterpret_cast<hipStream_t>(stream), "dpia_dot launch", split);
}

// ------------------------------------------------------------ no-alloc dot
// dpia_dot_noalloc keeps the chunk values and the arrival counter of a call
// in this file-scope device array instead of a caller workspace: bytes
// [0, kWsAlign) hold the counter (at a fixed place, so that 1-pass calls of
// any size find it at zero), the chunk values start at kWsAlign.  Every GPU
// the library runs on has its own copy, at its own address.
constexpr size_t kScratchBytes = size_t(1) << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

__global__ void scratch_clear_kernel(unsigned int* counter) {
  // the whole 256-byte block of the arrival counter
  if (threadIdx.x < kWsAlign / sizeof(unsigned int)) counter[threadIdx.x] = 0u;
}

namespace {

constexpr int kMaxDevices = 64;

struct ScratchSlot {
  std::once_flag once;
  void* ptr = nullptr;
  hipError_t err = hipSuccess;
};
ScratchSlot g_scratch[kMaxDevices];

// The current device's copy of `scratch` (set up on the first call on that
// device: its address, and the counter cleared by a kernel on `hs`).
dpia_status scratch_for_current_device(hipStream_t hs, void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "dpia_dot_noalloc: hipGetDevice");
  if (dev < 0 || dev >= kMaxDevices)
    return bad(DPIA_ERR_HIP, "dpia_dot_noalloc: device id beyond the supported 64");
  ScratchSlot& slot = g_scratch[dev];
  std::call_once(slot.once, [&] {
    void* ptr = nullptr;
    slot.err = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (slot.err != hipSuccess) return;
    unsigned int* counter = static_cast<unsigned int*>(ptr);
    void* args[] = {&counter};
    slot.err = hipLaunchKernel(reinterpret_cast<const void*>(scratch_clear_kernel), dim3(1),
                               dim3(64), args, 0, hs);
    if (slot.err == hipSuccess) slot.ptr = ptr;
  });
  if (slot.err != hipSuccess) return hip_fail(slot.err, "dpia_dot_noalloc: scratch set-up");
  *out = slot.ptr;
  return DPIA_OK;
}

}  // namespace

extern "C" dpia_status dpia_dot_noalloc(const dpia_strategy* s, dpia_dtype dt, int64_t n,
                                        const void* x, const void* y, void* out,
                                        dpia_dtype out_dt, dpia_stream_t stream) {
  Plan p;
  dpia_status st = dot_validate(s, dt, n, x, y, out, out_dt, &p);
  if (st != DPIA_OK) return st;
  if (p.partial_bytes > kScratchBytes - kWsAlign)
    return bad(DPIA_ERR_WORKSPACE,
               "the strategy's " + std::to_string(p.partial_bytes) +
                   " bytes of chunk values exceed the no-alloc scratch of " +
                   std::to_string(kScratchBytes - kWsAlign) + " bytes");
  hipStream_t hs = reinterpret_cast<hipStream_t>(stream);
  void* base = nullptr;
  st = scratch_for_current_device(hs, &base);
  if (st != DPIA_OK) return st;
  unsigned char* b = static_cast<unsigned char*>(base);
  return dot_launch(p, x, y, out, out_dt, b + kWsAlign, b, hs, "dpia_dot_noalloc launch");
}

extern "C" dpia_status dpia_asum(const dpia_strategy* s, dpia_dtype dt, int64_t n, const void* x,
                                 void* out, dpia_dtype out_dt, void* ws, size_t ws_bytes,
                                 dpia_stream_t stream) {
  Plan p;
  std::string detail;
  dpia_status st = make_plan(s, DPIA_OP_ASUM, dt, 0, n, &p, &detail);
  if (st != DPIA_OK) return bad(st, detail);
  if (out_dt != DPIA_F32) return bad(DPIA_ERR_DTYPE, "asum writes an F32 result");
  if (!out || (n > 0 && !x)) return bad(DPIA_ERR_NULL, "x and out must be non-NULL");
  if (n > 0 && !aligned16(x)) return bad(DPIA_ERR_SHAPE, "x must be 16-byte aligned");
  st = check_ws(p, ws, ws_bytes);
  if (st != DPIA_OK) return st;
  void* split = p.split_off ? static_cast<char*>(ws) + p.split_off : nullptr;
  const Plan q = thin_plan(p);
  hipError_t e = with_reduction(p, x, nullptr, [&](auto op, auto fin) {
    return launch_reduce<decltype(op), decltype(fin)::value>(
        q, op, out, 0, ws, static_cast<char*>(ws) + p.partial_bytes,
        reinterpret_cast<hipStream_t>(stream), split);
  });
  if (e != hipSuccess) return hip_fail(e, "dpia_asum launch");
  clear_detail();
  return DPIA_OK;
}

// The two stages of a 2-pass strategy as separate calls (see dpia.h).
extern "C" dpia_status dpia_chunks(const dpia_strategy* s, dpia_op op, dpia_dtype dt, int64_t n,
                                   const void* x, const void* y, void* chunks,
                                   size_t chunks_bytes, dpia_stream_t stream) {
  if (op != DPIA_OP_DOT && op != DPIA_OP_ASUM)
    return bad(DPIA_ERR_STRATEGY, "dpia_chunks takes DPIA_OP_DOT or DPIA_OP_ASUM");
  Plan p;
  std::string detail;
  dpia_status st = make_plan(s, op, dt, 0, n, &p, &detail);
  if (st != DPIA_OK) return bad(st, detail);
  const bool dot = op == DPIA_OP_DOT;
  if (n > 0 && (!x || (dot && !y))) return bad(DPIA_ERR_NULL, "input vectors must be non-NULL");
  if (n > 0 && (!aligned16(x) || (dot && !aligned16(y))))
    return bad(DPIA_ERR_SHAPE, "input vectors must be 16-byte aligned");
  const size_t need = static_cast<size_t>(p.values) * p.acc_bytes;
  if (p.items > 0 && !chunks) return bad(DPIA_ERR_NULL, "chunks must be non-NULL");
  if (chunks_bytes < need)
    return bad(DPIA_ERR_WORKSPACE, "chunks holds " + std::to_string(chunks_bytes) +
                                       " bytes, the strategy writes " + std::to_string(need));
  hipStream_t hs = reinterpret_cast<hipStream_t>(stream);
  hipError_t e = with_reduction(p, x, y, [&](auto op_v, auto fin) {
    using Op = decltype(op_v);
    constexpr int FINAL = decltype(fin)::value;
    const Plan q = thin_plan(p);
    ReduceArgs a = reduce_args<Op>(q, chunks, nullptr, nullptr, 0, false);
    return launch_chunks<Op, FINAL>(q, op_v, a, hs);
  });
  if (e != hipSuccess) return hip_fail(e, "dpia_chunks launch");
  clear_detail();
  return DPIA_OK;
}

extern "C" dpia_status dpia_fold(const dpia_strategy* s, dpia_op op, dpia_dtype dt, int64_t n,
                                 const void* chunks, void* out, dpia_dtype out_dt,
                                 dpia_stream_t stream) {
  if (op != DPIA_OP_DOT && op != DPIA_OP_ASUM)
    return bad(DPIA_ERR_STRATEGY, "dpia_fold takes DPIA_OP_DOT or DPIA_OP_ASUM");
  Plan p;
  std::string detail;
  dpia_status st = make_plan(s, op, dt, 0, n, &p, &detail);
  if (st != DPIA_OK) return bad(st, detail);
  if (!out || (p.items > 0 && !chunks)) return bad(DPIA_ERR_NULL, "chunks and out must be non-NULL");
  const dpia_dtype want = (dt == DPIA_I32) ? DPIA_I32 : DPIA_F32;
  if (!(out_dt == want || (out_dt == DPIA_F64 && p.final_f64)))
    return bad(DPIA_ERR_DTYPE, "output type does not match the strategy");
  hipStream_t hs = reinterpret_cast<hipStream_t>(stream);
  hipError_t e = with_reduction(p, nullptr, nullptr, [&](auto op_v, auto fin) {
    using Op = decltype(op_v);
    constexpr int FINAL = decltype(fin)::value;
    return launch_fold<Op, FINAL>(p.values, chunks, out, out_dt == DPIA_F64, hs);
  });
  if (e != hipSuccess) return hip_fail(e, "dpia_fold launch");
  clear_detail();
  return DPIA_OK;
}
