// y = A x under a DPIA strategy (gemv benchmark, Sec. 7.1):
//   join (mapWorkgroup (lam rows. map (lam row. ROWRED (zip row x)) rows)
//         (split R A))
// where ROWRED is the chunk reduction of the dot-product strategy (lane folds
// of C elements, then the combine of the L lanes).  With two row parts each
// half row is a chunk of its own and the halves are folded as (0 + h0) + h1.
// bf16 and fp8-e4m3 matrices are decoded exactly to binary32 before the
// multiply; fp8 rows are scaled after the reduction: y[r] = scale[r] * sum.
// No cross-work-group step: each team owns whole rows of y.
#pragma once

#include "device.h"
#include "fed.h"
#include "ops.h"
#include "rows.h"
#include "host.h"
#include "plan.h"

namespace dpia {

struct GemvArgs {
  int64_t m;
  int64_t k;
  int64_t lda;
  int W, L, C, team, teams_per_wg, team_lds_elems, parts;
  int stage_off;          // byte offset of the LDS staging region, -1: none
};

// Strided lane folds of RB rows at once: thread t holds lanes t*NV ..
// t*NV + NV-1 of each of the RB rows, so every x load serves RB rows.  Each
// row's lanes fold their own elements in increasing index, exactly as with
// one row per team.  `limit`: elements of the row part that exist.
// Row-blocked folds load their batch as two halves, one in flight while the
// other is folded.  With 4 rows per team the fp8 launch has one wavefront
// per SIMD, so a batch's decodes, products and sums otherwise ran with no
// loads of that SIMD in flight (measured at 16384^2, cache evicted, C=64
// L=256: 53.1 -> 50.6-50.9 us; bf16 C=32 L=512 98.5 -> 97.3 us).
template <class Op, int NV, int RB>
__device__ __forceinline__ void row_block_folds(const Op& op, const int64_t (&row)[RB],
                                                const bool (&act)[RB], int64_t lda, int64_t col0,
                                                int t, int L, int C, int limit,
                                                float (&acc)[RB][NV]) {
#pragma unroll
  for (int b = 0; b < RB; ++b)
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[b][v] = 0.0f;
  bool any = false;
#pragma unroll
  for (int b = 0; b < RB; ++b) any = any || act[b];
  if (!any) return;
  constexpr int U = Batch<NV, Op, kStrided>::U;
  const int rows = limit / L;
  const int nfull = rows < C ? rows : C;
  const int start = t * NV;
  int k = 0;
  if constexpr (U >= 2 && U % 2 == 0) {
    // two half batches: one in flight while the other is folded
    constexpr int H = U / 2;
    float xa[H][NV], xb[H][NV];
    typename Op::Code ca[H][RB][NV], cb[H][RB][NV];
    auto load_half = [&](int k0, float (&xv)[H][NV], typename Op::Code (&cc)[H][RB][NV]) {
#pragma unroll
      for (int u = 0; u < H; ++u) {
        const int64_t c = col0 + start + static_cast<int64_t>(k0 + u) * L;
        op.template load_x<NV>(c, xv[u]);
#pragma unroll
        for (int b = 0; b < RB; ++b) op.template load_codes<NV>(row[b], lda, c, cc[u][b]);
      }
    };
    auto fold_half = [&](const float (&xv)[H][NV], const typename Op::Code (&cc)[H][RB][NV]) {
#pragma unroll
      for (int u = 0; u < H; ++u)
#pragma unroll
        for (int b = 0; b < RB; ++b) {
          float av[NV];
          Op::template decode<NV>(cc[u][b], av);
#pragma unroll
          for (int v = 0; v < NV; ++v)
            acc[b][v] = Op::step(typename Op::Term{av[v], xv[u][v]}, acc[b][v]);
        }
    };
    if (k + U <= nfull) {
      load_half(k, xa, ca);
      for (; k + U <= nfull; k += U) {
        load_half(k + H, xb, cb);
        __builtin_amdgcn_sched_barrier(0);
        fold_half(xa, ca);
        __builtin_amdgcn_sched_barrier(0);
        if (k + U + H <= nfull) load_half(k + U, xa, ca);
        __builtin_amdgcn_sched_barrier(0);
        fold_half(xb, cb);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (k + H <= nfull) {   // the half batch loaded last
        fold_half(xa, ca);
        k += H;
      }
    }
  }
  for (; k + U <= nfull; k += U) {
    float xv[U][NV];
    typename Op::Code ca[U][RB][NV];   // codes: decoded only when folded
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t c = col0 + start + static_cast<int64_t>(k + u) * L;
      op.template load_x<NV>(c, xv[u]);
#pragma unroll
      for (int b = 0; b < RB; ++b) op.template load_codes<NV>(row[b], lda, c, ca[u][b]);
    }
    __builtin_amdgcn_sched_barrier(0);   // issue the whole batch first
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int b = 0; b < RB; ++b) {
        float av[NV];
        Op::template decode<NV>(ca[u][b], av);
#pragma unroll
        for (int v = 0; v < NV; ++v)
          acc[b][v] = Op::step(typename Op::Term{av[v], xv[u][v]}, acc[b][v]);
      }
  }
  // what is left (fewer than a half batch), in batches of 2 and 1 steps
  auto some = [&](auto nc) {
    constexpr int N = decltype(nc)::value;
    float xv[N][NV];
    typename Op::Code cc[N][RB][NV];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int64_t c = col0 + start + static_cast<int64_t>(k + u) * L;
      op.template load_x<NV>(c, xv[u]);
#pragma unroll
      for (int b = 0; b < RB; ++b) op.template load_codes<NV>(row[b], lda, c, cc[u][b]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < N; ++u)
#pragma unroll
      for (int b = 0; b < RB; ++b) {
        float av[NV];
        Op::template decode<NV>(cc[u][b], av);
#pragma unroll
        for (int v = 0; v < NV; ++v)
          acc[b][v] = Op::step(typename Op::Term{av[v], xv[u][v]}, acc[b][v]);
      }
    k += N;
  };
  if constexpr (U > 2)
    while (k + 2 <= nfull) some(ic<2>{});
  while (k < nfull) some(ic<1>{});
  if (nfull < C) {   // the last, partly existing row of the part
    const int o = start + nfull * L;
    float xv[NV], av[RB][NV];
    // its elements are loaded together (one wait on memory, not NV), then folded
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      if (o + v < limit) {
        xv[v] = op.x[col0 + o + v];
#pragma unroll
        for (int b = 0; b < RB; ++b) av[b][v] = op.load_a1(row[b], lda, col0 + o + v);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      if (o + v < limit) {
#pragma unroll
        for (int b = 0; b < RB; ++b)
          acc[b][v] = Op::step(typename Op::Term{av[b][v], xv[v]}, acc[b][v]);
      }
    }
  }
}

// LDS elements from one of a team's rows to the next, where lanes are combined
// one after the other: a slot for the row's first part, and other banks.
constexpr int kSeqPad = 4;

// The sum of L lane values in LDS from 0 in lane order, L a multiple of NV: the
// next NV values are read while the ones before are added.
template <int NV>
__device__ __forceinline__ float lanes_in_turn(const float* lanes, int L) {
  float r = PlainF32::zero(), g[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) g[v] = lanes[v];
  for (int l = NV; l < L; l += NV) {
    float next[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) next[v] = lanes[l + v];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int v = 0; v < NV; ++v) r = PlainF32::add(g[v], r);
#pragma unroll
    for (int v = 0; v < NV; ++v) g[v] = next[v];
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) r = PlainF32::add(g[v], r);
  return r;
}

// A sequential combine of one row is a chain of L additions that one thread
// does while its wavefront waits, so the rows of a team are combined side by
// side, a thread each (us, row after row and so; a work-group of 256 threads
// with 2 rows: fp8 6800 x 6656, C=13 L=512 52.9 19.3, 39.3; 20000 x 16384, C=32
// L=512 165 82.5, 97.3; bf16 17000 x 16384, C=32 L=512 137 104, 118).
template <class Op, int NV, int COMBINE, int RB>
__global__ void __launch_bounds__(256) gemv_block_kernel(Op op, GemvArgs a) {
  using T = float;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  T* lds = reinterpret_cast<T*>(lds_raw);
  const int team_id = threadIdx.x / a.team;
  const int t = threadIdx.x - team_id * a.team;
  T* scratch = lds + team_id * a.team_lds_elems;
  const int64_t per_wg = static_cast<int64_t>(a.teams_per_wg) * RB;
  for (int64_t base = static_cast<int64_t>(blockIdx.x) * per_wg; base < a.m;
       base += static_cast<int64_t>(gridDim.x) * per_wg) {
    int64_t row[RB];
    bool act[RB];
#pragma unroll
    for (int b = 0; b < RB; ++b) {
      const int64_t r = base + static_cast<int64_t>(team_id) * RB + b;
      act[b] = r < a.m;
      row[b] = act[b] ? r : 0;
    }
    float acc[RB][NV];
    if constexpr (COMBINE == kSeq) {
      const int pitch = a.L + kSeqPad;
      for (int part = 0; part < a.parts; ++part) {
        const int64_t left = a.k - static_cast<int64_t>(part) * a.W;
        const int lim = static_cast<int>(left < 0 ? 0 : (left < a.W ? left : a.W));
        row_block_folds<Op, NV, RB>(op, row, act, a.lda, static_cast<int64_t>(part) * a.W, t, a.L,
                                    a.C, lim, acc);
#pragma unroll
        for (int b = 0; b < RB; ++b)
#pragma unroll
          for (int v = 0; v < NV; ++v) scratch[b * pitch + t * NV + v] = acc[b][v];
        __syncthreads();
        for (int b = t; b < RB; b += a.team) {
          T* lanes = scratch + b * pitch;
          const T v = lanes_in_turn<NV>(lanes, a.L);
          if (part + 1 < a.parts) {
            lanes[a.L] = v;
          } else {
            // reduceSeq (+) 0 [h0, h1]
            const T r = a.parts == 2 ? tree_node<PlainF32>(lanes[a.L], v) : v;
            const int64_t q = base + static_cast<int64_t>(team_id) * RB + b;
            if (q < a.m) op.store(q, r);
          }
        }
        __syncthreads();
      }
    } else {
      T v[RB];
      const int lim0 = static_cast<int>(a.k < a.W ? a.k : a.W);
      row_block_folds<Op, NV, RB>(op, row, act, a.lda, 0, t, a.L, a.C, lim0, acc);
#pragma unroll
      for (int b = 0; b < RB; ++b) v[b] = combine_lanes<PlainF32, NV, COMBINE>(acc[b], t, a.team, a.L, scratch);
      if (a.parts == 2) {
        const int lim1 = static_cast<int>(a.k - a.W);
        row_block_folds<Op, NV, RB>(op, row, act, a.lda, a.W, t, a.L, a.C, lim1 > 0 ? lim1 : 0, acc);
#pragma unroll
        for (int b = 0; b < RB; ++b) {
          const T h1 = combine_lanes<PlainF32, NV, COMBINE>(acc[b], t, a.team, a.L, scratch);
          v[b] = tree_node<PlainF32>(v[b], h1);   // reduceSeq (+) 0 [h0, h1]
        }
      }
      if (t == 0) {
#pragma unroll
        for (int b = 0; b < RB; ++b)
          if (act[b]) op.store(row[b], v[b]);
      }
    }
  }
}

// MAXT: the largest work-group it is launched with (256 or 1024); the
// 256-thread build may use twice the registers of the 1024-thread one.
// STAGED: folded through LDS (see chunk_value; work-groups of at most 256).
template <class Op, int ORDER, int NV, int COMBINE, int MAXT, bool STAGED = false>
__global__ void __launch_bounds__(MAXT) gemv_kernel(Op op, GemvArgs a) {
  using T = typename Op::T;
  using A = typename Op::Arith;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  T* lds = reinterpret_cast<T*>(lds_raw);
  const int team_id = threadIdx.x / a.team;
  const int t = threadIdx.x - team_id * a.team;
  T* scratch = lds + team_id * a.team_lds_elems;
  float* stage = STAGED ? reinterpret_cast<float*>(lds_raw + a.stage_off) +
                              (threadIdx.x / kWave) * stage_floats(kWave)
                        : nullptr;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * a.teams_per_wg;
  for (int64_t base = static_cast<int64_t>(blockIdx.x) * a.teams_per_wg; base < a.m;
       base += stride) {
    const int64_t row = base + team_id;
    const bool active = row < a.m;
    const int64_t r = active ? row : 0;
    // elements of each row part that exist (k may stop short of W * parts:
    // the row is zero-extended)
    const int lim0 = static_cast<int>(a.k < a.W ? a.k : a.W);
    T v = chunk_value<Op, ORDER, NV, COMBINE, STAGED>(op.part(r, 0, a.lda, a.W), active, t, a.team,
                                                  a.L, a.C, lim0, scratch, stage);
    if (a.parts == 2) {
      const int lim1 = static_cast<int>(a.k - a.W);
      const T h1 = chunk_value<Op, ORDER, NV, COMBINE, STAGED>(op.part(r, 1, a.lda, a.W), active, t,
                                                           a.team, a.L, a.C, lim1 > 0 ? lim1 : 0,
                                                           scratch, stage);
      v = tree_node<A>(v, h1);   // reduceSeq (+) 0 [h0, h1]
    }
    if (active && t == 0) op.store(row, v);
  }
}

// Binary32 rows fed by loader wavefronts: teams of one thread (the strided
// order with L = NL lanes held as that thread's components, or one
// contiguous lane), strided teams of two threads (TPR below) and contiguous
// teams of L threads (one lane each), row parts of whole tiles.  The strategy's work-groups of R rows give each busy
// compute unit a wavefront or two (16384 rows of R = 128: 128 work-groups),
// too few loads in flight to stream A.  The rows are independent, so a
// hardware work-group here takes ROWS lane rows of its own, ROWS / team
// consecutive matrix rows: wave 0 folds them (lane q the Cel = W / team
// elements of lane q % team of its row, element e into component e % NL, in
// increasing e, as chunk_value's staged folds do), kFedLoaders wavefronts
// load A and x into the LDS ring.  The lanes are combined by combine_lanes
// over teams of `team` adjacent lanes of wave 0 and the parts by tree_node,
// as in gemv_kernel: every row's association is the strategy's.
// TPR = 2: strided teams of 2 threads holding 4 lanes each (L = 8);
// the ROWS ring rows are whole matrix row parts, and the team's threads fold
// their own 16-byte pieces of every step of the shared row (fed_fold).
// XR: x rows of a ring slot, 1 where a matrix row is one ring row (every
// team but the contiguous teams of L > 1 lanes), L for contiguous teams of
// L = 2 or 4 lanes (lane l reads x row l), 0: one x row per ring row.
template <class Op, int NL, int COMBINE, int ROWS, int TPR = 1, int XR = 0>
__global__ void __launch_bounds__(kWave * (1 + kFedLoaders)) gemv_fed_kernel(Op op, GemvArgs a) {
  using T = typename Op::T;
  using A = typename Op::Arith;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  float* ring = reinterpret_cast<float*>(lds_raw);
  const int team = TPR > 1 ? TPR : a.team;
  const int t = static_cast<int>(threadIdx.x) % team;
  // each team's combine region (its team * NL lane values)
  T* scratch = reinterpret_cast<T*>(ring + fed_ring_floats()) +
               (static_cast<int>(threadIdx.x) - t) * NL;
  const int wave = static_cast<int>(threadIdx.x) / kWave;
  const int lane = static_cast<int>(threadIdx.x) % kWave;
  const int row_lanes = TPR > 1 ? 1 : team;   // ring rows per matrix row
  const int cel = a.W / row_lanes;
  const int rows_per_wg = ROWS / row_lanes;
  for (int64_t row0 = static_cast<int64_t>(blockIdx.x) * rows_per_wg; row0 < a.m;
       row0 += static_cast<int64_t>(gridDim.x) * rows_per_wg) {
    T acc[NL];
    fed_fold<Op, NL, ROWS, true, TPR, XR>(op.part(row0, 0, a.lda, a.W), cel, wave, lane, 0,
                                            ring, acc, static_cast<int>(a.lda), row_lanes);
    T v = combine_lanes<A, NL, COMBINE>(acc, t, team, a.L, scratch);
    if (a.parts == 2) {
      fed_fold<Op, NL, ROWS, true, TPR, XR>(op.part(row0, 1, a.lda, a.W), cel, wave, lane, 0,
                                              ring, acc, static_cast<int>(a.lda), row_lanes);
      const T h1 = combine_lanes<A, NL, COMBINE>(acc, t, team, a.L, scratch);
      v = tree_node<A>(v, h1);   // reduceSeq (+) 0 [h0, h1]
    }
    if (wave == 0 && lane < ROWS * TPR && t == 0) op.store(row0 + lane / team, v);
  }
}

// Lane rows per work-group of gemv_fed_kernel for this plan, or 0 where it
// does not apply: teams of one thread, strided teams of two, or contiguous
// teams of at most 64 threads, binary32 A (the caller's check), every row part whole (k = W *
// parts) with lanes of at least 64 tiles of 64 elements, and m a multiple
// of the matrix rows per work-group.  The most lane rows that still give
// every compute unit a work-group.
template <int ROWS>
constexpr bool fed_gemv_fits(int64_t tiles) {
  // (a multiple of every depth fed_fold uses for these rows: 4 to 16 tiles)
  return tiles % fed_depth<ROWS, 1>() == 0;
}
// Strided teams of 2 threads of 4 lanes each (L = 8): ring rows are matrix
// rows, 16 or 32 of them (at most 64 folding lanes).  (Teams of 4 threads,
// 16 rows of 4 KB per round, measured no faster this way at 16384^2:
// strided C=1024 L=16 177.9 -> 175.1 us, C=512 L=16 with two parts 174.6
// -> 176.0 us; teams of 2: C=1024 L=8 with two parts 235.5 -> 181.8 us.)
inline int fed_gemv_rows(const Plan& p, int64_t m, int64_t lda) {
  if (m <= 0 || lda % 4 || lda > (int64_t(1) << 24)) return 0;
  if (p.order == DPIA_ORDER_STRIDED && p.nv == 4 && p.team == 2 && p.L == 8) {
    if (p.W % kFedStage || p.k != p.W * p.row_parts || p.W / kFedStage < 64) return 0;
    const int64_t tiles = p.W / kFedStage;
    if (m % 32 == 0 && m / 32 >= device_cus() && fed_gemv_fits<32>(tiles)) return 32;
    if (m % 16 == 0 && fed_gemv_fits<16>(tiles)) return 16;
    return 0;
  }
  const bool lanes = p.order == DPIA_ORDER_STRIDED
                         ? (p.team == 1 && p.nv == p.L && (p.L == 1 || p.L == 2 || p.L == 4))
                         : p.team == p.L && p.L <= 64 && (p.L & (p.L - 1)) == 0;
  if (!lanes || p.W % (int64_t(kFedStage) * p.team) || p.k != p.W * p.row_parts) return 0;
  // (lanes of 16 tiles measured slower than gemv_kernel: 16384^2 contiguous
  // C=1024 L=16 234.9 -> 248.3 us, L=8 with two parts 191.6 -> 251.0 us; a
  // work-group's pipeline fills and drains every 16 rounds)
  const int64_t tiles = p.W / p.team / kFedStage;
  if (tiles < 64) return 0;
  const int64_t cus = device_cus();
  const int64_t lane_rows = m * p.team;
  auto fits = [&](int rows, bool fill) {
    return rows % p.team == 0 && m % (rows / p.team) == 0 && (!fill || lane_rows / rows >= cus);
  };
  if (fits(64, true) && fed_gemv_fits<64>(tiles)) return 64;
  if (fits(32, true) && fed_gemv_fits<32>(tiles)) return 32;
  if (fits(16, false) && fed_gemv_fits<16>(tiles)) return 16;
  if (fits(64, false) && fed_gemv_fits<64>(tiles)) return 64;
  return 0;
}

template <class Op>
hipError_t launch_gemv_fed(const Plan& p, const Op& op, int64_t m, int64_t lda, int rows,
                           hipStream_t stream) {
  GemvArgs a{};
  a.m = m;
  a.k = p.k;
  a.lda = lda;
  a.W = static_cast<int>(p.W);
  a.L = static_cast<int>(p.L);
  a.C = static_cast<int>(p.C);
  // threads per row: strided teams of 1, 2 or 4 threads, contiguous teams of L
  a.team = p.order == DPIA_ORDER_STRIDED ? p.team : static_cast<int>(p.L);
  // matrix rows per work-group (ring rows are matrix rows for strided teams)
  a.teams_per_wg = p.order == DPIA_ORDER_STRIDED ? rows : rows / a.team;
  a.parts = p.row_parts;
  a.stage_off = -1;
  const int nl = p.order == DPIA_ORDER_STRIDED ? p.nv : 1;
  const int64_t grid = bounded_grid(m / a.teams_per_wg, p.max_grid, kWave * (1 + kFedLoaders));
  const size_t lds = sizeof(float) * fed_ring_floats() +
                     sizeof(typename Op::T) * kWave * (1 + kFedLoaders) * 4;
  auto go = [&](auto nlc, auto comb, auto rc) {
    constexpr int NL = decltype(nlc)::value;
    constexpr int COMBINE = decltype(comb)::value;
    constexpr int ROWS = decltype(rc)::value;
    auto kern = gemv_fed_kernel<Op, NL, COMBINE, ROWS, 1, 1>;
    if constexpr (NL == 1) {
      if (a.team == 2) kern = gemv_fed_kernel<Op, NL, COMBINE, ROWS, 1, 2>;
      else if (a.team == 4) kern = gemv_fed_kernel<Op, NL, COMBINE, ROWS, 1, 4>;
      else if (a.team > 4) kern = gemv_fed_kernel<Op, NL, COMBINE, ROWS, 1, 0>;
    }
    Op op_copy = op;
    void* args[] = {&op_copy, &a};
    return hipLaunchKernel(reinterpret_cast<const void*>(kern), dim3(grid),
                           dim3(kWave * (1 + kFedLoaders)), args, lds, stream);
  };
  auto by_rows = [&](auto nlc, auto comb) {
    return rows == 64 ? go(nlc, comb, ic<64>{})
                      : (rows == 32 ? go(nlc, comb, ic<32>{}) : go(nlc, comb, ic<16>{}));
  };
  auto by_combine = [&](auto nlc) {
    return p.combine == DPIA_COMBINE_TREE ? by_rows(nlc, ic<kTree>{}) : by_rows(nlc, ic<kSeq>{});
  };
  auto team_go = [&](auto comb, auto rc, auto tc) {
    auto kern = gemv_fed_kernel<Op, 4, decltype(comb)::value, decltype(rc)::value,
                                decltype(tc)::value, 1>;
    Op op_copy = op;
    void* args[] = {&op_copy, &a};
    return hipLaunchKernel(reinterpret_cast<const void*>(kern), dim3(grid),
                           dim3(kWave * (1 + kFedLoaders)), args, lds, stream);
  };
  auto team_rows = [&](auto comb) {
    return rows == 32 ? team_go(comb, ic<32>{}, ic<2>{}) : team_go(comb, ic<16>{}, ic<2>{});
  };
  if (p.order == DPIA_ORDER_STRIDED && a.team > 1)
    return p.combine == DPIA_COMBINE_TREE ? team_rows(ic<kTree>{}) : team_rows(ic<kSeq>{});
  return nl == 4 ? by_combine(ic<4>{}) : (nl == 2 ? by_combine(ic<2>{}) : by_combine(ic<1>{}));
}

// bf16 / fp8 rows in the strided order, whole 16-byte loads per lane group:
// RB rows per team at once, one wavefront's worth of teams per work-group.
// Rows are independent, so the work-group's size is free; small ones leave no
// compute unit idle while the last large ones end (measured at 16384^2, work-
// groups of 256 and of 64 threads: bf16 C=32 L=512 with 4 rows 104.0 and 83.5
// us, fp8 C=32 L=512 with 4 rows 58.9 and 45.5 us).
template <class Op>
bool gemv_blocks(const Plan& p) {
  return p.order == DPIA_ORDER_STRIDED && p.team <= 256 &&
         p.nv == kVecBytes / static_cast<int>(sizeof(typename Op::Code));
}

template <class Op, int RB>
hipError_t launch_gemv_block(const Plan& p, const Op& op, int64_t m, int64_t lda,
                             hipStream_t stream) {
  constexpr int NV = kVecBytes / static_cast<int>(sizeof(typename Op::Code));
  GemvArgs a{};
  a.m = m;
  a.k = p.k;
  a.lda = lda;
  a.W = static_cast<int>(p.W);
  a.L = static_cast<int>(p.L);
  a.C = static_cast<int>(p.C);
  a.team = p.team;
  // (never more teams than the plan's LDS is for: its work-groups hold at
  // least 64 threads)
  a.teams_per_wg = p.team < kWave ? kWave / p.team : 1;
  if (a.teams_per_wg > p.teams_per_wg) a.teams_per_wg = p.teams_per_wg;
  if (grid_is_bound(p, (m + a.teams_per_wg * RB - 1) / (a.teams_per_wg * RB))) {
    a.teams_per_wg = 256 / p.team;
    if (a.teams_per_wg > p.teams_per_wg) a.teams_per_wg = p.teams_per_wg;
  }
  const bool seq = p.combine == DPIA_COMBINE_SEQ;
  a.team_lds_elems = seq ? RB * (static_cast<int>(p.L) + kSeqPad) : (p.team > 64 ? p.team / 64 : 1);
  const size_t lds = (static_cast<size_t>(a.teams_per_wg) * a.team_lds_elems * sizeof(float) + 31) / 16 * 16;
  a.parts = p.row_parts;
  a.stage_off = -1;
  const int64_t per_wg = static_cast<int64_t>(a.teams_per_wg) * RB;
  const int64_t grid =
      bounded_grid((m + per_wg - 1) / per_wg, p.max_grid, a.teams_per_wg * p.team);
  auto kern = seq ? gemv_block_kernel<Op, NV, kSeq, RB> : gemv_block_kernel<Op, NV, kTree, RB>;
  Op op_copy = op;
  void* args[] = {&op_copy, &a};
  return hipLaunchKernel(reinterpret_cast<const void*>(kern), dim3(grid),
                         dim3(a.teams_per_wg * p.team), args, lds, stream);
}

// Contiguous binary32 rows, ROWS lane rows to a wavefront (rows.h):
// `teams_per_wg` matrix rows to a work-group at once.
template <class Op, int COMBINE, int ROWS, int D>
__global__ void __launch_bounds__(kWave* kRowsWaves) gemv_rows_kernel(Op op, GemvArgs a) {
  using T = typename Op::T;
  using A = typename Op::Arith;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int lane = static_cast<int>(threadIdx.x) & (kWave - 1);
  // wavefronts per row
  const int per_row = static_cast<int>(blockDim.x) / kWave / a.teams_per_wg;
  const int team = wave / per_row;
  const int t = static_cast<int>(threadIdx.x) - team * per_row * kWave;
  T* scratch = reinterpret_cast<T*>(lds_raw);          // (used by single rows only)
  T* lanes = reinterpret_cast<T*>(lds_raw + kRowsScratch) + team * a.L;
  float* stage = reinterpret_cast<float*>(lds_raw + a.stage_off) +
                 wave * rows_stage_floats<ROWS>(Op::View::kOps);
  const int slices = a.L / ROWS;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * a.teams_per_wg;
  for (int64_t r0 = static_cast<int64_t>(blockIdx.x) * a.teams_per_wg; r0 < a.m; r0 += stride) {
    const int64_t r = r0 + team;
    auto part = [&](int p) {
      const int64_t rest = a.k - static_cast<int64_t>(p) * a.W;
      const int limit = static_cast<int>(rest < 0 ? 0 : (rest < a.W ? rest : a.W));
      if (r < a.m) {
        const auto view = op.part(r, p, a.lda, a.W);
        for (int s = wave - team * per_row; s < slices; s += per_row) {
          T acc[1];
          rows_fold<Op, 1, ROWS, D, true>(view, s * ROWS, a.C, limit, stage, acc);
          if (ROWS == kWave || lane < ROWS) lanes[s * ROWS + lane] = acc[0];
        }
      }
      __syncthreads();
      const T v = combine_stored<A, COMBINE>(lanes, a.L, t, per_row * kWave, scratch);
      __syncthreads();   // the lane values may be written again
      return v;
    };
    T v = part(0);
    if (a.parts == 2) {
      const T h1 = part(1);
      v = tree_node<A>(v, h1);   // reduceSeq (+) 0 [h0, h1]
    }
    if (t == 0 && r < a.m) op.store(r, v);
  }
}

// Lane rows per wavefront of contiguous binary32 rows (0: gemv_kernel), by the
// same lines as a dot's chunks (rows_per_wave, reduce.h).  Measured, that and
// this (us; m x k, lanes in the launch):
//   256 x 16384  C=1024 L=16 (4,096)    39.4 17.7    C=32 L=512 13.6 7.3
//   1024 x 16384 C=512 L=32 (32,768)    23.9 19.0    C=256 L=64 (65,536) 19.1 17.4
//   1500 x 3001  C=192 L=16 (24,000)    14.8  9.9    C=32 L=512 17.8 11.4
//   8192^2       C=32 L=512             160  77      16384^2 C=32 L=512 625 225
// (8192 x 1000 under C=32 L=512, where 32 of a row's 512 lanes have elements,
// 43 and 49 us: rows much shorter than their lanes stay with gemv_kernel.)
// (32 rows take tiles of 64 elements: 759 x 1276, C=32 L=64, 4.0 4.6; C=64 is 9%
// faster in the mean.)
// A row tile is 128 elements of 16 rows, so lanes shorter than 96 mostly load
// nothing: rows win there only where the launch is small, or where the row's
// length is no multiple of 4 and gemv_kernel's last parts are loaded one by one
// (us, gemv_kernel and rows: 1024 x 512, C=32 L=16 3.4 4.2; 1024 x 2048, C=64
// L=32 4.6 5.3; 256 x 2048, C=64 L=32 4.4 4.2; 256 x 131, C=32 L=16 5.9 4.2;
// 256 x 2050, C=64 L=64 5.1 4.4; 256 x 1025, C=32 L=64 3.9 4.2).
inline bool gemv_rows_short(const Plan& p, int64_t lanes, int64_t cus) {
  const bool ragged = p.k % 4 != 0;
  if (p.C >= 64) return (p.L < kWave && lanes <= 32 * cus) || (ragged && lanes <= 64 * cus);
  return ragged && p.L < kWave && lanes <= 32 * cus;
}
inline int gemv_rows_per_wave(const Plan& p, int64_t m) {
  if (p.order != DPIA_ORDER_CONTIGUOUS || p.nv != 4 || p.C % 32) return 0;
  const int64_t lanes = m * p.L, cus = device_cus();
  if (p.L > 256) return p.L % kWave == 0 && 8 * p.k >= p.W * p.row_parts ? kWave : 0;
  if (p.L != 16 && p.L != 32 && p.L != kWave) return 0;
  if (lanes <= 128 * cus) return p.C >= 96 || gemv_rows_short(p, lanes, cus) ? 16 : 0;
  return p.L != 16 && p.C >= 64 && lanes <= 256 * cus ? 32 : 0;
}

template <class Op>
hipError_t launch_gemv_rows(const Plan& p, const Op& op, int64_t m, int64_t lda, int rows,
                            hipStream_t stream) {
  auto go = [&](auto comb, auto nrows) {
    constexpr int COMBINE = decltype(comb)::value;
    constexpr int ROWS = decltype(nrows)::value;
    constexpr int D = ROWS == kWave ? 1 : 2;           // tiles in flight
    const int64_t slices = p.L / ROWS;
    GemvArgs a{};
    a.m = m;
    a.k = p.k;
    a.lda = lda;
    a.W = static_cast<int>(p.W);
    a.L = static_cast<int>(p.L);
    a.C = static_cast<int>(p.C);
    a.parts = p.row_parts;
    a.teams_per_wg = rows_teams(slices, m, bounded_grid(device_cus(), p.max_grid, kWave));
    const int waves =
        slices >= kRowsWaves ? kRowsWaves : a.teams_per_wg * static_cast<int>(slices);
    a.stage_off = kRowsScratch +
                  static_cast<int>((a.teams_per_wg * p.L * sizeof(typename Op::T) + 15) / 16 * 16);
    const size_t lds = a.stage_off + sizeof(float) * static_cast<size_t>(waves) *
                                         rows_stage_floats<ROWS>(Op::View::kOps);
    const int64_t need = (m + a.teams_per_wg - 1) / a.teams_per_wg;
    const int64_t grid = bounded_grid(need, p.max_grid, kWave * waves);
    Op op_copy = op;
    void* args[] = {&op_copy, &a};
    auto kern = gemv_rows_kernel<Op, COMBINE, ROWS, D>;
    return hipLaunchKernel(reinterpret_cast<const void*>(kern), dim3(grid),
                           dim3(kWave * waves), args, lds, stream);
  };
  auto by_rows = [&](auto comb) {
    if (rows == 16) return go(comb, ic<16>{});
    if (rows == 32) return go(comb, ic<32>{});
    return go(comb, ic<kWave>{});
  };
  return p.combine == DPIA_COMBINE_TREE ? by_rows(ic<kTree>{}) : by_rows(ic<kSeq>{});
}

// The plan of strided binary32 rows with few lanes in all: one lane per thread
// with batches of 64 steps, as thin_plan (reduce.h) does for a dot.  Shorter
// lanes are in flight whole with four of them to a thread (us, that and one to
// a thread: 1024 rows of L=64, C=8 2.5 3.4, C=16 3.4 3.8, C=24 4.3 4.5, C=32
// 4.8 4.4, C=64 7.9 6.3; 64 rows of L=16, C=24 3.7 3.4, C=32 4.5 3.5, C=40
// 4.3 4.0; 256 of L=32, C=32 3.5 3.7).
inline Plan gemv_thin_plan(const Plan& p, int64_t m) {
  Plan q = p;
  q.nv = 1;
  q.team = static_cast<int>(q.L);
  q.teams_per_wg = q.team >= 256 ? 1 : 256 / q.team;
  while (q.teams_per_wg > 1 && (q.teams_per_wg / 2) * q.team >= kWave &&
         (m + q.teams_per_wg - 1) / q.teams_per_wg < 4 * device_cus())
    q.teams_per_wg /= 2;
  q.wg_threads = q.teams_per_wg * q.team;
  const size_t per_team = q.combine == DPIA_COMBINE_SEQ ? q.L : (q.team > kWave ? q.team / kWave : 1);
  q.lds_bytes = (static_cast<size_t>(q.teams_per_wg) * per_team * sizeof(float) + 31) / 16 * 16;
  q.stage = false;
  return q;
}

// (A bounded grid has to be large enough for work-groups of fewer than 256
// threads: 4096 x 1024, C=64 L=16 under 300 work-groups 12.3 us, 8.5 not thin.)
inline bool gemv_thin(const Plan& p, int64_t m) {
  if (p.order != DPIA_ORDER_STRIDED || p.nv != 4 || p.team < 4 || p.L > 256 ||
      m * p.L > 256 * static_cast<int64_t>(device_cus()) || p.C < 32)
    return false;
  const Plan q = gemv_thin_plan(p, m);
  return q.wg_threads >= 256 || !grid_is_bound(q, (m + q.teams_per_wg - 1) / q.teams_per_wg);
}

// Whether staged contiguous teams are launched one wavefront's worth (or one
// team) to a work-group instead of 256 threads.  Wavefronts that share a
// work-group hold its 18 KB regions each until the slowest is done; alone they
// come and go by themselves, which evens out the last round.  Measured, 256
// threads and this (us):
//   binary32  L=64  16384^2 C=256 185.5 180.5   16384 x 4096 C=64 56.2 54.8
//             L=32  8192^2 C=256 50.7 49.2      16384^2 C=512 186 182
//   bf16      L=64  16384 x 4096 C=64 47.8 43.8 4096^2 C=64 14.8 14.3
//             L=128 8192^2 C=64 50.8 47.3       16384 x 4096 C=32 58.0 53.6
//   fp8       L=64  16384 x 4096 C=64 38.4 34.8 8192^2 C=128 36.1 33.9
// and where it does not: binary32 L=128 (16384^2 C=128 189.5 192.9, 8192 x
// 1000 25.7 26.9), L=8 (16384^2 190.1 196.6); bf16 L=64 with longer lanes
// (16384^2 C=256 148.8 150.5), L=16 and 32 (8192^2 C=256 L=32 40.0 40.8).
inline bool gemv_by_wave(const Plan& p, bool f32) {
  if (!p.stage || p.order != DPIA_ORDER_CONTIGUOUS) return false;
  if (f32) return p.L == 32 || p.L == kWave;
  return p.L == 2 * kWave || (p.L == kWave && p.C <= 128);
}

inline GemvArgs gemv_args(const Plan& p, int64_t m, int64_t lda) {
  GemvArgs a{};
  a.m = m;
  a.k = p.k;
  a.lda = lda;
  a.W = static_cast<int>(p.W);
  a.L = static_cast<int>(p.L);
  a.C = static_cast<int>(p.C);
  a.team = p.team;
  a.teams_per_wg = p.teams_per_wg;
  a.team_lds_elems = (p.combine == DPIA_COMBINE_SEQ) ? static_cast<int>(p.L)
                                                     : (p.team > 64 ? p.team / 64 : 1);
  a.parts = p.row_parts;
  a.stage_off = p.stage ? static_cast<int>(p.stage_off) : -1;
  return a;
}

// A plan of gemv_thin_plan.
template <class Op>
hipError_t launch_gemv_thin(const Plan& p, const Op& op, int64_t m, int64_t lda,
                            hipStream_t stream) {
  GemvArgs a = gemv_args(p, m, lda);
  auto kern = p.combine == DPIA_COMBINE_TREE ? gemv_kernel<Op, kStrided, 1, kTree, 256>
                                             : gemv_kernel<Op, kStrided, 1, kSeq, 256>;
  Op op_copy = op;
  void* args[] = {&op_copy, &a};
  return hipLaunchKernel(reinterpret_cast<const void*>(kern), dim3(grid_size(p)),
                         dim3(p.wg_threads), args, p.lds_bytes, stream);
}

template <class Op, int MAXNV>
hipError_t launch_gemv(const Plan& p, const Op& op, int64_t m, int64_t lda, hipStream_t stream) {
  GemvArgs a = gemv_args(p, m, lda);
  Plan q = p;
  const int teams = p.team < kWave ? kWave / p.team : 1;
  if (teams < p.teams_per_wg && p.nv == MAXNV && gemv_by_wave(p, Op::kF32Rows) &&
      (p.max_grid == 0 || (m + teams - 1) / teams <= static_cast<int64_t>(p.max_grid))) {
    q.teams_per_wg = a.teams_per_wg = teams;
    q.wg_threads = teams * p.team;
    const size_t lanes = static_cast<size_t>(teams) * a.team_lds_elems * sizeof(typename Op::T);
    a.stage_off = static_cast<int>((lanes + 15) / 16 * 16);
    q.lds_bytes = a.stage_off +
                  static_cast<size_t>(q.wg_threads / kWave) * stage_floats(kWave) * sizeof(float);
  }
  const int64_t grid = grid_size(q);
  return with_order_combine(p.order, p.combine, [&](auto ord, auto comb) {
    constexpr int ORDER = decltype(ord)::value;
    constexpr int COMBINE = decltype(comb)::value;
    return with_nv<MAXNV>(p.nv, [&](auto nvc) {
      constexpr int NV = decltype(nvc)::value;
      auto kern = p.wg_threads <= 256 ? gemv_kernel<Op, ORDER, NV, COMBINE, 256>
                                      : gemv_kernel<Op, ORDER, NV, COMBINE, 1024>;
      if constexpr (ORDER == kContiguous && NV == MAXNV && !std::is_same<Op, GemvU32>::value) {
        if (p.stage) kern = gemv_kernel<Op, ORDER, NV, COMBINE, 256, true>;
      }
      if constexpr (ORDER == kStrided && Op::kF32Rows) {
        // (the staged fold loads 16-byte pieces of every row)
        if (p.stage && lda % 4 == 0) kern = gemv_kernel<Op, ORDER, NV, COMBINE, 256, true>;
      }
      Op op_copy = op;
      void* args[] = {&op_copy, &a};
      return hipLaunchKernel(reinterpret_cast<const void*>(kern), dim3(grid),
                             dim3(q.wg_threads), args, q.lds_bytes, stream);
    });
  });
}

}  // namespace dpia
