// dot and asum under a DPIA strategy (blocked dot product, Sec. 2.1 eq. (2);
// asum and dot are benchmarks of Sec. 7.1).
//
// Kernel 1 evaluates the mapWorkgroup level: every chunk of W = L*C elements
// is reduced by one team (lane folds, then the work-group combine) and its
// value is written to the workspace, partial[g] (the hoisted newGlobal
// temporary of Sec. 6.3: one slot per parforWorkgroup iteration).  The outer
// reduceSeq over partial[0..G) from +0 in chunk order then runs either in a
// second kernel (2 passes) or in the last work-group to finish (1 pass).  Both
// evaluate the same expression and give the same bits.
//
// 1 pass: every thread stores its chunk values device-coherently, waits until
// they are in memory, and meets the work-group at a barrier; then one thread
// counts the work-group's arrival (relaxed, last_to_arrive) and a second
// barrier hands its answer on.  The last work-group reads few values with
// device-coherent loads; where there are more, every wavefront that reads does
// an agent-scope acquire first and loads plainly (final_fold).  No work-group
// writes its L2 back.
#pragma once

#include <type_traits>

#include "device.h"
#include "fed.h"
#include "fold.h"
#include "ops.h"
#include "rows.h"
#include "host.h"
#include "plan.h"

namespace dpia {

struct ReduceArgs {
  int64_t items;          // G chunks
  int64_t values;         // values the outer fold reads (G * values per chunk)
  int64_t n;              // elements; the last chunk may be partly beyond n
  int64_t W;
  int L, C, team, teams_per_wg;
  int team_lds_elems;     // LDS elements of T per team
  int stage_off;          // byte offset of the LDS staging region, -1: none
  int one_pass;
  int out_f64;            // Kahan 64 only: write a double
  void* partials;
  unsigned int* counter;
  void* nodes;            // split teams: kSplitMax nodes per chunk, or nullptr
  unsigned int* node_cnt; // split teams: one arrival count per chunk
  void* out;
};

// The arrival of a 1-pass work-group (one thread calls this, when all of the
// work-group's chunk values are in memory): true for the last one of the
// launch.  The counter is left at zero.
__device__ __forceinline__ bool last_of(unsigned int* counter, unsigned count) {
  if (__hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != count - 1)
    return false;
  __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return true;
}

// The same for launches of many work-groups.  Arrivals at one word are taken
// one by one, about 9 ns each, and the work-groups of a launch end together;
// so more than 256 of them count in kArriveGroups words, and the last of each
// word in the first one (asum of 2^23, C=64 L=256, 512 work-groups 15.6 ->
// 13.0 us; 256 work-groups would lose 0.7 us by the second step).  The words
// fit the 256 bytes that a workspace keeps for them.
constexpr unsigned kArriveGroups = 32;
static_assert((1 + kArriveGroups) * sizeof(unsigned) <= kWsAlign, "the workspace's counters");
__device__ __forceinline__ bool last_to_arrive(unsigned int* counter) {
  if (gridDim.x <= 256) return last_of(counter, gridDim.x);
  const unsigned g = blockIdx.x % kArriveGroups;
  if (!last_of(counter + 1 + g, (gridDim.x - g + kArriveGroups - 1) / kArriveGroups)) return false;
  return last_of(counter, kArriveGroups);
}

// STAGED: the contiguous order through LDS (see chunk_value).
// MAXT: the largest work-group it is launched with (256 or 1024); the
// 256-thread build may use more registers than the 1024-thread one.
template <class Op, int ORDER, int NV, int COMBINE, int FINAL, int VEC, int MAXT, bool STAGED>
__global__ void __launch_bounds__(MAXT) reduce_kernel(Op op, ReduceArgs a) {
  using T = typename Op::T;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  __shared__ int is_last;
  T* lds = reinterpret_cast<T*>(lds_raw);
  const int team_id = threadIdx.x / a.team;
  const int t = threadIdx.x - team_id * a.team;
  T* scratch = lds + team_id * a.team_lds_elems;
  float* stage = STAGED ? reinterpret_cast<float*>(lds_raw + a.stage_off) +
                              (threadIdx.x / kWave) * stage_floats(kWave)
                        : nullptr;
  T* partials = static_cast<T*>(a.partials);
  const int64_t stride = static_cast<int64_t>(gridDim.x) * a.teams_per_wg;
  // parforWorkgroup as a grid-stride loop: every thread of a work-group
  // runs the same iterations, so the barriers inside are uniform
  for (int64_t base = static_cast<int64_t>(blockIdx.x) * a.teams_per_wg; base < a.items;
       base += stride) {
    const int64_t g = base + team_id;
    const bool active = g < a.items;
    const auto view = op.chunk(active ? g : 0, a.W);
    const int64_t rest = a.n - g * a.W;
    const int limit = static_cast<int>(rest < a.W ? rest : a.W);
    if constexpr (VEC == 1 && COMBINE != kNone) {
      const T v = chunk_value<Op, ORDER, NV, COMBINE, STAGED>(view, active, t, a.team, a.L, a.C,
                                                              limit, scratch, stage);
      if (active && t == 0) store_coherent(partials + g, v);
    } else {
      chunk_values_wide<Op, ORDER, NV, COMBINE, VEC, STAGED>(view, active, t, a.team, a.L, a.C,
                                                             limit, scratch, partials, g, stage);
    }
  }
  if (a.one_pass) {
    // (the protocol at the head of this file: own stores in memory, barrier,
    // arrival, barrier)
    wait_memory();
    __syncthreads();
    if (threadIdx.x == 0) {
      is_last = last_to_arrive(a.counter);
    }
    __syncthreads();
    if (is_last) {
      final_fold<typename Op::Arith, FINAL, true>(partials, a.values, a.out, a.out_f64, lds,
                                                  !one_sign<Op>);
    }
  }
}

#ifndef DPIA_FED
#define DPIA_FED 1
#endif

// The mapWorkgroup level of a strategy with few chunks, fed by loader
// wavefronts (fed.h): staged contiguous lanes (teams of 64, 128 or 256 lanes,
// one per thread) or scalar strided lanes.  Each work-group takes ROWS lanes
// of one chunk (a slice; L / ROWS slices per chunk), its wave 0 folds them,
// one lane per thread, and waves 1 .. kFedLoaders load.  Uncombined slices store their lanes' values.  A tree
// combine over a split team: each slice reduces its ROWS lanes with the
// team's butterfly levels below ROWS and stores that node (device-coherent);
// the slice whose arrival completes the chunk's count applies the levels
// from ROWS up to the team over the nodes in lane order, which is the same
// tree (the levels are hierarchical), and stores the chunk value.  Lane rows
// that are not whole (the last chunk, when W does not divide n) are folded
// by wave 0 alone, as reduce_kernel folds them.  The same chunk values, the
// same 1-pass arrival and fold as reduce_kernel.
template <class Op, int ORDER, int COMBINE, int FINAL, int VEC, int ROWS>
__global__ void __launch_bounds__(kWave*(1 + kFedLoaders)) fed_reduce_kernel(Op op,
                                                                               ReduceArgs a) {
  using T = typename Op::T;
  using A = typename Op::Arith;
  static_assert(COMBINE != kSeq, "a sequential combine has barriers of the team alone");
  extern __shared__ __align__(16) unsigned char lds_raw[];
  __shared__ int is_last;
  T* lds = reinterpret_cast<T*>(lds_raw);
  float* ring = reinterpret_cast<float*>(lds_raw + a.stage_off);
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int lane = threadIdx.x & (kWave - 1);
  T* partials = static_cast<T*>(a.partials);
  static_assert(ORDER == kContiguous || VEC == 1, "strided slices are scalar lanes");
  const int Cel = a.C * VEC;
  const int S = a.L / ROWS;   // slices per chunk
  for (int64_t w = blockIdx.x; w < a.items * S; w += gridDim.x) {
    const int64_t g = w / S;
    const int s = static_cast<int>(w % S);
    const int row0 = s * ROWS;
    const auto view = op.chunk(g, a.W);
    const int64_t rest = a.n - g * a.W;
    const int limit = static_cast<int>(rest < a.W ? rest : a.W);
    T acc[VEC];
    if constexpr (ORDER == kStrided) {
      if (limit == a.W)
        fed_fold_strided<Op, ROWS>(view, a.L, a.C, wave, lane, row0, ring, acc[0]);
      else if (wave == 0)
        lane_folds<OneLane<Op>, kStrided, 1>(view, lane < ROWS, row0 + lane, a.L, a.C, limit, acc);
    } else {
      if (limit == a.W)
        fed_fold<Op, VEC, ROWS>(view, Cel, wave, lane, row0, ring, acc);
      else if (wave == 0)
        contiguous_staged<Op, VEC>(view, lane < ROWS, row0 + lane, a.C, limit, acc, ring);
    }
    if (wave == 0) {
      if constexpr (COMBINE == kNone) {
        if (lane < ROWS) {
          const int64_t l = g * a.L + row0 + lane;
#pragma unroll
          for (int j = 0; j < VEC; ++j) store_coherent(partials + l * VEC + j, acc[j]);
        }
      } else if (S == 1) {
#pragma unroll
        for (int j = 0; j < VEC; ++j) {
          T one[1] = {acc[j]};
          const T c = combine_lanes<A, 1, COMBINE>(one, lane, kWave, a.L, lds);
          if (lane == 0) store_coherent(partials + g * VEC + j, c);
        }
      } else if constexpr (VEC == 1) {
        T one[1] = {acc[0]};
        const T node = combine_lanes<A, 1, COMBINE>(one, lane, ROWS, a.L, lds);
        T* nodes = static_cast<T*>(a.nodes) + g * kSplitMax;
        unsigned last = 0;
        if (lane == 0) {
          store_coherent(nodes + s, node);
          wait_memory();
          last = __hip_atomic_fetch_add(a.node_cnt + g, 1u, __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT) == static_cast<unsigned>(S - 1);
        }
        if (__shfl(last, 0)) {   // every slice's node is stored
          T v = lane < S ? load_coherent(nodes + lane) : A::zero();
          butterfly_levels<A>(v, lane, S);
          if (lane == 0) {
            store_coherent(partials + g, v);
            __hip_atomic_store(a.node_cnt + g, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
        }
      }
    }
    __syncthreads();   // the ring may be written for the next slice
  }
  if (a.one_pass) {
    wait_memory();
    __syncthreads();
    if (threadIdx.x == 0) {
      is_last = last_of(a.counter, gridDim.x);
    }
    __syncthreads();
    if (is_last) {
      final_fold<typename Op::Arith, FINAL, true>(partials, a.values, a.out, a.out_f64, lds,
                                                  !one_sign<Op>);
    }
  }
}

// Contiguous lanes, ROWS to a wavefront (rows.h): `teams_per_wg` chunks to a
// work-group at once, the staging regions at `stage_off`.
template <class Op, int COMBINE, int FINAL, int VEC, int ROWS, int D>
__global__ void __launch_bounds__(kWave* kRowsWaves) rows_reduce_kernel(Op op, ReduceArgs a) {
  using T = typename Op::T;
  using A = typename Op::Arith;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  __shared__ int is_last;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int lane = static_cast<int>(threadIdx.x) & (kWave - 1);
  // wavefronts per chunk
  const int per_chunk = static_cast<int>(blockDim.x) / kWave / a.teams_per_wg;
  const int chunk = wave / per_chunk;
  const int t = static_cast<int>(threadIdx.x) - chunk * per_chunk * kWave;
  T* scratch = reinterpret_cast<T*>(lds_raw);          // (used by single chunks only)
  T* lanes = reinterpret_cast<T*>(lds_raw + kRowsScratch) + chunk * a.L * VEC;
  float* stage = reinterpret_cast<float*>(lds_raw + a.stage_off) +
                 wave * rows_stage_floats<ROWS>(Op::View::kOps);
  T* partials = static_cast<T*>(a.partials);
  const int slices = a.L / ROWS;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * a.teams_per_wg;
  for (int64_t g0 = static_cast<int64_t>(blockIdx.x) * a.teams_per_wg; g0 < a.items;
       g0 += stride) {
    const int64_t g = g0 + chunk;
    if (g < a.items) {
      const auto view = op.chunk(g, a.W);
      const int64_t rest = a.n - g * a.W;
      const int limit = static_cast<int>(rest < a.W ? rest : a.W);
      for (int s = wave - chunk * per_chunk; s < slices; s += per_chunk) {
        T acc[VEC];
        rows_fold<Op, VEC, ROWS, D>(view, s * ROWS, a.C * VEC, limit, stage, acc);
        if (ROWS == kWave || lane < ROWS) {
          const int l = s * ROWS + lane;
#pragma unroll
          for (int j = 0; j < VEC; ++j) {
            if constexpr (COMBINE == kNone)
              store_coherent(partials + (g * a.L + l) * VEC + j, acc[j]);
            else
              lanes[j * a.L + l] = acc[j];
          }
        }
      }
    }
    if constexpr (COMBINE != kNone) {
      __syncthreads();
#pragma unroll
      for (int j = 0; j < VEC; ++j) {
        const T c = combine_stored<A, COMBINE>(lanes + j * a.L, a.L, t, per_chunk * kWave, scratch);
        if (t == 0 && g < a.items) store_coherent(partials + g * VEC + j, c);
      }
      __syncthreads();   // the lane values may be written for the next chunk
    }
  }
  if (a.one_pass) {
    wait_memory();
    __syncthreads();
    if (threadIdx.x == 0) is_last = last_to_arrive(a.counter);
    __syncthreads();
    if (is_last)
      final_fold<A, FINAL, true>(partials, a.values, a.out, a.out_f64, lds_raw, !one_sign<Op>);
  }
}

template <class A, int FINAL>
__global__ void __launch_bounds__(1024) final_kernel(const typename A::T* partials, int64_t G,
                                                     void* out, int out_f64, int signs) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  final_fold<A, FINAL>(partials, G, out, out_f64, lds_raw, signs != 0);
}

template <class Op>
ReduceArgs reduce_args(const Plan& p, void* partials, void* counter, void* out, int out_f64,
                       bool one_pass) {
  ReduceArgs a{};
  a.items = p.items;
  a.values = p.values;
  a.n = p.n;
  a.W = p.W;
  a.L = static_cast<int>(p.L);
  a.C = static_cast<int>(p.C);
  a.team = p.team;
  a.teams_per_wg = p.teams_per_wg;
  a.team_lds_elems = (p.combine == DPIA_COMBINE_SEQ) ? static_cast<int>(p.L)
                                                     : (p.team > 64 ? p.team / 64 : 1);
  a.stage_off = p.stage ? static_cast<int>(p.stage_off) : -1;
  a.out_f64 = out_f64;
  a.partials = partials;
  a.counter = static_cast<unsigned int*>(counter);
  a.out = out;
  a.one_pass = one_pass ? 1 : 0;
  return a;
}

// Calls f(order, combine, nv, vec constants) for a plan.  Vector and
// uncombined shapes exist for the plain operations only (WIDE).
template <bool WIDE, class F>
hipError_t with_reduce_shape(const Plan& p, F&& f) {
  constexpr int MAXNV = kVecBytes / static_cast<int>(sizeof(float));
  if (p.V == 1 && p.combine != DPIA_COMBINE_NONE) {
    return with_order_combine(p.order, p.combine, [&](auto ord, auto comb) {
      return with_nv<MAXNV>(p.nv, [&](auto nvc) { return f(ord, comb, nvc, ic<1>{}); });
    });
  }
  if constexpr (WIDE) {
    auto by_order = [&](auto comb, auto nvc, auto vec) {
      if (p.order == DPIA_ORDER_STRIDED) return f(ic<kStrided>{}, comb, nvc, vec);
      return f(ic<kContiguous>{}, comb, nvc, vec);
    };
    if (p.V == 1)
      return with_nv<MAXNV>(p.nv, [&](auto nvc) { return by_order(ic<kNone>{}, nvc, ic<1>{}); });
    auto by_combine = [&](auto vec) {
      if (p.combine == DPIA_COMBINE_TREE) return by_order(ic<kTree>{}, vec, vec);
      if (p.combine == DPIA_COMBINE_SEQ) return by_order(ic<kSeq>{}, vec, vec);
      return by_order(ic<kNone>{}, vec, vec);
    };
    if (p.V == 2) return by_combine(ic<2>{});
    if (p.V == 4) return by_combine(ic<4>{});
  }
  return hipErrorInvalidValue;
}

// The same for a plan of thin_lanes: strided scalar lanes in work-groups of at
// most 256 threads.
template <bool WIDE, class F>
hipError_t with_thin_shape(const Plan& p, F&& f) {
  if (p.order != DPIA_ORDER_STRIDED || p.V != 1 || p.wg_threads > 256)
    return hipErrorInvalidValue;
  return with_nv<4>(p.nv, [&](auto nvc) {
    if (p.combine == DPIA_COMBINE_TREE) return f(ic<kStrided>{}, ic<kTree>{}, nvc, ic<1>{});
    if (p.combine == DPIA_COMBINE_SEQ) return f(ic<kStrided>{}, ic<kSeq>{}, nvc, ic<1>{});
    if constexpr (WIDE) return f(ic<kStrided>{}, ic<kNone>{}, nvc, ic<1>{});
    return hipErrorInvalidValue;
  });
}

// Lane rows per work-group when a plan's chunks are folded by
// fed_reduce_kernel (0: they are not): staged contiguous lanes, one lane per
// thread, fewer chunks than compute units (otherwise the launch has
// wavefronts enough), and a chunk's tiles a multiple of the loaders' depth
// for that row count.  A compute unit streams at most about 37 GB/s, so the
// chunks' lanes are split over as many work-groups as the compute units
// allow: uncombined lanes into 2 or 4 slices of a 64-lane team, tree-combined
// teams of 64, 128 or 256 lanes into up to kSplitMax slices when the call
// brings the workspace's split region (`can_split`); a 64-lane tree team may
// also stay whole.
template <int NOPS>
int fed_rows_strided(const Plan& p, bool can_split) {
  // scalar strided lanes, L a power of two from 16 to 512, whole tiles of
  // kFedStrideRows steps; a tree needs the split region beyond one slice
  if (p.V != 1 || p.combine == DPIA_COMBINE_SEQ) return 0;
  if (p.L < 16 || p.L > 512 || (p.L & (p.L - 1)) || p.C % kFedStrideRows) return 0;
  const int64_t cus = device_cus();
  if (p.items > 2 * cus) return 0;
  const bool split = can_split && p.split_off;
  const int64_t ntiles = p.C / kFedStrideRows;
  auto fits = [&](int depth) { return ntiles >= depth && ntiles % depth == 0; };
  auto ok = [&](int rows, int depth, int64_t most) {
    const int64_t per = p.L / rows;
    if (rows > p.L || p.items * per > most || !fits(depth)) return false;
    if (p.combine == DPIA_COMBINE_TREE && per > 1 && (!split || per > kSplitMax)) return false;
    return true;
  };
  // one work-group per compute unit, else two (what their LDS allows)
  for (const int64_t most : {cus, 2 * cus}) {
    if (ok(16, fed_depth<16, NOPS>(), most)) return 16;
    if (ok(32, fed_depth<32, NOPS>(), most)) return 32;
    if (ok(kWave, fed_depth<kWave, NOPS>(), most)) return kWave;
  }
  return 0;
}

template <int NOPS>
int fed_rows(const Plan& p, bool can_split) {
  if (!DPIA_FED) return 0;
  if (p.op != DPIA_OP_DOT && p.op != DPIA_OP_ASUM) return 0;
  if (p.order == DPIA_ORDER_STRIDED) return fed_rows_strided<NOPS>(p, can_split);
  if (!p.stage || p.order != DPIA_ORDER_CONTIGUOUS) return 0;
  if (p.teams_per_wg != 1 || p.combine == DPIA_COMBINE_SEQ) return 0;
  if (p.V != 1 && p.V != 4) return 0;
  const bool split = can_split && p.split_off && p.combine == DPIA_COMBINE_TREE && p.V == 1;
  if (p.team != kWave && !(split && (p.team == 128 || p.team == 256))) return 0;
  const int64_t cus = device_cus();
  if (p.items >= cus || (p.C * p.V) % kFedStage) return 0;
  const int64_t ntiles = p.C * p.V / kFedStage;
  auto fits = [&](int depth) { return ntiles >= depth && ntiles % depth == 0; };
  if (p.combine == DPIA_COMBINE_NONE || split) {
    const int64_t per16 = p.team / 16, per32 = p.team / 32;   // slices per chunk
    if (per16 <= kSplitMax && p.items * per16 <= cus && fits(fed_depth<16, NOPS>())) return 16;
    if (per32 <= kSplitMax && p.items * per32 <= cus && fits(fed_depth<32, NOPS>())) return 32;
    if (p.items * (p.team / kWave) <= cus && fits(fed_depth<kWave, NOPS>())) return kWave;
    return 0;
  }
  return fits(fed_depth<kWave, NOPS>()) ? kWave : 0;
}

// The plan of a scalar strided launch with few lanes: one lane per thread (as
// far as a chunk's lanes fit 256 threads), for the operations' deep batches.
// A thread that holds 4 lanes brings 16 bytes per load, but there are a
// quarter as many threads, each with only as many loads in flight as it has
// registers.  What is in flight is lanes x batch: with one lane per thread a
// batch is 64 steps of it.  Measured, 4 lanes and 1 per thread, each with its
// best batch (us; lanes in the launch):
//   dot  2^26 C=8192 L=16 (8,192)    735   221    asum 531 143
//   dot  2^26 C=1024 L=64 (65,536)   97.5  90.8   asum 60.4 46.2
//   dot  2^25 C=512 L=256 (65,536)   52.0  44.5   asum 34.2 25.5
//   dot  2^23 C=256 L=64 (32,768)    26.6  16.8   asum 19.3 12.2
//   dot  2^20 C=256 L=16 (4,096)     26.9  11.7   asum 21.1 9.3
//   dot  2^25 C=256 L=16 (131,072)   67.4  70.3   asum 35.8 36.3
//   dot  2^26 C=256 L=64 (262,144)   99.9  101    asum 50.7 47.9
//   dot  2^26 C=64 L=64 (2^20)       127   116    asum 60.0 50.3
// Hence up to 256 lanes per compute unit; an asum, with one operand to keep
// in flight, also up to 512, and with a wavefront per chunk (L = 64) beyond
// (2 passes: C=16 2^26 69.1 68.6, 2^24 21.5 19.6; 1 pass: see below).
// Lanes that not even `nv` to a thread make a team of 256 threads are left to
// the plan as it is, with the operation's own batches: 64 steps of two lanes
// are 128 registers of loads, all that a thread of a larger work-group has
// (L=514 C=256, 60 chunks: Kahan 47.9 us, 74.8 with deep batches).
constexpr int kThinTeam = 256;
inline int thin_nv(const Plan& p) {
  int nv = 1;
  while (p.L / nv > kThinTeam && nv < p.nv) nv *= 2;
  return p.L / nv > kThinTeam ? 0 : nv;
}
// Lanes so short that four of them to a thread have them in flight whole gain
// nothing, and more threads cost (us; not thin and thin):
//   asum 2^22 C=8 L=64    9.4 11.0   C=16 8.7  8.7
//   dot  512 chunks of C=4 L=64 5.8 6.4   C=8 6.4 6.4
// A 1-pass launch pays for every work-group's arrival besides (last_of), so
// its lanes are one to a thread from 32 elements on (a dot with a last chunk in
// part from 16: 8 chunks of C=16 L=64 4.8 us not thin, 4.0 thin; whole 3.6,
// 3.7), and its work-groups hold 256 threads up to 64 (256 chunks of L=64, dot:
// C=16 5.7 us not thin, 7.9 in work-groups of one wavefront, 5.8 in full ones;
// C=32 7.2, 8.4, 6.7; C=64 8.9, 8.6, 7.4).  Teams of a few threads put so many
// chunks into a work-group that there are too few of those: such lanes are one
// to a thread whatever their length, from where it pays (1 pass, asum C=8, not
// thin and thin; lanes in the launch):
//   L=4   8,192 6.9 6.2    16,384 9.9 6.8   65,536 28.8 15.8
//   L=16  24,576 7.5 6.8   32,768 7.6 6.9   65,536 11.8 8.8
//   L=32  32,768 5.9 6.6   49,152 8.9 8.0   65,536 9.1 8.5
// Wider ones beyond 384 lanes per compute unit have work-groups enough, each
// thin one more to arrive (asum C=32 L=64, 65,536 lanes 9.7 9.0; 98,304 12.6
// 10.5; 131,072 10.8 11.1; 262,144 13.3 16.0; L=256, 98,304 10.1 9.3; 131,072
// 10.5 10.8).
constexpr int kThinRound = 64;     // elements a lane has in flight at once
inline bool thin_lanes(const Plan& p) {
  if (p.order != DPIA_ORDER_STRIDED || p.V != 1 || p.nv == 1 || !thin_nv(p)) return false;
  const int64_t lanes = p.items * p.L, cus = device_cus();
  if (p.passes == 1) {
    const bool part = p.op == DPIA_OP_DOT && p.n % p.W != 0;
    const int64_t narrow = p.L <= 8 ? 64 : p.L <= 16 ? 128 : p.L <= 32 ? 192 : INT64_MAX / cus;
    if (p.C < (part ? 16 : 32) && lanes < narrow * cus) return false;
    if (p.C < kThinRound && p.L >= kWave && lanes > 384 * cus) return false;
  } else if (p.L >= kWave && p.C < (p.op == DPIA_OP_ASUM ? 16 : 8)) {
    return false;
  }
  if (p.op == DPIA_OP_ASUM) return p.L == kWave || lanes <= 512 * cus;
  return lanes <= 256 * cus;
}

inline Plan thin_plan(const Plan& p) {
  if (!thin_lanes(p)) return p;
  Plan q = p;
  q.nv = thin_nv(p);
  if (q.nv == p.nv) return p;
  q.team = static_cast<int>(q.L / q.nv);
  q.teams_per_wg = q.team >= kThinTeam ? 1 : kThinTeam / q.team;
  while ((q.passes == 2 || q.C >= kThinRound) && q.teams_per_wg > 1 &&
         (q.teams_per_wg / 2) * q.team >= kWave &&
         (q.items + q.teams_per_wg - 1) / q.teams_per_wg <
             bounded_grid(device_cus(), q.max_grid, kThinTeam))
    q.teams_per_wg /= 2;
  q.wg_threads = q.teams_per_wg * q.team;
  size_t lds = 0;
  if (q.combine == DPIA_COMBINE_SEQ)
    lds = static_cast<size_t>(q.teams_per_wg) * q.L * q.acc_bytes;
  else if (q.combine == DPIA_COMBINE_TREE && q.team > kWave)
    lds = static_cast<size_t>(q.teams_per_wg) * (q.team / kWave) * q.acc_bytes;
  if (q.passes == 1 && lds < kFoldLds) lds = kFoldLds;
  q.lds_bytes = (lds + 16 + 15) / 16 * 16;
  return q;
}

// Lane rows per wavefront of a contiguous launch (0: contiguous_staged, 64
// lanes to a wavefront and a thread for each of a chunk's lanes).  Measured,
// that and with 16, 32 or 64 rows (us; lanes in the launch):
//   dot  2^20 C=256 L=16 (4,096)      15.8  16: 10.7     asum 12.6 9.0
//   dot  2^26 C=8192 L=16 (8,192)     339   16: 103      asum 242  73.6
//   dot  2^26 C=4096 L=64 (16,384)    178   16: 92  32: 114   asum 129  54.9
//   dot  2^25 C=1024 L=64 (32,768)    59.6  16: 52  32: 51.8  asum 41.8 35.9
//   dot  2^25 C=512 L=64 (65,536)     52.8  16: 51  32: 48.4  asum 29.9 34.2, 28.1
//   dot  2^23 C=64 L=64 (131,072)     22.2  16: 29.7 32: 23.8
// Chunks of 128 or 256 lanes give every work-group 4 wavefronts of 64 rows
// already; 32 rows help where two operands' rows are long, since a row is
// then read 256 bytes at a time (2^25 C=1024 L=256 70.7 -> 57.4 us, 2^26
// C=512 L=256 94 -> 86; asum 2^25 C=512 27.6 -> 30.6), up to 512 lanes per
// compute unit, 192 where the lanes are not whole wavefronts (L=96 C=512, 700
// chunks: 51.3 us, 56.4 in rows).  Longer teams had a thread per lane without
// staging (2^26 C=128 L=1024 304 -> 85.5 us).
// A row tile is 128 elements of 16 rows or 64 of 32, whether or not a row has
// them, so short lanes stay with contiguous_staged (us, that and rows):
//   dot  256 chunks of L=16  C=32 6.0 6.9    C=64 7.5 7.3   C=96 8.3 7.5
//   asum 256 chunks of L=32  C=32 5.7 6.9    C=64 6.4 6.8   C=96 7.5 7.4
//   asum 1024 chunks of L=64 C=128 11.5 12.1 C=256 17.3 18.6 C=384 23.4 22.9
//   dot  64 chunks of L=16   C=32 5.9 6.2    C=64 6.7 6.2
//        256 of L=16 C=64, 2 passes 7.1 6.6   360 8.7 7.5   512 7.4 7.6
// and the two-step arrival of a 1-pass launch of 512 work-groups costs what
// rows gain below 256 elements (asum, 512 chunks of L=64: C=128 12.0 13.3,
// C=256 16.1 16.1).
inline int rows_min_elems(const Plan& p, int rows, int64_t lanes) {
  if (rows == 32) return 384;
  if (p.passes == 1 && p.items * (p.L / rows) >= 2 * kRowsWaves * device_cus()) return 256;
  return p.op == DPIA_OP_DOT && lanes <= (p.passes == 1 ? 8 : 24) * device_cus() ? 64 : 96;
}
inline int rows_per_wave(const Plan& p) {
  if (p.order != DPIA_ORDER_CONTIGUOUS || p.dt != DPIA_F32 || p.nv != 4) return 0;
  if ((p.V != 1 && p.V != 4) || (p.C * p.V) % 32) return 0;
  const int64_t lanes = p.items * p.L, cus = device_cus();
  if (p.L > 256) return p.L % kWave == 0 ? kWave : 0;
  if (p.L > kWave)
    return p.op == DPIA_OP_DOT && p.C * p.V >= 512 && p.L % 32 == 0 &&
                   lanes <= (p.L % kWave ? 192 : 512) * cus ? 32 : 0;
  if (p.L != 16 && p.L != 32 && p.L != kWave) return 0;
  const int rows = lanes <= 128 * cus ? 16 : (p.L != 16 && lanes <= 256 * cus ? 32 : 0);
  return rows && p.C * p.V >= rows_min_elems(p, rows, lanes) ? rows : 0;
}

template <class Op, int FINAL>
hipError_t launch_rows(const Plan& p, const Op& op, const ReduceArgs& a, int rows,
                       hipStream_t stream) {
  constexpr int NOPS = Op::View::kOps;
  auto go = [&](auto comb, auto vec, auto nrows) {
    constexpr int COMBINE = decltype(comb)::value;
    constexpr int VEC = decltype(vec)::value;
    constexpr int ROWS = decltype(nrows)::value;
    // tiles in flight: a tile is 32 registers per operand
    constexpr int D = ROWS == kWave ? 1 : (NOPS == 1 ? 4 : 2);
    const int64_t slices = p.L / ROWS;
    ReduceArgs a_copy = a;
    a_copy.teams_per_wg =
        rows_teams(slices, p.items,
                   bounded_grid(a.one_pass ? device_cus() / 4 : device_cus(), p.max_grid, kWave));
    const int waves = slices >= kRowsWaves
                          ? kRowsWaves : a_copy.teams_per_wg * static_cast<int>(slices);
    a_copy.stage_off = kRowsScratch;
    if (COMBINE != kNone)
      a_copy.stage_off += static_cast<int>(
          (a_copy.teams_per_wg * p.L * VEC * sizeof(typename Op::T) + 15) / 16 * 16);
    const size_t lds = a_copy.stage_off + sizeof(float) * static_cast<size_t>(waves) *
                                              rows_stage_floats<ROWS>(NOPS);
    const int64_t need = (p.items + a_copy.teams_per_wg - 1) / a_copy.teams_per_wg;
    const int64_t grid = bounded_grid(need, p.max_grid, kWave * waves);
    Op op_copy = op;
    void* args[] = {&op_copy, &a_copy};
    auto kern = rows_reduce_kernel<Op, COMBINE, FINAL, VEC, ROWS, D>;
    return hipLaunchKernel(reinterpret_cast<const void*>(kern), dim3(grid),
                           dim3(kWave * waves), args, lds, stream);
  };
  auto by_rows = [&](auto comb, auto vec) {
    if (rows == 16) return go(comb, vec, ic<16>{});
    if (rows == 32) return go(comb, vec, ic<32>{});
    return go(comb, vec, ic<kWave>{});
  };
  auto by_combine = [&](auto vec) {
    if (p.combine == DPIA_COMBINE_TREE) return by_rows(ic<kTree>{}, vec);
    if (p.combine == DPIA_COMBINE_SEQ) return by_rows(ic<kSeq>{}, vec);
    if constexpr (FINAL == kFinalPlain) return by_rows(ic<kNone>{}, vec);
    return hipErrorInvalidValue;
  };
  if constexpr (FINAL == kFinalPlain)
    if (p.V == 4) return by_combine(ic<4>{});
  return by_combine(ic<1>{});
}

template <class Op, int FINAL>
hipError_t launch_fed(const Plan& p, const Op& op, const ReduceArgs& a, int rows,
                      hipStream_t stream) {
  const int64_t grid = p.items * (p.L / rows);
  // the ring from the start of the LDS: the kernel's combines within one
  // wavefront need no LDS, and the 1-pass fold uses it after the chunks
  size_t lds = static_cast<size_t>(fed_ring_floats()) * sizeof(float);
  lds = (lds + 16 + 15) / 16 * 16;
  Op op_copy = op;
  ReduceArgs a_copy = a;
  a_copy.stage_off = 0;
  void* args[] = {&op_copy, &a_copy};
  const bool strided = p.order == DPIA_ORDER_STRIDED;
  auto go = [&](auto comb, auto vec, auto nrows) {
    constexpr int COMBINE = decltype(comb)::value;
    constexpr int VEC = decltype(vec)::value;
    constexpr int ROWS = decltype(nrows)::value;
    auto kern = strided && VEC == 1
                    ? fed_reduce_kernel<Op, (VEC == 1 ? kStrided : kContiguous), COMBINE, FINAL,
                                        VEC, ROWS>
                    : fed_reduce_kernel<Op, kContiguous, COMBINE, FINAL, VEC, ROWS>;
    return hipLaunchKernel(reinterpret_cast<const void*>(kern), dim3(grid),
                           dim3(kWave * (1 + kFedLoaders)), args, lds, stream);
  };
  auto by_rows = [&](auto comb, auto vec) {
    if (rows == 16) return go(comb, vec, ic<16>{});
    if (rows == 32) return go(comb, vec, ic<32>{});
    return go(comb, vec, ic<kWave>{});
  };
  if constexpr (FINAL != kFinalPlain) {
    return by_rows(ic<kTree>{}, ic<1>{});   // compensated: scalar, combined lanes
  } else {
    if (p.combine == DPIA_COMBINE_TREE)
      return p.V == 4 ? go(ic<kTree>{}, ic<4>{}, ic<kWave>{}) : by_rows(ic<kTree>{}, ic<1>{});
    return p.V == 4 ? by_rows(ic<kNone>{}, ic<4>{}) : by_rows(ic<kNone>{}, ic<1>{});
  }
}

// The mapWorkgroup level: chunk values into `partials`; with one_pass the
// last work-group also folds them into `out`.
template <class Op, int FINAL>
hipError_t launch_chunks(const Plan& p, const Op& op, const ReduceArgs& a, hipStream_t stream) {
  if (p.items == 0) return hipSuccess;
  // (the loaders keep the tiles in flight, so deeper load batches would only
  // add registers)
  const bool can_split = a.nodes != nullptr;
  using Fed = typename BaseOp<Op>::type;
  if constexpr (Op::View::kStageable) {
    // (Loader wavefronts take 64-lane chunks whole, but a last chunk in part is
    // folded by one wavefront alone: 3,000,000 elements, C=512 L=64: 27.4 us,
    // 15.8 with 16 rows; without such a chunk 2^20, C=256 L=64 8.0 and 10.8, asum
    // of 2^21, C=512 8.3 and 12.5.  Kahan's chunks are whole.)
    const int per_wave = rows_per_wave(p);
    const int rows = fed_rows<Op::View::kOps>(p, can_split);
    if (rows && !(rows == kWave && per_wave == 16 && p.n % p.W != 0) &&
        (FINAL == kFinalPlain || (p.V == 1 && p.combine == DPIA_COMBINE_TREE)))
      return launch_fed<Fed, FINAL>(p, static_cast<const Fed&>(op), a, rows, stream);
    if (per_wave)
      return launch_rows<Fed, FINAL>(p, static_cast<const Fed&>(op), a, per_wave, stream);
  }
  const int64_t grid = grid_size(p);
  auto go = [&](auto ord, auto comb, auto nvc, auto vec) {
    constexpr int ORDER = decltype(ord)::value;
    constexpr int COMBINE = decltype(comb)::value;
    constexpr int NV = decltype(nvc)::value;
    constexpr int VEC = decltype(vec)::value;
    auto kern = reduce_kernel<Op, ORDER, NV, COMBINE, FINAL, VEC, 256, false>;
    if constexpr (!is_deep<Op>) {
      if (p.wg_threads > 256)
        kern = reduce_kernel<Op, ORDER, NV, COMBINE, FINAL, VEC, 1024, false>;
    }
    if constexpr (ORDER == kContiguous && NV == 4 && Op::View::kStageable) {
      if (p.stage) kern = reduce_kernel<Op, ORDER, NV, COMBINE, FINAL, VEC, 256, true>;
    }
    Op op_copy = op;
    ReduceArgs a_copy = a;
    void* args[] = {&op_copy, &a_copy};
    return hipLaunchKernel(reinterpret_cast<const void*>(kern), dim3(grid), dim3(p.wg_threads),
                           args, p.lds_bytes, stream);
  };
  if constexpr (is_deep<Op>)
    return with_thin_shape<FINAL == kFinalPlain>(p, go);
  else
    return with_reduce_shape<FINAL == kFinalPlain>(p, go);
}

// The outer reduceSeq over G chunk values, as a kernel of its own: 4
// wavefronts while one block of theirs holds the values (4,096, or 2,048
// pairs), else 16.
template <class Op, int FINAL>
hipError_t launch_fold(int64_t G, const void* partials, void* out, int out_f64,
                       hipStream_t stream) {
  using T = typename Op::T;
  const T* pp = static_cast<const T*>(partials);
  int signs = !one_sign<Op>;
  void* args[] = {&pp, &G, &out, &out_f64, &signs};
  auto kern = final_kernel<typename Op::Arith, FINAL>;
  const int threads = G > 4 * kWave * kFoldLaneValues<T> ? 1024 : 256;
  return hipLaunchKernel(reinterpret_cast<const void*>(kern), dim3(1), dim3(threads), args,
                         kFoldLds, stream);
}

// Both passes of a reduction: chunk values into `partials`, then the outer
// fold (1 pass: in the last work-group, which needs `counter` at zero and
// leaves it at zero; 2 passes: a second kernel).  `split`: the workspace's
// split region (p.split_off), or nullptr where the call has none.
template <class Op, int FINAL>
hipError_t launch_reduce(const Plan& p, const Op& op, void* out, int out_f64, void* partials,
                         void* counter, hipStream_t stream, void* split = nullptr) {
  const bool two_pass = p.passes == 2 || p.items == 0;
  ReduceArgs a = reduce_args<Op>(p, partials, counter, out, out_f64, !two_pass);
  if (split && p.split_off) {
    a.nodes = split;
    a.node_cnt = reinterpret_cast<unsigned int*>(
        static_cast<char*>(split) +
        (static_cast<size_t>(p.items) * kSplitMax * p.acc_bytes + kWsAlign - 1) / kWsAlign *
            kWsAlign);
  }
  hipError_t e = launch_chunks<Op, FINAL>(p, op, a, stream);
  if (e != hipSuccess || !two_pass) return e;
  return launch_fold<Op, FINAL>(p.values, partials, out, out_f64, stream);
}

}  // namespace dpia
