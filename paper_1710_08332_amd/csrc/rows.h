// Contiguous lanes folded ROWS to a wavefront (dot, asum, binary32 gemv rows).
//
// contiguous_staged gives every thread of a wavefront a lane, so a wavefront
// loads 64 rows 128 bytes at a time and a launch has a wavefront per 64 lanes.
// With few lanes that is few wavefronts, each waiting for its rows' tiles one
// after the other (a dot of 2^20 under C=256 L=16: 64 wavefronts, 8 tiles
// each); and a chunk of more than 256 lanes would need more LDS than a compute
// unit has.  Here a wavefront takes ROWS = 16, 32 or 64 lane rows: all its
// threads load (a tile is 2,048 elements per operand in any case, 128, 64 or
// 32 of each row: 512, 256 or 128 bytes in one piece), its first ROWS threads
// fold.  The lane values go to LDS, where the chunk's combine reads them, so
// a work-group may take the lanes of a chunk in several turns.  Which elements
// a lane folds, in which order, and the combine's tree are the strategy's.
#pragma once

#include "device.h"
#include "plan.h"

namespace dpia {

constexpr int kTileElems = 2048;                       // per operand and tile
template <int ROWS>
constexpr int rows_tile() { return kTileElems / ROWS; }
// (LDS row stride: an odd number of 16-byte units)
template <int ROWS>
constexpr int rows_stage_floats(int nops) { return nops * ROWS * (rows_tile<ROWS>() + 4); }

// A work-group has 4 wavefronts; they take a chunk's groups of ROWS lanes in
// turn, or, where a chunk has fewer than 4 such groups, 2 or 4 chunks at once.
// (With fewer chunks than that gives every compute unit a work-group, fewer
// chunks and wavefronts: rows_teams.)
// LDS: the combine's scratch (and, after the chunks, a 1-pass fold's) in the
// first kRowsScratch bytes, the lane values, the staging regions.
constexpr int kRowsWaves = 4;
constexpr int kRowsScratch = 512;
static_assert(kFoldLds <= kRowsScratch, "the fold's LDS");

// Chunks a work-group takes at once: fewer than its wavefronts have room for
// where that leaves fewer than `wgs` work-groups.  That is one per compute
// unit, but a quarter of it in a 1-pass launch, whose work-groups' arrivals
// are taken one by one (256 chunks of L=16, dot C=128: 256 work-groups 9.7 us,
// 64 of four chunks 8.6; asum 9.0, 7.5).
inline int rows_teams(int64_t slices, int64_t items, int64_t wgs) {
  int teams = slices >= kRowsWaves ? 1 : kRowsWaves / static_cast<int>(slices);
  while (teams > 1 && (items + teams - 1) / teams < wgs) teams /= 2;
  return teams;
}

// Rows row0 .. row0 + ROWS - 1 of a chunk (Cel elements each, a multiple of
// 32; `limit` elements of the chunk exist): lane r < ROWS folds row row0 + r
// into acc, element e into component e % VEC.  `stage`: this wavefront's
// rows_stage_floats.  D tiles in flight.  CACHED1: operand 1 is read with
// cached loads (a gemv's x).
template <class Op, int VEC, int ROWS, int D, bool CACHED1 = false, class View>
__device__ __forceinline__ void rows_fold(const View& view, int row0, int Cel, int limit,
                                          float* stage, typename Op::T (&acc)[VEC]) {
  constexpr int NOPS = View::kOps;
  constexpr int TE = rows_tile<ROWS>();
  constexpr int PV = TE / 4;                           // 16-byte parts of a row tile
  constexpr int RPL = kWave / PV;                      // rows one load instruction covers
  constexpr int N = ROWS / RPL;                        // load instructions per operand
  static_assert(N == 8 && RPL >= 1, "2,048 elements are 8 loads of a wavefront");
  constexpr int SR = TE + 4;
#pragma unroll
  for (int j = 0; j < VEC; ++j) acc[j] = Op::Arith::zero();
  if (limit <= row0 * Cel) return;                     // none of the rows exists
  const int lane = static_cast<int>(threadIdx.x) & (kWave - 1);
  const int part = lane % PV, first = lane / PV;
  const int base = (row0 + first) * Cel + part * 4;    // (below W < 2^31)
  const int ntiles = (Cel + TE - 1) / TE;
  const bool whole = limit >= (row0 + ROWS) * Cel;     // every row exists
  f32x4 regs[D][NOPS][N];
  auto load = [&](int o, int at) {
    const f32x4* g = reinterpret_cast<const f32x4*>(view.operand(o) + at);
    return CACHED1 && o == 1 ? ld<false>(g) : ld<DPIA_NT_LOADS != 0>(g);
  };
  auto gload = [&](f32x4 (&rg)[NOPS][N], int tile) {
    const int e = tile * TE + part * 4;
    if (whole && (tile + 1) * TE <= Cel) {
#pragma unroll
      for (int o = 0; o < NOPS; ++o)
#pragma unroll
        for (int i = 0; i < N; ++i)
          rg[o][i] = load(o, base + tile * TE + i * RPL * Cel);
    } else {
      // whole 16-byte parts that exist, zeros past them (which fold as the
      // identity: a chunk that is not whole is a plain operation's)
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const bool in = e < Cel && base + tile * TE + i * RPL * Cel + 4 <= limit;
#pragma unroll
        for (int o = 0; o < NOPS; ++o) {
          rg[o][i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
          if (in) rg[o][i] = load(o, base + tile * TE + i * RPL * Cel);
        }
      }
    }
  };
  auto stage_fold = [&](const f32x4 (&rg)[NOPS][N], int tile, auto&& next) {
#pragma unroll
    for (int o = 0; o < NOPS; ++o)
#pragma unroll
      for (int i = 0; i < N; ++i)
        *reinterpret_cast<f32x4*>(stage + (o * ROWS + first + i * RPL) * SR + part * 4) = rg[o][i];
    wave_lds_order();
    next();
    if (ROWS == kWave || lane < ROWS) {
      const float* mine = stage + lane * SR;
      auto four = [&](int j) {
        f32x4 v[NOPS];
#pragma unroll
        for (int o = 0; o < NOPS; ++o)
          v[o] = *reinterpret_cast<const f32x4*>(mine + o * ROWS * SR + j * 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i % VEC] = Op::step(View::term(v, i), acc[i % VEC]);
      };
      // (elements past the row's end, in a last tile, are not folded)
      const int parts = Cel - tile * TE < TE ? (Cel - tile * TE) / 4 : PV;
      for (int j = 0; j < parts; j += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) four(j + u);
      }
    }
    wave_lds_order();
  };
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (d < ntiles) gload(regs[d], d);
  for (int t0 = 0; t0 < ntiles; t0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int tile = t0 + d;
      if (tile < ntiles)
        stage_fold(regs[d], tile, [&] { if (tile + D < ntiles) gload(regs[d], tile + D); });
    }
  }
  // the chunk's last limit % 4 elements, by the lane whose row ends there
  if (!whole && (limit & 3) != 0) {
    const int e0 = limit & ~3;
    if (lane < ROWS && e0 >= (row0 + lane) * Cel && e0 < (row0 + lane + 1) * Cel) {
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        if (e0 + i < limit) {
          typename Op::Term z[1];
          view.template load<1>(e0 + i, z);
          acc[i % VEC] = Op::step(z[0], acc[i % VEC]);
        }
      }
    }
  }
}

// The combine of L lane values in LDS by a group of `threads` threads (64, 128
// or 256 of the work-group; t: the thread's place in its group).  Every thread
// of the work-group calls this together; the value is in its group's thread 0.
template <class A, int COMBINE>
__device__ __forceinline__ typename A::T combine_stored(const typename A::T* lanes, int L, int t,
                                                        int threads, typename A::T* scratch) {
  using T = typename A::T;
  if constexpr (COMBINE == kSeq) {
    T r = A::zero();
    if (t == 0)
      for (int l = 0; l < L; ++l) r = A::add(lanes[l], r);
    return r;
  } else {
    const int team = L < threads ? L : threads;        // powers of two
    auto run = [&](auto nl) {
      constexpr int NL = decltype(nl)::value;
      T v[NL];
#pragma unroll
      for (int i = 0; i < NL; ++i) v[i] = t < team ? lanes[t * NL + i] : A::zero();
      return combine_lanes<A, NL, kTree>(v, t, team, L, scratch);
    };
    const int nl = L / team;
    if (nl == 1) return run(std::integral_constant<int, 1>{});
    if (nl == 2) return run(std::integral_constant<int, 2>{});
    return run(std::integral_constant<int, 4>{});
  }
}

}  // namespace dpia
