// The outer reduceSeq of a strategy: the fold of G chunk values from 0 in
// chunk order, shared by the reduction kernels and the batched engine.
//
// The fold is a chain: every addition rounds, and takes the rounded value of
// the one before it.  Added one by one it runs at the rate one wavefront
// issues instructions, 3.8 ns a value with its LDS reads (32,768 values: 125
// us, more than the 2^29 bytes those values were computed from take to read).
// It is run in parallel here, with the same bits, as follows.
//
// Lane l of a wavefront holds E consecutive values and the chain reaches it
// with some start s_l.  Two binary32 numbers of one sign and exponent differ
// by a whole number of units in the last place, and adding a value v to
// either rounds at the same places, except that ties go to the even result:
// as long as the running value keeps its sign and exponent, what a lane's
// values add to the *bit pattern* of its start depends on the start's last
// bit alone.  So:
//  1. an ordinary prefix sum gives every lane an approximate start;
//  2. every lane folds its values, with the chain's own additions, from that
//     start with its last bit cleared and set: two displacements (d0, d1) of
//     the bit pattern;
//  3. displacements compose (the first decides the last bit that the second
//     sees), so a scan over the lanes gives every lane's start from the
//     wavefront's;
//  4. lanes whose running value leaves its binade (seen in step 2) have no
//     such displacement: the scan restarts behind them, and the chain is
//     walked from one to the next, folding their values from the now known
//     start;
//  5. every lane folds its values from the start it was given, and the result
//     has to be, bit for bit, the start its successor was given.  By
//     induction from the first lane all starts are then the chain's own.  A
//     lane that fails is treated as in 4 and the walk is done again.
// Steps 1 to 4 only guess; step 5 is the chain itself, so the result does not
// rest on any property of the values (infinities and NaN included).
// Wavefronts do 4 in turn and the rest at once.  Where most lanes change
// binade, and where there are few values, the lanes are folded one after
// another (E additions and one lane read each: 3.4 ns a value).
//
// Measured, a launch of the fold alone (12 us of it are the launch and its
// events), one by one before and now: 4,096 values 17.8 -> 12.2 us where all
// are positive, 13.9 us where they are normal (both signs: the sum crosses
// powers of two again and again near zero); 32,768 values 127 -> 13.3 and 124
// -> 51 us; 32,768 values alternating about +1 and -1, where every lane leaves
// its binade, 126 -> 117 us; 8,192 Kahan pairs 150 -> 29-49 us folded in
// binary32, 89 -> 13-32 us in binary64.
#pragma once

#include <type_traits>

#include "device.h"
#include "plan.h"

namespace dpia {

// Kahan pairs have value s - c, Sum2 pairs s + c; "64": the chunk values are
// folded in binary64.
enum : int {
  kFinalPlain = 0,
  kFinalKahan32 = 1,
  kFinalKahan64 = 2,
  kFinalSum2_32 = 3,
  kFinalSum2_64 = 4
};

template <class F>
struct FoldBits;
template <>
struct FoldBits<float> {
  using U = uint32_t;
  static constexpr int kMantissa = 23;
};
template <>
struct FoldBits<double> {
  using U = uint64_t;
  static constexpr int kMantissa = 52;
};

template <class F>
__device__ __forceinline__ typename FoldBits<F>::U to_bits(F v) {
  typename FoldBits<F>::U u;
  __builtin_memcpy(&u, &v, sizeof(F));
  return u;
}
template <class F>
__device__ __forceinline__ F from_bits(typename FoldBits<F>::U u) {
  F v;
  __builtin_memcpy(&v, &u, sizeof(F));
  return v;
}

// DPP controls: lane i reads lane i - N of its row of 16; the last lane of
// the row (of the half) before; lane i + 1 of the wavefront.
constexpr int kRowShr = 0x110, kRowBcast15 = 0x142, kRowBcast31 = 0x143;
constexpr int kWaveShl1 = 0x130, kWaveShr1 = 0x138;

// The value of the DPP source lane, or `old` where there is none.
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ uint32_t dpp(uint32_t old, uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(
      static_cast<int>(old), static_cast<int>(v), CTRL, ROWS, 0xF, false));
}
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ uint64_t dpp(uint64_t old, uint64_t v) {
  const uint32_t lo = dpp<CTRL, ROWS>(static_cast<uint32_t>(old), static_cast<uint32_t>(v));
  const uint32_t hi =
      dpp<CTRL, ROWS>(static_cast<uint32_t>(old >> 32), static_cast<uint32_t>(v >> 32));
  return static_cast<uint64_t>(hi) << 32 | lo;
}

// Lane `l`'s value (`l` uniform).
__device__ __forceinline__ uint32_t lane_read(uint32_t v, int l) {
  return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), l));
}
__device__ __forceinline__ uint64_t lane_read(uint64_t v, int l) {
  const uint64_t hi = lane_read(static_cast<uint32_t>(v >> 32), l);
  return hi << 32 | lane_read(static_cast<uint32_t>(v), l);
}
__device__ __forceinline__ float lane_read(float v, int l) {
  return from_bits<float>(lane_read(to_bits(v), l));
}
__device__ __forceinline__ double lane_read(double v, int l) {
  return from_bits<double>(lane_read(to_bits(v), l));
}

// The chain's additions over one lane's values (element first, as in reduce).
template <class F, int E>
__device__ __forceinline__ F fold_lane(const F (&v)[E], F a) {
#pragma unroll
  for (int j = 0; j < E; ++j) a = v[j] + a;
  return a;
}

// Inclusive prefix sums over the wavefront (approximate starts only).
template <class F>
__device__ __forceinline__ F wave_prefix(F x) {
  using U = typename FoldBits<F>::U;
  auto at = [&](auto u) { return from_bits<F>(u); };
  x += at(dpp<kRowShr + 1>(U(0), to_bits(x)));
  x += at(dpp<kRowShr + 2>(U(0), to_bits(x)));
  x += at(dpp<kRowShr + 4>(U(0), to_bits(x)));
  x += at(dpp<kRowShr + 8>(U(0), to_bits(x)));
  x += at(dpp<kRowBcast15, 0xA>(U(0), to_bits(x)));
  x += at(dpp<kRowBcast31, 0xC>(U(0), to_bits(x)));
  return x;
}

// Displacements of a bit pattern whose last bit is 0 (d0) or 1 (d1).
template <class U>
struct Displace {
  U d0, d1;
  // (by masks: written as a choice, the compiler indexes a copy in scratch)
  __device__ U of(U b) const { return d0 ^ ((d0 ^ d1) & (U(0) - (b & 1))); }
};

// `l`, then `r`.
template <class U>
__device__ __forceinline__ Displace<U> then(const Displace<U>& l, const Displace<U>& r) {
  return Displace<U>{l.d0 + ((l.d0 & 1) ? r.d1 : r.d0), l.d1 + ((l.d1 & 1) ? r.d0 : r.d1)};
}

// Inclusive scan over the wavefront, restarting at lane `head` (per lane: the
// last restart at or before it).
template <class U>
__device__ __forceinline__ Displace<U> displace_scan(Displace<U> d, int lane, int head) {
  auto step = [&](U s0, U s1, bool have) {
    const Displace<U> t = then(Displace<U>{s0, s1}, d);
    d.d0 = have ? t.d0 : d.d0;
    d.d1 = have ? t.d1 : d.d1;
  };
  const int row = lane & 15;
#define DPIA_SCAN_STEP(N)                                                                    \
  step(dpp<kRowShr + N>(U(0), d.d0), dpp<kRowShr + N>(U(0), d.d1), row >= N && lane - N >= head)
  DPIA_SCAN_STEP(1);
  DPIA_SCAN_STEP(2);
  DPIA_SCAN_STEP(4);
  DPIA_SCAN_STEP(8);
#undef DPIA_SCAN_STEP
  step(dpp<kRowBcast15, 0xA>(U(0), d.d0), dpp<kRowBcast15, 0xA>(U(0), d.d1),
       (lane & 16) != 0 && (lane & ~15) - 1 >= head);
  step(dpp<kRowBcast31, 0xC>(U(0), d.d0), dpp<kRowBcast31, 0xC>(U(0), d.d1),
       lane >= 32 && head <= 31);
  return d;
}

// Lane by lane: the chain over the first `lanes` lanes' values from `cur`;
// `start` receives the calling lane's start.
template <bool START, class F, int E>
__device__ __forceinline__ F walk_lanes(const F (&v)[E], F cur, int lanes, int lane, F& start) {
  for (int l = 0; l < lanes; ++l) {
    if constexpr (START) start = lane == l ? cur : start;
    cur = lane_read(fold_lane(v, cur), l);
  }
  return cur;
}

// A wavefront with more changes of binade than this, or whose starts fail
// step 5 more often than this, is folded lane by lane: a stop costs about 30
// instructions, a lane of walk_lanes 20.
constexpr int kFoldStops = 44;
constexpr int kFoldTries = 2;

// Values of type T that a lane of the fold holds.
template <class T>
constexpr int kFoldLaneValues = sizeof(T) > 4 ? 8 : 16;

// Slots of LDS a block's chain uses: per wavefront the sum of its values and
// the value its chain reaches, and one flag.
constexpr int kFoldWaves = 16;
constexpr int kFoldSlots = 2 * kFoldWaves + 1;

// The thread's index, as nothing that is known before the fold: what the fold
// derives from it would be held in registers all through a kernel that folds
// inside a loop (the one-launch batch: 135 registers, 3 wavefronts per SIMD,
// not 94 and 5).
__device__ __forceinline__ int fold_thread() {
  int t = static_cast<int>(threadIdx.x);
  asm volatile("" : "+v"(t));
  return t;
}

// The chain from `acc` over a block's values: lane l of wavefront w holds
// values (w * 64 + l) * E ..., zeros past the `lanes` lanes (of the first
// `waves` wavefronts) that hold any.  Every thread of the work-group calls
// this; acc ends as the chain's value in all of them, and `start` as the
// calling lane's start.  `walk`: a single wavefront folds its lanes in turn.
template <bool START, class F, int E>
__device__ __forceinline__ void block_chain(const F (&v)[E], F& acc, int lanes, int waves,
                                            F* slots, F& start, bool walk) {
  using U = typename FoldBits<F>::U;
  constexpr int kMant = FoldBits<F>::kMantissa;
  const int tid = fold_thread();
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int lane = tid & (kWave - 1);
  const bool mine = wave < waves;
  F* ends = slots + kFoldWaves;
  int* failed = reinterpret_cast<int*>(slots + 2 * kFoldWaves);
  wait_memory();   // the values are here: no wait is left in the loops below
  // 1. approximate starts
  F incl = F(0), own = F(0);
  bool in_turn = false;                          // lane by lane
  if (mine) {
    in_turn = walk && waves == 1;
    if (!in_turn) {
      own = fold_lane(v, F(0));
      incl = wave_prefix(own);
      if (lane == kWave - 1) slots[wave] = incl;
    }
  }
  if (tid == 0) *failed = 0;
  __syncthreads();
  // 2. displacements, and the lanes without (bad); 3. their scan
  Displace<U> d{0, 0}, inc{0, 0}, exc{0, 0};
  unsigned long long bad = 0;
  int head = 0;
  auto scan = [&] {
    // the last restart at or before this lane: a lane behind a stop
    const unsigned long long heads = (bad << 1 | 1ull) & (~0ull >> (63 - lane));
    head = 63 - __clzll(static_cast<long long>(heads));
    inc = displace_scan(d, lane, head);
    exc = Displace<U>{dpp<kWaveShr1>(U(0), inc.d0), dpp<kWaveShr1>(U(0), inc.d1)};
    if (lane == head) exc = Displace<U>{0, 0};
  };
  if (mine && !in_turn) {
    F p = acc;
    for (int w = 0; w < wave; ++w) p += slots[w];
    p += incl - own;
    const U b0 = to_bits(p) & ~U(1);
    F a0 = from_bits<F>(b0), a1 = from_bits<F>(b0 | 1), lo = a0, hi = a0;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      a0 = v[j] + a0;
      a1 = v[j] + a1;
      lo = fmin(lo, a0);
      hi = fmax(hi, a0);
    }
    d = Displace<U>{to_bits(a0) - b0, to_bits(a1) - (b0 | 1)};
    bad = __ballot((to_bits(lo) >> kMant) != (to_bits(hi) >> kMant));
    in_turn = __popcll(bad) > kFoldStops;
    if (!in_turn) scan();
  }
  for (int tries = 0;; ++tries) {
    // 4. the wavefronts in turn: from stop to stop
    U base = 0, end = 0;                         // base: the start of the lane's restart
    for (int w = 0; w < waves; ++w) {
      if (w == wave) {
        const F from = lane_read(w == 0 ? acc : ends[w - 1], 0);
        if (in_turn) {
          const int here = lanes - w * kWave < kWave ? lanes - w * kWave : kWave;
          end = to_bits(walk_lanes<START>(v, from, here, lane, start));
        } else {
          U cur = to_bits(from);
          base = cur;
          int h = 0;
          for (unsigned long long m = bad; m != 0; m &= m - 1) {
            const int b = __builtin_ctzll(m);
            const U s = cur + Displace<U>{lane_read(exc.d0, b), lane_read(exc.d1, b)}.of(cur);
            cur = lane_read(to_bits(fold_lane(v, from_bits<F>(s))), b);
            h = b + 1;
            base = lane >= h ? cur : base;
          }
          end = cur;
          if (h < kWave)
            end += Displace<U>{lane_read(inc.d0, 63), lane_read(inc.d1, 63)}.of(cur);
        }
        if (lane == 0) ends[w] = from_bits<F>(end);
      }
      __syncthreads();
      if (w == 0 && tid == 0) *failed = 0;
    }
    // 5. every lane's chain ends where its successor's starts
    if (mine && !in_turn) {
      const U st = base + exc.of(base);
      const U got = to_bits(fold_lane(v, from_bits<F>(st)));
      const U next = dpp<kWaveShl1>(end, st);
      const unsigned long long wrong = __ballot(got != next);
      if constexpr (START) start = from_bits<F>(st);
      if (wrong != 0) {
        bad |= wrong & (~wrong + 1);
        in_turn = tries >= kFoldTries || __popcll(bad) > kFoldStops;
        if (!in_turn) scan();
        if (lane == 0) *failed = 1;
      }
    }
    __syncthreads();
    if (*failed == 0) break;
  }
  acc = ends[waves - 1];
  __syncthreads();   // the slots are free again
}

static_assert(kFoldSlots * sizeof(double) <= kFoldLds, "the plan reserves the fold's LDS");

// The outer reduceSeq over the G chunk values, from the literal 0, in chunk
// order, and the strategy's result.  Every thread of the work-group calls
// this (at least one whole wavefront; at most 16 take part).  `lds`:
// kFoldLds bytes, 8-byte aligned.
// COHERENT: the chunk values were written by other work-groups of the same
// launch with store_coherent, which put them in memory.  Few are read with
// load_coherent; where more are, one agent-scope acquire in every wavefront
// that reads makes this compute unit's plain (wide) loads see them.  An acquire
// invalidates the compute unit's cache, which the other work-groups there go on
// using: with one for each of the 3,000 small folds of a one-launch batch it
// took 36 us, not 24.
// `signs`: the values may be of both signs.  Where one wavefront holds them all,
// their sum leaves its binade in most lanes then, and they are folded lane by
// lane (a dot's 513 to 900 values after the chunks' launch: scanned 8.4 to 9.8
// us a call, in turn 7.1 to 8.9, one by one 7.0 to 9.0); an asum's grows through
// a few binades (1,024 values: scanned 6.0, one by one 7.8).
template <class A, int FINAL, bool COHERENT = false>
__device__ __forceinline__ void final_fold(const typename A::T* partials, int64_t G, void* out,
                           int out_f64, void* lds, bool signs) {
  using T = typename A::T;
  constexpr int E = kFoldLaneValues<T>;
  // Up to this many lanes are folded lane by lane, from `signs` up to all (not
  // the pairs' binary32 chain, whose steps are ten instructions).
  constexpr int kFewLanes = 32;
  constexpr bool kPairs = FINAL == kFinalKahan32 || FINAL == kFinalSum2_32;
  const int tid = fold_thread();
  int whole = static_cast<int>(blockDim.x) / kWave;   // wavefronts without missing threads
  whole = whole < kFoldWaves ? whole : kFoldWaves;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const bool few = !std::is_integral_v<T> && G <= kFewLanes * E;
  const bool turns = G <= (signs && !kPairs ? kWave : kFewLanes) * E;
  const bool reads = std::is_integral_v<T> ? wave * kWave < G : !few && (wave == 0 || !turns);
  if constexpr (COHERENT) {
    if (reads) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  }
  if constexpr (std::is_integral_v<T>) {
    // addition modulo 2^32 is associative: any order gives the same bits
    T* sums = static_cast<T*>(lds);
    if (wave < whole) {
      T a = T(0);
      for (int64_t i = tid; i < G; i += whole * kWave) a += partials[i];
#pragma unroll
      for (int o = kWave / 2; o > 0; o >>= 1) a += __shfl_xor(a, o, kWave);
      if (lane == 0) sums[wave] = a;
    }
    __syncthreads();
    if (tid == 0) {
      T r = T(0);
      for (int w = 0; w < whole; ++w) r += sums[w];
      *static_cast<T*>(out) = r;
    }
    __syncthreads();
    return;
  } else {
    constexpr bool k64 = FINAL == kFinalKahan64 || FINAL == kFinalSum2_64;
    T acc = A::zero();
    double acc64 = 0.0;
    T v[E] = {};
    // this lane's values of the block at b (zeros past the end); one by one,
    // coherently, where ONE
    auto load = [&](int64_t b, auto one) {
      constexpr bool ONE = decltype(one)::value;
      const int64_t at = b + (static_cast<int64_t>(wave) * kWave + lane) * E;
      if constexpr (ONE) {
        // (past the end the last value is read again: no branch, and no wait,
        // between the loads)
#pragma unroll
        for (int j = 0; j < E; ++j) v[j] = load_coherent(partials + (at + j < G ? at + j : G - 1));
#pragma unroll
        for (int j = 0; j < E; ++j) v[j] = at + j < G ? v[j] : A::zero();
        return E;
      }
      if (at + E <= G) {
        __builtin_memcpy(v, partials + at, sizeof(v));
        return E;
      }
      int n = 0;
#pragma unroll
      for (int j = 0; j < E; ++j) {
        v[j] = A::zero();
        if (at + j < G) {
          v[j] = partials[at + j];
          ++n;
        }
      }
      return n;
    };
    auto value64 = [&](const T& e) {
      if constexpr (FINAL == kFinalKahan64)
        return static_cast<double>(e.s) - static_cast<double>(e.c);
      else if constexpr (FINAL == kFinalSum2_64)
        return static_cast<double>(e.s) + static_cast<double>(e.c);
      else
        return 0.0;
    };
    if (turns) {
      if (wave == 0) {
        if (COHERENT && few)
          load(0, std::bool_constant<COHERENT>{});
        else
          load(0, std::false_type{});
        const int lanes = static_cast<int>((G + E - 1) / E);
        if constexpr (k64) {
          double w[E];
#pragma unroll
          for (int j = 0; j < E; ++j) w[j] = value64(v[j]);
          double start;
          acc64 = walk_lanes<false>(w, acc64, lanes, lane, start);
        } else if constexpr (sizeof(T) == 4) {
          float start;
          acc = walk_lanes<false>(v, acc, lanes, lane, start);
        } else {
          for (int l = 0; l < lanes; ++l) {
            // (a zero pair changes no pair that is finite, and one that is not
            // has value NaN already)
            T a = acc;
#pragma unroll
            for (int j = 0; j < E; ++j) a = A::add(v[j], a);
            acc = T{lane_read(a.s, l), lane_read(a.c, l)};
          }
        }
      }
    } else {
      const int64_t block = static_cast<int64_t>(whole) * kWave * E;
      for (int64_t b = 0; b < G; b += block) {
        const int64_t left = G - b < block ? G - b : block;
        const int lanes = static_cast<int>((left + E - 1) / E);
        const int waves = (lanes + kWave - 1) / kWave;
        int n = 0;
        if (wave < waves) n = load(b, std::false_type{});
        if constexpr (k64) {
          double w[E], start;
#pragma unroll
          for (int j = 0; j < E; ++j) w[j] = value64(v[j]);
          block_chain<false>(w, acc64, lanes, waves, static_cast<double*>(lds), start, false);
        } else if constexpr (sizeof(T) == 4) {
          float start;
          block_chain<false>(v, acc, lanes, waves, static_cast<float*>(lds), start, false);
        } else {
          // pairs: the s parts are a chain of their own; from its running
          // values come the exact errors, and the c parts are a chain over
          // r.c and the error, in turn (c - e = c + (-e))
          float s[E], w[2 * E], start = 0.0f, cstart;
#pragma unroll
          for (int j = 0; j < E; ++j) s[j] = v[j].s;
          block_chain<true>(s, acc.s, lanes, waves, static_cast<float*>(lds), start, false);
          T l{start, 0.0f};
#pragma unroll
          for (int j = 0; j < E; ++j) {
            // (l.c = 0, r.c = 0: add's new c is -e, or e for Sum2)
            const T t = A::add(T{s[j], 0.0f}, T{l.s, 0.0f});
            w[2 * j] = v[j].c;
            w[2 * j + 1] = j < n ? t.c : 0.0f;
            l = t;
          }
          // (the errors are of both signs)
          block_chain<false>(w, acc.c, lanes, waves, static_cast<float*>(lds), cstart, G <= block);
        }
      }
    }
    if (tid == 0) {
      if constexpr (k64) {
        if (out_f64)
          *static_cast<double*>(out) = acc64;
        else
          *static_cast<float*>(out) = static_cast<float>(acc64);
      } else if constexpr (FINAL == kFinalKahan32) {
        *static_cast<float*>(out) = acc.s - acc.c;
      } else if constexpr (FINAL == kFinalSum2_32) {
        *static_cast<float*>(out) = acc.s + acc.c;
      } else {
        *static_cast<T*>(out) = acc;
      }
    }
    __syncthreads();   // the LDS is free again
  }
}

}  // namespace dpia
