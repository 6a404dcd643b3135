// Exact selection of nearest points on one wave: 64-bit keys (fp32 squared distance bits, index) compared
// as integers, a bitonic sort network on DPP lane patterns and the gfx950 row / half swaps, and a running
// top-64.  Distances are evaluated without fused multiply-add: every translation unit that includes this
// header is compiled with -ffp-contract=off.
#pragma once

#include "device_util.h"

namespace affmae {

typedef unsigned long long key_t;
constexpr key_t kKeyMax = ~0ull;

// fp32 squared distance, each operation rounded separately.
__device__ __forceinline__ float dist2(float ax, float ay, float bx, float by) {
#pragma clang fp contract(off)
  float dx = ax - bx;
  float dy = ay - by;
  float xx = dx * dx;
  float yy = dy * dy;
  return xx + yy;
}

__device__ __forceinline__ key_t make_key(float d2, int idx) {
  return ((key_t)__float_as_uint(d2) << 32) | (key_t)(uint32_t)idx;
}

__device__ __forceinline__ key_t shfl_key(key_t k, int src) {
  uint32_t lo = (uint32_t)k, hi = (uint32_t)(k >> 32);
  lo = __shfl(lo, src);
  hi = __shfl(hi, src);
  return ((key_t)hi << 32) | lo;
}

// The key held by lane (lane ^ J), J a power of two.
template <int J>
__device__ __forceinline__ key_t lane_xor_key(key_t k, int lane) {
  const uint32_t lo = lane_xor_u32<J>((uint32_t)k, lane);
  const uint32_t hi = lane_xor_u32<J>((uint32_t)(k >> 32), lane);
  return ((key_t)hi << 32) | lo;
}

// One compare-exchange step of a bitonic network: partner lane ^ J; the lane keeps
// the smaller key when keep_min.
template <int J>
__device__ __forceinline__ key_t exchange(key_t key, int lane, bool keep_min) {
  const key_t other = lane_xor_key<J>(key, lane);
  return ((key < other) == keep_min) ? key : other;
}
template <int K2, int J>
__device__ __forceinline__ key_t sort_stage(key_t key, int lane) {
  // blocks of K2 lanes alternate ascending / descending; within a block the lower lane of a pair keeps the minimum
  key = exchange<J>(key, lane, ((lane & K2) == 0) == ((lane & J) == 0));
  if constexpr (J > 1) key = sort_stage<K2, J / 2>(key, lane);
  return key;
}

// Sort one key per lane ascending across the 64 lanes of the wave.
__device__ __forceinline__ key_t wave_sort(key_t key, int lane) {
  key = sort_stage<2, 1>(key, lane);
  key = sort_stage<4, 2>(key, lane);
  key = sort_stage<8, 4>(key, lane);
  key = sort_stage<16, 8>(key, lane);
  key = sort_stage<32, 16>(key, lane);
  key = sort_stage<64, 32>(key, lane);  // lane & 64 == 0 everywhere: ascending
  return key;
}

// Input: bitonic across lanes.  Output: ascending across lanes.
__device__ __forceinline__ key_t wave_bitonic_merge(key_t key, int lane) {
  return sort_stage<64, 32>(key, lane);
}

// Keeps the 64 smallest keys seen so far, ascending across lanes.  `row` holds 64
// new keys in any order; `kth` is the lane whose key bounds what can still enter
// the first `kth+1` places.
__device__ __forceinline__ key_t topk_push(key_t best, key_t row, int lane, int kth) {
  key_t bound = shfl_key(best, kth);
  if (__ballot(row < bound) == 0ull) return best;  // wave-uniform: nothing can enter
  row = wave_sort(row, lane);
  key_t rev = shfl_key(row, kWave - 1 - lane);
  best = best < rev ? best : rev;  // the 64 smallest of both, bitonic
  return wave_bitonic_merge(best, lane);
}

// The value of the next lane (lane 63: its own): a whole-wave shift on the vector ALU.
__device__ __forceinline__ uint32_t next_lane_u32(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x130, 0xf, 0xf, false);  // wave_shl:1
}

// Sort of 64 distinct 32-bit keys, one per lane, ascending: a bitonic network whose compare-exchange is one lane move
// and one three-operand median.  With a third operand of 0 the median is the minimum, with all ones the maximum, so
// the lane's role in a step of distance J (keep the smaller or the larger key) is that operand: bit J of the lane
// number, spread over a word.  Blocks that the network sorts descending hold complemented keys meanwhile, so the
// roles are the same in every stage and six words serve all 21 steps.
__device__ __forceinline__ uint32_t umed3(uint32_t a, uint32_t b, uint32_t c) {
  const uint32_t lo = a < b ? a : b, hi = a < b ? b : a;
  const uint32_t m = hi < c ? hi : c;
  return lo > m ? lo : m;
}
template <int BIT>
__device__ __forceinline__ uint32_t lane_bit_word(int lane) {
  return (uint32_t)((lane << (31 - BIT)) >> 31);
}
template <int J>
__device__ __forceinline__ uint32_t sort_steps_u32(uint32_t key, int lane) {
  typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
  constexpr int BIT = J == 1 ? 0 : J == 2 ? 1 : J == 4 ? 2 : J == 8 ? 3 : J == 16 ? 4 : 5;
  const uint32_t role = lane_bit_word<BIT>(lane);
  if constexpr (J == 16) {
    const u32x2 t = __builtin_amdgcn_permlane16_swap(key, key, false, false);  // in every lane: its own key and its partner's
    key = umed3(t[0], t[1], role);
  } else if constexpr (J == 32) {
    const u32x2 t = __builtin_amdgcn_permlane32_swap(key, key, false, false);
    key = umed3(t[0], t[1], role);
  } else {
    key = umed3(key, lane_xor_u32<J>(key, lane), role);
  }
  if constexpr (J > 1) key = sort_steps_u32<J / 2>(key, lane);
  return key;
}
__device__ __forceinline__ uint32_t wave_sort_u32(uint32_t key, int lane) {
  const uint32_t f1 = lane_bit_word<1>(lane), f2 = lane_bit_word<2>(lane), f3 = lane_bit_word<3>(lane);
  const uint32_t f4 = lane_bit_word<4>(lane), f5 = lane_bit_word<5>(lane);
  key = sort_steps_u32<1>(key ^ f1, lane);
  key = sort_steps_u32<2>(key ^ (f1 ^ f2), lane);
  key = sort_steps_u32<4>(key ^ (f2 ^ f3), lane);
  key = sort_steps_u32<8>(key ^ (f3 ^ f4), lane);
  key = sort_steps_u32<16>(key ^ (f4 ^ f5), lane);
  return sort_steps_u32<32>(key ^ f5, lane);
}

// Sorts the `fill` (<= 64) keys of `pend` (LDS, owned by the wave), whose distances are at most t, ascending across
// the lanes; returns the lower half (index) of the lane's key, undefined from lane `fill` on (so callers queue at least
// as many as they use).  The 64-bit network costs ~170 vector instructions, once most of the search's time, so the order
// is found on 32-bit words (26 leading bits of distance / t, place in `pend`), ~65 instructions.  Where neighbouring
// words share their leading bits (equal or nearly equal distances) the keys themselves are fetched in that order and
// every neighbouring pair is compared in full: candidates of contiguous clusters are queued in index order, so equal
// distances pass; what does not (rare) goes through the 64-bit network.  The result is exact either way.
__device__ __forceinline__ uint32_t sort_queued(const key_t* pend, int fill, uint32_t t, int lane) {
  // (a scale that overflows, from a subnormal t, only makes the words useless as an order: the check below decides;
  // whatever the conversion makes of it, every word keeps its lane number, so the places stay a permutation)
  const float scale = 67108000.f * __builtin_amdgcn_rcpf(__uint_as_float(t));
  const uint32_t lead = (uint32_t)(__uint_as_float((uint32_t)(pend[lane] >> 32)) * scale);
  const uint32_t word = lane < fill ? (lead << 6) | (uint32_t)lane : 0xffffffc0u | (uint32_t)lane;
  const uint32_t sorted = wave_sort_u32(word, lane);
  const uint32_t from = sorted & 63u;
  const bool tie = (sorted ^ next_lane_u32(sorted)) < 64u;  // (lane 63 next to itself, and the pads next to each other)
  const unsigned long long below = fill < kWave ? (1ull << fill) - 1ull : ~0ull >> 1;
  if ((__ballot(tie) & below) != 0ull) {  // wave-uniform
    const key_t key = lane < fill ? pend[from] : kKeyMax;
    const uint32_t lo = (uint32_t)key, hi = (uint32_t)(key >> 32);
    const key_t next = ((key_t)next_lane_u32(hi) << 32) | next_lane_u32(lo);
    if (__ballot(key > next) != 0ull) {
      // (the lane number made opaque: nothing of the rare path is worth a register throughout the caller's loop)
      asm volatile("" : "+v"(lane));
      return (uint32_t)wave_sort(lane < fill ? pend[lane] : kKeyMax, lane);
    }
  }
  return (uint32_t)pend[from];
}

// Appends the candidates of one row at most t away to `pend` (64 keys; ROOM: they are known to fit, else those past
// its end are dropped); returns the number queued so far.  All lanes active.
template <bool ROOM = true>
__device__ __forceinline__ int queue_row(key_t* pend, int fill, uint32_t d2, uint32_t id, uint32_t t) {
  const bool in = d2 <= t;
  const unsigned long long mask = __builtin_amdgcn_ballot_w64(in);
  const int place =
      __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, (uint32_t)fill));
  if (in && (ROOM || place < kWave)) pend[place] = ((key_t)d2 << 32) | id;
  fill += __popcll(mask);
  return ROOM ? fill : min(fill, kWave);
}
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t x, int lane) {
  x = min(x, lane_xor_u32<1>(x, lane));
  x = min(x, lane_xor_u32<2>(x, lane));
  x = min(x, lane_xor_u32<4>(x, lane));
  x = min(x, lane_xor_u32<8>(x, lane));
  x = min(x, lane_xor_u32<16>(x, lane));
  x = min(x, lane_xor_u32<32>(x, lane));
  return __builtin_amdgcn_readfirstlane(x);
}

__device__ __forceinline__ bool finite_point(float x, float y) {
  return __builtin_isfinite(x) && __builtin_isfinite(y);
}

__device__ __forceinline__ key_t wave_min_key(key_t x, int lane) {
  const uint32_t hi = wave_min_u32((uint32_t)(x >> 32), lane);
  const uint32_t lo = wave_min_u32((uint32_t)(x >> 32) == hi ? (uint32_t)x : 0xffffffffu, lane);
  return ((key_t)hi << 32) | lo;
}
// The K nearest by their keys alone, each the smallest above the last one (keys are distinct), for points whose distances
// may be NaN: these sort by their bits, after every distance.  A path of its own, decided once per workgroup or wave from
// the coordinates (0.3 % of the search's time): inside select_nearest it cost the search of finite points 1 %, and as a
// running top 64 two registers too many for eight waves per SIMD, 5 - 10 %.
template <class KeyAt>
__device__ __forceinline__ uint32_t nearest_by_key(int rows, int K, int lane, KeyAt key_at) {
  uint32_t id = 0u;
  key_t last = 0ull;
#pragma unroll 1
  for (int i = 0; i < K; ++i) {
    key_t least = kKeyMax;
#pragma unroll 1
    for (int row = 0; row < rows; ++row) {
      const key_t key = key_at(row, lane);
      if ((i == 0 || key > last) && key < least) least = key;
    }
    last = wave_min_key(least, lane);
    if (lane == i) id = (uint32_t)last;
  }
  return id;
}

// The K nearest of the candidates that the caller holds in `rows` rows, one per lane and row: each(f) calls f(d2, low)
// for every row, d2 being the bit pattern of the lane's squared distance (ordered like the value, since d2 >= +0; above
// every distance's bits where the lane has no candidate) and low the lower half of its key, ordered like the index.
// key_at(row, lane) is any candidate's key (kKeyMax where the lane has none).  `pend`: 64 keys of LDS owned by the
// wave, 128 unless WIDE is kOneRow.  ORDERED: low ascends with row and lane.  Returns the lower halves of the keys in
// ascending order of the keys across the lanes (the first K are the answer).
//
// The wave looks for a distance threshold T with K <= #{d2 <= T} <= 64 by counting with ballots.  It starts from
// `guess` (the threshold that worked for the previous, nearby query, or an estimate; not 0) and scales it by wanted /
// found (the count grows like the area, i.e. like d2), then alternates bisection on the bit pattern with steps to the
// next larger distance (which end the search where many candidates share one).  Everything at or below T is nearer than
// everything above it, so the K nearest are among the counted candidates, which are sorted once.
// LINEAR, for queries that may lie away from all candidates (the count then grows late and steeply) and for counts that
// cost more than a few multiplications: once one threshold had too many, it interpolates between the closest ones with
// too few and too many, in place of scaling and, up to the 18th step, of bisecting (grid points up to half the frame
// away from 1024 tokens, 9 of them wanted: 3.7 steps a query without, 1.5 with it; with candidates in registers and
// queries among them it is the slower one, 77 us without and 98 with it for 8 images of 16384 tokens in 12 blobs).
// WIDE: where a count costs much, or the window would be next to nothing, it may be up to 128, and the K nearest of
// these are found in the same way (kTwoSearched) or by sorting both rows (kTwoSorted: 64-bit keys, ~400 instructions and
// registers for their lane masks).
// No such T exists when more candidates share a distance than the window takes: then the nearer ones and, in index order,
// as many of the equal ones as fit are sorted (candidates that are not ORDERED are merged row by row into a running top
// 64).  Either way the result is exact.  ORDERED: at least K candidates have a distance that is no NaN (the queue has
// nothing else); where a coordinate is not finite the caller takes nearest_by_key.
enum { kOneRow, kTwoSearched, kTwoSorted };
template <bool ORDERED, int WIDE, bool LINEAR, class Each, class KeyAt>
__device__ __forceinline__ uint32_t select_nearest(int rows, int K, uint32_t& guess, key_t* pend, int lane, Each each,
                                                   KeyAt key_at) {
  constexpr int most = WIDE != kOneRow ? 2 * kWave : kWave;
  // invariant: count(lo) = at_lo < K (lo = -1: nothing known), count(hi) = at_hi > most (at_hi = -1: hi = +inf, not counted)
  int lo = -1, hi = 0x7f800000, at_lo = 0, at_hi = -1;
  uint32_t t = __builtin_amdgcn_readfirstlane(guess);  // (a scalar, and known to be one)
#pragma unroll 1
  for (int it = 0; it < 96; ++it) {  // (from the 19th on every other step bisects: 31 of these end it)
    int n = 0;
    each([&](uint32_t d2, uint32_t) { n += __popcll(__ballot(d2 <= t)); });
    if (n >= K && n <= most) {
      guess = t;
      int fill = 0;
      // (compared again, as if with another threshold: the masks of the count, brought here as conditions, took two
      // instructions a row to become masks again; 8 images of 16384 tokens in 12 blobs 206.2 us with their plan, now 203.7)
      uint32_t same = t;
      asm volatile("" : "+s"(same));
      each([&](uint32_t d2, uint32_t low) { fill = queue_row(pend, fill, d2, low, same); });
      wave_lds_sync();
      if constexpr (WIDE != kOneRow) {
        if (n > kWave) {  // wave-uniform
          const key_t a = pend[lane], b = lane < n - kWave ? pend[kWave + lane] : kKeyMax;
          wave_lds_sync();
          if constexpr (WIDE == kTwoSorted) {
            asm volatile("" : "+v"(lane));  // its masks are made here, not held (spilled) throughout the caller's loop
            return (uint32_t)topk_push(wave_sort(a, lane), b, lane, K - 1);
          }
          uint32_t inner =
              __float_as_uint(__uint_as_float(t) * ((float)(K + kWave) * 0.5f * __builtin_amdgcn_rcpf((float)n)));
          return select_nearest<ORDERED, kOneRow, false>(
              2, K, inner, pend, lane,
              [&](auto f) {
                f((uint32_t)(a >> 32), (uint32_t)a);
                f((uint32_t)(b >> 32), (uint32_t)b);
              },
              [&](int row, int) -> key_t { return row ? b : a; });
        }
      }
      const uint32_t id = sort_queued(pend, fill, t, lane);
      wave_lds_sync();
      return id;
    }
    if (n < K) {
      lo = (int)t;
      at_lo = n;
    } else {
      hi = (int)t;
      at_hi = n;
    }
    if (hi - lo <= 1) break;  // neighbouring bit patterns straddle the window
    const float wanted = (float)(K + most) * 0.5f;
    auto scaled = [&] { return __uint_as_float(t) * (wanted * __builtin_amdgcn_rcpf((float)n)); };
    int next = -1;
    if (!LINEAR && it < 4) {
      if (n > 0) next = (int)__builtin_amdgcn_readfirstlane(__float_as_uint(scaled()));
    } else if (LINEAR ? it >= 4 && !(it & 1) : it & 1) {
      uint32_t above = 0xffffffffu;
      each([&](uint32_t d2, uint32_t) { above = min(above, (lo < 0 || d2 > (uint32_t)lo) ? d2 : 0xffffffffu); });
      next = (int)wave_min_u32(above, lane);
      if (next == hi) {  // nothing between: the distance hi has the surplus
        lo = hi - 1;
        break;
      }
    } else if (LINEAR && it < 18) {
      float x = n > 0 ? scaled() : __uint_as_float(t) * 4.f;
      if (at_hi >= 0) {
        const float from = lo < 0 ? 0.f : __uint_as_float((uint32_t)lo);
        float share = (wanted - (float)at_lo) * __builtin_amdgcn_rcpf((float)(at_hi - at_lo));
        if (lo >= 0) share = fminf(fmaxf(share, 0.0625f), 0.9375f);
        x = fmaf(__uint_as_float((uint32_t)hi) - from, share, from);
      }
      next = (int)__builtin_amdgcn_readfirstlane(__float_as_uint(x));
    }
    if (next <= lo || next >= hi) next = lo + (hi - lo) / 2;
    t = (uint32_t)next;
  }
  asm volatile("" : "+v"(lane));  // rare path: see sort_queued
  if (ORDERED) {
    int fill = 0;
    each([&](uint32_t d2, uint32_t low) { fill = queue_row(pend, fill, lo >= 0 && d2 <= (uint32_t)lo ? d2 : 0xffffffffu, low, (uint32_t)hi); });
    each([&](uint32_t d2, uint32_t low) { fill = queue_row<false>(pend, fill, d2 == (uint32_t)hi ? d2 : 0xffffffffu, low, (uint32_t)hi); });
    wave_lds_sync();
    const uint32_t id = sort_queued(pend, fill, (uint32_t)hi, lane);
    wave_lds_sync();
    return id;
  }
  key_t best = kKeyMax;
#pragma unroll 1
  for (int row = 0; row < rows; ++row) best = topk_push(best, key_at(row, lane), lane, K - 1);
  return (uint32_t)best;
}

}  // namespace affmae
