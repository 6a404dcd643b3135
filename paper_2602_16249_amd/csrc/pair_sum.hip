// The gathered half of the merging backward (paper, Sec. "AutoFocusFormer"): for every token
//   dfeat[token] = sum over the (anchor, neighbour) pairs that name it of weight[pair] * dout[anchor of the pair]
//   extra_sum[token] = sum of extra[pair] over the same pairs
// without floating-point atomics.
//
// One workgroup owns a range of an image's tokens: it picks the pairs that name one of them out of the image's, sorts
// them by token in LDS (counted, prefix-summed, placed), with the place of the pair's row in dout and its weight, and
// its waves add the rows up from there, G lanes of 16 bytes per row.  Neighbouring tokens are named by the same anchors,
// whose rows then come from the CU's own cache.  Before, one launch wrote every token's list to memory and a second one
// read, per 16 pairs of a token, the list, then the weights it named, then the rows; at C = 64 (bf16) half of the 16
// lanes that a token got had no channels.  8 images, 16384 tokens, 4096 anchors, K = 48, C = 64: 20.4 + 29.1 us and 4.6 for
// dp (which one workgroup of this launch adds up now); 25.5 us as here.
// (440 workgroups of 298 tokens: 33.8 us.)
// Bound by the chain of the sort (12 of its 16 us a workgroup: the anchors' masks, the pairs they point to, their weights:
// each step waits for memory) and then by the rows.  Two workgroups of 1024 threads per CU: 36.8 us with one (71
// registers).  Which anchors to look at is told by the cells of the image that their pairs name: 43.7 us with the lowest and highest
// token, which along a space-filling curve often lie far apart (of 4096 anchors 282 for 121 that do have a pair in 256 tokens).
// Where anchors crowd, a range has up to K pairs a token and its neighbours none: then the workgroups take the items that the launch before
// has listed, ranges with much to do first and in parts, the ranges without anchors last.  The same 8 images, us, whole backward, the
// two launches before / every workgroup its own range, with lists in memory where they do not fit / as here: anchors in a quarter of
// the frame 95 / 185 / 68, in a disc 97 / 183 / 78, by a smooth function of the place and some noise 95 / 177 / 67, at random 76 / 52.5 / 53.
// With parts of 3072 pairs instead of 4096 77, 86, 81 (three fifths of a part's time are the chain); with further parts behind all first
// ones instead of in front of the light ranges 87, 86, 84.
// Cells of more than 1024 groups come four at a time (one image of 262144 tokens, 65536 anchors: 155 us, one at a time 166); of fewer,
// the three that do not exist cost 0.8 us (16 images of 4096 tokens, this launch: 22.7 and 23.5).
// Places for 5120 pairs (the noted pairs make room for `extra`): with 4096 a range of the anchors at random did not fit in 3 of
// 40 batches, which then took 20 us longer.
// (The virtual tokens' backward, whose queries lie anywhere, would look at all pairs in every workgroup: 64.7 us for 17.3 +
// 39.0 + 4.7, 48 images of 8192 queries with 4 candidates.)
#include <algorithm>
#include <type_traits>

#include "cluster_common.h"
#include "device_util.h"
#include "launch.h"
#include "timing.h"

namespace affmae {
namespace {

constexpr int kSumThreads = 1024, kSumWaves = kSumThreads / kWave;
constexpr int kSumCap = 5 * kSumThreads;  // pairs of a workgroup's tokens that have a place in LDS
constexpr int kSumRange = 1024;           // most tokens of a workgroup
constexpr int kSumGroups = 8192;          // groups of pairs that a workgroup lists at a time

struct SumParams {
  const int32_t* pair_token;  // [B * ppi]: the pair's token, b * Nv + t
  const uint2* group_cells;   // which cells every `gs` consecutive pairs name
  PairCells cells;
  const uint4* dout;          // [B * ppi / row_pairs] rows of `pieces` 16-byte pieces
  const float *weights, *extra;
  uint4* dfeat;
  float* extra_sum;
  int32_t *crowds, *list;     // as in PairSumArgs
  int B, Nv, ppi, groups, gs, range, ranges, extras, pieces, row_pairs;
  uint32_t gs_magic, row_magic;
  const float* dp_part;       // dp = their sum, by one more workgroup, or nullptr
  int dp_n;
  float* dp;
};

template <typename T>
__device__ __forceinline__ void add_piece(const uint4& x, float w, float (&acc)[8]) {
  const uint32_t v[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if constexpr (sizeof(T) == 2) {
      acc[2 * e] = fmaf(w, __uint_as_float(v[e] << 16), acc[2 * e]);
      acc[2 * e + 1] = fmaf(w, __uint_as_float(v[e] & 0xffff0000u), acc[2 * e + 1]);
    } else {
      acc[e] = fmaf(w, __uint_as_float(v[e]), acc[e]);
    }
  }
}
template <typename T>
__device__ __forceinline__ uint4 pack_piece(const float (&a)[8]) {
  if constexpr (sizeof(T) == 2) return make_uint4(pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]), pack_bf16x2(a[4], a[5]), pack_bf16x2(a[6], a[7]));
  else return make_uint4(__float_as_uint(a[0]), __float_as_uint(a[1]), __float_as_uint(a[2]), __float_as_uint(a[3]));
}

// bits lo .. hi, 0 <= lo <= hi < 32
__device__ __forceinline__ uint32_t bit_range(int lo, int hi) { return (~0u >> (31 - (hi - lo))) << lo; }

// G: lanes per row (4, 8 or 16).  SPLIT: a wave per token, its 64 / G groups of lanes taking the token's pairs in turn
// (ranges of so few tokens that a group of lanes per token would leave lanes idle); otherwise G lanes per token.
template <typename T, int G, bool SPLIT>
__global__ __launch_bounds__(kSumThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void pair_sum_kernel(SumParams p) {
  __shared__ uint2 entry[kSumCap];  // row (its first piece in the image's dout), weight; before that: the listed groups
  __shared__ uint32_t hit_pair[kSumCap];  // pairs of the own tokens as they are found; then `extra` of the entries
  __shared__ uint16_t hit_token[kSumCap];
  float* const entry_extra = reinterpret_cast<float*>(hit_pair);
  __shared__ int32_t cnt[kSumRange];  // pairs per token; then the next free place of each; then where its list ends
  __shared__ int32_t wave_total[kSumWaves];
  __shared__ int32_t s_listed, s_hits, s_far;
  static_assert(kSumGroups * 4 <= kSumCap * 8, "the listed groups lie in the entries' place");
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  if (p.dp_part && blockIdx.x == gridDim.x - 1) {
    __shared__ float acc[kSumWaves];
    sum_parts(p.dp_part, 0, (size_t)p.dp_n, acc, p.dp);
    return;
  }
  // a range of an image's tokens, or a part of it
  const int at_extra = (int)blockIdx.x - p.B * p.ranges;
  const int b = at_extra < 0 ? blockIdx.x / p.ranges : at_extra / p.extras;
  int rg = at_extra < 0 ? blockIdx.x - b * p.ranges : p.ranges + at_extra - b * p.extras, part = 0, parts = 1;
  const uint2* group_cells = p.group_cells + (size_t)b * p.groups;
  if (p.extras) {
    const int item = p.crowds[(size_t)b * p.Nv + 1 + rg];
    if (item < 0) return;  // the whole workgroup
    parts = (item & (kSumMostParts - 1)) + 1;
    part = item / kSumMostParts & (kSumMostParts - 1);
    rg = item / (kSumMostParts * kSumMostParts);
  }
  const int each = parts == 1 ? p.range : (min(p.range, p.Nv - rg * p.range) + parts - 1) / parts;
  const int t0 = rg * p.range + part * each, span = min(each, min((rg + 1) * p.range, p.Nv) - t0);
  if (span <= 0) return;  // the whole workgroup (more parts than tokens)
  const int lo = b * p.ppi;  // the image's pairs
  cnt[tid] = 0;
  if (tid == 0) s_hits = 0;

  uint2 own;  // the cells that hold its tokens
  {
    const int lo_cell = exact_div(t0, p.cells.size, p.cells.magic), hi_cell = exact_div(t0 + span - 1, p.cells.size, p.cells.magic);
    const int r0 = lo_cell >> 5, r1 = hi_cell >> 5, c0 = lo_cell & 31, c1 = hi_cell & 31;
    if (p.cells.rows) {
      own.x = bit_range(r0, r1);
      own.y = hi_cell - lo_cell >= 31 ? ~0u : r0 == r1 ? bit_range(c0, c1) : bit_range(c0, 31) | bit_range(0, c1);
    } else {
      own.x = r0 == 0 ? bit_range(c0, r1 == 0 ? c1 : 31) : 0u;
      own.y = r1 == 1 ? bit_range(r0 == 1 ? c0 : 0, c1) : 0u;
    }
  }
  const int first = b * p.Nv + t0;
  // fn(tokens, pairs, in) for four pairs at a time, all lanes of a wave together, of the groups that name a token of these cells
  int32_t* glist = reinterpret_cast<int32_t*>(entry);
  auto each_pair = [&](auto&& fn) {
    for (int g0 = 0; g0 < p.groups; g0 += kSumGroups) {
      __syncthreads();  // the list before has been walked (and, the first time, the counters are set)
      if (tid == 0) s_listed = 0;
      __syncthreads();
      const int g1 = min(g0 + kSumGroups, p.groups);
      auto list_groups = [&](auto at_a_time) {
        constexpr int kU = decltype(at_a_time)::value;
        for (int gw = g0 + wave * kWave; gw < g1; gw += kU * kSumThreads) {
          uint2 named[kU];
#pragma unroll
          for (int u = 0; u < kU; ++u) named[u] = group_cells[min(gw + u * kSumThreads + lane, g1 - 1)];
          unsigned long long mask[kU];
          int found = 0;
#pragma unroll
          for (int u = 0; u < kU; ++u) {
            const bool x = (named[u].x & own.x) != 0u, y = (named[u].y & own.y) != 0u;
            mask[u] = __ballot(gw + u * kSumThreads + lane < g1 && (p.cells.rows ? x && y : x || y));
            found += __popcll(mask[u]);
          }
          int at = 0;
          if (lane == 0) at = atomicAdd(&s_listed, found);
          at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
          for (int u = 0; u < kU; ++u) {
            const int place = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask[u] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask[u], (uint32_t)at));
            if ((mask[u] >> lane) & 1ull) glist[place] = gw + u * kSumThreads + lane;
            at += __popcll(mask[u]);
          }
        }
      };
      if (g1 - g0 <= kSumThreads) list_groups(std::integral_constant<int, 1>{}); else list_groups(std::integral_constant<int, 4>{});
      __syncthreads();
      const int items = s_listed * p.gs;
      for (int i0 = 0; i0 < items; i0 += 4 * kSumThreads) {
        int pair[4], tok[4];
        bool in[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int at = i0 + u * kSumThreads + tid, i = min(at, items - 1);
          const int gi = exact_div(i, p.gs, p.gs_magic);
          in[u] = at < items;
          pair[u] = lo + glist[gi] * p.gs + (i - gi * p.gs);
          tok[u] = p.pair_token[pair[u]];
        }
        fn(tok, pair, in);
      }
    }
  };

  // the own tokens' pairs: counted and noted
  each_pair([&](const int (&tok)[4], const int (&pair)[4], const bool (&in)[4]) {
    unsigned long long mask[4];
    int found = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int rel = tok[u] - first;
      const bool own = in[u] && (unsigned)rel < (unsigned)span;
      mask[u] = __ballot(own);
      found += __popcll(mask[u]);
      if (own) atomicAdd(&cnt[rel], 1);
    }
    if (found == 0) return;  // wave-uniform
    int at = 0;
    if (lane == 0) at = atomicAdd(&s_hits, found);
    at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int place = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask[u] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask[u], (uint32_t)at));
      if (((mask[u] >> lane) & 1ull) && place < kSumCap) {
        hit_pair[place] = (uint32_t)pair[u];
        hit_token[place] = (uint16_t)(tok[u] - first);
      }
      at += __popcll(mask[u]);
    }
  });
  __syncthreads();
  // where each token's list starts
  const int mine = cnt[tid];
  int incl = mine;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int v = __shfl_up(incl, o);
    if (lane >= o) incl += v;
  }
  if (lane == kWave - 1) wave_total[wave] = incl;
  __syncthreads();
  int run = incl - mine, total = 0;
#pragma unroll
  for (int w = 0; w < kSumWaves; ++w) {
    const int t = wave_total[w];
    run += w < wave ? t : 0;
    total += t;
  }
  const bool fits = total <= kSumCap;
  cnt[tid] = run;
  // (lists that do not fit, where many pairs name few tokens, go to memory)
  if (!fits && tid == 0) s_far = atomicAdd(p.crowds + (size_t)b * p.Nv, total);
  __syncthreads();
  int32_t* const far = p.list + lo + (fits ? 0 : s_far);
  auto row_of = [&](int pair) { return (uint32_t)exact_div(pair - lo, p.row_pairs, p.row_magic) * (uint32_t)p.pieces; };
  if (fits) {
    constexpr int kMine = kSumCap / kSumThreads;
    int at[kMine];
    float extra[kMine];
#pragma unroll
    for (int u = 0; u < kMine; ++u) {
      const int i = u * kSumThreads + tid;
      if (i < total) {
        const int pair = (int)hit_pair[i];
        at[u] = atomicAdd(&cnt[hit_token[i]], 1);
        if (p.extra) extra[u] = p.extra[pair];
        entry[at[u]] = make_uint2(row_of(pair), __float_as_uint(p.weights[pair]));
      }
    }
    if (p.extra) {
      __syncthreads();  // hit_pair has been read
#pragma unroll
      for (int u = 0; u < kMine; ++u)
        if (u * kSumThreads + tid < total) entry_extra[at[u]] = extra[u];
    }
  } else {
    each_pair([&](const int (&tok)[4], const int (&pair)[4], const bool (&in)[4]) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int rel = tok[u] - first;
        if (in[u] && (unsigned)rel < (unsigned)span) far[atomicAdd(&cnt[rel], 1)] = pair[u];
      }
    });
    __threadfence_block();
  }
  __syncthreads();

  // the sums: N consumers of a token's list, this one the n-th, rows in flight four at a time
  constexpr int kGroupsOfLanes = kWave / G, kStep = SPLIT ? kGroupsOfLanes : 1;
  const int sub = lane & (G - 1), grp = lane / G;
  const uint4* rows = p.dout + (size_t)b * (p.ppi / p.row_pairs) * p.pieces;
  auto sums = [&](auto in_lds) {
  const int per_turn = SPLIT ? kSumWaves : kSumThreads / G;  // tokens at a time
  for (int r0 = 0; r0 < span; r0 += per_turn) {  // (workgroup-uniform)
    const int rel = r0 + (SPLIT ? wave : tid / G);
    const bool live = rel < span;
    const int l0 = live && rel > 0 ? cnt[rel - 1] : 0, l1 = live ? cnt[rel] : 0;
    const int from = l0 + (SPLIT ? grp : 0);
    auto at = [&](int i) -> uint2 {
      if constexpr (decltype(in_lds)::value) return entry[i];
      const int pair = far[i];
      return make_uint2(row_of(pair), __float_as_uint(p.weights[pair]));
    };
    for (int c0 = 0; c0 < p.pieces; c0 += G) {
      const int c = min(c0 + sub, p.pieces - 1);  // lanes past the row's end repeat its last piece (unused)
      float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      int i = from;
      for (; i + 3 * kStep < l1; i += 4 * kStep) {
        uint2 e[4];
        uint4 x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) e[u] = at(i + u * kStep);
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = rows[(size_t)(e[u].x + (uint32_t)c)];
#pragma unroll
        for (int u = 0; u < 4; ++u) add_piece<T>(x[u], __uint_as_float(e[u].y), acc);
      }
      if (i < l1) {  // up to three more: past the end the last one again, as zeros
        uint2 e[3];
        uint4 x[3];
#pragma unroll
        for (int u = 0; u < 3; ++u) e[u] = at(min(i + u * kStep, l1 - 1));
#pragma unroll
        for (int u = 0; u < 3; ++u) x[u] = rows[(size_t)(e[u].x + (uint32_t)c)];
#pragma unroll
        for (int u = 0; u < 3; ++u) {
          if (u > 0 && i + u * kStep >= l1) x[u] = make_uint4(0u, 0u, 0u, 0u);
          add_piece<T>(x[u], __uint_as_float(e[u].y), acc);
        }
      }
      if constexpr (SPLIT) {
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = lanes_sum<G, 32>(acc[e], lane);
      }
      if (live && c0 + sub < p.pieces && (!SPLIT || grp == 0)) p.dfeat[(size_t)(first + rel) * p.pieces + c] = pack_piece<T>(acc);
    }
    if (p.extra) {
      float x = 0.f;
      for (int i = l0 + (SPLIT ? lane : sub); i < l1; i += SPLIT ? kWave : G) x += decltype(in_lds)::value ? entry_extra[i] : p.extra[far[i]];
      x = lanes_sum<1, SPLIT ? 32 : G / 2>(x, lane);
      if (live && (SPLIT ? lane : sub) == 0) p.extra_sum[first + rel] = x;
    }
  }
  };
  if (fits) sums(std::true_type{}); else sums(std::false_type{});
}

}  // namespace

bool pair_sum_takes(const PairSumArgs& a) {
  auto al = [](const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; };
  const size_t row = (size_t)a.C * (a.dtype == 1 ? 2 : 4);
  if (row % 16 || !al(a.dout) || !al(a.dfeat)) return false;
  return (long long)(a.pairs_per_image / a.row_pairs) * (long long)(row / 16) < (1ll << 32);  // places of an image's rows
}

// Lanes per row of `pieces` 16-byte pieces.
static int pair_sum_lanes(int pieces) { return pieces <= 4 ? 4 : pieces <= 8 ? 8 : 16; }

PairSumShape pair_sum_shape(const PairSumArgs& a) {
  PairSumShape s;
  // tokens of a workgroup: two workgroups per CU, but on average no more pairs than three fifths of the places
  const int want = std::max(1, (512 + a.B - 1) / a.B);
  const long long fit = std::max(1ll, (long long)(kSumCap * 3 / 5) * a.Nv / std::max(1, a.pairs_per_image));
  const int range = (int)std::min({std::max(64ll, ((long long)a.Nv + want - 1) / want), fit, (long long)kSumRange});
  // A bit per range where there are no more than 64 of them; else rows, and a quarter of a range, so that the columns tell
  // neighbouring ranges apart, or as much as 1024 cells need.  (One of 64 parts of the image, a bit each, whatever the ranges are:
  // with one image of 262144 tokens, 64 channels, 65536 anchors of 48 pairs the whole backward took 176 us, and with 16384 tokens 19.4;
  // as here 148 and 18.8.  Rows for 64 ranges as well, an anchor's pairs lying in several: one image of 4096 tokens 14.6 instead of 14.1.)
  s.cells.rows = (a.Nv + range - 1) / range > 64;
  s.cells.size = s.cells.rows ? std::max((a.Nv + 1023) / 1024, range / 4) : (a.Nv + 63) / 64;
  s.cells.magic = div_magic(s.cells.size);
  const int pieces = (int)((size_t)a.C * (a.dtype == 1 ? 2 : 4) / 16);
  const int turn = kSumThreads / pair_sum_lanes(pieces);  // tokens at a time, with G lanes each: whole turns
  s.range = range > turn ? range / turn * turn : range;
  s.ranges = (a.Nv + s.range - 1) / s.range;
  s.range_magic = div_magic(s.range);
  s.front = a.pairs_per_image > kSumCap ? (a.B + 7) / 8 * 8 : 0;
  s.extras = s.front && s.ranges <= kSumMostRanges && (long long)s.range * a.row_pairs > kSumCrowd ? a.pairs_per_image / kSumPart : 0;
  return s;
}

hipError_t launch_pair_sum(const PairSumArgs& a, const PairSumShape& shape, hipStream_t stream) {
  SumParams p;
  p.pair_token = a.pair_token; p.group_cells = a.group_cells; p.cells = shape.cells;
  p.dout = static_cast<const uint4*>(a.dout); p.weights = a.weights; p.extra = a.extra;
  p.dfeat = static_cast<uint4*>(a.dfeat); p.extra_sum = a.extra_sum;
  p.crowds = a.crowds; p.list = a.list; p.extras = shape.extras;
  p.B = a.B; p.Nv = a.Nv; p.ppi = a.pairs_per_image; p.row_pairs = a.row_pairs; p.row_magic = div_magic(a.row_pairs);
  p.gs = a.group_size; p.groups = a.pairs_per_image / p.gs; p.gs_magic = div_magic(p.gs);
  p.pieces = (int)((size_t)a.C * (a.dtype == 1 ? 2 : 4) / 16);
  p.dp_part = a.dp_part; p.dp_n = a.dp_n; p.dp = a.dp;
  p.range = shape.range; p.ranges = shape.ranges;
  const dim3 grid((unsigned)(a.B * (p.ranges + p.extras) + (a.dp_part ? 1 : 0)));
  const int g = pair_sum_lanes(p.pieces);
  const bool split = p.range * g < kSumThreads / 2;
#define AFFMAE_SUM(T, G, SPLIT) \
  AFFMAE_LAUNCH("pair_sum_kernel", stream, (pair_sum_kernel<T, G, SPLIT>), grid, dim3(kSumThreads), 0, stream, p)
#define AFFMAE_SUM_G(T, SPLIT)             \
  do {                                     \
    if (g == 4) AFFMAE_SUM(T, 4, SPLIT);   \
    else if (g == 8) AFFMAE_SUM(T, 8, SPLIT); \
    else AFFMAE_SUM(T, 16, SPLIT);         \
  } while (0)
  if (a.dtype == 1) {
    if (split) AFFMAE_SUM_G(bf16_t, true); else AFFMAE_SUM_G(bf16_t, false);
  } else {
    if (split) AFFMAE_SUM_G(float, true); else AFFMAE_SUM_G(float, false);
  }
#undef AFFMAE_SUM_G
#undef AFFMAE_SUM
  return hipGetLastError();
}

}  // namespace affmae
