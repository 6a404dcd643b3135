// Plan of the cluster-tiled attention kernels, built from the neighbour table
// (paper, Sec. "Limitations": neighbourhood tables are cached per encoder stage
// and reused by every block; the plan is such a table in the layout the tiled
// kernels read, see PlanLayout).  Forward tables: a workgroup per group of four
// strips, a wave per strip of 16 queries.  Reverse tables (which strips touch a
// group of token tiles): one kernel that counts, places, files and sorts in LDS
// (large images: count, prefix sum, fill and sort kernels).
#include "cluster_common.h"
#include "launch.h"
#include "timing.h"

#include <algorithm>
#include <type_traits>

namespace affmae {
namespace {

struct PlanParams {
  const int32_t* nbr_idx;  // [B,N,K]
  const int32_t* near;     // [B,G,M]
  int N, K, S, M, G;
  uint32_t s_magic, tpc_magic, gpi_magic;
  int strips_per_image, groups_per_image, groups, uni_stride, pos_stride, jt_pairs, touch_stride;
  uint16_t* uni;
  uint8_t* pos;
  uint8_t* jt;
  unsigned long long* touch;
  int32_t* rev_count;
  int32_t* rev_offset;
  int32_t* rev_cursor;
  unsigned long long* rev_list;
  int group0;         // first group of this launch's slice (strip kernel)
  bool count_groups;  // the reverse tables are built by the count / scan / fill / sort kernels
};

__device__ __forceinline__ unsigned long long wave_or64(unsigned long long x) {
  uint32_t lo = wave_or32((uint32_t)x), hi = wave_or32((uint32_t)(x >> 32));
  return ((unsigned long long)hi << 32) | lo;
}

__global__ __launch_bounds__(256) void plan_zero_kernel(int32_t* a, int32_t* b, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    a[i] = 0;
    b[i] = 0;
  }
}

// inclusive prefix sum over the wave (all lanes active)
__device__ __forceinline__ int wave_prefix(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1, 2, 4, 8
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
  return x;
}

// A strip's candidate tiles are those of its near clusters, numbered by cluster and place (at most 64).  NE = entries per
// lane: 16 K / 64 rounded up to a multiple of 4 (the loops over a lane's entries are unrolled); the four lanes of a query
// share its list.  The pairs go to their bytes by plain LDS stores.
// Bound by the vector ALU, so whatever can be looked up in LDS is: TABLE, for images of at most kTableTiles token tiles,
// finds an entry's candidate by its tile in a table of bytes, the candidates in use by marks, an entry's slot in a table
// by candidate, and the places in the group's union by the prefix sum of a bit map of the image's tiles.  Without it an
// entry's cluster is compared with every near one, and a tile's place is searched in the lists of the group's strips.
// Whole plan, K = 48, S = 64, M = 8, with comparisons and searches throughout and now: 16 images of 16384 tokens 51.5 and
// 31.2 us (the kernel itself 42 and 21.5, 1230 and 480 vector instructions a strip), 16 of 4096 22.0 and 15.2, one of 1024
// 13.7 and 10.6; 4 images of 57344, the most that the table's place in LDS allows, 53.7 and 37.3, of 57360 54.1 and 48.2.
constexpr int kJtSlots = 16;  // slots whose j tiles are assembled in LDS at a time (4 KB per strip); few strips have more
constexpr int kTableTiles = 3584;
constexpr uint32_t kNoCandidate = 64, kNoPlace = 0xffff;
struct StripTables {            // in LDS, where the j tiles are assembled afterwards
  uint8_t candidate[kTableTiles];  // by token tile of the image
  uint8_t mark[128];               // by candidate
  uint16_t at[128];                // by candidate: where its slot's bytes start among the j tiles
};
static_assert(sizeof(StripTables) <= kJtSlots * 256 && kTableTiles % 16 == 0 && kTableTiles <= 64 * kWave, "");
__device__ __forceinline__ uint32_t slot_start(int slot) { return (uint32_t)((slot >> 1) * 512 + (slot & 1) * 4); }

template <int NE, bool TABLE>
__global__ __launch_bounds__(256) void pla_plan_kernel(PlanParams p) {
  __shared__ __align__(16) uint8_t jt_all[kGroup][kJtSlots * 256];
  __shared__ uint16_t tiles_all[kGroup][kMaxSlots];
  __shared__ __align__(8) uint32_t map_all[TABLE ? kGroup : 1][2 * kWave];  // TABLE: a strip's tiles, a bit each
  __shared__ int count_all[kGroup];
  __shared__ unsigned long long fresh_all[kGroup];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);  // uniform: keeps per-wave indices in SGPRs
  const int gi = p.group0 + blockIdx.x;
  const int b = exact_div(gi, p.groups_per_image, p.gpi_magic);
  const int si = (gi - b * p.groups_per_image) * kGroup + wave;
  const bool there = si < p.strips_per_image;  // the image's last group may have fewer strips
  const int q0 = min(si, p.strips_per_image - 1) * 16;  // first query, within the image
  const size_t sg = (size_t)b * p.strips_per_image + (q0 >> 4);
  const int c = fast_div(q0, p.s_magic);
  const int32_t* near_c = p.near + ((size_t)b * p.G + c) * p.M;
  const int tpc = p.S / 16;  // token tiles per cluster
  const int queries = there ? min(16, p.N - q0) : 0;  // the image's last strip may hold fewer than 16
  const int q = lane >> 2, j0 = lane & 3;  // this lane: places j0, j0 + 4, ... of the list of query q
  const int32_t* nbr = p.nbr_idx + ((size_t)b * p.N + q0) * p.K;
  const uint32_t row = (uint32_t)(min(q, max(queries, 1) - 1) * p.K);
  uint8_t* jt = jt_all[wave];
  StripTables& table = *reinterpret_cast<StripTables*>(jt);

  const int near_v = (lane < p.M) ? near_c[lane] : 0x7fffffff;  // lane m: the m-th near cluster (M <= 64)
  int tok[NE];
  bool inr[NE];
#pragma unroll
  for (int t = 0; t < NE; ++t) tok[t] = nbr[row + (uint32_t)min(4 * t + j0, p.K - 1)];
#pragma unroll
  for (int t = 0; t < NE; ++t) {
    const int n = tok[t];
    tok[t] = min(max(n, 0), p.N - 1);
    inr[t] = n == tok[t] && 4 * t + j0 < p.K && q < queries;  // queries past the end have no entries
  }
  // candidate tile of every (query, neighbour): clusters in ascending order, (token % S) / 16 inside
  const int lane_m = fast_div(lane, p.tpc_magic);
  int rank = 0;  // lane m: near clusters below the m-th one
  for (int m = 0; m < p.M; ++m) rank += __builtin_amdgcn_readlane(near_v, m) < near_v ? 1 : 0;
  const bool known = (uint32_t)near_v < (uint32_t)p.G;
  // lane c: the cluster of candidate c (one that is there twice goes to one place; -1: none)
  const int cl_by_rank = __builtin_amdgcn_ds_permute(rank << 2, known ? near_v + 1 : 0) - 1;
  const int cl = __builtin_amdgcn_ds_bpermute(lane_m << 2, cl_by_rank);
  const int my_tile = cl * tpc + (lane - lane_m * tpc);  // of candidate `lane`, within the image
  uint32_t at[NE];  // where an entry's byte lies among the j tiles
  unsigned long long mask;  // candidates in use
  if constexpr (TABLE) {
    for (int i = lane; i < (p.strips_per_image + 15) / 16; i += kWave)
      reinterpret_cast<u32x4*>(table.candidate)[i] = (u32x4)(kNoCandidate * 0x01010101u);
    table.mark[lane] = 0;
    *reinterpret_cast<unsigned long long*>(&map_all[wave][2 * lane]) = 0ull;
    wave_lds_sync();
    if (lane < p.M * tpc && cl >= 0 && my_tile < p.strips_per_image) table.candidate[my_tile] = (uint8_t)lane;
    wave_lds_sync();
#pragma unroll
    for (int t = 0; t < NE; ++t) {
      at[t] = table.candidate[tok[t] >> 4];
      at[t] = inr[t] ? at[t] : kNoCandidate;
    }
#pragma unroll
    for (int t = 0; t < NE; ++t) table.mark[at[t]] = 1;
    wave_lds_sync();
    mask = __builtin_amdgcn_ballot_w64(table.mark[lane] != 0);
  } else {
    int ecl[NE], ct[NE];
#pragma unroll
    for (int t = 0; t < NE; ++t) {
      ecl[t] = fast_div(tok[t], p.s_magic);
      ct[t] = -1;
    }
    for (int m = 0; m < p.M; ++m) {
      const int near_m = __builtin_amdgcn_readlane(near_v, m), rk = __builtin_amdgcn_readlane(rank, m);
#pragma unroll
      for (int t = 0; t < NE; ++t) ct[t] = (ecl[t] == near_m) ? rk * tpc : ct[t];
    }
    mask = 0;
#pragma unroll
    for (int t = 0; t < NE; ++t) {
      const int cand = ct[t] + ((tok[t] - ecl[t] * p.S) >> 4);
      const bool there_t = inr[t] && ct[t] >= 0;
      mask |= there_t ? 1ull << cand : 0ull;
      at[t] = there_t ? (uint32_t)cand : kNoCandidate;
    }
    mask = wave_or64(mask);
  }
  const int count = __popcll(mask);
  const bool used = (mask >> lane) & 1ull;
  const int my_slot = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
  if (used) tiles_all[wave][my_slot] = (uint16_t)my_tile;
  if constexpr (TABLE) {
    if (used) atomicOr(&map_all[wave][my_tile >> 5], 1u << (my_tile & 31));
    table.at[lane] = (uint16_t)slot_start(my_slot);
    if (lane == 0) table.at[kNoCandidate] = (uint16_t)kNoPlace;
    wave_lds_sync();
#pragma unroll
    for (int t = 0; t < NE; ++t) at[t] = table.at[at[t]];
  } else {
#pragma unroll
    for (int t = 0; t < NE; ++t)
      at[t] = at[t] == kNoCandidate ? kNoPlace : slot_start(__popcll(mask & ((1ull << at[t]) - 1ull)));
    if (lane == 0) count_all[wave] = count;
  }
  __syncthreads();
  // lane s: slot s, and its tile's place in the union of the group's strips
  const int T = lane < count ? (int)tiles_all[wave][lane] : 0x10000;
  int place, U;
  uint16_t* uni = p.uni + (size_t)gi * p.uni_stride;
  if constexpr (TABLE) {
    unsigned long long all = 0ull;  // lane i: tiles 64 i .. 64 i + 63
#pragma unroll
    for (int v = 0; v < kGroup; ++v) all |= *reinterpret_cast<const unsigned long long*>(&map_all[v][2 * lane]);
    const int n = __popcll(all), upto = wave_prefix(n);
    U = __builtin_amdgcn_readlane(upto, kWave - 1);
    const int from = (T >> 6) << 2;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)(uint32_t)all);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)(uint32_t)(all >> 32));
    place = __builtin_amdgcn_ds_bpermute(from, upto - n) + __popcll((((unsigned long long)hi << 32) | lo) & ((1ull << (T & 63)) - 1ull));
    if (lane < count) uni[1 + place] = (uint16_t)T;  // (from every strip that touches it)
  } else {
    // a tile's place in every strip's list by binary search; a strip is the first of the group to have the tile if no
    // earlier one does, and the place in the union is the number of firsts below
    int lb[kGroup];
    bool fresh = lane < count;
#pragma unroll
    for (int v = 0; v < kGroup; ++v) {
      const int n = count_all[v];
      int low = 0;
#pragma unroll
      for (int step = 32; step > 0; step >>= 1)
        if (low + step <= n && (int)tiles_all[v][low + step - 1] < T) low += step;
      if (low < n && (int)tiles_all[v][low] < T) ++low;  // (the steps add up to 63, a list may hold 64)
      lb[v] = low;
      if (v < wave && low < n && (int)tiles_all[v][low] == T) fresh = false;
    }
    const unsigned long long fm = __ballot(fresh);
    if (lane == 0) fresh_all[wave] = fm;
    __syncthreads();
    place = 0, U = 0;
#pragma unroll
    for (int v = 0; v < kGroup; ++v) {
      const unsigned long long f = fresh_all[v];
      place += __popcll(lb[v] >= kWave ? f : (f & ((1ull << lb[v]) - 1ull)));
      U += __popcll(f);
    }
    if (fresh) uni[1 + place] = (uint16_t)T;
  }
  if (wave == 0 && lane == 0) {
    uni[0] = (uint16_t)max(U, 1);  // (no tile at all only where the near clusters are not the table's: one that nobody uses)
    if (U == 0) uni[1] = (uint16_t)(q0 >> 4);
  }
  if (!there) return;  // (no workgroup barrier below)
  uint8_t* pos = p.pos + sg * p.pos_stride;
  if (lane < count) pos[1 + lane] = (uint8_t)place;
  if (lane == 0) pos[0] = (uint8_t)count;
  // groups of token tiles: a slot whose group differs from the slot's before starts one
  unsigned long long* touch = p.touch + sg * p.touch_stride;
  const int tg = T / kGroup;
  const int before = __shfl_up(tg, 1);
  const bool starts = lane < count && (lane == 0 || before != tg);
  const unsigned long long sm = __ballot(starts);
  if (starts) {
    uint32_t slots = 0xffffffffu;
#pragma unroll
    for (int d = 0; d < kGroup; ++d) {
      const int tile = lane + d < count ? (int)tiles_all[wave][lane + d] : 0x10000;
      if (tile / kGroup == tg) slots = (slots & ~(0xffu << (8 * (tile % kGroup)))) | ((uint32_t)(lane + d) << (8 * (tile % kGroup)));
    }
    touch[1 + __popcll(sm & ((1ull << lane) - 1ull))] = ((unsigned long long)(uint32_t)tg << 32) | slots;
    if (p.count_groups) atomicAdd(p.rev_count + (size_t)b * p.groups_per_image + tg, 1);
  }
  if (lane == 0) touch[0] = (unsigned long long)__popcll(sm);
  // j tiles
  u32x4* out = reinterpret_cast<u32x4*>(p.jt + sg * p.jt_pairs * 512);
  const uint32_t none = 2u * (uint32_t)p.K * 0x01010101u;
#pragma unroll
  for (int t = 0; t < NE; ++t) at[t] += (uint32_t)(((tok[t] & 12) << 5) | (tok[t] & 3)) + (uint32_t)q * 8u;
  for (int s0 = 0; s0 < count; s0 += kJtSlots) {
    const int ns = min(kJtSlots, (count - s0 + 1) & ~1);  // the second half of the last pair holds no neighbours
    for (int i = lane; i < ns * 16; i += kWave) reinterpret_cast<u32x4*>(jt)[i] = u32x4{none, none, none, none};
    wave_lds_sync();
#pragma unroll
    for (int t = 0; t < NE; ++t) {
      const uint32_t here = at[t] - (uint32_t)s0 * 256u;
      if (here < kJtSlots * 256u) jt[here] = (uint8_t)(2 * (4 * t + j0));
    }
    wave_lds_sync();
    for (int i = lane; i < ns * 16; i += kWave) out[s0 * 16 + i] = reinterpret_cast<const u32x4*>(jt)[i];
    wave_lds_sync();
  }
}

// Exclusive prefix sum of rev_count.  Workgroup j owns elements [1024 j, 1024 j + 1024): it first adds up
// everything before them (coalesced reads of a few hundred KB at most, all from L2), then scans its own.
// No workgroup waits for another.
__global__ __launch_bounds__(256) void plan_scan_kernel(const int32_t* __restrict__ count, int32_t* __restrict__ offset,
                                                       int n) {
  __shared__ int32_t part[4];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int first = blockIdx.x * 1024;
  int before = 0;
  for (int i = tid * 4; i < first; i += 1024) {  // first is a multiple of 1024: whole 16-byte pieces
    const int4 v = *reinterpret_cast<const int4*>(count + i);
    before += v.x + v.y + v.z + v.w;
  }
  // this thread's four elements
  const int at = first + tid * 4;
  int c[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) c[i] = (at + i < n) ? count[at + i] : 0;
  const int mine = c[0] + c[1] + c[2] + c[3];
  // wave-inclusive scan of (mine) and wave sum of (before)
  int incl = mine;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int v = __shfl_up(incl, o);
    if (lane >= o) incl += v;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o);
  if (lane == kWave - 1) part[wave] = incl;
  __shared__ int32_t before_all[4];
  if (lane == 0) before_all[wave] = before;
  __syncthreads();
  int base = before_all[0] + before_all[1] + before_all[2] + before_all[3];
  for (int w = 0; w < wave; ++w) base += part[w];
  int run = base + incl - mine;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (at + i < n) offset[at + i] = run;
    run += c[i];
  }
  if (at <= n - 1 && n - 1 < at + 4) offset[n] = run;  // the thread that owns the last element: run is the total
}

// Every strip appends itself to the list of each group of token tiles it touches.
__global__ __launch_bounds__(256) void plan_fill_kernel(PlanParams p, int strips) {
  const int lane = threadIdx.x & (kWave - 1);
  const int sg = blockIdx.x * (blockDim.x / kWave) + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (sg >= strips) return;
  const int b = sg / p.strips_per_image;
  const int strip = sg - b * p.strips_per_image;
  const unsigned long long* touch = p.touch + (size_t)sg * p.touch_stride;
  const int count = min((int)touch[0], p.touch_stride - 1);
  if (lane < count) {
    const unsigned long long t = touch[1 + lane];
    const size_t grp = (size_t)b * p.groups_per_image + (uint32_t)(t >> 32);
    const int at = atomicAdd(p.rev_cursor + grp, 1);
    p.rev_list[(size_t)p.rev_offset[grp] + at] = ((unsigned long long)(uint32_t)strip << 32) | (uint32_t)t;
  }
}

// How many of a list's n entries (at least one; in memory or in LDS) belong to a strip below `key`: a list is sorted by
// putting every entry at that place (its strips are distinct).  One wave, every lane its own key.
__device__ __forceinline__ int entries_below(const unsigned long long* list, int n, uint32_t key, int lane) {
  int rank = 0;
  for (int j0 = 0; j0 < n; j0 += kWave) {
    const uint32_t other = j0 + lane < n ? (uint32_t)(list[j0 + lane] >> 32) : ~0u;  // (behind the list: below no key)
    for (int j1 = 0; j1 < min(kWave, n - j0); j1 += 16)
#pragma unroll
      for (int j = 0; j < 16; ++j) rank += __builtin_amdgcn_readlane(other, j1 + j) < key ? 1 : 0;
  }
  return rank;
}

// Sorts one group's list ascending by strip.  One wave; lists of more than 64 entries (popular groups) by way of a copy.
// (One lane's insertion sort of a list of 96 held up the whole plan: 241 us for 27 now, B2 N20480 K16 S64 M8.)
__device__ __forceinline__ void sort_list(unsigned long long* list, unsigned long long* copy, int n, int lane) {
  if (n <= kWave) {
    const unsigned long long mine = lane < n ? list[lane] : ~0ull;
    const int rank = entries_below(list, n, (uint32_t)(mine >> 32), lane);
    if (lane < n) list[rank] = mine;  // every lane has read its element before any write lands (one wave)
    return;
  }
  for (int i = lane; i < n; i += kWave) copy[i] = list[i];
  __threadfence_block();  // (every lane reads what the others have written)
  for (int i0 = 0; i0 < n; i0 += kWave) {
    const unsigned long long mine = copy[min(i0 + lane, n - 1)];
    const int rank = entries_below(copy, n, (uint32_t)(mine >> 32), lane);
    if (i0 + lane < n) list[rank] = mine;
  }
}

__global__ __launch_bounds__(256) void plan_sort_kernel(PlanParams p) {
  const int lane = threadIdx.x & (kWave - 1);
  const int grp = blockIdx.x * (blockDim.x / kWave) + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (grp >= p.groups) return;
  // (the touch tables have been filed: their place, an entry per strip larger than the lists', takes the copies)
  const int at = __builtin_amdgcn_readfirstlane(p.rev_offset[grp]), n = __builtin_amdgcn_readfirstlane(p.rev_count[grp]);
  sort_list(p.rev_list + at, p.touch + at, n, lane);
}

// The reverse tables of images of at most kRevThreads strips, in one launch: a workgroup owns `own` consecutive groups
// of one image.  A thread reads the touch table of one of the image's strips, the workgroup counts every group's strips
// in LDS, prefix-sums the counts (an image's lists start at a place of their own, so nothing is needed of other images),
// files the strips of its own groups, and sorts these lists in LDS.
// Bound by the chain of these steps in each workgroup, which grows with the image's tiles, against counting with atomics
// in the strip kernel and four more launches (zero, scan, fill, sort: 4 - 6 us each, of the whole batch).  Whole plan, K =
// 48, one launch and four: one image of 64 / 256 / 512 / 1024 tiles 10 / 11 / 12.5 / 12.5 us and 19 us; 1024 tiles, 4 / 8 / 16 / 32
// images 15 / 19 / 26 / 39 us and 21 / 26 / 35 / 53 us.  (Not faster: the touch tables read twice and the lists sorted in memory; a
// list per token tile instead of per group; a list's places from LDS instead of broadcast lanes.)  Beyond 1024 tiles a thread would
// serve several strips.
// Images of a few tiles take a workgroup each and give it little to do (1 tile: 8 / 15 / 24 us at 256 / 1024 / 2048 images against
// 19; 4 tiles: 15 / 23 us at 768 / 1536 against 19 / 21; 16 tiles 24 / 38 us against 29 / 41): below 16 tiles, up to 768.
constexpr int kRevThreads = 1024, kRevGroups = kRevThreads / kGroup, kRevGroupsFew = 4, kRevImagesFew = 768;
constexpr int kRevSorted = 1024;  // entries of a workgroup's lists that are in LDS at a time
static_assert(kRevSorted >= kRevThreads, "room for a group's list of all the image's strips");
constexpr int kRevInline = 7;     // entries of a strip that its thread holds (most strips have fewer)
__global__ __launch_bounds__(kRevThreads) void plan_reverse_kernel(PlanParams p, int own) {
  __shared__ int32_t count[kRevGroups];   // strips per group
  __shared__ int32_t offset[kRevGroups];  // exclusive prefix, then the cursor of the own groups
  __shared__ int32_t part[kRevThreads / kWave];
  __shared__ unsigned long long sorted[kRevSorted];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int gpi = p.groups_per_image;
  const int shares = (gpi + own - 1) / own;
  const int block = gridDim.x % 8 == 0 ? xcd_contiguous_block(blockIdx.x, gridDim.x) : blockIdx.x;
  const int b = block / shares, first = (block - b * shares) * own, last = min(first + own, gpi);
  const size_t strip0 = (size_t)b * p.strips_per_image;
  const unsigned long long* row = p.touch + (strip0 + min(tid, p.strips_per_image - 1)) * p.touch_stride;
  unsigned long long w[1 + kRevInline];
#pragma unroll
  for (int i = 0; i <= kRevInline; ++i) w[i] = row[min(i, p.touch_stride - 1)];
  if (tid < kRevGroups) count[tid] = 0;
  __syncthreads();
  const int n = tid < p.strips_per_image ? min((int)w[0], p.touch_stride - 1) : 0;
  auto each = [&](auto f) {
#pragma unroll
    for (int s = 0; s < kRevInline; ++s) {
      const int grp = (int)(w[1 + s] >> 32);
      if (s < n && (uint32_t)grp < (uint32_t)gpi) f(grp, (uint32_t)w[1 + s]);
    }
    for (int s = kRevInline; s < n; ++s) {
      const unsigned long long t = row[1 + s];
      const int grp = (int)(t >> 32);
      if ((uint32_t)grp < (uint32_t)gpi) f(grp, (uint32_t)t);
    }
  };
  each([&](int grp, uint32_t) { atomicAdd(&count[grp], 1); });
  __syncthreads();
  // exclusive prefix: a group per thread
  const int mine = tid < kRevGroups ? count[tid] : 0;
  int incl = mine;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int v = __shfl_up(incl, o);
    if (lane >= o) incl += v;
  }
  if (lane == kWave - 1) part[wave] = incl;
  __syncthreads();
  int before = incl - mine;
  for (int i = 0; i < min(wave, kRevGroups / kWave); ++i) before += part[i];
  if (tid < kRevGroups) offset[tid] = before;
  const size_t list0 = strip0 * (p.touch_stride - 1);  // the image's lists
  if (tid >= first && tid < last) {
    p.rev_count[(size_t)b * gpi + tid] = mine;
    p.rev_offset[(size_t)b * gpi + tid] = (int32_t)(list0 + before);
  }
  __syncthreads();
  unsigned long long* list = p.rev_list + list0;
  // as many of the own groups at a time as have room for their lists in LDS (one has: it lists a strip once)
  for (int g0 = first, g1; g0 < last; g0 = g1) {
    const int base = offset[g0];
    g1 = last;
    if (offset[last - 1] + count[last - 1] - base > kRevSorted) {
      int total = count[g0];
      for (g1 = g0 + 1; g1 < last && total + count[g1] <= kRevSorted; ++g1) total += count[g1];
    }
    __syncthreads();  // (offset becomes the cursors)
    each([&](int grp, uint32_t slots) {
      if (grp >= g0 && grp < g1) sorted[atomicAdd(&offset[grp], 1) - base] = ((unsigned long long)(uint32_t)tid << 32) | slots;
    });
    __syncthreads();
    for (int grp = g0 + wave; grp < g1; grp += kRevThreads / kWave) {
      const int m = __builtin_amdgcn_readfirstlane(count[grp]), at = __builtin_amdgcn_readfirstlane(offset[grp]) - m;
      for (int i0 = 0; i0 < m; i0 += kWave) {
        const unsigned long long v = sorted[at - base + min(i0 + lane, m - 1)];
        const int rank = entries_below(sorted + (at - base), m, (uint32_t)(v >> 32), lane);
        if (i0 + lane < m) list[at + rank] = v;
      }
    }
    __syncthreads();
  }
}

}  // namespace

hipError_t launch_pla_plan(const int32_t* nbr_idx, const int32_t* near, int B, int N, int K, int S, int M, void* plan,
                           hipStream_t stream) {
  const PlanLayout L = make_plan_layout(B, N, K, S, M);
  char* base = static_cast<char*>(plan);
  PlanParams p;
  p.nbr_idx = nbr_idx; p.near = near;
  p.N = N; p.K = K; p.S = S; p.M = M; p.G = (N + S - 1) / S;  // the last cluster may be short
  p.s_magic = div_magic(S); p.tpc_magic = div_magic(S / 16); p.gpi_magic = div_magic(L.groups_per_image);
  p.strips_per_image = L.strips_per_image; p.groups_per_image = L.groups_per_image; p.groups = L.groups;
  p.uni_stride = L.uni_stride; p.pos_stride = L.pos_stride; p.jt_pairs = L.jt_pairs; p.touch_stride = L.touch_stride;
  p.uni = reinterpret_cast<uint16_t*>(base + L.uni_off);
  p.pos = reinterpret_cast<uint8_t*>(base + L.pos_off);
  p.jt = reinterpret_cast<uint8_t*>(base + L.jt_off);
  p.touch = reinterpret_cast<unsigned long long*>(base + L.touch_off);
  p.rev_count = reinterpret_cast<int32_t*>(base + L.rev_count_off);
  p.rev_offset = reinterpret_cast<int32_t*>(base + L.rev_offset_off);
  p.rev_cursor = reinterpret_cast<int32_t*>(base + L.rev_cursor_off);
  p.rev_list = reinterpret_cast<unsigned long long*>(base + L.rev_list_off);
  // One launch where it is the faster way (see plan_reverse_kernel), list places fit int32 and the threads a launch
  // (2^32 - 1).  256 workgroups share the groups, four or more each.
  const int gpi = L.groups_per_image;
  const int own = std::max(4, (int)((L.groups + 255ll) / 256));
  const long long shares = (long long)B * ((gpi + own - 1) / own);
  const bool one_launch = gpi < kRevGroupsFew ? B <= kRevImagesFew : L.strips_per_image <= kRevThreads;
  p.count_groups = !one_launch || (long long)L.strips * (L.touch_stride - 1) >= (1ll << 31) || shares * kRevThreads >= (1ll << 32);
  if (p.count_groups)
    AFFMAE_LAUNCH("plan_zero_kernel", stream, plan_zero_kernel, dim3((L.groups + 255) / 256), dim3(256), 0, stream,
                  p.rev_count, p.rev_cursor, L.groups);
  const int ne = (16 * K + kWave - 1) / kWave;
  for (long long g0 = 0; g0 < L.groups; g0 += kMaxBlocks) {
    p.group0 = (int)g0;
    const dim3 grid((unsigned)std::min((long long)L.groups - g0, kMaxBlocks));
    auto kernel = [&](auto table) {
      return ne <= 4 ? pla_plan_kernel<4, table.value> : ne <= 8 ? pla_plan_kernel<8, table.value>
             : ne <= 12 ? pla_plan_kernel<12, table.value> : pla_plan_kernel<kMaxEntries, table.value>;
    };
    AFFMAE_LAUNCH("pla_plan_kernel", stream, (L.strips_per_image <= kTableTiles ? kernel(std::true_type{}) : kernel(std::false_type{})),
                  grid, dim3(256), 0, stream, p);
  }
  if (!p.count_groups) {
    AFFMAE_LAUNCH("plan_reverse_kernel", stream, plan_reverse_kernel, dim3((unsigned)shares), dim3(kRevThreads), 0, stream, p, own);
    return hipGetLastError();
  }
  AFFMAE_LAUNCH("plan_scan_kernel", stream, plan_scan_kernel, dim3((L.groups + 1023) / 1024), dim3(256), 0, stream,
                p.rev_count, p.rev_offset, L.groups);
  AFFMAE_LAUNCH("plan_fill_kernel", stream, plan_fill_kernel, dim3((L.strips + 3) / 4), dim3(256), 0, stream, p, L.strips);
  AFFMAE_LAUNCH("plan_sort_kernel", stream, plan_sort_kernel, dim3((L.groups + 3) / 4), dim3(256), 0, stream, p);
  return hipGetLastError();
}

}  // namespace affmae
