// What the forward and the query-stationary backward kernel share: a workgroup of four waves serves a group of four
// strips for one head; the union of the token tiles that the strips touch is fetched into LDS once, straight from
// memory, and every wave walks the tiles of its own strip there.
//
// Before, every (strip, head) wave fetched its tiles itself, a pair at a time, through registers: a row crossed L1 and
// LDS 8.6 times where 3.7 are needed, and a strip of five pairs waited for memory five times in a row.  Clocked inside
// the kernels, such a chain, not a unit of the chip, was most of a wave's life.  Now everything that a strip needs is
// requested at its start: the tiles, its bias rows, its q rows and the j words of all its slots.
#pragma once

#include "cluster_common.h"
#include "launch.h"

#include <type_traits>

namespace affmae {

constexpr int kSpare = 8;   // tiles beyond the places in LDS whose rows wait in registers, two per wave
constexpr int kPairs = 12;  // pairs of slots whose j words are held in registers

struct GroupTables {
  const uint16_t* uni;
  const uint8_t* pos;
  const char* jt;
  int N, H, strips_per_image, groups_per_image, groups, uni_stride, pos_stride;
  uint32_t h_magic, gpi_magic;  // reciprocals of H and of groups_per_image
  // products that the kernels would form again and again (each below 2^32: see pla_cluster_supported)
  uint32_t row_bytes;  // of a token in q, k, v, out: all heads
  uint32_t img_bytes;  // ... of an image
  uint32_t img_pairs;  // N * H * K, values of an image in bias, dbias
  uint32_t jt_bytes;   // of a strip in the j table
};
// 64-bit product of 32-bit values: two scalar instructions instead of the eight of a 64-bit product
__device__ __forceinline__ size_t mul_u32(uint32_t a, uint32_t b) { return (size_t)a * b; }

// Values that a lane moves at a time between the bias (or dbias) rows in memory and those in LDS: 16 bytes where every row
// of K values starts at a multiple of them, else 4, else one value.
inline int bias_item(int K, const void* bias, const void* dbias) {
  const uintptr_t at = reinterpret_cast<uintptr_t>(bias) | reinterpret_cast<uintptr_t>(dbias);
  return K % 8 == 0 && at % 16 == 0 ? 8 : K % 2 == 0 && at % 4 == 0 ? 2 : 1;
}

// Bias from a relative-position table (REL of the kernels): kRelCells, the cells of the pairs come from memory, written by
// a kernel of their own; kRelDirect, every (strip, head) works its own out from the coordinates.
enum { kNoRel = 0, kRelCells = 1, kRelDirect = 2 };
struct RelSource {
  const bf16_t* table;    // [H][ncells]
  int ncells;
  const uint16_t* cells;  // [B,N,K] (kRelCells)
  const float2* coords;   // [B,N], nbr [B,N,K] (kRelDirect)
  const int32_t* nbr;
  float rate;
  int R;
};
// Calls of few heads, or of up to this many (token, head, neighbour) triples, work their cells out directly: two launches
// less in a step.  us forward + backward, cells from memory / directly: 47 / 41 up to 1 M triples, 90.2 / 85.5 at 6.3 M; with
// eight heads (the cells of a pair are worked out 8 times, and 24 bytes are gathered for 2 bytes read) 113 / 116 at 12.6 M, 220 /
// 232 at 25 M.  With few heads the cells' own kernel costs more at every size, R = 3 (R = 7 alike): one head 3 / 13 / 38 M
// 56 / 147 / 444 and 47 / 126 / 393, two heads 6 / 13 / 25 / 50 M 77 / 126 / 283 / 547 and 71 / 119 / 265 / 533; three heads
// 9 / 19 / 38 M 96 / 174 / 386 and 93 / 171 / 385, four heads 13 / 25 / 50 M 116 / 235 / 494 and 116 / 237 / 504.
constexpr int kRelDirectHeads = 3;
constexpr long long kRelDirectTriples = 10ll << 20;

inline GroupTables group_tables(const PlanLayout& L, const void* plan, int N, int H, int K) {
  const char* base = static_cast<const char*>(plan);
  GroupTables t;
  t.uni = reinterpret_cast<const uint16_t*>(base + L.uni_off);
  t.pos = reinterpret_cast<const uint8_t*>(base + L.pos_off);
  t.jt = base + L.jt_off;
  t.N = N; t.H = H;
  t.strips_per_image = L.strips_per_image; t.groups_per_image = L.groups_per_image; t.groups = L.groups;
  t.uni_stride = L.uni_stride; t.pos_stride = L.pos_stride;
  t.row_bytes = (uint32_t)H * kD * 2u; t.img_bytes = (uint32_t)N * t.row_bytes;
  t.img_pairs = (uint32_t)((long long)N * H * K); t.jt_bytes = (uint32_t)L.jt_pairs * 512u;
  t.h_magic = div_magic(H); t.gpi_magic = div_magic(L.groups_per_image);
  return t;
}

__device__ __forceinline__ f32x4 mfma32(const Frag8& a, const Frag8& b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b.v, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma16(const Frag4& a, const Frag4& b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a.v, b.v, c, 0, 0, 0);
}

// (see xcd_contiguous_block(block, blocks): neighbouring groups share rows)
__device__ __forceinline__ int xcd_contiguous_block() { return xcd_contiguous_block(blockIdx.x, gridDim.x); }

// The wave's strip, and the tiles of its group.  PL: places for tiles in LDS, RAG: N is not a multiple of 16 (only then
// do the row clamps exist in the code).
template <int PL, bool RAG>
struct TileWalk {
  const GroupTables& t;
  int lane, wave, g, r;  // lane = 16 g + r
  int gi, h, b, sg, q0, nq;
  bool live;  // the image's last group may have fewer than four strips
  uint32_t row_bytes;  // of a token, all heads
  size_t img_off;      // bytes before the image in q, k, v, out, ...
  const uint16_t* ul;
  const uint8_t* pl;
  const char* jt;
  const char *kimg, *vimg;
  char* tiles;  // PL x 2 KB: K rows, V rows of a tile, 16-byte pieces placed by tile_chunk
  int U, cnt;   // tiles of the union; the strip's slots
  int my_tile, my_pos, u_raw, cnt_raw;
  uint32_t lane_off, lane_off_max, tile_bytes;
  uint2 jw[kPairs];
  u32x4 sk[kSpare / kGroup], sv[kSpare / kGroup];

  __device__ __forceinline__ TileWalk(const GroupTables& tables, int gi_, int h_, char* lds_tiles) : t(tables), gi(gi_), h(h_), tiles(lds_tiles) {
    lane = threadIdx.x & (kWave - 1);
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);  // uniform: keeps per-wave indices in SGPRs
    g = lane >> 4;
    r = lane & 15;
    b = exact_div(gi, t.groups_per_image, t.gpi_magic);
    const int si_raw = (gi - b * t.groups_per_image) * kGroup + wave;
    live = si_raw < t.strips_per_image;
    const int si = min(si_raw, t.strips_per_image - 1);
    sg = b * t.strips_per_image + si;
    q0 = si * 16;
    // An image's last strip and last token tile may be short (N % 16 != 0): rows past the end are never addressed -
    // loads repeat the last real row (no pair refers to it, so it meets probability 0), stores are skipped.
    nq = RAG ? min(16, t.N - q0) : 16;
    row_bytes = t.row_bytes;
    img_off = mul_u32(b, t.img_bytes);
    ul = t.uni + mul_u32(gi, t.uni_stride) + 1;
    pl = t.pos + mul_u32(sg, t.pos_stride) + 1;
    jt = t.jt + mul_u32(sg, t.jt_bytes);
    u_raw = (int)ul[-1];
    cnt_raw = (int)pl[-1];
    my_tile = (int)ul[(uint32_t)min(lane, t.uni_stride - 2)];
    my_pos = (int)pl[(uint32_t)min(lane, t.pos_stride - 2)];
  }
  // first value of the strip's rows in [B,N,H,K] (the head's for `head`), in [B,N,H] and in [B,N,K] arrays
  __device__ __forceinline__ size_t pairs0(int K, int head) const { return mul_u32(b, t.img_pairs) + ((uint32_t)q0 * t.H + head) * K; }
  __device__ __forceinline__ size_t heads0() const { return mul_u32(b, (uint32_t)(t.N * t.H)) + (uint32_t)(q0 * t.H + h); }
  __device__ __forceinline__ size_t slots0(int K) const { return mul_u32(b, (uint32_t)(t.N * K)) + (uint32_t)(q0 * K); }
  // byte offset, within the image, of 16-byte piece `piece` of the head's row of query `q` of the strip
  __device__ __forceinline__ uint32_t query_piece(int q, int piece) const {
    return (uint32_t)(q0 + (RAG ? min(q, nq - 1) : q)) * row_bytes + (uint32_t)(h * kD * 2 + piece * 16);
  }
  __device__ __forceinline__ uint32_t tile_off(int tile) const {
    const uint32_t off = lane_off + (uint32_t)tile * tile_bytes;
    return RAG ? min(off, lane_off_max) : off;
  }
  // K and V rows of a tile straight into a place (16 bytes per lane, lane l's piece landing at 16 l, i.e. row l / 4,
  // place l % 4: the lane fetches the piece whose place that is)
  __device__ __forceinline__ void issue(int tile, int place) const {
    typedef const __attribute__((address_space(1))) void* gptr_t;
    typedef __attribute__((address_space(3))) void* lptr_t;
    const uint32_t off = tile_off(tile);
    char* dst = tiles + place * 2048;
    __builtin_amdgcn_global_load_lds((gptr_t)(kimg + off), (lptr_t)dst, 16, 0, 0);
    __builtin_amdgcn_global_load_lds((gptr_t)(vimg + off), (lptr_t)(dst + 1024), 16, 0, 0);
  }
  // everything that depends on the group's and the strip's own records
  __device__ __forceinline__ void request(const void* k, const void* v) {
    U = __builtin_amdgcn_readfirstlane(u_raw);
    cnt = min(__builtin_amdgcn_readfirstlane(cnt_raw), live ? kMaxSlots : 0);
    // the second half of an odd strip's last pair meets "no neighbour", on the rows of a tile that is there
    const int last_pos = __builtin_amdgcn_readlane(my_pos, max(cnt - 1, 0));
    my_pos = lane < cnt ? my_pos : last_pos;
    kimg = static_cast<const char*>(k) + img_off;
    vimg = static_cast<const char*>(v) + img_off;
    const int la = lane >> 2, lc = lane & 3;
    const uint32_t piece = (uint32_t)((lc ^ ((la >> 1) & 3)) * 16 + h * kD * 2);
    lane_off = (uint32_t)la * row_bytes + piece;
    lane_off_max = (uint32_t)(t.N - 1) * row_bytes + piece;
    tile_bytes = 16u * row_bytes;
#pragma unroll
    for (int i = 0; i < (PL + kGroup - 1) / kGroup; ++i)
      if (i * kGroup + wave < min(U, PL)) issue(__builtin_amdgcn_readlane(my_tile, i * kGroup + wave), i * kGroup + wave);
    // j words of the strip's pairs, two pairs a test (the second repeats the last pair where the strip ends before it)
    const int last_pair = (max(cnt, 1) - 1) >> 1;
#pragma unroll
    for (int i = 0; i < kPairs; ++i) {
      if (i & 1) asm volatile("" : "=v"(jw[i].x), "=v"(jw[i].y));  // any value where no slot is: no instruction
      else jw[i] = make_uint2(0u, 0u);  // the pair behind the last may be fetched: bytes as they come are odd addresses, and slow
      if (2 * (i & ~1) < cnt) jw[i] = *reinterpret_cast<const uint2*>(jt + (uint32_t)(((i & 1) ? min(i, last_pair) : i) * 512 + lane * 8));
    }
#pragma unroll
    for (int i = 0; i < kSpare / kGroup; ++i)
      if (PL + i * kGroup + wave < U) {
        const uint32_t off = tile_off(__builtin_amdgcn_readlane(my_tile, PL + i * kGroup + wave));
        sk[i] = *reinterpret_cast<const u32x4*>(kimg + off);
        sv[i] = *reinterpret_cast<const u32x4*>(vimg + off);
      }
  }
  // All requested rows are in LDS, and so is what the other waves wrote there.
  __device__ __forceinline__ void arrive() const {
    __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0): rows on their way to LDS count as vector loads
    __syncthreads();
  }
  // Up to P pairs, from the a-th on, of the slots below `end`.
  template <int P, class Frag, class Fetch, class Math>
  __device__ __forceinline__ void pairs(std::integral_constant<int, P>, Frag (&f)[2], int a, int end, int at, Fetch& fetch, Math& math) {
    fetch(f[0], jw[0].x, jw[0].y, __builtin_amdgcn_readlane(at, 2 * a), __builtin_amdgcn_readlane(at, 2 * a + 1));
#pragma unroll
    for (int i = 0; i < P; ++i) {
      if (2 * (a + i) >= end) break;
      if (i + 1 < P)
        fetch(f[(i + 1) & 1], jw[i + 1].x, jw[i + 1].y, __builtin_amdgcn_readlane(at, 2 * (a + i) + 2), __builtin_amdgcn_readlane(at, 2 * (a + i) + 3));
      __builtin_amdgcn_sched_barrier(0);
      math(f[i & 1], i < 2);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // The strip's slots by pairs.  fetch(frag, w0, w1, at0, at1) reads from LDS what a pair needs (j words w, tiles at byte
  // offsets at), math(frag, early) uses it (early: among the first pairs, see the forward kernel).  The next pair is fetched
  // before the present one's math: the compiler does not move loads over the branch between pairs by itself.
  // Unions of more than PL tiles go in stages: the first, of a pair or two as a rule, frees places for the tiles that wait in
  // registers; the rest is walked like a union that fits, the j words of the pairs that are done shifted out of the way.
  // (With every pair of both stages fetched only when the one before was done, the forward kernel was slower than with tiles
  // fetched per strip wherever unions are large and shared little: masked grids by up to 7 %, S = 16 by up to 16 %.  us, B6
  // N4096 H8 S16: K32 M8 20.9 -> 20.3, K64 M10 27.2 -> 26.0; B8 N16384 H4 K64 M10 blobs 57.8 -> 55.2; B64 N1024 H8 K48 S32 M8
  // 61.7 -> 59.2; B16 N16384 H4 K48 S64 M8 blobs 147 -> 142; what fits is as fast as before.)  Unions of more than PL + kSpare
  // tiles go on in eights.
  // APART: unions that fit have a loop of their own, without the pairs that only others have (the forward kernel is 1 - 2 %
  // faster with it; the query-stationary one is not, and with a relative-position table it has no registers left for two).
  template <bool APART, class Frag, class Fetch, class Math>
  __device__ __forceinline__ void walk(int K, Fetch fetch, Math math) {
    static_assert(2 * kPairs >= PL + kSpare, "the j words of two stages' slots are in registers");
    static_assert(kSpare % kGroup == 0 && (kSpare & (kSpare - 1)) == 0 && kSpare <= PL, "");
    const uint32_t none = 2u * (uint32_t)K * 0x01010101u;
    int at = min(my_pos, PL - 1) * 2048;
    if (APART && U <= PL) {
      Frag f[2];
      pairs(std::integral_constant<int, (PL + 1) / 2>{}, f, 0, cnt, at, fetch, math);
      return;
    }
    int a = 0, end = cnt;  // first pair and last slot of the main part
    if (APART || U > PL) {
      const int done = (int)__popcll(__ballot(lane < cnt && my_pos < min(kSpare, U - PL)));  // slots of the places to be freed
#pragma unroll
      for (int i = 0; i < kSpare / 2; ++i) {
        if (2 * i >= done) break;
        Frag f;
        fetch(f, jw[i].x, 2 * i + 1 < done ? jw[i].y : none, __builtin_amdgcn_readlane(at, 2 * i),
              __builtin_amdgcn_readlane(at, min(2 * i + 1, done - 1)));
        __builtin_amdgcn_sched_barrier(0);
        math(f, true);
        __builtin_amdgcn_sched_barrier(0);
      }
      __syncthreads();  // every wave is through with these places
#pragma unroll
      for (int i = 0; i < kSpare / kGroup; ++i)
        if (PL + i * kGroup + wave < U) {
          char* dst = tiles + (i * kGroup + wave) * 2048;
          reinterpret_cast<u32x4*>(dst)[lane] = sk[i];
          reinterpret_cast<u32x4*>(dst + 1024)[lane] = sv[i];
        }
      __syncthreads();
      a = done >> 1;
#pragma unroll
      for (int step = kSpare / 2; step > 0; step >>= 1)
        if (a & step) {
#pragma unroll
          for (int i = 0; i < kPairs; ++i) jw[i] = i + step < kPairs ? jw[i + step] : make_uint2(0u, 0u);
        }
      if (done & 1) jw[0].x = none;  // (its tile's place holds another tile now, whose rows meet probability 0)
      end = (int)__popcll(__ballot(lane < cnt && my_pos < PL + kSpare));
      if (end < cnt && (end & 1)) {
#pragma unroll
        for (int i = 0; i < kPairs; ++i)
          if (2 * (a + i) + 1 == end) jw[i].y = none;
      }
      at = min(my_pos < PL ? my_pos : my_pos - PL, PL - 1) * 2048;
    }
    Frag f[2];
    pairs(std::integral_constant<int, kPairs>{}, f, a, end, at, fetch, math);
    if (U <= PL + kSpare) return;
    const int last_pair = (max(cnt, 1) - 1) >> 1;
    auto words = [&](int i) { return *reinterpret_cast<const uint2*>(jt + (uint32_t)(min(i, last_pair) * 512 + lane * 8)); };
    for (int lo = PL + kSpare; lo < U; lo += kSpare) {
      const int hi = min(U, lo + kSpare);
      const int s0 = end, s1 = (int)__popcll(__ballot(lane < cnt && my_pos < hi));
      end = s1;
      const int next = (int)ul[min(lo + (lane & (kSpare - 1)), U - 1)];
      int i = s0 >> 1;
      uint2 w = words(i);
      __syncthreads();  // every wave is through with the tiles below lo
#pragma unroll
      for (int t = 0; t < kSpare / kGroup; ++t)
        if (lo + t * kGroup + wave < U) issue(__builtin_amdgcn_readlane(next, t * kGroup + wave), t * kGroup + wave);
      arrive();
      at = min(max(my_pos - lo, 0), PL - 1) * 2048;
      for (; max(2 * i, s0) < s1; ++i) {
        const uint2 after = words(i + 1);
        fetch(f[0], 2 * i >= s0 ? w.x : none, 2 * i + 1 < s1 ? w.y : none, __builtin_amdgcn_readlane(at, max(2 * i, s0)),
              __builtin_amdgcn_readlane(at, min(2 * i + 1, s1 - 1)));
        __builtin_amdgcn_sched_barrier(0);
        math(f[0], false);
        w = after;
      }
    }
  }
};

// Eight neighbours of a query (an item of the kernels, K a multiple of 8) on their way to cells (kRelDirect).
struct RelItem {
  typedef int i32x4 __attribute__((ext_vector_type(4), aligned(4)));  // (the table need not lie at a multiple of 16 bytes)
  i32x4 n0, n1;
  float2 ci;
  template <class Walk>
  __device__ __forceinline__ void request(const RelSource& s, const Walk& w, int K, int qc, int j0) {
    const i32x4* src = reinterpret_cast<const i32x4*>(s.nbr + w.slots0(K) + (uint32_t)(qc * K + j0));
    n0 = src[0];
    n1 = src[1];
    ci = (s.coords + mul_u32(w.b, w.t.N))[(uint32_t)(w.q0 + qc)];
  }
  template <class Walk>
  __device__ __forceinline__ void cells(const RelSource& s, const Walk& w, uint32_t (&out)[4]) const {
    const float2* cimg = s.coords + mul_u32(w.b, w.t.N);
    const int nn[8] = {n0.x, n0.y, n0.z, n0.w, n1.x, n1.y, n1.z, n1.w};
    float2 cn[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) cn[e] = cimg[(uint32_t)min(max(nn[e], 0), w.t.N - 1)];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      out[e] = (uint32_t)relpos_cell(cn[2 * e], ci, s.rate, s.R) | ((uint32_t)relpos_cell(cn[2 * e + 1], ci, s.rate, s.R) << 16);
  }
};
inline RelSource rel_source(const PlaArgs& a) {
  RelSource s;
  s.table = (const bf16_t*)a.rel_table;
  s.ncells = (2 * a.rel_R + 1) * (2 * a.rel_R + 1);
  s.cells = a.rel_cells;
  s.coords = (const float2*)a.rel_coords;
  s.nbr = a.nbr_idx;
  s.rate = a.rel_rate;
  s.R = a.rel_R;
  return s;
}

// Straight from memory into LDS (lane l's bytes land at dst + 16 l, or + 4 l).  By hand: for the compiler every LDS read might
// read what such a load still writes, and it would wait for what is on its way before it reads what is there.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"  // (m0 is reserved: written only for the next instruction, never held)
__device__ __forceinline__ void lds_load16(uint32_t dst, const char* base, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(off), "s"(base) : "m0", "memory");
}
__device__ __forceinline__ void lds_load4(uint32_t dst, const char* base, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(dst), "v"(off), "s"(base) : "m0", "memory");
}
#pragma clang diagnostic pop
__device__ __forceinline__ uint32_t lds_address(const void* p) { return (uint32_t)(size_t)(__attribute__((address_space(3))) const char*)p; }

// dk_blank, dv_blank [H,D] = sums over the strips of part [strips][H][2][D], in a fixed order: D / 8 workgroups per (head, which of the
// two), the i-th of them all, 8 channels each, 32 groups of 8 lanes; group j adds strips j, j + 32, ..., eight loads in flight (one at a
// time the few workgroups waited for one memory round trip per strip: 7.5 us at 753 strips).  `lds`: 256 words.
template <int D>
__device__ __forceinline__ void blank_sums(const float* part, int strips, int H, int i, float* lds, float* dk_blank, float* dv_blank) {
  constexpr int kParts = D / 8;
  const int which = (i / kParts) & 1, h = i / (2 * kParts);
  const int c = i % kParts * 8 + (threadIdx.x & 7), grp = threadIdx.x >> 3;
  float s = 0.f;
  for (int sg0 = grp; sg0 < strips; sg0 += 8 * 32) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int sg = sg0 + 32 * u;
      v[u] = part[(((size_t)min(sg, strips - 1) * H + h) * 2 + which) * D + c];
      if (sg >= strips) v[u] = 0.f;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) s += v[u];
  }
  lds[threadIdx.x] = s;
  __syncthreads();
  if (grp == 0) {
    float t = 0.f;
    for (int j = 0; j < 32; ++j) t += lds[j * 8 + threadIdx.x];
    (which ? dv_blank : dk_blank)[h * D + c] = t;
  }
}

}  // namespace affmae
