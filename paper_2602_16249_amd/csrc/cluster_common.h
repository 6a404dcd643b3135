// Shared definitions of the cluster-tiled attention kernels (bf16, d = 32).
//
// Tokens are handled in tiles of 16 consecutive tokens ("token tiles"); a strip
// is the token tile seen as 16 queries.  Because clusters hold a multiple of 16
// tokens in cluster order, a token tile never straddles clusters.
//
// The plan (built by pla_plan.hip from the neighbour table) describes, per
// strip, which token tiles hold at least one neighbour of one of its queries
// ("slots", at most kMaxSlots) and, for every (query, token) pair of a strip and a
// slot, where the token stands in the query's neighbour list (see PlanLayout).
#pragma once

#include "device_util.h"

namespace affmae {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;  // 16 bytes on their way through registers

constexpr int kD = 32;                 // channels per head
constexpr int kMaxSlots = 64;          // token tiles one strip may touch (M*S/16 <= 64)
constexpr int kMaxEntries = 16;        // 16 queries * K (<= 64) neighbours / 64 lanes

union Frag8 {
  bf16x8 v;
  uint4 u4;
  u32x4 x4;
  uint2 u2[2];
  uint32_t u[4];
  uint16_t h[8];
};

union Frag4 {
  s16x4 v;
  uint2 u2;
  uint32_t u[2];
  uint16_t h[4];
};

// Strips are taken in groups of kGroup consecutive ones of an image: the strips of a group touch mostly the same token
// tiles (14.7 different ones per group on a jittered grid where each strip touches 8.6; 18.9 and 12.1 in clumps), so one
// workgroup fetches the union once and each of its waves serves one strip from LDS.
constexpr int kGroup = 4;
static_assert(kGroup * kMaxSlots <= 256, "places in a group's union are bytes");

// Layout of the plan buffer.
//  uni     per group: how many token tiles its strips touch together, then these tiles, ascending.
//  pos     per strip: how many of them it touches itself (its "slots", ascending), then each slot's place in the union.
//  jt      per strip and slot, for every (query, token) of the 16 x 16 pairs, where the token stands in the query's
//          neighbour list: one byte, 2 j, or 2 K for "no neighbour".  It is at the same time the byte offset of the
//          pair's value in a row of K two-byte values with one more place behind them.  Two slots share a block of
//          512 bytes, lane (g, q) = 16 g + q of a wave finding its four bytes for tokens 4g..4g+3 of query q at
//          8 (16 g + q) for the first and 4 further on for the second: one 8-byte load serves a pair of slots.
//  touch   per strip: how many groups of token tiles it touches, then per such group the group's number (high half)
//          and the strip's slots of the group's four tiles (one byte each in the low half, 0xff: not touched).
//  rev     the same seen from the tiles: per group of token tiles the strips that touch it, ascending (the sums
//          formed along the list then do not depend on scheduling): strip (high half), slots of the four tiles.
// Bytes written per strip: 256 per slot (8 to 12 of them as a rule) against 32 K for a list of the pairs' cells, twice; in
// exchange no kernel sorts pairs or scatters values over a tile.  Room is kept for every slot that there may be.
struct PlanLayout {
  int strips;            // B * strips_per_image (also the number of token tiles)
  int strips_per_image;  // ceil(N / 16)
  int groups_per_image, groups;
  int max_slots;         // at most M * S / 16
  int K;
  int uni_stride;        // uint16 per group
  int pos_stride;        // uint8 per strip
  int jt_pairs;          // pairs of slots per strip
  int touch_stride;      // uint64 per strip
  size_t uni_off, pos_off, jt_off, touch_off;
  size_t rev_count_off;   // int32  [groups]
  size_t rev_offset_off;  // int32  [groups + 1]  where a group's list starts in rev_list
  size_t rev_cursor_off;  // int32  [groups]      build-time cursors
  size_t rev_list_off;    // uint64 [strips * (touch_stride - 1)]
  size_t total;
};

inline size_t plan_align(size_t n) { return (n + 255) / 256 * 256; }

inline PlanLayout make_plan_layout(int B, int N, int K, int S, int M) {
  PlanLayout L;
  L.strips_per_image = (N + 15) / 16;  // the last strip / token tile of an image may be short
  L.strips = (int)((long long)B * L.strips_per_image);
  L.groups_per_image = (L.strips_per_image + kGroup - 1) / kGroup;
  L.groups = B * L.groups_per_image;
  // a strip touches no more token tiles than its near clusters have, than the image has, and than it has neighbours
  L.max_slots = (int)((long long)M * S / 16);
  if (L.max_slots > L.strips_per_image) L.max_slots = L.strips_per_image;
  if (L.max_slots > 16 * K) L.max_slots = 16 * K;
  L.K = K;
  const int most = kGroup * L.max_slots < L.strips_per_image ? kGroup * L.max_slots : L.strips_per_image;
  L.uni_stride = (1 + most + 1) / 2 * 2;
  L.pos_stride = (1 + L.max_slots + 3) / 4 * 4;
  L.jt_pairs = (L.max_slots + 1) / 2;
  L.touch_stride = 1 + (L.max_slots < L.groups_per_image ? L.max_slots : L.groups_per_image);
  size_t off = 0;
  L.uni_off = off;
  off += plan_align((size_t)L.groups * L.uni_stride * sizeof(uint16_t));
  L.pos_off = off;
  off += plan_align((size_t)L.strips * L.pos_stride);
  L.jt_off = off;
  off += plan_align((size_t)L.strips * L.jt_pairs * 512);
  L.touch_off = off;
  off += plan_align((size_t)L.strips * L.touch_stride * sizeof(uint64_t));
  L.rev_count_off = off;
  off += plan_align((size_t)L.groups * sizeof(int32_t));
  L.rev_offset_off = off;
  off += plan_align(((size_t)L.groups + 1) * sizeof(int32_t));
  L.rev_cursor_off = off;
  off += plan_align((size_t)L.groups * sizeof(int32_t));
  L.rev_list_off = off;
  off += plan_align((size_t)L.strips * (L.touch_stride - 1) * sizeof(uint64_t));
  L.total = off;
  return L;
}

// A row of K two-byte values and the place behind them that "no neighbour" points to, an odd number of words: the places
// of "no neighbour" of the 16 rows, which most lanes read, lie in 16 banks (in one, with K = 62 and rows of 32 words, the
// forward kernel took 66 us against 45 at K = 64; B = 8, N = 4096, H = 8).
__host__ __device__ __forceinline__ int row_halves(int K) { return ((K / 2 + 1) | 1) * 2; }

// A launch has at most 2^32 - 1 threads: larger ones are cut into slices of workgroups of 256 (a multiple of 8 each).
constexpr long long kMaxBlocks = (1ll << 24) - 8;

// Division of a non-negative int by a small run-time constant through a 32-bit reciprocal (exact for the
// ranges used here: n * d < 2^31).  The reciprocal of 1 does not fit 32 bits: magic 0 stands for it.
__device__ __forceinline__ int fast_div(int n, uint32_t magic) {
  // (a sum, not a choice between the two: the choice on a uniform magic becomes a branch at every use)
  return (int)(__umulhi((uint32_t)n, magic) + (magic == 0u ? (uint32_t)n : 0u));
}
inline uint32_t div_magic(int d) { return d <= 1 ? 0u : (uint32_t)((1ull << 32) / (uint32_t)d) + 1u; }
// The same for any non-negative n and d >= 1: the reciprocal is rounded up, so the quotient it gives is at most
// one too large; one multiplication checks it.  (The compiler's own division by a run-time value is a chain of
// ~30 dependent instructions through the reciprocal unit, at the head of every wave.)
__device__ __forceinline__ int exact_div(int n, int d, uint32_t magic) {
  const uint32_t q = __umulhi((uint32_t)n, magic) + (magic == 0u ? (uint32_t)n : 0u);
  return (int)(q - (q * (uint32_t)d > (uint32_t)n ? 1u : 0u));
}

// Workgroups are dealt round-robin to the 8 XCDs (one L2 each); where neighbouring ones share what they read or write,
// give every XCD a contiguous range.  The grid is a multiple of 8.
__device__ __forceinline__ int xcd_contiguous_block(unsigned block, unsigned blocks) {
  const int per_xcd = blocks >> 3;
  return (block & 7) * per_xcd + (block >> 3);
}

__device__ __forceinline__ uint32_t wave_or32(uint32_t x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x |= __shfl_xor(x, o);
  return x;
}

// Reductions over the four lanes that hold one query's values (lanes r, r+16, r+32, r+48), on the
// VALU lane-swap instructions of gfx950: no trip through the LDS crossbar.
typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
__device__ __forceinline__ float group_max(float x) {
  u32x2 a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float m = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  u32x2 b = __builtin_amdgcn_permlane16_swap(__float_as_uint(m), __float_as_uint(m), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float group_sum(float x) {
  u32x2 a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float m = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  u32x2 b = __builtin_amdgcn_permlane16_swap(__float_as_uint(m), __float_as_uint(m), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Place, in 16-byte pieces, of piece `piece` (0..3) of row `row` (0..15) in a 1 KB LDS tile of 16 rows
// of 64 bytes.  The XOR spreads both access patterns of the kernels over the banks: lane (row lane/4, piece
// lane%4) writes (13.6 cycles per access whatever the XOR), lane (row lane%16, piece lane/16) reads (5.6 cycles
// with this XOR, 8.2 without).
__device__ __forceinline__ int tile_chunk(int row, int piece) {
  return row * 4 + (piece ^ ((row >> 1) & 3));
}

// ds_read_b64_tr_b16: inside a group of 16 lanes, lanes 4j..4j+3 address the four 8-byte quarters of a row j of
// 16 bf16 values (j = 0..3), and lane i of the group receives element i of rows 0..3: a 4 x 16 block read by
// columns.  With rows = tokens and columns = channels this is the transposed operand of an MFMA.
__device__ __forceinline__ uint2 lds_read_tr(const void* p) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  const s16x4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p);
  return __builtin_bit_cast(uint2, r);
}

// Byte offset, inside a staged 16 x 32 tile (layout of tile_chunk), that lane (r = lane % 16, g = lane / 16) gives
// to lds_read_tr to receive, for channel 16 dt + r, the values of rows 4g..4g+3: it addresses the quarter r % 4 of
// the 16 channels of row 4g + r / 4.
__device__ __forceinline__ int tile_tr_offset(int g, int r, int dt) {
  return tile_chunk(4 * g + (r >> 2), 2 * dt + ((r & 3) >> 1)) * 16 + (r & 1) * 8;
}

// Two fp32 -> packed bf16 (round to nearest even), low half first.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  typedef __attribute__((ext_vector_type(2))) float f32x2;
  f32x2 f = {lo, hi};
  bf16x2 b = __builtin_convertvector(f, bf16x2);
  return __builtin_bit_cast(uint32_t, b);
}

}  // namespace affmae
