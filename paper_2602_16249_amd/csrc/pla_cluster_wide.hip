// Cluster-tiled local attention where the probabilities and their products stay fp32: fp32 storage (head sizes 16, 32,
// 64) and bf16 storage with head sizes 16 and 64, on a cached plan (paper, Sec. "Flash-style Cluster Attention and Fast
// Decoder KNN": stream over tiles, never store the scores; the equation is FlashNbhdAttn).  Same preconditions as the
// kernels for bf16 and d = 32 (pla_cluster_fwd.hip, pla_cluster_bwd.hip), whose shape they share: a workgroup of four waves
// per (group of four strips, head), the union of the strips' token tiles in LDS, scores transposed, every pair's
// bias, p or dS found through its j byte; backward by a query-stationary and a key-stationary kernel, rows of p handed over.
// What differs: all products are v_mfma_f32_16x16x4_f32 on fp32 operands, so nothing that the gather kernels hold in 32
// bits is rounded; the union goes through LDS in stages, the next stage's tiles on their way while one is used.
//
// Bound by the matrix instructions (32 cycles each: 2, 3 and 3 times d / 4 of them per pair of strip and tile) and, with few
// workgroups, the chain at their start.  16384 tokens in 4 images, K = 48, two heads of 32 fp32 channels, us, gather kernels /
// here: forward 29 / 30 (14 tiles a strip; 9, on a grid without a mask: 28 / 16), query side 39 / 38, lists
// and key side 53 / 29.
#include "cluster_tiles.h"
#include "launch.h"
#include "timing.h"

#include <algorithm>

namespace affmae {
namespace {

template <typename T, int D>
struct WideRows {
  static constexpr int E = sizeof(T), RB = D * E, PCS = RB / 16;  // bytes and 16-byte pieces of a row
  static constexpr int TB = 16 * RB;                              // bytes of a tile's rows
  static constexpr int NI = (TB + 1023) / 1024;                   // loads into LDS of 64 x 16 bytes
  static constexpr int U = D / 16;                                // a lane's pieces of four channels: 16 u + 4 g ..
  static constexpr int kRowsPer256 = 256 / RB;
  // Piece `piece` of row `row` lies at place piece ^ swizzle(row): rows that share banks have different ones, so that 16 rows
  // are read at one piece, and 16 channels of 4 rows, with as few conflicts as their banks allow.
  static __device__ __forceinline__ int swizzle(int row) { return (row / kRowsPer256) & (PCS - 1); }
  static __device__ __forceinline__ int offset(int row, int ch) {
    const int byte = ch * E;
    return row * RB + (((byte >> 4) ^ swizzle(row)) << 4) + (byte & 15);
  }
  static __device__ __forceinline__ float one(const char* p) {
    if constexpr (E == 4) return *reinterpret_cast<const float*>(p);
    else return bf16_to_f32(*reinterpret_cast<const bf16_t*>(p));
  }
  static __device__ __forceinline__ void put_four(T* p, const f32x4& x) {
    if constexpr (E == 4) *reinterpret_cast<f32x4*>(p) = x;
    else *reinterpret_cast<u32x2*>(p) = u32x2{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3])};
  }
};

// exp(x) within a unit and a half of the last place, in 8 instructions against 13 of the library's (which take as long here as the products
// that they follow).  Cody and Waite's reduction with the constant in two parts: log2 e = kL + kLow, kL its nearest fp32 value; x
// log2 e = n + f, f rounded once and corrected by the rest, 2^f by the hardware, n into the exponent.  Below -104 the
// result is 0, so x is kept above -150: -inf would leave infinity minus infinity.
__device__ __forceinline__ float wide_exp(float x) {
  constexpr float kL = 1.44269504f, kLow = 1.92596299e-8f;  // log2 e = 1.442695040888963 = 1.44269502162933 + 0.00000001925963
  x = x < -150.f ? -150.f : x;  // (not a maximum: NaN stays NaN)
  const float n = __builtin_rintf(x * kL);
  const float f = fmaf(x, kLow, fmaf(x, kL, -n));
  return __builtin_ldexpf(__builtin_amdgcn_exp2f(f), (int)n);
}

// A row of K fp32 values, the place that "no neighbour" points to and one that nobody reads; an odd number of words.
__host__ __device__ __forceinline__ int wide_row(int K) { return (K + 2) | 1; }
constexpr int kMostWideRow = 67;
constexpr uint32_t kNotHeld = 0x7fc05a5au;  // a NaN that no arithmetic here makes

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// Four channels of a row as stored, and sums of products of two of them over the four lanes of a row and query: bf16 values go as
// they are (their products are exact in the bf16 instruction, its sums fp32; an eighth of the time).
template <typename T>
struct Four;
template <>
struct Four<float> {
  f32x4 x;
  __device__ __forceinline__ void load(const void* p) { x = *static_cast<const f32x4*>(p); }
  __device__ __forceinline__ f32x4 values() const { return x; }
};
template <>
struct Four<bf16_t> {
  Frag4 x;
  __device__ __forceinline__ void load(const void* p) { x.u2 = *static_cast<const uint2*>(p); }
  __device__ __forceinline__ f32x4 values() const {
    return f32x4{__uint_as_float(x.u[0] << 16), __uint_as_float(x.u[0] & 0xffff0000u), __uint_as_float(x.u[1] << 16), __uint_as_float(x.u[1] & 0xffff0000u)};
  }
};
// Dot products of N rows with the queries' (d channels; from c on).  fp32: four sums (eight with d = 64), added by pairs at the
// end, so that as few roundings lie one behind the other as where lanes add their parts up (with one sum the results were 1.4
// times as far from 64 bits).
template <int U, int N>
__device__ __forceinline__ void dots(const Four<float> (&a)[N][U], const Four<float> (&b)[U], f32x4 (&c)[N]) {
  constexpr int P = U < 4 ? 1 : 2;
  f32x4 part[N][P][4];
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int n = 0; n < N; ++n)
        part[n][u % P][e] = mfma4(a[n][u].x[e], b[u].x[e], u >= P ? part[n][u % P][e] : u + e ? f32x4{0.f, 0.f, 0.f, 0.f} : c[n]);
#pragma unroll
  for (int n = 0; n < N; ++n) {
    c[n] = (part[n][0][0] + part[n][0][1]) + (part[n][0][2] + part[n][0][3]);
    if constexpr (P == 2) c[n] += (part[n][1][0] + part[n][1][1]) + (part[n][1][2] + part[n][1][3]);
  }
}
template <int U, int N>
__device__ __forceinline__ void dots(const Four<bf16_t> (&a)[N][U], const Four<bf16_t> (&b)[U], f32x4 (&c)[N]) {
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int n = 0; n < N; ++n) c[n] = mfma16(a[n][u].x, b[u].x, c[n]);
}
// Sums over tokens (or queries) by A chains, for the same reason; total() adds them up.
template <int A, int U>
struct Chains {
  f32x4 a[A][U];
  __device__ __forceinline__ Chains() {
#pragma unroll
    for (int i = 0; i < A; ++i)
#pragma unroll
      for (int u = 0; u < U; ++u) a[i][u] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  __device__ __forceinline__ void total(f32x4 (&t)[U]) const {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if constexpr (A == 8) t[u] = ((a[0][u] + a[1][u]) + (a[2][u] + a[3][u])) + ((a[4][u] + a[5][u]) + (a[6][u] + a[7][u]));
      else if constexpr (A == 2) t[u] = a[0][u] + a[1][u];
      else if constexpr (A == 4) t[u] = (a[0][u] + a[1][u]) + (a[2][u] + a[3][u]);
      else t[u] = a[0][u];
    }
  }
};
// (bf16 results are rounded far above that: one chain)
template <typename T, int D>
constexpr int chains() { return sizeof(T) == 2 ? 1 : D <= 32 ? 8 : 4; }

// every load into LDS has landed, in every wave
__device__ __forceinline__ void lds_loads_arrive() {
  __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0): rows on their way to LDS count as vector loads
  __syncthreads();
}

struct WideParams {
  GroupTables t;
  const void *q, *k, *v, *bias, *k_blank, *v_blank, *out, *dout;
  const float* lse_in;
  int K, block0;
  uint32_t k_magic;
  float scale;
  void *o, *dq, *dk, *dv, *dbias;
  float* lse;
  char* hand;         // workspace [strips][H]: rows of p [16][wide_row], then -D [16]
  int block_bytes;
  float* blank_part;  // workspace [strips][H][2][D]: the strip's parts of dk_blank, dv_blank; or nullptr
  const int32_t *rev_offset, *rev_count;
  const unsigned long long* rev_list;
  int front, blank_blocks, strips;  // as in BwdParams (pla_cluster_bwd.hip): workgroups in front that add the parts up
  float *dk_blank, *dv_blank;
};

// The wave's strip and the tiles of its group.
template <typename T, int D, bool RAG>
struct WideStrip {
  typedef WideRows<T, D> R;
  int lane, wave, g, r, h, b, q0, nq, U, cnt;
  bool live;
  uint32_t sg;
  size_t img_off;
  const uint16_t* ul;
  const char* jt;
  int my_pos;
  __device__ __forceinline__ WideStrip(const GroupTables& t, int gi, int head) : h(head) {
    lane = threadIdx.x & (kWave - 1);
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    g = lane >> 4;
    r = lane & 15;
    b = exact_div(gi, t.groups_per_image, t.gpi_magic);
    const int si_raw = (gi - b * t.groups_per_image) * kGroup + wave;
    live = si_raw < t.strips_per_image;  // the image's last group may have fewer than four strips
    const int si = min(si_raw, t.strips_per_image - 1);
    sg = (uint32_t)(b * t.strips_per_image + si);
    q0 = si * 16;
    nq = RAG ? min(16, t.N - q0) : 16;  // rows past a short last strip repeat the last one, stores past it are skipped
    img_off = mul_u32(b, t.img_bytes);
    ul = t.uni + mul_u32(gi, t.uni_stride) + 1;
    const uint8_t* pl = t.pos + mul_u32(sg, t.pos_stride) + 1;
    jt = t.jt + mul_u32(sg, t.jt_bytes);
    my_pos = (int)pl[(uint32_t)min(lane, t.pos_stride - 2)];
    U = __builtin_amdgcn_readfirstlane((int)ul[-1]);
    cnt = min(__builtin_amdgcn_readfirstlane((int)pl[-1]), live ? kMaxSlots : 0);
  }
  __device__ __forceinline__ int query(int q) const { return q0 + (RAG ? min(q, nq - 1) : q); }
  // channels 16 u + 4 g .. + 3 of the head's row of query r, as the B operand of the products with K or V rows
  __device__ __forceinline__ void query_row(const GroupTables& t, const void* x, Four<T> (&f)[R::U]) const {
    const char* row = static_cast<const char*>(x) + img_off + ((uint32_t)query(r) * t.row_bytes + (uint32_t)(h * R::RB));
#pragma unroll
    for (int u = 0; u < R::U; ++u) f[u].load(row + (16 * u + 4 * g) * R::E);
  }
  // first value of the strip in [B,N,H,K] and [B,N,H] arrays
  __device__ __forceinline__ size_t pairs0(const GroupTables& t, int K) const { return mul_u32(b, t.img_pairs) + ((uint32_t)q0 * t.H + h) * K; }
  __device__ __forceinline__ size_t heads0(const GroupTables& t) const { return mul_u32(b, (uint32_t)(t.N * t.H)) + (uint32_t)(q0 * t.H + h); }
  // a strip's fp32 sums [channel 16 dt + 4 g + i][query r] to [B,N,H,D]
  __device__ __forceinline__ void store(const GroupTables& t, void* x, const f32x4 (&a)[R::U], float by) const {
    if (RAG && r >= nq) return;
    T* row = reinterpret_cast<T*>(static_cast<char*>(x) + img_off + ((uint32_t)(q0 + r) * t.row_bytes + (uint32_t)(h * R::RB)));
#pragma unroll
    for (int dt = 0; dt < R::U; ++dt) R::put_four(row + 16 * dt + 4 * g, a[dt] * by);
  }
};

// What a lane fetches of a tile with the n-th load: byte offset from the tile's first row (row clamped to the image at `tile`).
template <typename T, int D>
struct TileLanes {
  typedef WideRows<T, D> R;
  int row[R::NI];
  uint32_t piece[R::NI];
  __device__ __forceinline__ TileLanes(int lane, int h) {
#pragma unroll
    for (int n = 0; n < R::NI; ++n) {
      const int at = n * kWave + lane;
      row[n] = at / R::PCS;
      piece[n] = (uint32_t)((((at & (R::PCS - 1)) ^ R::swizzle(row[n])) << 4) + h * R::RB);
    }
  }
  template <bool RAG>
  __device__ __forceinline__ void load(uint32_t dst, const char* img, int tile, const GroupTables& t, int lane) const {
    if (R::TB >= 1024 || lane < R::TB / 16) {
#pragma unroll
      for (int n = 0; n < R::NI; ++n) {
        const int token = tile * 16 + row[n];
        lds_load16(dst + n * 1024u, img, (uint32_t)(RAG ? min(token, t.N - 1) : token) * t.row_bytes + piece[n]);
      }
    }
  }
};

// The wave's slots by pairs, the union's tiles by stages: PS tiles (K rows and V rows) straight into LDS, SP more wait in registers
// for the places of the first ones (with a reload in their stead the forward kernel stood still for 6000 of 40000 cycles), and
// what is left comes PS at a time.
template <typename T, int D, int PS, int SP, bool RAG>
struct WideWalk {
  typedef WideRows<T, D> R;
  static constexpr int NS = SP * 2 * R::TB / (kGroup * 1024);  // 16-byte pieces of the spare tiles per lane
  static_assert(SP <= PS && (NS * kGroup * 1024 == SP * 2 * R::TB), "");
  const WideStrip<T, D, RAG>& w;
  const GroupTables& t;
  char* lds;  // [PS][2 TB]
  const TileLanes<T, D> lanes;
  const char *kimg, *vimg;
  int ids;  // lane i: the i-th tile of the union (of the stage, behind the first PS + SP)
  u32x4 spare[NS ? NS : 1];
  uint32_t next[2];  // j words of the next pair
  __device__ __forceinline__ uint32_t word(int s) const {
    return *reinterpret_cast<const uint32_t*>(w.jt + ((uint32_t)(s >> 1) * 512u + (uint32_t)(s & 1) * 4u + (uint32_t)w.lane * 8u));
  }
  __device__ __forceinline__ WideWalk(const WideStrip<T, D, RAG>& strip, const GroupTables& tables, const void* k, const void* v, char* l)
      : w(strip), t(tables), lds(l), lanes(strip.lane, strip.h) {
    kimg = static_cast<const char*>(k) + w.img_off;
    vimg = static_cast<const char*>(v) + w.img_off;
    ids = (int)w.ul[(uint32_t)min(w.lane, t.uni_stride - 2)];
    next[0] = word(0);
    next[1] = word(1);
  }
  __device__ __forceinline__ int slots_below(int place) const { return (int)__popcll(__ballot(w.lane < w.cnt && w.my_pos < place)); }
  // n tiles, the first one's number in lane 0 of `ids`
  __device__ __forceinline__ void request(int n) {
    const uint32_t dst = lds_address(lds);
#pragma unroll
    for (int i = 0; i < (2 * PS + kGroup - 1) / kGroup; ++i) {
      const int at = i * kGroup + w.wave;  // K rows, V rows of tile 0, of tile 1, ...
      if (at < 2 * n) lanes.template load<RAG>(dst + (uint32_t)(at * R::TB), (at & 1) ? vimg : kimg, __builtin_amdgcn_readlane(ids, at >> 1), t, w.lane);
    }
  }
  __device__ __forceinline__ void request_first() {
    request(min(PS, w.U));
    if (NS && w.U > PS) {
#pragma unroll
      for (int i = 0; i < NS; ++i) {  // (behind the union's end: its last tile, which nobody uses there)
        const int block = i * kGroup + w.wave, at = block / R::NI;  // 1 KB of K rows or V rows
        const int piece = (block % R::NI) * kWave + w.lane, row = piece / R::PCS;
        const int token = __builtin_amdgcn_readlane(ids, min(PS + (at >> 1), w.U - 1)) * 16 + row;
        spare[i] = *reinterpret_cast<const u32x4*>(((at & 1) ? vimg : kimg) + ((uint32_t)(RAG ? min(token, t.N - 1) : token) * t.row_bytes +
                                                    (uint32_t)((((piece & (R::PCS - 1)) ^ R::swizzle(row)) << 4) + w.h * R::RB)));
      }
    }
  }
  // body(j words, tiles in LDS) for the slots from s0 on whose tiles lie below `end`, the tile at place `lo` being the first in LDS
  // (behind an odd number of them the last tile again, with `none` for words); returns the slot behind them
  template <class Body>
  __device__ __forceinline__ int stage(int s0, int lo, int end, uint32_t none, Body& body) {
    const int s1 = slots_below(end);
#pragma unroll 1
    for (int s = s0; s < s1; s += 2) {
      const bool two = s + 1 < s1;
      const uint32_t wd[2] = {next[0], two ? next[1] : none};
      const int after = min(two ? s + 2 : s + 1, w.cnt - 1);
      next[0] = word(after);
      next[1] = word(min(after + 1, w.cnt - 1));
      const int a = __builtin_amdgcn_readlane(w.my_pos, s) - lo, b = two ? __builtin_amdgcn_readlane(w.my_pos, s + 1) - lo : a;
      const char* const tile[2] = {lds + a * 2 * R::TB, lds + b * 2 * R::TB};
      body(wd, tile);
    }
    return max(s0, s1);
  }
  template <class Body>
  __device__ __forceinline__ void run(uint32_t none, Body&& body) {
    lds_loads_arrive();
    int s = stage(0, 0, PS, none, body);
    if (w.U <= PS) return;  // (the same for the four waves, as what follows)
    int lo = PS;
    if (NS) {
      __syncthreads();  // every wave is through with the places
#pragma unroll
      for (int i = 0; i < NS; ++i) *reinterpret_cast<u32x4*>(lds + (i * kGroup + w.wave) * 1024 + w.lane * 16) = spare[i];
      __syncthreads();
      s = stage(s, lo, lo + SP, none, body);
      lo += SP;
    }
    for (; lo < w.U; lo += PS) {
      ids = (int)w.ul[(uint32_t)min(lo + w.lane, w.U - 1)];
      __syncthreads();
      request(min(PS, w.U - lo));
      lds_loads_arrive();
      s = stage(s, lo, lo + PS, none, body);
    }
  }
};

// LDS of a workgroup's stages: as many tiles as leave room for two workgroups per CU beside the rows of K <= 64 values; and tiles
// that wait in registers, 32 of them a lane.
template <typename T, int D>
constexpr int fwd_stage() { return WideRows<T, D>::TB < 1024 ? 24 : WideRows<T, D>::TB <= 1024 ? 16 : WideRows<T, D>::TB <= 2048 ? 15 : 7; }
template <typename T, int D>
constexpr int query_stage() { return WideRows<T, D>::TB < 1024 ? 24 : WideRows<T, D>::TB <= 1024 ? 16 : WideRows<T, D>::TB <= 2048 ? 11 : 5; }
template <typename T, int D>
constexpr int spare_tiles() { return WideRows<T, D>::TB < 1024 ? 0 : WideRows<T, D>::TB <= 1024 ? 8 : WideRows<T, D>::TB <= 2048 ? 8 : 4; }
template <typename T, int D>
constexpr int key_chunk() { return WideRows<T, D>::TB <= 2048 ? 4 : 2; }

// The strip's bias rows, [query][wide_row], -inf behind them: all values are asked for first, then put down.
template <typename T, int D, bool RAG>
struct WideBias {
  static constexpr int kMost = 16;  // values per lane
  T x[kMost];
  template <int N>
  __device__ __forceinline__ void ask(const WideParams& p, const WideStrip<T, D, RAG>& w) {
    const T* src = static_cast<const T*>(p.bias) + w.pairs0(p.t, p.K);
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int i = min(u * kWave + w.lane, 16 * p.K - 1);
      const int qi = fast_div(i, p.k_magic), j = i - qi * p.K;
      x[u] = src[(uint32_t)(RAG ? min(qi, w.nq - 1) : qi) * p.t.H * p.K + j];
    }
  }
  __device__ __forceinline__ void request(const WideParams& p, const WideStrip<T, D, RAG>& w) {
#pragma unroll
    for (int u = 0; u < kMost; ++u) x[u] = 0;
    if (!p.bias) return;
    if (p.K <= 32) ask<kMost / 2>(p, w); else if (p.K <= 48) ask<kMost * 3 / 4>(p, w); else ask<kMost>(p, w);
  }
  __device__ __forceinline__ void put(const WideParams& p, const WideStrip<T, D, RAG>& w, float* rows, int RW) const {
#pragma unroll
    for (int u = 0; u < kMost; ++u) {
      const int i = u * kWave + w.lane;
      if (i < 16 * p.K) {
        const int qi = fast_div(i, p.k_magic);
        rows[i + qi * (RW - p.K)] = Elem<T>::load(&x[u]);
      }
    }
    if (w.lane < 16) rows[w.lane * RW + p.K] = -INFINITY;
  }
};

template <typename T>
__device__ __forceinline__ f32x4 blank_four(const T* head, int u, int g) {
  Four<T> f;
  f.load(head + 16 * u + 4 * g);
  return f.values();
}

template <typename T, int D, bool RAG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void pla_fwd_wide_kernel(WideParams p) {
  typedef WideRows<T, D> R;
  constexpr int PS = fwd_stage<T, D>();
  __shared__ __align__(16) char tiles[PS * 2 * R::TB];
  __shared__ float rows_all[kGroup][16 * kMostWideRow];
  const int blk = p.block0 + xcd_contiguous_block();
  const int gi = exact_div(blk, p.t.H, p.t.h_magic);
  if (gi >= p.t.groups) return;  // the whole workgroup
  const WideStrip<T, D, RAG> w(p.t, gi, blk - gi * p.t.H);
  const int g = w.g, r = w.r, h = w.h, RW = wide_row(p.K);
  float* rows = rows_all[w.wave];
  WideWalk<T, D, PS, spare_tiles<T, D>(), RAG> walk(w, p.t, p.k, p.v, tiles);
  Four<T> qf[R::U];
  w.query_row(p.t, p.q, qf);
  WideBias<T, D, RAG> bias_rows;
  bias_rows.request(p, w);
  walk.request_first();
  bias_rows.put(p, w, rows, RW);
  const char* row = reinterpret_cast<const char*>(rows + r * RW);
  int k_off[R::U], v_off[4][R::U];
#pragma unroll
  for (int u = 0; u < R::U; ++u) {
    k_off[u] = R::offset(r, 16 * u + 4 * g);
#pragma unroll
    for (int i = 0; i < 4; ++i) v_off[i][u] = R::TB + R::offset(4 * g + i, 16 * u + r);
  }
  // Exponentials relative to the largest score so far: the largest probability is exactly 1 then, as where it is known beforehand.
  // (A reference that moved only for scores 16 above it saved 1.5 us of 29, and out and the gradients were up to 5 % further
  // from 64 bits.)
  float ref = -INFINITY;
  double l_run = 0.;  // (in fp32, with out = sums * (1 / l), out was 1.5 % further from 64 bits than by the gather kernels)
  constexpr int A = chains<T, D>();
  Chains<A, R::U> sums;
  const uint32_t none = 2u * (uint32_t)p.K * 0x01010101u;
  walk.run(none, [&](const uint32_t (&wd)[2], const char* const (&tile)[2]) {
    Four<T> kf[2][R::U];
    float bias[8];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int u = 0; u < R::U; ++u) kf[tt][u].load(tile[tt] + k_off[u]);
#pragma unroll
    for (int i = 0; i < 8; ++i) bias[i] = *reinterpret_cast<const float*>(row + 2 * ((wd[i >> 2] >> (8 * (i & 3))) & 0xffu));
    f32x4 st[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};  // <k[token 4g+i], q[query r]>
    dots(kf, qf, st);
    float vt[8][R::U];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int u = 0; u < R::U; ++u) vt[i][u] = R::one(tile[i >> 2] + v_off[i & 3][u]);
    float pr[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) pr[i] = fmaf(p.scale, st[i >> 2][i & 3], bias[i]);
    const float mx = group_max(fmaxf(fmaxf(fmaxf(pr[0], pr[1]), fmaxf(pr[2], pr[3])), fmaxf(fmaxf(pr[4], pr[5]), fmaxf(pr[6], pr[7]))));
    if (__ballot(mx > ref) != 0ull) {
      const float to = mx > ref ? mx : ref;
      const float by = ref == -INFINITY ? 0.f : wide_exp(ref - to);
      ref = to;
      l_run *= (double)by;
#pragma unroll
      for (int a = 0; a < A; ++a)
#pragma unroll
        for (int u = 0; u < R::U; ++u) sums.a[a][u] *= by;
    }
    const float from = ref == -INFINITY ? 0.f : ref;
#pragma unroll
    for (int i = 0; i < 8; ++i) pr[i] = wide_exp(pr[i] - from);
    l_run += (double)(((pr[0] + pr[1]) + (pr[2] + pr[3])) + ((pr[4] + pr[5]) + (pr[6] + pr[7])));
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int u = 0; u < R::U; ++u) sums.a[i % A][u] = mfma4(vt[i][u], pr[i], sums.a[i % A][u]);  // out^T[channel 16u + 4g+i][query r]
  });
  if (!w.live) return;  // (no workgroup barrier below)
  f32x4 acc[R::U];
  sums.total(acc);
  double l_all = l_run;
#pragma unroll
  for (int o = 16; o < kWave; o <<= 1) l_all += __shfl_xor(l_all, o);
  if (p.k_blank) {
    const T *kb = static_cast<const T*>(p.k_blank) + h * D, *vb = static_cast<const T*>(p.v_blank) + h * D;
    float part = 0.f;
#pragma unroll
    for (int u = 0; u < R::U; ++u) {
      const f32x4 x = blank_four(kb, u, g), q4 = qf[u].values();
#pragma unroll
      for (int e = 0; e < 4; ++e) part = fmaf(q4[e], x[e], part);
    }
    const float sb = p.scale * group_sum(part);
    const float to = fmaxf(ref, sb);
    const float by = wide_exp(ref - to), pb = wide_exp(sb - to);
    l_all = l_all * (double)by + (double)pb;
    ref = to;
#pragma unroll
    for (int u = 0; u < R::U; ++u) acc[u] = acc[u] * by + blank_four(vb, u, g) * pb;
  }
  const float l_tot = (float)l_all;
  // sums / l, rounded once
  const float inv = 1.f / l_tot, l_rest = (float)(l_all - (double)l_tot);
#pragma unroll
  for (int u = 0; u < R::U; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float q0 = acc[u][e] * inv;
      const float rest = fmaf(-q0, l_rest, fmaf(-q0, l_tot, acc[u][e]));
      acc[u][e] = sizeof(T) == 2 ? q0 : fmaf(rest, inv, q0);
    }
  w.store(p.t, p.o, acc, 1.f);
  if (g == 0 && (!RAG || r < w.nq)) {
    // (the logarithm of the sum's mantissa: of the whole sum it is off by a unit of a value up to 20, more than lse's own rounding)
    const float e = (float)__builtin_amdgcn_frexp_expf(l_tot);
    (p.lse + w.heads0(p.t))[(uint32_t)(r * p.t.H)] = ref + fmaf(e, 0.693147180559945f, logf(__builtin_amdgcn_frexp_mantf(l_tot)));
  }
}

// Query side: p and dS of the strip's pairs, dq, dbias; rows of p and -D for the key side.
template <typename T, int D, bool RAG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void pla_bwd_wide_query_kernel(WideParams p) {
  typedef WideRows<T, D> R;
  constexpr int PS = query_stage<T, D>();
  __shared__ __align__(16) char tiles[PS * 2 * R::TB];
  __shared__ __align__(16) float rows_all[kGroup][2 * 16 * kMostWideRow];  // bias rows, then p in their place; rows of dS
  const int blk = p.block0 + xcd_contiguous_block();
  const int gi = exact_div(blk, p.t.H, p.t.h_magic);
  if (gi >= p.t.groups) return;  // the whole workgroup
  const WideStrip<T, D, RAG> w(p.t, gi, blk - gi * p.t.H);
  const int g = w.g, r = w.r, h = w.h, K = p.K, RW = wide_row(K);
  float *rows = rows_all[w.wave], *ds_rows = rows + 16 * RW;
  WideWalk<T, D, PS, spare_tiles<T, D>(), RAG> walk(w, p.t, p.k, p.v, tiles);
  Four<T> qf[R::U], gf[R::U];
  w.query_row(p.t, p.q, qf);
  w.query_row(p.t, p.dout, gf);
  WideBias<T, D, RAG> bias_rows;
  bias_rows.request(p, w);
  walk.request_first();
  // D of query r: <dout, out> where out is fp32.  Rounded to bf16 it would be too far off (gradients 6 - 10 % further from 64 bits): then
  // D = sum of p dP, known only at the end, so that the products go on with p dP and with p, and dS = p dP - D p.
  constexpr bool kLateD = sizeof(T) == 2;
  float Dq = 0.f;
  if constexpr (!kLateD) {
    Four<T> of[R::U];
    w.query_row(p.t, p.out, of);
#pragma unroll
    for (int u = 0; u < R::U; ++u) {
      const f32x4 x = gf[u].values(), y = of[u].values();
#pragma unroll
      for (int e = 0; e < 4; ++e) Dq = fmaf(x[e], y[e], Dq);
    }
    Dq = group_sum(Dq);
  }
  const float lse = (p.lse_in + w.heads0(p.t))[(uint32_t)((RAG ? min(r, w.nq - 1) : r) * p.t.H)];
  bias_rows.put(p, w, rows, RW);
  // pairs that the plan does not hold: dS is 0.  (kLateD: a mark, as p dP may be 0 where p is not, and D p is still to be taken off)
  for (int i = w.lane; i < 16 * RW; i += kWave) ds_rows[i] = kLateD ? __uint_as_float(kNotHeld) : 0.f;
  char *row = reinterpret_cast<char*>(rows + r * RW), *ds_row = reinterpret_cast<char*>(ds_rows + r * RW);
  int k_off[R::U], c_off[4][R::U];
#pragma unroll
  for (int u = 0; u < R::U; ++u) {
    k_off[u] = R::offset(r, 16 * u + 4 * g);
#pragma unroll
    for (int i = 0; i < 4; ++i) c_off[i][u] = R::offset(4 * g + i, 16 * u + r);
  }
  constexpr int A = kLateD ? 1 : D <= 32 ? 8 : 2;
  Chains<A, R::U> sums;
  Chains<1, kLateD ? R::U : 1> sums_p;
  const f32x4 nd = {-Dq, -Dq, -Dq, -Dq};
  const uint32_t none = 2u * (uint32_t)K;
  walk.run(none * 0x01010101u, [&](const uint32_t (&wd)[2], const char* const (&tile)[2]) {
    Four<T> kf[2][R::U], vf[2][R::U];
    float bias[8];
    uint32_t code[8];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int u = 0; u < R::U; ++u) {
        kf[tt][u].load(tile[tt] + k_off[u]);
        vf[tt][u].load(tile[tt] + R::TB + k_off[u]);
      }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      code[i] = (wd[i >> 2] >> (8 * (i & 3))) & 0xffu;
      bias[i] = *reinterpret_cast<const float*>(row + 2 * code[i]);
    }
    f32x4 st[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}}, dp[2] = {nd, nd};  // <k[token 4g+i], q[query r]>; <v[..], dout[..]> - D
    dots(kf, qf, st);
    dots(vf, gf, dp);
    float kt[8][R::U];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int u = 0; u < R::U; ++u) kt[i][u] = R::one(tile[i >> 2] + c_off[i & 3][u]);
    float ds[8], prs[8];  // (kLateD: p dP)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float pr = wide_exp(fmaf(p.scale, st[i >> 2][i & 3], bias[i]) - lse);
      prs[i] = pr;
      ds[i] = pr * dp[i >> 2][i & 3];
      const uint32_t at = code[i] == none ? none + 2u : code[i];  // "no neighbour": its place keeps its -inf
      *reinterpret_cast<float*>(row + 2 * at) = pr;
      *reinterpret_cast<float*>(ds_row + 2 * at) = ds[i];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int u = 0; u < R::U; ++u) {
        sums.a[i % A][u] = mfma4(kt[i][u], ds[i], sums.a[i % A][u]);  // dq^T[channel 16u + 4g+i][query r]
        if constexpr (kLateD) sums_p.a[0][u] = mfma4(kt[i][u], prs[i], sums_p.a[0][u]);
      }
    if (kLateD) Dq += ((ds[0] + ds[1]) + (ds[2] + ds[3])) + ((ds[4] + ds[5]) + (ds[6] + ds[7]));
  });
  if (!w.live) return;  // (no workgroup barrier below)
  f32x4 acc[R::U];
  sums.total(acc);
  if (kLateD) Dq = group_sum(Dq);
  const uint32_t unit = w.sg * p.t.H + h;
  if (p.k_blank) {
    // the blank column of query r: s = scale <q, k_blank>, p = exp(s - lse), dP = <dout, v_blank>, dS = p (dP - D)
    const T *kb = static_cast<const T*>(p.k_blank) + h * D, *vb = static_cast<const T*>(p.v_blank) + h * D;
    float sq = 0.f, gv = 0.f;
#pragma unroll
    for (int u = 0; u < R::U; ++u) {
      const f32x4 x = blank_four(kb, u, g), y = blank_four(vb, u, g), q4 = qf[u].values(), g4 = gf[u].values();
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        sq = fmaf(q4[e], x[e], sq);
        gv = fmaf(g4[e], y[e], gv);
      }
    }
    const float pb = (!RAG || r < w.nq) ? wide_exp(p.scale * group_sum(sq) - lse) : 0.f;  // no blank column for a query past the end
    gv = group_sum(gv);
    if (kLateD) Dq = fmaf(pb, gv, Dq);
    const float dsb = pb * (gv - Dq);
#pragma unroll
    for (int u = 0; u < R::U; ++u) acc[u] += blank_four(kb, u, g) * dsb;
    if (p.blank_part) {
      float* dst = p.blank_part + mul_u32(unit, 2 * D) + 4 * g;
#pragma unroll
      for (int u = 0; u < R::U; ++u) {
        f32x4 x = qf[u].values(), y = gf[u].values();
#pragma unroll
        for (int e = 0; e < 4; ++e) {  // sums over the strip's 16 queries
          x[e] = lanes_sum<1, 8>(p.scale * dsb * x[e], w.lane);
          y[e] = lanes_sum<1, 8>(pb * y[e], w.lane);
        }
        if (r == 0) {
          *reinterpret_cast<f32x4*>(dst + 16 * u) = x;
          *reinterpret_cast<f32x4*>(dst + D + 16 * u) = y;
        }
      }
    }
  }
  if constexpr (kLateD) {
#pragma unroll
    for (int u = 0; u < R::U; ++u) acc[u] -= sums_p.a[0][u] * Dq;
  }
  wave_lds_sync();
  if (w.lane < 16) rows[w.lane * RW + K] = 0.f;  // p of "no neighbour"
  if (kLateD && g == 0) ds_rows[r * RW + K] = Dq;
  wave_lds_sync();
  char* hand = p.hand + mul_u32(unit, p.block_bytes);
  for (int i = w.lane; i < 4 * RW; i += kWave) reinterpret_cast<u32x4*>(hand)[i] = reinterpret_cast<const u32x4*>(rows)[i];
  if (g == 0) reinterpret_cast<float*>(hand + 64 * RW)[r] = -Dq;
  if (p.dbias) {
    T* dst = static_cast<T*>(p.dbias) + w.pairs0(p.t, K);
    for (int i = w.lane; i < w.nq * K; i += kWave) {
      const int qi = fast_div(i, p.k_magic), j = i - qi * K;
      float ds = ds_rows[qi * RW + j];
      if (kLateD) ds = __float_as_uint(ds) == kNotHeld ? 0.f : fmaf(-ds_rows[qi * RW + K], rows[qi * RW + j], ds);
      Elem<T>::store(dst + ((uint32_t)qi * p.t.H * K + j), ds);
    }
  }
  w.store(p.t, p.dq, acc, p.scale);
}

// Key side: a wave per tile of 16 tokens; the strips that touch any of the workgroup's four tiles go through LDS, a chunk on its
// way while one is used.
template <typename T, int D, bool RAG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void pla_bwd_wide_key_kernel(WideParams p) {
  typedef WideRows<T, D> R;
  constexpr int NC = key_chunk<T, D>();
  constexpr int kHand = 64 * kMostWideRow + 64, kStrip = 2 * R::TB + kHand;  // q rows, dout rows, the strip's block of `hand`
  __shared__ __align__(16) char strips[2][NC][kStrip];
  __shared__ __align__(16) char jb_all[2][kGroup][NC][256];  // j bytes of (strip, own tile), 16 (token / 4) + query words
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int g = lane >> 4, r = lane & 15;
  if ((int)blockIdx.x < p.front) {  // the whole workgroup
    if ((int)blockIdx.x < p.blank_blocks) blank_sums<D>(p.blank_part, p.strips, p.t.H, blockIdx.x, reinterpret_cast<float*>(strips), p.dk_blank, p.dv_blank);
    return;
  }
  const int blk = p.block0 + xcd_contiguous_block(blockIdx.x - p.front, gridDim.x - p.front);
  const int gi = exact_div(blk, p.t.H, p.t.h_magic);
  if (gi >= p.t.groups) return;  // the whole workgroup
  const int h = blk - gi * p.t.H;
  const int b = exact_div(gi, p.t.groups_per_image, p.t.gpi_magic);
  const int tile_raw = (gi - b * p.t.groups_per_image) * kGroup + wave;
  const bool live = tile_raw < p.t.strips_per_image;
  const int t0 = min(tile_raw, p.t.strips_per_image - 1) * 16;
  const int nt = RAG ? min(16, p.t.N - t0) : 16;
  const size_t img_off = mul_u32(b, p.t.img_bytes);
  const uint32_t strip0 = (uint32_t)(b * p.t.strips_per_image);
  const int n = __builtin_amdgcn_readfirstlane(p.rev_count[gi]);
  const unsigned long long* list = p.rev_list + __builtin_amdgcn_readfirstlane(p.rev_offset[gi]);
  const int RW = wide_row(p.K);
  Four<T> vf[R::U];  // the tile's V rows: lane (token r, channels 16u + 4g ..)
  {
    const char* row = static_cast<const char*>(p.v) + img_off + ((uint32_t)(t0 + (RAG ? min(r, nt - 1) : r)) * p.t.row_bytes + (uint32_t)(h * R::RB));
#pragma unroll
    for (int u = 0; u < R::U; ++u) vf[u].load(row + (16 * u + 4 * g) * R::E);
  }
  const TileLanes<T, D> lanes(lane, h);
  const char *qimg = static_cast<const char*>(p.q) + img_off, *gimg = static_cast<const char*>(p.dout) + img_off;
  const char* jimg = p.t.jt + mul_u32(strip0, p.t.jt_bytes);
  const uint32_t lds_strips = lds_address(strips), lds_jb = lds_address(jb_all[0][wave]);
  const int hand_pieces = 4 * RW + 4;
  int g_off[R::U], c_off[4][R::U];
#pragma unroll
  for (int u = 0; u < R::U; ++u) {
    g_off[u] = R::TB + R::offset(r, 16 * u + 4 * g);
#pragma unroll
    for (int i = 0; i < 4; ++i) c_off[i][u] = R::offset(4 * g + i, 16 * u + r);
  }
  const int jb_off = ((r >> 2) * 16 + 4 * g) * 4 + (r & 3);
  const int p_off = 2 * R::TB + 4 * g * RW * 4, d_off = 2 * R::TB + 64 * RW + 16 * g;
  constexpr int A = chains<T, D>() < 4 ? 1 : 4;
  Chains<A, R::U> dks, dvs;
  for (int base = 0; base < n; base += kWave) {
    const int nb = min(kWave, n - base);
    const unsigned long long mine = lane < nb ? list[base + lane] : ~0ull;
    const uint32_t my_strip = (uint32_t)(mine >> 32), my_slot = ((uint32_t)mine >> (8 * wave)) & 0xffu;
    const uint32_t my_jt = my_strip * p.t.jt_bytes + (my_slot >> 1) * 512u + (my_slot & 1u) * 4u;
    const unsigned long long mask = __ballot(my_slot != 0xffu);
    auto request = [&](int c, int buf) {  // strips NC c .. of this part of the list, each wave its own ones
      const uint32_t on = (uint32_t)(mask >> (c * NC));
#pragma unroll
      for (int i = 0; i < NC; ++i)
        if (on & (1u << i))
          lds_load4(lds_jb + (uint32_t)((buf * kGroup * NC + i) * 256), jimg, (uint32_t)__builtin_amdgcn_readlane(my_jt, c * NC + i) + (uint32_t)lane * 8u);
      const int e = c * NC + wave;
      if (wave < NC && e < nb) {
        const int strip = (int)__builtin_amdgcn_readlane(my_strip, e);
        const uint32_t dst = lds_strips + (uint32_t)((buf * NC + wave) * kStrip);
        lanes.template load<RAG>(dst, qimg, strip, p.t, lane);
        lanes.template load<RAG>(dst + R::TB, gimg, strip, p.t, lane);
        const char* hand = p.hand + mul_u32((strip0 + (uint32_t)strip) * p.t.H + h, p.block_bytes);
#pragma unroll
        for (int i = 0; i < (kHand + 1023) / 1024; ++i)
          if (lane + i * kWave < hand_pieces) lds_load16(dst + 2 * R::TB + i * 1024u, hand, (uint32_t)(lane + i * kWave) * 16u);
      }
    };
    const int nc = (nb + NC - 1) / NC;
    __syncthreads();  // the part of the list before: its last chunk may still be read
    request(0, 0);
    for (int c = 0; c < nc; ++c) {
      lds_loads_arrive();  // chunk c is there; chunk c - 1 has been used
      if (c + 1 < nc) request(c + 1, (c + 1) & 1);
      const uint32_t on = (uint32_t)(mask >> (c * NC));
#pragma unroll 1
      for (int i = 0; i < NC; ++i) {
        if (!(on & (1u << i))) continue;
        const char* s = strips[c & 1][i];
        const char* jb = jb_all[c & 1][wave][i] + jb_off;
        uint32_t code[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) code[e] = *reinterpret_cast<const uint8_t*>(jb + 4 * e);
        Four<T> gf[1][R::U];
#pragma unroll
        for (int u = 0; u < R::U; ++u) gf[0][u].load(s + g_off[u]);
        f32x4 dp[1] = {*reinterpret_cast<const f32x4*>(s + d_off)};  // -D of queries 4g..4g+3
        float pr[4], gt[4][R::U], qt[4][R::U];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int u = 0; u < R::U; ++u) {
            gt[e][u] = R::one(s + R::TB + c_off[e][u]);
            qt[e][u] = R::one(s + c_off[e][u]);
          }
#pragma unroll
        for (int e = 0; e < 4; ++e) pr[e] = *reinterpret_cast<const float*>(s + p_off + e * RW * 4 + 2 * code[e]);
        // <dout[query 4g+e], v[token r]> - D
        dots(gf, vf, dp);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int u = 0; u < R::U; ++u) dvs.a[e % A][u] = mfma4(gt[e][u], pr[e], dvs.a[e % A][u]);  // dv^T[channel 16u + 4g+i][token r]
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int u = 0; u < R::U; ++u) dks.a[e % A][u] = mfma4(qt[e][u], pr[e] * dp[0][e], dks.a[e % A][u]);
      }
    }
  }
  if (!live || (RAG && r >= nt)) return;
  f32x4 dk[R::U], dv[R::U];
  dks.total(dk);
  dvs.total(dv);
  const size_t at = img_off + ((uint32_t)(t0 + r) * p.t.row_bytes + (uint32_t)(h * R::RB));
#pragma unroll
  for (int u = 0; u < R::U; ++u) {
    R::put_four(reinterpret_cast<T*>(static_cast<char*>(p.dk) + at) + 16 * u + 4 * g, dk[u] * p.scale);
    R::put_four(reinterpret_cast<T*>(static_cast<char*>(p.dv) + at) + 16 * u + 4 * g, dv[u]);
  }
}

size_t wide_hand_bytes(int K) { return (size_t)64 * wide_row(K) + 64; }
size_t wide_bwd_bytes(const PlaArgs& a) {
  const size_t strips = (size_t)a.B * ((a.N + 15) / 16);
  return plan_align(strips * a.H * wide_hand_bytes(a.K)) + (a.k_blank ? plan_align(strips * a.H * 2 * a.d * sizeof(float)) : 0);
}

WideParams wide_params(const PlaArgs& a, const void* plan, const PlanLayout& L) {
  WideParams p = {};
  p.t = group_tables(L, plan, a.N, a.H, a.K);
  p.t.row_bytes = (uint32_t)(a.H * a.d * (a.dtype == 1 ? 2 : 4));
  p.t.img_bytes = (uint32_t)a.N * p.t.row_bytes;
  p.q = a.q; p.k = a.k; p.v = a.v; p.bias = a.bias; p.k_blank = a.k_blank; p.v_blank = a.v_blank;
  p.K = a.K; p.k_magic = div_magic(a.K); p.scale = a.scale;
  return p;
}

template <typename T, int D>
hipError_t wide_fwd(const PlaArgs& a, const void* plan, hipStream_t stream) {
  const PlanLayout L = make_plan_layout(a.B, a.N, a.K, a.S, a.M);
  WideParams p = wide_params(a, plan, L);
  p.o = a.out; p.lse = a.lse;
  const long long blocks = (long long)L.groups * a.H;
  for (long long b0 = 0; b0 < blocks; b0 += kMaxBlocks) {
    p.block0 = (int)b0;
    const dim3 grid((unsigned)((std::min(blocks - b0, kMaxBlocks) + 7) / 8 * 8));
    if (a.N % 16) AFFMAE_LAUNCH("pla_fwd_wide_kernel", stream, (pla_fwd_wide_kernel<T, D, true>), grid, dim3(256), 0, stream, p);
    else AFFMAE_LAUNCH("pla_fwd_wide_kernel", stream, (pla_fwd_wide_kernel<T, D, false>), grid, dim3(256), 0, stream, p);
  }
  return hipGetLastError();
}

template <typename T, int D>
hipError_t wide_bwd(const PlaArgs& a, const void* plan, hipStream_t stream) {
  const PlanLayout L = make_plan_layout(a.B, a.N, a.K, a.S, a.M);
  const char* base = static_cast<const char*>(plan);
  WideParams p = wide_params(a, plan, L);
  p.out = a.out; p.dout = a.dout; p.lse_in = a.lse;
  p.dq = a.dq; p.dk = a.dk; p.dv = a.dv; p.dbias = a.dbias;
  p.rev_offset = reinterpret_cast<const int32_t*>(base + L.rev_offset_off);
  p.rev_count = reinterpret_cast<const int32_t*>(base + L.rev_count_off);
  p.rev_list = reinterpret_cast<const unsigned long long*>(base + L.rev_list_off);
  p.hand = static_cast<char*>(a.workspace);
  p.block_bytes = (int)wide_hand_bytes(a.K);
  p.strips = L.strips;
  if (a.k_blank && a.dk_blank) {
    p.blank_part = reinterpret_cast<float*>(p.hand + plan_align((size_t)L.strips * a.H * p.block_bytes));
    p.blank_blocks = 2 * a.H * D / 8;
    p.dk_blank = a.dk_blank; p.dv_blank = a.dv_blank;
  }
  const int front = (p.blank_blocks + 7) / 8 * 8;
  const long long blocks = (long long)L.groups * a.H, slice = kMaxBlocks - front;
  for (long long b0 = 0; b0 < blocks; b0 += slice) {
    p.block0 = (int)b0;
    const dim3 grid((unsigned)((std::min(blocks - b0, slice) + 7) / 8 * 8));
    if (a.N % 16) AFFMAE_LAUNCH("pla_bwd_wide_query_kernel", stream, (pla_bwd_wide_query_kernel<T, D, true>), grid, dim3(256), 0, stream, p);
    else AFFMAE_LAUNCH("pla_bwd_wide_query_kernel", stream, (pla_bwd_wide_query_kernel<T, D, false>), grid, dim3(256), 0, stream, p);
  }
  for (long long b0 = 0; b0 < blocks; b0 += slice) {
    p.block0 = (int)b0;
    p.front = b0 == 0 ? front : 0;
    const dim3 grid((unsigned)(p.front + (std::min(blocks - b0, slice) + 7) / 8 * 8));
    if (a.N % 16) AFFMAE_LAUNCH("pla_bwd_wide_key_kernel", stream, (pla_bwd_wide_key_kernel<T, D, true>), grid, dim3(256), 0, stream, p);
    else AFFMAE_LAUNCH("pla_bwd_wide_key_kernel", stream, (pla_bwd_wide_key_kernel<T, D, false>), grid, dim3(256), 0, stream, p);
  }
  return hipGetLastError();
}

}  // namespace

// Where these kernels are the better way.  Not in a call of fewer workgroups than CUs (a wave per strip of 16 tokens here, per
// token there): B1 N1000 H1 K48 d32 fp32, us, gather / here: forward 13 / 19, backward 27 / 44.  Above that it is a matter of the
// neighbours, as a tile's product costs the same for few as for many, and of how full the last of the rounds of 512 workgroups is that the
// chip holds: up to 512 .. 767 (1 .. 1.5 rounds) count as `some`, up to 1024 as `most`, and from there on, and near 512, as `full`.
// Gather kernels' time / here, forward and backward together (forward alone), on tables from masked, uniform and jittered tokens, S =
// 64, M = 8; S = 16 and 32 have fewer tiles a strip and are up to 1.3 times better:
//                  full                                 most                            some
//   bf16 d = 16    K 3 .. 64  1.7 - 3.4 (1.3 - 2.4)     1.6 - 2.2 (1.3 - 1.9)           1.3 - 1.7 (1.0 - 1.5)
//   bf16 d = 64    K 17 .. 64 1.11 - 2.0 (1.2 - 2.1)    1.0 - 1.12 (1.14 - 1.35)        K < 48 0.93 - 1.04, K >= 48 0.97 - 1.14 (0.88 - 1.04)
//                  K 9 .. 16  0.96 - 1.2 (0.91 - 1.26)  0.88 - 0.95                     0.77 - 0.93
//   fp32 d = 64    K 16 .. 64 1.14 - 2.7 (1.3 - 3.0)    1.03 - 1.36 (1.23 - 1.6)        K < 48 0.90 - 1.01, K >= 48 1.16 - 1.35 (1.2 - 1.6)
//   fp32 d = 32    K 17 .. 64 1.07 - 2.2 (0.93 - 1.7)   K >= 48 1.10 - 1.21 (0.88 - 0.93)   0.90 - 1.2, but the forward 0.71 - 0.92
//                  K = 16     0.79 - 1.1 (0.67 - 0.97)  K < 48 0.96 - 1.05 (0.87 - 1.0)
//   fp32 d = 16    K 3 .. 64  0.99 - 3.1 (0.88 - 1.7)   K >= 48 1.28 - 1.53 (0.85 - 0.9)    K < 16 1.05 - 1.16 (1.0); 1.01 - 1.45, but the
//                                                       K < 48 0.96 - 1.24 (0.8 - 1.1)      forward 0.76 - 1.0, from there on
// so the rule keeps out what is slower for a step by more than 4 %, or for a forward alone by more than 15 %.
// (fp32 d = 64, K = 9: dS was 4 % further from 64 bits than by the gather kernels.)
// (Forward and backward by one rule: the backward forms p = exp(s - lse) again, and is further from 64 bits where s is not rounded as
// in the forward: fp32, K = 9 .. 64, dq 1.09 - 1.18 times as far with the forward by the gather kernels as with both by them, 0.90 - 0.99 with
// both by these.  So it asks for nothing that only one direction knows; the workspace is what the gather kernels ask for.)
static bool wide_pays(const PlaArgs& a) {
  const long long blocks = (long long)a.B * ((a.N + 16 * kGroup - 1) / (16 * kGroup)) * a.H;
  if (blocks < 256) return false;
  const bool full = blocks >= 1024 || (blocks >= 448 && blocks <= 512), most = full || blocks >= 768;
  if (a.d == 64) return a.K >= (full ? (a.dtype == 1 ? 9 : 16) : most ? 17 : 48);
  if (a.dtype == 1) return a.K >= 3;
  if (a.d == 32) return full ? a.K >= 17 : most && a.K >= 48;
  return a.K >= 3 && (full || a.K < 16 || (most && a.K >= 48));
}
static bool wide_supported(const PlaArgs& a, const void* plan) {
  if (!plan || reinterpret_cast<uintptr_t>(plan) % 256) return false;
  if (a.dtype == 1 && a.d == kD) return false;
  PlaArgs s = a;  // the plan's own limits
  s.dtype = 1;
  s.d = kD;
  if (!pla_cluster_supported(s)) return false;
  // byte offsets, and places in [N,H,K] arrays, inside an image
  if ((long long)a.N * a.H * a.d * (a.dtype == 1 ? 2 : 4) >= (1ll << 32) || (long long)a.N * a.H * a.K >= (1ll << 32)) return false;
  return wide_pays(a) && wide_bwd_bytes(a) <= pla_bwd_general_workspace_bytes(a.B, a.N, a.H, a.K);
}
bool pla_fwd_wide_supported(const PlaArgs& a, const void* plan) { return wide_supported(a, plan); }
// (out, which the forward gave, as it did)
bool pla_bwd_wide_supported(const PlaArgs& a, const void* plan) {
  return wide_supported(a, plan) && a.out && reinterpret_cast<uintptr_t>(a.out) % 16 == 0;
}

#define AFFMAE_WIDE(IMPL)                                       \
  if (a.dtype == 0) {                                           \
    switch (a.d) {                                              \
      case 16: return IMPL<float, 16>(a, plan, stream);         \
      case 32: return IMPL<float, 32>(a, plan, stream);         \
      case 64: return IMPL<float, 64>(a, plan, stream);         \
    }                                                           \
  } else {                                                      \
    switch (a.d) {                                              \
      case 16: return IMPL<bf16_t, 16>(a, plan, stream);        \
      case 64: return IMPL<bf16_t, 64>(a, plan, stream);        \
    }                                                           \
  }                                                             \
  return hipErrorInvalidValue;

hipError_t launch_pla_fwd_wide(const PlaArgs& a, const void* plan, hipStream_t stream) { AFFMAE_WIDE(wide_fwd) }
hipError_t launch_pla_bwd_wide(const PlaArgs& a, const void* plan, hipStream_t stream) { AFFMAE_WIDE(wide_bwd) }

}  // namespace affmae
