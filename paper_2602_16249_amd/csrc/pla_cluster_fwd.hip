// Cluster-tiled local attention, forward (paper, Sec. "Flash-style Cluster
// Attention and Fast Decoder KNN": stream over tiles, never store the scores,
// fp32 softmax statistics; the equation is FlashNbhdAttn).
//
// Valid when tokens are stored in cluster order and every neighbour of a token
// lies in one of its cluster's M near clusters (the table affmae_knn builds), bf16
// storage, d = 32, S a multiple of 16.  Driven by the plan of pla_plan.hip.
//
// One wave per (strip of 16 queries, head), one workgroup per (group of four strips,
// head): see cluster_tiles.h for how the rows come in.  Per pair of token tiles the
// scores of all 16 x 32 (query, token) pairs come from two MFMAs on K rows and the
// strip's Q rows; they are computed transposed (tokens x queries) so that the
// probabilities leave the softmax already in the operand layout of the P.V MFMAs,
// whose V operand the transposing LDS read takes from the row-major tile.  A query
// attends only to its K neighbours: a pair's bias is read from the strip's rows in LDS
// at the place that its j byte gives, and "no neighbour" points to a place of -inf.
// (The other way round, the pairs' bias scattered into a tile of -inf, it took 5 KB
// a wave, several passes for a strip of many tiles, and a fill and 16 scattered
// writes per pass.)
//
// Bound by instruction issue and the two memory round trips at a wave's start; four
// workgroups per CU (39 KB of LDS at K = 48).  us, tiles fetched per (strip, head) / shared:
// B64 N1024 H8 K48 88 / 75, B16 N16384 blobs H4 K48 175 / 151, B8 N16384 H2 K48 40 / 39.  Where
// four strips of small clusters share few tiles it is slower than before: S = 16, M of 8 and more by
// 2 - 12 % (B6 N4096 H8, K32 M8 19.5 / 20.3, K64 M10 23.4 / 26.0; with the second stage's pairs
// fetched only when the one before was done 20.9 and 27.2).  22 tiles and three workgroups were not better.
#include "cluster_tiles.h"
#include "launch.h"
#include "timing.h"

#include <algorithm>

namespace affmae {
namespace {

constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.69314718055994531f;
// Token tiles held in LDS: as many as leave room for four workgroups per CU beside the rows of K values (K > 60: 33 words a
// row; with 16 places and three workgroups 40.1 us against 36.3 before the tiles were shared, K = 64, B = 8, N = 4096, H = 8).
constexpr int kMostPlaces = 16;
inline int places(int K) { return K <= 60 ? kMostPlaces : kMostPlaces - 1; }

struct FwdParams {
  GroupTables t;
  const bf16_t *q, *k, *v, *bias, *k_blank, *v_blank;
  int K, wave_bytes;
  int block0;                   // first workgroup of this launch's slice
  uint32_t item_magic;          // reciprocal of K / W, the items of a query
  float scale;
  RelSource rel;
  bf16_t* out;
  float* lse;
};

// What a pair of tiles needs from LDS.
struct FwdPair {
  Frag8 kf[2];      // K rows, lane (token r, channels 8g..8g+7)
  Frag8 vt[2];      // V^T, lane (channel 16 dt + r): tokens 4g..4g+3 of the first tile, then of the second
  uint16_t tb[8];   // bias of query r and these tokens
};

// Bias rows [query][row_halves] of the strip: a lane brings NT items of W values each, 8 when K is a multiple of 8, 2 when
// it is even, otherwise 1 (see bias_item).  REL: the values are looked up in the head's table, which the workgroup holds in LDS.
// RAG: N is not a multiple of 16.
template <int NT, int W, int PL, int REL, bool RAG>
__device__ __forceinline__ void pla_fwd_body(const FwdParams& p) {
  static_assert(!REL || W == 8, "the table form is built for 16-byte items");
  extern __shared__ __align__(16) char lds[];  // tiles, per wave bias rows, REL: the head's table
  const int blk = p.block0 + xcd_contiguous_block();
  const int gi = exact_div(blk, p.t.H, p.t.h_magic);
  if (gi >= p.t.groups) return;  // the whole workgroup
  TileWalk<PL, RAG> w(p.t, gi, blk - gi * p.t.H, lds);
  const int lane = w.lane, g = w.g, r = w.r, h = w.h, K = p.K;
  const int RH = row_halves(K);
  char* rows = lds + PL * 2048 + w.wave * p.wave_bytes;
  const char* table = lds + PL * 2048 + kGroup * p.wave_bytes;
  Frag8 qf;  // Q^T operand: lane (query r, channels 8g..8g+7)
  qf.x4 = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(p.q) + w.img_off + w.query_piece(r, g));
  constexpr int EW = W == 8 ? 4 : 1;  // 32-bit words per item
  const int per = K / W, items = 16 * per;
  uint32_t bw[NT][EW];
  int row_at[NT];
  RelItem item[REL == kRelDirect ? NT : 1];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int i = t * kWave + lane, ii = i < items ? i : 0;
    const int qi = fast_div(ii, p.item_magic);
    const int j0 = (ii - qi * per) * W;
    const int qc = RAG ? min(qi, w.nq - 1) : qi;
    row_at[t] = (qi * RH + j0) * 2;
#pragma unroll
    for (int e = 0; e < EW; ++e) bw[t][e] = 0u;
    if constexpr (REL == kRelDirect) {
      item[REL == kRelDirect ? t : 0].request(p.rel, w, K, qc, j0);
    } else if (REL) {  // the cells instead
      const u32x4 x = *reinterpret_cast<const u32x4*>(p.rel.cells + w.slots0(K) + (uint32_t)(qc * K + j0));
#pragma unroll
      for (int e = 0; e < EW; ++e) bw[t][e] = x[e];
    } else if (p.bias) {
      const bf16_t* src = p.bias + w.pairs0(K, h) + (uint32_t)qc * p.t.H * K + j0;
      if (W == 8) {
        const u32x4 x = *reinterpret_cast<const u32x4*>(src);
#pragma unroll
        for (int e = 0; e < EW; ++e) bw[t][e] = x[e];
      } else {
        bw[t][0] = W == 2 ? *reinterpret_cast<const uint32_t*>(src) : *src;
      }
    }
  }
  w.request(p.k, p.v);
  if (REL) {
    if constexpr (REL == kRelDirect) {
#pragma unroll
      for (int t = 0; t < NT; ++t) item[REL == kRelDirect ? t : 0].cells(p.rel, w, bw[t]);
    }
    for (int i = threadIdx.x; i < p.rel.ncells; i += 256) reinterpret_cast<bf16_t*>(lds + PL * 2048 + kGroup * p.wave_bytes)[i] = p.rel.table[h * p.rel.ncells + i];
    __syncthreads();
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (t * kWave + lane < items) {
      if (W == 1) {
        *reinterpret_cast<bf16_t*>(rows + row_at[t]) = (bf16_t)bw[t][0];
      } else {
#pragma unroll
        for (int e = 0; e < EW; ++e) {
          if (REL) {
            const uint32_t lo = *reinterpret_cast<const bf16_t*>(table + (bw[t][e] & 0xffffu) * 2u);
            const uint32_t hi = *reinterpret_cast<const bf16_t*>(table + (bw[t][e] >> 16) * 2u);
            bw[t][e] = lo | (hi << 16);
          }
          reinterpret_cast<uint32_t*>(rows + row_at[t])[e] = bw[t][e];
        }
      }
    }
  }
  if (lane < 16) reinterpret_cast<bf16_t*>(rows)[lane * RH + K] = 0xff80u;  // -inf
  const char* row = rows + r * RH * 2;
  const int rd_off = tile_chunk(r, g) * 16;
  const int vt_off0 = tile_tr_offset(g, r, 0) + 1024, vt_off1 = tile_tr_offset(g, r, 1) + 1024;
  const float scale = p.scale;
  asm volatile("" ::"s"(scale));  // read before the wait below: a scalar load in flight makes the LDS waits of the loop wait for all
  float l_run = 0.f;
  f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  f32x4 accw = {0.f, 0.f, 0.f, 0.f};  // sum of the rounded probabilities of query r, four times
  Frag8 ones;
#pragma unroll
  for (int i = 0; i < 4; ++i) ones.u[i] = 0x3f803f80u;
  auto fetch = [&](FwdPair& f, uint32_t w0, uint32_t w1, int at0, int at1) {
    const uint32_t wd[2] = {w0, w1};
    const char* t[2] = {lds + at0, lds + at1};
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) f.kf[tt].x4 = *reinterpret_cast<const u32x4*>(t[tt] + rd_off);
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int i = 0; i < 4; ++i) f.tb[4 * tt + i] = *reinterpret_cast<const uint16_t*>(row + ((wd[tt] >> (8 * i)) & 0xffu));
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      f.vt[0].u2[tt] = lds_read_tr(t[tt] + vt_off0);
      f.vt[1].u2[tt] = lds_read_tr(t[tt] + vt_off1);
    }
  };
  // Exponentials relative to the query's largest score in the first of the strip's first two pairs of tiles that holds a
  // neighbour of it (or 0 where neither does): no running maximum, no rescaling.  Scores that rise or stay far away are caught
  // at the end (a sum outside [2^-40, 2^60]): in fp32 and in bf16 operands, which have its exponents, probabilities keep their
  // relative precision in that range, and so do their sums.  Any reference would do but for the last digit: the largest
  // probability is exactly 1 then, which a bf16 operand holds without error.  Error of out against 64 bits with the first pair
  // alone / the first two / all pairs looked at: K9 S64 M4 2.057e-3 / 1.976e-3 / -, K48 S32 M8 2.217e-3 / 2.202e-3 / 2.191e-3;
  // us, B64 N1024 H8 K48 60.5 / 61.9 / 62.1, B8 N16384 H2 K48 27.9 / 28.2 / 28.6.
  float ref = -INFINITY, shift = 0.f;  // shift = -ref log2 e, rounded
  auto math = [&](const FwdPair& f, bool early) {
    f32x4 st[2];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      const f32x4 z = {0.f, 0.f, 0.f, 0.f};
      st[tt] = mfma32(f.kf[tt], qf, z);  // <k[token 4g+i], q[query r]>
    }
    float pr[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) pr[i] = fmaf(st[i >> 2][i & 3], scale, __uint_as_float((uint32_t)f.tb[i] << 16));
    if (early) {
      const float mx = group_max(fmaxf(fmaxf(fmaxf(pr[0], pr[1]), fmaxf(pr[2], pr[3])), fmaxf(fmaxf(pr[4], pr[5]), fmaxf(pr[6], pr[7]))));
      ref = ref == -INFINITY ? mx : ref;
      shift = ref == -INFINITY ? 0.f : -ref * kLog2e;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) pr[i] = __builtin_amdgcn_exp2f(fmaf(pr[i], kLog2e, shift));
    l_run += ((pr[0] + pr[1]) + (pr[2] + pr[3])) + ((pr[4] + pr[5]) + (pr[6] + pr[7]));
    Frag8 pf;  // P^T operand: k-slots 0..3 = first tile's tokens 4g..4g+3, 4..7 = second tile's
#pragma unroll
    for (int i = 0; i < 4; ++i) pf.u[i] = pack_bf16x2(pr[2 * i], pr[2 * i + 1]);
#pragma unroll
    for (int dt = 0; dt < 2; ++dt) acc[dt] = mfma32(f.vt[dt], pf, acc[dt]);
    accw = mfma32(ones, pf, accw);
  };
  w.arrive();
  w.template walk<true, FwdPair>(K, fetch, math);
  ref = ref == -INFINITY ? 0.f : ref;
  if (!w.live) return;  // (no workgroup barrier below)

  // The probabilities that entered the MFMAs were rounded to bf16.  out divides by the sum of the rounded ones (the weights
  // then add up to 1: a query with one neighbour gets its V row unchanged), lse takes the sum of the unrounded ones.
  float l_tot = group_sum(l_run);
  // The exponentials are 2^(s log2 e + shift) = 2^((s - ref) log2 e + rest), rest what the rounding of shift left (exact in
  // fp32).  So lse = ref + ln 2 (log2 of the sum - rest), the logarithm taken of the sum's mantissa (of the whole sum it is
  // off by a unit of a value of 6 or 7, as much as lse's own rounding).  From shift instead, lse was up to 10 % further from
  // 64 bits than with a reference in natural units throughout (5.9e-8 for 5.3e-8; B3 N4001 H3 K37).
  float rest = fmaf(ref, kLog2e, shift);
  // (the rows past the image's end have no neighbours and a sum of 0: they have no say)
  if (__ballot((!RAG || r < w.nq) && !(l_tot > 0x1p-40f && l_tot < 0x1p60f)) != 0ull) {
    // scores too far from 0 for some query (rare): the row maxima first, then the sums again, rows from memory
    auto tile_row = [&](int s) { return 16u * (uint32_t)w.ul[w.pl[s]]; };
    auto scores = [&](int s, uint32_t row0) {
      Frag8 kf;
      kf.x4 = *reinterpret_cast<const u32x4*>(w.kimg + (min(row0 + r, (uint32_t)p.t.N - 1u) * w.row_bytes + (uint32_t)(h * kD * 2 + g * 16)));
      const f32x4 z = {0.f, 0.f, 0.f, 0.f};
      f32x4 st = mfma32(kf, qf, z);
      const uint32_t wd = *reinterpret_cast<const uint32_t*>(w.jt + (s >> 1) * 512 + lane * 8 + (s & 1) * 4);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        st[i] = fmaf(st[i], scale, bf16_to_f32(*reinterpret_cast<const uint16_t*>(row + ((wd >> (8 * i)) & 0xffu))));
      return st;
    };
    float mx = -INFINITY;
    for (int s = 0; s < w.cnt; ++s) {
      const f32x4 st = scores(s, tile_row(s));
      mx = fmaxf(mx, fmaxf(fmaxf(st[0], st[1]), fmaxf(st[2], st[3])));
    }
    mx = group_max(mx);
    const float from = mx == -INFINITY ? 0.f : mx;
    ref = mx;  // (-inf where every neighbour is masked: a blank column takes it all then, however low its score)
    rest = 0.f;
    l_run = 0.f;
#pragma unroll
    for (int dt = 0; dt < 2; ++dt) acc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    accw = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < w.cnt; ++s) {
      const uint32_t row0 = tile_row(s);
      const f32x4 st = scores(s, row0);
      float pr[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        pr[i] = __builtin_amdgcn_exp2f((st[i] - from) * kLog2e);
        l_run += pr[i];
      }
      Frag4 pf;
      pf.u[0] = pack_bf16x2(pr[0], pr[1]);
      pf.u[1] = pack_bf16x2(pr[2], pr[3]);
#pragma unroll
      for (int dt = 0; dt < 2; ++dt) {
        Frag4 vt;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          vt.h[i] = *reinterpret_cast<const uint16_t*>(w.vimg + (min(row0 + 4 * g + i, (uint32_t)p.t.N - 1u) * w.row_bytes + (uint32_t)((h * kD + dt * 16 + r) * 2)));
        acc[dt] = mfma16(vt, pf, acc[dt]);
      }
      Frag4 ones4;
      ones4.u[0] = ones4.u[1] = 0x3f803f80u;
      accw = mfma16(ones4, pf, accw);
    }
    l_tot = group_sum(l_run);
  }
  float w_tot = accw[0];
  if (p.k_blank) {
    Frag8 kb;
    kb.u4 = *reinterpret_cast<const uint4*>(p.k_blank + h * kD + g * 8);
    float part = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) part = fmaf(bf16_to_f32(qf.h[i]), bf16_to_f32(kb.h[i]), part);
    const float sb = scale * group_sum(part);
    const float m_fin = fmaxf(ref, sb);
    const float alpha = __builtin_amdgcn_exp2f(fmaf(ref - m_fin, kLog2e, -rest));
    const float pb = __builtin_amdgcn_exp2f((sb - m_fin) * kLog2e);
    l_tot = l_tot * alpha + pb;
    w_tot = w_tot * alpha + pb;
    ref = m_fin;
    rest = 0.f;
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        acc[dt][i] = acc[dt][i] * alpha + pb * bf16_to_f32(p.v_blank[h * kD + dt * 16 + g * 4 + i]);
  }
  const float inv = __builtin_amdgcn_rcpf(w_tot);
  // out rows cross through the wave's rows: lane (query r, channels 16dt + 4g..+3) holds 8 bytes of 16-byte piece
  // 2dt + g/2 of row r; lane (row lane/4, piece lane%4) stores 16 bytes
  wave_lds_sync();
#pragma unroll
  for (int dt = 0; dt < 2; ++dt) {
    uint2 o;
    o.x = pack_bf16x2(acc[dt][0] * inv, acc[dt][1] * inv);
    o.y = pack_bf16x2(acc[dt][2] * inv, acc[dt][3] * inv);
    reinterpret_cast<uint2*>(rows)[tile_chunk(r, 2 * dt + (g >> 1)) * 2 + (g & 1)] = o;
  }
  wave_lds_sync();
  const int la = lane >> 2, lc = lane & 3;
  if (!RAG || la < w.nq)
    *reinterpret_cast<u32x4*>(reinterpret_cast<char*>(p.out) + w.img_off + w.query_piece(la, lc)) = reinterpret_cast<const u32x4*>(rows)[tile_chunk(la, lc)];
  if (g == 0 && (!RAG || r < w.nq))
    (p.lse + w.heads0())[(uint32_t)(r * p.t.H)] = ref + fmaf((float)__builtin_amdgcn_frexp_expf(l_tot), kLn2, (__builtin_amdgcn_logf(__builtin_amdgcn_frexp_mantf(l_tot)) - rest) * kLn2);
}

template <int NT, int PL, bool RAG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void pla_fwd_cluster_kernel(FwdParams p) {
  pla_fwd_body<NT, 8, PL, kNoRel, RAG>(p);
}
template <int NT, int PL, bool RAG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void pla_fwd_cluster_rel_kernel(FwdParams p) {
  pla_fwd_body<NT, 8, PL, kRelCells, RAG>(p);
}
template <int NT, int PL, bool RAG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void pla_fwd_cluster_rel_direct_kernel(FwdParams p) {
  pla_fwd_body<NT, 8, PL, kRelDirect, RAG>(p);
}
template <int NT, int PL, bool RAG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void pla_fwd_cluster_scalar_kernel(FwdParams p) {
  pla_fwd_body<NT, 1, PL, kNoRel, RAG>(p);
}
template <int NT, int PL, bool RAG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void pla_fwd_cluster_even_kernel(FwdParams p) {
  pla_fwd_body<NT, 2, PL, kNoRel, RAG>(p);
}

}  // namespace

bool pla_cluster_relpos_supported(const PlaArgs& a) {
  // the table form of the tiled kernels: 16-byte items, 8-byte coordinate pairs
  return pla_cluster_supported(a) && a.K % 8 == 0 && a.rel_coords && a.rel_table &&
         reinterpret_cast<uintptr_t>(a.rel_coords) % 8 == 0;
}

bool pla_cluster_relpos_direct(int B, int N, int H, int K) {
  return H <= kRelDirectHeads || (long long)B * N * H * K <= kRelDirectTriples;
}

bool pla_cluster_supported(const PlaArgs& a) {
  if (!a.near_clusters || a.dtype != 1 || a.d != kD) return false;
  if (a.S % 16 || a.S < 16) return false;                         // token tiles never straddle clusters
  if (a.M > (a.N + a.S - 1) / a.S) return false;
  if ((long long)a.M * a.S / 16 > kMaxSlots) return false;        // tile set of a strip is a 64-bit mask
  if (a.K > 64 || (a.N + 15) / 16 > 65535) return false;          // 16-bit plan entries and tile ids
  if ((long long)a.N * a.S >= (1ll << 31)) return false;          // range of the reciprocal division
  if ((long long)a.N * a.H * kD * 2 >= (1ll << 32)) return false; // 32-bit byte offsets inside an image's K / V
  return true;
}

size_t pla_plan_bytes(int B, int N, int K, int S, int M) { return make_plan_layout(B, N, K, S, M).total; }

hipError_t launch_pla_fwd_cluster(const PlaArgs& a, const void* plan, hipStream_t stream) {
  const PlanLayout L = make_plan_layout(a.B, a.N, a.K, a.S, a.M);
  FwdParams p;
  p.t = group_tables(L, plan, a.N, a.H, a.K);
  p.q = (const bf16_t*)a.q; p.k = (const bf16_t*)a.k; p.v = (const bf16_t*)a.v; p.bias = (const bf16_t*)a.bias;
  p.k_blank = (const bf16_t*)a.k_blank; p.v_blank = (const bf16_t*)a.v_blank;
  p.K = a.K;
  p.scale = a.scale;
  p.out = (bf16_t*)a.out; p.lse = a.lse;
  p.rel = rel_source(a);
  const int W = bias_item(a.K, a.bias, nullptr);
  p.item_magic = div_magic(a.K / W);
  p.wave_bytes = std::max(1024, (16 * row_halves(a.K) * 2 + 15) / 16 * 16);  // (out rows cross there: 1 KB)
  const bool full = places(a.K) == kMostPlaces;
  const size_t shared = places(a.K) * 2048 + kGroup * p.wave_bytes + (a.rel_table ? (size_t)p.rel.ncells * 2 : 0);
  const bool rag = a.N % 16 != 0;  // a short last strip / token tile per image: the variants with row clamps
  const long long blocks = (long long)L.groups * a.H;
  for (long long b0 = 0; b0 < blocks; b0 += kMaxBlocks) {
    // the XCD-contiguous mapping needs a grid that is a multiple of 8; surplus workgroups exit at once
    p.block0 = (int)b0;
    const dim3 grid((unsigned)((std::min(blocks - b0, kMaxBlocks) + 7) / 8 * 8));
#define AFFMAE_FWD_PL(KERNEL, NT, PL)                                                                                         \
  do {                                                                                                                         \
    if (rag) AFFMAE_LAUNCH("pla_fwd_cluster_kernel", stream, (KERNEL<NT, PL, true>), grid, dim3(256), shared, stream, p);      \
    else AFFMAE_LAUNCH("pla_fwd_cluster_kernel", stream, (KERNEL<NT, PL, false>), grid, dim3(256), shared, stream, p);         \
  } while (0)
#define AFFMAE_FWD(KERNEL, NT) AFFMAE_FWD_PL(KERNEL, NT, kMostPlaces)
#define AFFMAE_FWD_LAST(KERNEL, NT)  /* K > 48 among others */         \
  do {                                                                 \
    if (full) AFFMAE_FWD(KERNEL, NT);                                  \
    else AFFMAE_FWD_PL(KERNEL, NT, kMostPlaces - 1);                   \
  } while (0)
    if (a.rel_table && !a.rel_cells) {  // callers check pla_cluster_relpos_supported first
      if (2 * a.K <= kWave) AFFMAE_FWD(pla_fwd_cluster_rel_direct_kernel, 1); else AFFMAE_FWD_LAST(pla_fwd_cluster_rel_direct_kernel, 2);
    } else if (a.rel_table) {
      if (2 * a.K <= kWave) AFFMAE_FWD(pla_fwd_cluster_rel_kernel, 1); else AFFMAE_FWD_LAST(pla_fwd_cluster_rel_kernel, 2);
    } else if (W == 8) {
      if (2 * a.K <= kWave) AFFMAE_FWD(pla_fwd_cluster_kernel, 1); else AFFMAE_FWD_LAST(pla_fwd_cluster_kernel, 2);
    } else if (W == 2) {
      if (a.K <= 16) AFFMAE_FWD(pla_fwd_cluster_even_kernel, 2);
      else if (a.K <= 32) AFFMAE_FWD(pla_fwd_cluster_even_kernel, 4);
      else if (a.K <= 48) AFFMAE_FWD(pla_fwd_cluster_even_kernel, 6);
      else AFFMAE_FWD_LAST(pla_fwd_cluster_even_kernel, 8);
    } else {
      const int ent = (16 * a.K + kWave - 1) / kWave;
      if (ent <= 4) AFFMAE_FWD(pla_fwd_cluster_scalar_kernel, 4);
      else if (ent <= 8) AFFMAE_FWD(pla_fwd_cluster_scalar_kernel, 8);
      else if (ent <= 12) AFFMAE_FWD(pla_fwd_cluster_scalar_kernel, 12);
      else AFFMAE_FWD_LAST(pla_fwd_cluster_scalar_kernel, 16);
    }
#undef AFFMAE_FWD_LAST
#undef AFFMAE_FWD
#undef AFFMAE_FWD_PL
  }
  return hipGetLastError();
}

}  // namespace affmae
