// Cluster-tiled local attention, backward (chain rule on the FlashNbhdAttn
// equation of Sec. "Flash-style Cluster Attention and Fast Decoder KNN"; the
// paper prints no backward).  Same preconditions and plan as the forward
// kernel.  Two kernels:
//
//  query-stationary (one wave per strip of 16 queries and head, four strips a workgroup, rows
//    as in the forward kernel): recomputes the probabilities p from lse tile by tile exactly
//    as the forward pass forms the scores, forms dP - D = V dO^T - D with MFMAs, dS = p (dP - D)
//    with D = <dout, out>, accumulates dQ^T = K^T dS^T (K^T read from the staged rows with the
//    transposing LDS read), and puts p and dS of the real (query, neighbour) pairs into rows of
//    K values in LDS, at the place the pair's bias came from: dS in that order is dbias, and the
//    rows of p are handed to the other kernel as they are, with D of every query.  With blank
//    tokens the blank column joins every query's softmax: its dS feeds dq, and the strip's sums
//    for dk_blank / dv_blank go to the workspace, to be added up over the strips in a fixed
//    order beside the other kernel;
//
//  key-stationary (one wave per tile of 16 tokens and head, four tiles a workgroup): the workgroup
//    walks the strips that touch any of its tiles, four at a time, their q, dout and p rows
//    fetched into LDS once for all four tiles; each wave gathers the p of its tile's pairs (the
//    same j bytes), forms dS = p (dP - D) itself (one more MFMA on its own V rows: handing dS
//    over as well would cost 2 bytes per pair written and read again), and accumulates
//    dK^T = Q^T dS and dV^T = dO^T P in registers, so dk and dv are written once, without
//    atomics and in a fixed summation order.
//
// Bound by instruction issue, three (query) and four (key; above K = 60 three) workgroups per CU.  us, rows fetched per (strip, head) and
// (tile, head) / shared: query 127 / 114, key 88 / 82 (B64 N1024 H8 K48); 265 / 235, 187 / 173 (B16 N16384 blobs H4 K48).
#include "cluster_tiles.h"
#include "launch.h"
#include "timing.h"

#include <algorithm>

namespace affmae {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kRelBins = 128;  // bins of a workgroup's fp64 table

struct BwdParams {
  GroupTables t;
  const bf16_t *q, *k, *v, *bias, *out, *dout;
  const float* lse;
  const int32_t *rev_offset, *rev_count;
  const unsigned long long* rev_list;
  int K, block_bytes;           // block_bytes: of a (strip, head) in `hand`
  int block0;                   // first workgroup of this launch's slice
  uint32_t item_magic;          // reciprocal of K / W, the items of a query
  float scale;
  bf16_t *dq, *dk, *dv;
  bf16_t* ds;    // [B,N,H,K] dS = dbias, or nullptr when the caller does not want it
  char* hand;    // workspace [strips][H]: rows of p [16][row_halves] bf16, then -D [16] fp32
  const bf16_t *k_blank, *v_blank;  // [H,32] or nullptr
  float* blank_part;                // workspace [strips][H][2][32]: the strip's parts of dk_blank, dv_blank; or nullptr
  RelSource rel;    // REL kernels
  float* rel_part;  // workspace [groups][H][ncells]: every workgroup's sums of dS per bin (needs ncells <= kRelBins),
                    // or nullptr: then dS goes out through `ds` for the stand-alone table-gradient kernel
  // Sums over what the query-stationary kernel left in the workspace, by workgroups in front of the key-stationary ones (`front`
  // of them, a multiple of 8): see side_sums.
  int front, rel_entries, blank_blocks, strips;
  float *rel_dtable, *dk_blank, *dv_blank;
};

// ------------------------------------------------------------------------------------------------
// query-stationary kernel
struct BwdPair {
  Frag8 kf[2], vf[2];  // K and V rows, lane (token r, channels 8g..8g+7)
  Frag8 kt[2];         // K^T, lane (channel 16 dt + r): tokens 4g..4g+3 of the first tile, then of the second
  uint16_t tb[8];      // bias of query r and these tokens
  uint16_t at[8];      // their places
};

// Classes of K: up to 48, 60, 64.  Bytes of a wave's bias rows (the words of dS and p take twice that; the key-stationary
// kernel holds one such array a strip), and the token tiles that fit beside them with three workgroups per CU.  LDS is
// given out in pieces of 1280 bytes: three have 53760 bytes each (with 17 tiles, 54016 bytes, two ran: 135 us for 115).
template <int CL>
struct RowArray {
  static constexpr int bytes = CL == 0 ? 25 * 64 : CL == 1 ? 31 * 64 : 33 * 64;
  static constexpr int places = CL == 0 ? 16 : CL == 1 ? 14 : 13;
};

// Items per lane as in the forward kernel: NT of W slots each (W = 8, 2, 1).
// REL: the bias comes from the head's relative-position table, and the table's gradient is summed per
// workgroup (SUMS): each pair's dS is added to its bin in an fp64 table in LDS (ds_add_f64 runs at the speed of an integer
// LDS atomic on this chip; the fp32 form is several times slower) and the workgroup writes its table out at the end.
// RAG: N is not a multiple of 16 (only then do the row clamps and store tests below exist in the code).
template <int NT, int W, int CL, int REL, bool SUMS, bool RAG>
__device__ __forceinline__ void pla_bwd_query_body(const BwdParams& p) {
  static_assert(!SUMS || REL, "the table's gradient belongs to the table form");
  static_assert(!REL || W == 8, "the table form is built for 16-byte items");
  constexpr int PL = RowArray<CL>::places, RB = RowArray<CL>::bytes;
  __shared__ __align__(16) char tiles[PL * 2048];
  __shared__ __align__(16) char rows_all[kGroup][3 * RB];
  __shared__ __align__(16) double sums[SUMS ? kRelBins : 1];  // (one table for the four waves: with one each, two workgroups per CU)
  extern __shared__ __align__(16) char table[];  // REL: the head's table
  const int blk = p.block0 + xcd_contiguous_block();
  const int gi = exact_div(blk, p.t.H, p.t.h_magic);
  if (gi >= p.t.groups) return;  // the whole workgroup
  TileWalk<PL, RAG> w(p.t, gi, blk - gi * p.t.H, tiles);
  const int lane = w.lane, g = w.g, r = w.r, h = w.h, K = p.K;
  const int RH = row_halves(K);
  char* rows = rows_all[w.wave];
  const uint32_t unit = (uint32_t)w.sg * p.t.H + h;
  Frag8 qf, gf, of;  // lane (query r, channels 8g..8g+7) of q, dout, out
  {
    const size_t at = w.img_off + w.query_piece(r, g);
    qf.x4 = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(p.q) + at);
    gf.x4 = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(p.dout) + at);
    of.x4 = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(p.out) + at);
  }
  const float lse = (p.lse + w.heads0())[(uint32_t)((RAG ? min(r, w.nq - 1) : r) * p.t.H)];
  constexpr int EW = W == 8 ? 4 : 1;  // 32-bit words per item
  const int per = K / W, items = 16 * per;
  // Place of an item: byte offset in the bias rows, and element offset of its first value within the strip's
  // [token, head, :] rows, head 0.  Single values and pairs: worked out again at the end, not held (16 items of one value
  // took 177 registers, two wavefronts a SIMD).
  auto item_place = [&](int t, int ln, int& row_at, uint32_t& item_off, bool& live) {
    const int i = t * kWave + ln, ii = i < items ? i : 0;
    const int qi = fast_div(ii, p.item_magic);
    const int j0 = (ii - qi * per) * W;
    row_at = (qi * RH + j0) * 2;
    item_off = (uint32_t)(RAG ? min(qi, w.nq - 1) : qi) * p.t.H * K + j0;
    live = i < items && (!RAG || qi < w.nq);  // items of queries past the image's end: no dbias is written
  };
  uint32_t bw[NT][EW];
  RelItem item[REL == kRelDirect ? NT : 1];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    int row_at;
    uint32_t item_off;
    bool item_live;
    item_place(t, lane, row_at, item_off, item_live);
#pragma unroll
    for (int e = 0; e < EW; ++e) bw[t][e] = 0u;
    if constexpr (REL == kRelDirect) {
      const int ii = t * kWave + lane < items ? t * kWave + lane : 0, qi = fast_div(ii, p.item_magic);
      item[REL == kRelDirect ? t : 0].request(p.rel, w, K, RAG ? min(qi, w.nq - 1) : qi, (ii - qi * per) * W);
    } else if (REL) {  // the cells instead
      const int ii = t * kWave + lane < items ? t * kWave + lane : 0;
      const u32x4 x = reinterpret_cast<const u32x4*>(p.rel.cells + w.slots0(K))[RAG ? min(ii, w.nq * per - 1) : ii];
#pragma unroll
      for (int e = 0; e < EW; ++e) bw[t][e] = x[e];
    } else if (p.bias) {
      const bf16_t* src = p.bias + w.pairs0(K, h) + item_off;
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
    for (int i = threadIdx.x; i < p.rel.ncells; i += 256) reinterpret_cast<bf16_t*>(table)[i] = p.rel.table[h * p.rel.ncells + i];
    if (SUMS && threadIdx.x < kRelBins) sums[SUMS ? threadIdx.x : 0] = 0.;
    __syncthreads();
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (t * kWave + lane < items) {
      int row_at;
      uint32_t item_off;
      bool item_live;
      item_place(t, lane, row_at, item_off, item_live);
      if (W == 1) {
        *reinterpret_cast<bf16_t*>(rows + row_at) = (bf16_t)bw[t][0];
      } else {
#pragma unroll
        for (int e = 0; e < EW; ++e) {
          uint32_t x = bw[t][e];
          if (REL) x = *reinterpret_cast<const bf16_t*>(table + (x & 0xffffu) * 2u) | ((uint32_t)*reinterpret_cast<const bf16_t*>(table + (x >> 16) * 2u) << 16);
          reinterpret_cast<uint32_t*>(rows + row_at)[e] = x;
        }
      }
    }
  }
  if (lane < 16) reinterpret_cast<bf16_t*>(rows)[lane * RH + K] = 0xff80u;  // -inf where "no neighbour" points
  const char* row = rows + r * RH * 2;
  // dS (low half) and p (high half) of a pair in one word, laid out as the bias rows: half the writes of two arrays
  char* words = rows + RB;
  char* word_row = words + r * RH * 4;
  // (a slot whose token the plan does not hold - a table that breaks the promise - is not written below: its dS is 0)
#pragma unroll
  for (int i = 0; i < (2 * RB / 16 + kWave - 1) / kWave; ++i)
    if (i * kWave + lane < 2 * RB / 16) reinterpret_cast<u32x4*>(words)[i * kWave + lane] = u32x4{0u, 0u, 0u, 0u};
  const int rd_off = tile_chunk(r, g) * 16;
  const int tr_off0 = tile_tr_offset(g, r, 0), tr_off1 = tile_tr_offset(g, r, 1);
  const float scale = p.scale;
  asm volatile("" ::"s"(scale));  // read before the wait below (see the forward kernel)
  float Dq = 0.f;  // D of query r
#pragma unroll
  for (int i = 0; i < 8; ++i) Dq = fmaf(bf16_to_f32(gf.h[i]), bf16_to_f32(of.h[i]), Dq);
  Dq = group_sum(Dq);
  const float nl2 = -lse * kLog2e;
  f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  if (p.k_blank && w.live) {
    // the blank column of query r: s = scale <q, k_blank>, p = exp(s - lse), dP = <dout, v_blank>, dS = p (dP - D)
    Frag8 kb, vb;  // channels 8g..8g+7 of the head's blank rows
    kb.u4 = *reinterpret_cast<const uint4*>(p.k_blank + h * kD + g * 8);
    vb.u4 = *reinterpret_cast<const uint4*>(p.v_blank + h * kD + g * 8);
    float sq = 0.f, gv = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      sq = fmaf(bf16_to_f32(qf.h[i]), bf16_to_f32(kb.h[i]), sq);
      gv = fmaf(bf16_to_f32(gf.h[i]), bf16_to_f32(vb.h[i]), gv);
    }
    sq = group_sum(sq);
    gv = group_sum(gv);
    const float pb = (!RAG || r < w.nq) ? __builtin_amdgcn_exp2f(fmaf(scale * sq, kLog2e, nl2)) : 0.f;  // no blank column for a query past the end
    const float dsb = pb * (gv - Dq);
    // dq^T[channel 16dt + 4g + i][query r] += dS k_blank (the scale is applied when dq is written)
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[dt][i] = fmaf(dsb, bf16_to_f32(p.k_blank[h * kD + dt * 16 + g * 4 + i]), acc[dt][i]);
    if (p.blank_part) {
      // the strip's parts: dk_blank[c] = scale sum_r dS_r q[r][c], dv_blank[c] = sum_r p_r dout[r][c]; lane (r, g)
      // holds channels 8g..8g+7 of query r, so the sum over r runs over the 16 lanes of a row of the wave
      float pk[8], pv[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        pk[i] = lanes_sum<1, 8>(scale * dsb * bf16_to_f32(qf.h[i]), lane);
        pv[i] = lanes_sum<1, 8>(pb * bf16_to_f32(gf.h[i]), lane);
      }
      if (r == 0) {
        float* dst = p.blank_part + mul_u32(unit, 2 * kD) + g * 8;
        *reinterpret_cast<float4*>(dst) = make_float4(pk[0], pk[1], pk[2], pk[3]);
        *reinterpret_cast<float4*>(dst + 4) = make_float4(pk[4], pk[5], pk[6], pk[7]);
        *reinterpret_cast<float4*>(dst + kD) = make_float4(pv[0], pv[1], pv[2], pv[3]);
        *reinterpret_cast<float4*>(dst + kD + 4) = make_float4(pv[4], pv[5], pv[6], pv[7]);
      }
    }
  }
  auto fetch = [&](BwdPair& f, uint32_t w0, uint32_t w1, int at0, int at1) {
    const uint32_t wd[2] = {w0, w1};
    const char* t[2] = {tiles + at0, tiles + at1};
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      f.kf[tt].x4 = *reinterpret_cast<const u32x4*>(t[tt] + rd_off);
      f.vf[tt].x4 = *reinterpret_cast<const u32x4*>(t[tt] + 1024 + rd_off);
    }
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        f.at[4 * tt + i] = (uint16_t)((wd[tt] >> (8 * i)) & 0xffu);
        f.tb[4 * tt + i] = *reinterpret_cast<const uint16_t*>(row + f.at[4 * tt + i]);
      }
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      f.kt[0].u2[tt] = lds_read_tr(t[tt] + tr_off0);
      f.kt[1].u2[tt] = lds_read_tr(t[tt] + tr_off1);
    }
  };
  const f32x4 nd = {-Dq, -Dq, -Dq, -Dq};
  auto math = [&](const BwdPair& f, bool) {
    f32x4 st[2], dp[2];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      const f32x4 z = {0.f, 0.f, 0.f, 0.f};
      st[tt] = mfma32(f.kf[tt], qf, z);   // <k[token 4g+i], q[query r]>
      dp[tt] = mfma32(f.vf[tt], gf, nd);  // <v[token 4g+i], dout[query r]> - D
    }
    float pv[8], dsv[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      pv[i] = __builtin_amdgcn_exp2f(fmaf(fmaf(st[i >> 2][i & 3], scale, __uint_as_float((uint32_t)f.tb[i] << 16)), kLog2e, nl2));
      dsv[i] = pv[i] * dp[i >> 2][i & 3];
    }
    uint32_t both[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {  // ("no neighbour": zeros, behind the rows' ends)
      both[i] = pack_bf16x2(dsv[i], pv[i]);
      *reinterpret_cast<uint32_t*>(word_row + 2 * (int)f.at[i]) = both[i];
    }
    Frag8 dsf;  // dS^T operand: k-slots 0..3 = first tile's tokens 4g..4g+3, 4..7 = second tile's
#pragma unroll
    for (int i = 0; i < 4; ++i) dsf.u[i] = __builtin_amdgcn_perm(both[2 * i + 1], both[2 * i], 0x05040100u);
#pragma unroll
    for (int dt = 0; dt < 2; ++dt) acc[dt] = mfma32(f.kt[dt], dsf, acc[dt]);  // dq^T[channel 16dt + 4g+i][query r]
  };
  w.arrive();
  w.template walk<false, BwdPair>(K, fetch, math);
  if (w.live) {
    wave_lds_sync();
    // rows of p and -D to the other kernel
    char* hand = p.hand + mul_u32(unit, p.block_bytes);
    // two words' halves of one kind in one word
    auto halves = [](uint2 x, bool high) { return __builtin_amdgcn_perm(x.y, x.x, high ? 0x07060302u : 0x05040100u); };
    for (int i = lane; i < 2 * RH; i += kWave) {
      u32x4 x;
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = halves(reinterpret_cast<const uint2*>(words)[4 * i + e], true);
      reinterpret_cast<u32x4*>(hand)[i] = x;
    }
    if (g == 0) reinterpret_cast<float*>(hand + 32 * RH)[r] = -Dq;
    // dbias [token, head, slot]; whole 16-byte pieces when K is a multiple of 8
    if (SUMS || p.ds) {
      int ln = lane;
      if (W != 8) asm volatile("" : "+v"(ln));  // (the places are not held from above)
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        int row_at;
        uint32_t item_off;
        bool item_live;
        item_place(t, ln, row_at, item_off, item_live);
        const char* src = words + 2 * row_at;
        if (W == 8) {
          u32x4 x;
#pragma unroll
          for (int e = 0; e < EW; ++e) x[e] = halves(reinterpret_cast<const uint2*>(src)[e], false);
          if (item_live) {
            if (SUMS) {
#pragma unroll
              for (int e = 0; e < EW; ++e) {
                atomicAdd(&sums[SUMS ? (bw[t][e] & 0xffffu) : 0], (double)__uint_as_float(x[e] << 16));
                atomicAdd(&sums[SUMS ? (bw[t][e] >> 16) : 0], (double)__uint_as_float(x[e] & 0xffff0000u));
              }
            } else {
              *reinterpret_cast<u32x4*>(p.ds + w.pairs0(K, h) + item_off) = x;
            }
          }
        } else if (item_live) {
          bf16_t* dst = p.ds + w.pairs0(K, h) + item_off;
          if (W == 2) *reinterpret_cast<uint32_t*>(dst) = halves(*reinterpret_cast<const uint2*>(src), false);
          else *dst = *reinterpret_cast<const bf16_t*>(src);
        }
      }
    }
    // dq rows cross through the bias rows: lane (query r, channels 16dt + 4g..+3) holds 8 bytes of 16-byte piece
    // 2dt + g/2 of row r; lane (row lane/4, piece lane%4) stores 16 bytes
#pragma unroll
    for (int dt = 0; dt < 2; ++dt) {
      uint2 o;
      o.x = pack_bf16x2(acc[dt][0] * scale, acc[dt][1] * scale);
      o.y = pack_bf16x2(acc[dt][2] * scale, acc[dt][3] * scale);
      reinterpret_cast<uint2*>(rows)[tile_chunk(r, 2 * dt + (g >> 1)) * 2 + (g & 1)] = o;
    }
    wave_lds_sync();
    const int la = lane >> 2, lc = lane & 3;
    if (!RAG || la < w.nq)
      *reinterpret_cast<u32x4*>(reinterpret_cast<char*>(p.dq) + w.img_off + w.query_piece(la, lc)) = reinterpret_cast<const u32x4*>(rows)[tile_chunk(la, lc)];
  }
  if (SUMS) {
    __syncthreads();
    if (threadIdx.x < (unsigned)p.rel.ncells) (p.rel_part + mul_u32((uint32_t)gi * p.t.H + h, p.rel.ncells))[threadIdx.x] = (float)sums[SUMS ? threadIdx.x : 0];
  }
}

template <int NT, int CL, bool RAG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void pla_bwd_query_kernel(BwdParams p) {
  pla_bwd_query_body<NT, 8, CL, kNoRel, false, RAG>(p);
}
template <int NT, int CL, bool RAG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void pla_bwd_query_rel_kernel(BwdParams p) {
  pla_bwd_query_body<NT, 8, CL, kRelCells, true, RAG>(p);
}
template <int NT, int CL, bool RAG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void pla_bwd_query_rel_direct_kernel(BwdParams p) {
  pla_bwd_query_body<NT, 8, CL, kRelDirect, true, RAG>(p);
}
template <int NT, int CL, bool RAG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 3))) void pla_bwd_query_rel_ds_kernel(BwdParams p) {
  pla_bwd_query_body<NT, 8, CL, kRelCells, false, RAG>(p);
}
template <int NT, int CL, bool RAG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 3))) void pla_bwd_query_rel_ds_direct_kernel(BwdParams p) {
  pla_bwd_query_body<NT, 8, CL, kRelDirect, false, RAG>(p);
}
template <int NT, int CL, bool RAG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void pla_bwd_query_even_kernel(BwdParams p) {
  pla_bwd_query_body<NT, 2, CL, kNoRel, false, RAG>(p);
}
template <int NT, int CL, bool RAG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void pla_bwd_query_scalar_kernel(BwdParams p) {
  pla_bwd_query_body<NT, 1, CL, kNoRel, false, RAG>(p);
}

// ------------------------------------------------------------------------------------------------
// What is left to add up behind the query-stationary kernel, each in a fixed order, `i` being the workgroup:
//  rel_dtable[i] = sum over the groups of rel_part[group][i]  (i < rel_entries)
//  dk_blank, dv_blank = sums over the strips of blank_part
// As launches of their own, behind the key-stationary kernel, they took 5.0 us (2048 tables of 162 bins) and 3.5 us (753
// strips, 3 heads) and the gap before them, at the end of a step; here they run beside it.  Whole backward with the tables' sum in two
// launches behind / beside, us: 8 images of 16384 tokens (2048 tables of 162 bins) 91.9 / 85.3, 16 201.9 / 191.3, 32 391.7 / 376.7,
// 64 759.8 / 736.7, 32768 images of 64 tokens 600 / 540.
__device__ __forceinline__ void side_sums(const BwdParams& p, int i, float* lds) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  if (i < p.rel_entries) {
    float s = 0.f;
    for (int t = threadIdx.x; t < p.t.groups; t += 256) s += p.rel_part[(size_t)t * p.rel_entries + i];
    s = wave_sum(s);
    if (lane == 0) lds[wave] = s;
    __syncthreads();
    if (threadIdx.x == 0) p.rel_dtable[i] = (lds[0] + lds[1]) + (lds[2] + lds[3]);
    return;
  }
  i -= p.rel_entries;
  if (i < p.blank_blocks) blank_sums<kD>(p.blank_part, p.strips, p.t.H, i, lds, p.dk_blank, p.dv_blank);
}

// ------------------------------------------------------------------------------------------------
// key-stationary kernel
constexpr int kChunk = 4;  // strips in LDS at a time, one per wave to fetch; twice: the next chunk's rows fly during the math

// FRONT: workgroups of side_sums stand in front (the test alone cost calls without them 0.7 %)
template <int CL, bool RAG, bool FRONT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(CL == 2 ? 3 : 4, CL == 2 ? 3 : 4))) void pla_bwd_key_kernel(BwdParams p) {
  constexpr int kRows = RowArray<CL>::bytes;
  constexpr int kStrip = 2048 + kRows + 64;  // q rows, dout rows, the strip's block of `hand`
  __shared__ __align__(16) char strips[2][kChunk][kStrip];
  __shared__ __align__(16) char jb_all[2][kGroup][kChunk][256];  // j bytes of (strip, own tile), 16 (token / 4) + query words
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);  // uniform: keeps per-wave indices in SGPRs
  const int g = lane >> 4, r = lane & 15;
  if (FRONT && (int)blockIdx.x < p.front) {  // the whole workgroup
    side_sums(p, blockIdx.x, reinterpret_cast<float*>(strips));
    return;
  }
  const int blk = p.block0 + (FRONT ? xcd_contiguous_block(blockIdx.x - p.front, gridDim.x - p.front) : xcd_contiguous_block());
  const int gi = exact_div(blk, p.t.H, p.t.h_magic);
  if (gi >= p.t.groups) return;  // the whole workgroup
  const int h = blk - gi * p.t.H;
  const int b = exact_div(gi, p.t.groups_per_image, p.t.gpi_magic);
  const int tile_raw = (gi - b * p.t.groups_per_image) * kGroup + wave;
  const bool live = tile_raw < p.t.strips_per_image;
  const int t0 = min(tile_raw, p.t.strips_per_image - 1) * 16;  // the tile's first token, within the image
  // the image's last token tile and last strip may be short (N % 16 != 0): loads past the end repeat the last real row
  // (its p is 0: no pair refers to it), stores past the end are skipped
  const int nt = RAG ? min(16, p.t.N - t0) : 16;
  const uint32_t row_bytes = p.t.row_bytes;
  const size_t img_off = mul_u32(b, p.t.img_bytes);
  const uint32_t strip0 = (uint32_t)(b * p.t.strips_per_image);
  const int n = __builtin_amdgcn_readfirstlane(p.rev_count[gi]);
  const unsigned long long* list = p.rev_list + __builtin_amdgcn_readfirstlane(p.rev_offset[gi]);
  const int RH = row_halves(p.K);
  Frag8 vop;  // the tile's V rows: lane (token r, channels 8g..8g+7)
  vop.x4 = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(p.v) + img_off +
                                           ((uint32_t)(t0 + (RAG ? min(r, nt - 1) : r)) * row_bytes + (uint32_t)(h * kD * 2 + g * 16)));
  const int la = lane >> 2, lc = lane & 3;
  const uint32_t piece = (uint32_t)((lc ^ ((la >> 1) & 3)) * 16 + h * kD * 2);  // as TileWalk::issue
  const uint32_t lane_off = (uint32_t)la * row_bytes + piece, lane_off_max = (uint32_t)(p.t.N - 1) * row_bytes + piece;
  const uint32_t tile_bytes = 16u * row_bytes;
  const char* qimg = reinterpret_cast<const char*>(p.q) + img_off;
  const char* gimg = reinterpret_cast<const char*>(p.dout) + img_off;
  const int hand_pieces = 2 * RH + 4;
  const char* jimg = p.t.jt + mul_u32(strip0, p.t.jt_bytes);
  const uint32_t lds_strips = lds_address(strips);
  const uint32_t lds_jb = lds_address(jb_all[0][wave]);
  const int rd_off = tile_chunk(r, g) * 16;
  const int tr_off0 = tile_tr_offset(g, r, 0), tr_off1 = tile_tr_offset(g, r, 1);
  const int jb_off = ((r >> 2) * 16 + 4 * g) * 4 + (r & 3);
  const int prow = 4 * g * RH * 2;  // queries 4g..4g+3: rows of p
  const int d_off = 2048 + 32 * RH + 16 * g;
  f32x4 dk[2], dv[2];
#pragma unroll
  for (int dt = 0; dt < 2; ++dt) dk[dt] = dv[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int base = 0; base < n; base += kWave) {
    const int nb = min(kWave, n - base);
    const unsigned long long mine = lane < nb ? list[base + lane] : ~0ull;
    // what the loop needs of an entry, worked out for 64 of them at once: where the j bytes of its strip and the own tile
    // lie in the image's table, where the strip's rows start, and which entries touch the own tile at all
    const uint32_t my_strip = (uint32_t)(mine >> 32), my_slot = ((uint32_t)mine >> (8 * wave)) & 0xffu;
    const uint32_t my_jt = my_strip * p.t.jt_bytes + (my_slot >> 1) * 512u + (my_slot & 1u) * 4u;
    const uint32_t my_rows = my_strip * tile_bytes;
    const unsigned long long mask = __ballot(my_slot != 0xffu);
    auto request = [&](int c, int buf) {  // strips kChunk c .. of this part of the list
      const int e = c * kChunk + wave;
      if (e < nb) {
        uint32_t off = (uint32_t)__builtin_amdgcn_readlane(my_rows, e) + lane_off;
        if (RAG) off = min(off, lane_off_max);
        const uint32_t dst = lds_strips + (uint32_t)((buf * kChunk + wave) * kStrip);
        lds_load16(dst, qimg, off);
        lds_load16(dst + 1024u, gimg, off);
        const char* hand = p.hand + mul_u32((strip0 + (uint32_t)__builtin_amdgcn_readlane(my_strip, e)) * p.t.H + h, p.block_bytes);
#pragma unroll
        for (int i = 0; i < (CL == 2 ? 3 : 2); ++i)
          if (lane + i * kWave < hand_pieces) lds_load16(dst + 2048u + i * 1024u, hand, (uint32_t)(lane + i * kWave) * 16u);
      }
      const uint32_t on = (uint32_t)(mask >> (c * kChunk));
#pragma unroll
      for (int i = 0; i < kChunk; ++i)
        if (on & (1u << i))
          lds_load4(lds_jb + (uint32_t)((buf * kGroup * kChunk + i) * 256), jimg, (uint32_t)__builtin_amdgcn_readlane(my_jt, c * kChunk + i) + (uint32_t)lane * 8u);
    };
    auto compute = [&](int c, auto buf) {
      const uint32_t on = (uint32_t)(mask >> (c * kChunk));
#pragma unroll
      for (int i = 0; i < kChunk; ++i) {
        if (!(on & (1u << i))) continue;
        const char* s = strips[decltype(buf)::value][i];
        const char* jb = jb_all[decltype(buf)::value][wave][i] + jb_off;
        uint32_t code[4], pw[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) code[e] = *reinterpret_cast<const uint8_t*>(jb + 4 * e);
        Frag8 gf;  // dout, lane (query r, channels 8g..8g+7)
        gf.x4 = *reinterpret_cast<const u32x4*>(s + 1024 + rd_off);
        const f32x4 nd = *reinterpret_cast<const f32x4*>(s + d_off);  // -D of queries 4g..4g+3
        Frag4 qT[2], gT[2];  // lane (channel 16dt + r, queries 4g..4g+3)
        qT[0].u2 = lds_read_tr(s + tr_off0);
        qT[1].u2 = lds_read_tr(s + tr_off1);
        gT[0].u2 = lds_read_tr(s + 1024 + tr_off0);
        gT[1].u2 = lds_read_tr(s + 1024 + tr_off1);
#pragma unroll
        for (int e = 0; e < 4; ++e) pw[e] = *reinterpret_cast<const uint16_t*>(s + 2048 + prow + e * RH * 2 + code[e]);
        __builtin_amdgcn_sched_barrier(0);
        // <dout[query 4g+i], v[token r]> - D[query 4g+i]: the accumulator starts at -D
        const f32x4 dp = mfma32(gf, vop, nd);
        Frag4 pf, df;  // operand B of the 16x16x16 MFMA: lane (token r, queries 4g..4g+3)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          pf.u[e] = pw[2 * e] | (pw[2 * e + 1] << 16);
          df.u[e] = pack_bf16x2(__uint_as_float(pw[2 * e] << 16) * dp[2 * e], __uint_as_float(pw[2 * e + 1] << 16) * dp[2 * e + 1]);
        }
#pragma unroll
        for (int dt = 0; dt < 2; ++dt) {
          dv[dt] = mfma16(gT[dt], pf, dv[dt]);  // dv^T[channel 16dt + 4g+i][token r]
          dk[dt] = mfma16(qT[dt], df, dk[dt]);
        }
      }
    };
    const int nc = (nb + kChunk - 1) / kChunk;
    __syncthreads();  // the part of the list before: its last chunk may still be read
    request(0, 0);
    for (int c = 0; c < nc; c += 2) {
      __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
      __syncthreads();  // chunk c is there; chunk c - 1 has been used
      if (c + 1 < nc) request(c + 1, 1);
      compute(c, std::integral_constant<int, 0>{});
      if (c + 1 >= nc) break;
      __builtin_amdgcn_s_waitcnt(0x0070);
      __syncthreads();
      if (c + 2 < nc) request(c + 2, 0);
      compute(c + 1, std::integral_constant<int, 1>{});
    }
  }
  __syncthreads();
  if (!live) return;
  // dk / dv rows cross through LDS the other way: lane (token r, channels 16dt + 4g..+3) holds 8 bytes of 16-byte
  // piece 2dt + g/2 of row r; lane (row lane/4, piece lane%4) stores 16 bytes
  char* mine = strips[0][wave];
#pragma unroll
  for (int dt = 0; dt < 2; ++dt) {
    const int at = tile_chunk(r, 2 * dt + (g >> 1)) * 2 + (g & 1);
    uint2 o;
    o.x = pack_bf16x2(dk[dt][0] * p.scale, dk[dt][1] * p.scale);
    o.y = pack_bf16x2(dk[dt][2] * p.scale, dk[dt][3] * p.scale);
    reinterpret_cast<uint2*>(mine)[at] = o;
    o.x = pack_bf16x2(dv[dt][0], dv[dt][1]);
    o.y = pack_bf16x2(dv[dt][2], dv[dt][3]);
    reinterpret_cast<uint2*>(mine + 1024)[at] = o;
  }
  wave_lds_sync();
  if (!RAG || la < nt) {
    const size_t at = img_off + ((uint32_t)(t0 + la) * row_bytes + (uint32_t)(h * kD * 2 + lc * 16));
    *reinterpret_cast<u32x4*>(reinterpret_cast<char*>(p.dk) + at) = reinterpret_cast<const u32x4*>(mine)[tile_chunk(la, lc)];
    *reinterpret_cast<u32x4*>(reinterpret_cast<char*>(p.dv) + at) = reinterpret_cast<const u32x4*>(mine + 1024)[tile_chunk(la, lc)];
  }
}

}  // namespace

size_t pla_bwd_cluster_rel_workspace_bytes(int B, int N, int H, int R) {
  // tables of the workgroups (and room for 64 more, which callers' workspaces have always had)
  const size_t cells = (size_t)(2 * R + 1) * (2 * R + 1);
  const size_t groups = (size_t)B * ((N + 16 * kGroup - 1) / (16 * kGroup));
  return plan_align(groups * H * cells * sizeof(float)) + plan_align(64 * H * cells * sizeof(float));
}
bool pla_bwd_cluster_rel_sums(int R) { return (2 * R + 1) * (2 * R + 1) <= kRelBins; }

// bytes of a (strip, head) in the hand-over: rows of p, -D
static size_t hand_bytes(int K) { return (size_t)32 * row_halves(K) + 64; }

size_t pla_bwd_cluster_workspace_bytes(int B, int N, int H, int K, int S, int M) {
  const PlanLayout L = make_plan_layout(B, N, K, S, M);
  return plan_align((size_t)L.strips * H * hand_bytes(K)) +
         plan_align((size_t)L.strips * H * 2 * kD * sizeof(float));  // parts of the blank gradients
}

hipError_t launch_pla_bwd_cluster(const PlaArgs& a, const void* plan, void* workspace, hipStream_t stream) {
  const PlanLayout L = make_plan_layout(a.B, a.N, a.K, a.S, a.M);
  const char* base = static_cast<const char*>(plan);
  BwdParams p;
  p.t = group_tables(L, plan, a.N, a.H, a.K);
  p.q = (const bf16_t*)a.q; p.k = (const bf16_t*)a.k; p.v = (const bf16_t*)a.v; p.bias = (const bf16_t*)a.bias;
  p.out = (const bf16_t*)a.out; p.dout = (const bf16_t*)a.dout; p.lse = a.lse;
  p.rev_offset = reinterpret_cast<const int32_t*>(base + L.rev_offset_off);
  p.rev_count = reinterpret_cast<const int32_t*>(base + L.rev_count_off);
  p.rev_list = reinterpret_cast<const unsigned long long*>(base + L.rev_list_off);
  p.K = a.K; p.block_bytes = (int)hand_bytes(a.K);
  p.scale = a.scale;
  p.dq = (bf16_t*)a.dq; p.dk = (bf16_t*)a.dk; p.dv = (bf16_t*)a.dv;
  p.hand = static_cast<char*>(workspace);
  p.ds = (bf16_t*)a.dbias;
  p.k_blank = (const bf16_t*)a.k_blank; p.v_blank = (const bf16_t*)a.v_blank;
  p.blank_part = (a.k_blank && a.dk_blank)
                     ? reinterpret_cast<float*>(p.hand + plan_align((size_t)L.strips * a.H * hand_bytes(a.K)))
                     : nullptr;
  p.rel = rel_source(a);
  p.rel_part = a.rel_part;
  const int W = bias_item(a.K, a.bias, p.ds);
  p.item_magic = div_magic(a.K / W);
  const bool rag = a.N % 16 != 0;  // a short last strip / token tile per image: the variants with row clamps
  const int cl = a.K <= 48 ? 0 : a.K <= 60 ? 1 : 2;
  const size_t shared = a.rel_table ? (size_t)p.rel.ncells * 2 : 0;
  const long long blocks = (long long)L.groups * a.H;
  // the XCD-contiguous mapping needs a grid that is a multiple of 8; surplus workgroups exit at once
  for (long long b0 = 0; b0 < blocks; b0 += kMaxBlocks) {
    p.block0 = (int)b0;
    const dim3 grid((unsigned)((std::min(blocks - b0, kMaxBlocks) + 7) / 8 * 8));
#define AFFMAE_BWDQ(KERNEL, NT, CL)                                                                                               \
  do {                                                                                                                            \
    if (rag) AFFMAE_LAUNCH("pla_bwd_query_kernel", stream, (KERNEL<NT, CL, true>), grid, dim3(256), shared, stream, p);           \
    else AFFMAE_LAUNCH("pla_bwd_query_kernel", stream, (KERNEL<NT, CL, false>), grid, dim3(256), shared, stream, p);              \
  } while (0)
#define AFFMAE_BWDQ_LAST(KERNEL, NT)               \
  do {                                             \
    if (cl == 1) AFFMAE_BWDQ(KERNEL, NT, 1);       \
    else AFFMAE_BWDQ(KERNEL, NT, 2);               \
  } while (0)
    // (an item of 8 per lane covers K <= 32; two cover the rest)
#define AFFMAE_BWDQ_VEC(KERNEL)                       \
  do {                                                \
    if (2 * a.K <= kWave) AFFMAE_BWDQ(KERNEL, 1, 0);  \
    else if (cl == 0) AFFMAE_BWDQ(KERNEL, 2, 0);      \
    else AFFMAE_BWDQ_LAST(KERNEL, 2);                 \
  } while (0)
    // callers check pla_cluster_relpos_supported first
    if (a.rel_table && !a.rel_cells && a.rel_part) AFFMAE_BWDQ_VEC(pla_bwd_query_rel_direct_kernel);
    else if (a.rel_table && !a.rel_cells) AFFMAE_BWDQ_VEC(pla_bwd_query_rel_ds_direct_kernel);
    else if (a.rel_table && a.rel_part) AFFMAE_BWDQ_VEC(pla_bwd_query_rel_kernel);
    else if (a.rel_table) AFFMAE_BWDQ_VEC(pla_bwd_query_rel_ds_kernel);
    else if (W == 8) AFFMAE_BWDQ_VEC(pla_bwd_query_kernel);
    else if (W == 2) {
      if (a.K <= 16) AFFMAE_BWDQ(pla_bwd_query_even_kernel, 2, 0);
      else if (a.K <= 32) AFFMAE_BWDQ(pla_bwd_query_even_kernel, 4, 0);
      else if (cl == 0) AFFMAE_BWDQ(pla_bwd_query_even_kernel, 6, 0);
      else AFFMAE_BWDQ_LAST(pla_bwd_query_even_kernel, 8);
    } else {
      const int ent = (16 * a.K + kWave - 1) / kWave;
      if (ent <= 4) AFFMAE_BWDQ(pla_bwd_query_scalar_kernel, 4, 0);
      else if (ent <= 8) AFFMAE_BWDQ(pla_bwd_query_scalar_kernel, 8, 0);
      else if (cl == 0) AFFMAE_BWDQ(pla_bwd_query_scalar_kernel, 12, 0);
      else AFFMAE_BWDQ_LAST(pla_bwd_query_scalar_kernel, 16);
    }
#undef AFFMAE_BWDQ_VEC
#undef AFFMAE_BWDQ_LAST
#undef AFFMAE_BWDQ
  }
  const int cells = (2 * a.rel_R + 1) * (2 * a.rel_R + 1);
  p.rel_entries = a.rel_table && a.rel_part ? a.H * cells : 0;
  p.rel_dtable = a.rel_dtable;
  p.blank_blocks = p.blank_part ? 8 * a.H : 0;
  p.strips = L.strips;
  p.dk_blank = a.dk_blank; p.dv_blank = a.dv_blank;
  const int front = (p.rel_entries + p.blank_blocks + 7) / 8 * 8;
  const long long slice = kMaxBlocks - front;
  for (long long b0 = 0; b0 < blocks; b0 += slice) {
    p.block0 = (int)b0;
    p.front = b0 == 0 ? front : 0;
    const dim3 grid((unsigned)(p.front + (std::min(blocks - b0, slice) + 7) / 8 * 8));
#define AFFMAE_BWDK_RAG(CL, RAG)                                                                                                      \
  do {                                                                                                                                \
    if (p.front) AFFMAE_LAUNCH("pla_bwd_key_kernel", stream, (pla_bwd_key_kernel<CL, RAG, true>), grid, dim3(256), 0, stream, p);     \
    else AFFMAE_LAUNCH("pla_bwd_key_kernel", stream, (pla_bwd_key_kernel<CL, RAG, false>), grid, dim3(256), 0, stream, p);            \
  } while (0)
#define AFFMAE_BWDK(CL)                                                         \
  do {                                                                          \
    if (rag) AFFMAE_BWDK_RAG(CL, true); else AFFMAE_BWDK_RAG(CL, false);        \
  } while (0)
    if (cl == 0) AFFMAE_BWDK(0); else if (cl == 1) AFFMAE_BWDK(1); else AFFMAE_BWDK(2);
#undef AFFMAE_BWDK
#undef AFFMAE_BWDK_RAG
  }
  return hipGetLastError();
}

}  // namespace affmae
