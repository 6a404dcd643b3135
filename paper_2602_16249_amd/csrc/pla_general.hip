// Local attention over arbitrary neighbour tables (paper, Sec. "Flash-style
// Cluster Attention and Fast Decoder KNN", the FlashNbhdAttn equation), gather
// formulation: one wave per token, the neighbours' rows fetched straight from
// global memory.  This path makes no assumption about the table (any indices,
// repeats allowed: every slot is its own softmax column) and serves both storage
// types and every head size; the cluster-tiled kernels cover clustered bf16 tables with heads of 32 channels and, in
// calls large enough to fill the chip that come with a plan, fp32 and heads of 16 and 64 (pla_cluster_wide.hip).
//
// Lane layout, all three kernels: a head's row of D channels is PP = D / E pieces of 16 bytes (E = 4 fp32 or 8
// bf16 channels); lane (r, c) = (lane / PP, lane % PP) holds piece c of the r-th of the 64 / PP rows of a trip, so a
// load instruction fetches whole rows, PP lanes wide, and K neighbours take ceil(K * PP / 64) <= PP trips.  A dot
// product with the query's row is a partial sum per lane, added over the PP lanes of the row so that lane (r, c) ends
// with the value of trip c (scatter_sum): one neighbour per lane, so bias, exp, maximum, sum and dS are done once each
// and stored or loaded with one instruction, and a weight goes back to its row's lanes by a lane move (RowValues).  A
// weighted sum of rows is accumulated per lane and added over the rows at the end.  Scores are never stored.
// Bound by the vector ALU and by the latency of the row loads; so the loads of several trips are issued before the
// first is used.  16384 tokens, K = 48, two heads of 32 fp32 channels: forward 58 us, query side 71 us, key side 42 us
// with every lane of a row holding every score and one trip's rows in flight; 29.5, 39 and 36 us as here.
// Backward: the query-side kernel writes dq and dbias and keeps p and dS of every (query, slot) pair; dk and dv are
// gathered, not scattered: the pairs are filed per neighbour token (the list builder shared with the decoder's and
// the merging backward) and a wave per token adds dS q and p dout over its list - no floating-point atomics.
#include "cluster_common.h"
#include "device_util.h"
#include "launch.h"
#include "select_util.h"
#include "timing.h"

#include <hip/amd_detail/amd_hip_unsafe_atomics.h>

#include <type_traits>

namespace affmae {
namespace {

constexpr int kWavesPerBlock = 4;

// 16 bytes of a row as fp32 values (the first E of v)
template <typename T>
struct Piece;
template <>
struct Piece<float> {
  static constexpr int E = 4;
  typedef float4 Raw;
  static __device__ __forceinline__ Raw raw(const float* p) { return *reinterpret_cast<const float4*>(p); }
  static __device__ __forceinline__ void load(const float* p, float (&v)[8]) { unpack(raw(p), v); }
  static __device__ __forceinline__ void unpack(const Raw& x, float (&v)[8]) {
    v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
    v[4] = v[5] = v[6] = v[7] = 0.f;
  }
  static __device__ __forceinline__ void store(float* p, const float (&v)[8]) {
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
  }
};
template <>
struct Piece<bf16_t> {
  static constexpr int E = 8;
  typedef uint4 Raw;
  static __device__ __forceinline__ Raw raw(const bf16_t* p) { return *reinterpret_cast<const uint4*>(p); }
  static __device__ __forceinline__ void load(const bf16_t* p, float (&v)[8]) { unpack(raw(p), v); }
  static __device__ __forceinline__ void unpack(const Raw& x, float (&v)[8]) {
    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[2 * e] = __uint_as_float(w[e] << 16);
      v[2 * e + 1] = __uint_as_float(w[e] & 0xffff0000u);
    }
  }
  static __device__ __forceinline__ void store(bf16_t* p, const float (&v)[8]) {
    uint4 x;
    x.x = (uint32_t)f32_to_bf16(v[0]) | ((uint32_t)f32_to_bf16(v[1]) << 16);
    x.y = (uint32_t)f32_to_bf16(v[2]) | ((uint32_t)f32_to_bf16(v[3]) << 16);
    x.z = (uint32_t)f32_to_bf16(v[4]) | ((uint32_t)f32_to_bf16(v[5]) << 16);
    x.w = (uint32_t)f32_to_bf16(v[6]) | ((uint32_t)f32_to_bf16(v[7]) << 16);
    *reinterpret_cast<uint4*>(p) = x;
  }
};

// Sums and maxima over lanes whose numbers differ in the bits LO .. HI (powers of two), every lane receiving the
// result.  The exchanges run on the vector ALU (DPP patterns inside a row of 16 lanes, the row / half swaps across
// rows): a softmax row costs some fifty of them, and through the LDS crossbar they were most of the kernel's time.
// Nearest lanes first, unlike lanes_sum / lanes_max: with these the kernels took 0.6 % longer over 96 shapes (up to 4 %).
// All lanes of the wave must be active.
template <int J>
__device__ __forceinline__ float lane_xor_f(float x, int lane) {
  return __uint_as_float(lane_xor_u32<J>(__float_as_uint(x), lane));
}
template <int LO, int HI>
__device__ __forceinline__ float sum_bits(float x, int lane) {
  if constexpr (LO <= HI) {
    x += lane_xor_f<LO>(x, lane);
    return sum_bits<LO * 2, HI>(x, lane);
  } else {
    return x;
  }
}
template <int LO, int HI>
__device__ __forceinline__ float max_bits(float x, int lane) {
  if constexpr (LO <= HI) {
    x = fmaxf(x, lane_xor_f<LO>(x, lane));
    return max_bits<LO * 2, HI>(x, lane);
  } else {
    return x;
  }
}
// sum over the PP lanes of a row / over the 64 / PP rows of a trip (same piece) / over the wave
template <int PP>
__device__ __forceinline__ float row_sum(float x, int lane) { return sum_bits<1, PP / 2>(x, lane); }
template <int PP, int E>
__device__ __forceinline__ void rows_sum(float (&a)[8], int lane) {
#pragma unroll
  for (int i = 0; i < E; ++i) a[i] = sum_bits<PP, 32>(a[i], lane);
}
__device__ __forceinline__ float all_sum(float x, int lane) { return sum_bits<1, 32>(x, lane); }
__device__ __forceinline__ float all_max(float x, int lane) { return max_bits<1, 32>(x, lane); }
// exp(x) for x <= 0 or so: the library routine for fp32 storage (1e-5 bar), the hardware exp2 for bf16 storage
template <typename T>
__device__ __forceinline__ float exp_for(float x) {
  if constexpr (sizeof(T) == 2) return __builtin_amdgcn_exp2f(x * 1.4426950408889634f);
  else return expf(x);
}

// <a, b> over the 16 bytes at pa and pb: fp32 pieces by fused multiply-adds, bf16 pieces by four two-element dot
// instructions on the packed values (no unpacking)
__device__ __forceinline__ float dot_raw(const float4& a, const float4& b) {
  return fmaf(a.w, b.w, fmaf(a.z, b.z, fmaf(a.y, b.y, a.x * b.x)));
}
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
__device__ __forceinline__ float dot_raw(const uint4& a, const uint4& b) {
  float acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a.x), __builtin_bit_cast(bf16x2_t, b.x), 0.f, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a.y), __builtin_bit_cast(bf16x2_t, b.y), acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a.z), __builtin_bit_cast(bf16x2_t, b.z), acc, false);
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a.w), __builtin_bit_cast(bf16x2_t, b.w), acc, false);
}

// fn(t) for t = 0 .. N - 1, t a compile-time constant (a DPP pattern has to be one)
template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F&& fn) {
  if constexpr (I < N) {
    fn(std::integral_constant<int, I>{});
    static_for<N, I + 1>(fn);
  }
}

// d[t] holds this lane's part of a value of trip t; lane (r, c) receives the whole value of trip c % N, the sum of d[c % N]
// over the PP lanes of its row (row_scatter: N trips, a power of two up to PP).  Each step halves the values that a lane still carries: PP - 1 exchanges where the
// sum of every trip over all lanes takes PP log2(PP), and what follows is done once per value instead of once per lane.
template <int J, int N>
__device__ __forceinline__ float scatter_sum(const float (&d)[N], int lane) {
  if constexpr (N == 1) {
    return d[0];
  } else {
    float half[N / 2];
    const bool up = lane & J;
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
      const float keep = up ? d[2 * i + 1] : d[2 * i], give = up ? d[2 * i] : d[2 * i + 1];
      half[i] = keep + lane_xor_f<J>(give, lane);
    }
    return scatter_sum<2 * J>(half, lane);
  }
}

template <int PP, int N>
__device__ __forceinline__ float row_scatter(const float (&d)[N], int lane) {
  return sum_bits<N, PP / 2>(scatter_sum<1>(d, lane), lane);
}

// The way back: get<t>() is, in every lane of a row, the value that lane t of the row held.
template <int PP>
struct RowValues {
  uint32_t own, low, high;
  __device__ __forceinline__ RowValues(uint32_t x, int lane) : own(x), low(x), high(x) {
    if constexpr (PP == 8) {  // the row's first and second quad, in both quads
      const uint32_t other = lane_xor_u32<4>(x, lane);
      low = (lane & 4) ? other : x;
      high = (lane & 4) ? x : other;
    }
  }
  template <int T>
  __device__ __forceinline__ uint32_t get() const {
    static_assert(T < PP, "a lane of the row");
    if constexpr (PP == 16) return dpp_mov<0x150 + T>(own);           // row_newbcast
    else if constexpr (PP == 8) return dpp_mov<(T & 3) * 0x55>(T < 4 ? low : high);  // one lane of a quad
    else if constexpr (PP == 4) return dpp_mov<T * 0x55>(own);
    else return dpp_mov<T * 0x05 + (2 + T) * 0x50>(own);              // PP == 2: one lane of each pair
  }
  template <int T>
  __device__ __forceinline__ float getf() const { return __uint_as_float(get<T>()); }
};

// The neighbour rows of this lane in every trip: element offset of its piece in head 0 of the row (a row past the
// end repeats the last neighbour and gets weight 0).
template <int TR>
struct LaneRows {
  size_t off[TR];
};
template <int PP, int E, int TR>
__device__ __forceinline__ LaneRows<TR> lane_rows(int mynb, long long img_base, int C, int K, int lane) {
  constexpr int RPT = kWave / PP;
  const int rl = lane / PP, pc = lane % PP;
  LaneRows<TR> r;
#pragma unroll
  for (int t = 0; t < TR; ++t) {
    const int nbj = __shfl(mynb, min(t * RPT + rl, K - 1));
    r.off[t] = (size_t)(img_base + nbj) * C + (size_t)(pc * E);
  }
  return r;
}

// TR: trips that the K neighbours take at most: 1, 2 or PP.  With TR < PP the lanes c >= TR of a row repeat the values of
// lanes c % TR and do not count.  (With PP for every K the parts of trips that K does not reach were exchanged all the same:
// 12000 tokens, fp32, three heads of 64, K = 1: forward 37 us, 14 with one trip; eight heads, K = 8: 94 and 46 us.)
template <typename T, int D, int TR>
__global__ __launch_bounds__(256) void pla_fwd_general_kernel(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v, const T* __restrict__ bias,
    const int32_t* __restrict__ nbr_idx, const T* __restrict__ k_blank, const T* __restrict__ v_blank,
    long long tokens, int N, int H, int K, float scale, T* __restrict__ out, float* __restrict__ lse) {
  constexpr int E = Piece<T>::E, PP = D / E, RPT = kWave / PP;  // K <= RPT * TR
  constexpr bool kHoldV = TR <= 8;  // V rows loaded with the K rows, as far as the registers go
  constexpr int kBatch = TR < 8 ? TR : 4;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);  // token, image and their addresses: scalar
  const int rl = lane / PP, pc = lane % PP;
  const int C = H * D;
  const int trips = (K + RPT - 1) / RPT;
  for (long long tok = (long long)blockIdx.x * kWavesPerBlock + wave; tok < tokens;
       tok += (long long)gridDim.x * kWavesPerBlock) {
    const long long img_base = (tok / N) * N;  // first token of this image
    const int mynb = min(max(nbr_idx[tok * K + min(lane, K - 1)], 0), N - 1);
    const LaneRows<TR> rows = lane_rows<PP, E, TR>(mynb, img_base, C, K, lane);
    const int mine = pc * RPT + rl;  // the neighbour whose score this lane holds
    const bool valid = mine < K && pc < TR;
    for (int h = 0; h < H; ++h) {
      const auto qv = Piece<T>::raw(q + (tok * H + h) * D + pc * E);
      const float bj = (bias && valid) ? Elem<T>::load(bias + (tok * H + h) * K + mine) : 0.f;
      typename Piece<T>::Raw vr[TR];
      float part[TR];
#pragma unroll
      for (int t0 = 0; t0 < TR; t0 += kBatch) {
        typename Piece<T>::Raw kr[kBatch];
#pragma unroll
        for (int t = 0; t < kBatch; ++t)
          if (t0 + t < trips) {
            kr[t] = Piece<T>::raw(k + rows.off[t0 + t] + (size_t)h * D);
            if (kHoldV) vr[t0 + t] = Piece<T>::raw(v + rows.off[t0 + t] + (size_t)h * D);
          }
#pragma unroll
        for (int t = 0; t < kBatch; ++t) part[t0 + t] = t0 + t < trips ? dot_raw(qv, kr[t]) : 0.f;
      }
      const float dot = row_scatter<PP>(part, lane);  // (by every lane: also those past K hand on parts)
      const float s = valid ? fmaf(scale, dot, bj) : -INFINITY;
      float sb = -INFINITY, eb = 0.f;
      if (k_blank) {
        sb = scale * row_sum<PP>(dot_raw(qv, Piece<T>::raw(k_blank + (size_t)h * D + pc * E)), lane);
      }
      const float m = fmaxf(all_max(s, lane), sb);
      const float e = valid ? exp_for<T>(s - m) : 0.f;
      if (k_blank) eb = exp_for<T>(sb - m);
      const float z = all_sum(e, lane) + eb;
      const RowValues<PP> ew(__float_as_uint(e), lane);
      float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      static_for<TR>([&](auto t) {
        if (t < trips) {
          float vp[8];
          Piece<T>::unpack(kHoldV ? vr[t] : Piece<T>::raw(v + rows.off[t] + (size_t)h * D), vp);
          const float et = ew.template getf<t>();
#pragma unroll
          for (int i = 0; i < E; ++i) acc[i] = fmaf(et, vp[i], acc[i]);
        }
      });
      rows_sum<PP, E>(acc, lane);
      if (v_blank) {
        float vb[8];
        Piece<T>::load(v_blank + (size_t)h * D + pc * E, vb);
#pragma unroll
        for (int i = 0; i < E; ++i) acc[i] = fmaf(eb, vb[i], acc[i]);
      }
      if (rl == 0) {
        const float inv = 1.f / z;
#pragma unroll
        for (int i = 0; i < E; ++i) acc[i] *= inv;
        Piece<T>::store(out + (tok * H + h) * D + pc * E, acc);
      }
      if (lane == 0) lse[tok * H + h] = m + logf(z);
    }
  }
}

// Query side of the backward: dq, dbias, and p / dS of every (query, slot) pair for the key side; also the global
// token of every pair and the lowest and highest of a query's K, for the list builder.
template <typename T, int D, int TR>
__global__ __launch_bounds__(256) void pla_bwd_general_kernel(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v, const T* __restrict__ bias,
    const int32_t* __restrict__ nbr_idx, const T* __restrict__ k_blank, const T* __restrict__ v_blank,
    const float* __restrict__ lse, const T* __restrict__ dout, long long tokens, int N, int H, int K, float scale,
    T* __restrict__ dq, T* __restrict__ dbias, float* __restrict__ pw, float* __restrict__ dsw,
    int32_t* __restrict__ pair_tok, int2* __restrict__ bounds, float* __restrict__ dk_blank,
    float* __restrict__ dv_blank) {
  constexpr int E = Piece<T>::E, PP = D / E, RPT = kWave / PP;
  constexpr bool kHoldV = TR <= 8;
  extern __shared__ float smem[];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);  // token, image and their addresses: scalar
  const int rl = lane / PP, pc = lane % PP;
  const int C = H * D;
  const int trips = (K + RPT - 1) / RPT;
  const bool blank_grad = k_blank && dk_blank;
  float* bacc = smem + (size_t)wave * 2 * C;  // [2][C] running blank-row gradients of this wave
  if (blank_grad)
    for (int c = lane; c < 2 * C; c += kWave) bacc[c] = 0.f;

  for (long long tok = (long long)blockIdx.x * kWavesPerBlock + wave; tok < tokens;
       tok += (long long)gridDim.x * kWavesPerBlock) {
    const long long img_base = (tok / N) * N;
    const int mynb = min(max(nbr_idx[tok * K + min(lane, K - 1)], 0), N - 1);
    const LaneRows<TR> rows = lane_rows<PP, E, TR>(mynb, img_base, C, K, lane);
    {
      const int gtok = (int)(img_base + mynb);  // lanes >= K repeat the last neighbour
      if (lane < K) pair_tok[tok * K + lane] = gtok;
      int tmin = gtok, tmax = gtok;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        tmin = min(tmin, __shfl_xor(tmin, o));
        tmax = max(tmax, __shfl_xor(tmax, o));
      }
      if (lane == 0) bounds[tok] = make_int2(tmin, tmax);
    }
    const int mine = pc * RPT + rl;  // the neighbour whose p and dS this lane holds
    const bool valid = mine < K && pc < TR;
    for (int h = 0; h < H; ++h) {
      const T* qrow = q + (tok * H + h) * D + pc * E;
      const T* grow = dout + (tok * H + h) * D + pc * E;
      const float l = lse[tok * H + h];
      const auto qraw = Piece<T>::raw(qrow), graw = Piece<T>::raw(grow);
      typename Piece<T>::Raw kr[TR], vr[TR];
#pragma unroll
      for (int t = 0; t < TR; ++t)
        if (t < trips) {
          kr[t] = Piece<T>::raw(k + rows.off[t] + (size_t)h * D);
          if (kHoldV) vr[t] = Piece<T>::raw(v + rows.off[t] + (size_t)h * D);
        }
      const long long at = (tok * H + h) * K + mine;
      const float bj = (bias && valid) ? Elem<T>::load(bias + at) : 0.f;
      float part[TR], gpart[TR];
#pragma unroll
      for (int t = 0; t < TR; ++t) {
        part[t] = gpart[t] = 0.f;
        if (t < trips) {
          part[t] = dot_raw(qraw, kr[t]);
          gpart[t] = dot_raw(graw, kHoldV ? vr[t] : Piece<T>::raw(v + rows.off[t] + (size_t)h * D));
        }
      }
      const float dP = row_scatter<PP>(gpart, lane);
      const float dot = row_scatter<PP>(part, lane);
      const float p = valid ? exp_for<T>(fmaf(scale, dot, bj) - l) : 0.f;
      float pb = 0.f, dPb = 0.f, kb[8];
      if (k_blank) {
        const auto kbraw = Piece<T>::raw(k_blank + (size_t)h * D + pc * E);
        Piece<T>::unpack(kbraw, kb);
        pb = exp_for<T>(scale * row_sum<PP>(dot_raw(qraw, kbraw), lane) - l);
        dPb = row_sum<PP>(dot_raw(graw, Piece<T>::raw(v_blank + (size_t)h * D + pc * E)), lane);
      }
      const float Dsum = all_sum(valid ? p * dP : 0.f, lane) + pb * dPb;
      const float ds = valid ? p * (dP - Dsum) : 0.f;
      if (valid) {
        pw[at] = p;
        dsw[at] = ds;
        if (dbias) Elem<T>::store(dbias + at, ds);
      }
      const RowValues<PP> dsr(__float_as_uint(ds), lane);
      float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      static_for<TR>([&](auto t) {
        if (t < trips) {
          float kp[8];
          Piece<T>::unpack(kr[t], kp);
          const float dst = dsr.template getf<t>();
#pragma unroll
          for (int i = 0; i < E; ++i) acc[i] = fmaf(dst, kp[i], acc[i]);
        }
      });
      rows_sum<PP, E>(acc, lane);
      const float dsb = pb * (dPb - Dsum);
      if (k_blank) {
#pragma unroll
        for (int i = 0; i < E; ++i) acc[i] = fmaf(dsb, kb[i], acc[i]);
      }
      if (rl == 0) {
#pragma unroll
        for (int i = 0; i < E; ++i) acc[i] *= scale;
        Piece<T>::store(dq + (tok * H + h) * D + pc * E, acc);
        if (blank_grad) {
          float qv[8], gv[8];
          Piece<T>::load(qrow, qv);
          Piece<T>::load(grow, gv);
#pragma unroll
          for (int i = 0; i < E; ++i) {
            bacc[h * D + pc * E + i] += scale * dsb * qv[i];
            bacc[C + h * D + pc * E + i] += pb * gv[i];
          }
        }
      }
    }
  }
  if (blank_grad) {
    // one addition per workgroup and channel: every workgroup adds to the same 2 C words (12000 tokens, C = 64: the
    // backward took 238 us when every wave added its own, 73 us as here)
    __syncthreads();
    for (int c = threadIdx.x; c < 2 * C; c += kWavesPerBlock * kWave) {
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < kWavesPerBlock; ++w) s += smem[(size_t)w * 2 * C + c];
      unsafeAtomicAdd(c < C ? dk_blank + c : dv_blank + (c - C), s);
    }
  }
}

// Key side of the backward: dk[t] = scale * sum over the pairs (i, j) filed under token t of dS[i,j] q[i],
// dv[t] = sum of p[i,j] dout[i]; a pair id is i * K + j with i the query's global token.  Tokens that nobody lists get
// zero rows.
template <typename T, int D>
__global__ __launch_bounds__(256) void pla_bwd_general_key_kernel(
    const T* __restrict__ q, const T* __restrict__ dout, const float* __restrict__ pw, const float* __restrict__ dsw,
    const int32_t* __restrict__ offset, const int32_t* __restrict__ list, long long tokens, int H, int K,
    uint32_t k_magic, float scale, T* __restrict__ dk, T* __restrict__ dv) {
  constexpr int E = Piece<T>::E, PP = D / E, RPT = kWave / PP;
  constexpr int kBatch = PP < 8 ? PP : 8;  // trips whose rows are in flight together
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);  // token, image and their addresses: scalar
  const int rl = lane / PP, pc = lane % PP;
  for (long long tok = (long long)blockIdx.x * kWavesPerBlock + wave; tok < tokens;
       tok += (long long)gridDim.x * kWavesPerBlock) {
    const int lo = offset[tok], n = offset[tok + 1] - lo;
    for (int h = 0; h < H; ++h) {
      float ak[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, av[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      for (int base = 0; base < n; base += kWave) {
        // lane (r, c) fetches the pair that its row handles in trip c
        const int idx = base + pc * RPT + rl;
        const bool on = idx < n;
        const int pair = list[lo + min(idx, n - 1)];  // a place past the end repeats the last pair with weight 0
        const int i = exact_div(pair, K, k_magic), j = pair - i * K;
        const long long at = ((long long)i * H + h) * K + j;
        const RowValues<PP> qi((uint32_t)i, lane), ps(__float_as_uint(on ? pw[at] : 0.f), lane),
            dss(__float_as_uint(on ? dsw[at] : 0.f), lane);
        const int trips = (min(n - base, kWave) + RPT - 1) / RPT;
        static_for<PP / kBatch>([&](auto bt) {
          typename Piece<T>::Raw qr[kBatch], gr[kBatch];
          static_for<kBatch>([&](auto u) {
            if (bt * kBatch + u < trips) {
              const long long row = ((long long)(int)qi.template get<bt * kBatch + u>() * H + h) * D + pc * E;
              qr[u] = Piece<T>::raw(q + row);
              gr[u] = Piece<T>::raw(dout + row);
            }
          });
          static_for<kBatch>([&](auto u) {
            if (bt * kBatch + u < trips) {
              const float pt = ps.template getf<bt * kBatch + u>(), dst = dss.template getf<bt * kBatch + u>();
              float qp[8], gp[8];
              Piece<T>::unpack(qr[u], qp);
              Piece<T>::unpack(gr[u], gp);
#pragma unroll
              for (int c = 0; c < E; ++c) {
                ak[c] = fmaf(dst, qp[c], ak[c]);
                av[c] = fmaf(pt, gp[c], av[c]);
              }
            }
          });
        });
      }
      rows_sum<PP, E>(ak, lane);
      rows_sum<PP, E>(av, lane);
      if (rl == 0) {
#pragma unroll
        for (int c = 0; c < E; ++c) ak[c] *= scale;
        Piece<T>::store(dk + (tok * H + h) * D + pc * E, ak);
        Piece<T>::store(dv + (tok * H + h) * D + pc * E, av);
      }
    }
  }
}

__global__ __launch_bounds__(256) void fill_zero_kernel(float* __restrict__ p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0.f;
}

int grid_for(size_t n, int per_block, int cap) {
  size_t g = (n + per_block - 1) / per_block;
  if (g < 1) g = 1;
  if (g > (size_t)cap) g = cap;
  return (int)g;
}

size_t general_align(size_t n) { return (n + 255) & ~(size_t)255; }
struct GeneralBwdLayout {
  size_t p_off, ds_off, pair_off, bounds_off, offset_off, list_off, total;
};
GeneralBwdLayout general_bwd_layout(int B, int N, int H, int K) {
  GeneralBwdLayout L;
  const size_t tokens = (size_t)B * N, pairs = tokens * K;
  size_t off = 0;
  L.p_off = off;      off += general_align(pairs * H * sizeof(float));
  L.ds_off = off;     off += general_align(pairs * H * sizeof(float));
  L.pair_off = off;   off += general_align(pairs * sizeof(int32_t));
  L.bounds_off = off; off += general_align(tokens * 2 * sizeof(int32_t));
  L.offset_off = off; off += general_align((tokens + 1) * sizeof(int32_t));
  L.list_off = off;   off += general_align(pairs * sizeof(int32_t));
  L.total = off;
  return L;
}

// fn(TR) for the trips that K neighbours take
template <typename T, int D, typename F>
void by_trips(int K, F&& fn) {
  constexpr int PP = D / Piece<T>::E, RPT = kWave / PP;
  if (K <= RPT) return fn(std::integral_constant<int, 1>{});
  if constexpr (PP > 2) {
    if (K <= 2 * RPT) return fn(std::integral_constant<int, 2>{});
  }
  fn(std::integral_constant<int, PP>{});
}

template <typename T, int D>
hipError_t fwd_impl(const PlaArgs& a, hipStream_t stream) {
  const long long tokens = (long long)a.B * a.N;
  const int grid = grid_for((size_t)tokens, kWavesPerBlock, 1 << 20);
  by_trips<T, D>(a.K, [&](auto trips) {
    AFFMAE_LAUNCH("pla_fwd_general_kernel", stream, (pla_fwd_general_kernel<T, D, decltype(trips)::value>), dim3(grid), dim3(256), 0,
                  stream, (const T*)a.q, (const T*)a.k, (const T*)a.v, (const T*)a.bias, a.nbr_idx, (const T*)a.k_blank,
                  (const T*)a.v_blank, tokens, a.N, a.H, a.K, a.scale, (T*)a.out, a.lse);
  });
  return hipGetLastError();
}

template <typename T, int D>
hipError_t bwd_impl(const PlaArgs& a, hipStream_t stream) {
  const long long tokens = (long long)a.B * a.N;
  if (tokens * a.K >= (1ll << 31)) return hipErrorInvalidValue;  // pair ids are 32-bit
  const GeneralBwdLayout L = general_bwd_layout(a.B, a.N, a.H, a.K);
  char* ws = static_cast<char*>(a.workspace);
  float* pw = reinterpret_cast<float*>(ws + L.p_off);
  float* dsw = reinterpret_cast<float*>(ws + L.ds_off);
  int32_t* pair_tok = reinterpret_cast<int32_t*>(ws + L.pair_off);
  int2* bounds = reinterpret_cast<int2*>(ws + L.bounds_off);
  int32_t* offset = reinterpret_cast<int32_t*>(ws + L.offset_off);
  int32_t* list = reinterpret_cast<int32_t*>(ws + L.list_off);
  const bool blank_grad = a.k_blank && a.dk_blank;
  if (blank_grad) {
    AFFMAE_LAUNCH("fill_zero_kernel", stream, fill_zero_kernel, dim3(1), dim3(256), 0, stream, a.dk_blank, (size_t)a.H * D);
    AFFMAE_LAUNCH("fill_zero_kernel", stream, fill_zero_kernel, dim3(1), dim3(256), 0, stream, a.dv_blank, (size_t)a.H * D);
  }
  const size_t lds = blank_grad ? kWavesPerBlock * 2 * (size_t)a.H * D * sizeof(float) : 0;
  // With blank gradients every workgroup adds a running sum to the same words at its end, so bound the grid: four
  // workgroups per CU.
  const int grid = grid_for((size_t)tokens, kWavesPerBlock, blank_grad ? 1024 : (1 << 20));
  by_trips<T, D>(a.K, [&](auto trips) {
    AFFMAE_LAUNCH("pla_bwd_general_kernel", stream, (pla_bwd_general_kernel<T, D, decltype(trips)::value>), dim3(grid), dim3(256), lds,
                  stream, (const T*)a.q, (const T*)a.k, (const T*)a.v, (const T*)a.bias, a.nbr_idx, (const T*)a.k_blank,
                  (const T*)a.v_blank, a.lse, (const T*)a.dout, tokens, a.N, a.H, a.K, a.scale, (T*)a.dq, (T*)a.dbias, pw, dsw,
                  pair_tok, bounds, a.dk_blank, a.dv_blank);
  });
  const hipError_t e = launch_pair_lists(pair_tok, a.B, a.N, a.N * a.K, offset, list, stream,
                                         reinterpret_cast<const int32_t*>(bounds), a.K);
  if (e != hipSuccess) return e;
  const int kgrid = grid_for((size_t)tokens, kWavesPerBlock, 1 << 20);
  AFFMAE_LAUNCH("pla_bwd_general_key_kernel", stream, (pla_bwd_general_key_kernel<T, D>), dim3(kgrid), dim3(256), 0, stream,
                (const T*)a.q, (const T*)a.dout, pw, dsw, offset, list, tokens, a.H, a.K, div_magic(a.K), a.scale,
                (T*)a.dk, (T*)a.dv);
  return hipGetLastError();
}

}  // namespace

size_t pla_bwd_general_workspace_bytes(int B, int N, int H, int K) { return general_bwd_layout(B, N, H, K).total; }

#define AFFMAE_DISPATCH(IMPL)                                            \
  if (a.dtype == 0) {                                                    \
    switch (a.d) {                                                       \
      case 16: return IMPL<float, 16>(a, stream);                        \
      case 32: return IMPL<float, 32>(a, stream);                        \
      case 64: return IMPL<float, 64>(a, stream);                        \
    }                                                                    \
  } else {                                                               \
    switch (a.d) {                                                       \
      case 16: return IMPL<bf16_t, 16>(a, stream);                       \
      case 32: return IMPL<bf16_t, 32>(a, stream);                       \
      case 64: return IMPL<bf16_t, 64>(a, stream);                       \
    }                                                                    \
  }                                                                      \
  return hipErrorInvalidValue;

hipError_t launch_pla_fwd_general(const PlaArgs& a, hipStream_t stream) { AFFMAE_DISPATCH(fwd_impl) }
hipError_t launch_pla_bwd_general(const PlaArgs& a, hipStream_t stream) { AFFMAE_DISPATCH(bwd_impl) }

}  // namespace affmae
