// Internal device helpers shared by the HIP kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace affmae {

constexpr int kWave = 64;

typedef uint16_t bf16_t;  // bfloat16 bit pattern

__device__ __forceinline__ float bf16_to_f32(bf16_t x) { return __uint_as_float(((uint32_t)x) << 16); }

// Round to nearest, ties to even.  NaN stays NaN (quiet bit forced).
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)((u >> 16) | 0x0040u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}

template <typename T>
struct Elem;
template <>
struct Elem<float> {
  static __device__ __forceinline__ float load(const float* p) { return *p; }
  static __device__ __forceinline__ void store(float* p, float v) { *p = v; }
};
template <>
struct Elem<bf16_t> {
  static __device__ __forceinline__ float load(const bf16_t* p) { return bf16_to_f32(*p); }
  static __device__ __forceinline__ void store(bf16_t* p, float v) { *p = f32_to_bf16(v); }
};

// Load D contiguous elements (row start aligned to 16 bytes) into fp32 registers.
template <int D>
__device__ __forceinline__ void load_row(const float* p, float (&r)[D]) {
  const float4* p4 = reinterpret_cast<const float4*>(p);
#pragma unroll
  for (int t = 0; t < D / 4; ++t) {
    float4 x = p4[t];
    r[4 * t + 0] = x.x;
    r[4 * t + 1] = x.y;
    r[4 * t + 2] = x.z;
    r[4 * t + 3] = x.w;
  }
}
template <int D>
__device__ __forceinline__ void load_row(const bf16_t* p, float (&r)[D]) {
  const uint4* p4 = reinterpret_cast<const uint4*>(p);
#pragma unroll
  for (int t = 0; t < D / 8; ++t) {
    uint4 x = p4[t];
    uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      r[8 * t + 2 * e + 0] = __uint_as_float(w[e] << 16);
      r[8 * t + 2 * e + 1] = __uint_as_float(w[e] & 0xffff0000u);
    }
  }
}

// The word held by lane (lane ^ J), J a power of two, moved on the vector ALU: DPP lane
// patterns inside a row of 16 lanes, the gfx950 row / half swaps across rows.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_mov(uint32_t x) {
  // every pattern used here reads an existing lane, so no value is needed for lanes without a source: leaving it
  // undefined saves the instruction that would otherwise set it before every move
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xf, 0xf, true);
}
template <int J>
__device__ __forceinline__ uint32_t lane_xor_u32(uint32_t x, int lane) {
  typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
  if constexpr (J == 1) {
    return dpp_mov<0xB1>(x);  // quad_perm [1,0,3,2]
  } else if constexpr (J == 2) {
    return dpp_mov<0x4E>(x);  // quad_perm [2,3,0,1]
  } else if constexpr (J == 4) {
    return dpp_mov<0x1B>(dpp_mov<0x141>(x));  // reverse 8 lanes, then reverse each quad: i -> i ^ 7 ^ 3
  } else if constexpr (J == 8) {
    return dpp_mov<0x128>(x);  // rotate the row by 8
  } else if constexpr (J == 16) {
    const u32x2 t = __builtin_amdgcn_permlane16_swap(x, x, false, false);  // [0]: even rows doubled, [1]: odd rows
    return (lane & 16) ? t[0] : t[1];
  } else {
    const u32x2 t = __builtin_amdgcn_permlane32_swap(x, x, false, false);  // [0]: low half doubled, [1]: high half
    return (lane & 32) ? t[0] : t[1];
  }
}
// Sum over the lanes whose numbers differ in the bits LO .. HI (powers of two), largest distance first, every lane
// receiving it; all lanes of the wave must be active.  Through the LDS crossbar (shuffles) each step would wait for a
// trip to LDS and back.
template <int LO, int HI>
__device__ __forceinline__ float lanes_sum(float x, int lane) {
  if constexpr (LO <= HI) {
    x += __uint_as_float(lane_xor_u32<HI>(__float_as_uint(x), lane));
    x = lanes_sum<LO, HI / 2>(x, lane);
  }
  return x;
}
template <int LO, int HI>
__device__ __forceinline__ float lanes_max(float x, int lane) {
  if constexpr (LO <= HI) {
    x = fmaxf(x, __uint_as_float(lane_xor_u32<HI>(__float_as_uint(x), lane)));
    x = lanes_max<LO, HI / 2>(x, lane);
  }
  return x;
}
__device__ __forceinline__ float wave_max(float x) { return lanes_max<1, 32>(x, threadIdx.x & (kWave - 1)); }
__device__ __forceinline__ float wave_sum(float x) { return lanes_sum<1, 32>(x, threadIdx.x & (kWave - 1)); }

// *out = part[lo] + ... + part[hi - 1] by a workgroup of 1024 threads, in an order that is the same in every launch; part + lo is
// 16-byte aligned, `acc` LDS.
__device__ __forceinline__ void sum_parts(const float* __restrict__ part, size_t lo, size_t hi, float (&acc)[16], float* out) {
  float s = 0.f;
  const size_t n4 = (hi - lo) / 4;  // whole 16-byte pieces first
  for (size_t i = threadIdx.x; i < n4; i += 1024) {
    const float4 v = reinterpret_cast<const float4*>(part + lo)[i];
    s += (v.x + v.y) + (v.z + v.w);
  }
  for (size_t i = lo + n4 * 4 + threadIdx.x; i < hi; i += 1024) s += part[i];
  s = wave_sum(s);
  if ((threadIdx.x & (kWave - 1)) == 0) acc[threadIdx.x / kWave] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = 0.f;
    for (int w = 0; w < 16; ++w) t += acc[w];
    *out = t;
  }
}

// Orders LDS traffic between the lanes of one wave (no workgroup barrier).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Cell of a relative-position table (paper, Sec. "AutoFocusFormer": relative position from the 2-D token
// coordinates): along each axis clamp(rint((nbr - query) * rate), -R, R), in fp32 one operation at a time, ties
// to even; cell = (by + R) * (2R + 1) + bx + R.  Every kernel that needs a cell calls this, so that all of them
// take the same integer decision.  The clamped offsets are small integers held in fp32, so combining them with
// one fused multiply-add is exact; a NaN offset lands on -R (the median instruction returns the minimum then).
__device__ __forceinline__ float relpos_axis(float nbr, float query, float rate, float Rf) {
#pragma clang fp contract(off)
  const float d = nbr - query;
  const float t = d * rate;
  return __builtin_amdgcn_fmed3f(__builtin_rintf(t), -Rf, Rf);
}
__device__ __forceinline__ int relpos_cell(float2 nbr, float2 query, float rate, int R) {
  const float Rf = (float)R;
  const float c = __builtin_fmaf(relpos_axis(nbr.y, query.y, rate, Rf), (float)(2 * R + 1),
                                 relpos_axis(nbr.x, query.x, rate, Rf));
  return (int)c + (R * (2 * R + 1) + R);
}

}  // namespace affmae
