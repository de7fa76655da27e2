// Internal device helpers and types shared by the HIP sources of libswam
// (gfx950 only).  The host-side launcher declarations and their argument
// structs are in launchers.h.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define SWAM_SEL_MAXNP 4096   // selection sort capacity (next power of two >= N_s)
#define SWAM_MAX_NS_DEV 4096

namespace swam {

typedef uint16_t bf16_t;  // raw bf16 storage

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ float bf16_to_f32(bf16_t v) {
  return __uint_as_float(((uint32_t)v) << 16);
}

// Round to nearest even: one v_cvt_pk_bf16_f32 per pair (the same rounding in
// integer arithmetic takes nine VALU instructions).
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  return __builtin_bit_cast(bf16_t, (__bf16)f);
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  bf16x2 v;
  v[0] = (__bf16)lo;
  v[1] = (__bf16)hi;
  return __builtin_bit_cast(uint32_t, v);
}

// Physical 16-byte chunk of logical chunk c in row r of an LDS tile with
// 128-byte rows is c ^ lds_swz(r).  The LDS serves a ds_read_b128 in phases
// of 16 lanes and a 64-bit read in phases of 32 lanes over 64 four-byte banks;
// with this swizzle 16 consecutive rows at one logical chunk (the MFMA operand
// reads) and the transposed 64-bit reads of 8 rows x 64 bytes both hit every
// bank once per phase.  Only row bits 1..3 matter.
__device__ __forceinline__ int lds_swz(int r) {
  return ((r >> 1) & 3) | ((((r >> 1) ^ (r >> 3)) & 1) << 2);
}

template <typename T> struct Elem;
template <> struct Elem<float> {
  __device__ __forceinline__ static float load(const float* p) { return *p; }
  __device__ __forceinline__ static void store(float* p, float v) { *p = v; }
};
template <> struct Elem<bf16_t> {
  __device__ __forceinline__ static float load(const bf16_t* p) { return bf16_to_f32(*p); }
  __device__ __forceinline__ static void store(bf16_t* p, float v) { *p = f32_to_bf16(v); }
};

// 8 consecutive elements of a 16-byte aligned T row as fp32, and back
template <typename T>
__device__ __forceinline__ void load8(const T* p, float (&o)[8]) {
  if constexpr (sizeof(T) == 2) {
    const uint4 u = *reinterpret_cast<const uint4*>(p);
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      o[2 * e] = __uint_as_float(w[e] << 16);
      o[2 * e + 1] = __uint_as_float(w[e] & 0xFFFF0000u);
    }
  } else {
    const float4 a = reinterpret_cast<const float4*>(p)[0], b = reinterpret_cast<const float4*>(p)[1];
    o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w; o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
  }
}
template <typename T>
__device__ __forceinline__ void store8(T* p, const float (&v)[8]) {
  if constexpr (sizeof(T) == 2) {
    *reinterpret_cast<uint4*>(p) = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                                              pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
  } else {
    reinterpret_cast<float4*>(p)[0] = make_float4(v[0], v[1], v[2], v[3]);
    reinterpret_cast<float4*>(p)[1] = make_float4(v[4], v[5], v[6], v[7]);
  }
}

// Weights that a later launch reads, touched by spare workgroups of this one so
// that they come out of the caches there (p NULL: nothing to do).
struct Prefetch {
  const void* p = nullptr;
  int64_t bytes = 0;
};
// workgroup wg of n reads its share of q, 8 16-byte loads per thread in flight
__device__ __forceinline__ void prefetch_share(const Prefetch& q, int wg, int n) {
  const uint4* w = (const uint4*)q.p;
  const int64_t chunks = q.bytes / 16, step = (int64_t)n * blockDim.x;
  for (int64_t i = (int64_t)wg * blockDim.x + threadIdx.x; i < chunks; i += 8 * step) {
    uint4 v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = w[i + e * step < chunks ? i + e * step : i];
#pragma unroll
    for (int e = 0; e < 8; ++e) asm volatile("" ::"v"(v[e].x), "v"(v[e].y), "v"(v[e].z), "v"(v[e].w));
  }
}

__device__ __forceinline__ float warp_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}
__device__ __forceinline__ float warp_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}
__device__ __forceinline__ double warp_sum_d(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

}  // namespace swam
