// Shared pieces of the bf16 projection kernels: the fused epilogue functions,
// the workgroup-to-tile map and the buffer-to-LDS addressing helpers.
#pragma once
#include "launchers.h"

namespace swam {

__device__ __forceinline__ float gelu_tanh(float u) {
  // 0.5 u (1 + tanh(z)) = u / (1 + exp(-2 z)), z = sqrt(2/pi) (u + 0.044715 u^3);
  // exp(-2z) = exp2(-2 log2(e) z) on the hardware exp2, then the hardware reciprocal
  // (both about 1 ulp: far below the bf16 rounding of the stored result)
  const float z2 = -2.0f * 1.4426950408889634f * 0.7978845608028654f *
                   (u + 0.044715f * u * u * u);
  return u * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(z2));
}

template <int EPI>
__device__ __forceinline__ float epi_value(float acc, float bias, float gate, float resid) {
  if (EPI == EPI_BIAS) return acc + bias;
  if (EPI == EPI_BIAS_GELU) return gelu_tanh(acc + bias);
  return resid + gate * (acc + bias);
}

// Rotary position of a row (0 without a table).  The kernels look the positions
// of their rows up before the k loop: behind it, the index and the table are two
// memory latencies in a row per slice of the store.
__device__ __forceinline__ int qkpost_pos(int row, int M, const QkPost& qp) {
  if (qp.tab == nullptr) return 0;
  const int rr = min(row, M - 1);
  int pos;
  if (qp.pos_mode == 0) {
    pos = rr % qp.l_full;
  } else if (qp.pos_mode == 1) {
    pos = qp.gather[rr] % qp.l_full;
  } else {
    int b = 0;
    while (b + 1 < qp.n_seqs && qp.cu[b + 1] <= rr) ++b;
    pos = rr - qp.cu[b];
  }
  return min(max(pos, 0), qp.n_pos - 1);
}

// Store of 8 consecutive QKV columns of one row with the QK-norm / rotary
// embedding of q and k heads applied (the steps of qk_post_kernel on the
// projection rounded to bf16).  The 8 lanes storing one row's 64 columns are
// consecutive and aligned, and a wave's 64 columns are one head, so the head
// norm is a 3-step exchange; every lane takes part (the store is guarded).
__device__ __forceinline__ void qkpost_store(const float* v, const bf16_t* __restrict__ bias,
                                             bf16_t* C, int64_t ldc, int row, int col, int col0,
                                             int M, int N, int pos, const QkPost& qp) {
  float x[8];
  {
    const float4 v0 = *reinterpret_cast<const float4*>(v);
    const float4 v1 = *reinterpret_cast<const float4*>(v + 4);
    const float a[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
    uint4 bw = make_uint4(0u, 0u, 0u, 0u);
    if (col < N) bw = *reinterpret_cast<const uint4*>(bias + col);
    const uint32_t bb[4] = {bw.x, bw.y, bw.z, bw.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      // the projection is stored (rounded to bf16) before the post-processing
      x[2 * e] = bf16_to_f32(f32_to_bf16(a[2 * e] + __uint_as_float(bb[e] << 16)));
      x[2 * e + 1] = bf16_to_f32(f32_to_bf16(a[2 * e + 1] + __uint_as_float(bb[e] & 0xFFFF0000u)));
    }
  }
  if (col0 < 2 * qp.d) {                      // q or k head (wave-uniform)
    if (qp.qk_norm) {
      float ss = 0.0f;
#pragma unroll
      for (int e = 0; e < 8; ++e) ss = fmaf(x[e], x[e], ss);
      ss += __shfl_xor(ss, 1);
      ss += __shfl_xor(ss, 2);
      ss += __shfl_xor(ss, 4);
      const float r = rsqrtf(ss / 64.0f + 1e-6f);
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] *= r;
    }
    if (qp.tab != nullptr) {
      const float2* t = qp.tab + (int64_t)pos * 32 + ((col & 63) >> 1);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float2 cs = t[e];
        const float a = x[2 * e], b = x[2 * e + 1];
        x[2 * e] = a * cs.x - b * cs.y;
        x[2 * e + 1] = a * cs.y + b * cs.x;
      }
    }
  }
  if (row < M && col < N)
    *reinterpret_cast<uint4*>(C + (int64_t)row * ldc + col) =
        make_uint4(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(x[4], x[5]),
                   pack_bf16x2(x[6], x[7]));
}

constexpr int GEMM_BK = 64;
constexpr int GROUP_M = 8;

__device__ __forceinline__ void tile_of(int pid, int nwg, int tiles_m, int tiles_n, int& tm,
                                        int& tn) {
  // XCD remap: ids with equal (pid % 8) run on one XCD; give them consecutive ids.
  const int xcd = pid & 7;
  const int per = nwg >> 3, rem = nwg & 7;
  const int id = xcd * per + min(xcd, rem) + (pid >> 3);
  const int in_group = GROUP_M * tiles_n;
  const int group = id / in_group;
  const int first_m = group * GROUP_M;
  const int gsz = min(tiles_m - first_m, GROUP_M);
  tm = first_m + (id % in_group) % gsz;
  tn = (id % in_group) / gsz;
}

typedef __attribute__((address_space(3))) void lds_void_t;

// dword 3 of a raw buffer descriptor on gfx9-family parts (32-bit data format)
constexpr int SWAM_BUF_DWORD3 = 0x00020000;

// per-lane offset + wave-uniform step, formed at the point of use: an asm add
// keeps the compiler from hoisting one live VGPR per slab out of the k loop
__device__ __forceinline__ int vadd_sgpr(int v, int s) {
  int r;
  asm volatile("v_add_u32 %0, %1, %2" : "=v"(r) : "s"(s), "v"(v));
  return r;
}

// Ring kernel (k_ring.hip): tiles, arguments and launcher.
enum RingTile { RING_64x64 = 0, RING_64x128, RING_128x64, RING_128x128, RING_TILES };
struct RingPlan { int tile, splits; };
struct RingArgs {
  const void* A; int64_t lda;
  const void* B; int64_t ldb;
  const void* bias;
  const float* gate;
  void* C; int64_t ldc;
  int M, N, K;
  float* part;                 // [splits][M][N] partial sums when splits > 1
  QkPost qp;                   // bf16 QKV only
  void* Cs; const int32_t* smap;
};
// one projection of role `role` (GemmRole); splits > 1 leaves the partial sums
// in a.part and the epilogue to the caller
hipError_t launch_ring(int dtype, int role, const RingArgs& a, const RingPlan& p, hipStream_t st);

}  // namespace swam
