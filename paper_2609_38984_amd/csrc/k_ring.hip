// Projections of short token sets, C = epi(A . B^T + bias) with M up to a few
// thousand rows (bf16), and every fp32 projection.
//
// What bounds these is not the matrix cores but the read of the weights (a
// 192-row block of d = 1536 does 10.9 GFLOP on 57 MB of weights): a two-stage
// tile loop waits out one memory round trip per 64 columns of K with 16 KB in
// flight per workgroup.  Here the A and B tiles of NST k-stages of 64 form a
// ring in LDS; the DMA loads of stage kt + NST - 1 are issued before stage kt
// is multiplied and a counted vmcnt wait leaves the NST - 2 younger stages in
// flight: 48-64 KB per workgroup are on their way while a stage is multiplied
// (up to 96 KB on a CU that holds two workgroups), 24-32 KB during the wait.
//
// Tile (64 WM) x (64 WN): every wave holds a 64 x 64 accumulator block (four
// 32x32x16 MFMAs per 16 columns of K) and the WK waves of one block take
// different 16-column slices of each stage, so no operand fragment is read by
// two waves of a block; their sums meet in LDS in a fixed order in the
// epilogue.
// fp32: the same ring, tiles and LDS layout with 16-byte chunks of four floats
// (stages of 32 columns); a lane's chunk of A and of B feeds four 32x32x2 MFMAs,
// one column pair (c, c + 4) each, so the sums stay fp32 products in fp32
// accumulators.  Bound by the fp32 matrix rate (157 TFLOP/s nominal).
// `splits` > 1: that many workgroups share a tile along K and store fp32
// partial sums (EPI_PARTIAL) for splitk_epilogue or splitk_ln.
#include "gemm_common.h"

#include <algorithm>

namespace swam {

// wait until at most V vector-memory operations and no LDS operation of this
// wave are outstanding (vmcnt in bits 3:0 and 15:14, lgkmcnt in bits 11:8);
// the empty asm statements keep the compiler's memory operations on their side
template <int V>
__device__ __forceinline__ void wait_stage() {
  static_assert(V >= 0 && V < 64, "vmcnt is a 6-bit counter");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((V & 15) | (7 << 4) | ((V >> 4) << 14));
  asm volatile("" ::: "memory");
}

// one DMA instruction: 16 bytes per lane from the buffer at `off` to a 1 KB LDS slab
__device__ __forceinline__ void dma_slab(__amdgpu_buffer_rsrc_t r, uint4* slab, int off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t*)slab, 16, off, 0, 0, 0);
}

// acc += A B^T for one 16-byte chunk per lane of a 32-row A and B fragment.  The
// fragments are values of the vector type: read through a pointer to the LDS
// words the compiler waits for every DMA load in flight before each stage.
__device__ __forceinline__ void mma_chunk(bf16x8 a, bf16x8 b, f32x16& acc) {
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
}
__device__ __forceinline__ void mma_chunk(f32x4 a, f32x4 b, f32x16& acc) {
#pragma unroll
  for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e], acc, 0, 0, 0);
}
template <typename T> struct Chunk { typedef f32x4 type; };
template <> struct Chunk<bf16_t> { typedef bf16x8 type; };

template <int ROLE, typename T, int WM, int WN, int WK, int NST, int EPI>
__global__ void __launch_bounds__(WM * WN * WK * 64)
gemm_ring(const T* __restrict__ A, int64_t lda, const T* __restrict__ B, int64_t ldb,
          const T* __restrict__ bias, const float* __restrict__ gate, T* C, int64_t ldc,
          int M, int N, int K, int tiles_m, int tiles_n, int splits, float* __restrict__ part,
          const QkPost qp, T* Cs, const int32_t* __restrict__ smap) {
  constexpr int EPC = 16 / (int)sizeof(T), BK = 8 * EPC;   // elements per chunk, columns per stage
  constexpr int NW = WM * WN * WK, BM = 64 * WM, BN = 64 * WN;
  constexpr int A_INS = BM / 8 / NW, B_INS = BN / 8 / NW, INS = A_INS + B_INS;
  static_assert(A_INS * 8 * NW == BM && B_INS * 8 * NW == BN, "tile/waves mismatch");
  static_assert(4 % WK == 0, "the waves of a block split the four k-steps of a stage");
  constexpr int STAGE = (BM + BN) * 8;
  constexpr int EP_LD = 68;                           // fp32 row pitch of a staged 32 x 64 slice
  constexpr int RING = NST * STAGE, EPI_SLOTS = NW * 32 * EP_LD / 4;
  __shared__ uint4 ring[RING > EPI_SLOTS ? RING : EPI_SLOTS];   // [stage][A rows | B rows][8 chunks]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wk = wave % WK, wn = (wave / WK) % WN, wm = wave / (WK * WN);
  const int n_tiles = tiles_m * tiles_n;
  // consecutive ids per XCD, K slices slowest: the row tiles that read the
  // same weights run on one XCD
  const int nwg = n_tiles * splits, pid = blockIdx.x;
  const int xcd = pid & 7, per = nwg >> 3, rem = nwg & 7;
  const int id = xcd * per + min(xcd, rem) + (pid >> 3);
  const int z = id / n_tiles, t = id - z * n_tiles;
  const int in_group = GROUP_M * tiles_n, group = t / in_group, first_m = group * GROUP_M;
  const int gsz = min(tiles_m - first_m, GROUP_M);
  const int tm = first_m + (t % in_group) % gsz, tn = (t % in_group) / gsz;
  const int m0 = tm * BM, n0 = tn * BN;
  const int KT_all = K / BK;
  const int kt0 = KT_all * z / splits;
  const int KT = KT_all * (z + 1) / splits;

  // descriptors end with the tile's last valid row: rows of a ragged tile read
  // as zeros, and so does every load of a stage past KT (offset DEAD)
  constexpr int DEAD = 0x40000000;
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(A + (int64_t)m0 * lda), (short)0, (int)(min(M - m0, BM) * lda * (int)sizeof(T)), SWAM_BUF_DWORD3);
  const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(B + (int64_t)n0 * ldb), (short)0, (int)(min(N - n0, BN) * ldb * (int)sizeof(T)), SWAM_BUF_DWORD3);
  const int lrow = lane >> 3;
  int va[A_INS], vb[B_INS];
#pragma unroll
  for (int j = 0; j < A_INS; ++j) {
    const int r = (wave * A_INS + j) * 8 + lrow;
    va[j] = (int)(r * lda * (int)sizeof(T)) + 16 * ((lane & 7) ^ lds_swz(r));
  }
#pragma unroll
  for (int j = 0; j < B_INS; ++j) {
    const int r = (wave * B_INS + j) * 8 + lrow;
    vb[j] = (int)(r * ldb * (int)sizeof(T)) + 16 * ((lane & 7) ^ lds_swz(r));
  }
  auto issue = [&](int slot, int kt) {
    const int k2 = kt < KT ? kt * 128 : DEAD;
    uint4* as = ring + slot * STAGE;
#pragma unroll
    for (int j = 0; j < B_INS; ++j)
      dma_slab(rb, as + BM * 8 + (wave * B_INS + j) * 64, vadd_sgpr(vb[j], k2));
#pragma unroll
    for (int j = 0; j < A_INS; ++j)
      dma_slab(ra, as + (wave * A_INS + j) * 64, vadd_sgpr(va[j], k2));
  };

  // epilogue operands, requested ahead of the ring so that their latency is
  // not exposed after it: a lane stores runs of 8 columns (8 lanes per row),
  // the same columns in every run
  constexpr int RUNS = 4 / WK;                        // runs per lane and 32-row slice
  const int col = n0 + wn * 64 + (lane & 7) * 8;
  const bool col_ok = col < N;
  float gg[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  constexpr int VEC = (int)sizeof(T) / 2;             // 16-byte pieces of a run
  uint4 bw[VEC], res[2][RUNS][VEC];                   // unconverted: nothing waits for them yet
  int pos[2][RUNS];                                   // rotary positions of the lane's rows
  if constexpr (EPI == EPI_BIAS_QKPOST)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int it = 0; it < RUNS; ++it)
        pos[i][it] = qkpost_pos(m0 + wm * 64 + i * 32 + (wk * RUNS + it) * 8 + (lane >> 3), M, qp);
  if constexpr (EPI != EPI_PARTIAL && EPI != EPI_BIAS_QKPOST) {
#pragma unroll
    for (int p = 0; p < VEC; ++p)
      bw[p] = col_ok ? reinterpret_cast<const uint4*>(bias + col)[p] : make_uint4(0u, 0u, 0u, 0u);
    if constexpr (EPI == EPI_BIAS_GATED_RESIDUAL) {
      if (col_ok) load8(gate + col, gg);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int it = 0; it < RUNS; ++it) {
          const int row = m0 + wm * 64 + i * 32 + (wk * RUNS + it) * 8 + (lane >> 3);
#pragma unroll
          for (int p = 0; p < VEC; ++p)
            res[i][it][p] = (row < M && col_ok) ? reinterpret_cast<const uint4*>(C + (int64_t)row * ldc + col)[p]
                                                : make_uint4(0u, 0u, 0u, 0u);
        }
    }
  }

  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

#pragma unroll
  for (int p = 0; p < NST - 1; ++p) issue(p, kt0 + p);
  const int khalf = lane >> 5, r31 = lane & 31, sw = lds_swz(r31);
  int slot = 0, fill = NST - 1;
  for (int kt = kt0; kt < KT; ++kt) {
    // own loads of stage kt have landed and own reads of stage kt - 1 are done;
    // after the barrier so are everyone's, which frees slot `fill` (stage kt - 1)
    wait_stage<(NST - 2) * INS>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    issue(fill, kt + NST - 1);
    const uint4* as = ring + slot * STAGE + wm * 64 * 8;
    const uint4* bs = ring + slot * STAGE + (BM + wn * 64) * 8;
#pragma unroll
    for (int q = 0; q < 4 / WK; ++q) {
      const int chunk = (2 * (wk * (4 / WK) + q) + khalf) ^ sw;
      typename Chunk<T>::type af[2], bf[2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
        af[i] = __builtin_bit_cast(typename Chunk<T>::type, as[(i * 32 + r31) * 8 + chunk]);
#pragma unroll
      for (int j = 0; j < 2; ++j)
        bf[j] = __builtin_bit_cast(typename Chunk<T>::type, bs[(j * 32 + r31) * 8 + chunk]);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) mma_chunk(af[i], bf[j], acc[i][j]);
    }
    slot = slot + 1 == NST ? 0 : slot + 1;
    fill = fill + 1 == NST ? 0 : fill + 1;
  }
  wait_stage<0>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");

  // epilogue: 32-row slices of the WK partial blocks through LDS, summed in
  // block order
  float* stage = reinterpret_cast<float*>(ring);
  float bb[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if constexpr (EPI != EPI_PARTIAL && EPI != EPI_BIAS_QKPOST) load8(reinterpret_cast<const T*>(bw), bb);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    float* own = stage + wave * 32 * EP_LD;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        own[(8 * (r >> 2) + 4 * khalf + (r & 3)) * EP_LD + j * 32 + r31] = acc[i][j][r];
    __syncthreads();
#pragma unroll
    for (int it = 0; it < RUNS; ++it) {
      const int rl = (wk * RUNS + it) * 8 + (lane >> 3);
      const int row = m0 + wm * 64 + i * 32 + rl;
      float v[8];
#pragma unroll
      for (int p = 0; p < WK; ++p) {
        const float* q = stage + (((wm * WN + wn) * WK + p) * 32 + rl) * EP_LD + (lane & 7) * 8;
        const float4 a = reinterpret_cast<const float4*>(q)[0], b = reinterpret_cast<const float4*>(q)[1];
        const float w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = p == 0 ? w[e] : v[e] + w[e];
      }
      if constexpr (EPI == EPI_BIAS_QKPOST) {
        static_assert(sizeof(T) == 2, "the QK post-processing store is bf16");
        qkpost_store(v, bias, C, ldc, row, col, n0 + wn * 64, M, N, pos[i][it], qp);
      } else if (row < M && col_ok) {
        if constexpr (EPI == EPI_PARTIAL) {
          float* q = part + ((int64_t)z * M + row) * N + col;
          reinterpret_cast<float4*>(q)[0] = make_float4(v[0], v[1], v[2], v[3]);
          reinterpret_cast<float4*>(q)[1] = make_float4(v[4], v[5], v[6], v[7]);
        } else {
          T* dst = C + (int64_t)row * ldc + col;
          float rr[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
          if constexpr (EPI == EPI_BIAS_GATED_RESIDUAL) {
            load8(reinterpret_cast<const T*>(res[i][it]), rr);
            if (smap != nullptr) dst = Cs + (int64_t)smap[row] * ldc + col;
          }
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = epi_value<EPI>(v[e], bb[e], gg[e], rr[e]);
          store8(dst, v);
        }
      }
    }
    if (i == 0) __syncthreads();
  }
}

template <int ROLE, typename T, int WM, int WN, int WK, int NST, int EPI>
static hipError_t run_ring(const RingArgs& a, int splits, hipStream_t st) {
  const int tiles_m = (a.M + 64 * WM - 1) / (64 * WM), tiles_n = (a.N + 64 * WN - 1) / (64 * WN);
  hipLaunchKernelGGL((gemm_ring<ROLE, T, WM, WN, WK, NST, EPI>), dim3(tiles_m * tiles_n * splits),
                     dim3(WM * WN * WK * 64), 0, st, (const T*)a.A, a.lda, (const T*)a.B, a.ldb,
                     (const T*)a.bias, a.gate, (T*)a.C, a.ldc, a.M, a.N, a.K, tiles_m, tiles_n,
                     splits, a.part, a.qp, (T*)a.Cs, a.smap);
  return hipGetLastError();
}

template <int ROLE, typename T, int EPI>
static hipError_t run_ring_tile(const RingPlan& p, const RingArgs& a, hipStream_t st) {
  switch (p.tile) {
    case RING_64x64: return run_ring<ROLE, T, 1, 1, 4, 4, EPI>(a, p.splits, st);
    case RING_64x128: return run_ring<ROLE, T, 1, 2, 2, 3, EPI>(a, p.splits, st);
    case RING_128x64: return run_ring<ROLE, T, 2, 1, 2, 3, EPI>(a, p.splits, st);
    case RING_128x128: return run_ring<ROLE, T, 2, 2, 2, 3, EPI>(a, p.splits, st);
    default: return hipErrorInvalidValue;
  }
}

template <int ROLE, typename T, int EPI>
static hipError_t run_ring_role(const RingPlan& p, const RingArgs& a, hipStream_t st) {
  if (p.splits > 1) return run_ring_tile<ROLE, T, EPI_PARTIAL>(p, a, st);
  if constexpr (ROLE == ROLE_QKV && sizeof(T) == 2)
    if (a.qp.qk_norm || a.qp.tab != nullptr) return run_ring_tile<ROLE, T, EPI_BIAS_QKPOST>(p, a, st);
  return run_ring_tile<ROLE, T, EPI>(p, a, st);
}

template <typename T>
static hipError_t launch_ring_t(int role, const RingArgs& a, const RingPlan& p, hipStream_t st) {
  switch (role) {
    case ROLE_QKV: return run_ring_role<ROLE_QKV, T, EPI_BIAS>(p, a, st);
    case ROLE_UP: return run_ring_role<ROLE_UP, T, EPI_BIAS_GELU>(p, a, st);
    case ROLE_OUT: return run_ring_role<ROLE_OUT, T, EPI_BIAS_GATED_RESIDUAL>(p, a, st);
    case ROLE_DOWN: return run_ring_role<ROLE_DOWN, T, EPI_BIAS_GATED_RESIDUAL>(p, a, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_ring(int dtype, int role, const RingArgs& a, const RingPlan& p, hipStream_t st) {
  return dtype == 1 ? launch_ring_t<bf16_t>(role, a, p, st) : launch_ring_t<float>(role, a, p, st);
}

}  // namespace swam
