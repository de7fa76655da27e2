// Dense projections of the DiT block: C = epi(A . B^T + bias).
//
// A [M][K] activations and B [N][K] weights are both K-contiguous, so every
// MFMA operand is eight consecutive bf16 of one row.  bf16 path: workgroup
// tile BM x BN x 64, waves arranged WM x WN, each wave a grid of 32x32x16
// MFMA tiles with fp32 accumulators; A/B tiles double-buffered in LDS with a
// 16-byte-chunk XOR swizzle (chunk ^ lds_swz(row)) so the column reads of the
// MFMA operand layout are spread over all banks.  Workgroup ids are remapped
// so that each XCD (dispatch round-robins over 8) receives a contiguous run
// of tiles, grouped GROUP_M tile-rows deep, to share its L2.
// Epilogues (bias, tanh-GELU, gated residual) are fused into the store.
// Split K: when the output tiles cannot fill the 256 CUs (few rows, or a
// narrow N), grid.y workgroups share a tile along K, store fp32 partial sums,
// and one memory-bound pass sums them and applies the epilogue (or the
// epilogue and the LayerNorm that follows: launch_splitk_ln).
// Short token sets run the ring kernel of k_ring.hip instead (plan_gemm).
#include "gemm_common.h"
#include "score_unit.h"

#include <algorithm>

namespace swam {

// ---------------------------------------------------------------------------
// bf16 MFMA kernel
// ---------------------------------------------------------------------------
// one k-stage (64) of MFMAs from a staged A/B tile pair.  The operand
// fragments of k-step s + 1 are read from LDS while the MFMAs of k-step s
// run (two fragment sets), and the schedule interleaves one LDS read after
// each MFMA so the reads never queue behind a whole MFMA group.
template <int BM, int BN, int TM, int TN, int FM, int FN>
__device__ __forceinline__ void mma_stage(const uint4* __restrict__ as, const uint4* __restrict__ bs,
                                          int wm, int wn, int lane, f32x16 (&acc)[FM][FN]) {
  constexpr int KS = GEMM_BK / 16;
  // fragment reads of the next k-step paired with this k-step's MFMAs; with
  // fewer MFMAs than reads (the 96 x 32 wave tile) the rest follow as a group
  constexpr int PAIRS = FM * FN < FM + FN ? FM * FN : FM + FN;
  const int khalf = lane >> 5, r31 = lane & 31;
  const int sw = lds_swz(r31);   // rows differ from r31 by multiples of 32
  bf16x8 af[2][FM], bfr[2][FN];
  auto load = [&](int s, int buf) {
    const int chunk = (2 * s + khalf) ^ sw;
#pragma unroll
    for (int i = 0; i < FM; ++i)
      af[buf][i] = __builtin_bit_cast(bf16x8, as[(wm * TM + i * 32 + r31) * 8 + chunk]);
#pragma unroll
    for (int j = 0; j < FN; ++j)
      bfr[buf][j] = __builtin_bit_cast(bf16x8, bs[(wn * TN + j * 32 + r31) * 8 + chunk]);
  };
  load(0, 0);
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    if (s + 1 < KS) load(s + 1, (s + 1) & 1);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[s & 1][i], bfr[s & 1][j], acc[i][j],
                                                            0, 0, 0);
  }
  // schedule: the first fragment set, then per k-step (MFMA, LDS read) pairs
  // for the next set followed by the remaining MFMAs; the last k-step's MFMAs
  __builtin_amdgcn_sched_group_barrier(0x100, FM + FN, 0);
#pragma unroll
  for (int s = 0; s + 1 < KS; ++s) {
#pragma unroll
    for (int r = 0; r < PAIRS; ++r) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    if constexpr (FM + FN > PAIRS)
      __builtin_amdgcn_sched_group_barrier(0x100, FM + FN - PAIRS, 0);
    if constexpr (FM * FN > PAIRS)
      __builtin_amdgcn_sched_group_barrier(0x008, FM * FN - PAIRS, 0);
  }
  __builtin_amdgcn_sched_group_barrier(0x008, FM * FN, 0);
}

// Stage loads go global -> LDS directly (no registers) as buffer loads: each
// instruction moves 8 rows x 128 bytes; lane i lands at slot i of the 1 KB
// slab, i.e. row lane >> 3 and physical chunk lane & 7, so it fetches logical
// chunk (lane & 7) ^ lds_swz(row) -- the swizzle is applied on the global
// side.  The descriptors start at the tile's first row and end at the last
// row of the operand, so the rows of a ragged last tile read as zeros (the
// hardware range check) and every offset stays below 2^31.  A wave's slabs
// are 8 rows apart; only bit 3 of the row enters the swizzle, so two
// per-lane offsets (even / odd slab) plus a wave-uniform step address them
// all.
// ROLE (a GemmRole) only names the instantiation after the block's
// projection, so a kernel trace tells the four projections apart.
// SC: workgroups past the tile count (the grid's tail) score one layer
// instead (scoring units of score_unit.h, two per 8-wave workgroup at a time),
// on the CUs that the last round of tiles leaves idle; sa / n_units describe
// that work.
template <int ROLE, int BM, int BN, int WM, int WN, int EPI, bool SC = false>
__global__ void __launch_bounds__(WM * WN * 64)
gemm_bf16_nt(const bf16_t* __restrict__ A, int64_t lda, const bf16_t* __restrict__ B,
             int64_t ldb, const bf16_t* __restrict__ bias, const float* __restrict__ gate,
             bf16_t* C, int64_t ldc, int M, int N, int K, int tiles_m, int tiles_n,
             float* __restrict__ part, const QkPost qp, const ScoreArgs sa, int n_units,
             bf16_t* Cs, const int32_t* __restrict__ smap) {
  constexpr int NW = WM * WN;
  constexpr int TM = BM / WM, TN = BN / WN;
  constexpr int FM = TM / 32, FN = TN / 32;
  constexpr int A_INS = BM / 8 / NW, B_INS = BN / 8 / NW;
  static_assert(A_INS * 8 * NW == BM && B_INS * 8 * NW == BN, "tile/waves mismatch");
  __shared__ uint4 lds[2 * (BM + BN) * 8];   // [stage][A rows | B rows][8 chunks]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform
  const int n_tiles = tiles_m * tiles_n;
  if constexpr (SC) {
    static_assert(NW % 4 == 0, "scoring units take groups of four waves");
    if ((int)blockIdx.x >= n_tiles) {
      constexpr int G = NW / 4;
      const int group = wave >> 2;
      float (*sp)[16] = reinterpret_cast<float (*)[16]>(lds) + 4 * group;
      const int nsw = (int)gridDim.x - n_tiles;
      for (int base = ((int)blockIdx.x - n_tiles) * G; base < n_units; base += nsw * G) {
        __syncthreads();                 // the previous units' partial sums are consumed
        const int unit = base + group;
        score_unit_bf16(sa, unit, unit < n_units, wave & 3, lane, tid & 255, sp,
                        [] { __syncthreads(); });
      }
      return;
    }
  }
  int tm, tn;
  tile_of(blockIdx.x, n_tiles, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int wm = wave / WN, wn = wave % WN;
  const int lrow = lane >> 3;

  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(A + (int64_t)m0 * lda), (short)0,
      (int)min((int64_t)(M - m0) * lda * 2, (int64_t)0x7fffffff), SWAM_BUF_DWORD3);
  const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(B + (int64_t)n0 * ldb), (short)0,
      (int)min((int64_t)(N - n0) * ldb * 2, (int64_t)0x7fffffff), SWAM_BUF_DWORD3);
  // With an even slab count per wave, a wave's slabs start on a multiple of
  // 16 rows, so two offsets (even / odd slab) plus a 16-row step address them
  // all.  With an odd count bit 3 of a slab's first row alternates with the
  // wave, so every slab keeps its own offset.
  constexpr int NA = A_INS % 2 == 0 ? 2 : A_INS, NB = B_INS % 2 == 0 ? 2 : B_INS;
  int va[NA], vb[NB];
  if constexpr (A_INS % 2 == 0 && B_INS % 2 == 0) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int ch = (lane & 7) ^ lds_swz(8 * p + lrow);
      va[p] = (int)(((int64_t)(wave * A_INS * 8 + 8 * p + lrow) * lda + 8 * ch) * 2);
      vb[p] = (int)(((int64_t)(wave * B_INS * 8 + 8 * p + lrow) * ldb + 8 * ch) * 2);
    }
  } else {
#pragma unroll
    for (int p = 0; p < NA; ++p) {
      const int r = wave * A_INS * 8 + 8 * p + lrow;
      const int ch = (lane & 7) ^ lds_swz(A_INS % 2 == 0 ? 8 * p + lrow : r);
      va[p] = (int)(((int64_t)r * lda + 8 * ch) * 2);
    }
#pragma unroll
    for (int p = 0; p < NB; ++p) {
      const int r = wave * B_INS * 8 + 8 * p + lrow;
      const int ch = (lane & 7) ^ lds_swz(B_INS % 2 == 0 ? 8 * p + lrow : r);
      vb[p] = (int)(((int64_t)r * ldb + 8 * ch) * 2);
    }
  }
  const int step_a = (int)(16 * lda * 2), step_b = (int)(16 * ldb * 2);
  auto issue = [&](uint4* as, uint4* bs, int k0) {
#pragma unroll
    for (int j = 0; j < A_INS; ++j) {
      int off;
      if constexpr (A_INS % 2 == 0) off = vadd_sgpr(va[j & 1], (j >> 1) * step_a + k0 * 2);
      else off = vadd_sgpr(va[j], k0 * 2);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void_t*)(as + (wave * A_INS + j) * 64), 16,
                                               off, 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < B_INS; ++j) {
      int off;
      if constexpr (B_INS % 2 == 0) off = vadd_sgpr(vb[j & 1], (j >> 1) * step_b + k0 * 2);
      else off = vadd_sgpr(vb[j], k0 * 2);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_void_t*)(bs + (wave * B_INS + j) * 64), 16,
                                               off, 0, 0, 0);
    }
  };

  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  constexpr int CPR = TN / 8;                         // 8-column runs per row of a wave's columns
  constexpr int EP_IT = (32 * CPR + 63) / 64;         // runs per lane and 32-row slice
  int pos[EPI == EPI_BIAS_QKPOST ? FM : 1][EP_IT];    // rotary positions of the lane's rows
  if constexpr (EPI == EPI_BIAS_QKPOST)
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int it = 0; it < EP_IT; ++it)
        pos[i][it] = qkpost_pos(m0 + wm * TM + i * 32 + (lane + 64 * it) / CPR, M, qp);

  constexpr int STAGE = (BM + BN) * 8;
  // k-stages of this workgroup: all of them, or split slice blockIdx.y of gridDim.y
  const int KT_all = K / GEMM_BK;
  const int kt0 = (int)((int64_t)KT_all * blockIdx.y / gridDim.y);
  const int KT = (int)((int64_t)KT_all * (blockIdx.y + 1) / gridDim.y);
  issue(lds, lds + BM * 8, kt0 * GEMM_BK);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  for (int kt = kt0; kt < KT; ++kt) {
    uint4* cur = lds + ((kt - kt0) & 1) * STAGE;
    uint4* nxt = lds + ((kt - kt0 + 1) & 1) * STAGE;
    // prefetch stage kt + 1 into the other buffer (released by the previous barrier)
    if (kt + 1 < KT) issue(nxt, nxt + BM * 8, (kt + 1) * GEMM_BK);
    mma_stage<BM, BN, TM, TN, FM, FN>(cur, cur + BM * 8, wm, wn, lane, acc);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  }

  // Epilogue through LDS (the stage buffers are free after the last barrier):
  // each wave parks one 32-row slice of its tile as fp32, then every lane
  // handles 8 consecutive columns with 16-byte loads (bias, gate, residual) and
  // a 16-byte store, so each 8 lanes write one contiguous 128-byte row run.
  // A lane's column run is the same in every row it handles, so its bias and
  // gate are loaded once, and each slice's residual rows are requested one
  // slice ahead (one exposed memory latency per tile, not one per slice).
  constexpr int EP_LD = TN + 4;                       // fp32 row pitch of the staging slice
  static_assert((32 * CPR) % 64 == 0, "every lane handles whole runs");
  static_assert(EPI != EPI_BIAS_QKPOST || TN == 64, "a wave's columns must be one head");
  static_assert(NW * 32 * EP_LD * 4 <= (int)sizeof(lds), "epilogue staging exceeds LDS");
  float* stage = reinterpret_cast<float*>(lds) + wave * 32 * EP_LD;
  const int col0 = n0 + wn * TN;
  const int cl = (lane % CPR) * 8, col = col0 + cl;  // 64 is a multiple of CPR
  const bool col_ok = col < N;
  uint32_t bb[4] = {0u, 0u, 0u, 0u};
  float gg[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  uint4 res[2][EP_IT];                                // residual runs of slices i and i + 1
  auto load_res = [&](int i, uint4 (&r)[EP_IT]) {
#pragma unroll
    for (int it = 0; it < EP_IT; ++it) {
      const int row = m0 + wm * TM + i * 32 + (lane + 64 * it) / CPR;
      r[it] = (row < M && col_ok) ? *reinterpret_cast<const uint4*>(C + (int64_t)row * ldc + col)
                                  : make_uint4(0u, 0u, 0u, 0u);
    }
  };
  if constexpr (EPI != EPI_PARTIAL && EPI != EPI_BIAS_QKPOST) {
    if (col_ok) {
      const uint4 bw = *reinterpret_cast<const uint4*>(bias + col);
      bb[0] = bw.x; bb[1] = bw.y; bb[2] = bw.z; bb[3] = bw.w;
      if constexpr (EPI == EPI_BIAS_GATED_RESIDUAL) {
        const float4 g0 = *reinterpret_cast<const float4*>(gate + col);
        const float4 g1 = *reinterpret_cast<const float4*>(gate + col + 4);
        gg[0] = g0.x; gg[1] = g0.y; gg[2] = g0.z; gg[3] = g0.w;
        gg[4] = g1.x; gg[5] = g1.y; gg[6] = g1.z; gg[7] = g1.w;
      }
    }
    if constexpr (EPI == EPI_BIAS_GATED_RESIDUAL) load_res(0, res[0]);
  }
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    // the next slice's residual rows are requested before this slice is parked
    if constexpr (EPI == EPI_BIAS_GATED_RESIDUAL)
      if (i + 1 < FM) load_res(i + 1, res[(i + 1) & 1]);
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        stage[(8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * EP_LD + j * 32 + (lane & 31)] =
            acc[i][j][r];
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_s_waitcnt(0xc07f);                 // lgkmcnt(0): slice visible to the wave
    __builtin_amdgcn_wave_barrier();
    const int row0 = m0 + wm * TM + i * 32;
#pragma unroll
    for (int it = 0; it < EP_IT; ++it) {
      const int rl = (lane + 64 * it) / CPR;
      const int row = row0 + rl;
      if constexpr (EPI == EPI_BIAS_QKPOST) {
        qkpost_store(stage + rl * EP_LD + cl, bias, C, ldc, row, col, col0, M, N, pos[i][it], qp);
        continue;
      }
      if (EPI == EPI_PARTIAL && row < M && col_ok) {
        // fp32 partial sums of this K slice: part[slice][M][N]
        float* q = part + ((int64_t)blockIdx.y * M + row) * N + col;
        reinterpret_cast<float4*>(q)[0] = *reinterpret_cast<const float4*>(stage + rl * EP_LD + cl);
        reinterpret_cast<float4*>(q)[1] = *reinterpret_cast<const float4*>(stage + rl * EP_LD + cl + 4);
      } else if (EPI != EPI_PARTIAL && row < M && col_ok) {
        const float4 v0 = *reinterpret_cast<const float4*>(stage + rl * EP_LD + cl);
        const float4 v1 = *reinterpret_cast<const float4*>(stage + rl * EP_LD + cl + 4);
        const float v[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
        uint32_t rr[4] = {0u, 0u, 0u, 0u};
        if constexpr (EPI == EPI_BIAS_GATED_RESIDUAL) {
          const uint4 rw = res[i & 1][it];
          rr[0] = rw.x; rr[1] = rw.y; rr[2] = rw.z; rr[3] = rw.w;
        }
        uint32_t out[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float b0 = __uint_as_float(bb[e] << 16), b1 = __uint_as_float(bb[e] & 0xFFFF0000u);
          const float x0 = __uint_as_float(rr[e] << 16), x1 = __uint_as_float(rr[e] & 0xFFFF0000u);
          out[e] = pack_bf16x2(epi_value<EPI>(v[2 * e], b0, gg[2 * e], x0),
                               epi_value<EPI>(v[2 * e + 1], b1, gg[2 * e + 1], x1));
        }
        bf16_t* dst = C + (int64_t)row * ldc + col;
        if constexpr (EPI == EPI_BIAS_GATED_RESIDUAL)
          if (smap != nullptr) dst = Cs + (int64_t)smap[row] * ldc + col;
        *reinterpret_cast<uint4*>(dst) = make_uint4(out[0], out[1], out[2], out[3]);
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// Sum of the split-K partials and the epilogue: one thread per 8 columns of
// a row (16-byte loads and stores).
template <int ROLE, typename T, int EPI>
__global__ void __launch_bounds__(256)
splitk_epilogue(const float* __restrict__ part, int splits, int M, int N,
                const T* __restrict__ bias, const float* __restrict__ gate, T* C,
                int64_t ldc, T* Cs, const int32_t* __restrict__ smap) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int cpr = N / 8;
  if (id >= (int64_t)M * cpr) return;
  const int row = (int)(id / cpr), col = (int)(id % cpr) * 8;
  float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int z = 0; z < splits; ++z) {
    float q[8];
    load8(part + ((int64_t)z * M + row) * N + col, q);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] += q[e];
  }
  float bb[8], gg[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float rr[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  load8(bias + col, bb);
  T* dst = C + (int64_t)row * ldc + col;
  if (EPI == EPI_BIAS_GATED_RESIDUAL) {
    load8(dst, rr);
    load8(gate + col, gg);
    if (smap != nullptr) dst = Cs + (int64_t)smap[row] * ldc + col;
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = epi_value<EPI>(v[e], bb[e], gg[e], rr[e]);
  store8(dst, v);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
template <int ROLE, int BM, int BN, int WM, int WN, int EPI>
static hipError_t run_bf16(const void* A, int64_t lda, const void* B, int64_t ldb,
                           const void* bias, const float* gate, void* C, int64_t ldc, int M,
                           int N, int K, int splits, float* part, hipStream_t st,
                           const QkPost& qp = QkPost{}, void* Cs = nullptr,
                           const int32_t* smap = nullptr) {
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  if (splits <= 1) {
    hipLaunchKernelGGL((gemm_bf16_nt<ROLE, BM, BN, WM, WN, EPI>), dim3(tiles_m * tiles_n),
                       dim3(WM * WN * 64), 0, st, (const bf16_t*)A, lda, (const bf16_t*)B, ldb,
                       (const bf16_t*)bias, gate, (bf16_t*)C, ldc, M, N, K, tiles_m, tiles_n,
                       (float*)nullptr, qp, ScoreArgs{}, 0, (bf16_t*)Cs, smap);
    return hipGetLastError();
  }
  if constexpr (EPI == EPI_BIAS_QKPOST) {
    return hipErrorNotSupported;             // no split-K store with the QK post-processing
  } else {
    hipLaunchKernelGGL((gemm_bf16_nt<ROLE, BM, BN, WM, WN, EPI_PARTIAL>), dim3(tiles_m * tiles_n, splits),
                       dim3(WM * WN * 64), 0, st, (const bf16_t*)A, lda, (const bf16_t*)B, ldb,
                       (const bf16_t*)bias, gate, (bf16_t*)C, ldc, M, N, K, tiles_m, tiles_n, part,
                       QkPost{}, ScoreArgs{}, 0, (bf16_t*)nullptr, (const int32_t*)nullptr);
    return hipGetLastError();
  }
}

// Tile and K-split choice by modelled time: n rounds of a pipeline fill plus a
// step per 64 columns of K, and the pass over the partial sums when K is split.
// The 256x256 and 192x256 kernels fit one workgroup per CU and run in whole
// rounds of 256; two 128x128 or 192x128 workgroups share a CU and start as soon
// as a slot frees, so their rounds count in halves once a grid spills past one
// slot per CU, and a lone workgroup per CU takes 0.6 of a shared round.  The
// constants (us) are a fit to the four projections of d = 512, 1,088, 1,536 and
// 2,048 at 16 row counts from 1,100 to 17,472: choosing by this model and the
// ring kernel's runs within 0.5% of the best measured plan on average; one MFMA
// efficiency per tile and no fill, as used before, lost 5.7% (out projection at
// 1,400 x 1,536: 22.4 us on 128x128 tiles against 16.2 on the ring; down at
// 3,688: 192x128 without a split 87 us, 192x256 with two slices 68.9 and a pass
// that is the next LayerNorm's).
struct GemmPlan { int tile, splits; bool ring; double us; };
constexpr int GEMM_TILES = 4;
static const int TILE_BM[GEMM_TILES] = {256, 128, 192, 192};
static const int TILE_BN[GEMM_TILES] = {256, 128, 256, 128};
static const int TILE_PER_CU[GEMM_TILES] = {1, 2, 1, 2};
// wide_only: only tiles whose waves span 64 columns, without a split (the QK
// post-processing store needs one head per wave); ln_follows: the pass over the
// partial sums is the LayerNorm launch that follows anyway (3,472 x 1,536, three
// slices: 14 us against the 7.5 us of the LayerNorm it replaces)
static double split_pass_us(int splits, int64_t M, int64_t N, bool ln_follows) {
  if (splits <= 1) return 0.0;
  return ln_follows ? 0.5 + (double)splits * M * N * 4.0 / 5.0e6
                    : 3.0 + (double)(splits + 1) * M * N * 4.0 / 5.0e6;
}
static GemmPlan choose_gemm(int64_t M, int64_t N, int64_t K, int64_t ws_floats, bool ln_follows,
                            bool wide_only = false) {
  // 3 us of t0 stand for weights read cold, as the ring kernel's constants are
  const double t0[GEMM_TILES] = {6.14, 6.15, 4.46, 5.81}, fill[GEMM_TILES] = {4.23, 5.66, 6.45, 5.03},
               step[GEMM_TILES] = {1.55, 0.95, 1.209, 1.302}, lone[GEMM_TILES] = {1.0, 0.628, 1.0, 0.605};
  const int split_opts[6] = {1, 2, 3, 4, 6, 8};
  const int64_t kt = K / GEMM_BK;
  GemmPlan best{0, 1, false, 1e30};
  for (int i = 0; i < GEMM_TILES; ++i) {
    if (wide_only && i == 3) continue;
    const int64_t tiles = ((M + TILE_BM[i] - 1) / TILE_BM[i]) * ((N + TILE_BN[i] - 1) / TILE_BN[i]);
    for (int s : split_opts) {
      if (s > 1 && (wide_only || kt / s < 4 || (int64_t)s * M * N > ws_floats)) continue;
      const int64_t wgs = tiles * s;
      double n;
      if (TILE_PER_CU[i] == 1) n = (double)((wgs + 255) / 256);
      else if (wgs <= 256) n = lone[i];
      else n = std::max((double)wgs / 512.0, (double)((wgs + 255) / 256) / 2.0);
      double us = t0[i] + n * (fill[i] + step[i] * (double)((kt + s - 1) / s));
      // alone, the smaller tiles are level with 256x256 at the same modelled time;
      // within a step their extra operand traffic costs 3-5% (QKV at 12,059 rows:
      // 202 us on 192x128 against 192)
      if (i != 0) us *= 1.03;
      us += split_pass_us(s, M, N, ln_follows);
      if (us < best.us) best = {i, s, false, us};
    }
  }
  return best;
}

// The ring kernel's time for a plan: 256 CUs take `n` workgroups each (two
// share a CU's loads, so n counts them all), a workgroup costs a fill plus a
// step per 64 columns of K (a fifth more once the CUs run out of step), and
// split partial sums a pass of their own (shorter when the pass is the
// LayerNorm launch that follows anyway).  The constants are a fit to 350
// shapes with the weights read cold (M 64 .. 10,200, d 384 .. 2,048): choosing
// by the two models runs within 0.5% of the best measured plan on average
// (d = 1536, 192 rows: 11.0 / 10.7 / 14.0 / 17.7 us for QKV / out / up / down
// against 19.5 / 14.6 / 23.0 / 21.6 of the tile kernels, which win from about
// 1,000 rows at d = 1536, down projections from about 3,000).
constexpr int RING_BM[RING_TILES] = {64, 64, 128, 128};
constexpr int RING_BN[RING_TILES] = {64, 128, 64, 128};
// fp32 has no other kernel; its steps are bound by the fp32 matrix rate.
static GemmPlan choose_ring(int dtype, int64_t M, int64_t N, int64_t K, int64_t ws_floats,
                            bool ln_follows, int max_splits) {
  const double t0[RING_TILES] = {4.0, 4.8, 4.8, 1.5}, fill[RING_TILES] = {0.33, 0.17, 0.19, 3.5};
  const double step16[RING_TILES] = {0.215, 0.392, 0.392, 0.51},
               step32[RING_TILES] = {0.55, 1.05, 1.05, 2.1};
  const double* step = dtype == 1 ? step16 : step32;
  const int split_opts[6] = {1, 2, 3, 4, 6, 8};
  const int64_t kt = K / (dtype == 1 ? GEMM_BK : GEMM_BK / 2);
  GemmPlan best{0, 1, true, 1e30};
  for (int i = 0; i < RING_TILES; ++i) {
    const int64_t tiles = ((M + RING_BM[i] - 1) / RING_BM[i]) * ((N + RING_BN[i] - 1) / RING_BN[i]);
    for (int s : split_opts) {
      if (s > max_splits || (s > 1 && (kt / s < 4 || (int64_t)s * M * N > ws_floats))) continue;
      const int64_t n = (tiles * s + 255) / 256;
      double us = t0[i] + n * (fill[i] + step[i] * (double)((kt + s - 1) / s)) * (n > 1 ? 1.21 : 1.0);
      us += split_pass_us(s, M, N, ln_follows);
      if (us < best.us) best = {i, s, true, us};
    }
  }
  return best;
}

// the plan of one bf16 projection; ln_follows: a LayerNorm of the result is
// next (out and down projections)
static GemmPlan plan_gemm(int64_t M, int64_t N, int64_t K, int64_t ws_floats, bool ln_follows) {
  const GemmPlan c = choose_gemm(M, N, K, ws_floats, ln_follows);
  const GemmPlan r = choose_ring(1, M, N, K, ws_floats, ln_follows, 8);
  return r.us < c.us ? r : c;
}

template <int ROLE, typename T, int EPI>
static hipError_t run_epilogue(const float* ws, int splits, int M, int N, const void* bias,
                               const float* gate, void* C, int64_t ldc, void* Cs,
                               const int32_t* smap, hipStream_t st) {
  const int64_t n = (int64_t)M * (N / 8);
  hipLaunchKernelGGL((splitk_epilogue<ROLE, T, EPI>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                     ws, splits, M, N, (const T*)bias, gate, (T*)C, ldc, (T*)Cs, smap);
  return hipGetLastError();
}

// after a projection of `splits` K slices: the sum and epilogue, with the
// LayerNorm that follows where the caller asks for it
template <int ROLE, typename T, int EPI>
static hipError_t finish_splits(const float* ws, int splits, int M, int N, const void* bias,
                                const float* gate, void* C, int64_t ldc, void* Cs,
                                const int32_t* smap, LnNext* ln, hipStream_t st) {
  if (splits <= 1) return hipSuccess;
  if (ln == nullptr || N > LN_ROW_MAX)
    return run_epilogue<ROLE, T, EPI>(ws, splits, M, N, bias, gate, C, ldc, Cs, smap, st);
  ln->done = true;
  return launch_splitk_ln(sizeof(T) == 2, ws, splits, M, N, bias, gate, C, ln->h, ln->shift, ln->scale, st, ln->pf);
}

// ln (out and down projections): a LayerNorm of the result into ln->h follows;
// it shares the pass that sums the splits when K is split
template <int ROLE, int EPI>
static hipError_t dispatch_bf16(const void* A, int64_t lda, const void* B, int64_t ldb,
                                const void* bias, const float* gate, void* C, int64_t ldc,
                                int M, int N, int K, float* ws, int64_t ws_floats,
                                hipStream_t st, void* Cs = nullptr,
                                const int32_t* smap = nullptr, LnNext* ln = nullptr) {
  const GemmPlan p = plan_gemm(M, N, K, ws ? ws_floats : 0, ln != nullptr);
  hipError_t e;
  if (p.ring) {
    const RingArgs a{A, lda, B, ldb, bias, gate, C, ldc, M, N, K, ws, QkPost{}, Cs, smap};
    e = launch_ring(1, ROLE, a, {p.tile, p.splits}, st);
  } else if (p.tile == 0) {
    e = run_bf16<ROLE, 256, 256, 2, 4, EPI>(A, lda, B, ldb, bias, gate, C, ldc, M, N, K, p.splits, ws, st, QkPost{}, Cs, smap);
  } else if (p.tile == 2) {
    e = run_bf16<ROLE, 192, 256, 2, 4, EPI>(A, lda, B, ldb, bias, gate, C, ldc, M, N, K, p.splits, ws, st, QkPost{}, Cs, smap);
  } else if (p.tile == 3) {
    e = run_bf16<ROLE, 192, 128, 2, 4, EPI>(A, lda, B, ldb, bias, gate, C, ldc, M, N, K, p.splits, ws, st, QkPost{}, Cs, smap);
  } else {
    e = run_bf16<ROLE, 128, 128, 2, 2, EPI>(A, lda, B, ldb, bias, gate, C, ldc, M, N, K, p.splits, ws, st, QkPost{}, Cs, smap);
  }
  if (e != hipSuccess) return e;
  return finish_splits<ROLE, bf16_t, EPI>(ws, p.splits, M, N, bias, gate, C, ldc, Cs, smap, ln, st);
}

// The MLP up projection with one layer's scoring in the tail of its grid:
// the scoring workgroups are dispatched after every tile, i.e. into the last
// round, on the CUs its tiles leave idle there (at least 16 of them, or the
// caller scores on its side stream instead).
static int scored_idle_slots(const GemmPlan& p, int64_t M, int64_t N) {
  if (p.ring) return 0;
  const int bm = TILE_BM[p.tile], bn = TILE_BN[p.tile];
  if (p.splits != 1) return 0;
  const int64_t tiles = ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
  const int64_t slots = 256 * TILE_PER_CU[p.tile];
  const int64_t idle = (slots - tiles % slots) % slots;
  return idle >= 16 ? (int)idle : 0;
}

// the plan of a scored up projection: the ring kernel has no scoring tail, so
// it is taken only where it saves more than the events that the scoring on
// the side stream needs instead (about 8 us)
static GemmPlan plan_up_scored(int64_t M, int64_t N, int64_t K, int64_t ws_floats) {
  const GemmPlan p = plan_gemm(M, N, K, ws_floats, false), c = choose_gemm(M, N, K, ws_floats, false);
  return p.ring && scored_idle_slots(c, M, N) > 0 && c.us < p.us + 8.0 ? c : p;
}

int gemm_up_scored_slots(int64_t M, int64_t N, int64_t K, int64_t ws_floats) {
  if (M <= 0) return 0;
  return scored_idle_slots(plan_up_scored(M, N, K, ws_floats), M, N);
}

template <int BM, int BN, int WM, int WN>
static hipError_t run_up_scored(const void* A, int64_t lda, const void* B, int64_t ldb,
                                const void* bias, void* C, int64_t ldc, int M, int N, int K,
                                const ScoreArgs& sa, int n_sw, hipStream_t st) {
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  const int ktiles = (sa.n_s + 15) / 16;
  const int n_units = (sa.n_layers < 1 ? 1 : sa.n_layers) * sa.B * sa.F * ktiles;
  constexpr int G = WM * WN / 4;
  n_sw = std::min(n_sw, (n_units + G - 1) / G);
  hipLaunchKernelGGL((gemm_bf16_nt<ROLE_UP, BM, BN, WM, WN, EPI_BIAS_GELU, true>),
                     dim3(tiles_m * tiles_n + n_sw), dim3(WM * WN * 64), 0, st, (const bf16_t*)A,
                     lda, (const bf16_t*)B, ldb, (const bf16_t*)bias, (const float*)nullptr,
                     (bf16_t*)C, ldc, M, N, K, tiles_m, tiles_n, (float*)nullptr, QkPost{}, sa,
                     n_units, (bf16_t*)nullptr, (const int32_t*)nullptr);
  return hipGetLastError();
}

hipError_t launch_gemm_up_scored(const void* A, int64_t lda, const void* B, int64_t ldb,
                                 const void* bias, void* C, int64_t ldc, int64_t M, int64_t N,
                                 int64_t K, const ScoreArgs& sa, hipStream_t st,
                                 int64_t ws_floats) {
  if (M <= 0) return hipSuccess;
  const GemmPlan p = plan_up_scored(M, N, K, ws_floats);
  const int n_sw = scored_idle_slots(p, M, N);
  if (n_sw == 0) return hipErrorNotSupported;
  const int m = (int)M, n = (int)N, k = (int)K;
  if (p.tile == 0) return run_up_scored<256, 256, 2, 4>(A, lda, B, ldb, bias, C, ldc, m, n, k, sa, n_sw, st);
  if (p.tile == 2) return run_up_scored<192, 256, 2, 4>(A, lda, B, ldb, bias, C, ldc, m, n, k, sa, n_sw, st);
  if (p.tile == 3) return run_up_scored<192, 128, 2, 4>(A, lda, B, ldb, bias, C, ldc, m, n, k, sa, n_sw, st);
  return run_up_scored<128, 128, 2, 2>(A, lda, B, ldb, bias, C, ldc, m, n, k, sa, n_sw, st);
}

template <int ROLE, int EPI>
static hipError_t run_f32(const void* A, int64_t lda, const void* B, int64_t ldb,
                          const void* bias, const float* gate, void* C, int64_t ldc, int M,
                          int N, int K, float* ws, int64_t ws_floats, LnNext* ln, hipStream_t st) {
  const GemmPlan p = choose_ring(0, M, N, K, ws ? ws_floats : 0, ln != nullptr, 8);
  const RingArgs a{A, lda, B, ldb, bias, gate, C, ldc, M, N, K, ws, QkPost{}, nullptr, nullptr};
  const hipError_t e = launch_ring(0, ROLE, a, {p.tile, p.splits}, st);
  if (e != hipSuccess) return e;
  return finish_splits<ROLE, float, EPI>(ws, p.splits, M, N, bias, gate, C, ldc, nullptr, nullptr, ln, st);
}

hipError_t launch_gemm(int dtype, int role, const void* A, int64_t lda, const void* B,
                       int64_t ldb, const void* bias, const float* gate, void* C,
                       int64_t ldc, int64_t M, int64_t N, int64_t K, hipStream_t st,
                       float* ws, int64_t ws_floats, void* Cs, const int32_t* smap,
                       LnNext* ln) {
  if (M <= 0) return hipSuccess;
  if (ln != nullptr && ((role != ROLE_OUT && role != ROLE_DOWN) || smap != nullptr || ldc != N))
    return hipErrorNotSupported;             // LayerNorm of the plain residual stream only
  const int m = (int)M, n = (int)N, k = (int)K;
  if (smap != nullptr && (dtype != 1 || (role != ROLE_OUT && role != ROLE_DOWN) || Cs == nullptr))
    return hipErrorNotSupported;             // row scatter: bf16 gated-residual stores only
  if (dtype == 1) {
    switch (role) {
      case ROLE_QKV: return dispatch_bf16<ROLE_QKV, EPI_BIAS>(A, lda, B, ldb, bias, gate, C, ldc, m, n, k, ws, ws_floats, st);
      case ROLE_UP: return dispatch_bf16<ROLE_UP, EPI_BIAS_GELU>(A, lda, B, ldb, bias, gate, C, ldc, m, n, k, ws, ws_floats, st);
      case ROLE_OUT: return dispatch_bf16<ROLE_OUT, EPI_BIAS_GATED_RESIDUAL>(A, lda, B, ldb, bias, gate, C, ldc, m, n, k, ws, ws_floats, st, Cs, smap, ln);
      case ROLE_DOWN: return dispatch_bf16<ROLE_DOWN, EPI_BIAS_GATED_RESIDUAL>(A, lda, B, ldb, bias, gate, C, ldc, m, n, k, ws, ws_floats, st, Cs, smap, ln);
      default: return hipErrorInvalidValue;
    }
  }
  switch (role) {
    case ROLE_QKV: return run_f32<ROLE_QKV, EPI_BIAS>(A, lda, B, ldb, bias, gate, C, ldc, m, n, k, ws, ws_floats, nullptr, st);
    case ROLE_UP: return run_f32<ROLE_UP, EPI_BIAS_GELU>(A, lda, B, ldb, bias, gate, C, ldc, m, n, k, ws, ws_floats, nullptr, st);
    case ROLE_OUT: return run_f32<ROLE_OUT, EPI_BIAS_GATED_RESIDUAL>(A, lda, B, ldb, bias, gate, C, ldc, m, n, k, ws, ws_floats, ln, st);
    case ROLE_DOWN: return run_f32<ROLE_DOWN, EPI_BIAS_GATED_RESIDUAL>(A, lda, B, ldb, bias, gate, C, ldc, m, n, k, ws, ws_floats, ln, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_gemm_qkv(int dtype, const void* A, int64_t lda, const void* B, int64_t ldb,
                           const void* bias, void* C, int64_t ldc, int64_t M, int64_t N,
                           int64_t K, const QkPost& qp, hipStream_t st, float* ws,
                           int64_t ws_floats) {
  if (M <= 0) return hipSuccess;
  const bool post = qp.qk_norm || qp.tab != nullptr;
  if (dtype == 1 && post) {
    const GemmPlan p = choose_gemm(M, N, K, 0, false, true);
    const int m = (int)M, n = (int)N, k = (int)K;
    const GemmPlan r = choose_ring(1, M, N, K, 0, false, 1);
    if (r.us < p.us) {
      const RingArgs a{A, lda, B, ldb, bias, nullptr, C, ldc, m, n, k, nullptr, qp, nullptr, nullptr};
      return launch_ring(1, ROLE_QKV, a, {r.tile, 1}, st);
    }
    if (p.tile == 0)
      return run_bf16<ROLE_QKV, 256, 256, 2, 4, EPI_BIAS_QKPOST>(A, lda, B, ldb, bias, nullptr, C, ldc, m, n, k, 1, nullptr, st, qp);
    if (p.tile == 2)
      return run_bf16<ROLE_QKV, 192, 256, 2, 4, EPI_BIAS_QKPOST>(A, lda, B, ldb, bias, nullptr, C, ldc, m, n, k, 1, nullptr, st, qp);
    return run_bf16<ROLE_QKV, 128, 128, 2, 2, EPI_BIAS_QKPOST>(A, lda, B, ldb, bias, nullptr, C, ldc, m, n, k, 1, nullptr, st, qp);
  }
  const hipError_t e = launch_gemm(dtype, ROLE_QKV, A, lda, B, ldb, bias, nullptr, C, ldc, M, N, K,
                                   st, ws, ws_floats);
  if (e != hipSuccess || !post) return e;
  return launch_qk_post((float*)C, M, qp.d, qp.pos_mode, qp.gather, qp.cu, qp.n_seqs, qp.l_full, qp.tab,
                        qp.n_pos, qp.qk_norm, st);
}

}  // namespace swam
