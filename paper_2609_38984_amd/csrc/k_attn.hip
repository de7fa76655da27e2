// Softmax attention of the DiT block over the keys of each (dense or packed)
// sequence, writing O and the natural-log normaliser lambda of every query
// row and head (the normaliser the scorer reuses).
//
// bf16 path, one head per workgroup, 4 or 8 waves x 32 query rows:
//   S^T = K Q^T with 32x32x16 MFMA: K (64-key tile, LDS) is the A operand and
//   the wave's 32 query rows are the B operand held in registers, so the C
//   layout gives each lane ONE query (lane & 31) and 16 of every 32 keys;
//   the other 16 sit in lane ^ 32.  Row max / sum are in-lane plus one swap.
//   O^T = V^T P^T: P^T straight from the S^T accumulators is the B operand
//   (no shuffle); the V^T operand comes from transposed LDS reads of the
//   row-major V tile.  K and V tiles are DMA'd global -> LDS (no register
//   staging), double-buffered.  Online softmax in the log2 domain with the
//   1/8 scale folded into one FMA, tail-only masking and lazy rescaling.
// fp32 path: 32 query rows of one head per workgroup, its four waves taking
// every fourth 32-key tile, both products on 32x32x2 fp32 MFMAs.
#include "launchers.h"

#include <cfloat>
#include <type_traits>

namespace swam {

constexpr int ATT_BK = 64;      // keys per tile

template <int BQ>
__device__ __forceinline__ bool find_tile(const int32_t* cu, int n_seqs, int n_rows, int t,
                                          int& s0, int& s1, int& q0) {
  for (int b = 0; b < n_seqs; ++b) {
    const int e = min(max(cu[b + 1], 0), n_rows);
    const int a = min(max(cu[b], 0), e);
    const int nt = (e - a + BQ - 1) / BQ;
    if (t < nt) { s0 = a; s1 = e; q0 = a + t * BQ; return true; }
    t -= nt;
  }
  return false;
}

typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) void glb_void_t;
typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16;

// NW waves x 32 query rows per workgroup; WPE = minimum waves per SIMD the
// register allocation must allow (4 caps it at 128 VGPRs); SUB 64-key tiles
// share one LDS stage, i.e. one barrier and one DMA wait.
// KS = 2: two groups of NW waves take every other stage of keys for the same
// query rows, each with its own stage buffers; their (max, sum, O) are merged
// through LDS in group order.  A workgroup alone on its CU is bound by the
// serial chain over its key tiles (one wave per SIMD hides neither the LDS
// reads nor the exponentials), so half the chain is worth the merge; four groups
// are slower again (1,312 rows x 16 heads, 13%).  The launcher has the figures.
template <int NW, int WPE, int SUB, int KS>
__global__ void __launch_bounds__(NW * KS * 64) __attribute__((amdgpu_waves_per_eu(WPE, 8)))
attn_fwd_bf16(const bf16_t* __restrict__ qkv, bf16_t* __restrict__ out, float* __restrict__ lse,
     const int32_t* __restrict__ cu, int n_seqs, int n_heads, int n_rows, int n_wg, const Prefetch pf0,
     const Prefetch pf1) {
  constexpr int S = 2;                           // LDS stages (K and V tiles)
  constexpr int SK = SUB * ATT_BK;               // keys per stage: SUB tiles per barrier
  __shared__ uint4 kv[2][KS][S][SK * 8];          // K | V: [key][8 chunks], chunk ^ lds_swz(key)
  const int nwg = n_wg, pid = blockIdx.x;
  if (pid >= nwg) {                              // spare workgroups past the grid's tiles
    prefetch_share(pf0, pid - nwg, gridDim.x - nwg);
    prefetch_share(pf1, pid - nwg, gridDim.x - nwg);
    return;
  }
  const int xcd = pid & 7, per = nwg >> 3, rem = nwg & 7;
  const int id = xcd * per + min(xcd, rem) + (pid >> 3);
  const int slots = nwg / n_heads;
  const int h = id / slots;
  int s0, s1, q0;
  constexpr int BQ = 32 * NW;
  if (!find_tile<BQ>(cu, n_seqs, n_rows, id - h * slots, s0, s1, q0)) return;
  const int d = n_heads * 64;
  const int64_t ld = 3 * (int64_t)d;
  const int tid = threadIdx.x, lane = tid & 63, wave = (tid >> 6) % NW;
  const int kg = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane((tid >> 6) / NW);   // key group
  uint4 (&Ks)[S][SK * 8] = kv[0][kg];
  uint4 (&Vs)[S][SK * 8] = kv[1][kg];
  const int g = lane >> 5;
  const int qrow = q0 + wave * 32 + (lane & 31);
  const bool qvalid = qrow < s1;
  bf16x8 qf[4];
  {
    const bf16_t* qp = qkv + (int64_t)min(qrow, s1 - 1) * ld + h * 64;
#pragma unroll
    for (int s = 0; s < 4; ++s) qf[s] = __builtin_bit_cast(bf16x8, *(const uint4*)(qp + 8 * (2 * s + g)));
  }
  // K and V tiles go global -> LDS directly, row-major with the chunk swizzle
  // applied on the global side: each instruction moves an 8-row slab (1 KB),
  // lane i landing in row i >> 3, physical chunk i & 7.
  // (element offsets stay below 2^31: the launcher checks n_rows * 3d)
  const int lrow = lane >> 3;
  const int ld32 = 3 * d;
  const bf16_t* kbase = qkv + d + h * 64;
  const bf16_t* vbase = qkv + 2 * d + h * 64;
  constexpr int SLABS = SK / 8 / NW;             // 8-row slabs per wave and stage
  static_assert(SLABS * 8 * NW == SK, "every wave stages whole 8-row slabs");
  int lofs[SLABS];
#pragma unroll
  for (int j = 0; j < SLABS; ++j) {
    const int r0 = (SK / NW) * wave + 8 * j;
    lofs[j] = 8 * ((lane & 7) ^ lds_swz((r0 & 8) + lrow));
  }
  auto issue = [&](int buf, int kb) {
#pragma unroll
    for (int j = 0; j < SLABS; ++j) {
      const int r0 = (SK / NW) * wave + 8 * j;
      const int e = min(kb + r0 + lrow, s1 - 1) * ld32 + lofs[j];
      __builtin_amdgcn_global_load_lds((glb_void_t*)(kbase + e), (lds_void_t*)(&Ks[buf][r0 * 8]), 16, 0, 0);
      __builtin_amdgcn_global_load_lds((glb_void_t*)(vbase + e), (lds_void_t*)(&Vs[buf][r0 * 8]), 16, 0, 0);
    }
  };
  // PV operand (V^T fragment) from transposed LDS reads: within each 16-lane
  // group, lane a addresses V[key0 + (a >> 2)][hd0 + 4 (a & 3)] and lane i
  // receives V[key0 .. key0+3][hd0 + i], i.e. four consecutive keys of one
  // head-dim column (the k order the P^T accumulators provide).
  const int a16 = lane & 15, G = lane >> 4;
  // loop-invariant part of those addresses: key 32t + 16u + rlo (+ 8 for the
  // second read), column hd = 32ht + 16 (G & 1) + 4 (a16 & 3); the swizzle
  // sees only key bits 1..3, i.e. rlo and the +8
  const int rlo = 4 * g + (a16 >> 2);
  int vofs[2][2];
#pragma unroll
  for (int ht = 0; ht < 2; ++ht)
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      const int r = rlo + 8 * hf;
      const int hd = 32 * ht + 16 * (G & 1) + 4 * (a16 & 3);
      vofs[ht][hf] = r * 64 + 8 * ((hd >> 3) ^ lds_swz(r)) + (hd & 7);
    }
  // K fragment (logical chunk 2 s + g of key lane & 31) offsets in a tile
  int kofs[4];
#pragma unroll
  for (int s = 0; s < 4; ++s)
    kofs[s] = (lane & 31) * 8 + ((2 * s + g) ^ lds_swz(lane & 31));
  f32x16 o[2];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[t][r] = 0.0f;
  float m_run = -1e30f, l_run = 0.0f;
  const float sc = 1.4426950408889634f * 0.125f;
  const int nkt = (s1 - s0 + SK - 1) / SK;       // stages
  if (kg < nkt) issue(0, s0 + kg * SK);
  // one 64-key tile of stage buffer `cur` at key offset sub * 64; full tiles
  // carry no masking code, the ragged last one runs a copy with the key mask
  auto tile = [&](int cur, int sub, int kb, auto masked) {
    const uint4* Kt = &Ks[cur][sub * ATT_BK * 8];
    auto scores = [&](f32x16 (&st)[2]) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int r = 0; r < 16; ++r) st[t][r] = 0.0f;
        // keys 32 t + (lane & 31): the swizzle sees the same row bits for both
        // halves, so the half is a constant offset of 32 rows
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          bf16x8 kf = __builtin_bit_cast(bf16x8, Kt[kofs[s] + t * 32 * 8]);
          st[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[s], st[t], 0, 0, 0);
        }
      }
      if constexpr (decltype(masked)::value) {
        const int nvalid = s1 - kb;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int key = 32 * t + 8 * (r >> 2) + 4 * g + (r & 3);
            if (key >= nvalid) st[t][r] = -INFINITY;
          }
      }
    };
    // probabilities against the running max.  Their row sum bounds every one
    // of them, so a sum above 2^8 is the only case in which the running max
    // must move (lazy rescaling: each p stays <= 2^8 otherwise); the scores
    // are then recomputed (K is still staged) and the tile is redone against
    // the new max.  The first tile of a row always takes that path (the
    // running max starts at -1e30).
    bf16x8 pf[2][2];
    float psum0, psum1;
    auto probs = [&](const f32x16 (&st)[2]) {
      psum0 = 0.0f; psum1 = 0.0f;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int mm = 0; mm < 8; mm += 2) {
            const float p0 = __builtin_amdgcn_exp2f(fmaf(st[t][8 * u + mm], sc, -m_run));
            const float p1 = __builtin_amdgcn_exp2f(fmaf(st[t][8 * u + mm + 1], sc, -m_run));
            // row sums from the fp32 probabilities (the exported normaliser)
            psum0 += p0; psum1 += p1;
            pf[t][u][mm] = (__bf16)p0; pf[t][u][mm + 1] = (__bf16)p1;
          }
    };
    {
      f32x16 st[2];
      scores(st);
      probs(st);
    }
    if (__any(!(psum0 + psum1 <= 256.0f))) {
      // re-read K from LDS rather than keeping the first pass's fragments live
      asm volatile("" ::: "memory");
      f32x16 st[2];
      scores(st);
      float mx = st[0][0];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, st[t][r]);
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float m_new = fmaxf(m_run, mx * sc);
      const float corr = __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= corr;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t][r] *= corr;
      probs(st);
    }
    l_run += psum0 + psum1;
    const unsigned short* vs = reinterpret_cast<const unsigned short*>(&Vs[cur][sub * ATT_BK * 8]);
#pragma unroll
    for (int ht = 0; ht < 2; ++ht) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int e1 = vofs[ht][0] + (32 * t + 16 * u) * 64;
          const int e2 = vofs[ht][1] + (32 * t + 16 * u) * 64;
          const v4i16 x1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(vs + e1));
          const v4i16 x2 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(vs + e2));
          const uint2 w1 = __builtin_bit_cast(uint2, x1), w2 = __builtin_bit_cast(uint2, x2);
          const bf16x8 vf = __builtin_bit_cast(bf16x8, make_uint4(w1.x, w1.y, w2.x, w2.y));
          o[ht] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[t][u], o[ht], 0, 0, 0);
        }
    }
  };
  // iteration `it` of this group: stage it * KS + kg (none past the last one,
  // but every group keeps the barriers)
  static_assert(S == 2, "the prefetch goes to the other buffer");
  auto stage = [&](int it, auto masked) {
    const int cur = it & 1, kt = it * KS + kg;
    const int kb = s0 + kt * SK;
    // stage kt has landed (own DMA done, then everyone's via the barrier); the
    // barrier also releases the stage the next prefetch overwrites
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (kt + KS < nkt) issue(cur ^ 1, kb + KS * SK);
    if (KS > 1 && kt >= nkt) return;
#pragma unroll
    for (int sub = 0; sub < SUB; ++sub) {
      const int kbs = kb + sub * ATT_BK;
      if constexpr (decltype(masked)::value) {
        if (s1 > kbs) tile(cur, sub, kbs, std::true_type{});   // a no-op mask when full
      } else {
        tile(cur, sub, kbs, std::false_type{});
      }
    }
  };
  const int nfull = (s1 - s0) / SK / KS;          // iterations in which every stage is full
  const int nit = (nkt + KS - 1) / KS;
  for (int it = 0; it < nfull; ++it) stage(it, std::false_type{});
  for (int it = nfull; it < nit; ++it) stage(it, std::true_type{});
  float l_tot = l_run + __shfl_xor(l_run, 32);
  if constexpr (KS > 1) {
    // groups 1.. park their sums, group 0 adds them up in order
    constexpr int SLOT = 34 * 64;                 // floats per wave
    static_assert((KS - 1) * NW * SLOT * 4 <= (int)sizeof(kv), "merge space");
    float* ex = reinterpret_cast<float*>(kv);
    __syncthreads();                              // the last stages are consumed
    if (kg > 0) {
      float* e = ex + ((kg - 1) * NW + wave) * SLOT + lane;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) e[(16 * t + r) * 64] = o[t][r];
      e[32 * 64] = m_run;
      e[33 * 64] = l_tot;
    }
    __syncthreads();
    if (kg > 0) return;
    float mx = m_run;
#pragma unroll
    for (int k = 0; k < KS - 1; ++k) mx = fmaxf(mx, ex[(k * NW + wave) * SLOT + 32 * 64 + lane]);
    const float f0 = __builtin_amdgcn_exp2f(m_run - mx);
    l_tot *= f0;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[t][r] *= f0;
#pragma unroll
    for (int k = 0; k < KS - 1; ++k) {
      const float* e = ex + (k * NW + wave) * SLOT + lane;
      const float f = __builtin_amdgcn_exp2f(e[32 * 64] - mx);   // 0 for a group without keys
      l_tot = fmaf(e[33 * 64], f, l_tot);
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t][r] = fmaf(e[(16 * t + r) * 64], f, o[t][r]);
    }
    m_run = mx;
  }
  if (!qvalid) return;
  const float inv = 1.0f / l_tot;
  bf16_t* op = out + (int64_t)qrow * d + h * 64;
#pragma unroll
  for (int ht = 0; ht < 2; ++ht)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const int hd = 32 * ht + 8 * q4 + 4 * g;
      uint2 w;
      w.x = pack_bf16x2(o[ht][4 * q4 + 0] * inv, o[ht][4 * q4 + 1] * inv);
      w.y = pack_bf16x2(o[ht][4 * q4 + 2] * inv, o[ht][4 * q4 + 3] * inv);
      *(uint2*)(op + hd) = w;
    }
  if (lse != nullptr && g == 0)
    lse[(int64_t)qrow * n_heads + h] = (m_run + log2f(l_tot)) * 0.6931471805599453f;
}

// fp32: S^T = K Q^T and O^T = V^T P^T with 32x32x2 MFMAs in the operand roles
// of the bf16 kernel (one query per lane; the P^T accumulators are the B
// operand as they are, key pairs 4 apart).  K, Q and V fragments come straight
// from global memory: an MFMA takes 64 cycles for 4 or 16 bytes per lane, so
// the loads hide behind it and no tile is staged.  The four waves' partial
// (max, sum, O) over their keys are merged through LDS in a fixed order.  The
// key split keeps short sequences from running on a few CUs: 192 rows of 24
// heads are 144 workgroups (one wave per row and head took 106 us there).
__global__ void __launch_bounds__(256)
attn_fwd_f32(const float* __restrict__ qkv, float* __restrict__ out, float* __restrict__ lse,
             const int32_t* __restrict__ cu, int n_seqs, int n_heads, int n_rows) {
  constexpr int LD = 68;                         // fp32 pitch of a query's partial O row
  __shared__ float os[4][32][LD];
  __shared__ float ms[4][32], ls[4][32];
  const int h = blockIdx.y;
  int s0, s1, q0;
  if (!find_tile<32>(cu, n_seqs, n_rows, blockIdx.x, s0, s1, q0)) return;
  const int d = n_heads * 64;
  const int64_t ld = 3 * (int64_t)d;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 5, r31 = lane & 31;
  const float* kbase = qkv + d + h * 64;
  const float* vbase = qkv + 2 * d + h * 64 + r31;
  f32x4 qf[8];
  {
    const float* qp = qkv + (int64_t)min(q0 + r31, s1 - 1) * ld + h * 64;
#pragma unroll
    for (int s = 0; s < 8; ++s) qf[s] = *reinterpret_cast<const f32x4*>(qp + 4 * (2 * s + g)) * 0.125f;
  }
  f32x16 o[2];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[t][r] = 0.0f;
  // the running max starts at the lowest finite value: a first tile whose
  // logits are all minus infinity then adds nothing, where (-inf) - (-inf)
  // would make the wave's sums NaN
  float m = -FLT_MAX, l = 0.0f;
  for (int kb = s0 + 32 * wave; kb < s1; kb += 128) {
    const float* kp = kbase + (int64_t)min(kb + r31, s1 - 1) * ld;
    f32x4 kf[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) kf[s] = *reinterpret_cast<const f32x4*>(kp + 4 * (2 * s + g));
    float vf[2][16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float* vp = vbase + (int64_t)min(kb + 8 * (r >> 2) + 4 * g + (r & 3), s1 - 1) * ld;
      vf[0][r] = vp[0];
      vf[1][r] = vp[32];
    }
    f32x16 st;
#pragma unroll
    for (int r = 0; r < 16; ++r) st[r] = 0.0f;
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e) st = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[s][e], qf[s][e], st, 0, 0, 0);
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if (kb + 8 * (r >> 2) + 4 * g + (r & 3) >= s1) st[r] = -INFINITY;
      mx = fmaxf(mx, st[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float m_new = fmaxf(m, mx), corr = expf(m - m_new);
    m = m_new;
    l *= corr;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[t][r] *= corr;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float p = expf(st[r] - m_new);
      l += p;
      o[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[0][r], p, o[0], 0, 0, 0);
      o[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[1][r], p, o[1], 0, 0, 0);
    }
  }
  l += __shfl_xor(l, 32);
  if (g == 0) { ms[wave][r31] = m; ls[wave][r31] = l; }
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4)
      *reinterpret_cast<float4*>(&os[wave][r31][32 * t + 8 * q4 + 4 * g]) =
          make_float4(o[t][4 * q4], o[t][4 * q4 + 1], o[t][4 * q4 + 2], o[t][4 * q4 + 3]);
  __syncthreads();
  const int q = tid >> 3, c = (tid & 7) * 8, row = q0 + q;
  if (row >= s1) return;
  const float mt = fmaxf(fmaxf(ms[0][q], ms[1][q]), fmaxf(ms[2][q], ms[3][q]));
  float lt = 0.0f, acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float f = expf(ms[w][q] - mt);         // 0 for a wave without finite logits
    lt = fmaf(ls[w][q], f, lt);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = fmaf(os[w][q][c + e], f, acc[e]);
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] /= lt;
  store8(out + (int64_t)row * d + h * 64 + c, acc);
  if (lse != nullptr && (tid & 7) == 0) lse[(int64_t)row * n_heads + h] = mt + logf(lt);
}

hipError_t launch_attention(int dtype, const void* qkv, void* o, float* lse,
                            const int32_t* cu_seqlens, int n_seqs, int64_t n_rows,
                            int n_heads, hipStream_t st, Prefetch pf0, Prefetch pf1) {
  if (n_rows <= 0) return hipSuccess;
  if (dtype == 1) {
    if (n_rows * 3 * (int64_t)n_heads * 64 >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    // Four shapes, by how many workgroups of 64, 128 or 256 query rows there
    // are (at most, the lengths being on the device) and the mean length:
    //  - as long as every workgroup has a CU of its own, a key split, with the
    //    smallest row tile that still leaves it one (us; 64-row tiles split |
    //    128 split | 128 unsplit): 400 rows x 24 heads 8.3 | 10.0 | 10.2,
    //    1,312 x 8 14.6 | 17.6 | 20.8, 1,312 x 16 (336 tiles of 64 rows) 20.8 |
    //    18.7 | 22.2.  128-row tiles below 384 rows per sequence have too few
    //    keys to split (326 x 24: 9.3 | 9.3, 192 x 24: 7.7 | 7.0);
    //  - more workgroups of 128 rows than CUs but not of 256: 8 waves, so that
    //    no CU runs two in turn (8 waves | 4 waves: 1,312 x 28 27.4 | 29.5,
    //    2,400 x 24 47.6 | 51.1, 8,000 x 8 145 | 158; level at 600 x 64,
    //    17.4 | 17.3, and slower below, 375 x 10 x 8 sequences 14.1 | 13.5);
    //  - 8 waves again from 1.75 such workgroups per CU (3,744 rows x 32 heads,
    //    480 workgroups, 11% faster than 4 waves);
    //  - 4 waves between (2,600 x 24, 264 workgroups of 256 rows, 57 us against
    //    81; 3,472 x 24 102 against 111).
    const int64_t ns = n_seqs;
    const int slots8 = (int)((n_rows + 255 * ns) / 256);
    const int slots4 = (int)((n_rows + 127 * ns) / 128);
    const int slots2 = (int)((n_rows + 63 * ns) / 64);
    const int64_t len = n_rows / ns;
    const bf16_t* a = (const bf16_t*)qkv;
    bf16_t* ob = (bf16_t*)o;
    const int ni = (int)n_rows;
    const int n_pf = pf0.p || pf1.p ? PREFETCH_WGS : 0;
#define SWAM_ATT(NW_, WPE_, SUB_, KS_, SL_)                                                   \
  hipLaunchKernelGGL((attn_fwd_bf16<NW_, WPE_, SUB_, KS_>), dim3((SL_) * n_heads + n_pf),      \
                     dim3(NW_ * KS_ * 64), 0, st, a, ob, lse, cu_seqlens, n_seqs, n_heads, ni, \
                     (SL_) * n_heads, pf0, pf1)
    // the 8-wave kernel stages 128 keys per barrier (64 KB of LDS, two
    // workgroups per CU); the 4-wave ones keep 64 so four fit on a CU
    if ((int64_t)slots2 * n_heads <= 256)
      SWAM_ATT(2, 4, 1, 2, slots2);
    else if ((int64_t)slots4 * n_heads <= 256 && len >= 384)
      SWAM_ATT(4, 1, 1, 2, slots4);
    else if (((int64_t)slots4 * n_heads > 256 && (int64_t)slots8 * n_heads <= 256 && len >= 800) ||
             (n_rows + 255) / 256 * n_heads >= 7 * 64)
      SWAM_ATT(8, 4, 2, 1, slots8);
    else
      SWAM_ATT(4, 4, 1, 1, slots4);
#undef SWAM_ATT
  } else {
    hipLaunchKernelGGL(attn_fwd_f32, dim3((unsigned)((n_rows + 31) / 32 + n_seqs), n_heads), dim3(256),
                       0, st, (const float*)qkv, (float*)o, lse, cu_seqlens, n_seqs, n_heads, (int)n_rows);
  }
  return hipGetLastError();
}

}  // namespace swam
