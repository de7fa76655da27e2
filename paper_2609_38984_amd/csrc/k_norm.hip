// adaLN modulation vectors and the modulated LayerNorm of the DiT block.
//   mod = W_ada SiLU(t_emb) + b_ada        (all blocks of a step in one launch)
//   h   = LN(x) (1 + scale) + shift       (biased variance, eps 1e-6, no affine)
// One wavefront per output row (modulation) or per token row (LN); the row
// stays in registers between the mean and the variance pass.
#include "launchers.h"

namespace swam {

template <typename T>
__global__ void __launch_bounds__(256)
adaln_kernel(AdalnArgs args, const float* __restrict__ temb, int d_temb, int d6,
             float* __restrict__ mod) {
  const int blk = blockIdx.y;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= d6) return;
  const T* w = (const T*)args.w[blk] + (int64_t)row * d_temb;
  float acc = 0.0f;
  for (int k = lane; k < d_temb; k += 64) {
    const float t = temb[k];
    acc = fmaf(Elem<T>::load(w + k), t / (1.0f + expf(-t)), acc);
  }
  acc = warp_sum(acc);
  if (lane == 0) mod[(int64_t)blk * d6 + row] = acc + Elem<T>::load((const T*)args.b[blk] + row);
}

// bf16 weights, d_temb = 128: 16 lanes per output row (one 16-byte load of 8
// weights each), ADALN_RPG rows per 16-lane group (rows g, g + 16, ... of the
// workgroup's 16 * ADALN_RPG, so each round of loads reads 4 KB of
// consecutive rows), every load issued before the first reduction; SiLU(temb)
// once per lane instead of once per weight
constexpr int ADALN_RPG = 8;

__global__ void __launch_bounds__(256)
adaln_bf16_t128(AdalnArgs args, const float* __restrict__ temb, int d6,
                float* __restrict__ mod) {
  const int blk = blockIdx.y;
  const int g = threadIdx.x >> 4;
  const int row0 = blockIdx.x * (16 * ADALN_RPG) + g;
  const int k0 = (threadIdx.x & 15) * 8;
  const bf16_t* wb = (const bf16_t*)args.w[blk];
  uint4 w[ADALN_RPG];
#pragma unroll
  for (int j = 0; j < ADALN_RPG; ++j) {
    const int rr = min(row0 + 16 * j, d6 - 1);   // every lane joins the exchange
    w[j] = *reinterpret_cast<const uint4*>(wb + (int64_t)rr * 128 + k0);
  }
  float sl[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float t = temb[k0 + e];
    sl[e] = t / (1.0f + expf(-t));
  }
  const bf16_t* bb = (const bf16_t*)args.b[blk];
#pragma unroll
  for (int j = 0; j < ADALN_RPG; ++j) {
    const uint32_t p[4] = {w[j].x, w[j].y, w[j].z, w[j].w};
    float acc = 0.0f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc = fmaf(__uint_as_float(p[e] << 16), sl[2 * e], acc);
      acc = fmaf(__uint_as_float(p[e] & 0xFFFF0000u), sl[2 * e + 1], acc);
    }
    acc += __shfl_xor(acc, 1);
    acc += __shfl_xor(acc, 2);
    acc += __shfl_xor(acc, 4);
    acc += __shfl_xor(acc, 8);
    const int row = row0 + 16 * j;
    if ((threadIdx.x & 15) == 0 && row < d6)
      mod[(int64_t)blk * d6 + row] = acc + bf16_to_f32(bb[row]);
  }
}

hipError_t launch_adaln(int dtype, const AdalnArgs& a, int n_blk, const float* temb,
                        int d_temb, int d6, float* mod, hipStream_t st) {
  if (dtype == 1 && d_temb == 128) {
    hipLaunchKernelGGL(adaln_bf16_t128, dim3((d6 + 16 * ADALN_RPG - 1) / (16 * ADALN_RPG), n_blk),
                       dim3(256), 0, st, a, temb, d6, mod);
    return hipGetLastError();
  }
  dim3 grid((d6 + 3) / 4, n_blk);
  if (dtype == 1)
    hipLaunchKernelGGL(adaln_kernel<bf16_t>, grid, dim3(256), 0, st, a, temb, d_temb, d6, mod);
  else
    hipLaunchKernelGGL(adaln_kernel<float>, grid, dim3(256), 0, st, a, temb, d_temb, d6, mod);
  return hipGetLastError();
}

// bf16 rows: 16-byte chunks of 8 elements, up to CH chunks per lane (d <= 512 CH).
// GATHER: output row r reads input row gather[r] and also stores it unchanged
// to xp row r (the gather-pack of a sparse step fused into its first LN).
template <int CH, bool GATHER>
__global__ void __launch_bounds__(256)
ln_mod_bf16(const bf16_t* __restrict__ x, bf16_t* __restrict__ h,
            const float* __restrict__ shift, const float* __restrict__ scale, int64_t rows,
            int d, const int32_t* __restrict__ gather, bf16_t* __restrict__ xp) {
  const int64_t row =
      (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  if (row >= rows) return;
  const int nch = d >> 3;
  const int64_t src = GATHER ? (int64_t)gather[row] : row;
  const uint4* xr = (const uint4*)(x + src * d);
  float v[CH][8];
  float s = 0.0f;
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int ci = lane + 64 * c;
    if (ci < nch) {
      const uint4 w = xr[ci];
      if (GATHER) ((uint4*)(xp + row * d))[ci] = w;
      const uint32_t p[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[c][2 * e] = __uint_as_float(p[e] << 16);
        v[c][2 * e + 1] = __uint_as_float(p[e] & 0xFFFF0000u);
        s += v[c][2 * e] + v[c][2 * e + 1];
      }
    }
  }
  const float mean = warp_sum(s) / d;
  float q = 0.0f;
#pragma unroll
  for (int c = 0; c < CH; ++c)
    if (lane + 64 * c < nch)
#pragma unroll
      for (int e = 0; e < 8; ++e) { const float t = v[c][e] - mean; q += t * t; }
  const float rstd = rsqrtf(warp_sum(q) / d + 1e-6f);
  uint4* hr = (uint4*)(h + row * d);
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int ci = lane + 64 * c;
    if (ci < nch) {
      const int col = ci * 8;
      float o[8];
#pragma unroll
      for (int e = 0; e < 8; ++e)
        o[e] = (v[c][e] - mean) * rstd * (1.0f + scale[col + e]) + shift[col + e];
      uint4 w;
      w.x = pack_bf16x2(o[0], o[1]);
      w.y = pack_bf16x2(o[2], o[3]);
      w.z = pack_bf16x2(o[4], o[5]);
      w.w = pack_bf16x2(o[6], o[7]);
      hr[ci] = w;
    }
  }
}

// One workgroup per row, thread t holding the 8-column chunks t, t + blockDim,
// ... (up to CH) in registers between the passes:
//   LN_PLAIN : h = LN(x) (1 + scale) + shift
//   LN_GATHER: the same of x row gather[r], which is also stored to xp
//   LN_SPLIT : x += gate (sum of the split-K partial rows + bias), stored, and
//              h of that row (rounded to the storage type first)
// Latency-bound at the row counts that use it (a few hundred): one row per
// workgroup spreads them over all CUs.  LN_SPLIT replaces an epilogue pass and
// a LayerNorm pass (192 x 1536, 6 slices: 4.9 us against 4.7 + 4.7); fp32 rows
// took 18 us for 192 x 1536 with one wave re-reading its row in 4-byte loads.
enum LnRowMode { LN_PLAIN, LN_GATHER, LN_SPLIT };
template <typename T, int CH, int MODE>
__global__ void __launch_bounds__(256)
ln_row(const float* __restrict__ part, int splits, int64_t slice, const T* __restrict__ bias,
       const float* __restrict__ gate, const T* x, T* xp, T* __restrict__ h,
       const float* __restrict__ shift, const float* __restrict__ scale, int d,
       const int32_t* __restrict__ gather, int rows, const Prefetch pf) {
  __shared__ float red[2][4];
  const int64_t row = blockIdx.x;
  if (row >= rows) {                               // spare workgroups
    prefetch_share(pf, (int)row - rows, gridDim.x - rows);
    return;
  }
  const int64_t src = MODE == LN_GATHER ? (int64_t)gather[row] : row;
  const int nch = d >> 3, tid = threadIdx.x, wave = tid >> 6, nw = blockDim.x >> 6;
  float v[CH][8];
  float s = 0.0f;
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int ci = tid + (int)blockDim.x * c;
    if (ci >= nch) continue;
    const int col = ci * 8;
    load8(x + src * d + col, v[c]);
    if constexpr (MODE == LN_SPLIT) {
      float bb[8], gg[8], acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      load8(bias + col, bb);
      load8(gate + col, gg);
      const float* p = part + row * d + col;
#pragma unroll 4
      for (int z = 0; z < splits; ++z) {
        float q[8];
        load8(p + z * slice, q);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += q[e];
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        v[c][e] = v[c][e] + gg[e] * (acc[e] + bb[e]);
        if constexpr (sizeof(T) == 2) v[c][e] = bf16_to_f32(f32_to_bf16(v[c][e]));
      }
    }
    if constexpr (MODE != LN_PLAIN) store8(xp + row * d + col, v[c]);
#pragma unroll
    for (int e = 0; e < 8; ++e) s += v[c][e];
  }
  auto block_sum = [&](float t, float* r) {
    t = warp_sum(t);
    if ((tid & 63) == 0) r[wave] = t;
    __syncthreads();
    float u = r[0];
    for (int w = 1; w < nw; ++w) u += r[w];
    return u;
  };
  const float mean = block_sum(s, red[0]) / d;
  float q = 0.0f;
#pragma unroll
  for (int c = 0; c < CH; ++c)
    if (tid + (int)blockDim.x * c < nch)
#pragma unroll
      for (int e = 0; e < 8; ++e) { const float t = v[c][e] - mean; q += t * t; }
  const float var = block_sum(q, red[1]) / d + 1e-6f;
  const float rstd = sizeof(T) == 2 ? rsqrtf(var) : 1.0f / sqrtf(var);
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int ci = tid + (int)blockDim.x * c;
    if (ci >= nch) continue;
    const int col = ci * 8;
    float sc[8], sh[8];
    load8(scale + col, sc);
    load8(shift + col, sh);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[c][e] = (v[c][e] - mean) * rstd * (1.0f + sc[e]) + sh[e];
    store8(h + row * d + col, v[c]);
  }
}

template <typename T, int MODE>
static hipError_t run_ln_row(const float* part, int splits, int64_t rows, int d, const void* bias,
                             const float* gate, const void* x, void* xp, void* h,
                             const float* shift, const float* scale, const int32_t* gather,
                             hipStream_t st, Prefetch pf = {}) {
  const unsigned n_pf = pf.p ? PREFETCH_WGS : 0;
  const int nt = d <= 512 ? 64 : d <= 1024 ? 128 : d <= 1536 ? 192 : 256;
#define SWAM_LNR(CH_)                                                                           \
  hipLaunchKernelGGL((ln_row<T, CH_, MODE>), dim3((unsigned)rows + n_pf), dim3(nt), 0, st, part, \
                     splits, rows * d, (const T*)bias, gate, (const T*)x, (T*)xp, (T*)h, shift, \
                     scale, d, gather, (int)rows, pf)
  if (d <= 2048) SWAM_LNR(1);
  else SWAM_LNR(2);                                // d <= LN_ROW_MAX
#undef SWAM_LNR
  return hipGetLastError();
}

hipError_t launch_splitk_ln(int dtype, const float* part, int splits, int64_t rows, int d,
                            const void* bias, const float* gate, void* x, void* h,
                            const float* shift, const float* scale, hipStream_t st, Prefetch pf) {
  if (rows <= 0) return hipSuccess;
  if (d > LN_ROW_MAX) return hipErrorInvalidValue;
  return dtype == 1 ? run_ln_row<bf16_t, LN_SPLIT>(part, splits, rows, d, bias, gate, x, x, h, shift, scale, nullptr, st, pf)
                    : run_ln_row<float, LN_SPLIT>(part, splits, rows, d, bias, gate, x, x, h, shift, scale, nullptr, st, pf);
}

// fp32 rows wider than LN_ROW_MAX: two passes over global memory (rows are L1/L2 resident);
// gather != NULL: as the bf16 GATHER variant
__global__ void __launch_bounds__(256)
ln_mod_f32(const float* __restrict__ x, float* __restrict__ h, const float* __restrict__ shift,
           const float* __restrict__ scale, int64_t rows, int d,
           const int32_t* __restrict__ gather, float* __restrict__ xp) {
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= rows) return;
  const float* xr = x + (gather ? (int64_t)gather[row] : row) * d;
  float s = 0.0f;
  for (int c = lane; c < d; c += 64) {
    s += xr[c];
    if (gather) xp[row * d + c] = xr[c];
  }
  const float mean = warp_sum(s) / d;
  float q = 0.0f;
  for (int c = lane; c < d; c += 64) { const float t = xr[c] - mean; q += t * t; }
  const float rstd = 1.0f / sqrtf(warp_sum(q) / d + 1e-6f);
  for (int c = lane; c < d; c += 64)
    h[row * d + c] = (xr[c] - mean) * rstd * (1.0f + scale[c]) + shift[c];
}

template <bool GATHER>
static hipError_t ln_mod_any(int dtype, const void* x, void* h, const float* shift,
                             const float* scale, int64_t rows, int d, const int32_t* gather,
                             void* xp, hipStream_t st, Prefetch pf = {}) {
  if (rows <= 0) return hipSuccess;
  // bf16: a workgroup per row for short token sets (192 x 1536: 4.2 us against
  // 4.7), a wave per row otherwise
  if (dtype == 1 && rows <= SHORT_ROWS && d <= LN_ROW_MAX)
    return run_ln_row<bf16_t, GATHER ? LN_GATHER : LN_PLAIN>(nullptr, 0, rows, d, nullptr, nullptr, x, xp,
                                                             h, shift, scale, gather, st, pf);
  dim3 grid((unsigned)((rows + 3) / 4));
  if (dtype == 1) {
    const bf16_t* xb = (const bf16_t*)x;
    bf16_t* hb = (bf16_t*)h;
    bf16_t* pb = (bf16_t*)xp;
    if (d <= 1024)
      hipLaunchKernelGGL((ln_mod_bf16<2, GATHER>), grid, dim3(256), 0, st, xb, hb, shift, scale,
                         rows, d, gather, pb);
    else if (d <= 2048)
      hipLaunchKernelGGL((ln_mod_bf16<4, GATHER>), grid, dim3(256), 0, st, xb, hb, shift, scale,
                         rows, d, gather, pb);
    else
      hipLaunchKernelGGL((ln_mod_bf16<8, GATHER>), grid, dim3(256), 0, st, xb, hb, shift, scale,
                         rows, d, gather, pb);
  } else if (d <= LN_ROW_MAX) {
    return run_ln_row<float, GATHER ? LN_GATHER : LN_PLAIN>(nullptr, 0, rows, d, nullptr, nullptr, x, xp,
                                                            h, shift, scale, gather, st);
  } else {
    hipLaunchKernelGGL(ln_mod_f32, grid, dim3(256), 0, st, (const float*)x, (float*)h, shift,
                       scale, rows, d, GATHER ? gather : nullptr, (float*)xp);
  }
  return hipGetLastError();
}

hipError_t launch_ln_mod(int dtype, const void* x, void* h, const float* shift,
                         const float* scale, int64_t rows, int d, hipStream_t st, Prefetch pf) {
  return ln_mod_any<false>(dtype, x, h, shift, scale, rows, d, nullptr, nullptr, st, pf);
}

hipError_t launch_ln_mod_gather(int dtype, const void* x_full, const int32_t* gather, void* xp,
                                void* h, const float* shift, const float* scale, int64_t rows,
                                int d, hipStream_t st) {
  return ln_mod_any<true>(dtype, x_full, h, shift, scale, rows, d, gather, xp, st);
}

// ---------------------------------------------------------------------------
// backbone variants on the stored q and k: QK-norm (unit-gain RMS per head),
// then the rotary embedding at each row's original position
// ---------------------------------------------------------------------------
// [l_full][32] (cos, sin) of pos * 10000^(-2i/64), evaluated in float64
// cos / sin of position * 10000^(-2i/64) for positions [0, n_pos), i < 32
__global__ void rope_table_kernel(float2* __restrict__ tab, int n_pos) {
  const int id = blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= n_pos * 32) return;
  const int pos = id >> 5, i = id & 31;
  const double ang = (double)pos * pow(10000.0, -2.0 * i / 64.0);
  tab[id] = make_float2((float)cos(ang), (float)sin(ang));
}

hipError_t launch_rope_table(float2* tab, int n_pos, hipStream_t st) {
  hipLaunchKernelGGL(rope_table_kernel, dim3((n_pos * 32 + 255) / 256), dim3(256), 0, st, tab,
                     n_pos);
  return hipGetLastError();
}

// fp32 (the bf16 projections' store does the same: qkpost_store):
// one thread per 8 consecutive elements of q or k (a head is 8 threads, which
// are 8 consecutive lanes); pos_mode 0: row % l_full, 1: gather[row] % l_full,
// 2: row - cu[b] for the row's sequence b; positions are clamped to the
// table's n_pos rows
__global__ void __launch_bounds__(256)
qk_post_kernel(float* __restrict__ qkv, int64_t n_rows, int d, int pos_mode,
               const int32_t* __restrict__ gather, const int32_t* __restrict__ cu, int n_seqs,
               int l_full, const float2* __restrict__ tab, int n_pos, int qk_norm) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int chunks = 2 * d / 8;               // q and k columns of a row
  const bool live = id < n_rows * chunks;
  const int64_t row = live ? id / chunks : 0;
  const int c8 = live ? (int)(id % chunks) * 8 : 0;
  float* p = qkv + row * 3 * d + c8;
  float x[8];
  load8(p, x);
  if (qk_norm) {
    // the 8 lanes of a head are consecutive and aligned (chunks per row and per
    // head are multiples of 8); every lane takes part in the exchange
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
  if (!live) return;
  if (tab != nullptr) {
    int pos;
    if (pos_mode == 0) {
      pos = (int)(row % l_full);
    } else if (pos_mode == 1) {
      pos = gather[row] % l_full;
    } else {
      int b = 0;
      while (b + 1 < n_seqs && cu[b + 1] <= row) ++b;
      pos = (int)(row - cu[b]);
    }
    pos = min(max(pos, 0), n_pos - 1);
    const float2* t = tab + (int64_t)pos * 32 + ((c8 & 63) >> 1);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float2 cs = t[e];
      const float a = x[2 * e], b = x[2 * e + 1];
      x[2 * e] = a * cs.x - b * cs.y;
      x[2 * e + 1] = a * cs.y + b * cs.x;
    }
  }
  store8(p, x);
}

hipError_t launch_qk_post(float* qkv, int64_t n_rows, int d, int pos_mode, const int32_t* gather,
                          const int32_t* cu, int n_seqs, int l_full, const float2* tab, int n_pos,
                          int qk_norm, hipStream_t st) {
  if (n_rows <= 0) return hipSuccess;
  const int64_t n = n_rows * (2 * d / 8);
  hipLaunchKernelGGL(qk_post_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, qkv, n_rows, d,
                     pos_mode, gather, cu, n_seqs, l_full, tab, n_pos, qk_norm);
  return hipGetLastError();
}

}  // namespace swam
