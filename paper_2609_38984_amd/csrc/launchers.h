// Host-side launchers of the libswam kernels (one per kernel family, all
// asynchronous on the given stream) and their argument structs.
#pragma once
#include "common.h"

namespace swam {

// ---------------------------------------------------------------------------
// launchers (host side), one per kernel family; all asynchronous on `st`
// ---------------------------------------------------------------------------
// EPI_PARTIAL is internal to the bf16 split-K path (fp32 partial sums);
// EPI_BIAS_QKPOST to launch_gemm_qkv
enum Epilogue { EPI_BIAS = 0, EPI_BIAS_GELU = 1, EPI_BIAS_GATED_RESIDUAL = 2, EPI_PARTIAL = 3,
                EPI_BIAS_QKPOST = 4 };

// QK-norm / rotary embedding of the q and k columns of a QKV projection
// (the arguments of launch_qk_post): d = model width (q columns [0, d), k
// columns [d, 2d)); pos_mode 0 = dense rows (position row % l_full), 1 =
// packed rows (gather[row] % l_full), 2 = index inside the cu_seqlens
// sequence; tab = rotary table [n_pos][32] (NULL: no rotation).
struct QkPost {
  int d = 0, pos_mode = 0, n_seqs = 0, l_full = 1, n_pos = 1, qk_norm = 0;
  const int32_t* gather = nullptr;
  const int32_t* cu = nullptr;
  const float2* tab = nullptr;
};

// The four projections of a block; the role fixes the epilogue:
// QKV bias, UP bias + tanh-GELU, OUT and DOWN bias + gated residual.
enum GemmRole { ROLE_QKV = 0, ROLE_OUT = 1, ROLE_UP = 2, ROLE_DOWN = 3 };

// C[M][N] = epi(A[M][K] . B[N][K]^T + bias[N]); for the gated residual
// C[m][n] = C[m][n] + gate[n] * (acc + bias[n]) (C read then written).
// ws / ws_floats: fp32 workspace the bf16 path may use to split K when the
// output tiles alone cannot fill the CUs (partial sums, then one reduce +
// epilogue pass); NULL or too small means no split.
// smap (bf16 OUT / DOWN only): row m of the result goes to Cs[smap[m]] (same
// ldc) instead of C[m]; the residual is still read from C[m].  The scatter of
// a packed sequence's rows back into the full latent rides on the last
// projection this way.
// ln (OUT / DOWN without smap, ldc == N): where K is split, the pass that sums
// the splits also computes h = LN(result) (1 + scale) + shift and sets `done`;
// otherwise the caller launches that LayerNorm itself.
struct LnNext {
  void* h;
  const float *shift, *scale;
  Prefetch pf = {};      // weights of the projection after it
  bool done = false;
};
hipError_t launch_gemm(int dtype, int role, const void* A, int64_t lda, const void* B,
                       int64_t ldb, const void* bias, const float* gate, void* C,
                       int64_t ldc, int64_t M, int64_t N, int64_t K, hipStream_t st,
                       float* ws = nullptr, int64_t ws_floats = 0, void* Cs = nullptr,
                       const int32_t* smap = nullptr, LnNext* ln = nullptr);

// QKV projection C = A . B^T + bias followed by the QK-norm / rotary
// embedding of qp on its q and k columns: in the GEMM's store for bf16 (on the
// projection rounded to bf16; it then does not split K), a second launch for
// fp32.
hipError_t launch_gemm_qkv(int dtype, const void* A, int64_t lda, const void* B, int64_t ldb,
                           const void* bias, void* C, int64_t ldc, int64_t M, int64_t N,
                           int64_t K, const QkPost& qp, hipStream_t st, float* ws = nullptr,
                           int64_t ws_floats = 0);

// mod[blk][6d] = W_ada[blk] SiLU(temb) + b_ada[blk] for n_blk blocks at once.
struct AdalnArgs {
  const void* w[64];
  const void* b[64];
};
hipError_t launch_adaln(int dtype, const AdalnArgs& a, int n_blk, const float* temb,
                        int d_temb, int d6, float* mod, hipStream_t st);

// Token sets of at most SHORT_ROWS rows leave most CUs and the memory idle in
// attention and LayerNorm and then wait for cold weights in the projections, so
// PREFETCH_WGS spare workgroups of those launches read the weights ahead (192
// rows, d = 1536, weights from memory / read ahead: QKV 11.1 / 7.9 us, up 14.2 /
// 11.4, down 13.0 / 9.7, out 6.4 / 5.5; attention takes 2.1 us and LayerNorm 1.0
// us longer.  Spare workgroups in the projections themselves cost them more than
// they save: up 15.8 us).
// Only while a block's four matrices are at most READ_AHEAD_BYTES: a launch ends
// with its read, so what it reads has to fit into the time it would take alone.
// us per block with | without, weights from memory, 48 / 192 / 1,024 rows: d =
// 1,024 (25 MB) 38.5 | 42.2, 44.2 | 48.7, 76.0 | 78.0; 1,536 (57 MB) 48.7 | 51.5,
// 59.1 | 66.0, 124.6 | 138.8; 2,816 with an MLP ratio of 1 (95 MB; 64 rows first)
// 66.5 | 67.9, 80.2 | 86.4, 174.5 | 187.8; 2,048 (101 MB) 61.3 | 59.9, 81.5 | 82.3,
// 175.1 | 174.6; 3,072 (226 MB) 100.3 | 89.2, 139.9 | 129.9, 340.0 | 328.2; 4,096
// (403 MB) 153.5 | 122.5, 218.6 | 179.3, 519.5 | 486.4.  Reading only the first 6 to
// 36 MB of each launch's weights gained nothing above the line (2,048: 1-4% slower
// than none).  Weights that the caches already hold (a model of two blocks) cost
// 0-5% of a block up to d = 1,536.
constexpr int SHORT_ROWS = 1024;
constexpr int PREFETCH_WGS = 256;
constexpr int64_t READ_AHEAD_BYTES = 96000000;

// h[r] = LN(x[r]) (1 + scale) + shift; pf: see above (bf16, up to SHORT_ROWS rows)
hipError_t launch_ln_mod(int dtype, const void* x, void* h, const float* shift,
                         const float* scale, int64_t rows, int d, hipStream_t st, Prefetch pf = {});
// widest row that one workgroup's registers hold (the ln_row kernels)
constexpr int LN_ROW_MAX = 4096;
// the LayerNorm behind a projection whose K was split: x[r] += gate *
// (sum of the `splits` partial rows + bias), stored, and h[r] of that row;
// part is [splits][rows][d], d <= LN_ROW_MAX
hipError_t launch_splitk_ln(int dtype, const float* part, int splits, int64_t rows, int d,
                            const void* bias, const float* gate, void* x, void* h,
                            const float* shift, const float* scale, hipStream_t st,
                            Prefetch pf = {});
// the same on gathered rows: xp[r] = x_full[gather[r]] (the gather-pack) and
// h[r] = LN(xp[r]) (1 + scale) + shift, in one pass
hipError_t launch_ln_mod_gather(int dtype, const void* x_full, const int32_t* gather, void* xp,
                                void* h, const float* shift, const float* scale, int64_t rows,
                                int d, hipStream_t st);

// backbone variants: rotary table and QK-norm / RoPE of the stored q and k (fp32)
hipError_t launch_rope_table(float2* tab, int n_pos, hipStream_t st);
hipError_t launch_qk_post(float* qkv, int64_t n_rows, int d, int pos_mode, const int32_t* gather,
                          const int32_t* cu, int n_seqs, int l_full, const float2* tab, int n_pos,
                          int qk_norm, hipStream_t st);

// o = softmax(q k^T / 8) v per head inside each sequence; lse (optional).
// Sequence bounds are clamped to [0, n_rows].  pf0, pf1 (bf16): weights read ahead.
hipError_t launch_attention(int dtype, const void* qkv, void* o, float* lse,
                            const int32_t* cu_seqlens, int n_seqs, int64_t n_rows,
                            int n_heads, hipStream_t st, Prefetch pf0 = {}, Prefetch pf1 = {});

// Score kernels (mode A with lse, mode B computes lse first into lse_ws).
struct ScoreArgs {
  const void* q; int64_t q_seq, q_row;
  const void* k; int64_t k_seq, k_row;
  const float* lse;           // sequence b, query i, head h at lse + b*lse_seq + i*N_h + h
  int64_t lse_seq;
  float* s_out;               // sequence b, frame f at s_out + b*s_seq + f*N_s
  int64_t s_seq;
  const float* alpha;         // [g] device
  int B, F, n_s, H, n_heads;
  int n_layers;               // layers scored by one launch (>= 1)
  int64_t q_lay, k_lay, lse_lay, s_lay;   // element strides between layers
};
hipError_t launch_score(int dtype, const ScoreArgs& a, hipStream_t st);
// MLP up projection (bias + GELU) of a refresh step with one layer's scores
// (ScoreArgs, bf16) computed by extra workgroups in the tail of its grid, on
// the CUs its last round of tiles leaves idle; gemm_up_scored_slots returns
// how many that is for a shape (0: not applicable, the caller scores
// separately), and launch_gemm_up_scored returns hipErrorNotSupported then.
int gemm_up_scored_slots(int64_t M, int64_t N, int64_t K, int64_t ws_floats);
hipError_t launch_gemm_up_scored(const void* A, int64_t lda, const void* B, int64_t ldb,
                                 const void* bias, void* C, int64_t ldc, int64_t M, int64_t N,
                                 int64_t K, const ScoreArgs& sa, hipStream_t st,
                                 int64_t ws_floats);
hipError_t launch_lse_all(int dtype, const void* q, int64_t q_seq, int64_t q_row,
                          const void* kall, int64_t k_seq, int64_t k_row, int64_t n_keys,
                          int B, int H, int n_heads, float* lse_out, float* part_ws,
                          hipStream_t st);

// Score reduction (layer quality, core layers, V, A).
struct ReduceArgs {
  const float* s_all;  // [B][L][F][N_s]
  double* frame_sum;   // ws [B][L][F]
  double* frame_ent;   // ws [B][L][F]
  float* q;            // [B][L]
  int32_t* core;       // [B][k_layer_eff]
  float* v;            // [B][F][N_s]
  float* a;            // [B][N_s]
  int B, L, F, n_s, k_layer;
  float cv_penalty;
};
hipError_t launch_score_reduce(const ReduceArgs& a, hipStream_t st);

// buffers copied by one launch (word-aligned, whole words)
struct CopyList {
  static constexpr int MAX = 9;
  const void* src[MAX];
  void* dst[MAX];
  int64_t bytes[MAX];
  int n;
  void add(const void* s, void* d, int64_t b) {
    if (b <= 0) return;
    src[n] = s; dst[n] = d; bytes[n] = b; ++n;
  }
};
hipError_t launch_copy_list(const CopyList& c, hipStream_t st);

// Selection and packing metadata (pack_pos, gather, cu) of fixed budgets or a
// mass threshold.
struct SelectArgs {
  const float* v;      // [B][F][N_s]
  const float* a;      // [B][N_s]
  uint8_t* pool;       // ws [B][N_s] (mass threshold)
  uint8_t* core;       // ws [B][F][N_s]
  int32_t* keep_idx;   // [batch][F][k_max]
  int32_t* keep_cnt;   // [batch][F]
  int32_t* keep;       // ws [batch*L_full] 0/1 (mass threshold)
  int32_t* pack_pos;   // [batch*L_full]
  int32_t* gather;     // [batch*L_full]
  int32_t* cu;         // [batch+1]
  int B, F, n_s, k_core, k_anchor, k_max;
  int batch;               // B, or 2 B: sequence b + B keeps the positions of b
  int mass_num, mass_den;  // mass threshold as a fraction; den == 0: fixed K_c
  int n_ctx, n_act;
};
hipError_t launch_select(const SelectArgs& a, hipStream_t st);
// uniform keys in [0, 1) (top 24 bits of word 0 of Philox4x64-10 at counter
// (i, 0, 0, 0), key (seed, 0)) into v[i] for i < n, and zeros into a[n_a]
// (n_a <= n)
hipError_t launch_random_keys(float* v, int64_t n, float* a, int64_t n_a, uint64_t seed,
                              hipStream_t st);
// keep flags from an imported selection; rewrites keep_idx / keep_cnt ascending
hipError_t launch_keep_from_idx(const int32_t* in_idx, int32_t* keep_idx, int32_t* keep_cnt,
                                int32_t* keep, int B, int F, int n_s, int k_max, int n_ctx,
                                int n_act, hipStream_t st);
// exclusive scan of keep flags -> pack_pos, gather, cu_seqlens
hipError_t launch_packmap(const int32_t* keep, int32_t* pack_pos, int32_t* gather,
                          int32_t* cu, int B, int64_t l_full, hipStream_t st);
hipError_t launch_pack(const void* x_full, void* x_packed, const int32_t* gather,
                       int64_t rows, int64_t row_bytes, hipStream_t st);
hipError_t launch_unpack_scatter(const void* y_packed, void* y_full, const int32_t* gather,
                                 int64_t rows, int64_t row_bytes, hipStream_t st);
hipError_t launch_unpack_merge(const void* y_packed, const void* x_full, void* y_full,
                               const int32_t* pack_pos, int64_t rows, int64_t row_bytes,
                               hipStream_t st);
hipError_t launch_overlap(const float* p, const float* q, int64_t n_maps, int64_t n,
                          float* out, hipStream_t st);

// sampling update (k_sampler.hip)
// z_rows: latent rows of z; the latent rows of sequences past them (the
// unconditional partners of guidance pairs) read z row i - z_rows
hipError_t launch_embed(int dtype, const float* z, const void* w_in, const void* b_in, void* x,
                        int64_t n_lat_rows, int64_t z_rows, int l_lat, int l_full, int n_ctx,
                        int c, int d, hipStream_t st);
hipError_t launch_velocity(int dtype, const void* y, const int32_t* gather, int64_t n_items,
                           const void* w_v, const void* b_v, float* v, int l_lat, int l_full,
                           int n_ctx, int c, int d, hipStream_t st);
// pairs: v holds 2 * n_lat_rows rows (conditional, then unconditional) that
// are combined as v_u + guidance * (v_c - v_u) before the merge
hipError_t launch_sample_update(const float* v, float* v_cache, float* z, const int32_t* pack_pos,
                                float dsigma, int kind, int64_t n_lat_rows, int l_lat, int l_full,
                                int n_ctx, int n_fut, int c, int pairs, float guidance,
                                hipStream_t st);
hipError_t launch_copy(const void* src, void* dst, int64_t bytes, hipStream_t st);
// y_full row r = x_full row r where pack_pos[r] < 0 (the pruned rows)
hipError_t launch_copy_pruned(const void* x_full, void* y_full, const int32_t* pack_pos,
                              int64_t rows, int64_t row_bytes, hipStream_t st);

}  // namespace swam
