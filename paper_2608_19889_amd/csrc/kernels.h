// Host-side launchers of the gfx950 kernels.  Every launcher enqueues on the
// given stream and returns immediately; shapes are validated by the caller.
#pragma once
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.h"

namespace axon {

// Measurement hook: when the runtime arms this slot, the next kernel launched
// through klaunch() carries the two events in its own dispatch
// (hipExtLaunchKernelGGL), so their elapsed time is that kernel's execution.
struct TimingSlot {
  hipEvent_t start = nullptr, stop = nullptr;
};
extern thread_local TimingSlot g_timing_slot;

template <typename Kern, typename... Args>
void klaunch(Kern kern, dim3 grid, dim3 block, uint32_t shmem, hipStream_t s, Args... args) {
  if (g_timing_slot.start) {
    const TimingSlot t = g_timing_slot;
    g_timing_slot = TimingSlot{};
    hipExtLaunchKernelGGL(kern, grid, block, shmem, s, t.start, t.stop, 0, args...);
  } else {
    kern<<<grid, block, shmem, s>>>(args...);
  }
}

// Epilogues of the projection GEMMs (out[t][n] = sum_k X[t][k] * W[n][k]).
enum Epi : int {
  EPI_F32 = 0,    // out_f32[t * ldo + n] = acc
  EPI_RESID = 1,  // out_f32[t * ldo + n] = resid[t * ldo + n] + acc  (residual
                  // stream, float; resid null: out_f32)
  EPI_SILU = 2,   // W rows interleaved in blocks of 16 gate rows then 16 up rows;
                  // out_t[t * ldo + f] = silu(gate_f) * up_f
  EPI_ROPE = 4,   // bf16 fused QKV projection (rows in the rotation-pair order of
                  // the decode projections): bias + rotary embedding, then q ->
                  // q_out, k -> K pages, v -> transposed V pages
  // EPI_LSE, EPI_GU, EPI_DGU (training): X and bf16 outputs in the row-pair layout
  EPI_LSE = 3,    // EPI_F32 (no bias) and, per token and 64 columns, their largest
                  // value and the sum of exp(value - largest) (lse_part)
  EPI_GU = 6,     // the interleaved gate/up pre-activations kept (out_f32, rows of
                  // ldo) beside EPI_SILU's out_t (rows of ldo / 2)
  EPI_DGU = 7,    // acc = gradient of gated feature n; its gate/up pre-activations
                  // gu [T][2 ldo] give the gradients of both, bf16, interleaved
                  // like gu: out_t [T][2 ldo]
  EPI_HEAD = 8,   // logits out_f32 (may be null) and, per token and 32 (or 64) columns,
                  // the largest and its lowest index (am_val / am_idx)
  EPI_GELU = 5    // out_t[t * ldo + n] = gelu_tanh(acc + bias[n])  (GPT-2 MLP, bf16)
};
// EPI_F32 / EPI_RESID add EpiArgs::bias[n] to acc when it is set.

struct EpiArgs {
  float* out_f32;
  void* out_t;
  int ldo;
  const float* resid;
  int64_t part_stride;
  // EPI_ROPE.  Token t is at position t - cu[seq] of sequence seq (prefill,
  // len == nullptr) or at position len[t] of slot t (decode).
  const bf16* bias;  // [(H+2KV)hd] in the original head order, or null
  const float* cos_t;
  const float* sin_t;
  bf16* q_out;       // [T][H][hd]
  KVView kv;
  const int32_t* cu;
  int nseq;
  const int32_t* len;
  int H;
  // prefill entry e (tokens cu[e] .. cu[e+1]-1): cache slot ent_slot[e] and
  // position of its first token ent_base[e]; null: slot e, position 0
  const int32_t* ent_slot;
  const int32_t* ent_base;
  // grouped GEMM (mixture of experts): expert e multiplies its matrix W + e *
  // g_wstride with rows g_off[e] .. g_off[e+1]-1 of the grouped operand; row a
  // of it is X row g_xrow[a] (a when null), output row a.  g_toff[e] = sum of
  // ceil(rows / 256) over the experts before e.
  const int32_t* g_off;
  const int32_t* g_toff;
  const int32_t* g_xrow;
  int64_t g_wstride;
  int g_E;
  const float* gu;  // EPI_DGU
  // row-pair layout (xp_off) of the token operand X, and of the bf16 output
  // out_t of EPI_SILU and EPI_GU (there always 1); 0: row-major
  int xpair;
  int opair;
  // few-token GEMM (launch_gemm_few), EPI_SILU / EPI_ROPE / EPI_HEAD: the operand
  // is bf16(x * g) and the result is scaled by rsqrt(sum of squares / K + eps), the
  // sums in ss_n partials [ss_n][M]; null: no scaling
  const float* ss_in;
  int ss_n;
  float eps;
  const int32_t* slot;  // EPI_ROPE with len: the cache slot of token t (t when null)
  float* am_val;        // EPI_HEAD: [T][ceil(N / few_head_rows)]
  int32_t* am_idx;
  // EPI_LSE: [T][ceil(N / 64)] (largest, sum) of columns 64 i .. 64 i + 63
  float2* lse_part;
};
constexpr int LSE_COLS = 64;

// ---- GPT-2 rows (k_layernorm.hip).  Token t is at position len[t] (decode)
// or, with len null, ent_base[e] + t - cu[e] of its entry e (0-based when
// ent_base is null).
// x[t] = wte[tok[t]] + wpe[pos] (float; wte fragment-tiled, wpe row-major
// [P][D]); h[t] = LayerNorm(x[t]) * g + beta (bf16)
void launch_embed_pos_ln(const int32_t* tok, const bf16* wte, const bf16* wpe, const bf16* g, const bf16* beta,
                         float* x, bf16* h, int T, int D, int V, int P, float eps, const int32_t* cu, int nseq,
                         const int32_t* ent_base, const int32_t* len, hipStream_t s);
// h[i] = LayerNorm(x[r]) * g + beta with r = i, or r = cu_last[i+1]-1 (the
// last position of sequence i) when cu_last is set
void launch_layernorm(const float* x, const bf16* g, const bf16* beta, bf16* h, int rows, int D, float eps,
                      const int32_t* cu_last, hipStream_t s);
// dst[r][k] = src[k][perm ? perm[r] : r] (bf16): a [K][N] matrix stored
// [in][out] transposed to [N][K], rows optionally permuted
void launch_transpose_rows(const bf16* src, bf16* dst, int K, int N, const int32_t* perm, hipStream_t s);

// ---- backward pass (k_train.hip)
// loss over logits [T][ldl] (V real columns, ldl % 32 == 0) and targets
// (counted when in [0, V)), from the logits and their projection's EPI_LSE
// partials: loss[0] = mean cross-entropy, dlog [T][ldl] bf16 = its gradient
// (zero padding, row-pair layout); rowloss / valid / lse [T] and scal [1] scratch
void launch_ce_loss(const float* logits, int ldl, int V, const float2* lse_part, const int32_t* targets, int T,
                    float* rowloss, float* valid, float* lse, float* loss, float* scal, bf16* dlog, hipStream_t s);
// dst [K][Np] (row-major) = W^T for the fragment-tiled W [N][K]
void launch_untile_transpose(const bf16* W, int64_t N, int K, bf16* dst, int64_t Np, hipStream_t s);
// The row kernels below that reduce over tokens leave at most ROW_PARTS partial
// rows.  RMSNorm backward: dx (accumulate ? += : =), its bf16 copy dxb (row-pair
// layout) and the gain's gradient dg [D], from dy as np partials [T][D] ``stride``
// apart; part: ROW_PARTS x D floats; dgrow: [T][D] scratch, needed for D >
// NORM_BWD_COLS only.  D % 32 == 0.
constexpr int ROW_PARTS = 512, NORM_BWD_COLS = 8192;
void launch_norm_bwd(const float* x, const bf16* g, const float* dy, int np, int64_t stride, int T, int D, float eps,
                     float* dx, int accumulate, bf16* dxb, float* dg, float* part, float* dgrow, hipStream_t s);
// attention backward over nseq fresh sequences in slots 0.. (contiguous cache):
// dq [T][H][hd] and each query head's share of dk / dv, dkh / dvh [T][H][hd]
// (float), from q [T][H][hd] and o (row-pair layout) bf16, the gradient of o as
// np float partials ``stride`` apart (dob [T][H][hd] receives it in bf16) and the
// forward's log2-sum-exp lse [T][H]; dsum [T][H] scratch.  head_dim 64 or 128.
void launch_attn_bwd(const bf16* q, KVView kv, const bf16* o, const float* dof, int np, int64_t stride, bf16* dob,
                     const float* lse, float* dsum, const int32_t* cu, const int32_t* h_cu, int nseq, int T, int H,
                     float* dq, float* dkh, float* dvh, hipStream_t s);
// back through RoPE into the fused QKV row order (bf16, row-pair layout), the
// heads' shares of dk / dv summed; with dbq the bias gradients dbq / dbk / dbv too
// (bpart: ROW_PARTS x nq floats)
void launch_rope_bwd(const float* dq, const float* dkh, const float* dvh, const float* cos_t, const float* sin_t,
                     const int32_t* cu, int nseq, int T, int H, int KVh, int hd, bf16* dqkv, float* bpart, float* dbq,
                     float* dbk, float* dbv, hipStream_t s);
// dE [V][D] += the tokens' rows of dx [T][D]; clear: dE = 0 first (D % 4 == 0)
void launch_embed_bwd(const int32_t* tok, const float* dx, int T, int D, int V, float* dE, bool clear, hipStream_t s);

// ---- weight layout (k_layout.hip): fragment-tiled copy of row-major bf16
// W [N][K] (K % 32 == 0) into dst of round_up(N, 16) * K elements
void launch_tile_weight(const bf16* src, bf16* dst, int64_t N, int K, hipStream_t s);

// ---- row kernels (k_norm.hip); a bf16 embedding table is fragment-tiled.
// h_pair: h in the row-pair layout (xp_off; D % 32 == 0), else row-major.
template <typename T>
void launch_embed_rmsnorm(const int32_t* tok, const T* emb, const T* g, float* x, T* h, int rows, int D, int V,
                          float eps, hipStream_t s, bool h_pair = false);
template <typename T>
void launch_resid_rmsnorm(float* x, const float* parts, int nparts, int64_t part_stride, const T* g, T* h,
                          int rows, int D, float eps, const int32_t* cu_last, hipStream_t s, bool h_pair = false,
                          float* x_out = nullptr);  // nparts > 0: the new x goes to x_out (x when null)
// next[i] = argmax of logits row i, or (cu_last) of row cu_last[i+1]-1, the lowest
// index on ties; len[i] += 1 when set; am_val / am_idx: scratch of rows x
// ceil(V / 4096)
void launch_argmax(const float* logits, int rows, int V, float* am_val, int32_t* am_idx, int32_t* next, int32_t* len,
                   const int32_t* cu_last, hipStream_t s);
void launch_set_lengths(const int32_t* cu, int32_t* len, int n, hipStream_t s);
// len[ent_slot[e]] = ent_base[e] + cu[e+1] - cu[e] for the n entries of a step
void launch_set_step_lengths(const int32_t* cu, const int32_t* ent_slot, const int32_t* ent_base, int32_t* len,
                             int n, hipStream_t s);

// ---- projections (k_gemm.hip)
// Raises the dynamic LDS limits of the kernels below on the current device; once
// per device, before any of them is launched there.
hipError_t gemm_init_device();
// Many-token GEMM (prefill): bf16 MFMA tiles.  Requires K % 32 == 0, and N % 32 ==
// 0 except for EPI_F32, EPI_RESID and EPI_LSE (EPI_ROPE: the head dimension a
// multiple of 32).  ep.xpair: X in the row-pair
// layout (xp_off); ep.opair: the SiLU epilogue's output in that layout.
void launch_gemm_bf16(const bf16* W, const bf16* X, int N, int M, int K, int epi, const EpiArgs& ep,
                      hipStream_t s);
// The same GEMM for 17 .. 64 decode tokens (tiles of at most 64 tokens, row-major
// X, K % 32 == 0): EPI_ROPE, EPI_SILU, EPI_GELU, EPI_HEAD (any N).
void launch_gemm_few(const bf16* W, const bf16* X, int N, int M, int K, int epi, const EpiArgs& ep, hipStream_t s);
int few_head_rows(int N, int M, int K);  // columns per EPI_HEAD partial
// Grouped GEMM of the experts (ep.g_*): rows of all experts together at most
// max_rows; launches enough 256 x 256 tiles for any split of them over the
// experts (surplus workgroups exit at once).  EPI_F32 or EPI_SILU.
void launch_gemm_bf16_grouped(const bf16* W, const bf16* X, int N, int K, int max_rows, int epi, const EpiArgs& ep,
                              hipStream_t s);
// split K over gridDim.y = ksplit workgroup rows: float32 partials
// part[s * part_stride + m * N + n] (ksplit divides K / 32; tiles as for the
// unsplit GEMM).  gemm_ksplit: the split worth taking for an output of few 256-tiles
// (1: none).
void launch_gemm_bf16_split(const bf16* W, const bf16* X, int N, int M, int K, int ksplit, float* part,
                            int64_t part_stride, hipStream_t s, bool xpair = false);
int gemm_ksplit(int N, int M, int K);
// the split of a GEMM whose partials the next kernel sums (decode batches above
// 64, the backward pass): the least of its time and the partials' traffic
int gemm_ksplit_cost(int N, int M, int K, int max_split);
// Weight gradient dW = Y^T X over T token rows: out[r][c] = sum_t Y[t][r] X[t][c],
// Y [T][ldy] (R <= ldy columns used, ldy % 32 == 0), X [T][C] (C % 32 == 0), both
// in the row-pair layout.  The rows go to out [R][C], or
// back from the kernel row orders to the weight map's tensors: WGRAD_QKV out / out1
// / out2 = q / k / v, WGRAD_GU out / out1 = gate / up.  part: part_floats floats of
// scratch for a split over the tokens.
enum WgradMode : int { WGRAD_ROWS = 0, WGRAD_QKV = 1, WGRAD_GU = 2 };
void launch_wgrad(int mode, const bf16* Y, int ldy, int R, const bf16* X, int C, int T, float* out, float* out1,
                  float* out2, int hd, int H, int KVh, float* part, int64_t part_floats, hipStream_t s);
// float32 check-mode GEMM (any M): EPI_F32 / EPI_RESID.
void launch_gemm_f32(const float* W, const float* X, int N, int M, int K, int epi, const EpiArgs& ep,
                     hipStream_t s);
// a[t][f] = silu(gate) * up of the interleaved gate/up projection [M][2I]
void launch_silu_f32(const float* gu, float* a, int M, int I, hipStream_t s);
// ---- fused decode projections (k_gemv.hip)
enum GvEpi : int { GV_HEAD = 0, GV_RESID = 1, GV_SILU = 2, GV_ROPE = 3,
                   GV_PART = 4 /* the partials part[split][M][N] of gemv_shape(..).ksplit >= 1 K splits, for their
                                  consumer to sum in order (router) */,
                   GV_F32 = 5 /* grouped experts only: float rows out_f32[row][n] */,
                   GV_GELU = 6 /* out_t[t][n] = bf16(gelu_tanh(acc + bias[n])) */ };

struct GemvArgs {
  const bf16* W;  // [N][K]
  int N, K, M;
  // B operand X [M][K] bf16.  Normalized operand (ss_in != nullptr): X holds
  // bf16(x * g) and the result is scaled by rsqrt(sum of squares / K + eps)
  const bf16* X;
  const float* ss_in;  // [ss_n][M] partial sums of squares of the rows of x
  int ss_n;
  float eps;
  // epilogue outputs
  float* out_f32;  // GV_HEAD logits [M][ldo] (may be null) / GV_RESID x [M][ldo]
  int ldo;
  bf16* out_t;     // GV_SILU a [M][ldo]
  float* ss_out;   // GV_RESID: [N / gemv_rows][M], or null
  bf16* xg_out;    // GV_RESID: bf16(x * gain_next) [M][ldo], or null (then ss_out too)
  const bf16* gain_next;
  float* am_val;   // GV_HEAD: [M][N / gemv_rows] partial maxima
  int32_t* am_idx;
  // GV_ROPE: [(H+2KV)hd] in the original (unpermuted) order; GV_RESID /
  // GV_GELU: [N] added to acc; or null
  const bf16* bias;
  const float* cos_t;
  const float* sin_t;
  bf16* q_out;  // [M][H][hd]
  KVView kv;
  const int32_t* len;   // token t is at position len[t] ...
  const int32_t* slot;  // ... of cache slot slot[t] (t when null)
  int H;
  // split K (residual projections of 17..64 tokens, GV_PART): workspace of ksplit
  // * M * N floats (gemv_workspace_floats), owned by the caller
  float* part;
  // grouped experts (launch_gemv_grouped): expert e multiplies W + e *
  // g_wstride with its rows g_off[e] .. g_off[e+1]-1; row r reads X row
  // g_xrow[r] (row r when g_xrow is NULL) and writes output row r (M is an
  // upper bound of any expert's rows)
  const int32_t* g_off;
  const int32_t* g_xrow;
  int64_t g_wstride;
  // tile order (xt_off) of the token operands, up to 16 tokens, unsplit
  // fused projections only: x_tiled -- X is stored in it; out_tiled -- the
  // epilogue writes xg_out (GV_RESID) or out_t (GV_SILU) in it
  int x_tiled;
  int out_tiled;
};
constexpr int GEMV_MAX_M = 64;      // token columns one fused projection handles
constexpr int GV_RESID_ROWS = 1024;  // features per workgroup of the split-K residual epilogue
struct GvShape {
  int rows, ks, u;  // output rows per workgroup, wavefronts splitting K, k-steps of 32 per stage
  int ksplit;       // workgroups splitting K (1: fused epilogue; else partials, summed by their consumer)
  int wide = 0;     // 1: gemv_wide_kernel (4 wavefronts splitting the rows, ks unused); 2: launch_gemm_few
};
// floats of GemvArgs::part a launch of this shape needs (0: none)
int64_t gemv_workspace_floats(int N, int K, int M, int epi);
GvShape gemv_shape(int N, int K, int M, int epi);
int gemv_rows(int N, int K, int M, int epi);  // output rows per workgroup (ss partial count = N / rows)
// false (nothing launched) when M > GEMV_MAX_M, for GV_F32, or when the
// normalization does not match the epilogue (GV_SILU needs ss_in, GV_RESID,
// GV_GELU and GV_PART must not have it)
bool launch_gemv_fused(const GemvArgs& a, int epi, hipStream_t s);
void launch_argmax_final(const float* val, const int32_t* idx, int nparts, int M, int32_t* next, int32_t* len,
                         hipStream_t s);
// Few-token grouped expert projections (mixture-of-experts decode): a
// workgroup per (64-row block, expert), the expert's rows (at most a.M <= 64)
// gathered through g_xrow; GV_SILU (out_t rows, interleaved gate/up W) or
// GV_F32 (out_f32 rows).  false when a.M > 64.
bool launch_gemv_grouped(const GemvArgs& a, int epi, int n_experts, hipStream_t s);
// xg_tiled: xg in the tile order of the few-token projections (M <= 16)
void launch_embed_ss(const int32_t* tok, const bf16* emb, const bf16* g, float* x, bf16* xg, float* ss_out, int M,
                     int D, int V, hipStream_t s, bool xg_tiled = false);

// ---- float32 few-token projections (k_gemv_f32.hip): float weights [N][K]
// row-major (QKV rows in the rotation-pair order, gate/up interleaved in
// blocks of 16 rows), up to GEMV_F32_MAX_M tokens, the epilogues of
// GV_ROPE / GV_SILU (normalized operand), GV_RESID, GV_HEAD (normalized)
struct GemvF32Args {
  const float* W;
  int N, K, M;
  const float* X;       // [M][K]: x * g (normalized operand) or the plain operand
  const float* ss_in;   // [ss_n][M] partial sums of squares of x, or null
  int ss_n;
  float eps;
  float* out;           // GV_RESID x [M][ldo] (+=) / GV_SILU a [M][ldo] / GV_HEAD logits [M][ldo] or null
  int ldo;
  float* xg_out;        // GV_RESID: x * gain_next [M][ldo], or null
  const float* gain_next;
  float* ss_out;        // GV_RESID: [gemv_f32_parts(N)][M]
  float* am_val;        // GV_HEAD: [M][gemv_f32_parts(N)] per-workgroup maxima
  int32_t* am_idx;
  const float* bias;    // GV_ROPE: [(H+2KV)hd] in the original head order, or null
  const float* cos_t;
  const float* sin_t;
  float* q_out;         // [M][H][hd]
  KVView kv;
  const int32_t* len;   // token t at position len[t] of slot slot[t] (t when null)
  const int32_t* slot;
  int H;
};
constexpr int GEMV_F32_MAX_M = 16;
// false (nothing launched) for more than GEMV_F32_MAX_M tokens or a shape or
// normalization the epilogue does not take
bool launch_gemv_f32_fused(const GemvF32Args& a, int epi, hipStream_t s);
int gemv_f32_parts(int N, int epi);  // workgroups of a launch (partials per token)
// Short-context decode (attention recomputed by every workgroup of the O
// projection): whether a step of M tokens with contexts up to max_ctx keys
// qualifies, and the fused attention + residual O projection (a: the
// GV_RESID projection with K = H * hd; q [M][H][hd]; token t at position
// a.len[t] of slot a.slot[t]).  false (nothing launched) outside those limits.
bool attn_o_f32_fits(int M, int H, int KVh, int hd, int max_ctx);
bool launch_attn_o_f32(const GemvF32Args& a, const float* q, KVView kv, hipStream_t s);
void launch_embed_ss_f32(const int32_t* tok, const float* emb, const float* g, float* x, float* xg, float* ss_out,
                         int M, int D, int V, hipStream_t s);

// ---- bias + rotary + KV-cache write (k_rope.hip)
// qkv rows are sum_s parts[s][t][:] (+ bias): q heads, then k heads, then v heads.
// Token t belongs to entry e(t) of cu: prefill puts it in slot ent_slot[e] at
// position ent_base[e] + t - cu[e] (slot e, position t - cu[e] when the arrays
// are null); decode (len != nullptr) uses slot t at position len[t].
template <typename T>
void launch_rope_kv(const float* parts, int nparts, int64_t part_stride, const T* bias, const float* cos_t,
                    const float* sin_t, T* q_out, KVView kv, int T_tokens, int nseq, const int32_t* cu,
                    const int32_t* len, int H, hipStream_t s, const int32_t* ent_slot = nullptr,
                    const int32_t* ent_base = nullptr);

// ---- attention (k_attn.hip)
// Causal prefill attention over the cache; o [T][H*hd] (bf16 with o_pair: in
// the row-pair layout, xp_off with K = H*hd).  The workgroups cover
// the nseq entries listed in ents (device) / h_ents (host copy), or entries
// 0..nseq-1 when both are null; entry e's tokens cu[e] .. cu[e+1]-1 are at
// positions ent_base[e] + 0, 1, ... of slot ent_slot[e] and attend to every
// earlier key of that slot (null arrays: slot e from position 0).
template <typename T>
void launch_attn_prefill(const T* q, KVView kv, T* o, int T_tokens, int nseq, const int32_t* cu,
                         const int32_t* h_cu, int H, hipStream_t s, const int32_t* ents = nullptr,
                         const int32_t* h_ents = nullptr, const int32_t* ent_slot = nullptr,
                         const int32_t* ent_base = nullptr, float* lse = nullptr, bool o_pair = false);
// Decode attention: one query per slot at position len[b] (after the step's
// key/value were written), context len[b] + 1; keys split over
// plan_decode_splits() workgroups per (slot, kv head).  ``part`` holds
// B * H * splits * (hd + 2) floats; the last split of a (slot, kv head)
// merges them.
int plan_decode_splits(int B, int kv_heads, int max_ctx);
// Item b reads query row rows[b] and writes output row rows[b] (b when null),
// in cache slot slots[b] (b when null), at position len[b]; bf16 only for the
// indirection (the float32 path reaches such items through launch_attn_prefill).
// p[0 .. n) = 0, as a kernel (graph-capture safe)
void launch_zero_i32(int32_t* p, int n, hipStream_t s);
// cnt: int32 [B][kv heads], zero before the launch and left zero after it
// (split arrival counters).  o_tiled (bf16, B <= 16, no rows): o [B][H hd]
// in the tile order of the few-token projections (xt_off).
template <typename T>
void launch_attn_decode(const T* q, KVView kv, T* o, float* part, int32_t* cnt, int B, int H, const int32_t* len,
                        int max_ctx, hipStream_t s, const int32_t* rows = nullptr,
                        const int32_t* slots = nullptr, bool o_tiled = false);

// ---- mixture of experts (k_moe.hip)
// topi / topw [T][k]: the top_k experts of each token (E <= 256, k <= 8) from
// float logits [T][ldl] (the sum of nparts partials ``stride`` apart), and their
// softmax probabilities (over all E), divided by their sum when norm
void launch_moe_route(const float* logits, int nparts, int64_t stride, int ldl, int T, int E, int k, int norm,
                      int32_t* topi, float* topw, hipStream_t s);
// grouped-GEMM plan of the T*k choices: cnt [E], off / toff [E+1] (rows and
// 256-row tiles before each expert), xrow [T*k] (token of each grouped row),
// inv [T*k] (grouped row of choice t*k + j)
void launch_moe_plan(const int32_t* topi, int T, int E, int k, int32_t* cnt, int32_t* off, int32_t* toff,
                     int32_t* xrow, int32_t* inv, hipStream_t s);
// out[r] = h[xrow[r]] for r < rows (bf16 rows of D, D % 8 == 0)
void launch_moe_gather(const bf16* h, const int32_t* xrow, int rows, int D, bf16* out, hipStream_t s);
// x[t] += sum_j w[t][j] * y[inv[t*k+j]] (float rows of D, D % 4 == 0).  With
// xg: also xg = bf16(x * g) and per-token sums of squares of the new x in
// moe_combine_blocks(D) partials, ss_out[part * T + t].
inline int moe_combine_blocks(int D) { return (D / 4 + 255) / 256; }
void launch_moe_combine(float* x, const float* y, const int32_t* inv, const float* w, int T, int D, int k,
                        hipStream_t s, const bf16* g = nullptr, bf16* xg = nullptr, float* ss_out = nullptr);

}  // namespace axon
