// Backward pass of the Llama-family decoder (training): the loss, the
// reverse of each forward step that is not a projection, and the layout
// helpers that let the projection gradients run on the prefill GEMM.
//
// Every projection Y = X W^T (X [T][K], W [N][K]) has two gradients: dX = dY W,
// run by the prefill GEMM on W^T, and dW = dY^T X,
// so the weights get a transposed tiled copy once; the weight gradients read the
// token-major operands as they are (gemm_tn_256_kernel).  Every GEMM operand
// lies in the row-pair layout (xp_off).
//
// Attention backward recomputes the probabilities from the forward pass's
// per-(query, head) log2-sum-exp: P = 2^(s sc - lse) with sc = log2(e) /
// sqrt(hd); dP = dO V^T; dS = P (dP - D) with D = rowsum(dO O); dQ = dS K /
// sqrt(hd); dK = dS^T Q / sqrt(hd); dV = P^T dO, all on the matrix cores.
// A wavefront accumulates dQ of 32 queries of a head over the keys, or one query
// head's share of dK and dV of 32 keys over the later queries; the shares of a
// group's heads are summed in order.  No atomics, so every gradient but the
// embedding's is deterministic.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace axon {

constexpr float LOG2E = 1.4426950408889634f;

AXON_DEV float block_max(float v, float* red) {
  v = wave_max(v);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
  __syncthreads();
  if (lane == 0) red[w] = v;
  __syncthreads();
  float m = -INFINITY;
  for (int i = 0; i < nw; ++i) m = fmaxf(m, red[i]);
  return m;
}

// ---------------------------------------------------------------- the loss

// Row t: lse = log sum_v exp(logit_v) over v < V, merged from the np (largest,
// sum) partials of its 64-column pieces; a target in [0, V) counts (rowloss =
// lse - logit_target, valid = 1), any other value does not (0, 0).
__global__ void __launch_bounds__(256) ce_rows_kernel(const float* __restrict__ logits, int ldl, int V,
                                                      const float2* __restrict__ part, int np,
                                                      const int32_t* __restrict__ targets,
                                                      float* __restrict__ rowloss, float* __restrict__ valid,
                                                      float* __restrict__ lse_out) {
  __shared__ float red[16];
  const int t = blockIdx.x;
  const float2* row = part + (int64_t)t * np;
  float mx = -INFINITY;
  for (int i = threadIdx.x; i < np; i += 256) mx = fmaxf(mx, row[i].x);
  mx = block_max(mx, red);
  float sum = 0.f;
  for (int i = threadIdx.x; i < np; i += 256) sum += row[i].y * __expf(row[i].x - mx);
  sum = block_sum(sum, red);
  if (threadIdx.x == 0) {
    const float lse = mx + __logf(sum);
    const int tg = targets[t];
    const bool ok = tg >= 0 && tg < V;
    rowloss[t] = ok ? lse - logits[(int64_t)t * ldl + tg] : 0.f;
    valid[t] = ok ? 1.f : 0.f;
    lse_out[t] = lse;
  }
}

// loss = sum(rowloss) / N over the N counted rows (0 when none); scal[0] = 1/N
// (0 when none).  One workgroup, fixed summation order.
__global__ void __launch_bounds__(256) ce_reduce_kernel(const float* __restrict__ rowloss,
                                                        const float* __restrict__ valid, int T,
                                                        float* __restrict__ loss, float* __restrict__ scal) {
  __shared__ float red[16];
  float s = 0.f, n = 0.f;
  for (int t = threadIdx.x; t < T; t += 256) {
    s += rowloss[t];
    n += valid[t];
  }
  s = block_sum(s, red);
  n = block_sum(n, red);
  if (threadIdx.x == 0) {
    loss[0] = n > 0.f ? s / n : 0.f;
    scal[0] = n > 0.f ? 1.f / n : 0.f;
  }
}

// dlogits[t][v] = (softmax_v - [v == target]) / N for counted rows, else 0;
// columns V .. ldl-1 are zero; dlog in the row-pair layout.  8 columns per
// thread (ldl % 32 == 0), every load unconditional 16 bytes (the padding columns
// hold whatever the buffer held and are not used); 8 lanes fill one 128-byte line of
// a row pair.
__global__ void __launch_bounds__(256) ce_grad_kernel(const float* __restrict__ logits, int ldl, int V, int T,
                                                      const int32_t* __restrict__ targets,
                                                      const float* __restrict__ valid,
                                                      const float* __restrict__ lse, const float* __restrict__ scal,
                                                      bf16* __restrict__ dlog) {
  const int tid = threadIdx.x;
  const int t = blockIdx.y * 2 + ((tid >> 2) & 1);
  const int v0 = (blockIdx.x * 32 + (tid >> 3)) * 32 + (tid & 3) * 8;
  if (t >= T || v0 >= ldl) return;
  const float* row = logits + (int64_t)t * ldl + v0;
  const f32x4 lo = *(const f32x4*)row, hi = *(const f32x4*)(row + 4);
  const bool ok = valid[t] > 0.f;
  const float l = lse[t], inv = scal[0];
  const int tg = targets[t];
  bf16x8 o;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int v = v0 + j;
    const float x = j < 4 ? lo[j & 3] : hi[j & 3];
    const float g = (__expf(x - l) - (v == tg ? 1.f : 0.f)) * inv;
    o[j] = (bf16)(ok && v < V ? g : 0.f);
  }
  *(bf16x8*)(dlog + xp_off(t, v0, ldl)) = o;
}

// ---------------------------------------------------------------- layouts

// dst[k][n] = W[n][k] from the fragment-tiled W [N][K]; dst rows are Np
// apart (the caller zeroes columns N .. Np-1)
__global__ void __launch_bounds__(256) untile_transpose_kernel(const bf16* __restrict__ W, int64_t N, int K,
                                                               bf16* __restrict__ dst, int64_t Np) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;  // (n, k-chunk)
  const int kc = K / 8;
  if (q >= N * kc) return;
  const int64_t n = q / kc;
  const int c = (int)(q % kc);
  const bf16x8 v = *(const bf16x8*)(W + wt_chunk(n, c, K));
#pragma unroll
  for (int j = 0; j < 8; ++j) dst[(int64_t)(c * 8 + j) * Np + n] = v[j];
}

// ---------------------------------------------------------------- norms

// RMSNorm y = x r g, r = rsqrt(mean(x^2) + eps): dx (= or +=) r g dy - x r^3
// mean(g dy x), the gain's gradient dy x r summed over rows, and dx in bf16 (the
// next projections' operand, row-pair layout).  dy arrives as the np split-K
// partials of the GEMM that made it (in order).  HBM bound.  A workgroup takes
// ``rows`` rows, a thread the same columns (4 NV of them) of each, so the gain's
// terms stay in registers until one partial row per workgroup is left for the
// column sum; the next row's operands are loaded before this row's reduction (one
// barrier per row, its slots alternating).  The separate kernels for dx, the
// gain's terms through memory, their column sum, the partials' sum and the bf16
// copy took 100 us on 4096 x 2048; this one and the column sum 37 us (182 MB: 4.9 TB/s).
template <int NV>
__global__ void __launch_bounds__(256) norm_bwd_kernel(const float* __restrict__ x, const bf16* __restrict__ g,
                                                       const float* __restrict__ dy, int np, int64_t stride, int T,
                                                       int D, float eps, float* __restrict__ dx, int accumulate,
                                                       bf16* __restrict__ dxb, float* __restrict__ gpart, int rows) {
  __shared__ float red[2][2][4];
  const int tid = threadIdx.x, wave = tid >> 6;
  const int t0 = blockIdx.x * rows, t1 = min(T, t0 + rows);
  int col[NV];
  bool own[NV];
  f32x4 gv[NV], gsum[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int c = (v * 256 + tid) * 4;
    own[v] = c < D;
    col[v] = min(c, D - 4);  // columns past D: the last ones again, not counted
    const bf16x4 b = *(const bf16x4*)(g + col[v]);
    gv[v] = f32x4{(float)b[0], (float)b[1], (float)b[2], (float)b[3]};
    gsum[v] = f32x4{};
  }
  f32x4 xn[NV], dn[NV], an[NV];
  auto load = [&](int t) {
    const int64_t base = (int64_t)t * D;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      xn[v] = *(const f32x4*)(x + base + col[v]);
      dn[v] = *(const f32x4*)(dy + base + col[v]);
      an[v] = accumulate ? *(const f32x4*)(dx + base + col[v]) : f32x4{};
    }
    for (int p = 1; p < np; ++p)
#pragma unroll
      for (int v = 0; v < NV; ++v) dn[v] += *(const f32x4*)(dy + p * stride + base + col[v]);
  };
  load(t0);
  for (int t = t0; t < t1; ++t) {
    f32x4 xc[NV], dc[NV], ac[NV];
    float ss = 0.f, sgd = 0.f;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      xc[v] = xn[v];
      dc[v] = dn[v];
      ac[v] = an[v];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        ss += own[v] ? xc[v][j] * xc[v][j] : 0.f;
        sgd += own[v] ? gv[v][j] * dc[v][j] * xc[v][j] : 0.f;
      }
    }
    if (t + 1 < t1) load(t + 1);
    ss = wave_sum(ss);
    sgd = wave_sum(sgd);
    const int par = (t - t0) & 1;
    if ((tid & 63) == 0) {
      red[par][0][wave] = ss;
      red[par][1][wave] = sgd;
    }
    __syncthreads();
    ss = (red[par][0][0] + red[par][0][1]) + (red[par][0][2] + red[par][0][3]);
    sgd = (red[par][1][0] + red[par][1][1]) + (red[par][1][2] + red[par][1][3]);
    const float r = rsqrtf(ss / (float)D + eps), c = r * r * r * sgd / (float)D;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const f32x4 o = ac[v] + (gv[v] * dc[v] * r - xc[v] * c);
      gsum[v] += dc[v] * xc[v] * r;
      if (own[v]) {
        *(f32x4*)(dx + (int64_t)t * D + col[v]) = o;
        *(bf16x4*)(dxb + xp_off(t, col[v], D)) = bf16x4{(bf16)o[0], (bf16)o[1], (bf16)o[2], (bf16)o[3]};
      }
    }
  }
#pragma unroll
  for (int v = 0; v < NV; ++v)
    if (own[v]) *(f32x4*)(gpart + (int64_t)blockIdx.x * D + col[v]) = gsum[v];
}

// The same for D past the register form (8192): dgrow [T][D] receives the
// gain's terms, which colsum_part_kernel sums.
__global__ void __launch_bounds__(256) norm_bwd_wide_kernel(const float* __restrict__ x, const bf16* __restrict__ g,
                                                            const float* __restrict__ dy, int np, int64_t stride, int D,
                                                            float eps, float* __restrict__ dx, int accumulate,
                                                            bf16* __restrict__ dxb, float* __restrict__ dgrow) {
  __shared__ float red[16];
  const int64_t t = blockIdx.x, base = t * D;
  auto grad = [&](int i) {
    float d = dy[base + i];
    for (int p = 1; p < np; ++p) d += dy[p * stride + base + i];
    return d;
  };
  float ss = 0.f, sgd = 0.f;
  for (int i = threadIdx.x; i < D; i += 256) {
    const float xv = x[base + i];
    ss += xv * xv;
    sgd += (float)g[i] * grad(i) * xv;
  }
  ss = block_sum(ss, red);
  sgd = block_sum(sgd, red);
  const float r = rsqrtf(ss / (float)D + eps), c = r * r * r * sgd / (float)D;
  for (int i = threadIdx.x; i < D; i += 256) {
    const float xv = x[base + i], d = grad(i);
    const float v = r * (float)g[i] * d - xv * c + (accumulate ? dx[base + i] : 0.f);
    dx[base + i] = v;
    dxb[xp_off(t, i, D)] = (bf16)v;
    dgrow[base + i] = d * xv * r;
  }
}

// column sums of src [T][C] over rows chunk*rpc ..: part[chunk][c]
__global__ void __launch_bounds__(256) colsum_part_kernel(const float* __restrict__ src, int T, int C, int rpc,
                                                          float* __restrict__ part) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= C) return;
  const int t0 = blockIdx.y * rpc, t1 = min(T, t0 + rpc);
  float s = 0.f;
  for (int t = t0; t < t1; ++t) s += src[(int64_t)t * C + c];
  part[(int64_t)blockIdx.y * C + c] = s;
}

// The column sum's second pass: column c of part [n][C], the partials in 16
// interleaved groups of fixed order, then the groups in order.  Columns below
// c1 go to d0, below c2 to d1, the rest to d2.
__global__ void __launch_bounds__(1024) colsum_final_kernel(const float* __restrict__ part, int n, int C,
                                                            float* __restrict__ d0, int c1, float* __restrict__ d1,
                                                            int c2, float* __restrict__ d2) {
  __shared__ float sums[16][64];
  const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int c = blockIdx.x * 64 + lane;
  float s = 0.f;
  for (int i0 = grp; i0 < n; i0 += 16 * 8) {
    float v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = part[(int64_t)min(i0 + q * 16, n - 1) * C + min(c, C - 1)];
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (i0 + q * 16 < n) s += v[q];
  }
  sums[grp][lane] = s;
  __syncthreads();
  if (grp > 0 || c >= C) return;
  s = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) s += sums[i][lane];
  if (c < c1) d0[c] = s;
  else if (c < c2) d1[c - c1] = s;
  else d2[c - c2] = s;
}

// ---------------------------------------------------------------- attention

// dO in bf16 from the np split-K partials of its GEMM (in order), and D[t][h] =
// sum_d dO[t][h][d] O[t][h][d] (dO rounded; O in the row-pair layout).  A thread
// takes 8 dims.
template <int HD>
__global__ void __launch_bounds__(256) attn_bwd_do_kernel(const float* __restrict__ dof, int np, int64_t stride,
                                                          const bf16* __restrict__ o, int T, int H,
                                                          bf16* __restrict__ dob, float* __restrict__ dsum) {
  constexpr int LPH = HD / 8;  // lanes of a head
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t th = min(idx / LPH, (int64_t)T * H - 1);  // past the end: the last head again, not stored
  const int d0 = (int)(idx % LPH) * 8, t = (int)(th / H), h = (int)(th % H);
  const float* src = dof + th * HD + d0;
  f32x4 lo = *(const f32x4*)src, hi = *(const f32x4*)(src + 4);
  for (int p = 1; p < np; ++p) {
    lo += *(const f32x4*)(src + p * stride);
    hi += *(const f32x4*)(src + p * stride + 4);
  }
  const bf16x8 ov = *(const bf16x8*)(o + xp_off(t, h * HD + d0, H * HD));
  bf16x8 b;
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    b[j] = (bf16)(j < 4 ? lo[j & 3] : hi[j & 3]);
    s += (float)b[j] * (float)ov[j];
  }
  // over the 8 or 16 lanes of the head (see wave_sum)
  s += dpp_move<0xB1>(s);
  s += dpp_move<0x4E>(s);
  s += dpp_move<0x141>(s);
  if constexpr (LPH == 16) s += dpp_move<0x140>(s);
  if (idx / LPH >= (int64_t)T * H) return;
  *(bf16x8*)(dob + th * HD + d0) = b;
  if (d0 == 0) dsum[th] = s;
}

// ---- MFMA attention backward.  v_mfma_f32_32x32x16_bf16 with lane L, half
// hl = L / 32, column c = L % 32: A operand = row c, k = 8 hl .. 8 hl + 7;
// B operand = column c, the same k; accumulator element i = row (i/4)*8 +
// 4 hl + i%4, column c.  The accumulator of a 32 x 32 block therefore holds,
// per lane, 16 rows of one column: taken 8 at a time (k-steps kk = 0, 1) it
// is directly a B operand whose k slot (hl, j) stands for row kk*16 +
// (j/4)*8 + 4 hl + j%4, and the A operand of that product reads its rows in
// the same order: two runs of 4 consecutive positions, each one transposing LDS
// read (read_tr8).
//
// Both kernels share a sequence's tiles among the 4 wavefronts of a workgroup
// (32 queries or keys each, 128 together) through a ring of LDS stages filled by
// direct copies: dQ streams 32-key tiles of the cache's K and V^T blocks, dK / dV
// 32-query tiles of Q and dO rows with their statistics.  Rows, columns and both
// transposes come from the one tile.  One wavefront per block reading packed,
// transposed copies from L2 waited for each block's loads in turn (1B shape, 8 x
// 512 tokens: dQ 130 us, dK / dV 136, the copies 71; now 47 and 74).  The launch
// bounds keep the accumulators out of the second register file half (67 and 88 us
// without), except dK / dV of head dimension 128: 256 + 159 registers, one
// wavefront per SIMD.

// the ``rows``-position block blk of the sequences in order: (sequence, first position)
AXON_DEV void locate_block(const int32_t* __restrict__ cu, int nseq, int blk, int rows, int& e, int& p0) {
  for (e = 0; e < nseq - 1; ++e) {
    const int nb = (cu[e + 1] - cu[e] + rows - 1) / rows;
    if (blk < nb) break;
    blk -= nb;
  }
  p0 = blk * rows;
}

constexpr int BWD_ROWS = 128;  // queries (dQ) or keys (dK / dV) of a workgroup

// dS as a bf16 pair hi + lo: a row of dS sums to zero, so dQ = dS K and dK =
// dS^T Q cancel, and rounding dS to one bf16 would leave an error of 2^-9 of the
// row's absolute sum times the keys' (queries') common part
AXON_DEV void split_bf16(float v, bf16& hi, bf16& lo) {
  hi = (bf16)v;
  lo = (bf16)(v - (float)hi);
}

// dQ of 128 queries (one head): over the key tiles up to the last query, S^T =
// K Q^T and dP^T = V dO^T (k = head dim), then dQ^T += K^T dS^T (k = the tile's 32
// keys).  Workgroups of late queries (the most tiles) come first.
template <int HD, int S>
__global__ void __launch_bounds__(256, HD == 64 ? 3 : 2) attn_bwd_dq_kernel(const bf16* __restrict__ q, const bf16* __restrict__ dob,
                                                          KVView kv, const float* __restrict__ lse,
                                                          const float* __restrict__ dsum,
                                                          const int32_t* __restrict__ cu, int nseq, int H,
                                                          float* __restrict__ dq) {
  constexpr int KL = HD / 64, LPT = 2 * KL;  // copies per wavefront and tile: K, and with V
  constexpr int PANEL = HD * 4, STAGE = 2 * PANEL;  // 16-byte chunks: 32 keys of K; K and V
  __shared__ bf16x8 ring[S * STAGE];
  int e, q0;
  locate_block(cu, nseq, gridDim.x - 1 - blockIdx.x, BWD_ROWS, e, q0);
  const int h = blockIdx.y, KVh = kv.kv_heads, kvh = h / (H / KVh);
  const int tok0 = cu[e], N = cu[e + 1] - tok0;
  const int tid = threadIdx.x, lane = tid & 63, hl = lane >> 5, c = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qw = q0 + wave * 32, myq = qw + c;
  const bf16* ks = (const bf16*)kv.k + ((int64_t)e * KVh + kvh) * kv.ps * HD;
  const bf16* vs = (const bf16*)kv.v + ((int64_t)e * KVh + kvh) * kv.ps * HD;
  // keys past the sequence read its last key, V^T blocks past it its last block
  auto issue = [&](int kt) {
    bf16x8* base = ring + (kt % S) * STAGE;
#pragma unroll
    for (int j = 0; j < KL; ++j) {
      const int i = j * 4 + wave, ch = i * 64 + lane, r = ch % (2 * HD);
      const int key = min(kt * 32 + ch / (2 * HD) * 16 + r % 16, N - 1);
      load_lds16(ks + (int64_t)(key >> 4) * 16 * HD + r / 16 * 128 + (key & 15) * 8, base + i * 64);
      const int blk = min(kt * 2 + ch / (2 * HD), (N - 1) >> 4);
      load_lds16(vs + (int64_t)blk * 16 * HD + r * 8, base + PANEL + i * 64);
    }
  };
  const int nkt = (min(N, q0 + BWD_ROWS) + 31) / 32;  // tiles of the workgroup
  const int mine = qw < N ? (min(N, qw + 32) + 31) / 32 : 0;
#pragma unroll
  for (int st = 0; st < S - 1; ++st)
    if (st < nkt) issue(st);

  const int64_t tq = tok0 + min(myq, N - 1);  // columns past the sequence read its last query (not stored)
  bf16x8 qf[HD / 16], df[HD / 16];
#pragma unroll
  for (int s = 0; s < HD / 16; ++s) {
    qf[s] = *(const bf16x8*)(q + (tq * H + h) * HD + s * 16 + hl * 8);
    df[s] = *(const bf16x8*)(dob + (tq * H + h) * HD + s * 16 + hl * 8);
  }
  const float sc = LOG2E / sqrtf((float)HD);
  const float l2 = lse[tq * H + h], Dq = dsum[tq * H + h];
  f32x16 acc[HD / 32];
#pragma unroll
  for (int b = 0; b < HD / 32; ++b) acc[b] = f32x16{};
  // lane offsets inside a tile (elements): K row c; V^T read, 16 keys (lane / 16)
  // % 2 of dims 8 hl + (lane % 16) / 4; K^T read, keys 4 hl + (lane % 16) / 4 of
  // dims 16 ((lane / 16) % 2) + 4 (lane % 4)
  const int g16 = (lane >> 4) & 1, r4 = (lane >> 2) & 3, c4 = lane & 3;
  const int krow = (c >> 4) * 16 * HD + hl * 128 + (c & 15) * 8;
  const int vtr = g16 * 16 * HD + (hl * 8 + r4) * 16 + c4 * 4;
  const int ktr = (g16 * 2 + (c4 >> 1)) * 128 + (hl * 4 + r4) * 8 + (c4 & 1) * 4;
  for (int kt = 0; kt < nkt; ++kt) {
    wait_loads<LPT, S - 2>(min(S - 2, nkt - 1 - kt));
    phase_barrier();
    if (kt + S - 1 < nkt) issue(kt + S - 1);
    if (kt >= mine) continue;  // wave-uniform; the barriers are at the top
    const bf16* K = (const bf16*)(ring + (kt % S) * STAGE);
    const bf16* V = K + PANEL * 8;
    f32x16 st = {}, dpt = {};
#pragma unroll
    for (int s = 0; s < HD / 16; ++s) {
      st = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8*)(K + krow + s * 256), qf[s], st, 0, 0, 0);
      dpt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_tr8(V + vtr + s * 256, V + vtr + s * 256 + 64), df[s], dpt, 0,
                                                    0, 0);
    }
    bf16x8 dsh[2], dsl[2];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int key = kt * 32 + (i >> 2) * 8 + hl * 4 + (i & 3);
      const float p = __builtin_amdgcn_exp2f(st[i] * sc - l2);
      const float ds = key <= myq && myq < N ? p * (dpt[i] - Dq) : 0.f;
      bf16 hi, lo;
      split_bf16(ds, hi, lo);
      dsh[i >> 3][i & 7] = hi;
      dsl[i >> 3][i & 7] = lo;
    }
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int b = 0; b < HD / 32; ++b) {
        const bf16* p = K + kk * 16 * HD + b * 512 + ktr;
        const bf16x8 a = read_tr8(p, p + 64);
        acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, dsh[kk], acc[b], 0, 0, 0);
        acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, dsl[kk], acc[b], 0, 0, 0);
      }
  }
  if (myq >= N) return;
  const float rs = 1.f / sqrtf((float)HD);
  float* out = dq + ((int64_t)(tok0 + myq) * H + h) * HD;
#pragma unroll
  for (int b = 0; b < HD / 32; ++b)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int d = b * 32 + g * 8 + hl * 4;
      *(f32x4*)(out + d) = f32x4{acc[b][g * 4] * rs, acc[b][g * 4 + 1] * rs, acc[b][g * 4 + 2] * rs,
                                 acc[b][g * 4 + 3] * rs};
    }
}

// dK and dV of 128 keys from one query head h = blockIdx.y (kv head h / group):
// over the query tiles from the first key on, S = Q K^T and dP = dO V^T (k =
// head dim), then dV^T += dO^T P and dK^T += Q^T dS (k = the tile's 32
// queries).  Writes the head's share into dk / dv [T][H][hd] (the heads of a
// group are summed by rope_bwd_kernel).
template <int HD, int S>
__global__ void __launch_bounds__(256, HD == 64 ? 2 : 1) attn_bwd_dkv_kernel(const bf16* __restrict__ q, const bf16* __restrict__ dob,
                                                           KVView kv, const float* __restrict__ lse,
                                                           const float* __restrict__ dsum,
                                                           const int32_t* __restrict__ cu, int nseq, int H,
                                                           float* __restrict__ dk, float* __restrict__ dv) {
  constexpr int RL = HD / 64, LPT = 2 * RL + 1;     // copies per wavefront and tile: Q rows; with dO and statistics
  constexpr int CH = HD / 8;                        // 16-byte chunks of a row
  constexpr int PANEL = 32 * CH, STAGE = 2 * PANEL;
  __shared__ bf16x8 ring[S * STAGE];
  __shared__ float stats[S][4][64];  // per wavefront (its own copy): 32 log2-sum-exp, 32 D
  int e, k0;
  locate_block(cu, nseq, blockIdx.x, BWD_ROWS, e, k0);
  const int h = blockIdx.y, KVh = kv.kv_heads, kvh = h / (H / KVh);
  const int tok0 = cu[e], N = cu[e + 1] - tok0;
  const int tid = threadIdx.x, lane = tid & 63, hl = lane >> 5, c = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kw = k0 + wave * 32, mykey = kw + c;
  const bf16* ks = (const bf16*)kv.k + ((int64_t)e * KVh + kvh) * kv.ps * HD;
  const bf16* vs = (const bf16*)kv.v + ((int64_t)e * KVh + kvh) * kv.ps * HD;
  const int g16 = (lane >> 4) & 1, r4 = (lane >> 2) & 3, c4 = lane & 3;

  // this wavefront's keys as B operands: K rows from the cache, V rows through a
  // transposing read of its V^T blocks (staged in the ring before its first use);
  // keys past the sequence: its last key (block), not stored
  bf16x8 kf[HD / 16], vf[HD / 16];
  {
    static_assert(S * STAGE >= 4 * 4 * HD, "the ring holds every wavefront's V tile");
    bf16x8* tile = ring + wave * 4 * HD;
#pragma unroll
    for (int j = 0; j < HD / 16; ++j) {
      const int ch = j * 64 + lane, blk = min((kw >> 4) + ch / (2 * HD), (N - 1) >> 4);
      load_lds16(vs + (int64_t)blk * 16 * HD + ch % (2 * HD) * 8, tile + j * 64);
    }
    const int key = min(mykey, N - 1);
#pragma unroll
    for (int s = 0; s < HD / 16; ++s)
      kf[s] = *(const bf16x8*)(ks + (int64_t)(key >> 4) * 16 * HD + (s * 2 + hl) * 128 + (key & 15) * 8);
    wait_loads<1, 0>(0);
    const bf16* p = (const bf16*)tile + g16 * 16 * HD + (hl * 8 + r4) * 16 + c4 * 4;
#pragma unroll
    for (int s = 0; s < HD / 16; ++s) vf[s] = read_tr8(p + s * 256, p + s * 256 + 64);
    __syncthreads();  // every V tile has been read: the ring is free
  }

  // chunk c of tile row r sits at chunk c ^ key(r): 16 rows' reads of one chunk
  // hit distinct banks
  auto swzkey = [](int r) { return HD == 64 ? (r >> 1) & 7 : r & 15; };
  const int qt0 = k0 / 32, nqt = (N + 31) / 32;
  auto issue = [&](int qt) {  // rows past the sequence read its last query
    bf16x8* base = ring + ((qt - qt0) % S) * STAGE;
#pragma unroll
    for (int j = 0; j < RL; ++j) {
      const int i = j * 4 + wave, ch = i * 64 + lane, row = ch / CH, cc = ch % CH ^ swzkey(row);
      const int64_t at = ((int64_t)(tok0 + min(qt * 32 + row, N - 1)) * H + h) * HD + cc * 8;
      load_lds16(q + at, base + i * 64);
      load_lds16(dob + at, base + PANEL + i * 64);
    }
    load_lds4((lane < 32 ? lse : dsum) + (int64_t)(tok0 + min(qt * 32 + c, N - 1)) * H + h,
              &stats[(qt - qt0) % S][wave][0]);
  };
#pragma unroll
  for (int st = 0; st < S - 1; ++st)
    if (qt0 + st < nqt) issue(qt0 + st);

  const float sc = LOG2E / sqrtf((float)HD);
  f32x16 akk[HD / 32], avv[HD / 32];
#pragma unroll
  for (int b = 0; b < HD / 32; ++b) {
    akk[b] = f32x16{};
    avv[b] = f32x16{};
  }
  for (int qt = qt0; qt < nqt; ++qt) {
    wait_loads<LPT, S - 2>(min(S - 2, nqt - 1 - qt));
    phase_barrier();
    if (qt + S - 1 < nqt) issue(qt + S - 1);
    if (qt * 32 < kw || kw >= N) continue;  // wave-uniform; the barriers are at the top
    const bf16* Q = (const bf16*)(ring + ((qt - qt0) % S) * STAGE);
    const bf16* O = Q + PANEL * 8;
    f32x16 sq = {}, dpq = {};
#pragma unroll
    for (int s = 0; s < HD / 16; ++s) {
      const int at = c * HD + ((s * 2 + hl) ^ swzkey(c)) * 8;
      sq = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8*)(Q + at), kf[s], sq, 0, 0, 0);
      dpq = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8*)(O + at), vf[s], dpq, 0, 0, 0);
    }
    const float* stt = &stats[(qt - qt0) % S][wave][0];
    f32x4 lq[4], dq4[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      lq[g] = *(const f32x4*)(stt + g * 8 + hl * 4);
      dq4[g] = *(const f32x4*)(stt + 32 + g * 8 + hl * 4);
    }
    // P in bf16, dS as a bf16 pair
    bf16x8 pb[2], dsh[2], dsl[2];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int qi = qt * 32 + (i >> 2) * 8 + hl * 4 + (i & 3);
      const bool ok = qi < N && mykey <= qi;
      const float p = ok ? __builtin_amdgcn_exp2f(sq[i] * sc - lq[i >> 2][i & 3]) : 0.f;
      pb[i >> 3][i & 7] = (bf16)p;
      const float ds = ok ? p * (dpq[i] - dq4[i >> 2][i & 3]) : 0.f;
      bf16 hi, lo;
      split_bf16(ds, hi, lo);
      dsh[i >> 3][i & 7] = hi;
      dsl[i >> 3][i & 7] = lo;
    }
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      // rows of the transposing reads: queries kk * 16 + 4 hl + (lane % 16) / 4, + 8
      const int r0 = kk * 16 + hl * 4 + r4, r1 = r0 + 8;
#pragma unroll
      for (int b = 0; b < HD / 32; ++b) {
        const int ch = b * 4 + g16 * 2 + (c4 >> 1), sub = (c4 & 1) * 4;
        const int a0 = r0 * HD + (ch ^ swzkey(r0)) * 8 + sub, a1 = r1 * HD + (ch ^ swzkey(r1)) * 8 + sub;
        const bf16x8 ao = read_tr8(O + a0, O + a1);
        const bf16x8 aq = read_tr8(Q + a0, Q + a1);
        avv[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ao, pb[kk], avv[b], 0, 0, 0);
        akk[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aq, dsh[kk], akk[b], 0, 0, 0);
        akk[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aq, dsl[kk], akk[b], 0, 0, 0);
      }
    }
  }
  if (mykey >= N) return;
  const float rs = 1.f / sqrtf((float)HD);
  const int64_t orow = ((int64_t)(tok0 + mykey) * H + h) * HD;
#pragma unroll
  for (int b = 0; b < HD / 32; ++b)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int d = b * 32 + g * 8 + hl * 4;
      *(f32x4*)(dk + orow + d) = f32x4{akk[b][g * 4] * rs, akk[b][g * 4 + 1] * rs, akk[b][g * 4 + 2] * rs,
                                       akk[b][g * 4 + 3] * rs};
      *(f32x4*)(dv + orow + d) = f32x4{avv[b][g * 4], avv[b][g * 4 + 1], avv[b][g * 4 + 2], avv[b][g * 4 + 3]};
    }
}

// Gradients at the rotated q / k and at v back through RoPE (the transpose of
// a rotation rotates by the opposite angle) into the fused QKV layout: dqkv
// [T][nq] bf16 in the projection's row order (within a head, groups of 8 = 4
// first halves and their partners), row-pair layout.  dkh / dvh hold a share per
// query head; a kv head's are summed in head order.  A thread owns one 8-row
// group (16-byte loads and stores) over ``rows`` tokens, so that with bpart the
// bias gradient's column sums [workgroup][nq] (original row order) stay in
// registers.  One thread per rotation pair, with the share sum and a float32 copy
// of dqkv for the bias as passes of their own, took 46 us on 4096 x 3072; this
// kernel 27 us (125 MB).
__global__ void __launch_bounds__(128) rope_bwd_kernel(const float* __restrict__ dq, const float* __restrict__ dkh,
                                                       const float* __restrict__ dvh, const float* __restrict__ cos_t,
                                                       const float* __restrict__ sin_t,
                                                       const int32_t* __restrict__ cu, int nseq, int T, int H,
                                                       int KVh, int hd, bf16* __restrict__ dqkv,
                                                       float* __restrict__ bpart, int rows) {
  const int half = hd / 2, NH = H + 2 * KVh, nq = NH * hd, group = H / KVh;
  const int item = blockIdx.x * 128 + threadIdx.x;
  if (item >= nq / 8) return;
  const int hh = item / (hd / 8), i0 = item % (hd / 8) * 4;  // rotation pairs i0 .. i0 + 3 of head hh
  const int t0 = blockIdx.y * rows, t1 = min(T, t0 + rows);
  const bool rot = hh < H + KVh;
  const float* src = hh < H ? dq : hh < H + KVh ? dkh : dvh;
  const int head = hh < H ? hh : (hh - H - (rot ? 0 : KVh)) * group, nsum = hh < H ? 1 : group;
  int e = seq_of_token(cu, nseq, t0);
  f32x4 s1 = {}, s2 = {};
  for (int t = t0; t < t1; ++t) {
    while (t >= cu[e + 1]) ++e;  // sequences are not empty
    const float* p = src + ((int64_t)t * H + head) * hd + i0;
    f32x4 y1 = *(const f32x4*)p, y2 = *(const f32x4*)(p + half);
    for (int g = 1; g < nsum; ++g) {
      y1 += *(const f32x4*)(p + g * hd);
      y2 += *(const f32x4*)(p + g * hd + half);
    }
    if (rot) {
      const int64_t at = (int64_t)(t - cu[e]) * half + i0;
      const f32x4 c = *(const f32x4*)(cos_t + at), sn = *(const f32x4*)(sin_t + at);
      const f32x4 x1 = y1 * c + y2 * sn;
      y2 = y2 * c - y1 * sn;
      y1 = x1;
    }
    *(bf16x8*)(dqkv + xp_off(t, (int64_t)item * 8, nq)) =
        bf16x8{(bf16)y1[0], (bf16)y1[1], (bf16)y1[2], (bf16)y1[3], (bf16)y2[0], (bf16)y2[1], (bf16)y2[2], (bf16)y2[3]};
    s1 += y1;
    s2 += y2;
  }
  if (bpart) {
    float* b = bpart + (int64_t)blockIdx.y * nq + hh * hd + i0;
    *(f32x4*)b = s1;
    *(f32x4*)(b + half) = s2;
  }
}

// dst[0 .. 4 n4) = 0.  A kernel, since a caller may capture the step and
// memory-set nodes have given wrong results on a graph's later replays.  HBM
// bound: 152064 x 3584 floats 309 us (7.05 TB/s), the memory-set 327.
__global__ void __launch_bounds__(256) zero_f32_kernel(float* __restrict__ dst, int64_t n4) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n4) *(f32x4*)(dst + i * 4) = f32x4{};
}

// dE[tok[t]] += dx[t] (tokens repeat, hence atomic additions)
__global__ void __launch_bounds__(256) embed_bwd_kernel(const int32_t* __restrict__ tok, const float* __restrict__ dx,
                                                        int D, int V, float* __restrict__ dE) {
  const int t = blockIdx.x;
  const int id = min(max(tok[t], 0), V - 1);
  for (int d = threadIdx.x; d < D; d += 256) atomicAdd(dE + (int64_t)id * D + d, dx[(int64_t)t * D + d]);
}

// ---------------------------------------------------------------- launchers

void launch_ce_loss(const float* logits, int ldl, int V, const float2* lse_part, const int32_t* targets, int T,
                    float* rowloss, float* valid, float* lse, float* loss, float* scal, bf16* dlog, hipStream_t s) {
  ce_rows_kernel<<<T, 256, 0, s>>>(logits, ldl, V, lse_part, (V + LSE_COLS - 1) / LSE_COLS, targets, rowloss, valid,
                                   lse);
  ce_reduce_kernel<<<1, 256, 0, s>>>(rowloss, valid, T, loss, scal);
  ce_grad_kernel<<<dim3((ldl / 32 + 31) / 32, (T + 1) / 2), 256, 0, s>>>(logits, ldl, V, T, targets, valid, lse, scal,
                                                                       dlog);
}

void launch_untile_transpose(const bf16* W, int64_t N, int K, bf16* dst, int64_t Np, hipStream_t s) {
  const int64_t n = N * (K / 8);
  if (n > 0) untile_transpose_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(W, N, K, dst, Np);
}

// rows per workgroup of the row kernels that leave one partial per workgroup:
// at most ROW_PARTS partials
static int row_chunk(int T) { return (T + ROW_PARTS - 1) / ROW_PARTS; }

static void colsum_final(const float* part, int n, int C, float* d0, int c1, float* d1, int c2, float* d2,
                         hipStream_t s) {
  colsum_final_kernel<<<(C + 63) / 64, 1024, 0, s>>>(part, n, C, d0, c1, d1, c2, d2);
}

void launch_norm_bwd(const float* x, const bf16* g, const float* dy, int np, int64_t stride, int T, int D, float eps,
                     float* dx, int accumulate, bf16* dxb, float* dg, float* part, float* dgrow, hipStream_t s) {
  if (T <= 0) return;
  const int rows = row_chunk(T), n = (T + rows - 1) / rows;
  if (D > NORM_BWD_COLS) {
    norm_bwd_wide_kernel<<<T, 256, 0, s>>>(x, g, dy, np, stride, D, eps, dx, accumulate, dxb, dgrow);
    colsum_part_kernel<<<dim3((D + 255) / 256, n), 256, 0, s>>>(dgrow, T, D, rows, part);
  } else {
    auto go = [&](auto kern) {
      kern<<<n, 256, 0, s>>>(x, g, dy, np, stride, T, D, eps, dx, accumulate, dxb, part, rows);
    };
    if (D <= 1024) go(norm_bwd_kernel<1>);
    else if (D <= 2048) go(norm_bwd_kernel<2>);
    else if (D <= 4096) go(norm_bwd_kernel<4>);
    else go(norm_bwd_kernel<8>);
  }
  colsum_final(part, n, D, dg, D, nullptr, D, nullptr, s);
}

void launch_attn_bwd(const bf16* q, KVView kv, const bf16* o, const float* dof, int np, int64_t stride, bf16* dob,
                     const float* lse, float* dsum, const int32_t* cu, const int32_t* h_cu, int nseq, int T, int H,
                     float* dq, float* dkh, float* dvh, hipStream_t s) {
  if (T <= 0) return;
  int blocks = 0;
  for (int e = 0; e < nseq; ++e) blocks += (h_cu[e + 1] - h_cu[e] + BWD_ROWS - 1) / BWD_ROWS;
  const dim3 grid(blocks, H);
  const unsigned nd = (unsigned)(((int64_t)T * H * kv.hd / 8 + 255) / 256);
  if (kv.hd == 64) {
    attn_bwd_do_kernel<64><<<nd, 256, 0, s>>>(dof, np, stride, o, T, H, dob, dsum);
    attn_bwd_dq_kernel<64, 4><<<grid, 256, 0, s>>>(q, dob, kv, lse, dsum, cu, nseq, H, dq);
    attn_bwd_dkv_kernel<64, 4><<<grid, 256, 0, s>>>(q, dob, kv, lse, dsum, cu, nseq, H, dkh, dvh);
  } else {
    attn_bwd_do_kernel<128><<<nd, 256, 0, s>>>(dof, np, stride, o, T, H, dob, dsum);
    attn_bwd_dq_kernel<128, 3><<<grid, 256, 0, s>>>(q, dob, kv, lse, dsum, cu, nseq, H, dq);
    attn_bwd_dkv_kernel<128, 3><<<grid, 256, 0, s>>>(q, dob, kv, lse, dsum, cu, nseq, H, dkh, dvh);
  }
}

void launch_rope_bwd(const float* dq, const float* dkh, const float* dvh, const float* cos_t, const float* sin_t,
                     const int32_t* cu, int nseq, int T, int H, int KVh, int hd, bf16* dqkv, float* bpart, float* dbq,
                     float* dbk, float* dbv, hipStream_t s) {
  if (T <= 0) return;
  const int nq = (H + 2 * KVh) * hd, rows = row_chunk(T), n = (T + rows - 1) / rows;
  rope_bwd_kernel<<<dim3((nq / 8 + 127) / 128, n), 128, 0, s>>>(dq, dkh, dvh, cos_t, sin_t, cu, nseq, T, H, KVh, hd,
                                                               dqkv, dbq ? bpart : nullptr, rows);
  if (dbq) colsum_final(bpart, n, nq, dbq, H * hd, dbk, (H + KVh) * hd, dbv, s);
}

void launch_embed_bwd(const int32_t* tok, const float* dx, int T, int D, int V, float* dE, bool clear, hipStream_t s) {
  const int64_t n4 = (int64_t)V * D / 4;
  if (clear) zero_f32_kernel<<<(unsigned)((n4 + 255) / 256), 256, 0, s>>>(dE, n4);
  if (T > 0) embed_bwd_kernel<<<T, 256, 0, s>>>(tok, dx, D, V, dE);
}

}  // namespace axon
