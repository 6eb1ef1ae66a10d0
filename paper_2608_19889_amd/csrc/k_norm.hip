// Row kernels: embedding gather + RMSNorm, residual reduction + RMSNorm,
// greedy argmax, slot-length bookkeeping.  All are HBM/latency bound; rows are
// read with 16-byte vector accesses, one workgroup per row.
#include "common.h"
#include "kernels.h"

namespace axon {

// 4 consecutive elements of a T row as floats
AXON_DEV f32x4 load4(const float* p) { return *(const f32x4*)p; }
AXON_DEV f32x4 load4(const bf16* p) {
  bf16x4 v = *(const bf16x4*)p;
  return f32x4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
}
AXON_DEV void store4(float* p, f32x4 v) { *(f32x4*)p = v; }
AXON_DEV void store4(bf16* p, f32x4 v) {
  *(bf16x4*)p = bf16x4{(bf16)v[0], (bf16)v[1], (bf16)v[2], (bf16)v[3]};
}

// element i of embedding row id: bf16 tables are fragment-tiled (they double
// as the tied output head), float tables are row-major
AXON_DEV const float* emb_at(const float* e, int id, int i, int D) { return e + (int64_t)id * D + i; }
AXON_DEV const bf16* emb_at(const bf16* e, int id, int i, int D) { return e + wt_chunk(id, i >> 3, D) + (i & 7); }

// x[r,:] = E[tok[r],:] (as float); h[r,:] = x * rsqrt(mean(x^2) + eps) * g
template <typename T>
__global__ void __launch_bounds__(256) embed_rmsnorm_kernel(const int32_t* __restrict__ tok,
                                                            const T* __restrict__ emb,
                                                            const T* __restrict__ g,
                                                            float* __restrict__ x, T* __restrict__ h,
                                                            int D, int V, float eps, int h_pair) {
  __shared__ float red[16];
  const int r = blockIdx.x;
  const int id = min(max(tok[r], 0), V - 1);  // ids outside [0, V) are clamped, never dereferenced
  float* xr = x + (int64_t)r * D;
  float ss = 0.f;
  for (int i = threadIdx.x * 4; i < D; i += blockDim.x * 4) {
    f32x4 v = load4(emb_at(emb, id, i, D));
    store4(xr + i, v);
    ss += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
  }
  ss = block_sum(ss, red);
  const float inv = rsqrtf(ss / (float)D + eps);
  for (int i = threadIdx.x * 4; i < D; i += blockDim.x * 4) {
    f32x4 v = load4(emb_at(emb, id, i, D)), gv = load4(g + i);
    store4(h + (h_pair ? xp_off(r, i, D) : (int64_t)r * D + i),
           f32x4{v[0] * inv * gv[0], v[1] * inv * gv[1], v[2] * inv * gv[2], v[3] * inv * gv[3]});
  }
}

// Optionally x[r,:] += sum_s parts[s][r,:] (split-K partial products of the
// projection that feeds the residual), then h[i,:] = rmsnorm(x[r,:]) * g with
// r = i, or r = cu[i+1]-1 (last position of sequence i) when ``cu_last`` is set;
// h rows in the row-pair layout when h_pair is set (both kernels).
template <typename T>
__global__ void __launch_bounds__(256) resid_rmsnorm_kernel(const float* x, float* x_out,
                                                            const float* __restrict__ parts,
                                                            int nparts, int64_t part_stride,
                                                            const T* __restrict__ g, T* __restrict__ h,
                                                            int D, float eps,
                                                            const int32_t* __restrict__ cu_last, int h_pair) {
  __shared__ float red[16];
  const int i_out = blockIdx.x;
  const int r = cu_last ? cu_last[i_out + 1] - 1 : i_out;
  const float* xr = x + (int64_t)r * D;
  float* xo = x_out + (int64_t)r * D;
  float ss = 0.f;
  for (int i = threadIdx.x * 4; i < D; i += blockDim.x * 4) {
    f32x4 v = load4(xr + i);
    if (nparts > 0) {
      // in order, 4 parts' loads in flight per round
      for (int s0 = 0; s0 < nparts; s0 += 4) {
        f32x4 p[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) p[q] = load4(parts + min(s0 + q, nparts - 1) * part_stride + (int64_t)r * D + i);
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (s0 + q < nparts) v += p[q];
      }
      store4(xo + i, v);
    }
    ss += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
  }
  ss = block_sum(ss, red);
  const float inv = rsqrtf(ss / (float)D + eps);
  for (int i = threadIdx.x * 4; i < D; i += blockDim.x * 4) {
    f32x4 v = load4(xo + i), gv = load4(g + i);
    store4(h + (h_pair ? xp_off(i_out, i, D) : (int64_t)i_out * D + i),
           f32x4{v[0] * inv * gv[0], v[1] * inv * gv[1], v[2] * inv * gv[2], v[3] * inv * gv[3]});
  }
}

// Partial argmax of a logits row: workgroup (chunk, i) writes the largest of
// row r's columns ARGMAX_COLS chunk .. and its lowest index (a row of -inf or
// NaN: -inf and no index); launch_argmax_final merges the chunks.  r = i, or
// cu_last[i+1]-1 when ``cu_last`` is set (last position of sequence i in a
// packed all-positions logits matrix).  HBM bound: one workgroup per row, 160
// rows of 128256 columns, kept too few loads in flight (63 us; chunks of 4096
// columns with 16 independent loads per thread and the merge 18 us).
constexpr int ARGMAX_COLS = 4096;
__global__ void __launch_bounds__(256) argmax_part_kernel(const float* __restrict__ logits, int V,
                                                          float* __restrict__ val, int32_t* __restrict__ idx,
                                                          const int32_t* __restrict__ cu_last) {
  __shared__ float sv[4];
  __shared__ int si[4];
  const int i_out = blockIdx.y;
  const int r = cu_last ? cu_last[i_out + 1] - 1 : i_out;
  const float* row = logits + (int64_t)r * V;
  const int c0 = blockIdx.x * ARGMAX_COLS + threadIdx.x;
  float v[ARGMAX_COLS / 256];
#pragma unroll
  for (int j = 0; j < ARGMAX_COLS / 256; ++j) v[j] = row[min(c0 + j * 256, V - 1)];  // past the row: its last column
  float best = -INFINITY;
  int bi = 0x7fffffff;
#pragma unroll
  for (int j = 0; j < ARGMAX_COLS / 256; ++j)
    if (v[j] > best) { best = v[j]; bi = min(c0 + j * 256, V - 1); }  // ascending scan: first maximum per thread
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    const float ov = __shfl_xor(best, m, 64);
    const int oi = __shfl_xor(bi, m, 64);
    if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { sv[w] = best; si[w] = bi; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < 4; ++k)
      if (sv[k] > best || (sv[k] == best && si[k] < bi)) { best = sv[k]; bi = si[k]; }
    val[(int64_t)i_out * gridDim.x + blockIdx.x] = best;
    idx[(int64_t)i_out * gridDim.x + blockIdx.x] = bi;
  }
}

__global__ void set_lengths_kernel(const int32_t* __restrict__ cu, int32_t* __restrict__ len, int n) {
  int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < n) len[b] = cu[b + 1] - cu[b];
}

__global__ void set_step_lengths_kernel(const int32_t* __restrict__ cu, const int32_t* __restrict__ ent_slot,
                                        const int32_t* __restrict__ ent_base, int32_t* __restrict__ len, int n) {
  int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n) len[ent_slot[e]] = ent_base[e] + cu[e + 1] - cu[e];
}

// ---------------------------------------------------------------- launchers

template <typename T>
void launch_embed_rmsnorm(const int32_t* tok, const T* emb, const T* g, float* x, T* h, int rows, int D, int V,
                          float eps, hipStream_t s, bool h_pair) {
  if (rows <= 0) return;
  embed_rmsnorm_kernel<T><<<rows, 256, 0, s>>>(tok, emb, g, x, h, D, V, eps, h_pair ? 1 : 0);
}

template <typename T>
void launch_resid_rmsnorm(float* x, const float* parts, int nparts, int64_t part_stride, const T* g, T* h,
                          int rows, int D, float eps, const int32_t* cu_last, hipStream_t s, bool h_pair,
                          float* x_out) {
  if (rows <= 0) return;
  resid_rmsnorm_kernel<T><<<rows, 256, 0, s>>>(x, nparts > 0 && x_out ? x_out : x, parts, nparts, part_stride, g, h, D,
                                               eps, cu_last, h_pair ? 1 : 0);
}

void launch_argmax(const float* logits, int rows, int V, float* am_val, int32_t* am_idx, int32_t* next, int32_t* len,
                   const int32_t* cu_last, hipStream_t s) {
  if (rows <= 0) return;
  const int chunks = (V + ARGMAX_COLS - 1) / ARGMAX_COLS;
  argmax_part_kernel<<<dim3(chunks, rows), 256, 0, s>>>(logits, V, am_val, am_idx, cu_last);
  launch_argmax_final(am_val, am_idx, chunks, rows, next, len, s);
}

void launch_set_lengths(const int32_t* cu, int32_t* len, int n, hipStream_t s) {
  if (n <= 0) return;
  set_lengths_kernel<<<(n + 255) / 256, 256, 0, s>>>(cu, len, n);
}

void launch_set_step_lengths(const int32_t* cu, const int32_t* ent_slot, const int32_t* ent_base, int32_t* len,
                             int n, hipStream_t s) {
  if (n <= 0) return;
  set_step_lengths_kernel<<<(n + 255) / 256, 256, 0, s>>>(cu, ent_slot, ent_base, len, n);
}

template void launch_embed_rmsnorm<float>(const int32_t*, const float*, const float*, float*, float*, int, int,
                                          int, float, hipStream_t, bool);
template void launch_embed_rmsnorm<bf16>(const int32_t*, const bf16*, const bf16*, float*, bf16*, int, int, int,
                                         float, hipStream_t, bool);
template void launch_resid_rmsnorm<float>(float*, const float*, int, int64_t, const float*, float*, int, int,
                                          float, const int32_t*, hipStream_t, bool, float*);
template void launch_resid_rmsnorm<bf16>(float*, const float*, int, int64_t, const bf16*, bf16*, int, int,
                                         float, const int32_t*, hipStream_t, bool, float*);

}  // namespace axon
