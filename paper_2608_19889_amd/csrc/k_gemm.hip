// Projection GEMMs: out[t][n] = sum_k X[t][k] * W[n][k] (the F.linear
// convention: W is [out, in], X is tokens x in).  bf16 W is fragment-tiled
// (wt_chunk), float W and both X row-major.
//
// Both operands are K-contiguous, so the kernels compute C^T = W X^T with W as
// the MFMA A operand (rows = output features) and X as the B operand (columns
// = tokens): every lane's operand fragment is 8 consecutive k values, one
// 16-byte load, from either operand.
#include <vector>

#include "common.h"
#include "kernels.h"

namespace axon {

// Kernels that take more dynamic LDS than the runtime grants by itself (64 KB)
// need their limit raised on every device that runs them.  Each instance a
// launcher refers to enters itself here when the library is loaded, and
// gemm_init_device raises all limits on the current device, so that no launch --
// under capture, in a step that must not allocate, from several threads, on a
// second device -- depends on an earlier one.
struct LdsKernel {
  const void* kern;
  int bytes;
};
static std::vector<LdsKernel>& lds_kernels() {
  static std::vector<LdsKernel> v;
  return v;
}
template <auto KERN, int BYTES>
struct LdsLimit {
  static const bool entered;
};
template <auto KERN, int BYTES>
const bool LdsLimit<KERN, BYTES>::entered = (lds_kernels().push_back({(const void*)KERN, BYTES}), true);

hipError_t gemm_init_device() {
  for (const LdsKernel& k : lds_kernels()) {
    const hipError_t e = hipFuncSetAttribute(k.kern, hipFuncAttributeMaxDynamicSharedMemorySize, k.bytes);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

AXON_DEV float silu_f(float z) { return z / (1.f + __expf(-z)); }

// Store (for the residual stream, added to r) four consecutive output columns
// of which ``left`` are inside the matrix.
template <bool ADD>
AXON_DEV void store_cols(float* p, const float* r, f32x4 v, int left) {
  if (left >= 4) {
    if constexpr (ADD) v += *(const f32x4*)r;
    *(f32x4*)p = v;
  } else {
    for (int j = 0; j < left; ++j) p[j] = ADD ? r[j] + v[j] : v[j];
  }
}

// EPI_ROPE epilogue of one 32 x 32 accumulator block of the fused QKV
// projection: rows nb .. nb+31 (32-aligned, so inside one head), token t;
// v[i] = C[nb + (i/4)*8 + (lane/32)*4 + i%4][t].  Within a head the rows come
// in groups of 8: rotation-pair first halves i0 .. i0+3, then their partners
// i0+hd/2 .. i0+hd/2+3, so lane L < 32 holds first halves and lane L + 32 the
// partners for the same token, and one exchange across the half-wavefronts
// pairs them (both lanes of a pair share t, so they are active together).
// Bias first, then rotate-half RoPE at the token's position; q -> q_out, k ->
// its K page block, v (unrotated) -> its transposed V page block.
// The token's cache slot and position (rope_token) are looked up before the
// k-loop: the lookup is a chain of dependent loads (a binary search over the
// sequence offsets) whose latency the k-loop hides.
struct RopeTok {
  int slot, pos;
};
AXON_DEV RopeTok rope_token(const EpiArgs& ep, int t) {
  if (ep.len) return {ep.slot ? ep.slot[t] : t, ep.len[t]};
  const int e = seq_of_token(ep.cu, ep.nseq, t);
  return {ep.ent_slot ? ep.ent_slot[e] : e, (ep.ent_base ? ep.ent_base[e] : 0) + t - ep.cu[e]};
}
AXON_DEV void rope_block(const EpiArgs& ep, int nb, int t, RopeTok tok, const f32x16& v, int lane) {
  const int hd = ep.kv.hd, half = hd / 2, KVh = ep.kv.kv_heads;
  const int head = nb / hd;
  const bool first = lane < 32;
  const bool rotate = head < ep.H + KVh;  // q and k heads (v is stored unrotated)
  // every operand of the block is loaded before its first store: the stores
  // may alias the tables as far as the compiler knows, so loads issued
  // between them would cost one memory round trip per 8-row group
  bf16x4 bb[4];
  f32x4 cs[4], sn[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int i0 = ((nb % hd + g * 8) / 8) * 4;  // first rotation pair of the 8-row group
    const int e0 = first ? i0 : i0 + half;       // element index of this lane's first value
    bb[g] = ep.bias ? *(const bf16x4*)(ep.bias + head * hd + e0) : bf16x4{};
    cs[g] = f32x4{};
    sn[g] = f32x4{};
    if (rotate) {
      cs[g] = *(const f32x4*)(ep.cos_t + (int64_t)tok.pos * half + i0);
      sn[g] = *(const f32x4*)(ep.sin_t + (int64_t)tok.pos * half + i0);
    }
  }
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int i0 = ((nb % hd + g * 8) / 8) * 4;
    const int e0 = first ? i0 : i0 + half;
    float x[4], xp[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      x[j] = v[g * 4 + j] + (float)bb[g][j];
      xp[j] = lane_xor32(x[j]);
    }
    if (rotate) {
      bf16x4 y;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        y[j] = (bf16)(first ? x[j] * cs[g][j] - xp[j] * sn[g][j] : x[j] * cs[g][j] + xp[j] * sn[g][j]);
      if (head < ep.H) *(bf16x4*)(ep.q_out + ((int64_t)t * ep.H + head) * hd + e0) = y;
      else *(bf16x4*)((bf16*)ep.kv.k + k_el(ep.kv, tok.slot, head - ep.H, tok.pos, e0)) = y;  // 4 dims contiguous
    } else {
      bf16* vc = (bf16*)ep.kv.v;
#pragma unroll
      for (int j = 0; j < 4; ++j) vc[v_el(ep.kv, tok.slot, head - ep.H - KVh, tok.pos, e0 + j)] = (bf16)x[j];
    }
  }
}

// physical 16-byte chunk of logical chunk c in row r of an LDS panel with CH
// chunks per row.  The LDS serves 256 bytes (64 banks) per cycle, so the 16
// lanes of a ds_read_b128 phase (16 consecutive rows, one logical chunk) must
// land in 16 distinct 16-byte bank groups: with 128-byte rows two rows share
// a 256-byte bank line, so the XOR key is row / 2 (row / 4 for 64-byte rows).
template <int CH>
AXON_DEV int swz(int r, int c) {
  if constexpr (CH == 8) return c ^ ((r >> 1) & 7);
  else return c ^ ((r >> 2) & 3);
}

// Store one finished 32 x 32 accumulator block: rows nb .. nb+31 (nb < N),
// token t (t < M; output row t), v[i] = C[nb + (i/4)*8 + (lane/32)*4 + i%4][t].
// part: offset of this workgroup's split-K partial in ep.out_f32 (0: unsplit).
template <int EPI>
AXON_DEV void store_block(const EpiArgs& ep, int nb, int t, RopeTok tok, const f32x16& v, int lane, int N,
                          int64_t part) {
  if constexpr (EPI == EPI_ROPE) {
    rope_block(ep, nb, t, tok, v, lane);
  } else if constexpr (EPI == EPI_SILU || EPI == EPI_GU) {
    // rows nb..nb+15 are gate rows, nb+16..nb+31 the matching up rows
    // (features (nb / 32) * 16 .. +15: inside one 32-feature slice)
    const int64_t f0 = (nb / 32) * 16;
    const int lda = EPI == EPI_GU ? ep.ldo / 2 : ep.ldo;
    if constexpr (EPI == EPI_GU) {
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *(f32x4*)(ep.out_f32 + (int64_t)t * ep.ldo + nb + g * 8 + (lane >> 5) * 4) =
            f32x4{v[g * 4], v[g * 4 + 1], v[g * 4 + 2], v[g * 4 + 3]};
    }
    // (EPI_GU's is always the row-pair layout, but known at compile time the 4096 x
    // 16384 x 2048 GEMM took 319 us, against 311 with the choice left in)
    bf16* out = (bf16*)ep.out_t + (ep.opair ? xp_off(t, f0, lda) : (int64_t)t * lda + f0);
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const int f = g * 8 + (lane >> 5) * 4;
      bf16x4 o;
#pragma unroll
      for (int j = 0; j < 4; ++j) o[j] = (bf16)(silu_f(v[g * 4 + j]) * v[8 + g * 4 + j]);
      *(bf16x4*)(out + f) = o;
    }
  } else if constexpr (EPI == EPI_DGU) {
    // a = silu(g) u: dg = da u s (1 + g (1 - s)), du = da g s, s = sigmoid(g).
    // Feature nb + 16 j + i sits at columns 2 nb + 32 j + i (gate), + 16 (up);
    // both slices of 32 columns are loaded before the first store
    const int half = (lane >> 5) * 4;
    const float* gr = ep.gu + (int64_t)t * 2 * ep.ldo + 2 * nb + half;
    f32x4 gv[4], uv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      gv[q] = *(const f32x4*)(gr + (q >> 1) * 32 + (q & 1) * 8);
      uv[q] = *(const f32x4*)(gr + (q >> 1) * 32 + (q & 1) * 8 + 16);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t c0 = 2 * (int64_t)nb + (q >> 1) * 32;
      bf16* out = (bf16*)ep.out_t + xp_off(t, c0, 2 * ep.ldo) + (q & 1) * 8 + half;
      bf16x4 dg, du;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float gg = gv[q][j], d = v[q * 4 + j], sg = 1.f / (1.f + __expf(-gg));
        dg[j] = (bf16)(d * uv[q][j] * sg * (1.f + gg * (1.f - sg)));
        du[j] = (bf16)(d * gg * sg);
      }
      *(bf16x4*)out = dg;
      *(bf16x4*)(out + 16) = du;
    }
  } else if constexpr (EPI == EPI_GELU) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int n = nb + g * 8 + (lane >> 5) * 4;  // N % 32 == 0: all 4 rows exist
      const bf16x4 bb = *(const bf16x4*)(ep.bias + n);
      bf16x4 o;
#pragma unroll
      for (int j = 0; j < 4; ++j) o[j] = (bf16)gelu_tanh_f(v[g * 4 + j] + (float)bb[j]);
      *(bf16x4*)((bf16*)ep.out_t + (int64_t)t * ep.ldo + n) = o;
    }
  } else {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int n = nb + g * 8 + (lane >> 5) * 4;
      if (n >= N) continue;
      float* p = ep.out_f32 + part + (int64_t)t * ep.ldo + n;
      f32x4 o = {v[g * 4 + 0], v[g * 4 + 1], v[g * 4 + 2], v[g * 4 + 3]};
      if (ep.bias) {
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] += (float)ep.bias[min(n + j, N - 1)];
      }
      const float* r = EPI == EPI_RESID && ep.resid ? ep.resid + (int64_t)t * ep.ldo + n : p;
      store_cols<EPI == EPI_RESID>(p, r, o, N - n);
    }
  }
}

// EPI_LSE: the log-sum-exp partial of 64 columns nb .. nb+63 of token t (two
// accumulator blocks; the two lanes of a token hold 16 rows of each).  Costs
// the epilogue 64 exponentials per token; a pass over the logits for the same
// statistics read them twice (1.19 ms for 4096 x 128256 floats).
AXON_DEV void store_lse(const EpiArgs& ep, int nb, int t, const f32x16& v0, const f32x16& v1, int lane, int N) {
  const int half = (lane >> 5) * 4;
  float m = -INFINITY;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int n = nb + (i >> 2) * 8 + half + (i & 3);
    if (n < N) m = fmaxf(m, v0[i]);
    if (n + 32 < N) m = fmaxf(m, v1[i]);
  }
  m = fmaxf(m, lane_xor32(m));
  const float ref = m == -INFINITY ? 0.f : m;  // 64 columns of -inf: sum 0
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int n = nb + (i >> 2) * 8 + half + (i & 3);
    if (n < N) s += __expf(v0[i] - ref);
    if (n + 32 < N) s += __expf(v1[i] - ref);
  }
  s += lane_xor32(s);
  if (lane < 32) ep.lse_part[(int64_t)t * ((N + LSE_COLS - 1) / LSE_COLS) + nb / LSE_COLS] = float2{m, s};
}

// EPI_HEAD: the largest logit of a wavefront's AN blocks of token t (rows nb ..)
// and its lowest index, one partial per token; the logits themselves if wanted.
template <int AN>
AXON_DEV void store_head(const EpiArgs& ep, int nb, int t, const f32x16 (&v)[AN], int lane, int N) {
  const int half = (lane >> 5) * 4;
  float best = -INFINITY;
  int bi = 0x7fffffff;
#pragma unroll
  for (int a = 0; a < AN; ++a)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int n = nb + a * 32 + g * 8 + half;
      const f32x4 o = {v[a][g * 4], v[a][g * 4 + 1], v[a][g * 4 + 2], v[a][g * 4 + 3]};
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (n + j < N && o[j] > best) {
          best = o[j];
          bi = n + j;
        }
      if (ep.out_f32 && n < N) {
        float* p = ep.out_f32 + (int64_t)t * ep.ldo + n;
        // rows of an odd vocabulary are not 16-byte aligned
        if (ep.ldo % 4 == 0 && n + 4 <= N) *(f32x4*)p = o;
        else
          for (int j = 0; j < min(4, N - n); ++j) p[j] = o[j];
      }
    }
  const float ov = lane_xor32(best);
  const int oi = __float_as_int(lane_xor32(__int_as_float(bi)));
  if (ov > best || (ov == best && oi < bi)) {
    best = ov;
    bi = oi;
  }
  if (lane < 32) {
    const int64_t at = (int64_t)t * ((N + 32 * AN - 1) / (32 * AN)) + nb / (32 * AN);
    ep.am_val[at] = best;
    ep.am_idx[at] = bi;
  }
}

// Workgroup -> tile: each XCD (workgroup id mod 8) receives a contiguous range
// of tiles, walked in groups of 8 token tiles so that neighbouring tiles
// share operand panels in that XCD's L2.
AXON_DEV void tile_order(int bid, int gx, int gy, int& pn, int& pm) {
  const int G = gx * gy;
  int logical = bid;
  const int full = G / 8 * 8;
  if (bid < full) logical = (bid % 8) * (full / 8) + bid / 8;
  constexpr int GROUP = 8;
  const int per_group = GROUP * gx;
  const int gid = logical / per_group;
  const int first_m = gid * GROUP;
  const int gsize = min(gy - first_m, GROUP);
  pm = first_m + (logical % per_group) % gsize;
  pn = (logical % per_group) / gsize;
}

// ============================================================================
// Prefill GEMM of few tiles (short prompts, decode batches above 64, narrow
// outputs): WN x WM wavefronts, each owning AN x AM blocks of
// v_mfma_f32_32x32x16_bf16, over a ring of S stages of KU k-units of 32.
// What bounds these shapes is how many operand bytes a CU keeps in flight, so
// operands go straight to LDS (global_load_lds_dwordx4) S stages ahead,
// with one barrier per stage.  A W panel is copied tile by tile (a 16 x 32
// fragment tile is 1 KB in memory and in LDS: its lanes' reads are contiguous
// per 16 lanes, no swizzle); token rows are 64 bytes per unit, swizzled by the
// lane's source chunk (swz<4>); the next k-tile's fragments are read from LDS
// under this one's MFMAs.  Each output is one ascending chain of MFMAs
// over k, as in the 256 x 256 kernel: the same bits from every tile shape.
// gridDim.y = ksplit > 1 (float32 partials): workgroup row y takes k-share y.
// ============================================================================
template <int WN, int WM, int AN, int AM, int KU, int S>
struct RingShape {
  static constexpr int NW = WN * WM, BN = 32 * WN * AN, BM = 32 * WM * AM;
  static constexpr int WL = KU * BN / 16, XL = KU * BM / 16;  // 1 KB loads of a stage
  static constexpr int LPT = (WL + XL) / NW;                  // per wavefront
  static constexpr int STAGE = (WL + XL) * 64;                // 16-byte chunks
  static constexpr int LDS_BYTES = S * STAGE * 16;
  static_assert(WL % NW == 0 && XL % NW == 0, "a load instruction is W or X for every wavefront");
};

template <int EPI, bool XP, int WN, int WM, int AN, int AM, int KU, int S>
__global__ void __launch_bounds__(64 * WN * WM) gemm_ring_kernel(const bf16* __restrict__ W,
                                                                 const bf16* __restrict__ X, int N, int M, int K,
                                                                 EpiArgs ep) {
  using R = RingShape<WN, WM, AN, AM, KU, S>;
  extern __shared__ bf16x8 lds2[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = wave / WM, wm = wave % WM;
  int pn, pm;
  tile_order(blockIdx.x, (N + R::BN - 1) / R::BN, (M + R::BM - 1) / R::BM, pn, pm);
  const int n0 = pn * R::BN, m0 = pm * R::BM;
  const int nu = K / 32 / (int)gridDim.y;  // k-units of this workgroup (KU divides it)
  const int nk = nu / KU, ub = (int)blockIdx.y * nu;

  // this wavefront's loads of a stage, j < LPT: load q = j * NW + wave, W tile
  // (unit q / (BN/16), row block q % (BN/16)), then X tiles of 16 token rows;
  // row blocks and rows past the edge read the last one (never stored)
  const bf16* src[R::LPT];
#pragma unroll
  for (int j = 0; j < R::LPT; ++j) {
    if (j < R::WL / R::NW) {
      const int q = j * R::NW + wave, u = q / (R::BN / 16), blk = q % (R::BN / 16);
      const int nb = min(n0 / 16 + blk, (N - 1) / 16);
      src[j] = W + ((int64_t)nb * (K / 32) + ub + u) * 512 + lane * 8;
    } else {
      const int q = (j - R::WL / R::NW) * R::NW + wave, u = q / (R::BM / 16), blk = q % (R::BM / 16);
      const int row = blk * 16 + (lane >> 2), c = swz<4>(row, lane & 3);
      const int64_t m = min(m0 + row, M - 1);
      const int64_t k = (int64_t)(ub + u) * 32 + c * 8;
      src[j] = X + (XP ? xp_off(m, k, K) : m * K + k);
    }
  }
  auto issue = [&](int kt) {
    bf16x8* base = lds2 + (kt % S) * R::STAGE;
#pragma unroll
    for (int j = 0; j < R::LPT; ++j) {
      const bool w = j < R::WL / R::NW;
      const bf16* p = src[j] + (int64_t)kt * (KU * (w ? 512 : XP ? 64 : 32));
      __builtin_amdgcn_global_load_lds((const void*)p,
                                       (__attribute__((address_space(3))) void*)(base + (j * R::NW + wave) * 64), 16, 0,
                                       0);
    }
  };

  f32x16 acc[AN][AM];
#pragma unroll
  for (int a = 0; a < AN; ++a)
#pragma unroll
    for (int b = 0; b < AM; ++b) acc[a][b] = f32x16{};
  RopeTok tok[AM] = {};
#pragma unroll
  for (int st = 0; st < S; ++st)
    if (st < nk) issue(st);
  if constexpr (EPI == EPI_ROPE) {  // behind the first stages' loads
#pragma unroll
    for (int b = 0; b < AM; ++b) tok[b] = rope_token(ep, min(m0 + (wm * AM + b) * 32 + (lane & 31), M - 1));
  }
  // the token's normalization factor (few-token form), behind the same loads
  constexpr bool NORM = !XP && (EPI == EPI_SILU || EPI == EPI_ROPE || EPI == EPI_HEAD);
  float inv[AM];
  if constexpr (NORM) {
#pragma unroll
    for (int b = 0; b < AM; ++b) {
      inv[b] = 1.f;
      if (ep.ss_in) {
        const int t = min(m0 + (wm * AM + b) * 32 + (lane & 31), M - 1);
        float ss = 0.f;
        for (int j0 = 0; j0 < ep.ss_n; j0 += 8) {  // in order, 8 loads in flight
          float r[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) r[q] = ep.ss_in[(int64_t)min(j0 + q, ep.ss_n - 1) * M + t];
#pragma unroll
          for (int q = 0; q < 8; ++q)
            if (j0 + q < ep.ss_n) ss += r[q];
        }
        inv[b] = rsqrtf(ss / (float)K + ep.eps);
      }
    }
  }

  struct Frags {
    bf16x8 a[KU * 2][AN], b[KU * 2][AM];
  };
  auto read_frags = [&](int kt, Frags& f) {
    const bf16x8* la = lds2 + (kt % S) * R::STAGE;
    const bf16x8* lb = la + R::WL * 64;
#pragma unroll
    for (int u = 0; u < KU; ++u)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const int ch = ks * 2 + (lane >> 5);
#pragma unroll
        for (int a = 0; a < AN; ++a) {
          const int blk = u * (R::BN / 16) + (wn * AN + a) * 2 + ((lane >> 4) & 1);
          f.a[u * 2 + ks][a] = la[blk * 64 + (lane & 15) + 16 * ch];
        }
#pragma unroll
        for (int b = 0; b < AM; ++b) {
          const int r = (wm * AM + b) * 32 + (lane & 31);
          f.b[u * 2 + ks][b] = lb[u * (R::BM * 4) + r * 4 + swz<4>(r, ch)];
        }
      }
  };
  // k-tile kt, its fragments in ``cur``: stage kt + 1 has landed (``after``
  // later stages of this wavefront's loads stay in flight) and, after the
  // barrier, every wavefront's share of it is visible and every wavefront
  // holds its fragments of stage kt, whose buffer takes the loads of k-tile
  // kt + S; the next fragments are read under this k-tile's MFMAs
  auto ktile = [&](int kt, const Frags& cur, Frags& nxt, bool more, bool do_issue, int after) {
    __builtin_amdgcn_sched_barrier(0);
    // lgkmcnt(0) as the builtin: the compiler then knows that ``cur`` has
    // arrived and does not wait for the next fragments in front of the MFMAs
    __builtin_amdgcn_s_waitcnt(0xC07F);
    if (more) {
      wait_loads<R::LPT, S - 2>(after);
      phase_barrier();
      read_frags(kt + 1, nxt);
      if (do_issue) issue(kt + S);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int q = 0; q < KU * 2; ++q)
#pragma unroll
      for (int a = 0; a < AN; ++a)
#pragma unroll
        for (int b = 0; b < AM; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur.a[q][a], cur.b[q][b], acc[a][b], 0, 0, 0);
  };
  Frags f0, f1;
  wait_loads<R::LPT, S - 1>(min(S - 1, nk - 1));
  phase_barrier();
  read_frags(0, f0);
  int kt = 0;
  for (; kt + 1 + S < nk; kt += 2) {  // steady state: constant arguments
    ktile(kt, f0, f1, true, true, S - 2);
    ktile(kt + 1, f1, f0, true, true, S - 2);
  }
  for (; kt < nk; kt += 2) {
    ktile(kt, f0, f1, kt + 1 < nk, kt + S < nk, min(S - 2, nk - 2 - kt));
    if (kt + 1 < nk) ktile(kt + 1, f1, f0, kt + 2 < nk, kt + 1 + S < nk, min(S - 2, nk - 3 - kt));
  }

#pragma unroll
  for (int b = 0; b < AM; ++b) {
    const int t = m0 + (wm * AM + b) * 32 + (lane & 31);
    if constexpr (NORM) {
      if (ep.ss_in)
#pragma unroll
        for (int a = 0; a < AN; ++a) acc[a][b] *= inv[b];
    }
    if constexpr (EPI == EPI_HEAD) {
      f32x16 v[AN];
#pragma unroll
      for (int a = 0; a < AN; ++a) v[a] = acc[a][b];
      const int nb = n0 + wn * AN * 32;
      if (t < M && nb < N) store_head<AN>(ep, nb, t, v, lane, N);
      continue;
    }
    if (t >= M) continue;
    if constexpr (EPI == EPI_LSE) {
#pragma unroll
      for (int a = 0; a + 1 < AN; a += 2) {
        const int nb = n0 + (wn * AN + a) * 32;
        if (nb < N) store_lse(ep, nb, t, acc[a][b], acc[a + 1][b], lane, N);
      }
    }
#pragma unroll
    for (int a = 0; a < AN; ++a) {
      const int nb = n0 + (wn * AN + a) * 32;
      if (nb < N) store_block<EPI>(ep, nb, t, tok[b], acc[a][b], lane, N, (int64_t)blockIdx.y * ep.part_stride);
    }
  }
}

// ============================================================================
// Large prefill GEMM: 256 (W rows) x 256 (tokens) tiles, k-tiles of 32, 8
// wavefronts run as two groups that take turns on the matrix cores
// ("ping-pong").  Group g = wave / 4 owns W rows g*128 .. g*128+127 of the
// tile; wave (g, c) owns tokens c*64 .. c*64+63: 4 x 2 blocks of
// v_mfma_f32_32x32x16_bf16.  Waves w and w + 4 share a SIMD, and the groups
// run one phase apart: while one group issues a k-tile's 16 MFMAs, the other
// reads its next fragments from LDS and issues its share of the global->LDS
// loads, then a barrier swaps the roles.  The matrix core of every SIMD thus
// always has one wavefront's uninterrupted MFMA run in flight, and LDS
// latency and load issue are hidden behind it.
// Operands go straight from global memory to LDS (global_load_lds_dwordx4:
// lane L of an instruction writes 16 bytes at LDS offset 16 L) into a ring of
// STAGES k-tiles (32 KB each), issued STAGES-1 tiles ahead; the bank swizzle
// of the 64-byte panel rows is produced by choosing which global chunk each
// lane loads.
// Workgroups are renumbered so that each XCD (workgroup id mod 8) receives a
// contiguous range of tiles, walked in groups of 8 token tiles so that
// neighbouring tiles share operand panels in that XCD's L2.
// ============================================================================
namespace pf2 {
constexpr int BN = 256, BM = 256, BK = 32, STAGES = 4;
constexpr int CH = BK / 8;            // 16-byte chunks per panel row
constexpr int PANEL = BN * CH;        // chunks per operand panel
constexpr int STAGE = 2 * PANEL;      // W panel + X panel
constexpr int LPT = PANEL / 512;      // load instructions per operand per wave per k-tile
constexpr int ROWSTEP = 512 / CH;     // panel rows between a lane's consecutive chunks
constexpr int LDS_BYTES = STAGES * STAGE * 16;
}

// Wait until at most ``after`` k-tiles' loads of this wavefront are in flight
// (2 * LPT load instructions per k-tile).
AXON_DEV void wait_tiles(int after) {
  using namespace pf2;
  static_assert(2 * 2 * LPT <= 63, "vmcnt range");
  if (after >= 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * 2 * LPT) : "memory");
  else if (after == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * LPT) : "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// GROUPED: the mixture-of-experts form (EpiArgs::g_*): workgroup L takes n-tile
// L % gx of m-tile L / gx in the experts' tile sequence; that m-tile belongs to
// expert e (g_toff[e] <= L / gx < g_toff[e+1]), covers its local rows
// m0 .. m0+255 of M = g_off[e+1] - g_off[e], reads X row g_xrow[g_off[e] +
// row] and writes output row g_off[e] + row.
// XP: X in the row-pair layout (xp_off), so a k-tile's two 64-byte pieces of a
// row pair are one 128-byte line.
template <int EPI, bool GROUPED = false, bool XP = false>
__global__ void __launch_bounds__(512, 1) gemm_bf16_256_kernel(const bf16* __restrict__ W,
                                                               const bf16* __restrict__ X, int N, int M, int K,
                                                               EpiArgs ep) {
  using namespace pf2;
  static_assert(STAGES >= 3 && STAGES - 2 <= 2, "wait_tiles covers up to 2 later tiles");
  static_assert(CH == 4, "the W chunk address below assumes one 32-wide tile per k-tile");
  extern __shared__ bf16x8 lds2[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: scalar branches only
  const int grp = wave >> 2, wc = wave & 3;
  const int gx = (N + BN - 1) / BN;
  int pn, pm, n0, m0, rowbase = 0;
  if constexpr (GROUPED) {
    const int mt = blockIdx.x / gx;
    if (mt >= ep.g_toff[ep.g_E]) return;  // surplus workgroup: exits before any barrier
    int lo = 0, hi = ep.g_E - 1;          // the expert: largest e with g_toff[e] <= mt
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (ep.g_toff[mid] <= mt) lo = mid; else hi = mid - 1;
    }
    const int e = lo;
    pn = blockIdx.x % gx;
    pm = mt - ep.g_toff[e];
    rowbase = ep.g_off[e];
    M = ep.g_off[e + 1] - rowbase;  // this expert's rows (>= 1: it has an m-tile)
    W += (int64_t)e * ep.g_wstride;
  } else {
    tile_order(blockIdx.x, gx, (M + BM - 1) / BM, pn, pm);
  }
  n0 = pn * BN;
  m0 = pm * BM;

  // this lane's chunks of a stage: q = (i * 8 + wave) * 64 + lane, i < LPT,
  // row q / CH, logical chunk swz(row, q % CH) (swz is its own inverse)
  const int lrow0 = (wave * 64 + lane) / CH, lch = lane % CH;
  const int64_t rowblk = (int64_t)(K >> 5) * 512;  // elements per 16-row block of tiled W
  auto issue = [&](int stage, int k0) {
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      const int row = lrow0 + i * ROWSTEP;
      const int c = swz<CH>(row, lch);
      const int n = min(n0 + row, N - 1), m = min(m0 + row, M - 1);  // rows past the edge: any valid row
      // wt_chunk(n, k0 / 8 + c, K) with k0 a multiple of 32
      const bf16* ws = W + ((int64_t)(n >> 4) * rowblk + (int64_t)k0 * 16 + ((n & 15) + 16 * c) * 8);
      int64_t xr = m;
      if constexpr (GROUPED) xr = ep.g_xrow ? ep.g_xrow[rowbase + m] : rowbase + m;
      const bf16* xs = XP ? X + xp_off(xr, k0 + c * 8, K) : X + xr * K + k0 + c * 8;
      bf16x8* base = lds2 + stage * STAGE + (i * 8 + wave) * 64;
      __builtin_amdgcn_global_load_lds((const void*)ws, (__attribute__((address_space(3))) void*)base, 16, 0, 0);
      __builtin_amdgcn_global_load_lds((const void*)xs, (__attribute__((address_space(3))) void*)(base + PANEL),
                                       16, 0, 0);
    }
  };

  f32x16 acc[4][2];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = f32x16{};
  RopeTok tok[2] = {};

  // split K (gridDim.y > 1, float32 partials): this workgroup's share of
  // the k-tiles (gridDim.y divides K / BK)
  const int nk = K / BK / (int)gridDim.y;
  const int kbase = (int)blockIdx.y * nk * BK;
#pragma unroll
  for (int st = 0; st < STAGES - 1; ++st)
    if (st < nk) issue(st, kbase + st * BK);
  if constexpr (EPI == EPI_ROPE) {  // behind the first stages' loads
#pragma unroll
    for (int b = 0; b < 2; ++b) tok[b] = rope_token(ep, rowbase + min(m0 + wc * 64 + b * 32 + (lane & 31), M - 1));
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (grp == 1) phase_barrier();  // group 1 runs one phase behind group 0

  bf16x8 fa[2][4], fb[2][2];
  // one k-tile: do_issue -- issue the loads of k-tile kt + STAGES - 1;
  // after -- k-tiles of this wavefront's loads left in flight by its wait
  auto ktile = [&](int kt, bool do_issue, int after) {
    // ---- memory phase: fragments of k-tile kt, loads of k-tile kt+STAGES-1
    // into the buffer of k-tile kt-1, which both groups have read (group 1
    // in the phase that just ended)
    const bf16x8* la = lds2 + (kt % STAGES) * STAGE;
    const bf16x8* lb = la + PANEL;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int ch = ks * 2 + (lane >> 5);
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const int r = grp * 128 + a * 32 + (lane & 31);
        fa[ks][a] = la[r * CH + swz<CH>(r, ch)];
      }
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int r = wc * 64 + b * 32 + (lane & 31);
        fb[ks][b] = lb[r * CH + swz<CH>(r, ch)];
      }
    }
    const int kn = kt + STAGES - 1;
    if (do_issue) issue(kn % STAGES, kbase + kn * BK);
    // group 1's share of k-tile kt+1 must land before group 0 reads it in
    // the phase after the coming barrier; group 0 waits for its own share at
    // the end of its compute phase
    if (grp == 1) wait_tiles(after);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    phase_barrier();
    // ---- compute phase
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks][a], fb[ks][b], acc[a][b], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    if (grp == 0) wait_tiles(after);
    phase_barrier();
  };
  // steady state with constant arguments (no scalar branches around the
  // loads and waits: 1-3% on the 7B shapes), then the last STAGES - 1
  // k-tiles, which issue nothing and leave fewer k-tiles in flight
  static_assert(STAGES == 4, "the tail below peels STAGES - 1 k-tiles");
  int kt = 0;
  for (; kt + STAGES - 1 < nk; ++kt) ktile(kt, true, STAGES - 2);
#pragma unroll
  for (int j = 0; j < STAGES - 1; ++j)
    if (kt < nk) {
      ktile(kt, false, min(STAGES - 2, nk - 2 - kt));
      ++kt;
    }
  if (grp == 0) phase_barrier();  // same barrier count in both groups

  // SiLU epilogue staged through LDS (the ring is idle: every load has landed
  // and, after the barrier, every fragment has been read), so that global
  // memory sees 256-byte rows instead of 8-byte pieces (gate/up GEMM on the
  // 7B shape: 3% faster)
  if constexpr (EPI == EPI_SILU) {
    // 256 tokens x 128 gated features in bf16, rows 272 bytes apart (a
    // half-wavefront's 32 tokens hit distinct bank pairs), then 256-byte rows
    constexpr int LD = 136;
    bf16* st = (bf16*)lds2;
    __syncthreads();
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int tl = wc * 64 + b * 32 + (lane & 31);
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          bf16x4 v;
#pragma unroll
          for (int j = 0; j < 4; ++j) v[j] = (bf16)(silu_f(acc[a][b][g * 4 + j]) * acc[a][b][8 + g * 4 + j]);
          *(bf16x4*)(st + tl * LD + grp * 64 + a * 16 + g * 8 + (lane >> 5) * 4) = v;
        }
    }
    __syncthreads();
    const int nf = min(128, (N - n0) / 2);  // N % 32 == 0
    for (int idx = tid; idx < 256 * 16; idx += 512) {
      // row-major output: 16 chunks of a token row in consecutive lanes; the
      // row-pair layout: 8 lanes fill one 128-byte line (4 chunks of 32
      // features of each row of a pair), then the pair's next 32 features
      const int tl = ep.opair ? ((idx >> 5) << 1) | ((idx >> 2) & 1) : idx >> 4;
      const int ch = ep.opair ? (((idx >> 3) & 3) << 2) | (idx & 3) : idx & 15;
      if (m0 + tl < M && ch * 8 < nf) {
        const int64_t t = rowbase + m0 + tl, f = n0 / 2 + ch * 8;
        *(bf16x8*)((bf16*)ep.out_t + (ep.opair ? xp_off(t, f, ep.ldo) : t * ep.ldo + f)) =
            *(const bf16x8*)(st + tl * LD + ch * 8);
      }
    }
    return;
  }
  // epilogue: acc[a][b][i] = C[n][t],
  //   n = n0 + grp*128 + a*32 + (i/4)*8 + (lane/32)*4 + i%4,  t = m0 + wc*64 + b*32 + lane%32
  // (grouped: output row rowbase + t)
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int tl = m0 + wc * 64 + b * 32 + (lane & 31);
    if (tl >= M) continue;
    const int t = rowbase + tl;
    if constexpr (EPI == EPI_LSE) {
#pragma unroll
      for (int a = 0; a < 4; a += 2) {
        const int nb = n0 + grp * 128 + a * 32;
        if (nb < N) store_lse(ep, nb, t, acc[a][b], acc[a + 1][b], lane, N);
      }
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const int nb = n0 + grp * 128 + a * 32;
      if (nb < N) store_block<EPI>(ep, nb, t, tok[b], acc[a][b], lane, N, (int64_t)blockIdx.y * ep.part_stride);
    }
  }
}

// ============================================================================
// Weight-gradient GEMM: out[r][c] = sum_t Y[t][r] X[t][c] over T token rows
// (dW = dY^T X), both operands token-major as the backward pass leaves them.
// The schedule, tile and ring of the 256 x 256 kernel; a k-tile is 32 token
// rows of 256 columns of either operand (X the MFMA A operand, Y the B
// operand), and the transposition the fragments need is done by the LDS read
// itself: ds_read_tr16_b64, where 16 lanes read 4 token rows of 16 columns
// (lane i: row i / 4, columns 4 (i % 4) ..) and lane i receives column i's 4
// values.  A wavefront's read touches 8 token rows of 64 bytes; rows 512 bytes
// apart would share 16 banks, so a row's 64-byte segments are permuted by the
// row (segment ^ row % 4, by the chunk a lane loads).  Token rows past T read
// row T - 1; their Y values are zeroed in the last k-tile.
// The transposed copies it replaces (both operands through LDS tiles, X also
// fragment-tiled) took 2.4 ms of the 21.1 ms 1B-shaped 4-layer training step.
// Y and X lie in the row-pair layout (xp_off).
// ============================================================================
struct TnArgs {
  const bf16* Y;  // [T][ldy], output row r = column r
  const bf16* X;  // [T][ldx], output column c = column c
  int R, C, T, ldy, ldx;
  float* out;     // WGRAD_ROWS: [R][C]; split K: partials [split][R][C]
  // WGRAD_QKV / WGRAD_GU: the rows' own tensors (q, k, v / gate, up)
  float *out1, *out2;
  int hd, H, KVh;
};
// Row r of the gradient's destination.  WGRAD_QKV: heads q, k, v, a head's
// rows in groups of 8 = 4 first halves and their rotation partners; WGRAD_GU:
// 16 gate rows, then the 16 matching up rows.
template <int MODE>
AXON_DEV float* wgrad_row(const TnArgs& a, int r) {
  if constexpr (MODE == WGRAD_QKV) {
    const int hh = r / a.hd, rr = r % a.hd, g = rr / 8, j = rr % 8;
    const int64_t row = (int64_t)hh * a.hd + (j < 4 ? 4 * g + j : a.hd / 2 + 4 * g + j - 4);
    if (hh < a.H) return a.out + row * a.C;
    if (hh < a.H + a.KVh) return a.out1 + (row - (int64_t)a.H * a.hd) * a.C;
    return a.out2 + (row - (int64_t)(a.H + a.KVh) * a.hd) * a.C;
  } else if constexpr (MODE == WGRAD_GU) {
    const int64_t row = r / 32 * 16 + r % 16;
    return (r % 32 < 16 ? a.out : a.out1) + row * a.C;
  } else {
    return a.out + (int64_t)r * a.C;
  }
}

template <int MODE>
__global__ void __launch_bounds__(512, 1) gemm_tn_256_kernel(TnArgs g) {
  using namespace pf2;
  extern __shared__ bf16x8 lds2[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave >> 2, wc = wave & 3;
  int pn, pm;
  tile_order(blockIdx.x, (g.C + BN - 1) / BN, (g.R + BM - 1) / BM, pn, pm);
  const int n0 = pn * BN, m0 = pm * BM;

  // split K (gridDim.y): k-tiles kb .. kb + nk - 1 of ceil(T / 32)
  const int nkt = (g.T + BK - 1) / BK, per = (nkt + gridDim.y - 1) / gridDim.y;
  const int kb = min((int)blockIdx.y * per, nkt), nk = min(nkt - kb, per);

  // load i of a wavefront: token rows 4 wave + 2 i, + 1 of the k-tile, 32 chunks
  // of 8 columns each; columns past the operand read its last 8 (never stored)
  const int lrow = wave * 4 + (lane >> 5), pch = lane & 31;
  auto at = [&](int ld, int t, int c) -> int64_t { return xp_off(t, min(c, ld - 8), ld); };
  // a k-tile's 32 token rows are 32 ld elements: addresses are a fixed offset plus
  // that, except in a k-tile that passes T
  const int c0 = (pch ^ ((lrow & 3) << 2)) * 8, c1 = (pch ^ (((lrow + 2) & 3) << 2)) * 8;
  const bf16* xs[2] = {g.X + at(g.ldx, lrow, n0 + c0), g.X + at(g.ldx, lrow + 2, n0 + c1)};
  const bf16* ys[2] = {g.Y + at(g.ldy, lrow, m0 + c0), g.Y + at(g.ldy, lrow + 2, m0 + c1)};
  auto issue = [&](int stage, int kt) {
    const bool tail = (kt + 1) * BK > g.T;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const bf16* px = xs[i] + (int64_t)kt * BK * g.ldx;
      const bf16* py = ys[i] + (int64_t)kt * BK * g.ldy;
      if (tail) {
        const int t = min(kt * BK + lrow + i * 2, g.T - 1), c = i ? c1 : c0;
        px = g.X + at(g.ldx, t, n0 + c);
        py = g.Y + at(g.ldy, t, m0 + c);
      }
      bf16x8* base = lds2 + stage * STAGE + (wave * 2 + i) * 64;
      __builtin_amdgcn_global_load_lds((const void*)px, (__attribute__((address_space(3))) void*)base, 16, 0, 0);
      __builtin_amdgcn_global_load_lds((const void*)py, (__attribute__((address_space(3))) void*)(base + PANEL), 16, 0,
                                       0);
    }
  };

  f32x16 acc[4][2];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = f32x16{};
#pragma unroll
  for (int st = 0; st < STAGES - 1; ++st)
    if (st < nk) issue(st, kb + st);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (grp == 1) phase_barrier();  // group 1 runs one phase behind group 0

  // element offset of this lane's first read of column block cb (32 columns):
  // token row 8 (lane / 32) + (lane % 16) / 4, columns cb * 32 + 16 ((lane / 16)
  // % 2) + 4 (lane % 4) ..
  auto frag_at = [&](int cb) {
    const int row = (lane >> 5) * 8 + ((lane >> 2) & 3);
    const int ch = (cb * 4 + ((lane >> 4) & 1) * 2 + ((lane >> 1) & 1)) ^ (((lane >> 2) & 3) << 2);
    return row * 256 + ch * 8 + (lane & 1) * 4;
  };
  int offa[4], offb[2];
#pragma unroll
  for (int a = 0; a < 4; ++a) offa[a] = frag_at(grp * 4 + a);
#pragma unroll
  for (int b = 0; b < 2; ++b) offb[b] = frag_at(wc * 2 + b);
  // 8 token rows (ks * 16 + 8 (lane / 32) ..) of this lane's column
  auto read8 = [&](const bf16* p, int off, int ks) {
    return read_tr8(p + off + ks * 16 * 256, p + off + (ks * 16 + 4) * 256);
  };

  bf16x8 fa[2][4], fb[2][2];
  auto ktile = [&](int kt, bool do_issue, int after, bool last) {
    const bf16* la = (const bf16*)(lds2 + (kt % STAGES) * STAGE);
    const bf16* lb = la + PANEL * 8;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int a = 0; a < 4; ++a) fa[ks][a] = read8(la, offa[a], ks);
#pragma unroll
      for (int b = 0; b < 2; ++b) fb[ks][b] = read8(lb, offb[b], ks);
    }
    const int kn = kt + STAGES - 1;
    if (do_issue) issue(kn % STAGES, kb + kn);
    if (grp == 1) wait_tiles(after);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (last && (kb + kt + 1) * BK > g.T) {  // token rows past T contribute nothing
      const int t0 = (kb + kt) * BK + (lane >> 5) * 8;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int j = 0; j < 8; ++j)
            if (t0 + ks * 16 + j >= g.T) fb[ks][b][j] = (bf16)0.f;
    }
    phase_barrier();
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks][a], fb[ks][b], acc[a][b], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    if (grp == 0) wait_tiles(after);
    phase_barrier();
  };
  int kt = 0;
  for (; kt + STAGES - 1 < nk; ++kt) ktile(kt, true, STAGES - 2, false);
#pragma unroll
  for (int j = 0; j < STAGES - 1; ++j)
    if (kt < nk) {
      ktile(kt, false, min(STAGES - 2, nk - 2 - kt), kt == nk - 1);
      ++kt;
    }
  if (grp == 0) phase_barrier();  // same barrier count in both groups

#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int r = m0 + wc * 64 + b * 32 + (lane & 31);
    if (r >= g.R) continue;
    float* row = gridDim.y > 1 ? g.out + ((int64_t)blockIdx.y * g.R + r) * g.C : wgrad_row<MODE>(g, r);
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = n0 + grp * 128 + a * 32 + q * 8 + (lane >> 5) * 4;  // C % 32 == 0
        if (c < g.C)
          *(f32x4*)(row + c) = f32x4{acc[a][b][q * 4], acc[a][b][q * 4 + 1], acc[a][b][q * 4 + 2], acc[a][b][q * 4 + 3]};
      }
  }
}

// the split partials summed in order into the gradient's rows
template <int MODE>
__global__ void __launch_bounds__(256) wgrad_sum_kernel(TnArgs g, const float* __restrict__ parts, int nparts) {
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= (int64_t)g.R * g.C) return;
  const int r = (int)(i / g.C), c = (int)(i % g.C);
  f32x4 v = {};
  for (int s0 = 0; s0 < nparts; s0 += 4) {
    f32x4 p[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) p[q] = *(const f32x4*)(parts + min(s0 + q, nparts - 1) * ((int64_t)g.R * g.C) + i);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (s0 + q < nparts) v += p[q];
  }
  *(f32x4*)(wgrad_row<MODE>(g, r) + c) = v;
}

template <int MODE>
static void launch_tn(TnArgs g, float* part, int64_t part_floats, hipStream_t s) {
  auto kern = gemm_tn_256_kernel<MODE>;
  (void)LdsLimit<gemm_tn_256_kernel<MODE>, pf2::LDS_BYTES>::entered;
  const int tiles = ((g.R + 255) / 256) * ((g.C + 255) / 256), nkt = (g.T + 31) / 32;
  // few tiles: split the tokens towards 256 workgroups, at least 16 k-tiles each
  int ks = 1;
  while (ks < 8 && tiles * ks * 2 <= 256 && nkt / (ks * 2) >= 16 && (int64_t)ks * 2 * g.R * g.C <= part_floats) ks *= 2;
  if (ks == 1) {
    klaunch(kern, dim3(tiles, 1), dim3(512), pf2::LDS_BYTES, s, g);
    return;
  }
  TnArgs p = g;
  p.out = part;
  const int64_t n4 = (int64_t)g.R * g.C / 4;
  const dim3 grid(tiles, ks), sums((unsigned)((n4 + 255) / 256));
  // a timed launch starts its events with the GEMM and stops with the sum
  const TimingSlot t = g_timing_slot;
  g_timing_slot = TimingSlot{};
  if (t.start) {
    hipExtLaunchKernelGGL(kern, grid, dim3(512), pf2::LDS_BYTES, s, t.start, nullptr, 0, p);
    hipExtLaunchKernelGGL(wgrad_sum_kernel<MODE>, sums, dim3(256), 0, s, nullptr, t.stop, 0, g, part, ks);
  } else {
    kern<<<grid, 512, pf2::LDS_BYTES, s>>>(p);
    wgrad_sum_kernel<MODE><<<sums, 256, 0, s>>>(g, part, ks);
  }
}

void launch_wgrad(int mode, const bf16* Y, int ldy, int R, const bf16* X, int C, int T, float* out, float* out1,
                  float* out2, int hd, int H, int KVh, float* part, int64_t part_floats, hipStream_t s) {
  if (T <= 0 || R <= 0 || C <= 0) return;
  const TnArgs g{Y, X, R, C, T, ldy, C, out, out1, out2, hd, H, KVh};
  switch (mode) {
    case WGRAD_ROWS: launch_tn<WGRAD_ROWS>(g, part, part_floats, s); return;
    case WGRAD_QKV: launch_tn<WGRAD_QKV>(g, part, part_floats, s); return;
    case WGRAD_GU: launch_tn<WGRAD_GU>(g, part, part_floats, s); return;
  }
}

// the 256 x 256 kernel instance
template <int EPI, bool GROUPED, bool XP>
static auto kern_256() {
  (void)LdsLimit<gemm_bf16_256_kernel<EPI, GROUPED, XP>, pf2::LDS_BYTES>::entered;
  return gemm_bf16_256_kernel<EPI, GROUPED, XP>;
}

template <int EPI>
static void launch_grouped(const bf16* W, const bf16* X, int N, int K, int max_rows, const EpiArgs& ep,
                           hipStream_t s) {
  // sum over experts of ceil(rows_e / 256) <= ceil(max_rows / 256) + E
  const int64_t mtiles = (max_rows + pf2::BM - 1) / pf2::BM + ep.g_E;
  const int64_t tiles = mtiles * ((N + pf2::BN - 1) / pf2::BN);
  klaunch(kern_256<EPI, true, false>(), dim3((unsigned)tiles), dim3(512), pf2::LDS_BYTES, s, W, X, N, 0, K, ep);
}

// one ring kernel instance
template <int EPI, bool XP, int WN, int WM, int AN, int AM, int KU, int S>
static void launch_ring_shape(const bf16* W, const bf16* X, int N, int M, int K, int ksplit, const EpiArgs& ep,
                              hipStream_t s) {
  using R = RingShape<WN, WM, AN, AM, KU, S>;
  auto kern = gemm_ring_kernel<EPI, XP, WN, WM, AN, AM, KU, S>;
  (void)LdsLimit<gemm_ring_kernel<EPI, XP, WN, WM, AN, AM, KU, S>, R::LDS_BYTES>::entered;
  const int tiles = ((N + R::BN - 1) / R::BN) * ((M + R::BM - 1) / R::BM);
  klaunch(kern, dim3(tiles, ksplit), dim3(64 * R::NW), R::LDS_BYTES, s, W, X, N, M, K, ep);
}

// Tile shapes of the projection GEMM and what one 32-deep k-unit of a tile
// costs a CU (ns, from timing every shape on weights streamed from HBM, K
// 2048 to 18944, 24 to 2048 tokens).  A CU's time is the sum of its tiles'
// whether one or two workgroups share it, so the launch takes the shape of
// the smallest rounds x cost, rounds = tiles over 256 CUs rounded up: large
// tiles do more per operand byte, small ones leave fewer CUs idle.  Every
// shape gives the same bits.  us at 3584 x 3584 (N x K): 93 tokens 128x128
// tiles 33, 64x64 16, 32x64 14; 700 tokens 128x128 35, 64x64 40, 256x256 79;
// 1500 tokens 256x128 52, 128x128 60, 256x256 81.  The 128x128 kernel before
// this one, staged through registers one k-tile ahead, took 74-80 for all.  The
// costs are a plain float32 store's: they leave out what the RoPE epilogue and
// float32 logits add (1.6 to 2.5 times the cost on a short K).
enum Tile : int { T256x256, T256x128, T128x128, T128x64, T64x64, T32x64, T32x32, TILES };
struct TileCost {
  int bn, bm, ku, ns;
};
static constexpr TileCost TILE_COST[TILES] = {{256, 256, 1, 660}, {256, 128, 1, 420}, {128, 128, 1, 265},
                                              {128, 64, 1, 190},  {64, 64, 2, 120},   {32, 64, 2, 80},
                                              {32, 32, 2, 71}};
static Tile pick_tile(int N, int M, int K, int ksplit, int64_t* ns = nullptr, int first = T256x256,
                      int end = TILES) {
  const int units = K / 32 / ksplit;
  Tile best = (Tile)first;
  int64_t least = INT64_MAX;
  for (int i = first; i < end; ++i) {
    const TileCost& t = TILE_COST[i];
    if (units % t.ku) continue;  // a stage is ku whole k-units
    const int64_t tiles = (int64_t)((N + t.bn - 1) / t.bn) * ((M + t.bm - 1) / t.bm) * ksplit;
    const int64_t cost = (tiles + 255) / 256 * t.ns;
    if (cost < least) {
      least = cost;
      best = (Tile)i;
    }
  }
  if (ns) *ns = least * units;
  return best;
}

template <int EPI, bool XP>
static void launch_tiles(const bf16* W, const bf16* X, int N, int M, int K, int ksplit, const EpiArgs& ep,
                         hipStream_t s) {
  if constexpr (EPI == EPI_LSE) {
    // a wavefront owns pairs of 32-row blocks
    switch (pick_tile(N, M, K, ksplit, nullptr, T256x256, T64x64)) {
      case T256x128: launch_ring_shape<EPI, XP, 4, 2, 2, 2, 1, 4>(W, X, N, M, K, ksplit, ep, s); return;
      case T128x128: launch_ring_shape<EPI, XP, 2, 2, 2, 2, 1, 4>(W, X, N, M, K, ksplit, ep, s); return;
      case T128x64: launch_ring_shape<EPI, XP, 2, 2, 2, 1, 1, 6>(W, X, N, M, K, ksplit, ep, s); return;
      default: break;
    }
  } else
  switch (pick_tile(N, M, K, ksplit)) {
    case T256x128: launch_ring_shape<EPI, XP, 4, 2, 2, 2, 1, 4>(W, X, N, M, K, ksplit, ep, s); return;
    case T128x128: launch_ring_shape<EPI, XP, 2, 2, 2, 2, 1, 4>(W, X, N, M, K, ksplit, ep, s); return;
    case T128x64: launch_ring_shape<EPI, XP, 2, 2, 2, 1, 1, 6>(W, X, N, M, K, ksplit, ep, s); return;
    case T64x64: launch_ring_shape<EPI, XP, 2, 2, 1, 1, 2, 5>(W, X, N, M, K, ksplit, ep, s); return;
    case T32x64: launch_ring_shape<EPI, XP, 1, 2, 1, 1, 2, 5>(W, X, N, M, K, ksplit, ep, s); return;
    case T32x32: launch_ring_shape<EPI, XP, 1, 1, 1, 1, 2, 8>(W, X, N, M, K, ksplit, ep, s); return;
    default: break;
  }
  const int tiles = ((N + pf2::BN - 1) / pf2::BN) * ((M + pf2::BM - 1) / pf2::BM);
  klaunch(kern_256<EPI, false, XP>(), dim3(tiles, ksplit), dim3(512), pf2::LDS_BYTES, s, W, X, N, M, K, ep);
}

// The few-token form keeps to tiles of at most 64 tokens.  Against the
// row-splitting projection kernel with its tokens staged through registers and,
// on narrow outputs, a K split with an epilogue kernel (us, weights from HBM, 32
// tokens): QKV 6144 x 2048 16.9 -> 9.9, shared gate/up 5632 x 2048 14.8 -> 9.3,
// head 102400 x 2048 98 -> 84; 40 tokens: gate/up 37888 x 3584 66 -> 56.  The
// costs put 128x64 before 64x64 on that head (84.3 us, 64x64 80.4), and a 256x64
// tile, not built, timed 57.6 us on 37888 x 3584 at 64 tokens (64x64 62.3).
template <int EPI>
static void launch_few(const bf16* W, const bf16* X, int N, int M, int K, const EpiArgs& ep, hipStream_t s) {
  switch (pick_tile(N, M, K, 1, nullptr, T128x64)) {
    case T64x64: launch_ring_shape<EPI, false, 2, 2, 1, 1, 2, 5>(W, X, N, M, K, 1, ep, s); return;
    case T32x64: launch_ring_shape<EPI, false, 1, 2, 1, 1, 2, 5>(W, X, N, M, K, 1, ep, s); return;
    case T32x32: launch_ring_shape<EPI, false, 1, 1, 1, 1, 2, 8>(W, X, N, M, K, 1, ep, s); return;
    default: launch_ring_shape<EPI, false, 2, 2, 2, 1, 1, 6>(W, X, N, M, K, 1, ep, s); return;
  }
}

int few_head_rows(int N, int M, int K) { return pick_tile(N, M, K, 1, nullptr, T128x64) == T128x64 ? 64 : 32; }

void launch_gemm_few(const bf16* W, const bf16* X, int N, int M, int K, int epi, const EpiArgs& ep, hipStream_t s) {
  if (M <= 0) return;
  switch (epi) {
    case EPI_ROPE: launch_few<EPI_ROPE>(W, X, N, M, K, ep, s); return;
    case EPI_SILU: launch_few<EPI_SILU>(W, X, N, M, K, ep, s); return;
    case EPI_GELU: launch_few<EPI_GELU>(W, X, N, M, K, ep, s); return;
    case EPI_HEAD: launch_few<EPI_HEAD>(W, X, N, M, K, ep, s); return;
    default: return;
  }
}

void launch_gemm_bf16_split(const bf16* W, const bf16* X, int N, int M, int K, int ksplit, float* part,
                            int64_t part_stride, hipStream_t s, bool xpair) {
  if (M <= 0) return;
  EpiArgs ep{};
  ep.out_f32 = part;
  ep.ldo = N;
  ep.part_stride = part_stride;
  if (xpair) launch_tiles<EPI_F32, true>(W, X, N, M, K, ksplit, ep, s);
  else launch_tiles<EPI_F32, false>(W, X, N, M, K, ksplit, ep, s);
}

int gemm_ksplit(int N, int M, int K) {
  if (M < 256 || N < 256) return 1;
  const int tiles = ((N + 255) / 256) * ((M + 255) / 256);
  if (tiles >= 160) return 1;
  const int nk = K / 32;
  for (int ks : {2, 4})
    if (tiles * ks >= 200 && nk % ks == 0 && nk / ks >= 8) return ks;
  return nk % 2 == 0 && nk / 2 >= 8 ? 2 : 1;
}

int gemm_ksplit_cost(int N, int M, int K, int max_split) {
  const int units = K / 32;
  int best = 1;
  int64_t least = INT64_MAX;
  for (int ks = 1; ks <= max_split; ks *= 2) {
    if (units % ks || units / ks < 8) break;
    int64_t ns = 0;
    pick_tile(N, M, K, ks, &ns);
    // each further split writes and reads M x N floats more (~5000 bytes per
    // ns): worth it on a long K or a small output, not on a short K
    ns += (int64_t)(ks - 1) * M * N * 8 / 5000;
    if (ns < least) {
      least = ns;
      best = ks;
    }
  }
  return best;
}

void launch_gemm_bf16_grouped(const bf16* W, const bf16* X, int N, int K, int max_rows, int epi, const EpiArgs& ep,
                              hipStream_t s) {
  if (max_rows <= 0) return;
  if (epi == EPI_SILU) launch_grouped<EPI_SILU>(W, X, N, K, max_rows, ep, s);
  else launch_grouped<EPI_F32>(W, X, N, K, max_rows, ep, s);
}

void launch_gemm_bf16(const bf16* W, const bf16* X, int N, int M, int K, int epi, const EpiArgs& ep,
                      hipStream_t s) {
  if (M <= 0) return;
#define AXON_TILES(E)                                                  \
  case E:                                                              \
    if (ep.xpair) launch_tiles<E, true>(W, X, N, M, K, 1, ep, s);      \
    else launch_tiles<E, false>(W, X, N, M, K, 1, ep, s);              \
    return;
  switch (epi) {
    AXON_TILES(EPI_F32)
    AXON_TILES(EPI_RESID)
    AXON_TILES(EPI_SILU)
    AXON_TILES(EPI_ROPE)
    // the training step's: row-pair operands only
    case EPI_LSE: launch_tiles<EPI_LSE, true>(W, X, N, M, K, 1, ep, s); return;
    case EPI_GU: launch_tiles<EPI_GU, true>(W, X, N, M, K, 1, ep, s); return;
    case EPI_DGU: launch_tiles<EPI_DGU, true>(W, X, N, M, K, 1, ep, s); return;
    case EPI_GELU: launch_tiles<EPI_GELU, false>(W, X, N, M, K, 1, ep, s); return;  // GPT-2: row-major only
    default: return;
  }
#undef AXON_TILES
}

// ============================================================================
// float32 check-mode GEMM: 64 x 64 tiles, k-step 16, 256 threads with a 4 x 4
// register block each, operands staged k-major in LDS.  Dot products use
// compensated (Kahan) float32 summation, so their error does not grow with K.
// ============================================================================
template <int EPI>
__global__ void __launch_bounds__(256) gemm_f32_kernel(const float* __restrict__ W, const float* __restrict__ X,
                                                       int N, int M, int K, EpiArgs ep) {
  __shared__ float ws[16][68], xs[16][68];
  const int tid = threadIdx.x;
  const int n0 = blockIdx.x * 64, m0 = blockIdx.y * 64;
  const int lr = tid >> 2, lk = (tid & 3) * 4;
  const int tf = tid & 15, tt = tid >> 4;
  float acc[4][4] = {}, comp[4][4] = {};
  for (int k0 = 0; k0 < K; k0 += 16) {
    {
      const int n = n0 + lr, m = m0 + lr;
      f32x4 wv = {}, xv = {};
      if (n < N) {
        for (int j = 0; j < 4; ++j) wv[j] = (k0 + lk + j < K) ? W[(int64_t)n * K + k0 + lk + j] : 0.f;
      }
      if (m < M) {
        for (int j = 0; j < 4; ++j) xv[j] = (k0 + lk + j < K) ? X[(int64_t)m * K + k0 + lk + j] : 0.f;
      }
      for (int j = 0; j < 4; ++j) { ws[lk + j][lr] = wv[j]; xs[lk + j][lr] = xv[j]; }
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      float a[4], b[4];
      for (int i = 0; i < 4; ++i) { a[i] = ws[kk][tf * 4 + i]; b[i] = xs[kk][tt * 4 + i]; }
      for (int i = 0; i < 4; ++i)
        for (int j = 0; j < 4; ++j) {
          const float y = fmaf(a[i], b[j], -comp[i][j]);
          const float t = acc[i][j] + y;
          comp[i][j] = (t - acc[i][j]) - y;
          acc[i][j] = t;
        }
    }
    __syncthreads();
  }
  for (int j = 0; j < 4; ++j) {
    const int t = m0 + tt * 4 + j;
    if (t >= M) continue;
    for (int i = 0; i < 4; ++i) {
      const int n = n0 + tf * 4 + i;
      if (n >= N) continue;
      float* p = ep.out_f32 + (int64_t)t * ep.ldo + n;
      if constexpr (EPI == EPI_RESID) *p += acc[i][j];
      else *p = acc[i][j];
    }
  }
}

// ============================================================================
// float32 check mode, one token (M <= MT): a wavefront per weight row, lanes
// along K with 16-byte loads, compensated (Kahan) per-lane sums reduced across
// the wavefront by shuffles.  K % 4 == 0.
// ============================================================================
template <int EPI, int MT>
__global__ void __launch_bounds__(256) gemv_f32_kernel(const float* __restrict__ W, const float* __restrict__ X,
                                                       int N, int M, int K, EpiArgs ep) {
  const int lane = threadIdx.x & 63;
  const int n = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (n >= N) return;  // whole wavefronts only: no barrier follows
  float acc[MT], comp[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) acc[t] = comp[t] = 0.f;
  const float* wr = W + (int64_t)n * K;
  for (int k = lane * 4; k < K; k += 256) {
    const f32x4 w = *(const f32x4*)(wr + k);
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      if (t >= M) break;
      const f32x4 x = *(const f32x4*)(X + (int64_t)t * K + k);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float y = fmaf(w[j], x[j], -comp[t]);
        const float u = acc[t] + y;
        comp[t] = (u - acc[t]) - y;
        acc[t] = u;
      }
    }
  }
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    if (t >= M) break;
    const float v = wave_sum(acc[t]);
    if (lane == 0) {
      float* p = ep.out_f32 + (int64_t)t * ep.ldo + n;
      if constexpr (EPI == EPI_RESID) *p += v;
      else *p = v;
    }
  }
}

// ============================================================================
// float32 check mode, 2..32 tokens: the token rows are staged through LDS in
// k-chunks of 256 (double-buffered; the next chunk's loads are issued before
// the current chunk is used and stored after it), and each wavefront computes two weight rows for
// every token, lanes along K with compensated (Kahan) per-lane sums and a
// butterfly sum across the wavefront: the token operand is read from HBM once
// per workgroup instead of once per weight row.  Workgroup = 8 rows x MT
// tokens (token groups along gridDim.y, so that there are enough wavefronts
// for the compensated sums).  K % 4 == 0.
// ============================================================================
template <int EPI, int MT>
__global__ void __launch_bounds__(256) gemv_f32_lds_kernel(const float* __restrict__ W, const float* __restrict__ X,
                                                           int N, int M, int K, EpiArgs ep) {
  constexpr int KC = 256;
  __shared__ f32x4 xs[2][MT][KC / 4];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  // token group blockIdx.y: tokens MT y .. MT y + MT - 1
  X += (int64_t)blockIdx.y * MT * K;
  ep.out_f32 += (int64_t)blockIdx.y * MT * ep.ldo;
  M = min(MT, M - (int)blockIdx.y * MT);
  const int n0 = blockIdx.x * 8 + 2 * w, n1 = n0 + 1;
  const float* w0 = W + (int64_t)min(n0, N - 1) * K;
  const float* w1 = W + (int64_t)min(n1, N - 1) * K;
  float acc0[MT], cmp0[MT], acc1[MT], cmp1[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) acc0[t] = cmp0[t] = acc1[t] = cmp1[t] = 0.f;
  const int nch = (K + KC - 1) / KC;
  // chunk c of the token rows: loaded into registers (MT * KC / 1024 16-byte
  // pieces per thread), then written to xs[c & 1] (zeros past K and past M)
  constexpr int SP = MT * (KC / 4) / 256;
  f32x4 sv[SP];
  auto stage_load = [&](int c) {
#pragma unroll
    for (int r = 0; r < SP; ++r) {
      const int i = tid + r * 256, t = i / (KC / 4), k = c * KC + 4 * (i % (KC / 4));
      sv[r] = *(const f32x4*)(X + (int64_t)min(t, M - 1) * K + min(k, K - 4));
    }
  };
  auto stage_store = [&](int c) {
#pragma unroll
    for (int r = 0; r < SP; ++r) {
      const int i = tid + r * 256, t = i / (KC / 4), q = i % (KC / 4), k = c * KC + 4 * q;
      xs[c & 1][t][q] = t < M && k < K ? sv[r] : f32x4{};
    }
  };
  stage_load(0);
  stage_store(0);
  f32x4 wv0 = *(const f32x4*)(w0 + min(lane * 4, K - 4)), wv1 = *(const f32x4*)(w1 + min(lane * 4, K - 4));
  __syncthreads();
  for (int c = 0; c < nch; ++c) {
    if (c + 1 < nch) stage_load(c + 1);
    const int k = c * KC + lane * 4;
    const f32x4 a0 = wv0, a1 = wv1;
    if (c + 1 < nch) {
      const int kn = min(k + KC, K - 4);
      wv0 = *(const f32x4*)(w0 + kn);
      wv1 = *(const f32x4*)(w1 + kn);
    }
    if (k < K) {
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        const f32x4 x = xs[c & 1][t][lane];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float y = fmaf(a0[j], x[j], -cmp0[t]);
          float u = acc0[t] + y;
          cmp0[t] = (u - acc0[t]) - y;
          acc0[t] = u;
          y = fmaf(a1[j], x[j], -cmp1[t]);
          u = acc1[t] + y;
          cmp1[t] = (u - acc1[t]) - y;
          acc1[t] = u;
        }
      }
    }
    // the buffer of chunk c + 1 was last read in chunk c - 1, before the
    // barrier that ended it
    if (c + 1 < nch) stage_store(c + 1);
    __syncthreads();
  }
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    if (t >= M) break;
    const float v0 = wave_sum(acc0[t] - cmp0[t]), v1 = wave_sum(acc1[t] - cmp1[t]);
    if (lane == 0) {
      float* p = ep.out_f32 + (int64_t)t * ep.ldo;
      if (n0 < N) p[n0] = EPI == EPI_RESID ? p[n0] + v0 : v0;
      if (n1 < N) p[n1] = EPI == EPI_RESID ? p[n1] + v1 : v1;
    }
  }
}

void launch_gemm_f32(const float* W, const float* X, int N, int M, int K, int epi, const EpiArgs& ep,
                     hipStream_t s) {
  if (M <= 0) return;
  if (M <= 32 && K % 4 == 0) {
    const bool r = epi == EPI_RESID;
    if (M <= 1) {
      const dim3 g((N + 3) / 4);
      r ? klaunch(gemv_f32_kernel<EPI_RESID, 1>, g, dim3(256), 0, s, W, X, N, M, K, ep)
        : klaunch(gemv_f32_kernel<EPI_F32, 1>, g, dim3(256), 0, s, W, X, N, M, K, ep);
      return;
    }
    const dim3 g((N + 7) / 8, (M + 7) / 8);
    r ? klaunch(gemv_f32_lds_kernel<EPI_RESID, 8>, g, dim3(256), 0, s, W, X, N, M, K, ep)
      : klaunch(gemv_f32_lds_kernel<EPI_F32, 8>, g, dim3(256), 0, s, W, X, N, M, K, ep);
    return;
  }
  dim3 grid((N + 63) / 64, (M + 63) / 64);
  if (epi == EPI_RESID) klaunch(gemm_f32_kernel<EPI_RESID>, grid, dim3(256), 0, s, W, X, N, M, K, ep);
  else klaunch(gemm_f32_kernel<EPI_F32>, grid, dim3(256), 0, s, W, X, N, M, K, ep);
}

__global__ void __launch_bounds__(256) silu_f32_kernel(const float* __restrict__ gu, float* __restrict__ a, int M,
                                                       int I) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)M * I) return;
  const int t = (int)(idx / I), f = (int)(idx % I);
  const float* p = gu + (int64_t)t * 2 * I + (f / 16) * 32 + f % 16;  // gate; up 16 later
  a[idx] = silu_f(p[0]) * p[16];
}

void launch_silu_f32(const float* gu, float* a, int M, int I, hipStream_t s) {
  const int64_t n = (int64_t)M * I;
  if (n > 0) silu_f32_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(gu, a, M, I);
}

}  // namespace axon
