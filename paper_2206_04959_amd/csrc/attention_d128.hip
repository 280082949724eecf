// Causal attention at head dimension 128 in bf16, forward and backward: 64-row
// padded tiles, one LDS stage of two blocks, even and odd 64-row blocks on
// the two halves of a workgroup.  Same layout, grid rows and results contract as
// the kernels for d = 64 and 96.
//
// Kept for its rounding, not its speed: 2 x 2048 x 6 heads takes 39 us forward
// and 109 us backward against 29.6 and 80 with 32-row tiles loaded a step ahead,
// but on the 20B-shaped shard (2048 keys, peaked softmax) the largest error of a
// LayerNorm-1 input gradient against 64 bits is 1.94e-2 with these, and 2.10e-2
// with the 32-row kernels (2.08e-2 with only their backward): beyond the bar of
// 2e-2 for bf16.
#include <math.h>

#include <atomic>
#include <type_traits>

#include "attention.h"

namespace merak {

// A [64 rows][D] bf16 tile in LDS with rows padded to LD elements: 16-byte
// reads of 16 consecutive rows hit distinct banks, the transposing reads of 4
// consecutive rows at most two-way.  LD * 2 is a multiple of 16, so the tile is
// exactly kChunks wave-instructions of 16-byte-per-lane direct loads.
constexpr int D = 128, KS = D / 16, DT = D / 32;
constexpr int LD = D + 24;
constexpr int kChunks = LD / 8;            // 16-byte chunks per padded row
constexpr int kTileBytes = 64 * LD * 2;    // = kChunks * 1024

// One wave's plan for copying rows 0..63 of a tensor (row stride gs
// elements) into the padded tile with loads that write LDS directly: lane i of
// instruction q fills chunk 64 q + i (padding chunks re-read a data chunk).
// The per-lane element offsets are computed once.
struct TileLoad {
  uint32_t off[kChunks];
  __device__ __forceinline__ void init(size_t gs, int lane) {
#pragma unroll
    for (int q = 0; q < kChunks; ++q) {
      const int c = q * 64 + lane;
      const int row = c / kChunks, ch = c % kChunks;
      off[q] = (uint32_t)(row * gs) + (uint32_t)(ch < D / 8 ? ch : 0) * 8u;
    }
  }
  __device__ __forceinline__ void issue(char* lds, const bf16_t* src) const {
#pragma unroll
    for (int q = 0; q < kChunks; ++q)
      __builtin_amdgcn_global_load_lds(src + off[q], (MERAK_LDS void*)(lds + q * 1024), 16, 0, 0);
  }
};

// 64 floats (one per lane) into LDS with a direct load.
__device__ __forceinline__ void wave_vec_load(char* lds, const float* src, int lane) {
  __builtin_amdgcn_global_load_lds(src + lane, (MERAK_LDS void*)lds, 4, 0, 0);
}

// 8 consecutive elements of row `row` from column `col` of a padded tile.
__device__ __forceinline__ bf16x8_t frag_row(const char* tile, int row, int col) {
  return *reinterpret_cast<const bf16x8_t*>(tile + (row * LD + col) * 2);
}

// MFMA operand of X^T taken from a natural tile X[row][col]: lane l gets
// column col0 + l % 32 and rows kb + 4 (l / 32) + 0..3 (elements 0..3) and
// kb + 8 + 4 (l / 32) + 0..3 (elements 4..7), the key order of an accumulator
// reused as the 16-deep operand.  Two transposing LDS reads: in each 16-lane
// group, lane j fetches 4 columns of row (j / 4) and lane i receives column i of
// the 4 rows.
__device__ __forceinline__ bf16x8_t frag_tr(const char* tile, int kb, int col0, int lane) {
  const int row = kb + (lane >> 5) * 4 + ((lane & 15) >> 2);
  const int col = col0 + ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
  const char* p = tile + (row * LD + col) * 2;
  const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((MERAK_LDS s16x4_t*)p);
  const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((MERAK_LDS s16x4_t*)(p + 8 * LD * 2));
  const s16x8_t v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(bf16x8_t, v);
}

// One LDS stage of four tiles (two 64-row blocks of two tensors); the loads of the
// next block pair are issued after the current pair has been used.
constexpr size_t kLdsBytes = (size_t)4 * kTileBytes;

// ---------------------------------------------------------------------------
// bf16 forward.  A workgroup owns 64 query rows of one (batch, head); wave w
// takes the 32 rows of group w % 2 against the even (w < 2) or odd 64-key
// blocks, and the two halves are merged at the end (online-softmax merge).
// The stage holds the K and V tiles of two key blocks.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) attn_fwd_bf16_d128(int S, int H, int Bm, int mstride,
                                                          const bf16_t* __restrict__ qkv, bf16_t* __restrict__ o,
                                                          float* __restrict__ lse, float scale_log2) {
  extern __shared__ __align__(16) char smem[];  // [K blk a, K blk b, V blk a, V blk b]

  // Grid (heads, sequences, row blocks), row block slowest: the whole grid
  // runs longest rows first.
  const int b = seq_index(blockIdx.y, Bm, mstride), hh = blockIdx.x;
  const int qt = gridDim.z - 1 - blockIdx.z;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int qg = wave & 1, kh = wave >> 1;
  const int q0 = qt * 64 + qg * 32;
  const int q = q0 + l32;
  const size_t rs = (size_t)3 * H * D;
  const bf16_t* base = qkv + (size_t)b * S * rs;
  const bf16_t* Qp = base + hh * D;
  const bf16_t* Kp = base + (size_t)H * D + hh * D;
  const bf16_t* Vp = base + (size_t)2 * H * D + hh * D;

  bf16x8_t qf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) qf[ks] = frag_kc(Qp + (size_t)q * rs + ks * 16 + hf * 8);

  const int n_kb = qt + 1;  // key blocks 0..qt reach the tile's last row
  const int n_it = (n_kb + 1) / 2;
  TileLoad tl;
  tl.init(rs, lane);
  const bf16_t* lsrc = (wave >> 1) ? Vp : Kp;
  auto load_pair = [&](int it) {  // wave w: tile w of the stage
    const int blk = 2 * it + (wave & 1);
    if (blk < n_kb) tl.issue(smem + wave * kTileBytes, lsrc + (size_t)blk * 64 * rs);
  };

  f32x16_t oacc[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[t][r] = 0.0f;
  float m = -INFINITY, l = 0.0f;

  // S = K Q^T of key block kb (LDS tile Kt) for this wave's 32 queries.
  auto scores = [&](const char* Kt, f32x16_t (&s)[2]) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[t][r] = 0.0f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        s[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_row(Kt, t * 32 + l32, ks * 16 + hf * 8), qf[ks],
                                                       s[t], 0, 0, 0);
    }
  };
  // Causal mask, online softmax and O^T += V^T P^T with key block kb (tile Vt).
  auto softmax_pv = [&](const char* Vt, int k0, f32x16_t (&s)[2]) {
    // s[t][r]: key k0 + t*32 + (r/4)*8 + 4*hf + r%4, query q.  Only a block
    // that reaches past the wave's first query needs the causal mask.
    float mloc = -INFINITY;
    if (k0 + 63 > q0) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = k0 + t * 32 + (r >> 2) * 8 + hf * 4 + (r & 3);
          const float v = key > q ? -INFINITY : s[t][r] * scale_log2;
          s[t][r] = v;
          mloc = fmaxf(mloc, v);
        }
    } else {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          s[t][r] *= scale_log2;
          mloc = fmaxf(mloc, s[t][r]);
        }
    }
    mloc = fmaxf(mloc, __shfl_xor(mloc, 32, 64));
    const float mnew = fmaxf(m, mloc);
    if (__ballot(mnew > m)) {  // rescale only when some row's maximum grew
      const float alpha = __builtin_amdgcn_exp2f(m - mnew);
      l *= alpha;
#pragma unroll
      for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[t][r] *= alpha;
      m = mnew;
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = __builtin_amdgcn_exp2f(s[t][r] - m);
        s[t][r] = p;
        l += p;
      }
    bf16x8_t pb[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) pb[g] = cvt8(s[g >> 1], (g & 1) * 8);
    // O^T[d][q] += V^T[d][key] P^T[key][q]
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_tr(Vt, g * 16, dt * 32, lane), pb[g], oacc[dt],
                                                           0, 0, 0);
  };

  for (int it = 0; it < n_it; ++it) {
    __syncthreads();  // every wave is done with the previous block pair
    load_pair(it);
    __syncthreads();  // this block pair landed
    const int kb = 2 * it + kh, k0 = kb * 64;
    if (kb >= n_kb || k0 > q0 + 31) continue;
    f32x16_t s[2];
    scores(smem + kh * kTileBytes, s);
    softmax_pv(smem + (2 + kh) * kTileBytes, k0, s);
  }

  // Merge the two key halves of each query group (partial m, l, O^T).
  constexpr int XS = 2 + DT * 16;
  static_assert((size_t)128 * XS * 4 <= kLdsBytes, "merge buffer fits the tiles");
  float* xch = reinterpret_cast<float*>(smem) + (size_t)(qg * 64 + lane) * XS;
  __syncthreads();
  if (kh == 1) {
    xch[0] = m;
    xch[1] = l;
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) xch[2 + t * 16 + r] = oacc[t][r];
  }
  __syncthreads();
  if (kh == 1) return;
  const float m1 = xch[0], l1 = xch[1];
  const float mt = fmaxf(m, m1);
  const float a0 = __builtin_amdgcn_exp2f(m - mt), a1 = __builtin_amdgcn_exp2f(m1 - mt);
  float lt = l * a0 + l1 * a1;
  lt += __shfl_xor(lt, 32, 64);
  const float inv = 1.0f / lt;
  bf16_t* orow = o + ((size_t)b * S + q) * H * D + hh * D;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        v[e] = (oacc[dt][4 * g + e] * a0 + xch[2 + dt * 16 + 4 * g + e] * a1) * inv;
      store4(orow + dt * 32 + g * 8 + hf * 4, v);
    }
  if (hf == 0) lse[((size_t)b * H + hh) * S + q] = (mt + log2f(lt)) * kLn2;
}

// ---------------------------------------------------------------------------
// bf16 backward: dK, dV (KV-parallel).  A workgroup owns 64 keys of one
// (batch, head); wave w takes the 32 keys of group w % 2 against the even
// (w < 2) or odd 64-query blocks from the diagonal on, and the two partial sums
// are added at the end.  The stage holds the Q and dO tiles (and lse, delta)
// of two query blocks.  P is rebuilt from lse.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
    attn_bwd_dkdv_bf16_d128(int S, int H, int Bm, int mstride, const bf16_t* __restrict__ qkv,
                            const bf16_t* __restrict__ dout, const float* __restrict__ lse,
                            const float* __restrict__ delta, bf16_t* __restrict__ dqkv, float scale_log2, float scale) {
  extern __shared__ __align__(16) char smem[];  // [Q a, Q b, dO a, dO b], then lse/delta
  float* vecs = reinterpret_cast<float*>(smem + kLdsBytes);  // [lse a|b, delta a|b]

  // Grid (heads, sequences, key blocks), key block slowest: early keys see the
  // most queries, so the whole grid runs longest columns first.
  const int b = seq_index(blockIdx.y, Bm, mstride), hh = blockIdx.x;
  const int kt = blockIdx.z;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int kg = wave & 1, qh = wave >> 1;
  const int kw0 = kt * 64 + kg * 32;
  const int key = kw0 + l32;
  const size_t rs = (size_t)3 * H * D;
  const size_t ors = (size_t)H * D;
  const bf16_t* base = qkv + (size_t)b * S * rs;
  const bf16_t* Qp = base + hh * D;
  const bf16_t* Kp = base + (size_t)H * D + hh * D;
  const bf16_t* Vp = base + (size_t)2 * H * D + hh * D;
  const bf16_t* dOp = dout + (size_t)b * S * ors + hh * D;
  const float* lse_p = lse + ((size_t)b * H + hh) * S;
  const float* del_p = delta + ((size_t)b * H + hh) * S;

  bf16x8_t kf[KS], vf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    kf[ks] = frag_kc(Kp + (size_t)key * rs + ks * 16 + hf * 8);
    vf[ks] = frag_kc(Vp + (size_t)key * rs + ks * 16 + hf * 8);
  }
  f32x16_t dk[DT], dv[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) dk[t][r] = dv[t][r] = 0.0f;

  const int n_qb = S / 64 - kt;  // query blocks kt .. S/64-1
  const int n_it = (n_qb + 1) / 2;
  const bool is_do = (wave >> 1) != 0;
  const size_t lgs = is_do ? ors : rs;
  TileLoad tl;
  tl.init(lgs, lane);
  const bf16_t* lsrc = is_do ? dOp : Qp;
  const float* vsrc = is_do ? del_p : lse_p;
  auto load_pair = [&](int it) {
    const int blk = kt + 2 * it + (wave & 1);
    if (2 * it + (wave & 1) < n_qb) {
      tl.issue(smem + wave * kTileBytes, lsrc + (size_t)blk * 64 * lgs);
      float* v = vecs + (wave & 1) * 64 + (is_do ? 128 : 0);
      if (is_do) wave_vec_load(reinterpret_cast<char*>(v), vsrc + (size_t)blk * 64, lane);
      else v[lane] = vsrc[(size_t)blk * 64 + lane] * kLog2e;  // lse staged in log2 units
    }
  };

  for (int it = 0; it < n_it; ++it) {
    __syncthreads();
    load_pair(it);
    __syncthreads();
    const int qb = kt + 2 * it + qh, qs = qb * 64;
    if (2 * it + qh >= n_qb || qs + 63 < kw0) continue;
    const char* Qt = smem + qh * kTileBytes;
    const char* dOt = smem + (2 + qh) * kTileBytes;
    const float* lse_s = vecs + qh * 64;
    const float* del_s = lse_s + 128;

    // The two 32-query halves of the block one after the other (smaller live
    // register set); each dK/dV accumulator still takes its four 16-query
    // groups in order 0..3, so the sums are those of the whole block.
    const bool diag = qs < kw0 + 32;  // some query of the block precedes some key of the wave
    // Query qs + qi precedes this lane's key iff qi < key - qs.  With the lane's
    // part of qi (4 hf) folded in, one compare against a constant per score
    // decides; off the diagonal the limit is below every qi and masks nothing.
    const int mlim = (diag ? key - qs : -1) - hf * 4;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      f32x16_t p, dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) p[r] = dp[r] = 0.0f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        p = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_row(Qt, t * 32 + l32, ks * 16 + hf * 8), kf[ks], p, 0,
                                                    0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_row(dOt, t * 32 + l32, ks * 16 + hf * 8), vf[ks], dp,
                                                     0, 0, 0);
      }
      // p[r]: query qs + t*32 + (r/4)*8 + 4*hf + r%4, key `key`.
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int qc = t * 32 + (r >> 2) * 8 + (r & 3);
        const int qi = qc + hf * 4;
        float pv = __builtin_amdgcn_exp2f(fmaf(p[r], scale_log2, -lse_s[qi]));
        if (qc < mlim) pv = 0.0f;
        p[r] = pv;
        dp[r] = pv * (dp[r] - del_s[qi]);
      }
      const bf16x8_t pb[2] = {cvt8(p, 0), cvt8(p, 8)};
      const bf16x8_t sb[2] = {cvt8(dp, 0), cvt8(dp, 8)};
      // dV^T[d][key] += dO^T[d][q] P[q][key];  dK^T[d][key] += Q^T[d][q] dS[q][key]
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int gg = 0; gg < 2; ++gg) {
          const int g = 2 * t + gg;
          dv[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_tr(dOt, g * 16, dt * 32, lane), pb[gg], dv[dt],
                                                           0, 0, 0);
          dk[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_tr(Qt, g * 16, dt * 32, lane), sb[gg], dk[dt],
                                                           0, 0, 0);
        }
    }
  }

  // Add the two query halves.
  constexpr int XS = 2 * DT * 16;
  static_assert((size_t)128 * XS * 4 <= kLdsBytes, "merge buffer fits the tiles");
  float* xch = reinterpret_cast<float*>(smem) + (size_t)(kg * 64 + lane) * XS;
  __syncthreads();
  if (qh == 1) {
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        xch[t * 16 + r] = dk[t][r];
        xch[DT * 16 + t * 16 + r] = dv[t][r];
      }
  }
  __syncthreads();
  if (qh == 1) return;
  bf16_t* krow = dqkv + ((size_t)b * S + key) * rs + (size_t)H * D + hh * D;
  bf16_t* vrow = krow + (size_t)H * D;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      float a[4], c[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        a[e] = (dk[dt][4 * g + e] + xch[dt * 16 + 4 * g + e]) * scale;
        c[e] = dv[dt][4 * g + e] + xch[DT * 16 + dt * 16 + 4 * g + e];
      }
      store4(krow + dt * 32 + g * 8 + hf * 4, a);
      store4(vrow + dt * 32 + g * 8 + hf * 4, c);
    }
}

// ---------------------------------------------------------------------------
// bf16 backward: dQ (Q-parallel), the forward's layout: 64 query rows per
// workgroup, 2 query groups x 2 key halves, K and V tiles of two key blocks in the
// stage, partial dQ sums added at the end.  It also writes delta for its rows,
// which the dK/dV kernel launched after it reads.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
    attn_bwd_dq_bf16_d128(int S, int H, int Bm, int mstride, const bf16_t* __restrict__ qkv,
                          const bf16_t* __restrict__ o, const bf16_t* __restrict__ dout,
                          const float* __restrict__ lse, float* __restrict__ delta, bf16_t* __restrict__ dqkv,
                          float scale_log2, float scale) {
  extern __shared__ __align__(16) char smem[];

  const int b = seq_index(blockIdx.y, Bm, mstride), hh = blockIdx.x;  // grid as in the forward
  const int qt = gridDim.z - 1 - blockIdx.z;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int qg = wave & 1, kh = wave >> 1;
  const int q0 = qt * 64 + qg * 32;
  const int q = q0 + l32;
  const size_t rs = (size_t)3 * H * D;
  const size_t ors = (size_t)H * D;
  const bf16_t* base = qkv + (size_t)b * S * rs;
  const bf16_t* Qp = base + hh * D;
  const bf16_t* Kp = base + (size_t)H * D + hh * D;
  const bf16_t* Vp = base + (size_t)2 * H * D + hh * D;
  const bf16_t* dOp = dout + (size_t)b * S * ors + hh * D;

  bf16x8_t qf[KS], of[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    qf[ks] = frag_kc(Qp + (size_t)q * rs + ks * 16 + hf * 8);
    of[ks] = frag_kc(dOp + (size_t)q * ors + ks * 16 + hf * 8);
  }
  const float lse2 = lse[((size_t)b * H + hh) * S + q] * kLog2e;
  // delta = dO . O over the head dimension for this query: the lane holds
  // half of the row's elements (the fragments above), lane ^ 32 the other
  // half.  Written out for the dK/dV kernel, which runs after this one.
  float del;
  {
    const bf16_t* Op = o + (size_t)b * S * ors + hh * D;
    float part = 0.0f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      float ov[8], dv[8];
      load8(Op + (size_t)q * ors + ks * 16 + hf * 8, ov);
      load8(dOp + (size_t)q * ors + ks * 16 + hf * 8, dv);
#pragma unroll
      for (int e = 0; e < 8; ++e) part += dv[e] * ov[e];
    }
    del = part + __shfl_xor(part, 32, 64);
    if (kh == 0 && hf == 0) delta[((size_t)b * H + hh) * S + q] = del;
  }
  f32x16_t dq[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) dq[t][r] = 0.0f;

  const int n_kb = qt + 1;
  const int n_it = (n_kb + 1) / 2;
  TileLoad tl;
  tl.init(rs, lane);
  const bf16_t* lsrc = (wave >> 1) ? Vp : Kp;
  auto load_pair = [&](int it) {
    const int blk = 2 * it + (wave & 1);
    if (blk < n_kb) tl.issue(smem + wave * kTileBytes, lsrc + (size_t)blk * 64 * rs);
  };

  for (int it = 0; it < n_it; ++it) {
    __syncthreads();
    load_pair(it);
    __syncthreads();
    const int kb = 2 * it + kh, k0 = kb * 64;
    if (kb >= n_kb || k0 > q0 + 31) continue;
    const char* Kt = smem + kh * kTileBytes;
    const char* Vt = smem + (2 + kh) * kTileBytes;
    f32x16_t p[2], dp[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
      for (int r = 0; r < 16; ++r) p[t][r] = dp[t][r] = 0.0f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        p[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_row(Kt, t * 32 + l32, ks * 16 + hf * 8), qf[ks], p[t],
                                                       0, 0, 0);
        dp[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_row(Vt, t * 32 + l32, ks * 16 + hf * 8), of[ks],
                                                        dp[t], 0, 0, 0);
      }
    }
    // the causal mask only on a block that reaches past the wave's first query
    auto probs = [&](auto diag_c) {
      constexpr bool DIAG = decltype(diag_c)::value;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int kk = k0 + t * 32 + (r >> 2) * 8 + hf * 4 + (r & 3);
          float pv = __builtin_amdgcn_exp2f(fmaf(p[t][r], scale_log2, -lse2));
          if (DIAG && kk > q) pv = 0.0f;
          dp[t][r] = pv * (dp[t][r] - del);
        }
    };
    if (k0 + 63 > q0) probs(std::true_type{});
    else probs(std::false_type{});
    bf16x8_t sb[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) sb[g] = cvt8(dp[g >> 1], (g & 1) * 8);
    // dQ^T[d][q] += K^T[d][key] dS^T[key][q]
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        dq[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_tr(Kt, g * 16, dt * 32, lane), sb[g], dq[dt], 0, 0, 0);
  }

  constexpr int XS = DT * 16;
  static_assert((size_t)128 * XS * 4 <= kLdsBytes, "merge buffer fits the tiles");
  float* xch = reinterpret_cast<float*>(smem) + (size_t)(qg * 64 + lane) * XS;
  __syncthreads();
  if (kh == 1) {
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) xch[t * 16 + r] = dq[t][r];
  }
  __syncthreads();
  if (kh == 1) return;
  bf16_t* qrow = dqkv + ((size_t)b * S + q) * rs + hh * D;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      float a[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] = (dq[dt][4 * g + e] + xch[dt * 16 + 4 * g + e]) * scale;
      store4(qrow + dt * 32 + g * 8 + hf * 4, a);
    }
}

hipError_t launch_attention_fwd_d128(int B, int S, int H, int G, int mstride, const void* qkv, void* o, float* lse,
                                     hipStream_t st) {
  const float scale = 1.0f / sqrtf((float)D);
  static std::atomic<uint64_t> ok{0};
  hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(attn_fwd_bf16_d128), kLdsBytes, ok);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((attn_fwd_bf16_d128), dim3(H, G * B, S / 64), dim3(256), kLdsBytes, st, S, H, B, mstride,
                     (const bf16_t*)qkv, (bf16_t*)o, lse, scale * kLog2e);
  return hipGetLastError();
}

hipError_t launch_attention_bwd_d128(int B, int S, int H, int G, int mstride, const void* qkv, const void* o,
                                     const float* lse, const void* dout, void* dqkv, float* delta, hipStream_t st) {
  const float scale = 1.0f / sqrtf((float)D);
  constexpr size_t lds_q = kLdsBytes, lds_k = kLdsBytes + 256 * sizeof(float);
  static_assert(lds_k <= 160 * 1024, "LDS budget");
  static std::atomic<uint64_t> ok_k{0}, ok_q{0};
  hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(attn_bwd_dkdv_bf16_d128), lds_k, ok_k);
  if (e == hipSuccess) e = allow_dynamic_lds(reinterpret_cast<const void*>(attn_bwd_dq_bf16_d128), lds_q, ok_q);
  if (e != hipSuccess) return e;
  // dQ first: it also forms delta, which dK/dV reads.
  const dim3 grid(H, G * B, S / 64);
  hipLaunchKernelGGL((attn_bwd_dq_bf16_d128), grid, dim3(256), lds_q, st, S, H, B, mstride, (const bf16_t*)qkv,
                     (const bf16_t*)o, (const bf16_t*)dout, lse, delta, (bf16_t*)dqkv, scale * kLog2e, scale);
  hipLaunchKernelGGL((attn_bwd_dkdv_bf16_d128), grid, dim3(256), lds_k, st, S, H, B, mstride, (const bf16_t*)qkv,
                     (const bf16_t*)dout, lse, delta, (bf16_t*)dqkv, scale * kLog2e, scale);
  return hipGetLastError();
}

}  // namespace merak
