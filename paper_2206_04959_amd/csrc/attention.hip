// Causal self-attention on a rank's local heads, forward and backward.
//
// Layout: packed qkv [batch, seq, 3, heads, d] (row stride 3*heads*d), output
// o [batch, seq, heads, d], log-sum-exp lse [batch, heads, seq] (natural log of
// sum_j exp(s_ij), s = q k^T / sqrt(d)).  Keys j > i are masked.
//
// bf16 path at d = 64 and 96 (d = 128 is in attention_d128.hip;
// v_mfma_f32_32x32x16_bf16, fp32 softmax): flash-style tiling so the
// seq x seq score matrix never reaches HBM (the method published as
// FlashAttention, Dao et al. 2022; the gfx950 tiling below is our own).
//   * forward: a workgroup owns 64 query rows of one (batch, head); its four
//     waves are two groups of 32 rows times the even and odd 32-key tiles,
//     merged at the end with the online-softmax merge.  A wave computes the
//     transposed score tile S^T = K Q^T so that each lane owns one query
//     column; the softmax then needs only a lane-half exchange, and P^T stays
//     in registers as the second operand of O^T += V^T P^T.  K and V tiles sit
//     in LDS in their natural [key][d] layout; V^T fragments come from
//     transposing LDS reads.
//   * backward, deterministic (no atomics): a Q-parallel kernel accumulates dQ
//     and also forms delta_i = rowsum(dO_i * O_i) for its rows; a KV-parallel
//     kernel, run after it, accumulates dK and dV.  Both rebuild P from the
//     stored lse.
// The 32x32 accumulator layout is: lane l holds column l%32 and rows
// (r/4)*8 + (l/32)*4 + r%4 for r = 0..15.  When such an accumulator feeds the
// next MFMA as its 16-deep operand, the MFMA's k index 8*(l/32)+e is taken to
// mean row (e/4)*8 + (l/32)*4 + e%4 of that 16-row group; the other operand is
// read with transposing LDS reads in the same key order (two 8-byte reads).
//
// fp32 check mode: the same split with fp32 matrix instructions, fp32 throughout.
#include <math.h>
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "attention.h"

namespace merak {

// Work of one workgroup: sequence, head and 64-row block.
struct AttnSlot {
  int z, hh, blk;  // launch batch, head, row block counted from the one with the most work
};

// Order of the grid's workgroups (1-D grid of H * B * n_blk).  Workgroups go to
// the 8 XCDs round-robin; each XCD takes whole (sequence, head) pairs, so that a
// pair's streamed rows are fetched into one L2 only, in chunks of `chunk` pairs
// whose rows fit that L2 together, and within a chunk the blocks with the most
// work first.  The pairs left over by the division come before that, their
// blocks spread over all XCDs.  `fold`: the second half of the blocks runs in
// reverse order (see attn_order).
struct AttnOrder {
  int n_blk, chunk, fold;
};
__device__ __forceinline__ AttnSlot attn_slot(int id, int H, int n_pairs, const AttnOrder& ord) {
  const int full = n_pairs >> 3, left = n_pairs & 7;
  int pair, blk;
  if (id < left * ord.n_blk) {
    pair = full * 8 + id % left;
    blk = id / left;
  } else {
    id -= left * ord.n_blk;
    const int x = id & 7, i = id >> 3;  // i-th workgroup of one XCD
    const int c = i / (ord.chunk * ord.n_blk), in = i - c * ord.chunk * ord.n_blk;
    const int c0 = c * ord.chunk, cs = min(ord.chunk, full - c0);
    pair = x * full + c0 + in % cs;
    blk = in / cs;
  }
  const int half = (ord.n_blk + 1) >> 1;
  if (ord.fold && blk >= half) blk = ord.n_blk - 1 - (blk - half);
  return {pair / H, pair % H, blk};
}

// ---------------------------------------------------------------------------
// 32-row tiles for the streaming operands.  A [32 rows][D] bf16 tile is stored
// without padding; the 16-byte chunk c of row r sits in slot pos(c, r) of its
// row, chosen so that both kinds of fragment reads are free of bank conflicts
// (64 banks of 4 bytes): a row read takes one chunk of 16 consecutive rows per
// pass, a transposing read four neighbouring chunks of four consecutive rows.
// pos() depends on r mod 16 only.
// ---------------------------------------------------------------------------
template <int D>
struct SwTile {
  static constexpr int ROWB = D * 2;        // bytes per row
  static constexpr int CH = D / 8;          // 16-byte chunks per row
  static constexpr int BYTES = 32 * ROWB;
  static constexpr int NI = BYTES / 1024;   // 16-byte-per-lane wave loads per tile
  static constexpr __host__ __device__ int pos(int c, int r) {
    if constexpr (D == 64) return c ^ ((((r >> 1) & 1) << 2) | ((r >> 2) & 3));
    else return (c + ((r >> 2) & 3)) % CH;
  }
  static constexpr __host__ __device__ int chunk_at(int p, int r) {  // inverse of pos in c
    if constexpr (D == 96) return (p + CH - ((r >> 2) & 3)) % CH;
    else return pos(p, r);
  }
};

// 16-byte-per-lane global -> LDS load: lane i writes LDS bytes [lds_addr + 16 i,
// lds_addr + 16 i + 16).  Inline assembly, because the compiler would make
// every later LDS read wait for it; the kernels order these loads themselves
// (dma_wait).  An M0 write needs one wait state before it.
typedef int32_t i32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ i32x4_t buffer_words(const void* p) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  return i32x4_t{(int32_t)__builtin_amdgcn_readfirstlane((uint32_t)a),
                 (int32_t)__builtin_amdgcn_readfirstlane((uint32_t)((a >> 32) & 0xffffu)), 0x7fffffff, 0x00020000};
}
__device__ __forceinline__ void dma16(i32x4_t rsrc, uint32_t lds_addr, uint32_t voff) {
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds"
               :
               : "v"(voff), "s"(rsrc), "{m0}"(lds_addr)
               : "memory");
}
// Wait until at most N of this wave's vector-memory operations are outstanding.
template <int N>
__device__ __forceinline__ void dma_wait() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// Wait for this wave's LDS reads (before a load overwrites what they read).
__device__ __forceinline__ void lds_wait() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// One wave's plan for loading a tile from rows of stride `gs` elements.
template <int D>
struct TileDma {
  uint32_t voff[SwTile<D>::NI];
  __device__ __forceinline__ void init(size_t gs, int lane) {
#pragma unroll
    for (int q = 0; q < SwTile<D>::NI; ++q) {
      const int idx = q * 64 + lane, r = idx / SwTile<D>::CH, p = idx % SwTile<D>::CH;
      voff[q] = (uint32_t)((size_t)r * gs * 2) + (uint32_t)SwTile<D>::chunk_at(p, r) * 16u;
    }
  }
  __device__ __forceinline__ void issue(uint32_t lds_addr, const bf16_t* rows) const {
    const i32x4_t rsrc = buffer_words(rows);
#pragma unroll
    for (int q = 0; q < SwTile<D>::NI; ++q) dma16(rsrc, lds_addr + q * 1024, voff[q]);
  }
};

// Fragment reads of a tile: row(ks) is the MFMA operand with lane l holding row
// l % 32 and columns 16 ks + 8 (l / 32) + 0..7; tr(kb, dt) the transposed one,
// lane l holding column 32 dt + l % 32 and rows kb + 4 (l / 32) + 0..3, then
// kb + 8 + 4 (l / 32) + 0..3 (the row order of an accumulator reused as the
// 16-deep operand), from two transposing LDS reads.
template <int D>
struct TileFrag {
  using ST = SwTile<D>;
  int ro[D / 16], lo[D / 32], hi[D / 32];
  __device__ __forceinline__ void init(int lane) {
    const int l32 = lane & 31, hf = lane >> 5;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) ro[ks] = l32 * ST::ROWB + ST::pos(2 * ks + hf, l32) * 16;
    const int r = hf * 4 + ((lane & 15) >> 2), cl = ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1);
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) {
      lo[dt] = r * ST::ROWB + ST::pos(dt * 4 + cl, r) * 16 + (lane & 1) * 8;
      hi[dt] = (r + 8) * ST::ROWB + ST::pos(dt * 4 + cl, r + 8) * 16 + (lane & 1) * 8;
    }
  }
  __device__ __forceinline__ bf16x8_t row(const char* tile, int ks) const {
    return *reinterpret_cast<const bf16x8_t*>(tile + ro[ks]);
  }
  __device__ __forceinline__ bf16x8_t tr(const char* tile, int kb, int dt) const {
    const char* t = tile + kb * ST::ROWB;
    const s16x4_t a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((MERAK_LDS s16x4_t*)(t + lo[dt]));
    const s16x4_t b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((MERAK_LDS s16x4_t*)(t + hi[dt]));
    const s16x8_t v = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
    return __builtin_bit_cast(bf16x8_t, v);
  }
};

// Keeps a value's computation where it is written (between two MFMAs), rather
// than sunk to its use.
__device__ __forceinline__ float pinned(float v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Value of the other half-wave's matching lane combined with this lane's.
__device__ __forceinline__ float half_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_sum(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Waits for this wave's loads and joins the workgroup barrier: the tiles that
// were on their way can be read, and all waves are done with the tiles of the
// step before.
__device__ __forceinline__ void step_barrier() {
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// ---------------------------------------------------------------------------
// bf16 forward.  A workgroup owns 64 query rows of one (batch, head); wave w
// takes the 32 rows of group w % 2 against the even (w < 2) or odd 32-key
// tiles, and the two halves are merged at the end (online-softmax merge).
//
// The matrix and the vector units take about equal time here, so each wave
// overlaps them itself: step t issues the MFMAs of S(t + 1) and of the
// P V product of tile t one at a time between the softmax instructions of tile
// t.  K and V tiles sit in two-slot rings, loaded one step ahead; one barrier
// per step.  Small tiles and 157 registers (d = 96) let three workgroups share
// a CU.  What bounds it: on small grids the longest row block's chain (0.57 us a
// step at d = 96: one pair takes 12.7 us at 1024 rows, 21.8 at 2048), on large ones
// the vector unit (16 exponentials, 60 other instructions and 12 MFMAs of 32 cycles
// per 32 x 32 tile).  Against 64-key blocks with padded tiles and no overlap inside
// a wave: 4 x 1024 x 8 heads of 96 18.8 -> 16.5 us, 4 x 2048 x 25 of 96 159 -> 118.
// A third slot was 4% faster on the first of these and 6% slower on the second (two
// workgroups per CU).
// ---------------------------------------------------------------------------
template <int D>
constexpr size_t fwd_lds_bytes() { return (size_t)8 * SwTile<D>::BYTES; }

template <int D>
__global__ void __launch_bounds__(256, 2) attn_fwd_bf16(int S, int H, int Bm, int mstride,
                                                        const bf16_t* __restrict__ qkv, bf16_t* __restrict__ o,
                                                        float* __restrict__ lse, float scale_log2, int n_pairs,
                                                        AttnOrder ord) {
  using ST = SwTile<D>;
  constexpr int KS = D / 16, DT = D / 32, TB = ST::BYTES;
  extern __shared__ __align__(16) char smem[];  // [slot][K even, K odd, V even, V odd]

  const AttnSlot slot = attn_slot(blockIdx.x, H, n_pairs, ord);
  const int b = seq_index(slot.z, Bm, mstride), hh = slot.hh;
  const int qt = ord.n_blk - 1 - slot.blk;  // the last rows see the most keys
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qg = wave & 1, kh = wave >> 1;
  const int q0 = qt * 64 + qg * 32;
  const int q = q0 + l32;
  const size_t rs = (size_t)3 * H * D;
  const bf16_t* base = qkv + (size_t)b * S * rs;
  const bf16_t* Qp = base + hh * D;

  // Wave w loads tile w of a step: K (w < 2) or V of the even or odd keys.
  const int nt = qt + 1;  // steps; tile t of half kh holds keys 64 t + 32 kh ..
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(MERAK_LDS char*)smem) + wave * TB;
  const bf16_t* lsrc = base + (size_t)(1 + kh) * H * D + hh * D + (size_t)(wave & 1) * 32 * rs;
  TileDma<D> dma;
  dma.init(rs, lane);
  auto load = [&](int t) {
    if (t < nt) dma.issue(lds0 + (t & 1) * 4 * TB, lsrc + (size_t)t * 64 * rs);
  };
  TileFrag<D> fr;
  fr.init(lane);
  bf16x8_t qf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) qf[ks] = frag_kc(Qp + (size_t)q * rs + ks * 16 + hf * 8);
  load(0);
  // The wait for the query fragments belongs here: left to their first use it
  // would also cover the tile loads.
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qf[ks]));

  f32x16_t oacc[DT], s;
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[t][r] = 0.0f;
  float m = -INFINITY, nm = 0.0f;  // running maximum (scaled, log2 units); -m, 0 before the first score
  float l[2] = {0.0f, 0.0f};       // sum, in two parts

  // Causal mask of tile t's scores: x[r] is key 64 t + 32 kh + (r/4)*8 + 4*hf +
  // r%4, query q.  Only the last tiles reach past a query.
  auto mask = [&](f32x16_t& x, int t) {
    const int lim = q - (64 * t + 32 * kh) - hf * 4;
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if ((r >> 2) * 8 + (r & 3) > lim) x[r] = -INFINITY;
  };
  // The running maximum after a tile whose own maximum (this lane's half) is mx.
  auto new_max = [&](float mx) {
    mx = half_max(mx) * scale_log2;
    if (__ballot(mx > m)) {  // rescale only when some row's maximum grew
      const float mnew = fmaxf(m, mx);
      // a row without any score yet keeps its (zero) sums: no -inf - -inf
      nm = mnew == -INFINITY ? 0.0f : -mnew;
      const float alpha = __builtin_amdgcn_exp2f(m + nm);
      m = mnew;
      l[0] *= alpha;
      l[1] *= alpha;
#pragma unroll
      for (int u = 0; u < DT; ++u)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[u][r] *= alpha;
    }
  };

  step_barrier();
  if (wave < 2) load(1);
  {
    const char* Kt = smem + kh * TB;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.0f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.row(Kt, ks), qf[ks], s, 0, 0, 0);
    if (nt == 1) mask(s, 0);
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
    new_max(mx);
  }

  // Step t, with t % 2 = SLOT known at compile time (tile addresses become
  // instruction offsets).
  auto step = [&](int t, auto slot_c) {
    constexpr int SLOT = decltype(slot_c)::value;
    // K(t + 1) and V(t) are there; K(t) and V(t - 1) are no longer needed
    step_barrier();
    load(wave < 2 ? t + 2 : t + 1);
    const char* Kt = smem + ((SLOT ^ 1) * 4 + kh) * TB;  // past the last step: stale, its scores are not used
    const char* Vt = smem + (SLOT * 4 + 2 + kh) * TB;
    bf16x8_t kf[KS], vf[2][DT], pb[2];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kf[ks] = fr.row(Kt, ks);
    // Softmax of tile t in stages, so that no instruction waits for the one
    // before it: all exponents first (while the K fragments are on their way),
    // the exponentials between the MFMAs, each added to the sum two later.
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = pinned(fmaf(s[r], scale_log2, nm));
    }
    auto prob = [&](int r) {
      s[r] = pinned(__builtin_amdgcn_exp2f(s[r]));
      if (r >= 2) l[r & 1] = pinned(l[r & 1] + s[r - 2]);
    };
    f32x16_t sn;
#pragma unroll
    for (int r = 0; r < 16; ++r) sn[r] = 0.0f;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < KS; ++u) {
      sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[u], qf[u], sn, 0, 0, 0);
      vf[u / DT][u % DT] = fr.tr(Vt, (u / DT) * 16, u % DT);
#pragma unroll
      for (int r = 10 * u / KS; r < 10 * (u + 1) / KS; ++r) prob(r);
      __builtin_amdgcn_sched_barrier(0);
    }
    pb[0] = cvt8(s, 0);
    // O^T[d][q] += V^T[d][key] P^T[key][q]
#pragma unroll
    for (int u = 0; u < DT; ++u) {
      oacc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[0][u], pb[0], oacc[u], 0, 0, 0);
#pragma unroll
      for (int r = 10 + 6 * u / DT; r < 10 + 6 * (u + 1) / DT; ++r) prob(r);
      __builtin_amdgcn_sched_barrier(0);
    }
    l[0] += s[14];
    l[1] += s[15];
    pb[1] = cvt8(s, 8);
    float mx = sn[0];
#pragma unroll
    for (int u = 0; u < DT; ++u) {
      oacc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[1][u], pb[1], oacc[u], 0, 0, 0);
      if (u > 0) {
#pragma unroll
        for (int r = 1 + 15 * (u - 1) / (DT - 1); r < 1 + 15 * u / (DT - 1); ++r) mx = fmaxf(mx, sn[r]);
        mx = pinned(mx);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    s = sn;
    if (t + 1 == nt - 1) {
      mask(s, t + 1);
      mx = s[0];
#pragma unroll
      for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
    }
    if (t + 1 < nt) new_max(mx);
  };
  for (int t = 0; t < nt; t += 2) {
    step(t, std::integral_constant<int, 0>{});
    if (t + 1 < nt) step(t + 1, std::integral_constant<int, 1>{});
  }

  // Merge the two key halves of each query group (partial m, l, O^T).
  constexpr int XS = 2 + DT * 16;
  static_assert((size_t)128 * XS * 4 <= fwd_lds_bytes<D>(), "merge buffer fits the tiles");
  float* xch = reinterpret_cast<float*>(smem) + (size_t)(qg * 64 + lane) * XS;
  __syncthreads();
  if (kh == 1) {
    xch[0] = m;
    xch[1] = l[0] + l[1];
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
  const float lt = half_sum((l[0] + l[1]) * a0 + l1 * a1);
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
// (w < 2) or odd 32-query tiles from the diagonal on; the two partial sums are
// added at the end.  Q and dO tiles sit in two-slot rings, loaded one step
// ahead, with one barrier per step.  P is rebuilt from lse.  Within a step the
// MFMAs run back to back: S, then dP beside the exponentials of P, then
// dV += dO^T P beside dS = P (dP - delta), then dK += Q^T dS; each product's
// fragments are read beside the one before it.  What bounds it: the chain of
// steps of the first key block (0.70 us each at d = 96: one pair takes 15.5 us at
// 1024 rows, 26.7 at 2048), with two workgroups per CU (254 registers at d = 96).
// Against 64-query blocks loaded after a barrier and used after the next: 4 x 1024
// x 8 heads of 96 35.1 -> 24.9 us, 4 x 2048 x 25 of 96 256 -> 206.
// ---------------------------------------------------------------------------
template <int D>
constexpr size_t bwd_lds_bytes() { return (size_t)8 * SwTile<D>::BYTES + 2 * 2 * 64 * sizeof(float); }

template <int D>
__global__ void __launch_bounds__(256, 2)
    attn_bwd_dkdv_bf16(int S, int H, int Bm, int mstride, const bf16_t* __restrict__ qkv,
                       const bf16_t* __restrict__ dout, const float* __restrict__ lse,
                       const float* __restrict__ delta, bf16_t* __restrict__ dqkv, float scale_log2, float scale,
                       int n_pairs, AttnOrder ord) {
  using ST = SwTile<D>;
  constexpr int KS = D / 16, DT = D / 32, TB = ST::BYTES;
  extern __shared__ __align__(16) char smem[];  // [slot][Q even, Q odd, dO even, dO odd], then lse/delta
  float* const vecs = reinterpret_cast<float*>(smem + 8 * TB);  // [slot][half][lse 32, delta 32]

  const AttnSlot slot = attn_slot(blockIdx.x, H, n_pairs, ord);
  const int b = seq_index(slot.z, Bm, mstride), hh = slot.hh;
  const int kt = slot.blk;  // early keys see the most queries
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave & 1, qh = wave >> 1;
  const int key = kt * 64 + kg * 32 + l32;
  const size_t rs = (size_t)3 * H * D;
  const size_t ors = (size_t)H * D;
  const bf16_t* base = qkv + (size_t)b * S * rs;
  const bf16_t* Kp = base + (size_t)H * D + hh * D;
  const bf16_t* Vp = base + (size_t)2 * H * D + hh * D;

  // Wave w loads tile w of a step (Q or dO of the even or odd queries) and the
  // 32 lse or delta values that go with it; the values pass through a register,
  // fetched a step before they are written to LDS.  lse is staged in log2 units.
  const int nt = S / 64 - kt;  // steps; tile t of half q holds queries 64 (kt + t) + 32 q ..
  const bool is_do = wave >= 2;
  const size_t lgs = is_do ? ors : rs;
  const bf16_t* lsrc = (is_do ? dout + (size_t)b * S * ors : base) + hh * D + (size_t)(kt * 64 + (wave & 1) * 32) * lgs;
  const float* vsrc = (is_do ? delta : lse) + ((size_t)b * H + hh) * S + kt * 64 + (wave & 1) * 32 + l32;
  const float vscale = is_do ? 1.0f : kLog2e;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(MERAK_LDS char*)smem) + wave * TB;
  float* const vdst = vecs + (wave & 1) * 64 + (is_do ? 32 : 0) + l32;
  TileDma<D> dma;
  dma.init(lgs, lane);
  auto load = [&](int t) {
    if (t < nt) dma.issue(lds0 + (t & 1) * 4 * TB, lsrc + (size_t)t * 64 * lgs);
  };
  TileFrag<D> fr;
  fr.init(lane);
  bf16x8_t kf[KS], vf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    kf[ks] = frag_kc(Kp + (size_t)key * rs + ks * 16 + hf * 8);
    vf[ks] = frag_kc(Vp + (size_t)key * rs + ks * 16 + hf * 8);
  }
  float vnext = vsrc[0];
  load(0);
  // The wait for these loads belongs here: left to their first use it would
  // also cover later tile loads.
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(kf[ks]), "+v"(vf[ks]));
  vdst[0] = vnext * vscale;
  if (nt > 1) vnext = vsrc[64];

  f32x16_t dk[DT], dv[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) dk[t][r] = dv[t][r] = 0.0f;

  auto step = [&](int t, auto slot_c) {
    constexpr int SLOT = decltype(slot_c)::value;
    step_barrier();  // this step's tiles are there; those of the step before are no longer needed
    if (t + 1 < nt) {
      vdst[(SLOT ^ 1) * 128] = vnext * vscale;
      if (t + 2 < nt) vnext = vsrc[(size_t)(t + 2) * 64];
    }
    load(t + 1);
    const char* Qt = smem + (SLOT * 4 + qh) * TB;
    const char* dOt = smem + (SLOT * 4 + 2 + qh) * TB;
    const float* vec = vecs + SLOT * 128 + qh * 64 + hf * 4;
    f32x16_t p, dp;
#pragma unroll
    for (int r = 0; r < 16; ++r) p[r] = dp[r] = 0.0f;
    // Each product's fragments are read while the one before it runs.
    static_assert(KS == 2 * DT, "as many row fragments as transposed ones");
    bf16x8_t fa[KS], fb[KS];
    f32x4_t ls[4], de[4];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) fa[ks] = fr.row(Qt, ks);
#pragma unroll
    for (int g = 0; g < 4; ++g) ls[g] = *reinterpret_cast<const f32x4_t*>(vec + g * 8);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      p = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks], kf[ks], p, 0, 0, 0);
      fb[ks] = fr.row(dOt, ks);
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[ks], vf[ks], dp, 0, 0, 0);
      fa[ks] = fr.tr(dOt, (ks / DT) * 16, ks % DT);
#pragma unroll
      for (int r = 16 * ks / KS; r < 16 * (ks + 1) / KS; ++r)
        p[r] = pinned(__builtin_amdgcn_exp2f(fmaf(p[r], scale_log2, -ls[r >> 2][r & 3])));
      __builtin_amdgcn_sched_barrier(0);
    }
    // p[r]: query 64 (kt + t) + 32 qh + (r/4)*8 + 4*hf + r%4, key `key`.  Masked
    // after the exponential, so that a query's non-finite lse reaches no key after it.
    if (t == 0) {  // the only tiles with queries before a key
      const int lim = key - (kt * 64 + qh * 32) - hf * 4;
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if ((r >> 2) * 8 + (r & 3) < lim) p[r] = 0.0f;
    }
    __builtin_amdgcn_sched_barrier(0);
    const bf16x8_t pb[2] = {cvt8(p, 0), cvt8(p, 8)};
#pragma unroll
    for (int g = 0; g < 4; ++g) de[g] = *reinterpret_cast<const f32x4_t*>(vec + 32 + g * 8);
    // dV^T[d][key] += dO^T[d][q] P[q][key];  dK^T[d][key] += Q^T[d][q] dS[q][key]
#pragma unroll
    for (int u = 0; u < KS; ++u) {
      dv[u % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[u], pb[u / DT], dv[u % DT], 0, 0, 0);
      fb[u] = fr.tr(Qt, (u / DT) * 16, u % DT);
#pragma unroll
      for (int r = 16 * u / KS; r < 16 * (u + 1) / KS; ++r) p[r] = pinned(p[r] * (dp[r] - de[r >> 2][r & 3]));
      __builtin_amdgcn_sched_barrier(0);
    }
    const bf16x8_t sb[2] = {cvt8(p, 0), cvt8(p, 8)};
#pragma unroll
    for (int u = 0; u < KS; ++u)
      dk[u % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[u], sb[u / DT], dk[u % DT], 0, 0, 0);
  };
  for (int t = 0; t < nt; t += 2) {
    step(t, std::integral_constant<int, 0>{});
    if (t + 1 < nt) step(t + 1, std::integral_constant<int, 1>{});
  }

  // Add the two query halves: the even half's waves finish dK, the odd half's
  // dV, each handing over the other.
  static_assert((size_t)4 * DT * 4096 <= (size_t)8 * TB, "merge buffer fits the tiles");
  char* const mine = smem + (kg * 2 + qh) * DT * 4096 + lane * 16;
  const char* const theirs = smem + (kg * 2 + (qh ^ 1)) * DT * 4096 + lane * 16;
  auto put = [&](const f32x16_t (&a)[DT]) {
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<f32x4_t*>(mine + (t * 4 + i) * 1024) =
            f32x4_t{a[t][4 * i], a[t][4 * i + 1], a[t][4 * i + 2], a[t][4 * i + 3]};
  };
  auto finish = [&](const f32x16_t (&a)[DT], bf16_t* row, float f) {
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f32x4_t o = *reinterpret_cast<const f32x4_t*>(theirs + (t * 4 + i) * 1024);
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (a[t][4 * i + e] + o[e]) * f;
        store4(row + t * 32 + i * 8 + hf * 4, v);
      }
  };
  __syncthreads();
  if (qh == 0) put(dv);
  else put(dk);
  __syncthreads();
  bf16_t* krow = dqkv + ((size_t)b * S + key) * rs + (size_t)H * D + hh * D;
  if (qh == 0) finish(dk, krow, scale);
  else finish(dv, krow + (size_t)H * D, 1.0f);
}

// ---------------------------------------------------------------------------
// bf16 backward: dQ (Q-parallel), the forward's layout: 64 query rows per
// workgroup, 2 query groups x even / odd 32-key tiles, K and V tiles in two-slot
// rings, partial dQ sums added at the end.  It also writes delta for its rows,
// which the dK/dV kernel launched after it reads.  Against 64-key blocks loaded
// after a barrier and used after the next: 4 x 1024 x 8 heads of 96 25.3 -> 21.0 us,
// 4 x 2048 x 25 of 96 206 -> 164.
// ---------------------------------------------------------------------------
template <int D>
__global__ void __launch_bounds__(256, 2) attn_bwd_dq_bf16(int S, int H, int Bm, int mstride,
                                                           const bf16_t* __restrict__ qkv,
                                                           const bf16_t* __restrict__ o,
                                                           const bf16_t* __restrict__ dout,
                                                           const float* __restrict__ lse, float* __restrict__ delta,
                                                           bf16_t* __restrict__ dqkv, float scale_log2, float scale,
                                                           int n_pairs, AttnOrder ord) {
  using ST = SwTile<D>;
  constexpr int KS = D / 16, DT = D / 32, TB = ST::BYTES;
  extern __shared__ __align__(16) char smem[];  // [slot][K even, K odd, V even, V odd]

  const AttnSlot slot = attn_slot(blockIdx.x, H, n_pairs, ord);
  const int b = seq_index(slot.z, Bm, mstride), hh = slot.hh;
  const int qt = ord.n_blk - 1 - slot.blk;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qg = wave & 1, kh = wave >> 1;
  const int q = qt * 64 + qg * 32 + l32;
  const size_t rs = (size_t)3 * H * D;
  const size_t ors = (size_t)H * D;
  const bf16_t* base = qkv + (size_t)b * S * rs;
  const bf16_t* Qp = base + hh * D;
  const bf16_t* dOp = dout + (size_t)b * S * ors + hh * D;

  const int nt = qt + 1;  // steps; tile t of half kh holds keys 64 t + 32 kh ..
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(MERAK_LDS char*)smem) + wave * TB;
  const bf16_t* lsrc = base + (size_t)(1 + kh) * H * D + hh * D + (size_t)(wave & 1) * 32 * rs;
  TileDma<D> dma;
  dma.init(rs, lane);
  auto load = [&](int t) {
    if (t < nt) dma.issue(lds0 + (t & 1) * 4 * TB, lsrc + (size_t)t * 64 * rs);
  };
  TileFrag<D> fr;
  fr.init(lane);
  load(0);
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
      unpack8(__builtin_bit_cast(u32x4_t, of[ks]), dv);
#pragma unroll
      for (int e = 0; e < 8; ++e) part += dv[e] * ov[e];
    }
    del = half_sum(part);
    if (kh == 0 && hf == 0) delta[((size_t)b * H + hh) * S + q] = del;
  }
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qf[ks]), "+v"(of[ks]));
  f32x16_t dq[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) dq[t][r] = 0.0f;

  auto step = [&](int t, auto slot_c) {
    constexpr int SLOT = decltype(slot_c)::value;
    step_barrier();  // this step's tiles are there; those of the step before are no longer needed
    load(t + 1);
    const char* Kt = smem + (SLOT * 4 + kh) * TB;
    const char* Vt = smem + (SLOT * 4 + 2 + kh) * TB;
    f32x16_t p, dp;
#pragma unroll
    for (int r = 0; r < 16; ++r) p[r] = dp[r] = 0.0f;
    // Each product's fragments are read while the one before it runs.
    static_assert(KS == 2 * DT, "as many row fragments as transposed ones");
    bf16x8_t fa[KS], fb[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) fa[ks] = fr.row(Kt, ks);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      p = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks], qf[ks], p, 0, 0, 0);
      fb[ks] = fr.row(Vt, ks);
      __builtin_amdgcn_sched_barrier(0);
    }
    // p[r]: key 64 t + 32 kh + (r/4)*8 + 4*hf + r%4, query q.
    if (t == nt - 1) {  // the only tiles that reach past a query
      const int lim = q - (64 * t + 32 * kh) - hf * 4;
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if ((r >> 2) * 8 + (r & 3) > lim) p[r] = -INFINITY;
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[ks], of[ks], dp, 0, 0, 0);
      fa[ks] = fr.tr(Kt, (ks / DT) * 16, ks % DT);
#pragma unroll
      for (int r = 16 * ks / KS; r < 16 * (ks + 1) / KS; ++r)
        p[r] = pinned(__builtin_amdgcn_exp2f(fmaf(p[r], scale_log2, -lse2)));
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) p[r] *= dp[r] - del;
    const bf16x8_t sb[2] = {cvt8(p, 0), cvt8(p, 8)};
    // dQ^T[d][q] += K^T[d][key] dS^T[key][q]
#pragma unroll
    for (int u = 0; u < KS; ++u)
      dq[u % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[u], sb[u / DT], dq[u % DT], 0, 0, 0);
  };
  for (int t = 0; t < nt; t += 2) {
    step(t, std::integral_constant<int, 0>{});
    if (t + 1 < nt) step(t + 1, std::integral_constant<int, 1>{});
  }

  // Add the two key halves; each finishes half of the columns.
  constexpr int DH = (DT + 1) / 2;  // 32-column groups finished by the even half
  static_assert((size_t)4 * DH * 4096 <= (size_t)8 * TB, "merge buffer fits the tiles");
  char* const mine = smem + (qg * 2 + kh) * DH * 4096 + lane * 16;
  const char* const theirs = smem + (qg * 2 + (kh ^ 1)) * DH * 4096 + lane * 16;
  auto put = [&](int dt, int at) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *reinterpret_cast<f32x4_t*>(mine + (at * 4 + i) * 1024) =
          f32x4_t{dq[dt][4 * i], dq[dt][4 * i + 1], dq[dt][4 * i + 2], dq[dt][4 * i + 3]};
  };
  bf16_t* qrow = dqkv + ((size_t)b * S + q) * rs + hh * D;
  auto finish = [&](int dt, int at) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f32x4_t x = *reinterpret_cast<const f32x4_t*>(theirs + (at * 4 + i) * 1024);
      float a[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] = (dq[dt][4 * i + e] + x[e]) * scale;
      store4(qrow + dt * 32 + i * 8 + hf * 4, a);
    }
  };
  __syncthreads();
  if (kh == 0) {
#pragma unroll
    for (int dt = DH; dt < DT; ++dt) put(dt, dt - DH);
  } else {
#pragma unroll
    for (int dt = 0; dt < DH; ++dt) put(dt, dt);
  }
  __syncthreads();
  if (kh == 0) {
#pragma unroll
    for (int dt = 0; dt < DH; ++dt) finish(dt, dt);
  } else {
#pragma unroll
    for (int dt = DH; dt < DT; ++dt) finish(dt, dt - DH);
  }
}

// ---------------------------------------------------------------------------
// fp32 check mode, on the fp32 matrix instruction (v_mfma_f32_32x32x2_f32: fp32
// products and sums).  A workgroup owns 32 rows of one (batch, head); each of
// its four waves takes every fourth 32-row tile of the other sequence axis, and
// the four partial results are merged at the end in wave order.  Operands come
// straight from global memory: the 32x32x2 product's k index h of its step j
// of chunk c is taken to mean column 8 c + 4 h + j (h = lane / 32), so a lane
// reads 16 bytes of its row; products over the tile's rows take an accumulator
// register as one operand (rows (r/4)*8 + 4 h + r%4) and one row segment of 32
// columns as the other.  What bounds it: small calls are a chain of a few
// tiles (a tile is 2 x 4096 cycles of MFMAs at d = 128).  One thread per row,
// as before, took 221 + 422 us forward and backward at 2 x 128 x 4 heads of 64.
// ---------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ void rows_f32(const float* p, f32x4_t (&f)[D / 8]) {
#pragma unroll
  for (int c = 0; c < D / 8; ++c) f[c] = *reinterpret_cast<const f32x4_t*>(p + 8 * c);
}

// x[row of a][row of b] = a . b over the D columns.
template <int D>
__device__ __forceinline__ void dot_f32(const f32x4_t (&a)[D / 8], const f32x4_t (&b)[D / 8], f32x16_t& x) {
#pragma unroll
  for (int r = 0; r < 16; ++r) x[r] = 0.0f;
#pragma unroll
  for (int c = 0; c < D / 8; ++c)
#pragma unroll
    for (int j = 0; j < 4; ++j) x = __builtin_amdgcn_mfma_f32_32x32x2f32(a[c][j], b[c][j], x, 0, 0, 0);
}

// acc[column][lane's row] += sum over the tile's 32 rows of t[row][column] x[row].
// `t`: the tile's first row plus the lane's 4 h rows and l32 columns.
template <int D>
__device__ __forceinline__ void accumulate_f32(const float* t, size_t ld, const f32x16_t& x, f32x16_t (&acc)[D / 32]) {
#pragma unroll
  for (int r = 0; r < 16; ++r)
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
      acc[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(t[(size_t)((r >> 2) * 8 + (r & 3)) * ld + dt * 32], x[r], acc[dt],
                                                     0, 0, 0);
}

template <int D>
constexpr size_t f32_lds_bytes() { return (size_t)4 * D * 32 * 4 + 4 * 64 * 4; }

// Sum of the four waves' accumulators, times f, to `out` (the lane's row, first
// column).  Returns whether one of the lane's results is not finite.
template <int D>
__device__ __forceinline__ bool merge_f32(char* smem, const f32x16_t (&acc)[D / 32], float f, float* out, int wave,
                                          int lane) {
  float* part = reinterpret_cast<float*>(smem);
  __syncthreads();
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) part[((wave * (D / 32) + dt) * 16 + r) * 64 + lane] = acc[dt][r];
  __syncthreads();
  bool odd = false;
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt) {  // wave w: registers 4 w .. 4 w + 3 of every column group
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = 0.0f;
#pragma unroll
      for (int w = 0; w < 4; ++w) v[e] += part[((w * (D / 32) + dt) * 16 + wave * 4 + e) * 64 + lane];
      v[e] *= f;
      odd |= !(fabsf(v[e]) < INFINITY);
    }
    store4(out + dt * 32 + wave * 8 + (lane >> 5) * 4, v);
  }
  return odd;
}

// Results that are not finite.  The products take masked terms as 0 times a value
// of the diagonal tile, which is NaN where that value is not finite: a token's NaN
// would reach rows that the mask keeps from it.  So a lane whose results (D / 32
// groups of 4 columns, `col` the first) are not all finite forms them once more,
// term by term over the rows that it does see, and replaces those that were not.
// Nothing of it runs on finite results; a test of the values in the products made
// the kernels 15-20% slower.
template <int D>
__device__ __forceinline__ void replace_f32(float* out, const f32x4_t (&v)[D / 32], float f) {
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (!(fabsf(out[dt * 32 + e]) < INFINITY)) out[dt * 32 + e] = v[dt][e] * f;
}

template <int D>
__device__ __forceinline__ float row_dot_f32(const float* a, const float* b) {
  float s = 0.0f;
#pragma unroll 4
  for (int d = 0; d < D; ++d) s += a[d] * b[d];
  return s;
}

template <int D>
__device__ __forceinline__ void add_f32(f32x4_t (&acc)[D / 32], float a, float p, const float* v) {
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt) acc[dt] = acc[dt] * a + p * *reinterpret_cast<const f32x4_t*>(v + dt * 32);
}

template <int D>
__global__ void __launch_bounds__(256) attn_fwd_f32(int S, int H, int Bm, int mstride, const float* __restrict__ qkv,
                                                    float* __restrict__ o, float* __restrict__ lse, float scale) {
  extern __shared__ __align__(16) char smem[];
  const int b = seq_index(blockIdx.x / H, Bm, mstride), hh = blockIdx.x % H;
  const int qt = gridDim.y - 1 - blockIdx.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, hf = lane >> 5;
  const int q = qt * 32 + l32;
  const size_t rs = (size_t)3 * H * D;
  const float* base = qkv + (size_t)b * S * rs + (size_t)hh * D;
  const float* Kp = base + (size_t)H * D;
  const float* Vp = Kp + (size_t)H * D;
  f32x4_t qf[D / 8];
  rows_f32<D>(base + (size_t)q * rs + 4 * hf, qf);
  f32x16_t oacc[D / 32];
#pragma unroll
  for (int t = 0; t < D / 32; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[t][r] = 0.0f;
  float m = -INFINITY, l = 0.0f;
  for (int t = wave; t <= qt; t += 4) {
    f32x4_t kf[D / 8];
    f32x16_t s;
    rows_f32<D>(Kp + (size_t)(t * 32 + l32) * rs + 4 * hf, kf);
    dot_f32<D>(kf, qf, s);  // s[r]: key 32 t + (r/4)*8 + 4*hf + r%4, query q
    float mloc = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = t * 32 + (r >> 2) * 8 + hf * 4 + (r & 3) > q ? -INFINITY : s[r] * scale;
      mloc = fmaxf(mloc, s[r]);
    }
    const float mn = fmaxf(m, half_max(mloc));
    const float alpha = expf(m - mn);  // every tile has an unmasked key for each query
    l *= alpha;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = expf(s[r] - mn);
      l += s[r];
    }
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[dt][r] *= alpha;
    m = mn;
    accumulate_f32<D>(Vp + (size_t)(t * 32 + hf * 4) * rs + l32, rs, s, oacc);
  }
  // Online-softmax merge: common maximum and sum of each row, then plain sums.
  float* ml = reinterpret_cast<float*>(smem + (size_t)4 * D * 32 * 4);
  l = half_sum(l);
  if (hf == 0) {
    ml[wave * 64 + l32] = m;
    ml[wave * 64 + 32 + l32] = l;
  }
  __syncthreads();
  float mt = -INFINITY, lt = 0.0f;
#pragma unroll
  for (int w = 0; w < 4; ++w) mt = fmaxf(mt, ml[w * 64 + l32]);
#pragma unroll
  for (int w = 0; w < 4; ++w) lt += ml[w * 64 + 32 + l32] * expf(ml[w * 64 + l32] - mt);
  const float a = expf(m - mt) / lt;
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[dt][r] *= a;
  float* orow = o + (((size_t)b * S + q) * H + hh) * D;
  const bool odd = merge_f32<D>(smem, oacc, 1.0f, orow, wave, lane);
  if (wave == 0 && hf == 0) lse[((size_t)b * H + hh) * S + q] = mt + logf(lt);
  if (!odd) return;
  const int col = wave * 8 + hf * 4;
  f32x4_t acc[D / 32] = {};
  m = -INFINITY;
  l = 0.0f;
  for (int j = 0; j <= q && l == l; ++j) {
    const float s = row_dot_f32<D>(base + (size_t)q * rs, Kp + (size_t)j * rs) * scale;
    const float mn = fmaxf(m, s), alpha = expf(m - mn), p = expf(s - mn);
    l = l * alpha + p;
    add_f32<D>(acc, alpha, p, Vp + (size_t)j * rs + col);
    m = mn;
  }
  replace_f32<D>(orow + col, acc, 1.0f / l);
}

// dQ, and delta = dO . O of its rows for the dK/dV kernel launched after it.
// (At most two waves per SIMD: with three at d = 64 the loads are issued later, 35.0
// against 33.3 us for the backward of 1 x 256 x 4 heads.)
template <int D>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 2)))
    attn_bwd_dq_f32(int S, int H, int Bm, int mstride, const float* __restrict__ qkv, const float* __restrict__ o,
                    const float* __restrict__ dout, const float* __restrict__ lse, float* __restrict__ delta,
                    float* __restrict__ dqkv, float scale) {
  extern __shared__ __align__(16) char smem[];
  const int b = seq_index(blockIdx.x / H, Bm, mstride), hh = blockIdx.x % H;
  const int qt = gridDim.y - 1 - blockIdx.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, hf = lane >> 5;
  const int q = qt * 32 + l32;
  const size_t rs = (size_t)3 * H * D, row = (((size_t)b * S + q) * H + hh) * D;
  const float* base = qkv + (size_t)b * S * rs + (size_t)hh * D;
  const float* Kp = base + (size_t)H * D;
  const float* Vp = Kp + (size_t)H * D;
  f32x4_t qf[D / 8], of[D / 8];
  rows_f32<D>(base + (size_t)q * rs + 4 * hf, qf);
  rows_f32<D>(dout + row + 4 * hf, of);
  const float L = lse[((size_t)b * H + hh) * S + q];
  float part = 0.0f;
#pragma unroll
  for (int c = 0; c < D / 8; ++c) {
    const f32x4_t ov = *reinterpret_cast<const f32x4_t*>(o + row + 4 * hf + 8 * c);
#pragma unroll
    for (int e = 0; e < 4; ++e) part += of[c][e] * ov[e];
  }
  const float del = half_sum(part);
  if (wave == 0 && hf == 0) delta[((size_t)b * H + hh) * S + q] = del;
  f32x16_t dq[D / 32];
#pragma unroll
  for (int t = 0; t < D / 32; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) dq[t][r] = 0.0f;
  for (int t = wave; t <= qt; t += 4) {
    f32x4_t f[D / 8];
    f32x16_t p, dp;
    rows_f32<D>(Kp + (size_t)(t * 32 + l32) * rs + 4 * hf, f);
    dot_f32<D>(f, qf, p);
    rows_f32<D>(Vp + (size_t)(t * 32 + l32) * rs + 4 * hf, f);
    dot_f32<D>(f, of, dp);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const bool masked = t * 32 + (r >> 2) * 8 + hf * 4 + (r & 3) > q;
      p[r] = masked ? 0.0f : expf(p[r] * scale - L) * (dp[r] - del);
    }
    accumulate_f32<D>(Kp + (size_t)(t * 32 + hf * 4) * rs + l32, rs, p, dq);
  }
  float* qo = dqkv + ((size_t)b * S + q) * rs + (size_t)hh * D;
  if (!merge_f32<D>(smem, dq, scale, qo, wave, lane)) return;
  const int col = wave * 8 + hf * 4;
  f32x4_t acc[D / 32] = {};
  float ds = 0.0f;
  for (int j = 0; j <= q && ds == ds; ++j) {
    const float s = row_dot_f32<D>(base + (size_t)q * rs, Kp + (size_t)j * rs);
    ds = expf(s * scale - L) * (row_dot_f32<D>(dout + row, Vp + (size_t)j * rs) - del);
    add_f32<D>(acc, 1.0f, ds, Kp + (size_t)j * rs + col);
  }
  replace_f32<D>(qo + col, acc, scale);
}

template <int D>
__global__ void __launch_bounds__(256) attn_bwd_dkdv_f32(int S, int H, int Bm, int mstride,
                                                         const float* __restrict__ qkv,
                                                         const float* __restrict__ dout,
                                                         const float* __restrict__ lse,
                                                         const float* __restrict__ delta, float* __restrict__ dqkv,
                                                         float scale) {
  extern __shared__ __align__(16) char smem[];
  const int b = seq_index(blockIdx.x / H, Bm, mstride), hh = blockIdx.x % H;
  const int kt = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, hf = lane >> 5;
  const int key = kt * 32 + l32;
  const size_t rs = (size_t)3 * H * D, ors = (size_t)H * D;
  const float* base = qkv + (size_t)b * S * rs + (size_t)hh * D;
  const float* dop = dout + (size_t)b * S * ors + (size_t)hh * D;
  const float* lp = lse + ((size_t)b * H + hh) * S;
  const float* dlp = delta + ((size_t)b * H + hh) * S;
  f32x4_t kf[D / 8], vf[D / 8];
  rows_f32<D>(base + (size_t)key * rs + (size_t)H * D + 4 * hf, kf);
  rows_f32<D>(base + (size_t)key * rs + (size_t)2 * H * D + 4 * hf, vf);
  f32x16_t dk[D / 32], dv[D / 32];
#pragma unroll
  for (int t = 0; t < D / 32; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) dk[t][r] = dv[t][r] = 0.0f;
  for (int t = kt + wave; t < S / 32; t += 4) {
    f32x4_t f[D / 8];
    f32x16_t p, dp;
    rows_f32<D>(base + (size_t)(t * 32 + l32) * rs + 4 * hf, f);
    dot_f32<D>(f, kf, p);  // p[r]: query 32 t + (r/4)*8 + 4*hf + r%4, key `key`
    rows_f32<D>(dop + (size_t)(t * 32 + l32) * ors + 4 * hf, f);
    dot_f32<D>(f, vf, dp);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int q = t * 32 + (r >> 2) * 8 + hf * 4 + (r & 3);
      p[r] = q < key ? 0.0f : expf(p[r] * scale - lp[q]);
      dp[r] = p[r] * (dp[r] - dlp[q]);
    }
    accumulate_f32<D>(dop + (size_t)(t * 32 + hf * 4) * ors + l32, ors, p, dv);
    accumulate_f32<D>(base + (size_t)(t * 32 + hf * 4) * rs + l32, rs, dp, dk);
  }
  float* ko = dqkv + ((size_t)b * S + key) * rs + (size_t)H * D + (size_t)hh * D;
  float* vo = ko + (size_t)H * D;
  const bool odd_k = merge_f32<D>(smem, dk, scale, ko, wave, lane);
  const bool odd_v = merge_f32<D>(smem, dv, 1.0f, vo, wave, lane);
  if (!odd_k && !odd_v) return;
  const int col = wave * 8 + hf * 4;
  const float* kr = base + (size_t)key * rs + (size_t)H * D;
  f32x4_t ak[D / 32] = {}, av[D / 32] = {};
  float p = 0.0f;
  for (int i = key; i < S && p == p; ++i) {
    const float *qr = base + (size_t)i * rs, *dor = dop + (size_t)i * ors;
    p = expf(row_dot_f32<D>(qr, kr) * scale - lp[i]);
    add_f32<D>(av, 1.0f, p, dor + col);
    add_f32<D>(ak, 1.0f, p * (row_dot_f32<D>(dor, kr + (size_t)H * D) - dlp[i]), qr + col);
  }
  replace_f32<D>(ko + col, ak, scale);
  replace_f32<D>(vo + col, av, 1.0f);
}

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------
// Explicit instantiations of the bf16 kernels (the host pass then always emits
// their launch stubs).
#define MERAK_ATTN_INST(D)                                                                                        \
  template __global__ void attn_fwd_bf16<D>(int, int, int, int, const bf16_t* __restrict__, bf16_t* __restrict__, \
                                            float* __restrict__, float, int, AttnOrder);                         \
  template __global__ void attn_bwd_dkdv_bf16<D>(int, int, int, int, const bf16_t* __restrict__,                 \
                                                 const bf16_t* __restrict__, const float* __restrict__,          \
                                                 const float* __restrict__, bf16_t* __restrict__, float, float,  \
                                                 int, AttnOrder);                                                \
  template __global__ void attn_bwd_dq_bf16<D>(int, int, int, int, const bf16_t* __restrict__,                   \
                                               const bf16_t* __restrict__, const bf16_t* __restrict__,           \
                                               const float* __restrict__, float* __restrict__,                   \
                                               bf16_t* __restrict__, float, float, int, AttnOrder);
MERAK_ATTN_INST(64)
MERAK_ATTN_INST(96)
#undef MERAK_ATTN_INST

// Allow a kernel's dynamic LDS beyond the default limit on the current device.
template <typename K>
static hipError_t allow_lds(K kern, size_t bytes, std::atomic<uint64_t>& done) {
  return allow_dynamic_lds(reinterpret_cast<const void*>(kern), bytes, done);
}

// Streamed rows of a (sequence, head) pair: 4 D bytes per token.  A chunk's
// rows are kept to half of an XCD's 4 MB L2: without chunks, 100 pairs of 2048
// rows at d = 96 (0.8 MB each) took 136 us forward, 171 for dQ and 215 for dK and dV
// instead of 132, 164 and 206 (at d = 64, 0.5 MB each, 84, 100 and 141 instead of
// 91, 102 and 137).  Up to
// 512 workgroups (two per CU) are resident together, the second half of them
// beside the first in dispatch order, so there the second half runs shortest
// first (4 x 8 pairs of 1024 rows: 17.0 -> 16.5 us); larger grids run longest
// first throughout, which leaves the short blocks for the end.
static AttnOrder attn_order(int n_pairs, int S, int D) {
  AttnOrder o;
  o.n_blk = S / 64;
  o.chunk = (int)std::max<long long>(1, (2LL << 20) / ((long long)S * D * 4));
  o.fold = (long long)n_pairs * o.n_blk <= 512;
  return o;
}

template <int D>
static hipError_t fwd_bf16(int B, int S, int H, int G, int mstride, const void* qkv, void* o, float* lse,
                           hipStream_t st) {
  if constexpr (D == 128) {
    return launch_attention_fwd_d128(B, S, H, G, mstride, qkv, o, lse, st);
  } else {
    constexpr size_t lds = fwd_lds_bytes<D>();
    static std::atomic<uint64_t> ok{0};
    hipError_t e = allow_lds(attn_fwd_bf16<D>, lds, ok);
    if (e != hipSuccess) return e;
    const int n_pairs = H * G * B;
    hipLaunchKernelGGL((attn_fwd_bf16<D>), dim3((unsigned)n_pairs * (S / 64)), dim3(256), lds, st, S, H, B, mstride,
                       (const bf16_t*)qkv, (bf16_t*)o, lse, 1.0f / sqrtf((float)D) * kLog2e, n_pairs,
                       attn_order(n_pairs, S, D));
    return hipGetLastError();
  }
}

template <int D>
static hipError_t fwd_d(int dtype, int B, int S, int H, int G, int mstride, const void* qkv, void* o, float* lse,
                        hipStream_t st) {
  if (dtype == DT_BF16) return fwd_bf16<D>(B, S, H, G, mstride, qkv, o, lse, st);
  constexpr size_t lds = f32_lds_bytes<D>();
  static std::atomic<uint64_t> ok{0};
  hipError_t e = allow_lds(attn_fwd_f32<D>, lds, ok);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((attn_fwd_f32<D>), dim3((unsigned)(H * G * B), S / 32), dim3(256), lds, st, S, H, B, mstride,
                     (const float*)qkv, (float*)o, lse, 1.0f / sqrtf((float)D));
  return hipGetLastError();
}

template <int D>
static hipError_t bwd_bf16(int B, int S, int H, int G, int mstride, const void* qkv, const void* o, const float* lse,
                           const void* dout, void* dqkv, float* delta, hipStream_t st) {
  if constexpr (D == 128) {
    return launch_attention_bwd_d128(B, S, H, G, mstride, qkv, o, lse, dout, dqkv, delta, st);
  } else {
    const float scale = 1.0f / sqrtf((float)D);
    constexpr size_t lds_q = fwd_lds_bytes<D>(), lds_k = bwd_lds_bytes<D>();
    static_assert(lds_k <= 160 * 1024, "LDS budget");
    static std::atomic<uint64_t> ok_k{0}, ok_q{0};
    hipError_t e = allow_lds(attn_bwd_dkdv_bf16<D>, lds_k, ok_k);
    if (e == hipSuccess) e = allow_lds(attn_bwd_dq_bf16<D>, lds_q, ok_q);
    if (e != hipSuccess) return e;
    // dQ first: it also forms delta, which dK/dV reads.
    const int n_pairs = H * G * B;
    const dim3 grid((unsigned)n_pairs * (S / 64));
    const AttnOrder ord = attn_order(n_pairs, S, D);
    hipLaunchKernelGGL((attn_bwd_dq_bf16<D>), grid, dim3(256), lds_q, st, S, H, B, mstride, (const bf16_t*)qkv,
                       (const bf16_t*)o, (const bf16_t*)dout, lse, delta, (bf16_t*)dqkv, scale * kLog2e, scale,
                       n_pairs, ord);
    hipLaunchKernelGGL((attn_bwd_dkdv_bf16<D>), grid, dim3(256), lds_k, st, S, H, B, mstride, (const bf16_t*)qkv,
                       (const bf16_t*)dout, lse, delta, (bf16_t*)dqkv, scale * kLog2e, scale, n_pairs, ord);
    return hipGetLastError();
  }
}

template <int D>
static hipError_t bwd_d(int dtype, int B, int S, int H, int G, int mstride, const void* qkv, const void* o,
                        const float* lse, const void* dout, void* dqkv, float* delta, hipStream_t st) {
  if (dtype == DT_BF16) return bwd_bf16<D>(B, S, H, G, mstride, qkv, o, lse, dout, dqkv, delta, st);
  const float scale = 1.0f / sqrtf((float)D);
  constexpr size_t lds = f32_lds_bytes<D>();
  static std::atomic<uint64_t> ok_k{0}, ok_q{0};
  hipError_t e = allow_lds(attn_bwd_dkdv_f32<D>, lds, ok_k);
  if (e == hipSuccess) e = allow_lds(attn_bwd_dq_f32<D>, lds, ok_q);
  if (e != hipSuccess) return e;
  const dim3 grid((unsigned)(H * G * B), S / 32);
  hipLaunchKernelGGL((attn_bwd_dq_f32<D>), grid, dim3(256), lds, st, S, H, B, mstride, (const float*)qkv,
                     (const float*)o, (const float*)dout, lse, delta, (float*)dqkv, scale);
  hipLaunchKernelGGL((attn_bwd_dkdv_f32<D>), grid, dim3(256), lds, st, S, H, B, mstride, (const float*)qkv,
                     (const float*)dout, lse, delta, (float*)dqkv, scale);
  return hipGetLastError();
}

hipError_t launch_attention_fwd(int dtype, int batch, int seq, int heads, int d, const void* qkv, void* o,
                                float* lse, hipStream_t stream, int members, int member_stride) {
  if (batch <= 0 || seq <= 0 || heads <= 0 || members <= 0) return hipSuccess;
  if (seq % 64 != 0 || (members > 1 && member_stride < batch)) return hipErrorInvalidValue;
  switch (d) {
    case 64: return fwd_d<64>(dtype, batch, seq, heads, members, member_stride, qkv, o, lse, stream);
    case 96: return fwd_d<96>(dtype, batch, seq, heads, members, member_stride, qkv, o, lse, stream);
    case 128: return fwd_d<128>(dtype, batch, seq, heads, members, member_stride, qkv, o, lse, stream);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_attention_bwd(int dtype, int batch, int seq, int heads, int d, const void* qkv, const void* o,
                                const float* lse, const void* dout, void* dqkv, float* delta, hipStream_t stream,
                                int members, int member_stride) {
  if (batch <= 0 || seq <= 0 || heads <= 0 || members <= 0) return hipSuccess;
  if (seq % 64 != 0 || (members > 1 && member_stride < batch)) return hipErrorInvalidValue;
  switch (d) {
    case 64: return bwd_d<64>(dtype, batch, seq, heads, members, member_stride, qkv, o, lse, dout, dqkv, delta, stream);
    case 96: return bwd_d<96>(dtype, batch, seq, heads, members, member_stride, qkv, o, lse, dout, dqkv, delta, stream);
    case 128:
      return bwd_d<128>(dtype, batch, seq, heads, members, member_stride, qkv, o, lse, dout, dqkv, delta, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace merak
