// Helpers shared by the attention kernels (attention.hip, attention_d128.hip).
#pragma once

#include "common.h"
#include "kernels.h"

namespace merak {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x8_t __attribute__((ext_vector_type(8)));
#define MERAK_LDS __attribute__((address_space(3)))

// Eight accumulator values narrowed to an MFMA operand, four packed
// conversion instructions.
__device__ __forceinline__ bf16x8_t cvt8(const f32x16_t& a, int base) {
  typedef float f32x8_t __attribute__((ext_vector_type(8)));
  f32x8_t v;
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = a[base + e];
  return __builtin_convertvector(v, bf16x8_t);
}

__device__ __forceinline__ bf16x8_t frag_kc(const bf16_t* p) { return *reinterpret_cast<const bf16x8_t*>(p); }

// Sequence index of launch batch z when a launch covers several members (for
// example the sub-micro-batches that share a stream), each of Bm consecutive
// sequences, members mstride sequences apart.  Every tensor is addressed by
// sequence (rows b * S + i, lse and delta rows (b * H + h) * S + i), so the
// kernels need nothing else to work on such a group.
__device__ __forceinline__ int seq_index(int z, int Bm, int mstride) { return (z / Bm) * mstride + z % Bm; }

}  // namespace merak
