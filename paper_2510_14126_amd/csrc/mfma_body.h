// Types, packing and the 16x16 K stage layout of the matrix-core kernels
// (gfx950).
#pragma once

#include "kernels.h"
#include "pa_device.h"

namespace pa {
namespace mfma {

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef float floatx2_t __attribute__((ext_vector_type(2)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));
typedef float floatx16_t __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) floatx2_t lds_floatx2_t;
typedef __attribute__((address_space(3))) floatx4_t lds_floatx4_t;
typedef __attribute__((address_space(3))) short4_t lds_short4_t;
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) u32x4_t lds_u32x4_t;

constexpr int kWaves = 4;                     // wavefronts per workgroup
constexpr int kKPitch = 256;                  // LDS bytes per staged K token row (head_dim 128)
// Log2 units by which a score must exceed the running max before the
// accumulators are rescaled: probabilities stay <= 2^8.
constexpr float kLazyRescale = 8.0f;

// Two fp32 values rounded to nearest even as a packed bf16 pair.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  const floatx2_t x = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2_t));
}

// Value of query column 4q+r (held by lane 4q+r) for the accumulator rows
// of lane group q.
__device__ __forceinline__ float column_value(float x, int q, int r) {
  const int xi = __builtin_bit_cast(int, x);
  const float c0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, r));
  const float c1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, 4 + r));
  const float c2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, 8 + r));
  const float c3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, 12 + r));
  return q == 0 ? c0 : (q == 1 ? c1 : (q == 2 ? c2 : c3));
}

// Row of the K tile that lane (q, n) supplies as A row n: token 4(n%4) + n/4.
__device__ __forceinline__ int k_arow(int n) { return 4 * (n & 3) + (n >> 2); }

// LDS byte offset of 16-byte chunk c of token row r in a staged K tile:
// rows of 256 bytes, chunk c at position c ^ k_arow(r).  Writers (16 lanes
// per row, chunks 0..15) and A-operand readers (lane (q, n): row k_arow(n),
// chunk 4s+q, i.e. position (4s+q) ^ n since k_arow is its own inverse) then
// touch 16 distinct positions per instruction, with no padding.
__device__ __forceinline__ int k_stage(int r, int c) { return r * kKPitch + ((c ^ k_arow(r)) << 4); }

}  // namespace mfma
}  // namespace pa
