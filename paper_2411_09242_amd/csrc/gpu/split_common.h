// fp32 values as three bf16 ones, for products on the bf16 matrix cores
// (the method and its exceptions: k_gemm_f32_split.hip).
#pragma once

#include "gemm_common.h"

namespace fluid {

// Both operands are multiplied by 2^24 before they are split, and the sums
// by 2^-48: the lowest bit of any fp32 value, 2^-149, becomes 2^-125, so that
// every part of every value is a normal bf16 number (without the scale an
// operand of 1e-36 keeps 16 bits, one of 1e-40 two).
constexpr float kSplitScale = 0x1p24f, kSplitUnscale = 0x1p-48f;

// The three bf16 parts of the scaled pair (a, b): plane 0 the leading parts.
__device__ __forceinline__ void split2(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l) {
  a *= kSplitScale;
  b *= kSplitScale;
  h = pack_bf16(a, b);
  a -= __uint_as_float(h << 16);
  b -= __uint_as_float(h & 0xffff0000u);
  m = pack_bf16(a, b);
  a -= __uint_as_float(m << 16);
  b -= __uint_as_float(m & 0xffff0000u);
  l = pack_bf16(a, b);
}

// Eight consecutive k of one row to the three planes (16 bytes each).
__device__ __forceinline__ void split_put(const float* v, uint8_t* dst, int plane) {
  uint32_t h[4], m[4], l[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) split2(v[2 * i], v[2 * i + 1], h[i], m[i], l[i]);
  *(uint4*)dst = make_uint4(h[0], h[1], h[2], h[3]);
  *(uint4*)(dst + plane) = make_uint4(m[0], m[1], m[2], m[3]);
  *(uint4*)(dst + 2 * plane) = make_uint4(l[0], l[1], l[2], l[3]);
}

// The six products of 16 k of FI x FJ blocks (planes of A and B).  acc: the
// leading products h h'; low: the five others, 2^-8 smaller, so that they
// cost the large sums no roundings.
template <int FI, int FJ>
__device__ __forceinline__ void split_mul(const bf16x8 (&a)[3][FI], const bf16x8 (&b)[3][FJ], f32x16 (&acc)[FI][FJ],
                                          f32x16 (&low)[FI][FJ]) {
  constexpr int PA[5] = {0, 1, 1, 0, 2}, PB[5] = {1, 0, 1, 2, 0};
#pragma unroll
  for (int t = 4; t >= 0; --t)
#pragma unroll
    for (int i = 0; i < FI; ++i)
#pragma unroll
      for (int j = 0; j < FJ; ++j)
        low[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[PA[t]][i], b[PB[t]][j], low[i][j], 0, 0, 0);
#pragma unroll
  for (int i = 0; i < FI; ++i)
#pragma unroll
    for (int j = 0; j < FJ; ++j)
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0][i], b[0][j], acc[i][j], 0, 0, 0);
}

__device__ __forceinline__ float bload4(Rsrc r, uint32_t off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}

// Chunk position of the 16-byte chunk c (8 k) of row r, for rows of 32, 64
// or 128 k (64, 128 or 256 bytes): c ^ split_swz(r), so that the rows that
// one MFMA operand read touches, and neighbouring rows' writes, spread over
// the banks (conflicts: none for rows of 128 k, 29% of the LDS cycles for 64,
// a third for 32).
template <int BK>
__device__ __forceinline__ int split_swz(int r) {
  return BK == 32 ? (((r >> 1) ^ (r >> 3)) & 3) : BK == 64 ? (r & 7) : (r & 15);
}

}  // namespace fluid
