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

__device__ __forceinline__ float bload4(Rsrc r, uint32_t off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}

// Chunk position of the 16-byte chunk c (8 k) of row r, for rows of 32, 64
// or 128 k (64, 128 or 256 bytes): c ^ split_swz(r), so that neither the
// rows that one MFMA operand read touches nor neighbouring rows' writes
// share a bank.
template <int BK>
__device__ __forceinline__ int split_swz(int r) {
  return BK == 32 ? (((r >> 1) ^ (r >> 3)) & 3) : BK == 64 ? (r & 7) : (r & 15);
}

}  // namespace fluid
