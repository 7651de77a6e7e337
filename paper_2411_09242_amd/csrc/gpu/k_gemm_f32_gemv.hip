// fp32 products of at most four rows with a K-contiguous weight (the fully
// connected layers of a network run on one image): tile 6 for those
// operands where K is long enough (the rule and both sides' times: row_product
// in dispatch.cpp).  Such a product reads its weight once and is bound by that; the
// 16 x 32 tile kernel has N / 32 workgroups, too few loads in flight, and
// multiplies twelve or more rows of padding.  Here a workgroup of four
// wavefronts takes four columns: its threads read 4 KiB runs of each
// column's K values, sixteen bytes a lane, with the rows of A from the
// caches, and the lanes' sums are added across the wavefront and through LDS
// in wavefront order.  Everything is fp32; a lane's chain is K / 256 long.
// The three dense layers of the VGG-16-shaped network (25088, 4096, 4096 x
// 4096, 4096, 1000) with it: 975 -> 906 us for the network, where they took
// 114, 22 and 20 us (3.6, 3.0 and 0.8 TB/s).
#include <type_traits>

#include "gemm_common.h"
#include "launch.h"

namespace fluid {

// Columns 4 bid .. 4 bid + 3 of the product p.
template <int MR, bool RES>
__device__ __forceinline__ void gemv_f32_cols(const GemmParams& p, uint32_t bid) {
  constexpr int NC = 4, U = MR == 1 ? 4 : 2;
  __shared__ float part[4][NC * MR];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t n0 = bid * NC;
  const float* A = (const float*)p.A;
  const float* B = (const float*)p.B;
  // rows past M and columns past N are clamped onto the first: never stored
  const float *a[MR], *b[NC];
#pragma unroll
  for (int m = 0; m < MR; ++m) a[m] = A + ((uint32_t)m < p.M ? row_off(p, m, p.a_m1, p.a_m2) : 0);
#pragma unroll
  for (int c = 0; c < NC; ++c) b[c] = B + (int64_t)(n0 + c < p.N ? n0 + c : n0) * p.b_n;
  float acc[NC][MR];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int m = 0; m < MR; ++m) acc[c][m] = 0.f;
  auto run = [&](auto UC, uint32_t k) {
    constexpr int UN = decltype(UC)::value;
    float4 w[UN][NC], x[UN][MR];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
#pragma unroll
      for (int c = 0; c < NC; ++c) w[u][c] = *(const float4*)(b[c] + k + 1024 * u);
#pragma unroll
      for (int m = 0; m < MR; ++m) x[u][m] = *(const float4*)(a[m] + k + 1024 * u);
    }
#pragma unroll
    for (int u = 0; u < UN; ++u)
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int m = 0; m < MR; ++m) {
          float s = acc[c][m];
          s = fmaf(x[u][m].x, w[u][c].x, s);
          s = fmaf(x[u][m].y, w[u][c].y, s);
          s = fmaf(x[u][m].z, w[u][c].z, s);
          acc[c][m] = fmaf(x[u][m].w, w[u][c].w, s);
        }
  };
  // K is a multiple of 4 (K-contiguous operands move in 16-byte pieces)
  uint32_t k = 4u * tid;
  for (; k + 1024u * (U - 1) < p.K; k += 1024u * U) run(std::integral_constant<int, U>(), k);
  for (; k < p.K; k += 1024u) run(std::integral_constant<int, 1>(), k);
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int m = 0; m < MR; ++m) {
      const float s = wave_sum(acc[c][m]);
      if (lane == 0) part[wave][c * MR + m] = s;
    }
  __syncthreads();
  if (tid < NC * MR) {
    const uint32_t n = n0 + tid / MR, m = tid % MR;
    if (n < p.N && m < p.M) {
      const float s = part[0][tid] + part[1][tid] + part[2][tid] + part[3][tid];
      ((float*)p.C)[row_off(p, m, p.c_m1, p.c_m2) + (int32_t)n * p.c_n] = gemm_epi<RES>(p, 0, m, n, s);
    }
  }
}

template <int MR, bool RES>
__global__ __launch_bounds__(256) void gemv_f32_kernel(GemmParams p) {
  gemv_f32_cols<MR, RES>(p, blockIdx.x);
}

// The members of a group share the rows and the epilogue instance; each
// workgroup runs four columns of its member.
template <int MR, bool RES>
__global__ __launch_bounds__(256) void gemv_f32_group_kernel(GemmGroup G) {
  uint32_t i = 0;
  while (i + 1 < G.n && blockIdx.x >= G.tiles[i + 1]) ++i;
  gemv_f32_cols<MR, RES>(G.p[i], blockIdx.x - G.tiles[i]);
}

hipError_t launch_gemv_f32(const NodeKernel& k, hipStream_t s) {
  const GemmParams& p = k.gemm;
  if (p.M > 4 || p.G != 1) return hipErrorInvalidValue;
  const dim3 grid(p.tiles_n);
#define FLUID_GEMV(MRv)                                                                        \
  do {                                                                                         \
    if (p.rop) hipLaunchKernelGGL((gemv_f32_kernel<MRv, true>), grid, dim3(256), 0, s, p);     \
    else hipLaunchKernelGGL((gemv_f32_kernel<MRv, false>), grid, dim3(256), 0, s, p);          \
  } while (0)
  if (p.M == 1) FLUID_GEMV(1);
  else if (p.M == 2) FLUID_GEMV(2);
  else FLUID_GEMV(4);
#undef FLUID_GEMV
  return hipGetLastError();
}

hipError_t launch_gemv_f32_group(const NodeKernel& k, const GemmGroup& G, hipStream_t s) {
  if (!k.gemm_row || G.n < 1 || G.n > (uint32_t)kMaxGroup) return hipErrorInvalidValue;
  for (uint32_t i = 0; i < G.n; ++i)
    if (G.p[i].M != k.gemm.M || G.p[i].G != 1) return hipErrorInvalidValue;
  const dim3 grid(G.tiles[G.n]);
#define FLUID_GEMVG(MRv)                                                                              \
  do {                                                                                                \
    if (k.gemm.rop) hipLaunchKernelGGL((gemv_f32_group_kernel<MRv, true>), grid, dim3(256), 0, s, G); \
    else hipLaunchKernelGGL((gemv_f32_group_kernel<MRv, false>), grid, dim3(256), 0, s, G);           \
  } while (0)
  if (k.gemm.M == 1) FLUID_GEMVG(1);
  else if (k.gemm.M == 2) FLUID_GEMVG(2);
  else FLUID_GEMVG(4);
#undef FLUID_GEMVG
  return hipGetLastError();
}

}  // namespace fluid
