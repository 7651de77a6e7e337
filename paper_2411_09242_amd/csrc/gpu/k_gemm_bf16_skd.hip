// bf16 GEMM for few output tiles (a decoder's projections of a short prompt),
// both operands K-contiguous: the kernel behind tiles 2, 3 and 4 for those
// operands.  Such a product is bound by its loads in flight: with loads into
// registers (gemm_sk_kernel, which keeps the other operand layouts) a 333 x
// 1024 x 1024 product reads its 45 MB of L2 traffic at 4 TB/s.  Here, as in
// the fp32 tiles 6 and 7:
//
//  * a workgroup owns a (32 FM) x 32 tile, its W wavefronts a slice of K each;
//    the partial tiles are summed through LDS in wavefront order;
//    FM 1 over 4 (tile 2) or 8 wavefronts (tile 3), FM 2 over 4 (tile 4);
//  * operands go to LDS by DMA, 64 k (a whole 128-byte line of a row) at a
//    time, each wavefront into NS stages of its own, without a barrier in the
//    loop; nothing is loaded past the slice.
//
// Measured (M x K x N, tiles 2 / 3 / 4, weights from HBM, us; before: loads
// into registers): 16 x 1024 x 1024 7.6 / 6.2 / 8.8 -> 4.8 / 4.8 / 5.7, 333 x
// 1024 x 1024 10.9 / 12.3 / 10.6 -> 6.2 / 6.5 / 6.6, 333 x 1024 x 2816 20.3 /
// 23.2 / 19.4 -> 10.6 / 10.9 / 15.2, 333 x 2816 x 1024 23.7 / 25.6 / 19.8 ->
// 9.5 / 11.7 / 9.2, 700 x 2048 x 5464 127 / 152 / 111 -> 72 / 73 / 66.  At
// 333 rows the DMA of both operands' rows by every tile that needs them is
// what bounds it.  Two stages over 4 wavefronts and one over 8, so that two
// workgroups share a CU: with one stage more 8.1 / 8.1 us at 333 x 1024 x 1024.
//
// LDS, per 64-k group: rows of 128 bytes, chunk c (8 k) of row r at c ^ (r %
// 8), so that the rows of one MFMA operand read touch every bank.
// MFMA 32x32x16 bf16: lane l holds row l % 32, k 8 (l / 32) .. + 7 of A and B.
#include "gemm_common.h"
#include "launch.h"

namespace fluid {

namespace {

typedef __attribute__((address_space(3))) void lds_void;

}  // namespace

template <int W, int FM, int NS, bool RES>
__global__ __launch_bounds__(64 * W) void gemm_bf16_skd_kernel(GemmParams p) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass does not know the DMA's 16 bytes
  constexpr int TM = 32 * FM, TN = 32, RP = TN + 1;
  constexpr int WB = 4096 * (FM + 1);  // a wavefront's 64-k group: A, then B
  constexpr int ND = 4 * (FM + 1);     // DMA instructions per group
  static_assert(NS * W * WB <= 160 * 1024 && NS * WB >= 4 * TM * RP && (NS - 1) * ND < 64, "LDS, vmcnt");
  __shared__ __attribute__((aligned(1024))) uint8_t lds[W][NS][WB];
  const TileCoord tc = tile_coord(p, TM, TN);
  // causal attention: a tile entirely above the diagonal is never read; a
  // row block's A is zero past its last row, so K stops there
  if ((p.causal & 1u) && tc.n0 > tc.m0 + TM - 1) return;
  const uint32_t Kc = (p.causal & 2u) ? min(p.K, tc.m0 + TM) : p.K;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, lh = lane >> 5;
  const Rsrc ra = make_rsrc(p.A, p.a_bytes);
  const Rsrc rb = make_rsrc(p.B, p.b_bytes);
  // this wavefront's K slice [kbeg, kend), a multiple of 16 long
  const uint32_t kw = ((Kc + 16u * W - 1u) / (16u * W)) * 16u;
  const uint32_t kbeg = wave * kw;
  const uint32_t kend = min(Kc, kbeg + kw);
  const uint32_t ng = kend > kbeg ? (kend - kbeg + 63u) / 64u : 0u;

  // DMA sources: byte offset of the lane's piece at k = kbeg and the k it
  // starts at.  Rows past M and columns past N only feed outputs that are
  // never stored: they are clamped onto row / column 0.  k outside the slice
  // reads as zero (kOOB); Kc and the slices are multiples of the piece's 8 k.
  const uint32_t pk = kbeg + 8u * ((lane & 7) ^ (lane >> 3));
  uint32_t a_src[4 * FM], b_src[4];
#pragma unroll
  for (int i = 0; i < 4 * FM; ++i) {
    const uint32_t m = tc.m0 + 8 * i + (lane >> 3);
    a_src[i] = 2u * (uint32_t)(tc.a_base + (m < p.M ? row_off(p, m, p.a_m1, p.a_m2) : 0) + (int32_t)pk);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t n = tc.n0 + 8 * j + (lane >> 3);
    b_src[j] = 2u * (uint32_t)(tc.b_base + (int32_t)(n < p.N ? n : 0) * p.b_n + (int32_t)pk);
  }
  auto load = [&](uint32_t st, uint32_t g) {
    uint8_t* dst = lds[wave][st];
    const bool in = pk + 64u * g < kend;
#pragma unroll
    for (int i = 0; i < 4 * FM; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void*)(dst + 1024 * i), 16, in ? a_src[i] + 128u * g : kOOB, 0, 0, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_void*)(dst + 4096 * FM + 1024 * j), 16,
                                               in ? b_src[j] + 128u * g : kOOB, 0, 0, 0);
  };

  f32x16 acc[FM];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
  // A group's operands by 16-k step.  The LDS reads and their wait are one
  // asm block: the compiler would put a wait for every DMA in flight before
  // a read that it can see.
  const uint32_t rd = (uint32_t)(uintptr_t)(lds_void*)lds[wave][0] + 128 * lr + ((lh ^ (lr & 7)) << 4);
  auto compute = [&](uint32_t st) {
    const uint32_t p0 = rd + st * WB, p1 = p0 ^ 32u, p2 = p0 ^ 64u, p3 = p0 ^ 96u;
    bf16x8 a[FM][4], b[4];
    if constexpr (FM == 1)
      asm volatile(
          "ds_read_b128 %0, %8\nds_read_b128 %4, %8 offset:4096\nds_read_b128 %1, %9\nds_read_b128 %5, %9 offset:4096\n"
          "ds_read_b128 %2, %10\nds_read_b128 %6, %10 offset:4096\nds_read_b128 %3, %11\n"
          "ds_read_b128 %7, %11 offset:4096\ns_waitcnt lgkmcnt(0)"
          : "=&v"(a[0][0]), "=&v"(a[0][1]), "=&v"(a[0][2]), "=&v"(a[0][3]), "=&v"(b[0]), "=&v"(b[1]), "=&v"(b[2]),
            "=&v"(b[3])
          : "v"(p0), "v"(p1), "v"(p2), "v"(p3)
          : "memory");
    else
      asm volatile(
          "ds_read_b128 %0, %12\nds_read_b128 %4, %12 offset:4096\nds_read_b128 %8, %12 offset:8192\n"
          "ds_read_b128 %1, %13\nds_read_b128 %5, %13 offset:4096\nds_read_b128 %9, %13 offset:8192\n"
          "ds_read_b128 %2, %14\nds_read_b128 %6, %14 offset:4096\nds_read_b128 %10, %14 offset:8192\n"
          "ds_read_b128 %3, %15\nds_read_b128 %7, %15 offset:4096\nds_read_b128 %11, %15 offset:8192\n"
          "s_waitcnt lgkmcnt(0)"
          : "=&v"(a[0][0]), "=&v"(a[0][1]), "=&v"(a[0][2]), "=&v"(a[0][3]), "=&v"(a[FM - 1][0]), "=&v"(a[FM - 1][1]),
            "=&v"(a[FM - 1][2]), "=&v"(a[FM - 1][3]), "=&v"(b[0]), "=&v"(b[1]), "=&v"(b[2]), "=&v"(b[3])
          : "v"(p0), "v"(p1), "v"(p2), "v"(p3)
          : "memory");
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < FM; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][s], b[s], acc[i], 0, 0, 0);
  };
  // waits until at most the `rest` newest groups are in flight
  auto arrived = [&](uint32_t rest) {
    asm volatile("" ::: "memory");
    switch (min(rest, (uint32_t)NS - 1)) {
      case 0: __builtin_amdgcn_s_waitcnt(vmcnt_imm(0)); break;
      case 1: __builtin_amdgcn_s_waitcnt(vmcnt_imm(ND)); break;
      default: __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * ND)); break;
    }
    asm volatile("" ::: "memory");
  };
  static_assert(NS <= 3, "arrived");

  // group g travels through stage g % NS, NS groups in flight; no other
  // wavefront touches the stage, so the loop has no barrier
  const uint32_t first = min(ng, (uint32_t)NS);
  for (uint32_t g = 0; g < first; ++g) load(g, g);
  uint32_t g = 0, st = 0;
  for (; g + NS < ng; ++g) {
    arrived(NS - 1);
    compute(st);
    load(st, g + NS);  // the reads of the stage are done: compute waited for them
    st = st + 1 == NS ? 0 : st + 1;
  }
  for (; g < ng; ++g) {
    arrived(ng - 1 - g);
    compute(st);
    st = st + 1 == NS ? 0 : st + 1;
  }

  float* red = (float*)lds;
  __syncthreads();  // every wavefront is past its last read of its stages
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v)
      red[(wave * TM + 32 * i + 8 * (v / 4) + 4 * lh + (v % 4)) * RP + lr] = acc[i][v];
  __syncthreads();
  uint16_t* C = (uint16_t*)p.C;
  auto value = [&](int ml, int nl, uint32_t m, uint32_t n) {
    float sum = 0.f;
#pragma unroll
    for (int q = 0; q < W; ++q) sum += red[(q * TM + ml) * RP + nl];
    return gemm_epi<RES>(p, tc.r_base, m, n, sum);
  };
  if (p.c_n == 1) {
    // a thread writes 4 consecutive columns of one row
    for (int e = tid; e < TM * TN / 4; e += 64 * W) {
      const int ml = e / (TN / 4), nl = 4 * (e % (TN / 4));
      const uint32_t m = tc.m0 + ml, n = tc.n0 + nl;
      if (m >= p.M || n >= p.N) continue;
      uint16_t* c = C + tc.c_base + row_off(p, m, p.c_m1, p.c_m2) + (int32_t)n;
      uint16_t o[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) o[t] = n + t < p.N ? f32_to_bf16(value(ml, nl + t, m, n + t)) : (uint16_t)0;
      if (n + 3 < p.N && ((uintptr_t)c & 7u) == 0) {
        *(uint2*)c = make_uint2(o[0] | ((uint32_t)o[1] << 16), o[2] | ((uint32_t)o[3] << 16));
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (n + t < p.N) c[t] = o[t];
      }
    }
  } else {
    // consecutive threads on consecutive rows
    for (int e = tid; e < TM * TN; e += 64 * W) {
      const int ml = e % TM, nl = e / TM;
      const uint32_t m = tc.m0 + ml, n = tc.n0 + nl;
      if (m >= p.M || n >= p.N) continue;
      C[tc.c_base + row_off(p, m, p.c_m1, p.c_m2) + (int32_t)n * p.c_n] = f32_to_bf16(value(ml, nl, m, n));
    }
  }
#endif
}

hipError_t launch_gemm_bf16_skd(const NodeKernel& k, hipStream_t s) {
  const GemmParams& p = k.gemm;
  const dim3 grid(p.tiles_m * p.tiles_n * p.G);
#define FLUID_SKD(Wv, FMv, NSv)                                                                                   \
  do {                                                                                                            \
    if (p.rop) hipLaunchKernelGGL((gemm_bf16_skd_kernel<Wv, FMv, NSv, true>), grid, dim3(64 * Wv), 0, s, p);      \
    else hipLaunchKernelGGL((gemm_bf16_skd_kernel<Wv, FMv, NSv, false>), grid, dim3(64 * Wv), 0, s, p);           \
  } while (0)
  switch (k.gemm_tile) {
    case 2: FLUID_SKD(4, 1, 2); break;
    case 3: FLUID_SKD(8, 1, 1); break;
    case 4: FLUID_SKD(4, 2, 2); break;
    default: return hipErrorInvalidValue;
  }
#undef FLUID_SKD
  return hipGetLastError();
}

}  // namespace fluid
