// fp32 GEMM for small M (the projections of a short sequence: M = 128 or 512
// tokens), MFMA 16x16x4 f32.  Such a GEMM has too few 32 x 32 output tiles to
// fill 256 compute units, and each tile's K loop is short, so it is bound by
// how many loads are in flight, not by the matrix cores.  Here:
//
//  * a workgroup owns one (16 FM) x 32 output tile and W wavefronts split
//    its K range into W contiguous slices; at the end the W partial tiles
//    are summed through LDS in wavefront order (a fixed order: the result
//    does not depend on timing);
//  * both operands go to LDS by DMA (`buffer_load ... lds`, 16 bytes per
//    lane), each wavefront into stages of its own (no barrier in the loop),
//    three 16-k groups in flight; a K-contiguous operand comes in 64-byte row
//    pieces, half a line.  Nothing is loaded past the slice: it would cost as
//    much issue time as a real load.
//
// Measured (M K N, weights from HBM; before: loads straight into registers):
// 128 x 3072 x 768 15.8 -> 13.3 us, 128 x 768 x 3072 on a K-contiguous weight
// 17.1 -> 14.2, 512 x 3072 x 768 38.4 -> 31.0 (16 x 32); 512 x 768 x 3072
// 33.8 -> 29.4 (32 x 32).  What bounds it: at 128 x 3072 x 768 the DMA alone
// takes 12.5 us and the LDS reads and MFMAs alone 11.6, 1.7 of each the launch
// (113 MB in 10.8 us, 55 GB/s for each of the 192 workgroups).
// Three stages, so that two or three workgroups share a CU, against six:
// 13.3 and 14.3 us there, 36.8 and 56 at 512 x 768 x 3072; sixteen
// wavefronts, a K order rotated by tile row and XCD-contiguous tile columns
// were no faster.
//
// LDS, per 16-k group: a K-contiguous operand as 16 rows of 64 bytes, chunk
// c of row r at c ^ (r / 4); an M- or N-contiguous one as rows of 16 or 32
// values per k, row k in slot 4 (k % 4) + k / 4, so that the four k that
// one MFMA step reads are neighbours: no bank conflicts either way.  A lane
// reads two neighbouring columns of a 32-wide row at once, one for each MFMA
// block, and the epilogue knows block j's column i as 2 i + j.
//
// MFMA 16x16x4 f32 operand layout: lane l holds A[l % 16][k = l / 16] and
// B[k = l / 16][l % 16]; the result lane l holds D[4 (l / 16) + v][l % 16].
// Step s of a 16-k group uses, in the k slot l / 16, the real k
// 4 (l / 16) + s, the same for A and B.
#include <type_traits>

#include "gemm_common.h"
#include "launch.h"

namespace fluid {

namespace {

constexpr int SK_TN = 32;            // output tile columns
constexpr int SK_FN = 2;             // 16 x 16 blocks across a tile
typedef __attribute__((address_space(3))) void lds_void;

}  // namespace

// One workgroup's tile: tile `bid` of the product p.
template <int W, int SK_FM, int NS, int AM, int BMD, bool RES>
__device__ __forceinline__ void gemm_f32_dl_tile(const GemmParams& p, uint32_t bid) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass knows neither the DMA's 16 bytes nor the registers
  constexpr int SK_TM = 16 * SK_FM;
  constexpr int SK_RP = SK_FM == 1 ? SK_TN + 1 : SK_TN;  // reduction row pitch (floats): fits a stage
  constexpr int WB = 1024 * (SK_FM + 2);  // a wavefront's 16-k group: A, then B
  constexpr int ND = SK_FM + 2;           // DMA instructions per group
  static_assert(NS * W * WB <= 160 * 1024 && NS * WB >= 4 * SK_TM * SK_RP, "LDS");
  __shared__ __attribute__((aligned(1024))) uint8_t lds[W][NS][WB];
  const TileCoord tc = tile_coord_at(p, bid, SK_TM, SK_TN);
  // causal attention: a tile entirely above the diagonal is never read; a
  // row block's A is zero past its last row, so K stops there
  if ((p.causal & 1u) && tc.n0 > tc.m0 + SK_TM - 1) return;
  const uint32_t Kc = (p.causal & 2u) ? min(p.K, tc.m0 + SK_TM) : p.K;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lq = lane >> 4;
  const Rsrc ra = make_rsrc(p.A, p.a_bytes);
  const Rsrc rb = make_rsrc(p.B, p.b_bytes);
  // this wavefront's K slice [kbeg, kend), a multiple of 16 long
  const uint32_t kw = ((Kc + 16u * W - 1u) / (16u * W)) * 16u;
  const uint32_t kbeg = wave * kw;
  const uint32_t kend = min(Kc, kbeg + kw);
  const uint32_t ng = kend > kbeg ? (kend - kbeg + 15u) / 16u : 0u;

  // DMA sources: element offset of the lane's piece at k = kbeg and the k it
  // starts at.  Rows past M and columns past N only feed outputs that are
  // never stored: they are clamped onto row / column 0.  k outside the slice
  // reads as zero (kOOB).
  int32_t a_src[SK_FM], b_src[2];
  uint32_t a_k[SK_FM], b_k[2];
#pragma unroll
  for (int i = 0; i < SK_FM; ++i) {
    if constexpr (AM == GM_K) {
      const int row = lane >> 2, c = (lane & 3) ^ ((row >> 2) & 3);
      const uint32_t m = tc.m0 + 16 * i + row;
      a_k[i] = kbeg + 4 * c;
      a_src[i] = tc.a_base + (m < p.M ? row_off(p, m, p.a_m1, p.a_m2) : 0) + (int32_t)a_k[i];
    } else {
      const int L = 4 * SK_FM;  // lanes per row of 16 SK_FM values
      const int slot = (64 / L) * i + lane / L, r = 4 * (slot & 3) + (slot >> 2);
      const uint32_t m = tc.m0 + 4 * (lane % L);
      a_k[i] = kbeg + r;
      a_src[i] = tc.a_base + (m < p.M ? row_off(p, m, p.a_m1, p.a_m2) : 0) + (int32_t)a_k[i] * p.a_k;
    }
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if constexpr (BMD == GM_K) {
      const int row = lane >> 2, c = (lane & 3) ^ ((row >> 2) & 3);
      const uint32_t n = tc.n0 + 16 * j + row;
      b_k[j] = kbeg + 4 * c;
      b_src[j] = tc.b_base + (int32_t)(n < p.N ? n : 0) * p.b_n + (int32_t)b_k[j];
    } else {
      const int slot = 8 * j + (lane >> 3), r = 4 * (slot & 3) + (slot >> 2);
      const uint32_t n = tc.n0 + 4 * (lane & 7);
      b_k[j] = kbeg + r;
      b_src[j] = tc.b_base + (int32_t)(n < p.N ? n : 0) + (int32_t)b_k[j] * p.b_k;
    }
  }
  const int32_t a_step = AM == GM_K ? 16 : 16 * p.a_k, b_step = BMD == GM_K ? 16 : 16 * p.b_k;
  auto load = [&](uint32_t st, uint32_t g) {
    uint8_t* dst = lds[wave][st];

#pragma unroll
    for (int i = 0; i < SK_FM; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void*)(dst + 1024 * i), 16,
                                               a_k[i] + 16 * g < kend ? 4u * (uint32_t)(a_src[i] + (int32_t)g * a_step) : kOOB,
                                               0, 0, 0);
#pragma unroll
    for (int j = 0; j < 2; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_void*)(dst + 1024 * (SK_FM + j)), 16,
                                               b_k[j] + 16 * g < kend ? 4u * (uint32_t)(b_src[j] + (int32_t)g * b_step) : kOOB,
                                               0, 0, 0);
  };

  f32x4 acc[SK_FM][SK_FN];
#pragma unroll
  for (int i = 0; i < SK_FM; ++i)
#pragma unroll
    for (int j = 0; j < SK_FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // A group's operands, a[block][step] and b[block][step].  The LDS reads and
  // their wait are one asm block: the compiler would put a wait for every
  // DMA in flight before a read that it can see.
  const uint32_t a_rd = (uint32_t)(uintptr_t)(lds_void*)lds[wave][0] +
                        (AM == GM_K ? 64 * lr + ((lq ^ ((lr >> 2) & 3)) << 4) : 64 * SK_FM * lq + 4 * SK_FM * lr);
  const uint32_t b_rd = (uint32_t)(uintptr_t)(lds_void*)lds[wave][0] + 1024 * SK_FM +
                        (BMD == GM_K ? 64 * lr + ((lq ^ ((lr >> 2) & 3)) << 4) : 128 * lq + 8 * lr);
  auto compute = [&](uint32_t st) {
    const uint32_t pa = a_rd + st * WB, pb = b_rd + st * WB;
    float a[SK_FM][4], b[SK_FN][4];
    f32x4 a0, a1, b0, b1;      // K-contiguous: a block's four steps
    f32x2 c0, c1, c2, c3;      // A M-contiguous, 32 rows: both blocks of a step
    float e0, e1, e2, e3;      // A M-contiguous, 16 rows
    f32x2 d0, d1, d2, d3;      // B N-contiguous: both blocks of a step
#define FLUID_RD_A_K1 "ds_read_b128 %0, %[pa]\n"
#define FLUID_RD_A_K2 "ds_read_b128 %0, %[pa]\nds_read_b128 %1, %[pa] offset:1024\n"
#define FLUID_RD_A_M1                                                                                       \
  "ds_read_b32 %0, %[pa]\nds_read_b32 %1, %[pa] offset:256\nds_read_b32 %2, %[pa] offset:512\nds_read_b32 %3, " \
  "%[pa] offset:768\n"
#define FLUID_RD_A_M2                                                                                         \
  "ds_read_b64 %0, %[pa]\nds_read_b64 %1, %[pa] offset:512\nds_read_b64 %2, %[pa] offset:1024\nds_read_b64 %3, " \
  "%[pa] offset:1536\n"
#define FLUID_RD_B_K "ds_read_b128 %[b0], %[pb]\nds_read_b128 %[b1], %[pb] offset:1024\ns_waitcnt lgkmcnt(0)"
#define FLUID_RD_B_N                                                                                              \
  "ds_read_b64 %[d0], %[pb]\nds_read_b64 %[d1], %[pb] offset:512\nds_read_b64 %[d2], %[pb] offset:1024\nds_read_b64 " \
  "%[d3], %[pb] offset:1536\ns_waitcnt lgkmcnt(0)"
#define FLUID_RD(RA, ...)                                                                                          \
  do {                                                                                                             \
    if constexpr (BMD == GM_K)                                                                                     \
      asm volatile(RA FLUID_RD_B_K                                                                                 \
                   : __VA_ARGS__, [b0] "=&v"(b0), [b1] "=&v"(b1)                                                    \
                   : [pa] "v"(pa), [pb] "v"(pb)                                                                    \
                   : "memory");                                                                                    \
    else                                                                                                           \
      asm volatile(RA FLUID_RD_B_N                                                                                 \
                   : __VA_ARGS__, [d0] "=&v"(d0), [d1] "=&v"(d1), [d2] "=&v"(d2), [d3] "=&v"(d3)                     \
                   : [pa] "v"(pa), [pb] "v"(pb)                                                                    \
                   : "memory");                                                                                    \
  } while (0)
    if constexpr (AM == GM_K && SK_FM == 1) FLUID_RD(FLUID_RD_A_K1, "=&v"(a0));
    else if constexpr (AM == GM_K) FLUID_RD(FLUID_RD_A_K2, "=&v"(a0), "=&v"(a1));
    else if constexpr (SK_FM == 1) FLUID_RD(FLUID_RD_A_M1, "=&v"(e0), "=&v"(e1), "=&v"(e2), "=&v"(e3));
    else FLUID_RD(FLUID_RD_A_M2, "=&v"(c0), "=&v"(c1), "=&v"(c2), "=&v"(c3));
#undef FLUID_RD
#undef FLUID_RD_A_K1
#undef FLUID_RD_A_K2
#undef FLUID_RD_A_M1
#undef FLUID_RD_A_M2
#undef FLUID_RD_B_K
#undef FLUID_RD_B_N
    if constexpr (AM == GM_K) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        a[0][s] = a0[s];
        if constexpr (SK_FM == 2) a[1][s] = a1[s];
      }
    } else if constexpr (SK_FM == 1) {
      a[0][0] = e0, a[0][1] = e1, a[0][2] = e2, a[0][3] = e3;
    } else {
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i][0] = c0[i], a[i][1] = c1[i], a[i][2] = c2[i], a[i][3] = c3[i];
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if constexpr (BMD == GM_K) {
#pragma unroll
        for (int s = 0; s < 4; ++s) b[j][s] = j ? b1[s] : b0[s];
      } else {
        b[j][0] = d0[j], b[j][1] = d1[j], b[j][2] = d2[j], b[j][3] = d3[j];
      }
    }
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < SK_FM; ++i)
#pragma unroll
        for (int j = 0; j < SK_FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][s], b[j][s], acc[i][j], 0, 0, 0);
  };
  // waits until at most the `rest` newest groups are in flight
  auto arrived = [&](uint32_t rest) {
    asm volatile("" ::: "memory");
    switch (min(rest, (uint32_t)NS - 1)) {
      case 0: __builtin_amdgcn_s_waitcnt(vmcnt_imm(0)); break;
      case 1: __builtin_amdgcn_s_waitcnt(vmcnt_imm(ND)); break;
      case 2: __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * ND)); break;
      case 3: __builtin_amdgcn_s_waitcnt(vmcnt_imm(3 * ND)); break;
      case 4: __builtin_amdgcn_s_waitcnt(vmcnt_imm(4 * ND)); break;
      default: __builtin_amdgcn_s_waitcnt(vmcnt_imm(5 * ND)); break;
    }
    asm volatile("" ::: "memory");
  };

  // group g travels through stage g % NS, NS groups in flight; no other
  // wavefront touches the stage, so the loop has no barrier.  No load past
  // the slice: it would cost as much issue time as a real one.
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

  // row / column of a block's MFMA index: a row of 32 M- or N-contiguous
  // values gives a lane two neighbouring ones, one for each block
  auto m_of = [&](int i, int r) { return AM == GM_K || SK_FM == 1 ? 16 * i + r : 2 * r + i; };
  auto n_of = [&](int j, int c) { return BMD == GM_K ? 16 * j + c : 2 * c + j; };
  float* red = (float*)lds;
  __syncthreads();  // every wavefront is past its last read of its stages
  // partial tiles -> LDS, then every thread sums W partials of some outputs
#pragma unroll
  for (int i = 0; i < SK_FM; ++i)
#pragma unroll
    for (int j = 0; j < SK_FN; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        red[(wave * SK_TM + m_of(i, 4 * lq + v)) * SK_RP + n_of(j, lr)] = acc[i][j][v];
  __syncthreads();
  float* C = (float*)p.C;
  if (p.cmode == 2) {
    // M-contiguous C: a thread writes 4 consecutive rows of one column
    for (int e = tid; e < SK_TM * SK_TN / 4; e += 64 * W) {
      const int c = e / (SK_TM / 4), r0 = (e % (SK_TM / 4)) * 4;
      const uint32_t n = tc.n0 + c, m0 = tc.m0 + r0;
      if (n >= p.N) continue;
      float o[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        float sum = 0.f;
        for (int w = 0; w < W; ++w) sum += red[(w * SK_TM + r0 + t) * SK_RP + c];
        o[t] = gemm_epi<RES>(p, tc.r_base, m0 + t, n, sum);
      }
      // four rows m0..m0+3 lie in one M2 run (M2 % 4 == 0 in this mode)
      if (m0 + 3 < p.M) {
        *(float4*)(C + tc.c_base + row_off(p, m0, p.c_m1, p.c_m2) + (int32_t)n * p.c_n) = make_float4(o[0], o[1], o[2], o[3]);
      } else {
        for (int t = 0; t < 4; ++t)
          if (m0 + t < p.M) C[tc.c_base + row_off(p, m0 + t, p.c_m1, p.c_m2) + (int32_t)n * p.c_n] = o[t];
      }
    }
  } else {
    // a thread writes 4 consecutive columns of one row (one 16-byte store
    // when C is N-contiguous)
    for (int e = tid; e < SK_TM * SK_TN / 4; e += 64 * W) {
      const int r = e / (SK_TN / 4), c0 = (e % (SK_TN / 4)) * 4;
      const uint32_t m = tc.m0 + r, n0 = tc.n0 + c0;
      if (m >= p.M) continue;
      float o[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        float sum = 0.f;
        for (int w = 0; w < W; ++w) sum += red[(w * SK_TM + r) * SK_RP + c0 + t];
        o[t] = n0 + t < p.N ? gemm_epi<RES>(p, tc.r_base, m, n0 + t, sum) : sum;
      }
      const int32_t base = tc.c_base + row_off(p, m, p.c_m1, p.c_m2);
      if (p.cmode == 1 && n0 + 3 < p.N && ((uintptr_t)(C + base + (int32_t)n0) & 15u) == 0) {
        *(float4*)(C + base + (int32_t)n0) = make_float4(o[0], o[1], o[2], o[3]);
      } else {
        for (int t = 0; t < 4; ++t)
          if (n0 + t < p.N) C[base + (int32_t)(n0 + t) * p.c_n] = o[t];
      }
    }
  }
#endif
}

template <int W, int SK_FM, int NS, int AM, int BMD, bool RES>
__global__ __launch_bounds__(64 * W) void gemm_f32_dl_kernel(GemmParams p) {
  gemm_f32_dl_tile<W, SK_FM, NS, AM, BMD, RES>(p, blockIdx.x);
}

// The members of a group share tile shape, operand modes and epilogue
// instance; each workgroup runs one tile of its member.
template <int W, int SK_FM, int NS, int AM, int BMD, bool RES>
__global__ __launch_bounds__(64 * W) void gemm_f32_dl_group_kernel(GemmGroup G) {
  uint32_t i = 0;
  while (i + 1 < G.n && blockIdx.x >= G.tiles[i + 1]) ++i;
  gemm_f32_dl_tile<W, SK_FM, NS, AM, BMD, RES>(G.p[i], blockIdx.x - G.tiles[i]);
}

hipError_t launch_gemm_f32_dl(const NodeKernel& k, hipStream_t s) {
  const GemmParams& p = k.gemm;
  const dim3 grid(p.tiles_m * p.tiles_n * p.G);
#define FLUID_F32DL(Wv, FMv, NSv, AMv, BMv)                                                                     \
  do {                                                                                                     \
    if (p.rop) hipLaunchKernelGGL((gemm_f32_dl_kernel<Wv, FMv, NSv, AMv, BMv, true>), grid, dim3(64 * Wv), 0, s, p); \
    else hipLaunchKernelGGL((gemm_f32_dl_kernel<Wv, FMv, NSv, AMv, BMv, false>), grid, dim3(64 * Wv), 0, s, p);      \
  } while (0)
#define FLUID_F32DL_W(Wv, FMv, NSv)                                                          \
  if (k.amode == GM_K && k.bmode == GM_MN) FLUID_F32DL(Wv, FMv, NSv, GM_K, GM_MN);           \
  else if (k.amode == GM_K && k.bmode == GM_K) FLUID_F32DL(Wv, FMv, NSv, GM_K, GM_K);        \
  else if (k.amode == GM_MN && k.bmode == GM_MN) FLUID_F32DL(Wv, FMv, NSv, GM_MN, GM_MN);    \
  else if (k.amode == GM_MN && k.bmode == GM_K) FLUID_F32DL(Wv, FMv, NSv, GM_MN, GM_K);      \
  else return hipErrorInvalidValue;
  // tile 6: 16 x 32 over 8 wavefronts; tile 7: 32 x 32 over 4
  if (k.gemm_tile == 6) {
    FLUID_F32DL_W(8, 1, 3)
  } else {
    FLUID_F32DL_W(4, 2, 3)
  }
#undef FLUID_F32DL_W
#undef FLUID_F32DL
  return hipGetLastError();
}

hipError_t launch_gemm_f32_dl_group(const NodeKernel& k, const GemmGroup& G, hipStream_t s) {
  if (k.dtype != DT_F32 || (k.gemm_tile != 6 && k.gemm_tile != 7) || G.n < 1 || G.n > (uint32_t)kMaxGroup)
    return hipErrorInvalidValue;
  const bool res = k.gemm.rop != 0;
  const dim3 grid(G.tiles[G.n]);
#define FLUID_F32DLG(Wv, FMv, NSv, AMv, BMv)                                                                          \
  do {                                                                                                           \
    if (res) hipLaunchKernelGGL((gemm_f32_dl_group_kernel<Wv, FMv, NSv, AMv, BMv, true>), grid, dim3(64 * Wv), 0, s, G); \
    else hipLaunchKernelGGL((gemm_f32_dl_group_kernel<Wv, FMv, NSv, AMv, BMv, false>), grid, dim3(64 * Wv), 0, s, G);    \
  } while (0)
#define FLUID_F32DLG_W(Wv, FMv, NSv)                                                          \
  if (k.amode == GM_K && k.bmode == GM_MN) FLUID_F32DLG(Wv, FMv, NSv, GM_K, GM_MN);           \
  else if (k.amode == GM_K && k.bmode == GM_K) FLUID_F32DLG(Wv, FMv, NSv, GM_K, GM_K);        \
  else if (k.amode == GM_MN && k.bmode == GM_MN) FLUID_F32DLG(Wv, FMv, NSv, GM_MN, GM_MN);    \
  else if (k.amode == GM_MN && k.bmode == GM_K) FLUID_F32DLG(Wv, FMv, NSv, GM_MN, GM_K);      \
  else return hipErrorInvalidValue;
  if (k.gemm_tile == 6) {
    FLUID_F32DLG_W(8, 1, 3)
  } else {
    FLUID_F32DLG_W(4, 2, 3)
  }
#undef FLUID_F32DLG_W
#undef FLUID_F32DLG
  return hipGetLastError();
}

}  // namespace fluid
