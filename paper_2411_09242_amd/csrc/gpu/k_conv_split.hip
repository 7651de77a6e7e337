// Convolution (no padding, stride 1, one group) as an implicit GEMM on the
// bf16 matrix cores, every fp32 value split into three bf16 ones and a
// product summed from six (k_gemm_f32_split.hip), for any layout of the
// input and output.
//
//   y[n, o, i, j] = sum_{c, u, v} x[n, c, i+u, j+v] * w[o, c, u, v] + b[o]
//
// Rows m are output pixels, (n, i, j), or (n, j, i) where H is the input's
// unit-stride dim (512 -> 512 at 14 x 14 126 -> 68 us in that layout), columns
// output channels o, the reduction runs over k = (c, u, v), the weight's own
// order.  In any layout x[n, c, i+u, j+v] sits at row_offset(m) +
// col_offset(k), so the unfolded input is never built.  The lanes of a
// wavefront load 64 consecutive pixels of one k, k and its offset in scalar
// registers; a lane's eight k of one pixel are one 16-byte LDS write per bf16
// plane.  The weight rows are K-contiguous.
//
// BM x BN tile, eight wavefronts as KS groups of WM x WN, group s taking the
// s-th 16 k of every K-tile of 16 KS (partial sums added in group order):
//   128 x 64, KS 4 (wavefronts of 64 x 64): the wide layers;
//   64 x 64, KS 4 (64 x 32): fewer pixels, 100 to 200 tiles;
//   64 x 32, KS 8 (64 x 32): layers with fewer tiles than compute units,
//   where a tile's K-tiles must be few.
// Measured against the fp32 MFMA kernel's best (3 x 3, C -> Co at H x W):
// 64 -> 64 at 224 72 -> 56 us, 128 -> 128 at 112 76 -> 48 (128 x 64); 256 ->
// 256 at 56 77 -> 53, 128 -> 256 43 -> 31 (64 x 64); 512 -> 512 at 28 121 ->
// 67, 256 -> 512 65 -> 38 (64 x 32); at 14 x 14 (64 tiles) both take 63-66.
// For three input channels the fp32 kernels are faster (64 at 224 x 224: 17
// and 29 us).  At 56 x 56 the matrix cores are busy 23% of the time, VALU 44%,
// LDS 30%: the split, its LDS writes and reads and the MFMAs share a barrier
// per K-tile and overlap little.  Tried, slower: two and three
// register sets ahead, MFMAs interleaved with the split by scheduling
// groups; no faster: (c, u, v) stepped in scalar registers.
#include "launch.h"
#include "split_common.h"

namespace fluid {

namespace {

// Offset of row m, strides of the batch, the outer and the inner pixel dim.
__device__ __forceinline__ int32_t conv_row_off(const ConvParams& p, uint32_t m, int32_t sn, int32_t so, int32_t si) {
  const uint32_t n = fdiv(m, p.ohw_div);
  const uint32_t r = m - n * p.OHW;
  const uint32_t i = fdiv(r, p.pi_div);
  const uint32_t j = r - i * p.PI;
  return (int32_t)n * sn + (int32_t)i * so + (int32_t)j * si;
}

}  // namespace

// WV: weight rows in 16-byte loads (K % 4 == 0 and an aligned weight)
template <int BM, int BN, int WM, int WN, int KS, bool WV>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void conv_f32_split_kernel(ConvParams p) {
  constexpr int T = 512, BK = 16 * KS, CH = BK / 8;
  static_assert(64 * WM * WN * KS == T && BM % 64 == 0, "eight wavefronts");
  constexpr int FI = BM / WM / 32, FJ = BN / WN / 32, NB = FI * FJ;
  constexpr int NA = BM * CH / T, NBL = BN * CH / T;   // chunks of 8 k a thread carries
  static_assert(NA * T == BM * CH && NBL * T == BN * CH, "tile shape");
  constexpr int APL = BM * BK * 2, BPL = BN * BK * 2;  // bytes of one plane
  constexpr int STAGE = 3 * (APL + BPL);
  constexpr int OWN = 4 * NB / KS;                     // 4-row pieces a wavefront finishes
  constexpr int RED = T / 64 * (4 * NB - OWN) * 1024;
  static_assert(OWN * KS == 4 * NB && 2 * STAGE >= RED && 2 * STAGE <= 160 * 1024, "LDS");
  __shared__ __attribute__((aligned(1024))) uint8_t lds[2 * STAGE];
  const uint32_t tm = blockIdx.x / p.tiles_n, tn = blockIdx.x - tm * p.tiles_n;
  const uint32_t m0 = tm * BM, n0 = tn * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave / (WM * WN), wpos = wave % (WM * WN);
  const int wm = wpos / WN, wn = wpos % WN;
  const int lr = lane & 31, lh = lane >> 5;
  const Rsrc rx = make_rsrc(p.x, p.x_bytes);
  const Rsrc rw = make_rsrc(p.w, p.w_bytes);

  // Pixels past M and channels past Co are clamped onto the first (they only
  // feed outputs that are never stored); only k past K has to read as zero.
  uint32_t a_off[NA], b_off[NBL];  // byte offsets of the pixel, of the weight row's chunk
  int a_k[NA], b_k[NBL];
  int a_lds[NA], b_lds[NBL];
#pragma unroll
  for (int q = 0; q < NA; ++q) {
    const int c = q * T + tid;
    const int row = c % BM, kc = __builtin_amdgcn_readfirstlane(c / BM);
    const uint32_t m = m0 + row;
    a_off[q] = 4u * (uint32_t)(m < p.M ? conv_row_off(p, m, p.x_n, p.x_po, p.x_pi) : 0);
    a_k[q] = 8 * kc;
    a_lds[q] = row * BK * 2 + ((kc ^ split_swz<BK>(row)) << 4);
  }
#pragma unroll
  for (int q = 0; q < NBL; ++q) {
    const int c = q * T + tid;
    const int row = c / CH, kc = c % CH;
    const uint32_t o = n0 + row;
    b_off[q] = 4u * ((o < p.Co ? o : 0) * p.K + 8 * kc);
    b_k[q] = 8 * kc;
    b_lds[q] = 3 * APL + row * BK * 2 + ((kc ^ split_swz<BK>(row)) << 4);
  }

  struct Regs {
    float a[NA][8], b[NBL][8];
  };
  auto gload = [&](Regs& R, uint32_t k0) {
    // lane 8 q + h forms the column offset of k h of chunk q; the loads take
    // it from there as a scalar
    int ak = a_k[0];
#pragma unroll
    for (int q = 1; q < NA; ++q) ak = lane >= 8 * q ? a_k[q] : ak;
    const uint32_t kl = k0 + ak + (lane & 7);
    const uint32_t c = fdiv(kl, p.khw_div), r = kl - c * p.KHW, u = fdiv(r, p.kw_div), v = r - u * p.KW;
    const int32_t cl = 4 * ((int32_t)c * p.x_c + (int32_t)u * p.x_h + (int32_t)v * p.x_w);
#pragma unroll
    for (int q = 0; q < NA; ++q)
#pragma unroll
      for (int h = 0; h < 8; ++h) {
        const bool in = k0 + a_k[q] + h < p.K;
        R.a[q][h] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                  rx, in ? a_off[q] : kOOB,
                                                  in ? __builtin_amdgcn_readlane(cl, 8 * q + h) : 0, 0));
      }
#pragma unroll
    for (int q = 0; q < NBL; ++q) {
      const uint32_t k = k0 + b_k[q], off = b_off[q] + 4u * k0;
      if constexpr (WV) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint4 w = bload16(rw, k + 4 * h < p.K ? off + 16u * h : kOOB);
          R.b[q][4 * h] = __uint_as_float(w.x), R.b[q][4 * h + 1] = __uint_as_float(w.y);
          R.b[q][4 * h + 2] = __uint_as_float(w.z), R.b[q][4 * h + 3] = __uint_as_float(w.w);
        }
      } else {
#pragma unroll
        for (int h = 0; h < 8; ++h) R.b[q][h] = bload4(rw, k + h < p.K ? off + 4u * h : kOOB);
      }
    }
  };
  auto lstore = [&](const Regs& R, int st) {
    uint8_t* s = lds + st * STAGE;
#pragma unroll
    for (int q = 0; q < NA; ++q) split_put(R.a[q], s + a_lds[q], APL);
#pragma unroll
    for (int q = 0; q < NBL; ++q) split_put(R.b[q], s + b_lds[q], BPL);
  };

  f32x16 acc[FI][FJ], low[FI][FJ];
#pragma unroll
  for (int i = 0; i < FI; ++i)
#pragma unroll
    for (int j = 0; j < FJ; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = low[i][j][v] = 0.f;
  int a_rd[FI], b_rd[FJ];
#pragma unroll
  for (int i = 0; i < FI; ++i) {
    const int r = wm * 32 * FI + 32 * i + lr;
    a_rd[i] = r * BK * 2 + (((2 * grp + lh) ^ split_swz<BK>(r)) << 4);
  }
#pragma unroll
  for (int j = 0; j < FJ; ++j) {
    const int r = wn * 32 * FJ + 32 * j + lr;
    b_rd[j] = 3 * APL + r * BK * 2 + (((2 * grp + lh) ^ split_swz<BK>(r)) << 4);
  }
  bf16x8 a[3][FI], b[3][FJ];
  auto fread = [&](int st) {
    const uint8_t* s = lds + st * STAGE;
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) {
#pragma unroll
      for (int i = 0; i < FI; ++i) a[pl][i] = *(const bf16x8*)(s + a_rd[i] + pl * APL);
#pragma unroll
      for (int j = 0; j < FJ; ++j) b[pl][j] = *(const bf16x8*)(s + b_rd[j] + pl * BPL);
    }
  };

  // K-tile t is multiplied from stage t % 2 while tile t+1, loaded into
  // registers during tile t-1, is split into the other stage and tile t+2
  // is loaded; loads past the end of K read zeros without touching memory
  const uint32_t nt = (p.K + BK - 1) / BK;
  Regs R;
  gload(R, 0);
  lstore(R, 0);
  gload(R, BK);
  __syncthreads();
  for (uint32_t t = 0; t < nt; ++t) {
    fread(t & 1);
    lstore(R, (t + 1) & 1);
    gload(R, (t + 2) * BK);
    split_mul(a, b, acc, low);
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < FI; ++i)
#pragma unroll
    for (int j = 0; j < FJ; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = (acc[i][j][v] + low[i][j][v]) * kSplitUnscale;

  // The groups' partial sums, in pieces of four rows of a 32 x 32 block:
  // group g finishes pieces g OWN .. +OWN-1 and parks the others.
  float4* red = (float4*)lds;
  auto parked = [&](int g, int e) {
    return ((g * WM * WN + wpos) * (4 * NB - OWN) + (e / OWN > g ? e - OWN : e)) * 64 + lane;
  };
  float out[OWN][4];
  auto combine = [&]() {
#pragma unroll
    for (int e = 0; e < 4 * NB; ++e)
      if (e / OWN != grp) {
        const f32x16& x = acc[e / 4 / FJ][e / 4 % FJ];
        const int v = 4 * (e % 4);
        red[parked(grp, e)] = make_float4(x[v], x[v + 1], x[v + 2], x[v + 3]);
      }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4 * NB; ++e)
      if (e / OWN == grp) {
        const f32x16& x = acc[e / 4 / FJ][e / 4 % FJ];
        float* y = out[e % OWN];
#pragma unroll
        for (int t = 0; t < 4; ++t) y[t] = x[4 * (e % 4) + t];
#pragma unroll
        for (int g = 0; g < KS; ++g)
          if (g != grp) {
            const float4 z = red[parked(g, e)];
            y[0] += z.x, y[1] += z.y, y[2] += z.z, y[3] += z.w;
          }
      }
  };
  combine();
  bool bad = false;
#pragma unroll
  for (int e = 0; e < OWN; ++e)
#pragma unroll
    for (int t = 0; t < 4; ++t) bad |= !(fabsf(out[e][t]) <= 3.4028234663852886e38f);
  if (__syncthreads_or(bad)) {
    // the exceptions of the split: the tile again with the fp32 MFMA, the
    // groups taking KS runs of K.  Step t of sixteen k takes, in the k slot
    // lane / 32, the real k 8 (lane / 32) + t of both operands; the next
    // sixteen k are in flight.
    const uint32_t kg = (p.K + 16u * KS - 1u) / (16u * KS) * 16u;
    const uint32_t kb = (uint32_t)grp * kg, ke = min(p.K, kb + kg);
    uint32_t ao[FI], bo[FJ];
#pragma unroll
    for (int i = 0; i < FI; ++i) {
      const uint32_t m = m0 + wm * 32 * FI + 32 * i + lr;
      ao[i] = 4u * (uint32_t)(m < p.M ? conv_row_off(p, m, p.x_n, p.x_po, p.x_pi) : 0);
    }
#pragma unroll
    for (int j = 0; j < FJ; ++j) {
      const uint32_t o = n0 + wn * 32 * FJ + 32 * j + lr;
      bo[j] = 4u * ((o < p.Co ? o : 0) * p.K);
    }
    struct Octs {
      float a[FI][8], b[FJ][8];
    };
    auto octs = [&](Octs& O, uint32_t k1) {
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const uint32_t k = k1 + t;
        const uint32_t c = fdiv(k, p.khw_div), r = k - c * p.KHW, u = fdiv(r, p.kw_div), v = r - u * p.KW;
        const uint32_t co = 4u * (uint32_t)((int32_t)c * p.x_c + (int32_t)u * p.x_h + (int32_t)v * p.x_w);
#pragma unroll
        for (int i = 0; i < FI; ++i) O.a[i][t] = bload4(rx, k < ke ? ao[i] + co : kOOB);
        if constexpr (!WV) {
#pragma unroll
          for (int j = 0; j < FJ; ++j) O.b[j][t] = bload4(rw, k < ke ? bo[j] + 4u * k : kOOB);
        }
      }
      if constexpr (WV) {
#pragma unroll
        for (int j = 0; j < FJ; ++j)
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const uint4 w = bload16(rw, k1 + 4 * h < ke ? bo[j] + 4u * (k1 + 4 * h) : kOOB);
            O.b[j][4 * h] = __uint_as_float(w.x), O.b[j][4 * h + 1] = __uint_as_float(w.y);
            O.b[j][4 * h + 2] = __uint_as_float(w.z), O.b[j][4 * h + 3] = __uint_as_float(w.w);
          }
      }
    };
#pragma unroll
    for (int i = 0; i < FI; ++i)
#pragma unroll
      for (int j = 0; j < FJ; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    Octs nx;
    octs(nx, kb + 8 * lh);
    for (uint32_t k0 = kb; k0 < ke; k0 += 16) {
      const Octs O = nx;
      octs(nx, k0 + 16 + 8 * lh);
#pragma unroll
      for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int i = 0; i < FI; ++i)
#pragma unroll
          for (int j = 0; j < FJ; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(O.a[i][t], O.b[j][t], acc[i][j], 0, 0, 0);
    }
    combine();
  }

#pragma unroll
  for (int e = 0; e < 4 * NB; ++e) {
    if (e / OWN != grp) continue;
    const uint32_t o = n0 + wn * 32 * FJ + 32 * (e / 4 % FJ) + lr;
    if (o >= p.Co) continue;
    const float bo = p.bias ? p.bias[o] : 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const uint32_t m = m0 + wm * 32 * FI + 32 * (e / 4 / FJ) + 8 * (e % 4) + 4 * lh + t;
      if (m < p.M) p.y[conv_row_off(p, m, p.y_n, p.y_po, p.y_pi) + (int32_t)o * p.y_c] = out[e % OWN][t] + bo;
    }
  }
}

hipError_t launch_conv_split(const NodeKernel& k, hipStream_t s) {
  const ConvParams& p = k.conv;
  const uint32_t bm = k.conv_bm;
  const uint32_t grid = ((p.M + bm - 1) / bm) * p.tiles_n;
  const bool wv = p.K % 4 == 0 && ((uintptr_t)p.w & 15u) == 0;
#define FLUID_CS(BMv, BNv, WMv, WNv, KSv)                                                                       \
  do {                                                                                                          \
    if (wv) hipLaunchKernelGGL((conv_f32_split_kernel<BMv, BNv, WMv, WNv, KSv, true>), dim3(grid), dim3(512), 0, s, p); \
    else hipLaunchKernelGGL((conv_f32_split_kernel<BMv, BNv, WMv, WNv, KSv, false>), dim3(grid), dim3(512), 0, s, p);   \
  } while (0)
  if (bm == 128 && k.conv_tile == 64) FLUID_CS(128, 64, 2, 1, 4);
  else if (bm == 64 && k.conv_tile == 64) FLUID_CS(64, 64, 1, 2, 4);
  else if (bm == 64 && k.conv_tile == 32) FLUID_CS(64, 32, 1, 1, 8);
  else return hipErrorInvalidValue;
#undef FLUID_CS
  return hipGetLastError();
}

}  // namespace fluid
