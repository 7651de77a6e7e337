// fp32 GEMM on the bf16 matrix cores, for a K- or M-contiguous A and an N-
// or K-contiguous B.  Every fp32 value x is written exactly as the sum of
// three bf16 values (24 = 3 x 8 significant bits):
//   h = bf16(x),  m = bf16(x - h),  l = bf16(x - h - m)
// (both differences are exact; the decomposition of Henry, Tang and Heinecke,
// "Leveraging the bfloat16 Artificial Intelligence Datatype For
// Higher-Precision Computations", ARITH 2019), and a product a b is summed
// from the six partial products h h', h m', m h', m m', h l', l h', each
// exact in the fp32 accumulator's input; of the dropped ones m l' and l m'
// are at most 2^-25 of |a b| each, together the rounding of one fp32
// multiply-add.  The bf16 cores run 16 times the fp32 ones' rate, so six
// products still leave 2.7 times the fp32 matrix peak, and an accumulator is
// rounded once per 16 k of a product (6 / 16 per k) instead of every 2 k by
// the fp32 MFMA.  The operands are scaled (split_common.h), so that this
// holds for every finite operand, subnormal ones too.
//
// Exceptions of the split, all found after the product: an infinity or NaN
// (its x - h is NaN), a value of 2^104 or more (its scaled h is an infinity)
// and a sum that reaches 2^80 leave a non-finite accumulator.  A workgroup
// that sees one recomputes its tile with the fp32 MFMA straight from memory,
// so that infinities, NaN and values up to the largest float behave as in
// fp32 (4096 x 1024 x 4096 with a NaN in every row takes 465 us, 262 on the
// fp32 tile of that size).
#include "launch.h"
#include "split_common.h"

namespace fluid {

namespace {

// Tile of workgroup b: the tiles are dealt to the eight XCDs (b % 8) in
// contiguous ranges, walked within a batch in bands of four tile rows, so
// that the workgroups running on one XCD at a time share rows of A and
// columns of B in its L2.
__device__ __forceinline__ TileCoord split_tile(const GemmParams& p, uint32_t BM, uint32_t BN) {
  const uint32_t total = gridDim.x, b = blockIdx.x;
  const uint32_t x = b & 7, per = total >> 3, rem = total & 7;
  const uint32_t lin = x * per + min(x, rem) + (b >> 3);
  const uint32_t per_g = p.tiles_m * p.tiles_n;
  const uint32_t g = lin / per_g, r = lin - g * per_g;
  const uint32_t band = r / (4 * p.tiles_n), first = 4 * band;
  const uint32_t rows = min(4u, p.tiles_m - first);
  const uint32_t q = r - band * 4 * p.tiles_n;
  return tile_coord_lin(p, g * per_g + (first + q % rows) * p.tiles_n + q / rows, BM, BN);
}

}  // namespace

// BM x BN tile; KS groups of WM x WN wavefronts of 64 x 64 each, group s
// multiplying the s-th ST * 16 k of every K-tile (partial sums added in
// group order at the end).  A CU holds one workgroup of eight wavefronts, so
// that every SIMD has two to issue from:
//  * 256 x 128 (KS 1): 1.5 times the MFMAs per split element and per LDS
//    write of the smaller tile; K-contiguous A only (with an M-contiguous
//    one it spills 15 to 22 VGPRs).
//  * 128 x 128 (KS 2): where the larger tile would leave CUs idle; two groups
//    over K rather than 64 x 32 wavefront tiles, which would read LDS half as
//    much again per MFMA.
//  Which of them runs: split_tile_of in dispatch.cpp.
// Measured (weights from HBM) against the fp32 MFMA tiles of the same size that
// they replace: 128 x 128 at 4096 x 1024 x 1024 (M N K) 49-52 us, was 83.7, and
// 4096 x 1024 x 4096 164-173, was 267; 256 x 128 at 4096 x 4096 x 1024 167 us
// (206 TFLOP/s, 1.23 PFLOP/s of bf16 MFMA), was 276.  Bound: at those sizes
// the matrix cores are busy 62% and 59% of the time, VALU 50 and 45%, LDS 47
// and 41% (a third of that bank conflicts).  Tried: the groups in
// alternating MFMA and split phases (two barriers per K-tile) 8% slower; a
// second register set, loads two K-tiles ahead, 0 to 10% slower; the six
// products in one accumulator as fast, but with 2.6 times the error.
template <int BM, int BN, int WM, int WN, int KS, int ST, bool AK, bool BKC, bool RES>
__global__ __launch_bounds__(64 * WM * WN * KS) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_f32_split_kernel(GemmParams p) {
  constexpr int T = 64 * WM * WN * KS, BK = 16 * KS * ST, CH = BK / 8;
  constexpr int FI = BM / WM / 32, FJ = BN / WN / 32, NB = FI * FJ;
  constexpr int NA = BM * CH / T, NBL = BN * CH / T;  // chunks of 8 k a thread carries
  static_assert(NA * T == BM * CH && NBL * T == BN * CH && NB % KS == 0, "tile shape");
  constexpr int APL = BM * BK * 2, BPL = BN * BK * 2;  // bytes of one plane
  constexpr int STAGE = 3 * (APL + BPL);
  constexpr int OWN = NB / KS;                         // blocks a wavefront finishes
  constexpr int RED = KS > 1 ? T / 64 * (NB - OWN) * 4096 : 0;
  constexpr int LDS = 2 * STAGE > RED ? 2 * STAGE : RED;
  __shared__ __attribute__((aligned(1024))) uint8_t lds[LDS];
  const TileCoord tc = split_tile(p, BM, BN);
  // causal attention: a tile entirely above the diagonal is never read; a
  // row block's A is zero past its last row, so K stops there
  if ((p.causal & 1u) && tc.n0 > tc.m0 + BM - 1) return;
  const uint32_t kend = (p.causal & 2u) ? min(p.K, tc.m0 + BM) : p.K;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave / (WM * WN), wpos = wave % (WM * WN);
  const int wm = wpos / WN, wn = wpos % WN;
  const int lr = lane & 31, lh = lane >> 5;
  const Rsrc ra = make_rsrc(p.A, p.a_bytes);
  const Rsrc rb = make_rsrc(p.B, p.b_bytes);

  // Chunk q of a thread.  K-contiguous operand: CH lanes cover a row's K-tile
  // (two 16-byte loads per chunk); M- or N-contiguous: the lanes of a
  // wavefront take neighbouring rows at one k, eight 4-byte loads, each 256
  // contiguous bytes, and the packing of two k into a dword transposes.
  // Rows past M or N are clamped onto row 0 (they only feed outputs that
  // are never stored); only k past K has to read as zero.
  int32_t a_off[NA], b_off[NBL];  // element offset without the K-tile's k0
  int a_k[NA], b_k[NBL];          // first k of the chunk within the K-tile
  int a_lds[NA], b_lds[NBL];      // its byte offset within a plane
#pragma unroll
  for (int q = 0; q < NA; ++q) {
    const int c = q * T + tid;
    const int row = AK ? c / CH : c % BM, kc = AK ? c % CH : c / BM;
    const uint32_t m = tc.m0 + row;
    a_off[q] = tc.a_base + (m < p.M ? row_off(p, m, p.a_m1, p.a_m2) : 0) + 8 * kc * (AK ? 1 : p.a_k);
    a_k[q] = 8 * kc;
    a_lds[q] = row * BK * 2 + ((kc ^ split_swz<BK>(row)) << 4);
  }
#pragma unroll
  for (int q = 0; q < NBL; ++q) {
    const int c = q * T + tid;
    const int row = BKC ? c / CH : c % BN, kc = BKC ? c % CH : c / BN;
    const uint32_t n = tc.n0 + row;
    b_off[q] = tc.b_base + (n < p.N ? (int32_t)n * (BKC ? p.b_n : 1) : 0) + 8 * kc * (BKC ? 1 : p.b_k);
    b_k[q] = 8 * kc;
    b_lds[q] = 3 * APL + row * BK * 2 + ((kc ^ split_swz<BK>(row)) << 4);
  }

  struct Regs {
    float a[NA][8], b[NBL][8];
  };
  // a chunk: 8 k from k; off = element offset of its first k
  auto chunk = [&](Rsrc r, float* v, int32_t off, uint32_t k, bool kc, int32_t ks) {
    if (kc) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint4 u = bload16(r, k + 4 * h < kend ? 4u * (uint32_t)(off + 4 * h) : kOOB);
        v[4 * h] = __uint_as_float(u.x), v[4 * h + 1] = __uint_as_float(u.y);
        v[4 * h + 2] = __uint_as_float(u.z), v[4 * h + 3] = __uint_as_float(u.w);
      }
    } else {
#pragma unroll
      for (int h = 0; h < 8; ++h) v[h] = bload4(r, k + h < kend ? 4u * (uint32_t)(off + h * ks) : kOOB);
    }
  };
  auto gload = [&](Regs& R, uint32_t k0) {
#pragma unroll
    for (int q = 0; q < NA; ++q)
      chunk(ra, R.a[q], a_off[q] + (int32_t)k0 * (AK ? 1 : p.a_k), k0 + a_k[q], AK, p.a_k);
#pragma unroll
    for (int q = 0; q < NBL; ++q)
      chunk(rb, R.b[q], b_off[q] + (int32_t)k0 * (BKC ? 1 : p.b_k), k0 + b_k[q], BKC, p.b_k);
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

  // operand addresses: lane l reads row l % 32 of its block, chunk
  // 2 grp + l / 32 (MFMA 32x32x16 bf16: lane l holds A[l%32][8(l/32)..+7])
  int a_rd[FI], b_rd[FJ];
#pragma unroll
  for (int i = 0; i < FI; ++i) {
    const int r = wm * 32 * FI + 32 * i + lr;
    a_rd[i] = r * BK * 2 + (((2 * ST * grp + lh) ^ split_swz<BK>(r)) << 4);
  }
#pragma unroll
  for (int j = 0; j < FJ; ++j) {
    const int r = wn * 32 * FJ + 32 * j + lr;
    b_rd[j] = 3 * APL + r * BK * 2 + (((2 * ST * grp + lh) ^ split_swz<BK>(r)) << 4);
  }
  struct Frag {
    bf16x8 a[3][FI], b[3][FJ];
  };
  auto fread = [&](Frag& F, int st, int sx) {
    const uint8_t* s = lds + st * STAGE;
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) {
#pragma unroll
      for (int i = 0; i < FI; ++i) F.a[pl][i] = *(const bf16x8*)(s + (a_rd[i] ^ (sx << 5)) + pl * APL);
#pragma unroll
      for (int j = 0; j < FJ; ++j) F.b[pl][j] = *(const bf16x8*)(s + (b_rd[j] ^ (sx << 5)) + pl * BPL);
    }
  };

  // K-tile t is multiplied from stage t % 2 while tile t+1, loaded into
  // registers during tile t-1, is split into the other stage and tile t+2
  // is loaded.  Loads past the end of K read zeros without touching memory.
  const uint32_t nt = (kend + BK - 1) / BK;
  Regs R;
  gload(R, 0);
  lstore(R, 0);
  gload(R, BK);
  __syncthreads();
  for (uint32_t t = 0; t < nt; t += 2) {
#define FLUID_SPLIT_STEP(U)                                                          \
  if (t + U < nt) {                                                                  \
    Frag F;                                                                          \
    fread(F, U, 0);                                                                  \
    lstore(R, 1 - U);                                                                \
    gload(R, (t + U + 2) * BK);                                                      \
    split_mul(F.a, F.b, acc, low);                                                   \
    if constexpr (ST == 2) {                                                         \
      fread(F, U, 1);                                                                \
      split_mul(F.a, F.b, acc, low);                                                 \
    } else {                                                                         \
      _Pragma("unroll") for (int z = 0; z < 6 * NB; ++z) {                           \
        __builtin_amdgcn_sched_group_barrier(8, 1, 0); /* an MFMA, then */           \
        __builtin_amdgcn_sched_group_barrier(2, 5, 0); /* five VALU of the split */  \
      }                                                                              \
    }                                                                                \
    __syncthreads();                                                                 \
  }
    FLUID_SPLIT_STEP(0)
    FLUID_SPLIT_STEP(1)
#undef FLUID_SPLIT_STEP
  }
#pragma unroll
  for (int i = 0; i < FI; ++i)
#pragma unroll
    for (int j = 0; j < FJ; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = (acc[i][j][v] + low[i][j][v]) * kSplitUnscale;

  // the groups' partial sums: every wavefront parks the blocks that other
  // groups finish and adds theirs to its own, in group order
  auto combine = [&]() {
    if constexpr (KS > 1) {
      float4* red = (float4*)lds;
      auto parked = [&](int g, int b) {  // place of block b of group g, which does not finish it
        return (g * WM * WN + wpos) * (NB - OWN) + (b / OWN > g ? b - OWN : b);
      };
#pragma unroll
      for (int b = 0; b < NB; ++b)
        if (b / OWN != grp)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const f32x16& x = acc[b / FJ][b % FJ];
            red[parked(grp, b) * 256 + v * 64 + lane] =
                make_float4(x[4 * v], x[4 * v + 1], x[4 * v + 2], x[4 * v + 3]);
          }
      __syncthreads();
#pragma unroll
      for (int b = 0; b < NB; ++b)
        if (b / OWN == grp)
#pragma unroll
          for (int g = 0; g < KS; ++g)
            if (g != grp)
#pragma unroll
              for (int v = 0; v < 4; ++v) {
                const float4 y = red[parked(g, b) * 256 + v * 64 + lane];
                f32x16& x = acc[b / FJ][b % FJ];
                x[4 * v] += y.x, x[4 * v + 1] += y.y, x[4 * v + 2] += y.z, x[4 * v + 3] += y.w;
              }
    }
  };
  combine();
  bool bad = false;
#pragma unroll
  for (int b = 0; b < NB; ++b)
    if (KS == 1 || b / OWN == grp)
#pragma unroll
      for (int v = 0; v < 16; ++v) bad |= !(fabsf(acc[b / FJ][b % FJ][v]) <= 3.4028234663852886e38f);
  if (__syncthreads_or(bad)) {
    // the exceptions of the split: the tile again with the fp32 MFMA, the
    // groups taking KS runs of K.  Step t of eight k takes, in the k slot
    // lane / 32, the real k 4 (lane / 32) + t of both operands; the next
    // eight k are in flight.
    const uint32_t kg = (kend + 8u * KS - 1u) / (8u * KS) * 8u;
    const uint32_t kb = (uint32_t)grp * kg, ke = min(kend, kb + kg);
    int32_t ao[FI], bo[FJ];
#pragma unroll
    for (int i = 0; i < FI; ++i) {
      const uint32_t m = tc.m0 + wm * 32 * FI + 32 * i + lr;
      ao[i] = tc.a_base + (m < p.M ? row_off(p, m, p.a_m1, p.a_m2) : 0);
    }
#pragma unroll
    for (int j = 0; j < FJ; ++j) {
      const uint32_t n = tc.n0 + wn * 32 * FJ + 32 * j + lr;
      bo[j] = tc.b_base + (n < p.N ? (int32_t)n * p.b_n : 0);
    }
    struct Quads {
      float a[FI][4], b[FJ][4];
    };
    auto quad = [&](Rsrc r, float* q, int32_t off, uint32_t k, bool kc, int32_t ks) {
      if (kc) {
        const uint4 u = bload16(r, k < ke ? 4u * (uint32_t)(off + (int32_t)k) : kOOB);
        q[0] = __uint_as_float(u.x), q[1] = __uint_as_float(u.y);
        q[2] = __uint_as_float(u.z), q[3] = __uint_as_float(u.w);
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) q[t] = bload4(r, k + t < ke ? 4u * (uint32_t)(off + (int32_t)(k + t) * ks) : kOOB);
      }
    };
    auto quads = [&](Quads& Q, uint32_t k) {
#pragma unroll
      for (int i = 0; i < FI; ++i) quad(ra, Q.a[i], ao[i], k, AK, p.a_k);
#pragma unroll
      for (int j = 0; j < FJ; ++j) quad(rb, Q.b[j], bo[j], k, BKC, p.b_k);
    };
#pragma unroll
    for (int i = 0; i < FI; ++i)
#pragma unroll
      for (int j = 0; j < FJ; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    Quads nx;
    quads(nx, kb + 4 * lh);
    for (uint32_t k0 = kb; k0 < ke; k0 += 8) {
      const Quads Q = nx;
      quads(nx, k0 + 8 + 4 * lh);
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < FI; ++i)
#pragma unroll
          for (int j = 0; j < FJ; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(Q.a[i][t], Q.b[j][t], acc[i][j], 0, 0, 0);
    }
    combine();
  }

  float* C = (float*)p.C;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    if (KS > 1 && b / OWN != grp) continue;
    f32x16& x = acc[b / FJ][b % FJ];
    const uint32_t mf = tc.m0 + wm * 32 * FI + 32 * (b / FJ) + 4 * lh, n = tc.n0 + wn * 32 * FJ + 32 * (b % FJ) + lr;
    epi16<RES>(p, tc.r_base, mf, n, x);
#pragma unroll
    for (int vg = 0; vg < 4; ++vg) {
      const uint32_t mb = mf + 8 * vg;
      if (n >= p.N || mb >= p.M) continue;
      if (p.cmode == 2) {
        const int32_t o = tc.c_base + row_off(p, mb, p.c_m1, p.c_m2) + (int32_t)n * p.c_n;
        *(float4*)(C + o) = make_float4(x[4 * vg], x[4 * vg + 1], x[4 * vg + 2], x[4 * vg + 3]);
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const uint32_t m = mb + t;
          if (m < p.M) C[tc.c_base + row_off(p, m, p.c_m1, p.c_m2) + (int32_t)n * p.c_n] = x[4 * vg + t];
        }
      }
    }
  }
}

template <int BM, int BN, int WM, int WN, int KS, int ST>
hipError_t split_go(const NodeKernel& k, hipStream_t s) {
  const GemmParams& p = k.gemm;
  const dim3 grid(p.tiles_m * p.tiles_n * p.G);
#define FLUID_FS(AKv, BKv)                                                                                    \
  do {                                                                                                        \
    if (p.rop)                                                                                                \
      hipLaunchKernelGGL((gemm_f32_split_kernel<BM, BN, WM, WN, KS, ST, AKv, BKv, true>), grid,                   \
                         dim3(64 * WM * WN * KS), 0, s, p);                                                   \
    else                                                                                                      \
      hipLaunchKernelGGL((gemm_f32_split_kernel<BM, BN, WM, WN, KS, ST, AKv, BKv, false>), grid,                  \
                         dim3(64 * WM * WN * KS), 0, s, p);                                                   \
  } while (0)
  const bool ak = k.amode == GM_K, bk = k.bmode == GM_K;
  if (ak && bk) FLUID_FS(true, true);
  else if (ak) FLUID_FS(true, false);
  else if constexpr (BM == 128) {
    if (bk) FLUID_FS(false, true);
    else FLUID_FS(false, false);
  } else return hipErrorInvalidValue;
#undef FLUID_FS
  return hipGetLastError();
}

hipError_t launch_gemm_f32_split(const NodeKernel& k, hipStream_t s) {
  if (k.dtype != DT_F32 || (k.amode != GM_K && k.amode != GM_MN) || (k.bmode != GM_K && k.bmode != GM_MN) ||
      (k.gemm_tile != 8 && k.gemm_tile != 9))
    return hipErrorInvalidValue;
  return k.gemm_tile == 8 ? split_go<256, 128, 4, 2, 1, 2>(k, s) : split_go<128, 128, 2, 2, 2, 1>(k, s);
}

}  // namespace fluid
