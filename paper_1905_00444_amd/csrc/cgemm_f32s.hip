// FP32 complex GEMM on the bfloat16 matrix cores, C[m][n] = sum_k A(m, k) B(n, k) (paper Sec. III-E, the "G"
// of transpose-GEMM-transpose), for products large enough that cgemm_f32.hip's FP32 MFMAs bound them.
//
// An FP32 number is the sum of three bfloat16 numbers, x = x0 + x1 + x2 (8 bits each, rounded to nearest, so
// |x1| <= 2^-9 |x| and |x2| <= 2^-18 |x|), and a bfloat16 MFMA multiplies 13 times faster than an FP32
// one.  x y is taken as x0 y0 + (x0 y1 + x1 y0) + (x1 y1 + x0 y2 + x2 y0); what is left out is below 2^-26 |x y|,
// a quarter of an FP32 product's own rounding.
//
// What the instruction does to its sums (probed): a lane group's 8 products are aligned to the largest and cut at
// 2^-24 of it, and the accumulator operand, where it is the smaller, as well and downwards.  A sum that is kept
// in the instruction therefore loses the remainder when large products cancel, and always on the same side: of
// amplitudes of 5x5 and 6x6 circuits of depth 32 with every CZ an identity, whose path sums cancel, the errors
// were seven and three times those of FP32 MFMAs.  So the product of the first planes starts from zero in every
// K-tile of 16 and is added with FP32 rounding, and A is negated in the middle half of K, which leaves no bias; the
// five small products keep accumulators in the instruction, 2^-8 below, which are negated there too.  Relative
// errors per amplitude there (rms; FP32 MFMAs / all sums in the instruction / here): 4x4 1.3e-6 / 1.1e-6 / 9e-7, 4x5
// 2.1e-6 / 1.9e-6 / 1.4e-6, 5x5 2.3e-6 / 1.7e-5 / 3.3e-6, 6x6 5.3e-6 / 1.7e-5 / 8.9e-6.  Of products, norm-wise: normal
// entries, 4096 x 1024 x 128, 3.2e-8 / 1.0e-8 / 7.6e-9, same-sign entries over 20 binades, K = 1024, 2.2e-7 / - / 5.9e-8.
// Callers who want FP32 MFMAs throughout have QF_PLAN_PLAIN_FP32 and the variant f32.  Products below K = 128 stay
// on FP32 MFMAs, where HBM is half of their time and six products gained least (2^15 x 64 x 64 by 64 619 us, 539 with
// all sums in the instruction).
//
// Bound by VALU issue beside the MFMAs (conversions: 11 instructions per complex element staged; the
// arrangement of B: 2 per element and plane read), so tiles are as large as the launch allows.
// Layout as in cgemm_f32.hip: 16 complex columns take two MFMA tiles, one that multiplies (br, -bi) and gives
// real parts, one that multiplies (bi, br); LDS holds three planes of [row][16 k], rows padded to 80 bytes.
//
// Operands are scaled by 2^20, so that all planes of any normal FP32 number are bfloat16 numbers.  Operands from
// 2^108 on, infinities and NaNs, and results from 2^88 on, leave sums that are not finite: a wave that sees
// one computes its results again as plain FP32 sums.
//
// Measured (MI355X, FP32 MFMAs / all sums in the instruction / here): 4096^3 140 / 238 / 231 TFLOP/s, 2^18 x 256 x 256
// 134 / 198 / 193, 64 products of 256^3 123 / 188 / 181, 16 of them 97 / 109 / 97; 1500 x 700 x 300 39 / 33 / 36 us, the 7x7
// slices 388 / 206 / 234 ms.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <algorithm>
#include <type_traits>
#include "cgemm_f32.h"

namespace qf {

constexpr int kSRow = 20;  // dwords per LDS row of a plane: 16 complex and padding
constexpr float kSScale = 0x1p20f;  // of both operands: the third plane of 2^-126 is then a bfloat16 number

// Accumulators of 16 rows x 16 complex columns (element order of F32Acc): the products of the first
// planes, and the small ones.
struct F32sAcc {
  f4 re, im, re_low, im_low;
  __device__ __forceinline__ float2 at(int r) const {
    constexpr float s = 1.f / (kSScale * kSScale);
    return make_float2((re[r] + re_low[r]) * s, (im[r] + im_low[r]) * s);
  }
};

// A thread's pairs into the three planes of a tile, ROWS kSRow dwords apart.
template <int T, int ROWS, class Loader>
__device__ __forceinline__ void f32s_stage(uint32_t* lds, const Loader& l, float scale) {
  l.each([&](int row, int k, float4 v) {
    uint32_t* d = lds + row * kSRow + k;
    v = make_float4(v.x * scale, v.y * scale, v.z * scale, v.w * scale);
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const uint32_t a = pack_bf16x2(v.x, v.y), b = pack_bf16x2(v.z, v.w);
      if constexpr (T == 0) {
        *reinterpret_cast<uint2*>(d + p * ROWS * kSRow) = make_uint2(a, b);
      } else {
        d[p * ROWS * kSRow] = a;
        d[p * ROWS * kSRow + kSRow] = b;
      }
      if (p < 2)
        v = make_float4(v.x - bf16_lo_to_f32(a), v.y - bf16_hi_to_f32(a), v.z - bf16_lo_to_f32(b),
                        v.w - bf16_hi_to_f32(b));
    }
  });
}

// The products of a K-tile: plane p of rows 16 i + (lane's) from pa, of columns 16 j + l16 from pb.  The product of
// the first planes is taken from zero and added here, times the sign that A was staged with.
template <int TM, int TN, int BM, int BN, bool CONJ>
__device__ __forceinline__ void f32s_multiply(const uint32_t* pa, const uint32_t* pb, float sign,
                                              F32sAcc (&acc)[TM][TN]) {
  u4 a[3][TM];
#pragma unroll
  for (int p = 0; p < 3; ++p)
#pragma unroll
    for (int i = 0; i < TM; ++i) a[p][i] = *reinterpret_cast<const u4*>(pa + (p * BM + 16 * i) * kSRow);
  auto product = [](const u4& x, const u4& y, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, x), __builtin_bit_cast(bf8, y), c, 0, 0, 0);
  };
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    u4 re[3], im[3];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const u4 b = *reinterpret_cast<const u4*>(pb + (p * BN + 16 * j) * kSRow);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        // (br, -bi) and (bi, br); conjugated: (br, bi) and (-bi, br)
        re[p][e] = CONJ ? b[e] : b[e] ^ 0x80000000u;
        im[p][e] = __builtin_amdgcn_alignbit(b[e], b[e], 16) ^ (CONJ ? 0x00008000u : 0u);
      }
    }
    constexpr int order[5][2] = {{2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}};
#pragma unroll
    for (int o = 0; o < 5; ++o) {
      const int p = order[o][0], q = order[o][1];
#pragma unroll
      for (int i = 0; i < TM; ++i) acc[i][j].re_low = product(a[p][i], re[q], acc[i][j].re_low);
#pragma unroll
      for (int i = 0; i < TM; ++i) acc[i][j].im_low = product(a[p][i], im[q], acc[i][j].im_low);
    }
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    f4 r[TM], m[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) r[i] = product(a[0][i], re[0], zero);
#pragma unroll
    for (int i = 0; i < TM; ++i) m[i] = product(a[0][i], im[0], zero);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc[i][j].re[e] = fmaf(sign, r[i][e], acc[i][j].re[e]);
        acc[i][j].im[e] = fmaf(sign, m[i][e], acc[i][j].im[e]);
      }
  }
}

// Whether the wave holds a result that is not finite.
template <int TM, int TN>
__device__ __forceinline__ bool f32s_out_of_range(const F32sAcc (&acc)[TM][TN]) {
  float z = 0.f;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float2 v = acc[i][j].at(r);
        z = fmaf(v.x, 0.f, z);
        z = fmaf(v.y, 0.f, z);
      }
  return __any(!(z == 0.f));
}

// The wave's results as plain FP32 sums over k0 .. k0 + klen - 1.
template <int TM, int TN, int TA, int TB, bool CONJ, bool MAPA, bool GA, bool GB>
__device__ __forceinline__ float f32s_plain(const F32Args& g, const float2* A, const float2* B, float2* C,
                                            const Renorm& rn, int64_t m, int64_t n, int64_t k0, int64_t klen,
                                            float unscale) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4;
  float mx = 0.f;
#pragma unroll 1
  for (int t = 0; t < TM * TN * 4; ++t) {
    const int64_t x = m + 16 * (t / (4 * TN)) + 4 * (t & 3) + lg, y = n + 16 * (t / 4 % TN) + l16;
    if (x >= g.M || y >= g.N) continue;
    float2 c = make_float2(0.f, 0.f);
#pragma unroll 1
    for (int64_t k = k0; k < k0 + klen; ++k) {
      float2 a, b;
      if constexpr (GB) b = B[map_row(g.mb, (uint32_t)y) | map_bits<12>((uint32_t)k, g.mb.k)];
      else b = TB == 0 ? B[y * g.ldb + k] : B[k * g.ldb + y];
      if constexpr (GA) a = A[map_row(g.ma, (uint32_t)x) | map_bits<12>((uint32_t)k, g.ma.k)];
      else if constexpr (MAPA) a = A[c_row(g.amap, TA == 0 ? x : k, g.lda) + c_col(g.amap, TA == 0 ? k : x)];
      else a = TA == 0 ? A[x * g.lda + k] : A[k * g.lda + x];
      if (CONJ) b.y = -b.y;
      c.x = fmaf(a.x, b.x, c.x);
      c.x = fmaf(-a.y, b.y, c.x);
      c.y = fmaf(a.x, b.y, c.y);
      c.y = fmaf(a.y, b.x, c.y);
    }
    c = make_float2(c.x * unscale, c.y * unscale);
    C[c_index(rn, x, y, g.N)] = c;
    mx = fmaxf(mx, cmax(c));
  }
  return mx;
}

template <int WM, int WN, int TM, int TN>
struct F32sTile {
  static constexpr int threads = 64 * WM * WN, BM = 16 * WM * TM, BN = 16 * WN * TN;
  static constexpr int dwords = 3 * (BM + BN) * kSRow;
  // Two LDS stages and one barrier per K-tile where few workgroups fit a CU anyway: 128 x 128 tiles on 2^18 x 256 x
  // 256 718 -> 682 us, 4096^3 2.41 -> 2.34 ms; 64 x 64 tiles lose an overlapping workgroup by it (1024^3 61 -> 63 us).
  static constexpr int stages = BM * BN >= 128 * 128 ? 2 : 1;
};

template <int WM, int WN, int TM, int TN, int TA, int TB, bool CONJ, bool EDGE, bool GA, bool GB>
__global__ void __launch_bounds__(64 * WM * WN)
cgemm_f32s(F32Args g) {
  using Tile = F32sTile<WM, WN, TM, TN>;
  constexpr int BM = Tile::BM, BN = Tile::BN, NTH = Tile::threads;
  __shared__ __attribute__((aligned(16))) uint32_t lds[Tile::stages * Tile::dwords];

  const uint32_t tiles_m = (uint32_t)((g.M + BM - 1) / BM), tiles_n = (uint32_t)((g.N + BN - 1) / BN);
  const F32Place at = f32_place(blockIdx.x, tiles_m, tiles_n, gridDim.x, BM, BN);
  const int64_t m0 = at.m0, n0 = at.n0;
  const bool partial = gridDim.y > 1;
  const int64_t k0 = blockIdx.y * g.kc;
  const int64_t klen = EDGE ? (g.K - k0 < g.kc ? g.K - k0 : g.kc) : g.kc;
  const float2* A = g.A + (g.ma.on ? map_base(g.ma, at.batch, g.sa) : at.batch * g.sa);
  const float2* B = g.B + (g.mb.on ? map_base(g.mb, at.batch, g.sb) : at.batch * g.sb);
  float2* C = partial ? g.P + ((int64_t)blockIdx.y * g.batch + at.batch) * g.M * g.N : g.C + at.batch * g.sc;

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = (wave / WN) * (16 * TM), wc = (wave % WN) * (16 * TN);
  const int l16 = lane & 15, lg = lane >> 4;

  constexpr bool MAPA = TB == 1;
  std::conditional_t<GA, F32Gather<BM, NTH>, F32Loader<BM, NTH, TA, EDGE, MAPA>> la;
  std::conditional_t<GB, F32Gather<BN, NTH>, F32Loader<BN, NTH, TB, EDGE, false>> lb;
  if constexpr (GA) la.init_gather(A, g.ma, m0, k0);
  else if constexpr (MAPA) la.init_map(A, m0, k0);
  else la.init(A + (TA == 0 ? m0 * g.lda : m0), g.lda, k0);
  if constexpr (GB) lb.init_gather(B, g.mb, n0, k0);
  else lb.init(B + (TB == 0 ? n0 * g.ldb : n0), g.ldb, k0);
  const int64_t ml = g.M - m0, nl = g.N - n0;  // rows and columns that exist from the tile's first on

  float unscale = 1.f;
  Renorm rn = renorm_of(g.rn, at.batch);
  if (!partial) {
    float s0, s1;
    renorm_begin<P_FP32>(rn, nullptr, nullptr, m0 == 0 && n0 == 0, s0, s1, unscale);
  }

  F32sAcc acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
      acc[i][j].re = acc[i][j].im = acc[i][j].re_low = acc[i][j].im_low = (f4){0.f, 0.f, 0.f, 0.f};

  const int nk = (int)((klen + kFBK - 1) / kFBK);
  auto fetch = [&](int t) {
    if constexpr (GA) la.load_gather((int64_t)t * kFBK, g.ma);
    else la.load((int64_t)t * kFBK, g.lda, ml, klen, g.amap);
    if constexpr (GB) lb.load_gather((int64_t)t * kFBK, g.mb);
    else lb.load((int64_t)t * kFBK, g.ldb, nl, klen, g.amap);
  };
  auto stage_of = [&](int t) { return lds + (Tile::stages == 2 ? (t & 1) * Tile::dwords : 0); };
  const int first_turned = (nk + 3) / 4, last_turned = (3 * nk + 3) / 4;  // K-tiles with A negated
  auto turned = [&](int t) { return t >= first_turned && t < last_turned; };
  auto turn = [&] {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        acc[i][j].re_low = -acc[i][j].re_low;
        acc[i][j].im_low = -acc[i][j].im_low;
      }
  };
  auto stage = [&](int t) {
    f32s_stage<TA, BM>(stage_of(t), la, turned(t) ? -kSScale : kSScale);
    f32s_stage<TB, BN>(stage_of(t) + 3 * BM * kSRow, lb, kSScale);
  };
  fetch(0);
  if constexpr (Tile::stages == 2) {
    stage(0);
    if (nk > 1) fetch(1);
    __syncthreads();
  }
  // A loop over each part of K (A as it is, negated, as it is) rather than a test in one, around which the compiler
  // moves the accumulators of every K-tile.
  int t = 0;
#pragma unroll 1
  for (int part = 0; part < 3; ++part) {
    const int end = part == 0 ? first_turned : part == 1 ? last_turned : nk;
    const float sign = part == 1 ? -1.f : 1.f;
    if (part > 0) turn();
    for (; t < end; ++t) {
      if constexpr (Tile::stages == 1) {
        stage(t);
        __syncthreads();
        if (t + 1 < nk) fetch(t + 1);
      } else if (t + 1 < nk) {
        stage(t + 1);
        if (t + 2 < nk) fetch(t + 2);
      }
      const uint32_t* st = stage_of(t);
      f32s_multiply<TM, TN, BM, BN, CONJ>(st + (wr + 4 * (l16 & 3) + (l16 >> 2)) * kSRow + 4 * lg,
                                          st + (3 * BM + wc + l16) * kSRow + 4 * lg, sign, acc);
      __syncthreads();
    }
  }

  if (partial) rn.om_nh = 0;
  const uint32_t seen = partial ? 0u : seen_amax(rn);
  float mx;
  if (f32s_out_of_range<TM, TN>(acc))
    mx = f32s_plain<TM, TN, TA, TB, CONJ, MAPA, GA, GB>(g, A, B, C, rn, m0 + wr, n0 + wc, k0, klen, unscale);
  else
    mx = f32_store<TM, TN, EDGE>(C, rn, m0 + wr, n0 + wc, g.M, g.N, unscale, acc);
  if (rn.c && !partial) raise_amax<WM * WN>(rn.c, mx, seen, reinterpret_cast<float*>(lds));
}

template <int WM, int WN, int TM, int TN, int TA, int TB, bool CONJ>
static hipError_t f32s_launch(hipStream_t st, const F32Args& g, int split) {
  using Tile = F32sTile<WM, WN, TM, TN>;
  const int64_t tiles = ((g.M + Tile::BM - 1) / Tile::BM) * ((g.N + Tile::BN - 1) / Tile::BN) * g.batch;
  if (!grid_takes(tiles, Tile::threads)) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)tiles, (unsigned)split), block(Tile::threads);
  const bool whole = g.M % Tile::BM == 0 && g.N % Tile::BN == 0 && g.kc % kFBK == 0 && g.kc * split == g.K;
  auto run = [&](auto* kernel) {
    hipLaunchKernelGGL(kernel, grid, block, 0, st, g);
    return hipGetLastError();
  };
  if constexpr (TA == 0 && TB == 0 && !CONJ) {
    if (g.ma.on == 1 && g.mb.on == 1) return run(cgemm_f32s<WM, WN, TM, TN, 0, 0, false, false, true, true>);
    if (g.ma.on == 1) return run(cgemm_f32s<WM, WN, TM, TN, 0, 0, false, false, true, false>);
    if (g.mb.on == 1) return run(cgemm_f32s<WM, WN, TM, TN, 0, 0, false, false, false, true>);
  }
  if (whole) return run(cgemm_f32s<WM, WN, TM, TN, TA, TB, CONJ, false, false, false>);
  return run(cgemm_f32s<WM, WN, TM, TN, TA, TB, CONJ, true, false, false>);
}

// The largest tile that gives each of the 256 CUs a workgroup: 128 x 128 against 64 x 64 on 4096^3 2.34 / 2.67 ms,
// on 64 products of 256^3 44 / 50 us.  A result does not depend on the tile.
template <int TA, int TB, bool CONJ>
static hipError_t f32s_pick(hipStream_t st, const F32Args& g, int split) {
  auto blocks = [&](int64_t bm, int64_t bn) { return ((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn) * g.batch * split; };
  if (g.M >= 128 && g.N >= 128 && blocks(128, 128) >= 256) return f32s_launch<4, 2, 2, 4, TA, TB, CONJ>(st, g, split);
  if (blocks(64, 64) >= 256) return f32s_launch<2, 2, 2, 2, TA, TB, CONJ>(st, g, split);
  if (blocks(64, 32) >= 256) return f32s_launch<2, 2, 2, 1, TA, TB, CONJ>(st, g, split);
  return f32s_launch<2, 2, 1, 1, TA, TB, CONJ>(st, g, split);
}

// From 2^24 products on (256^3, where a single product is 7% slower and 64 of them 35% faster), and from 64
// rows and columns: half a tile of zeros costs more than the faster MFMAs bring.
bool f32s_takes(int64_t M, int64_t N, int64_t K) {
  return M >= 64 && N >= 64 && K >= 128 && (double)M * (double)N * (double)K >= (double)(1 << 24);
}

hipError_t launch_f32s(hipStream_t st, const F32Args& g, int split, bool env, bool side) {
  if (!env) return f32s_pick<0, 0, false>(st, g, split);
  return side ? f32s_pick<1, 1, true>(st, g, split) : f32s_pick<0, 1, true>(st, g, split);
}

} // namespace qf
