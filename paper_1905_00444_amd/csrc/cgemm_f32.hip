// FP32 complex GEMM on MFMA for every shape, C[m][n] = sum_k A(m, k) B(n, k) (paper Sec. III-E, the
// "G" of transpose-GEMM-transpose; cgemm.hip describes the real embedding and the renormalisation).
//
// Bound by the matrix cores (v_mfma_f32_16x16x4_f32: 32 cycles for 2048 flop), or by HBM where N and K are
// short.  Measured counters say that VALU instructions take their cycles from FP32 MFMAs (busy cycles of
// the two add up to the time), so the layout leaves the loop next to none:
//   * 16 complex columns take two MFMA tiles, one that multiplies (br, -bi) and gives the real parts, one
//     that multiplies (bi, br) and gives the imaginary parts.  Both read the same registers of B, the only
//     arithmetic is the sign of bi, and a lane ends up with whole complex results: an epilogue without
//     exchanges whose stores are full 128-byte lines.
//   * The sum over k may run in any order, so MFMA s of a K-step of 16 complex takes in lane group lg the
//     real k = 16 (s / 4) + 4 lg + s % 4: a lane's operands of four MFMAs are 16 contiguous bytes of its row,
//     and the four lane groups read 64 contiguous bytes of each row, in LDS or HBM.
//
// Tiles are staged in LDS, [row][k] with rows of 16 complex padded to 36 dwords (the 16-byte reads of 8
// rows cover all banks once); either operand may lie in HBM with k or with its row index contiguous.  Two
// LDS stages, operands fetched two K-tiles ahead, one barrier per K-tile.  Waves that wait at a barrier, for
// LDS or to issue a load issue no MFMA, so many small workgroups that run apart beat few large ones:
// 8192^3 runs at 140 TFLOP/s on 64 x 32 tiles (five workgroups per CU), 141 on 64 x 64 (four), 135 on
// 128 x 64 (two) and 137 on 256 x 128 (one).  Loading operands straight into MFMA registers, without LDS or
// barriers, gave 104 to 135.
//
// EDGE instances take any M, N and K: rows and columns past the end read as zeros and are not stored.
//
// Every accumulator receives its products in the same order in all tiles: a result does not depend on the
// tile that a launch picks, so the choice may follow the batch.  K is cut into chunks (gridDim.y > 1) by
// the shape alone.
//
// Measured (MI355X, before / here): 1500 x 700 x 300 1.27 ms as one thread per output, 42 us; 256^3 products of a
// 4 x 4 circuit in launches of 64 chains 331 us (two 256 x 128 tiles, K split in four), 70 us in one pass over
// K; 64 products of 2^15 x 64 x 64 785 us on 128 x 64 tiles, 619 (111 TFLOP/s, 3.5 TB/s); four slices of the
// 7x7 (1+32+1) circuit 442 and 388 ms.  The large ones (K >= 128) have since gone to cgemm_f32s.hip.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <algorithm>
#include <type_traits>
#include "cgemm_f32.h"

namespace qf {

constexpr int kFRow = 36;      // dwords per LDS row

// A thread's pairs into a tile of [row][k].
template <int T, class Loader>
__device__ __forceinline__ void f32_stage(float* lds, const Loader& l) {
  l.each([&](int row, int k, float4 v) {
    float* d = lds + row * kFRow + 2 * k;
    if constexpr (T == 0) {
      *reinterpret_cast<float4*>(d) = v;
    } else {
      *reinterpret_cast<float2*>(d) = make_float2(v.x, v.y);
      *reinterpret_cast<float2*>(d + kFRow) = make_float2(v.z, v.w);
    }
  });
}

// Accumulators of 16 rows x 16 complex columns: element r of lane (l16, lg) is row 4 r + lg of column l16
// (MFMA row 4 lg + r: A's rows are read in that order), so one store instruction writes four neighbouring
// rows, which under an output map are contiguous memory.
struct F32Acc {
  f4 re, im;
  __device__ __forceinline__ float2 at(int r) const { return make_float2(re[r], im[r]); }
};

template <int TM, int TN>
__device__ __forceinline__ void f32_zero(F32Acc (&acc)[TM][TN]) {
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j].re = acc[i][j].im = (f4){0.f, 0.f, 0.f, 0.f};
}

// The products of half a K-step: a[i] and b[j] hold this lane's 16 bytes (2 complex) of row / column l16.
template <int TM, int TN, bool CONJ>
__device__ __forceinline__ void f32_multiply(const f4 (&a)[TM], const f4 (&b)[TN], F32Acc (&acc)[TM][TN]) {
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      // real row s & 1 of [[br, bi], [-bi, br]] (conjugated: [[br, -bi], [bi, br]])
      const float own = b[j][s], other = b[j][s ^ 1];
      const float p = ((s & 1) && !CONJ) ? -own : own;
      const float q = (!(s & 1) && CONJ) ? -other : other;
#pragma unroll
      for (int i = 0; i < TM; ++i)
        acc[i][j].re = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][s], p, acc[i][j].re, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < TM; ++i)
        acc[i][j].im = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][s], q, acc[i][j].im, 0, 0, 0);
    }
}

template <int WM, int WN, int TM, int TN>
struct F32Tile {
  static constexpr int threads = 64 * WM * WN, BM = 16 * WM * TM, BN = 16 * WN * TN;
  static constexpr int stage = (BM + BN) * kFRow;  // dwords
};

template <int WM, int WN, int TM, int TN, int TA, int TB, bool CONJ, bool EDGE, bool GA, bool GB>
__global__ void __launch_bounds__(64 * WM * WN)
cgemm_f32(F32Args g) {
  using Tile = F32Tile<WM, WN, TM, TN>;
  constexpr int BM = Tile::BM, BN = Tile::BN, NTH = Tile::threads;
  __shared__ __attribute__((aligned(16))) float lds[2 * Tile::stage];

  const int64_t tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
  const F32Place at = f32_place(blockIdx.x, (uint32_t)tiles_m, (uint32_t)tiles_n, gridDim.x, BM, BN);
  const int64_t m0 = at.m0, n0 = at.n0, batch = at.batch;
  const bool partial = gridDim.y > 1;
  const int64_t k0 = blockIdx.y * g.kc;
  const int64_t klen = EDGE ? (g.K - k0 < g.kc ? g.K - k0 : g.kc) : g.kc;
  float2* C = partial ? g.P + ((int64_t)blockIdx.y * g.batch + batch) * g.M * g.N : g.C + batch * g.sc;

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = (wave / WN) * (16 * TM), wc = (wave % WN) * (16 * TN);
  const int l16 = lane & 15, lg = lane >> 4;

  const float2* A = g.A + (g.ma.on ? map_base(g.ma, batch, g.sa) : batch * g.sa);
  const float2* B = g.B + (g.mb.on ? map_base(g.mb, batch, g.sb) : batch * g.sb);
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
  Renorm rn = renorm_of(g.rn, batch);
  if (!partial) {
    float s0, s1;
    renorm_begin<P_FP32>(rn, nullptr, nullptr, m0 == 0 && n0 == 0, s0, s1, unscale);
  }

  F32Acc acc[TM][TN];
  f32_zero(acc);

  const int nk = (int)((klen + kFBK - 1) / kFBK);
  auto fetch = [&](int t) {
    if constexpr (GA) la.load_gather((int64_t)t * kFBK, g.ma);
    else la.load((int64_t)t * kFBK, g.lda, ml, klen, g.amap);
    if constexpr (GB) lb.load_gather((int64_t)t * kFBK, g.mb);
    else lb.load((int64_t)t * kFBK, g.ldb, nl, klen, g.amap);
  };
  auto stage = [&](int t) {
    float* st = lds + (t & 1) * Tile::stage;
    f32_stage<TA>(st, la);
    f32_stage<TB>(st + BM * kFRow, lb);
  };
  fetch(0);
  stage(0);
  if (nk > 1) fetch(1);
  __syncthreads();
  for (int t = 0; t < nk; ++t) {
    const float* LA = lds + (t & 1) * Tile::stage + (wr + 4 * (l16 & 3) + (l16 >> 2)) * kFRow + 4 * lg;
    const float* LB = lds + (t & 1) * Tile::stage + (BM + wc + l16) * kFRow + 4 * lg;
    f4 a[2][TM], b[2][TN];
    auto read = [&](int h) {
#pragma unroll
      for (int i = 0; i < TM; ++i) a[h][i] = *reinterpret_cast<const f4*>(LA + 16 * i * kFRow + 16 * h);
#pragma unroll
      for (int j = 0; j < TN; ++j) b[h][j] = *reinterpret_cast<const f4*>(LB + 16 * j * kFRow + 16 * h);
    };
    read(0);
    if (t + 1 < nk) {  // staged and fetched under this tile's products
      stage(t + 1);
      if (t + 2 < nk) fetch(t + 2);
    }
    read(1);
    f32_multiply<TM, TN, CONJ>(a[0], b[0], acc);
    f32_multiply<TM, TN, CONJ>(a[1], b[1], acc);
    __syncthreads();
  }

  if (partial) rn.om_nh = 0;
  const uint32_t seen = partial ? 0u : seen_amax(rn);
  const float mx = f32_store<TM, TN, EDGE>(C, rn, m0 + wr, n0 + wc, g.M, g.N, unscale, acc);
  if (rn.c && !partial) raise_amax<WM * WN>(rn.c, mx, seen, lds);
}

template <int WM, int WN, int TM, int TN, int TA, int TB, bool CONJ>
static hipError_t f32_launch(hipStream_t st, const F32Args& g, int split) {
  using Tile = F32Tile<WM, WN, TM, TN>;
  const int64_t tiles = ((g.M + Tile::BM - 1) / Tile::BM) * ((g.N + Tile::BN - 1) / Tile::BN) * g.batch;
  if (!grid_takes(tiles, Tile::threads)) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)tiles, (unsigned)split), block(Tile::threads);
  // whole tiles and pairs of elements that never straddle a row's end
  const bool whole = g.M % Tile::BM == 0 && g.N % Tile::BN == 0 && g.kc % kFBK == 0 && g.kc * split == g.K;
  auto run = [&](auto* kernel) {
    hipLaunchKernelGGL(kernel, grid, block, 0, st, g);
    return hipGetLastError();
  };
  if constexpr (TA == 0 && TB == 0 && !CONJ) {
    if (g.ma.on == 1 && g.mb.on == 1) return run(cgemm_f32<WM, WN, TM, TN, 0, 0, false, false, true, true>);
    if (g.ma.on == 1) return run(cgemm_f32<WM, WN, TM, TN, 0, 0, false, false, true, false>);
    if (g.mb.on == 1) return run(cgemm_f32<WM, WN, TM, TN, 0, 0, false, false, false, true>);
  }
  if (whole) return run(cgemm_f32<WM, WN, TM, TN, TA, TB, CONJ, false, false, false>);
  return run(cgemm_f32<WM, WN, TM, TN, TA, TB, CONJ, true, false, false>);
}

// Tile of a launch: 64 x 64 where that gives every CU its four workgroups (4096^3: 140 against 138 TFLOP/s
// on 64 x 32 tiles, 2^20 x 256 x 256: 135 / 131, 2^21 x 64 x 64: 105 / 103), else the largest that still
// gives the 256 CUs a workgroup each.  Thin products (N <= 16) get the tiles of that width: a wider tile
// would multiply zeros.
template <int TA, int TB, bool CONJ>
static hipError_t f32_pick(hipStream_t st, const F32Args& g, int split, int want) {
  auto blocks = [&](int64_t bm, int64_t bn) { return ((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn) * g.batch * split; };
  int tile = want;
  if (tile == F32_AUTO || tile == F32_PLAIN) {
    if (g.N <= 16) tile = g.M >= 128 && blocks(128, 16) >= 256 ? F32_128X16 : F32_32X16;
    else if (g.M >= 64 && g.N >= 64 && blocks(64, 64) >= 1024) tile = F32_64X64;
    else if (g.M >= 64 && blocks(64, 32) >= 256) tile = F32_64X32;
    else tile = F32_32X32;
  }
  switch (tile) {
    case F32_64X64: return f32_launch<2, 2, 2, 2, TA, TB, CONJ>(st, g, split);
    case F32_64X32: return f32_launch<2, 2, 2, 1, TA, TB, CONJ>(st, g, split);
    case F32_128X16: return f32_launch<4, 1, 2, 1, TA, TB, CONJ>(st, g, split);
    case F32_32X16: return f32_launch<2, 1, 1, 1, TA, TB, CONJ>(st, g, split);
    default: return f32_launch<2, 2, 1, 1, TA, TB, CONJ>(st, g, split);
  }
}

static hipError_t f32_args(F32Args& g, int64_t M, int64_t N, int64_t K, const float2* A, const float2* B, float2* C,
                           int64_t batch, int64_t sa, int64_t sb, int64_t sc, const Renorm& rn, int* split, float2* P) {
  if (M < 1 || N < 1 || K < 1 || batch < 1 || *split < 1) return hipErrorInvalidValue;
  g.M = M; g.N = N; g.K = K;
  g.A = A; g.B = B; g.C = C;
  g.batch = batch; g.sa = sa; g.sb = sb; g.sc = sc;
  g.kc = *split > 1 ? ((K + *split - 1) / *split + kFBK - 1) / kFBK * kFBK : K;
  *split = (int)((K + g.kc - 1) / g.kc);  // whole K-tiles per chunk: every chunk holds some of K
  g.P = P;
  g.rn = rn;
  return hipSuccess;
}

hipError_t launch_cgemm_f32(hipStream_t st, int64_t M, int64_t N, int64_t K, const float2* A, const float2* B,
                            float2* C, int64_t batch, int64_t sa, int64_t sb, int64_t sc, const Renorm& rn, int* split,
                            float2* P, int tile, const OpMap* ma, const OpMap* mb) {
  F32Args g;
  if (ma) g.ma = *ma;
  if (mb) g.mb = *mb;
  const hipError_t e = f32_args(g, M, N, K, A, B, C, batch, sa, sb, sc, rn, split, P);
  if (e != hipSuccess) return e;
  g.lda = K;
  g.ldb = K;
  if (tile == F32_AUTO && f32s_takes(M, N, K)) return launch_f32s(st, g, *split, false, false);
  return f32_pick<0, 0, false>(st, g, *split, tile);
}

hipError_t launch_cgemm_f32_env(hipStream_t st, int side, int64_t M, int64_t N, int64_t K, const float2* env,
                                const float2* other, float2* out, int64_t batch, const Renorm& map, int* split,
                                float2* P, bool plain) {
  // out[rows][K] = sum over the other index of env and conj(other): rows = M (side 0) or N (side 1)
  F32Args g;
  const int64_t rows = side ? N : M, sum = side ? M : N;
  const hipError_t e = f32_args(g, rows, K, sum, env, other, out, batch, M * N, sum * K, rows * K, Renorm{}, split, P);
  if (e != hipSuccess) return e;
  g.lda = N;  // env's plain row pitch
  g.ldb = K;
  g.amap = map;
  if (!plain && f32s_takes(g.M, g.N, g.K)) return launch_f32s(st, g, *split, true, side);
  return side ? f32_pick<1, 1, true>(st, g, *split, F32_AUTO) : f32_pick<0, 1, true>(st, g, *split, F32_AUTO);
}

} // namespace qf
