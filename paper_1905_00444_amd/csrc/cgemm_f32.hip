// FP32 complex GEMM on MFMA for every shape, C[m][n] = sum_k A(m, k) B(n, k) (paper Sec. III-E, the
// "G" of transpose-GEMM-transpose; cgemm.hip describes the real embedding and the renormalisation).
//
// One kernel template covers the 256 x 128 tile of the large contractions down to 32 x 16 and 128 x 8
// tiles for thin products.  v_mfma_f32_16x16x4_f32 takes 32 cycles for 2048 flop, so a wave needs one
// 4-byte LDS operand read per 32 MFMA-cycles and operand layout is free: LDS tiles are [row][k] with
// rows of 16 complex plus 8 bytes (34 dwords, 2 mod 32), which lands the 16 rows x 2 dwords of an
// operand read in distinct banks, and either operand may lie in HBM with k or with its row index
// contiguous (the transposition happens in the LDS store).  Two LDS stages, operands fetched two K-tiles
// ahead into registers, one barrier per K-tile of 16 complex.
//
// Every accumulator receives its products in the order of k, four reals (two complex) per MFMA,
// whatever the tile: a result does not depend on the tile that a launch picks, so the choice may
// follow the batch.  K is cut into chunks (gridDim.y > 1) by the shape alone.
//
// Measured (whole passes, MI355X): 1500 x 700 x 300 1.27 ms as one thread per output, 42 us here; the
// 256^3 products of a 4 x 4 circuit in launches of 64 chains 332 us (two 256 x 128 tiles, K split in four)
// against 60 us on 128 x 64 tiles; 2^20 x 16 x 256 4.7 ms as one thread per output, 0.5 ms on 128 x 16.
//
// EDGE instances take any M, N and K: rows and columns past the end read as zeros and are not stored.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <algorithm>
#include "cgemm_common.h"

namespace qf {

constexpr int kFBK = 16;       // complex k per K-tile
constexpr int kFRow = 34;      // dwords per LDS row

struct F32Args {
  int64_t M, N, K;
  const float2* A;
  const float2* B;
  float2* C;
  int64_t lda, ldb;      // elements between rows (k contiguous) or between k's (row index contiguous)
  int64_t sa, sb, sc;    // batch strides
  int64_t kc;            // k per chunk
  float2* P;             // partial tiles [chunk][batch][M][N] when gridDim.y > 1
  int conj_b;
  Renorm rn;
};

// Loads of one operand tile (ROWS x 16 complex) into registers: pairs of neighbours along the
// contiguous index.  T = 0: k contiguous, 8 threads per row; T = 1: rows contiguous.
template <int ROWS, int NTH, int T, bool EDGE>
struct F32Loader {
  static constexpr int pairs = ROWS * kFBK / 2;
  static constexpr int per = (pairs + NTH - 1) / NTH;
  static constexpr bool partial = pairs % NTH != 0;
  const float2* p[per];
  int row[per], k[per];   // of the pair's first element
  float4 r[per];

  __device__ __forceinline__ void init(const float2* base, int64_t ld, int64_t k0) {
#pragma unroll
    for (int i = 0; i < per; ++i) {
      const int id = (int)threadIdx.x + i * NTH;
      if constexpr (T == 0) {
        row[i] = id >> 3;
        k[i] = 2 * (id & 7);
        p[i] = base + row[i] * ld + k0 + k[i];
      } else {
        row[i] = 2 * (id % (ROWS / 2));
        k[i] = id / (ROWS / 2);
        p[i] = base + (k0 + k[i]) * ld + row[i];
      }
    }
  }
  // Tile at kt (k relative to the chunk); rows_left / k_left: elements that exist (EDGE).
  __device__ __forceinline__ void load(int64_t kt, int64_t ld, int64_t rows_left, int64_t k_left) {
#pragma unroll
    for (int i = 0; i < per; ++i) {
      if (partial && (int)threadIdx.x + i * NTH >= pairs) continue;
      const float2* q = p[i] + (T == 0 ? kt : kt * ld);
      if constexpr (!EDGE) {
        r[i] = *reinterpret_cast<const float4*>(q);
      } else {
        const int64_t kk = kt + k[i];
        const bool first = row[i] < rows_left && kk < k_left;
        const bool second = T == 0 ? row[i] < rows_left && kk + 1 < k_left : row[i] + 1 < rows_left && kk < k_left;
        float2 a = make_float2(0.f, 0.f), b = a;
        if (first) a = q[0];
        if (second) b = q[1];
        r[i] = make_float4(a.x, a.y, b.x, b.y);
      }
    }
  }
  __device__ __forceinline__ void store(float* lds) const {
#pragma unroll
    for (int i = 0; i < per; ++i) {
      if (partial && (int)threadIdx.x + i * NTH >= pairs) continue;
      float* d = lds + row[i] * kFRow + 2 * k[i];
      *reinterpret_cast<float2*>(d) = make_float2(r[i].x, r[i].y);
      *reinterpret_cast<float2*>(d + (T == 0 ? 2 : kFRow)) = make_float2(r[i].z, r[i].w);
    }
  }
};

template <int WM, int WN, int TM, int TN>
struct F32Tile {
  static constexpr int threads = 64 * WM * WN, BM = 16 * WM * TM, BN = 8 * WN * TN;
  static constexpr int stage = (BM + BN) * kFRow;  // dwords
};

template <int WM, int WN, int TM, int TN, int TA, int TB, bool EDGE>
__global__ void __launch_bounds__(64 * WM * WN)
cgemm_f32(F32Args g) {
  using Tile = F32Tile<WM, WN, TM, TN>;
  constexpr int BM = Tile::BM, BN = Tile::BN, NTH = Tile::threads;
  __shared__ __attribute__((aligned(16))) float lds[2 * Tile::stage];

  // consecutive tiles on one XCD (8 XCDs, dealt round-robin), rasterised in groups of row tiles
  const int64_t tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
  const int64_t ntiles = tiles_m * tiles_n;
  int64_t bid = blockIdx.x;
  if ((ntiles & 7) == 0) bid = (bid & 7) * (ntiles >> 3) + (bid >> 3);
  const int64_t group = BM >= 256 ? 4 : 8;
  const int64_t per_group = group * tiles_n;
  const int64_t first_m = bid / per_group * group;
  const int64_t gsize = (tiles_m - first_m) < group ? (tiles_m - first_m) : group;
  const int64_t m0 = (first_m + (bid % per_group) % gsize) * BM;
  const int64_t n0 = (bid % per_group) / gsize * BN;

  const int64_t batch = blockIdx.z;
  const bool partial = gridDim.y > 1;
  const int64_t k0 = blockIdx.y * g.kc;
  const int64_t klen = EDGE ? (g.K - k0 < g.kc ? g.K - k0 : g.kc) : g.kc;
  float2* C = partial ? g.P + ((int64_t)blockIdx.y * gridDim.z + batch) * g.M * g.N : g.C + batch * g.sc;

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wr = (wave / WN) * (16 * TM), wc = (wave % WN) * (8 * TN);
  const int l16 = lane & 15, lg = lane >> 4, q = l16 & 1;
  // A: dword 4s + lg of its row.  B: entry (part, q) of [[br, bi], [-bi, br]], part = lg & 1: chosen by
  // address, the sign flipped where the entry is -bi (or, conjugated, where it is bi)
  const int b_word = 2 * (lg >> 1) + ((lg & 1) ^ q);
  const int part = lg & 1;
  const uint32_t b_flip = (part != q && (g.conj_b ? q == 1 : q == 0)) ? 0x80000000u : 0u;

  F32Loader<BM, NTH, TA, EDGE> la;
  F32Loader<BN, NTH, TB, EDGE> lb;
  la.init(g.A + batch * g.sa + (TA == 0 ? m0 * g.lda : m0), g.lda, k0);
  lb.init(g.B + batch * g.sb + (TB == 0 ? n0 * g.ldb : n0), g.ldb, k0);
  const int64_t ml = g.M - m0, nl = g.N - n0;

  float unscale = 1.f;
  if (!partial) {
    float s0, s1;
    renorm_begin<P_FP32>(g.rn, nullptr, nullptr, s0, s1, unscale);
  }

  f4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = (f4){0.f, 0.f, 0.f, 0.f};

  const int nk = (int)((klen + kFBK - 1) / kFBK);
  auto fetch = [&](int t) {
    la.load((int64_t)t * kFBK, g.lda, ml, klen);
    lb.load((int64_t)t * kFBK, g.ldb, nl, klen);
  };
  auto stage = [&](int t) {
    float* st = lds + (t & 1) * Tile::stage;
    la.store(st);
    lb.store(st + BM * kFRow);
  };
  fetch(0);
  stage(0);
  if (nk > 1) fetch(1);
  __syncthreads();
  for (int t = 0; t < nk; ++t) {
    const float* LA = lds + (t & 1) * Tile::stage + (wr + l16) * kFRow + lg;
    const float* LB = lds + (t & 1) * Tile::stage + (BM + wc + (l16 >> 1)) * kFRow + b_word;
#pragma unroll 2
    for (int s = 0; s < kFBK / 2; ++s) {
      float a[TM];
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = LA[16 * i * kFRow + 4 * s];
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const float b = __uint_as_float(__float_as_uint(LB[8 * j * kFRow + 4 * s]) ^ b_flip);
#pragma unroll
        for (int i = 0; i < TM; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b, acc[i][j], 0, 0, 0);
      }
    }
    if (t + 1 < nk) {
      stage(t + 1);
      if (t + 2 < nk) fetch(t + 2);
    }
    __syncthreads();
  }

  // lane holds real column (n, q) for rows 4 lg .. 4 lg + 3 of each tile; the partner lane (l ^ 1)
  // holds the other part, and after the exchange each lane owns two complex results
  float mx = 0.f;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const f4 v = acc[i][j] * unscale;
      const float s0 = q ? v[0] : v[2], s1 = q ? v[1] : v[3];
      const float r0 = __shfl_xor(s0, 1), r1 = __shfl_xor(s1, 1);
      const int64_t row = m0 + wr + 16 * i + 4 * lg + (q ? 2 : 0);
      const int64_t col = n0 + wc + 8 * j + (l16 >> 1);
      float2 o0, o1;
      if (q) { o0 = make_float2(r0, v[2]); o1 = make_float2(r1, v[3]); }
      else { o0 = make_float2(v[0], r0); o1 = make_float2(v[1], r1); }
      if (!EDGE || (row < g.M && col < g.N)) C[partial ? row * g.N + col : c_index(g.rn, row, col, g.N)] = o0;
      if (!EDGE || (row + 1 < g.M && col < g.N))
        C[partial ? (row + 1) * g.N + col : c_index(g.rn, row + 1, col, g.N)] = o1;
      mx = fmaxf(mx, fmaxf(cmax(o0), cmax(o1)));  // zeros past the edge
    }
  if (g.rn.c && !partial) record_amax(g.rn.c, mx);
}

template <int WM, int WN, int TM, int TN, int TA, int TB>
static void f32_launch(hipStream_t st, const F32Args& g, int64_t batch, int split) {
  using Tile = F32Tile<WM, WN, TM, TN>;
  const int64_t tiles = ((g.M + Tile::BM - 1) / Tile::BM) * ((g.N + Tile::BN - 1) / Tile::BN);
  const dim3 grid((unsigned)tiles, (unsigned)split, (unsigned)batch), block(Tile::threads);
  // whole tiles and pairs of elements that never straddle a row's end
  const bool whole = g.M % Tile::BM == 0 && g.N % Tile::BN == 0 && g.kc % kFBK == 0 && g.kc * split == g.K;
  if (whole)
    hipLaunchKernelGGL((cgemm_f32<WM, WN, TM, TN, TA, TB, false>), grid, block, 0, st, g);
  else
    hipLaunchKernelGGL((cgemm_f32<WM, WN, TM, TN, TA, TB, true>), grid, block, 0, st, g);
}

// Tile of a launch.  The larger the tile, the fewer operand reads per product (a 256 x 128 tile reads
// each operand element from LDS for 64 to 128 outputs), so the largest one is taken that still gives the
// 256 CUs a workgroup each; below that, smaller tiles spread the launch.  Thin products (N <= 16) get
// the tiles of their width: a wider tile would multiply zeros.
template <int TA, int TB>
static void f32_pick(hipStream_t st, const F32Args& g, int64_t batch, int split, int want) {
  auto blocks = [&](int64_t bm, int64_t bn) { return ((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn) * batch * split; };
  int tile = want;
  if (tile == F32_AUTO) {
    if (g.N <= 8 && g.M >= 128) tile = F32_128X8;
    else if (g.N <= 16) tile = g.M >= 128 && blocks(128, 16) >= 256 ? F32_128X16 : F32_32X16;
    else if (g.M >= 256 && g.N >= 128 && blocks(256, 128) >= 256) tile = F32_256X128;
    else if (g.M >= 128 && g.N >= 64 && blocks(128, 64) >= 256) tile = F32_128X64;
    else if (g.M >= 64 && blocks(64, 32) >= 256) tile = F32_64X32;
    else tile = F32_32X32;
  }
  switch (tile) {
    case F32_256X128: f32_launch<4, 2, 4, 8, TA, TB>(st, g, batch, split); return;
    case F32_128X64: f32_launch<2, 2, 4, 4, TA, TB>(st, g, batch, split); return;
    case F32_64X32: f32_launch<2, 2, 2, 2, TA, TB>(st, g, batch, split); return;
    case F32_128X16: f32_launch<4, 1, 2, 2, TA, TB>(st, g, batch, split); return;
    case F32_128X8: f32_launch<4, 1, 2, 1, TA, TB>(st, g, batch, split); return;
    case F32_32X16: f32_launch<2, 1, 1, 2, TA, TB>(st, g, batch, split); return;
    default: f32_launch<2, 2, 1, 2, TA, TB>(st, g, batch, split); return;
  }
}

hipError_t launch_cgemm_f32(hipStream_t st, int64_t M, int64_t N, int64_t K, const float2* A, const float2* B,
                            float2* C, int64_t batch, int64_t sa, int64_t sb, int64_t sc, const Renorm& rn, int* split,
                            float2* P, int tile, int ta, int tb, int conj_b) {
  if (M < 1 || N < 1 || K < 1 || batch < 1 || *split < 1) return hipErrorInvalidValue;
  F32Args g;
  g.M = M; g.N = N; g.K = K;
  g.A = A; g.B = B; g.C = C;
  g.lda = ta ? M : K;
  g.ldb = tb ? N : K;
  g.sa = sa; g.sb = sb; g.sc = sc;
  g.kc = *split > 1 ? ((K + *split - 1) / *split + kFBK - 1) / kFBK * kFBK : K;
  *split = (int)((K + g.kc - 1) / g.kc);  // whole K-tiles per chunk: every chunk holds some of K
  g.P = P;
  g.conj_b = conj_b;
  g.rn = rn;
  if (ta == 0 && tb == 0) f32_pick<0, 0>(st, g, batch, *split, tile);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

} // namespace qf
