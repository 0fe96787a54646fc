// Complex GEMM, the "G" of the transpose-GEMM-transpose contraction (paper Sec. III-E):
//   C[m][n] = sum_k A[m][k] * B[n][k]   (complex64 in HBM; A and B both K-contiguous).
//
// The paper runs complex FP32 CGEMM on V100 CUDA cores.  On gfx950 the products run on MFMA
// through the real embedding of complex multiplication: with A viewed as a real M x 2K matrix
// (re, im interleaved, exactly its complex64 memory layout) and B expanded to a real 2K x 2N
// matrix whose 2x2 blocks are [[br, bi], [-bi, br]], the real product is C as a real M x 2N
// matrix, again (re, im) interleaved.  The expansion is never stored: each lane builds its
// B operand from the complex values in LDS by negating or swapping halves.  The algorithmic
// count 8 M N K of the paper's formula F = 8 sqrt(v0 v1 v2) equals the real MFMA work.
//
// Precisions (the operand conversion happens when a K-tile is staged into LDS):
//   FP32   : v_mfma_f32_16x16x4_f32 on the FP32 operands (cgemm_f32.hip); large products as six bfloat16
//            products (cgemm_f32s.hip).
//   BF16X3 : x = hi + lo with hi = bf16(x), lo = bf16(x - hi); C += hi*hi + hi*lo + lo*hi on
//            v_mfma_f32_16x16x32_bf16 with FP32 accumulation (the lo*lo term, about 2^-16
//            relative, is dropped).
//   FP16   : x * 2^s rounded to fp16 with s chosen from the operand's max magnitude so the
//            largest entry lands near 2^14; v_mfma_f32_16x16x32_f16, FP32 accumulation; the
//            epilogue multiplies by 2^-(sA+sB), which is exact.
//
// Renormalisation (paper Sec. III-E: normalise the inputs, renormalise at the end), done with
// powers of two so that it is exact: every stored tensor X carries a device-side exponent E_X
// (true values = stored * 2^E_X) and the max magnitude of its stored values.  A renormalised
// GEMM stores C * 2^-(e_A + e_B), e_X the binary exponent of X's max magnitude, so stored
// values stay near 1 whatever the true scale; E_C = E_A + E_B + e_A + e_B is written by one
// thread, C's max magnitude is gathered in the epilogue (one atomic max per workgroup), and the FP64
// slice sum applies 2^E of the root.
//
// Tiling: 256 threads = 4 waves as 2 x 2; a wave owns WTM x WTN MFMA tiles of 16 rows x 16 real
// columns (8 complex); block tile BM = 32 WTM rows x BN = 16 WTN complex columns; K-tiles of
// 32 complex.  Global loads for the next K-tile are issued into registers before the current
// tile's MFMAs, then converted and stored to LDS.  Rows are padded by 16 bytes in LDS.
// Workgroups are remapped so consecutive tiles of the launch share an XCD (8 XCDs, round-robin dispatch)
// and rasterised in groups of row-tiles for L2 reuse: 16 split-BF16 products of 256^3 take 16.2 us, 18.0 with
// each chain's tiles dealt to all XCDs.  K-tiles fetched three ahead instead of one: 17.0.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>
#include <algorithm>
#include <string>
#include "cgemm_f32.h"

namespace qf {

constexpr int kBK = 32;          // complex k per K-tile
constexpr int kThreads = 256;

__global__ void renorm_reset(NodeScale* c) {
  if (threadIdx.x < kScaleSlots) c[blockIdx.x].slot[threadIdx.x].amax = 0u;
}

hipError_t launch_renorm_reset(hipStream_t st, const Renorm& rn, int64_t batch) {
  hipLaunchKernelGGL(renorm_reset, dim3(rn.c_step ? (unsigned)batch : 1u), dim3(64), 0, st, rn.c);
  return hipGetLastError();
}

// Split-K launches (gridDim.y > 1): workgroup y contracts K-chunk y of length kc and writes its
// raw partial tile to P[y][batch][M][N]; cgemm_split_reduce sums the chunks in ascending order
// (deterministic) and applies the renormalisation.  A partial keeps only the FP16 operand scales
// (undone here); the renormalisation exponent is applied by the reduction.
template <int PREC>
__device__ __forceinline__ void scales_for(const Renorm& rn, const uint32_t* amaxA, const uint32_t* amaxB,
                                           bool partial, bool first, float& scale_a, float& scale_b, float& unscale) {
  if (!partial) {
    renorm_begin<PREC>(rn, amaxA, amaxB, first, scale_a, scale_b, unscale);
    return;
  }
  int s_a = 0, s_b = 0;
  if constexpr (PREC == P_FP16) {
    if (rn.c) {
      s_a = 14 - renorm_exp(rn.a);
      s_b = 14 - renorm_exp(rn.b);
    } else {
      s_a = fp16_shift(amaxA);
      s_b = fp16_shift(amaxB);
    }
  }
  scale_a = ldexpf(1.f, s_a);
  scale_b = ldexpf(1.f, s_b);
  unscale = ldexpf(1.f, -(s_a + s_b));
}

// Sum of the chunks in ascending order: a workgroup takes 32 consecutive outputs, its 8 groups of 32 lanes read
// whole 256-byte runs of 32 chunks at a time (four chunks' rows per group) into LDS, and the first group adds
// them.  Bound by reading the chunks once, or by latency where they are few (32 x 32 outputs of 64 chunks).
constexpr int kReduceOut = 32, kReduceGroups = 8, kReduceSlots = 32;

// A grid's z (the batch elements of P_z, C) where the elements keep scales of their own, else one z for all.
__global__ void __launch_bounds__(256)
cgemm_split_reduce(const float2* __restrict__ P, int split, int64_t batch, int64_t MN, int64_t N, int64_t sc,
                   float2* __restrict__ C, Renorm rn) {
  __shared__ float2 part[kReduceSlots][kReduceOut];
  float sa_, sb_, unscale;
  const int64_t chunk = batch * MN;
  if (rn.c_step) {
    rn = renorm_of(rn, blockIdx.z);
    P += blockIdx.z * MN;
    C += blockIdx.z * sc;
    batch = 1;
  }
  renorm_begin<P_FP32>(rn, nullptr, nullptr, blockIdx.x == 0, sa_, sb_, unscale);
  const int64_t total = batch * MN;
  const int lane = threadIdx.x % kReduceOut, t = threadIdx.x / kReduceOut;
  float mx = 0.f;
  for (int64_t i0 = (int64_t)blockIdx.x * kReduceOut; i0 < total; i0 += (int64_t)gridDim.x * kReduceOut) {
    const int64_t i = i0 + lane;
    float2 sum = make_float2(0.f, 0.f);
    for (int y0 = 0; y0 < split; y0 += kReduceSlots) {
      float2 v[kReduceSlots / kReduceGroups];
#pragma unroll
      for (int u = 0; u < kReduceSlots / kReduceGroups; ++u) {
        const int y = y0 + t + u * kReduceGroups;
        v[u] = i < total && y < split ? P[(int64_t)y * chunk + i] : make_float2(0.f, 0.f);
      }
#pragma unroll
      for (int u = 0; u < kReduceSlots / kReduceGroups; ++u) part[t + u * kReduceGroups][lane] = v[u];
      __syncthreads();
      if (t == 0) {
        const int n = split - y0 < kReduceSlots ? split - y0 : kReduceSlots;
#pragma unroll 8
        for (int k = 0; k < n; ++k) sum = make_float2(sum.x + part[k][lane].x, sum.y + part[k][lane].y);
      }
      __syncthreads();
    }
    if (t == 0 && i < total) {
      const float2 o = make_float2(sum.x * unscale, sum.y * unscale);
      const int64_t b = i / MN, e = i - b * MN, m = e / N;
      C[b * sc + c_index(rn, m, e - m * N, N)] = o;
      mx = fmaxf(mx, cmax(o));
    }
  }
  if (rn.c) record_amax(rn.c, mx);
}

template <int PREC>
struct LdsRow;  // bytes per complex element in LDS per plane
template <> struct LdsRow<P_BF16X3> { static constexpr int elem = 4, planes = 2; };
template <> struct LdsRow<P_FP16> { static constexpr int elem = 4, planes = 1; };

// Rows are read in 16-byte chunks and padded by 16 bytes.
template <int PREC, int ROWS>
struct TileLds {
  static constexpr int row_bytes = kBK * LdsRow<PREC>::elem + 16;
  static constexpr int plane_bytes = ROWS * row_bytes;
  static constexpr int bytes = plane_bytes * LdsRow<PREC>::planes;
};

// Stage ROWS x 32 complex (held as float4 = 2 complex per register) into LDS with conversion.
// Row of a thread's pair i and the pair's place in the row: pairs run along k, or (rows) along the rows.
template <int ROWS>
__device__ __forceinline__ void pair_of(int i, bool rows, int& row, int& c4) {
  const int idx = threadIdx.x + i * kThreads;
  row = rows ? idx % ROWS : idx >> 4;
  c4 = rows ? idx / ROWS : idx & 15;
}

template <int PREC, int ROWS>
__device__ __forceinline__ void stage_tile(char* lds, const float4 (&r)[ROWS * 16 / kThreads], float scale,
                                           bool rows = false) {
  constexpr int per = ROWS * 16 / kThreads;
#pragma unroll
  for (int i = 0; i < per; ++i) {
    int row, c4;  // c4: pair of complex k = 2*c4, 2*c4+1
    pair_of<ROWS>(i, rows, row, c4);
    const float4 v = r[i];
    if constexpr (PREC == P_BF16X3) {
      const uint32_t h0 = pack_bf16x2(v.x, v.y), h1 = pack_bf16x2(v.z, v.w);
      const uint32_t l0 = pack_bf16x2(v.x - bf16_lo_to_f32(h0), v.y - bf16_hi_to_f32(h0));
      const uint32_t l1 = pack_bf16x2(v.z - bf16_lo_to_f32(h1), v.w - bf16_hi_to_f32(h1));
      char* base = lds + row * TileLds<PREC, ROWS>::row_bytes + c4 * 8;
      *reinterpret_cast<uint2*>(base) = make_uint2(h0, h1);
      *reinterpret_cast<uint2*>(base + TileLds<PREC, ROWS>::plane_bytes) = make_uint2(l0, l1);
    } else {
      const uint32_t h0 = pack_f16x2(v.x * scale, v.y * scale), h1 = pack_f16x2(v.z * scale, v.w * scale);
      *reinterpret_cast<uint2*>(lds + row * TileLds<PREC, ROWS>::row_bytes + c4 * 8) = make_uint2(h0, h1);
    }
  }
}

template <int ROWS>
__device__ __forceinline__ void load_tile(float4 (&r)[ROWS * 16 / kThreads], const float2* __restrict__ p,
                                          int64_t ld, int64_t k0) {
  constexpr int per = ROWS * 16 / kThreads;
  const int tid = threadIdx.x;
#pragma unroll
  for (int i = 0; i < per; ++i) {
    const int idx = tid + i * kThreads;
    const int row = idx >> 4, c4 = idx & 15;
    r[i] = *reinterpret_cast<const float4*>(p + row * ld + k0 + 2 * c4);
  }
}

// The loads of an operand that is read through an OpMap (see F32Gather): p is its element (tile's first row, k = 0).
template <int ROWS>
__device__ __forceinline__ void gather_tile(float4 (&r)[ROWS * 16 / kThreads], const float2* __restrict__ p,
                                            const OpMap& m, const uint32_t (&at)[ROWS * 16 / kThreads], uint32_t k0) {
  const uint32_t off = map_bits<12>(k0, m.k), second = 1u << (m.k & 31);
#pragma unroll
  for (int i = 0; i < ROWS * 16 / kThreads; ++i) {
    const float2* q = p + (at[i] | off);
    const float2 a = q[0], b = q[second];
    r[i] = make_float4(a.x, a.y, b.x, b.y);
  }
}
template <int ROWS>
__device__ __forceinline__ void gather_places(uint32_t (&at)[ROWS * 16 / kThreads], const OpMap& m, int64_t row0) {
  const uint32_t r0 = map_row(m, (uint32_t)row0);
#pragma unroll
  for (int i = 0; i < ROWS * 16 / kThreads; ++i) {
    int row, c4;
    pair_of<ROWS>(i, m.row_fast, row, c4);
    at[i] = r0 | map_bits<7>(row, m.row[0]) | map_bits<5>(2 * c4, m.k);
  }
}

template <int PREC, int WTM, int WTN, bool GA, bool GB>
__global__ void __launch_bounds__(kThreads)
cgemm_mfma(int64_t M, int64_t N, int64_t K, const float2* __restrict__ A, const float2* __restrict__ B,
           float2* __restrict__ C, int64_t sa, int64_t sb, int64_t sc, const uint32_t* amaxA,
           const uint32_t* amaxB, Renorm rn, int64_t kc, float2* __restrict__ P, int64_t nbatch, OpMap ma, OpMap mb) {
  constexpr int BM = 32 * WTM, BN = 16 * WTN;
  using LA = TileLds<PREC, BM>;
  using LB = TileLds<PREC, BN>;
  __shared__ __attribute__((aligned(16))) char lds[LA::bytes + LB::bytes];
  char* ldsA = lds;
  char* ldsB = lds + LA::bytes;

  // tile mapping: XCD-contiguous remap over the whole launch (an XCD's L2 then holds its own chains'
  // operands), then grouped rasterisation over row tiles
  const int64_t tiles_m = M / BM, tiles_n = N / BN;
  const int64_t ntiles = tiles_m * tiles_n, total = ntiles * nbatch;
  int64_t bid = blockIdx.x;
  if ((total & 7) == 0) bid = (bid & 7) * (total >> 3) + (bid >> 3);
  const int64_t batch = bid / ntiles;
  bid -= batch * ntiles;
  const int64_t group = 8;
  const int64_t per_group = group * tiles_n;
  const int64_t gidx = bid / per_group;
  const int64_t first_m = gidx * group;
  const int64_t gsize = (tiles_m - first_m) < group ? (tiles_m - first_m) : group;
  const int64_t tm = first_m + (bid % per_group) % gsize;
  const int64_t tn = (bid % per_group) / gsize;

  const bool partial = gridDim.y > 1;
  const uint32_t k0 = blockIdx.y * (uint32_t)kc;
  uint32_t pa[GA ? BM * 16 / kThreads : 1], pb[GB ? BN * 16 / kThreads : 1];
  if constexpr (GA) {
    A += map_base(ma, batch, sa);
    gather_places<BM>(pa, ma, tm * BM);
  } else {
    A += (ma.on ? map_base(ma, batch, sa) : batch * sa) + tm * BM * K + blockIdx.y * kc;
  }
  if constexpr (GB) {
    B += map_base(mb, batch, sb);
    gather_places<BN>(pb, mb, tn * BN);
  } else {
    B += (mb.on ? map_base(mb, batch, sb) : batch * sb) + tn * BN * K + blockIdx.y * kc;
  }
  if (partial) {
    C = P + ((int64_t)blockIdx.y * nbatch + batch) * M * N;
  } else {
    C += batch * sc;
  }

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wr = (wave >> 1) * (16 * WTM);   // wave's first row in the block tile
  const int wc = (wave & 1) * (8 * WTN);     // wave's first complex column
  const int l16 = lane & 15, lg = lane >> 4;

  float scale_a, scale_b, unscale;
  rn = renorm_of(rn, batch);
  scales_for<PREC>(rn, amaxA, amaxB, partial, tm == 0 && tn == 0, scale_a, scale_b, unscale);

  f4 acc[WTM][WTN];
#pragma unroll
  for (int i = 0; i < WTM; ++i)
#pragma unroll
    for (int j = 0; j < WTN; ++j) acc[i][j] = (f4){0.f, 0.f, 0.f, 0.f};

  float4 ra[BM * 16 / kThreads], rb[BN * 16 / kThreads];
  auto fetch = [&](int64_t kt) {
    if constexpr (GA) gather_tile<BM>(ra, A, ma, pa, k0 + (uint32_t)(kt * kBK));
    else load_tile<BM>(ra, A, K, kt * kBK);
    if constexpr (GB) gather_tile<BN>(rb, B, mb, pb, k0 + (uint32_t)(kt * kBK));
    else load_tile<BN>(rb, B, K, kt * kBK);
  };
  fetch(0);
  const int64_t nk = kc / kBK;
  for (int64_t kt = 0; kt < nk; ++kt) {
    stage_tile<PREC, BM>(ldsA, ra, scale_a, GA && ma.row_fast);
    stage_tile<PREC, BN>(ldsB, rb, scale_b, GB && mb.row_fast);
    __syncthreads();
    if (kt + 1 < nk) fetch(kt + 1);
    // 2 chunks of 16 complex k; lane group lg holds complex k 4*lg .. 4*lg+3 (8 real k)
    const BExpand bx(l16 & 1);
#pragma unroll
    for (int c = 0; c < kBK / 16; ++c) {
      u4 ah[WTM], al[WTM];
#pragma unroll
      for (int i = 0; i < WTM; ++i) {
        const char* p = ldsA + (wr + 16 * i + l16) * LA::row_bytes + (16 * c + 4 * lg) * 4;
        ah[i] = *reinterpret_cast<const u4*>(p);
        if constexpr (PREC == P_BF16X3) al[i] = *reinterpret_cast<const u4*>(p + LA::plane_bytes);
      }
#pragma unroll
      for (int j = 0; j < WTN; ++j) {
        const char* p = ldsB + (wc + 8 * j + (l16 >> 1)) * LB::row_bytes + (16 * c + 4 * lg) * 4;
        u4 bh = *reinterpret_cast<const u4*>(p);
#pragma unroll
        for (int e = 0; e < 4; ++e) bh[e] = bx(bh[e]);
        if constexpr (PREC == P_BF16X3) {
          u4 bl = *reinterpret_cast<const u4*>(p + LB::plane_bytes);
#pragma unroll
          for (int e = 0; e < 4; ++e) bl[e] = bx(bl[e]);
          const bf8 vbh = __builtin_bit_cast(bf8, bh), vbl = __builtin_bit_cast(bf8, bl);
#pragma unroll
          for (int i = 0; i < WTM; ++i)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, al[i]), vbh, acc[i][j], 0, 0, 0);
#pragma unroll
          for (int i = 0; i < WTM; ++i)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, ah[i]), vbl, acc[i][j], 0, 0, 0);
#pragma unroll
          for (int i = 0; i < WTM; ++i)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, ah[i]), vbh, acc[i][j], 0, 0, 0);
        } else {
          const h8 vb = __builtin_bit_cast(h8, bh);
#pragma unroll
          for (int i = 0; i < WTM; ++i)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, ah[i]), vb, acc[i][j], 0, 0, 0);
        }
      }
    }
    __syncthreads();
  }

  const uint32_t seen = partial ? 0u : seen_amax(rn);
  float mx = 0.f;
  Renorm om = rn;
  if (partial) om.om_nh = 0;
  const int64_t col0 = tn * BN + wc + 2 * (l16 >> 2);
#pragma unroll
  for (int i = 0; i < WTM; ++i) {
    float2* c = C + c_row(om, tm * BM + wr + 16 * i + 4 * lg + (l16 & 3), N);
#pragma unroll
    for (int j = 0; j < WTN; ++j) {
      const f4 o = quad_transpose(acc[i][j] * unscale);
      *reinterpret_cast<f4*>(c + c_col(om, col0 + 8 * j)) = o;
      mx = fmaxf(mx, cmax4(o));
    }
  }
  if (rn.c && !partial) raise_amax<kThreads / 64>(rn.c, mx, seen, reinterpret_cast<float*>(lds));
}

// Large shapes, BF16-family products: 512 threads = 8 waves as 4 (M) x 2 (N); a wave owns
// 4 x 8 MFMA tiles (64 rows x 64 complex columns); block tile 256 rows x 128 complex columns;
// K-tiles of 16 complex (one 16x16x32 MFMA step).  Two LDS stages: while the MFMAs consume one
// stage, the next K-tile (already in registers) is converted and stored into the other, and the
// K-tile after it is fetched from global memory; one barrier per K-tile.  LDS rows are 16
// complex (64 B per plane) padded to 80 B, which spreads the 16-byte reads of 16 consecutive
// rows over all banks.
constexpr int kV2Threads = 512;
constexpr int kV2BM = 256, kV2BN = 128, kV2BK = 16;
constexpr int kV2Row = 80;                      // bytes per LDS row (64 + 16 pad)
constexpr int kV2PlaneA = kV2BM * kV2Row;       // 20 KiB
constexpr int kV2PlaneB = kV2BN * kV2Row;       // 10 KiB

template <int PREC>
struct V2 {
  static constexpr int planes = PREC == P_BF16X3 ? 2 : 1;
  static constexpr int stage = planes * (kV2PlaneA + kV2PlaneB);
};

template <int PREC>
__device__ __forceinline__ void v2_store(char* st, const float4 (&ra)[4], const float4 (&rb)[2], float sa, float sb) {
  const int tid = threadIdx.x;
  constexpr int planes = V2<PREC>::planes;
  char* A = st;
  char* B = st + planes * kV2PlaneA;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = (tid >> 3) + 64 * i, c = tid & 7;  // c: complex pair 2c, 2c+1
    const float4 v = ra[i];
    char* dst = A + row * kV2Row + c * 8;
    if constexpr (PREC == P_BF16X3) {
      const uint32_t h0 = pack_bf16x2(v.x, v.y), h1 = pack_bf16x2(v.z, v.w);
      const uint32_t l0 = pack_bf16x2(v.x - bf16_lo_to_f32(h0), v.y - bf16_hi_to_f32(h0));
      const uint32_t l1 = pack_bf16x2(v.z - bf16_lo_to_f32(h1), v.w - bf16_hi_to_f32(h1));
      *reinterpret_cast<uint2*>(dst) = make_uint2(h0, h1);
      *reinterpret_cast<uint2*>(dst + kV2PlaneA) = make_uint2(l0, l1);
    } else {
      *reinterpret_cast<uint2*>(dst) = make_uint2(pack_f16x2(v.x * sa, v.y * sa), pack_f16x2(v.z * sa, v.w * sa));
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = (tid >> 3) + 64 * i, c = tid & 7;
    const float4 v = rb[i];
    char* dst = B + row * kV2Row + c * 8;
    if constexpr (PREC == P_BF16X3) {
      const uint32_t h0 = pack_bf16x2(v.x, v.y), h1 = pack_bf16x2(v.z, v.w);
      const uint32_t l0 = pack_bf16x2(v.x - bf16_lo_to_f32(h0), v.y - bf16_hi_to_f32(h0));
      const uint32_t l1 = pack_bf16x2(v.z - bf16_lo_to_f32(h1), v.w - bf16_hi_to_f32(h1));
      *reinterpret_cast<uint2*>(dst) = make_uint2(h0, h1);
      *reinterpret_cast<uint2*>(dst + kV2PlaneB) = make_uint2(l0, l1);
    } else {
      *reinterpret_cast<uint2*>(dst) = make_uint2(pack_f16x2(v.x * sb, v.y * sb), pack_f16x2(v.z * sb, v.w * sb));
    }
  }
}

__device__ __forceinline__ void v2_load(float4 (&ra)[4], float4 (&rb)[2], const float2* __restrict__ A,
                                        const float2* __restrict__ B, int64_t K, int64_t k0) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = (tid >> 3) + 64 * i, c = tid & 7;
    ra[i] = *reinterpret_cast<const float4*>(A + row * K + k0 + 2 * c);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = (tid >> 3) + 64 * i, c = tid & 7;
    rb[i] = *reinterpret_cast<const float4*>(B + row * K + k0 + 2 * c);
  }
}

template <int PREC>
__global__ void __launch_bounds__(kV2Threads)
cgemm_v2(int64_t M, int64_t N, int64_t K, const float2* __restrict__ A, const float2* __restrict__ B,
         float2* __restrict__ C, int64_t sa, int64_t sb, int64_t sc, const uint32_t* amaxA, const uint32_t* amaxB,
         Renorm rn, int64_t kc, float2* __restrict__ P) {
  __shared__ __attribute__((aligned(16))) char lds[2 * V2<PREC>::stage];
  constexpr int planes = V2<PREC>::planes;

  const int64_t tiles_m = M / kV2BM, tiles_n = N / kV2BN;
  const int64_t ntiles = tiles_m * tiles_n;
  int64_t bid = blockIdx.x;
  if ((ntiles & 7) == 0) bid = (bid & 7) * (ntiles >> 3) + (bid >> 3);
  const int64_t group = 8;
  const int64_t per_group = group * tiles_n;
  const int64_t gidx = bid / per_group;
  const int64_t first_m = gidx * group;
  const int64_t gsize = (tiles_m - first_m) < group ? (tiles_m - first_m) : group;
  const int64_t tm = first_m + (bid % per_group) % gsize;
  const int64_t tn = (bid % per_group) / gsize;

  const int64_t batch = blockIdx.z;
  const bool partial = gridDim.y > 1;
  A += batch * sa + tm * kV2BM * K + blockIdx.y * kc;
  B += batch * sb + tn * kV2BN * K + blockIdx.y * kc;
  if (partial) {
    C = P + ((int64_t)blockIdx.y * gridDim.z + batch) * M * N;
  } else {
    C += batch * sc;
  }

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wr = (wave >> 1) * 64;  // first row of the wave
  const int wc = (wave & 1) * 64;   // first complex column of the wave
  const int l16 = lane & 15, lg = lane >> 4, q = l16 & 1;
  const BExpand bx(q);

  float scale_a, scale_b, unscale;
  rn = renorm_of(rn, batch);
  scales_for<PREC>(rn, amaxA, amaxB, partial, tm == 0 && tn == 0, scale_a, scale_b, unscale);

  f4 acc[4][8];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = (f4){0.f, 0.f, 0.f, 0.f};

  float4 ra[4], rb[2];
  const int64_t nk = kc / kV2BK;
  v2_load(ra, rb, A, B, K, 0);
  v2_store<PREC>(lds, ra, rb, scale_a, scale_b);
  if (nk > 1) v2_load(ra, rb, A, B, K, kV2BK);
  __syncthreads();
  for (int64_t kt = 0; kt < nk; ++kt) {
    const char* st = lds + (kt & 1) * V2<PREC>::stage;
    const char* LA = st;
    const char* LB = st + planes * kV2PlaneA;
    u4 ah[4], al[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const char* p = LA + (wr + 16 * i + l16) * kV2Row + lg * 16;
      ah[i] = *reinterpret_cast<const u4*>(p);
      if constexpr (PREC == P_BF16X3) al[i] = *reinterpret_cast<const u4*>(p + kV2PlaneA);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const char* p = LB + (wc + 8 * j + (l16 >> 1)) * kV2Row + lg * 16;
      u4 bh = *reinterpret_cast<const u4*>(p);
#pragma unroll
      for (int e = 0; e < 4; ++e) bh[e] = bx(bh[e]);
      if constexpr (PREC == P_BF16X3) {
        u4 bl = *reinterpret_cast<const u4*>(p + kV2PlaneB);
#pragma unroll
        for (int e = 0; e < 4; ++e) bl[e] = bx(bl[e]);
        const bf8 vbh = __builtin_bit_cast(bf8, bh), vbl = __builtin_bit_cast(bf8, bl);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, al[i]), vbh, acc[i][j], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, ah[i]), vbl, acc[i][j], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, ah[i]), vbh, acc[i][j], 0, 0, 0);
      } else {
        const h8 vb = __builtin_bit_cast(h8, bh);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, ah[i]), vb, acc[i][j], 0, 0, 0);
      }
    }
    if (kt + 1 < nk) {
      v2_store<PREC>(lds + ((kt + 1) & 1) * V2<PREC>::stage, ra, rb, scale_a, scale_b);
      if (kt + 2 < nk) v2_load(ra, rb, A, B, K, (kt + 2) * kV2BK);
    }
    __syncthreads();
  }

  const uint32_t seen = partial ? 0u : seen_amax(rn);
  float mx = 0.f;
  Renorm om = rn;
  if (partial) om.om_nh = 0;
  const int64_t col0 = tn * kV2BN + wc + 2 * (l16 >> 2);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float2* c = C + c_row(om, tm * kV2BM + wr + 16 * i + 4 * lg + (l16 & 3), N);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const f4 o = quad_transpose(acc[i][j] * unscale);
      *reinterpret_cast<f4*>(c + c_col(om, col0 + 8 * j)) = o;
      mx = fmaxf(mx, cmax4(o));
    }
  }
  if (rn.c && !partial) raise_amax<kV2Threads / 64>(rn.c, mx, seen, reinterpret_cast<float*>(lds));
}

// Small or thin shapes: one thread per output element, FP32 complex FMA over K.
__global__ void __launch_bounds__(256)
cgemm_simt(int64_t M, int64_t N, int64_t K, const float2* __restrict__ A, const float2* __restrict__ B,
           float2* __restrict__ C, int64_t sa, int64_t sb, int64_t sc, Renorm rn) {
  float scale_a, scale_b, unscale;
  const int64_t batch = blockIdx.z;
  rn = renorm_of(rn, batch);
  renorm_begin<P_FP32>(rn, nullptr, nullptr, blockIdx.x == 0, scale_a, scale_b, unscale);
  float mx = 0.f;
  A += batch * sa;
  B += batch * sb;
  C += batch * sc;
  const int64_t total = M * N;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int64_t m = idx / N, n = idx - m * N;
    const float2* a = A + m * K;
    const float2* b = B + n * K;
    float cr = 0.f, ci = 0.f;
    for (int64_t k = 0; k < K; ++k) {
      const float2 x = a[k], y = b[k];
      cr = fmaf(x.x, y.x, cr);
      cr = fmaf(-x.y, y.y, cr);
      ci = fmaf(x.x, y.y, ci);
      ci = fmaf(x.y, y.x, ci);
    }
    const float2 o = make_float2(cr * unscale, ci * unscale);
    C[c_index(rn, m, n, N)] = o;
    mx = fmaxf(mx, cmax(o));
  }
  if (rn.c) record_amax(rn.c, mx);
}

// Short K, narrow N, long M (a large tensor absorbing one small world-line): B (N x K) is staged
// in LDS; thread t computes outputs (m, 4g .. 4g+3) with m = t / (N/4), so consecutive threads
// write consecutive 32-byte groups of C and the threads sharing a row read the same A row.
constexpr int kSkinnyMaxB = 4096;  // complex elements of B held in LDS

// B is held transposed in LDS (Bs[k][n]); thread (m, g) computes outputs n = g + t N/4 (t < 4), so
// for each k the lanes of a wave read consecutive 8-byte words of one LDS row (no bank conflicts)
// and write consecutive complex numbers of C (coalesced).  Each output sums k in ascending order.
__global__ void __launch_bounds__(256)
cgemm_skinny(int64_t M, int64_t N, int64_t K, const float2* __restrict__ A, const float2* __restrict__ B,
             float2* __restrict__ C, int64_t sa, int64_t sb, int64_t sc, Renorm rn, OpMap ma, OpMap mb) {
  __shared__ float2 Bs[kSkinnyMaxB];
  float scale_a, scale_b, unscale;
  const int64_t batch = blockIdx.z;
  rn = renorm_of(rn, batch);
  renorm_begin<P_FP32>(rn, nullptr, nullptr, blockIdx.x == 0, scale_a, scale_b, unscale);
  float mx = 0.f;
  A += ma.on ? map_base(ma, batch, sa) : batch * sa;
  B += mb.on ? map_base(mb, batch, sb) : batch * sb;
  C += batch * sc;
  const int n_ = (int)N, k_ = (int)K;
  for (int i = threadIdx.x; i < n_ * k_; i += 256) {
    const int n = i / k_, k = i - n * k_;
    Bs[k * n_ + n] = B[mb.on == 1 ? map_row(mb, n) | map_bits<6>(k, mb.k) : (uint32_t)i];
  }
  __syncthreads();
  const int Q = n_ / 4;
  const int64_t total = M * Q;
  for (int64_t o = (int64_t)blockIdx.x * 256 + threadIdx.x; o < total; o += (int64_t)gridDim.x * 256) {
    int64_t m = o / Q;
    const int g = (int)(o - m * Q);
    const float2* a = A + (ma.on == 1 ? (int64_t)map_row(ma, (uint32_t)m) : m * K);
    float cr[4] = {0.f, 0.f, 0.f, 0.f}, ci[4] = {0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < k_; ++k) {
      const float2 x = a[ma.on == 1 ? map_bits<6>(k, ma.k) : (uint32_t)k];
      const float2* brow = Bs + k * n_ + g;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float2 y = brow[t * Q];
        cr[t] = fmaf(x.x, y.x, cr[t]);
        cr[t] = fmaf(-x.y, y.y, cr[t]);
        ci[t] = fmaf(x.x, y.y, ci[t]);
        ci[t] = fmaf(x.y, y.x, ci[t]);
      }
    }
    if (rn.rp_on) m = map_bits<12>((uint32_t)m & 0xfff, rn.rp[0]) | map_bits<12>((uint32_t)m >> 12, rn.rp[1]);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float2 v = make_float2(cr[t] * unscale, ci[t] * unscale);
      C[c_index(rn, m, g + t * Q, N)] = v;
      mx = fmaxf(mx, cmax(v));
    }
  }
  if (rn.c) record_amax(rn.c, mx);
}

// Few outputs, long K (e.g. the last contraction of two halves into a scalar): one workgroup per output
// element, threads stride over K with eight loads of each operand in flight, then a workgroup
// reduction.  Bound by latency (one workgroup) or, over many outputs, by reading the operands.
constexpr int kDotUnroll = 8;

template <int NTH>
__global__ void __launch_bounds__(NTH)
cgemm_splitk(int64_t M, int64_t N, int64_t K, const float2* __restrict__ A, const float2* __restrict__ B,
             float2* __restrict__ C, int64_t sa, int64_t sb, int64_t sc, Renorm rn) {
  __shared__ float red[2][NTH / 64];
  float scale_a, scale_b, unscale;
  const int64_t batch = blockIdx.z;
  rn = renorm_of(rn, batch);
  renorm_begin<P_FP32>(rn, nullptr, nullptr, blockIdx.x == 0, scale_a, scale_b, unscale);
  const int64_t out = blockIdx.x;  // m * N + n
  const int64_t m = out / N, n = out - m * N;
  const float2* a = A + batch * sa + m * K;
  const float2* b = B + batch * sb + n * K;
  float cr = 0.f, ci = 0.f;
  auto add = [&](float2 x, float2 y) {
    cr = fmaf(x.x, y.x, cr);
    cr = fmaf(-x.y, y.y, cr);
    ci = fmaf(x.x, y.y, ci);
    ci = fmaf(x.y, y.x, ci);
  };
  int64_t k = threadIdx.x;
  for (; k + (kDotUnroll - 1) * NTH < K; k += kDotUnroll * NTH) {
    float2 x[kDotUnroll], y[kDotUnroll];
#pragma unroll
    for (int u = 0; u < kDotUnroll; ++u) {
      x[u] = a[k + u * NTH];
      y[u] = b[k + u * NTH];
    }
#pragma unroll
    for (int u = 0; u < kDotUnroll; ++u) add(x[u], y[u]);
  }
  for (; k < K; k += NTH) add(a[k], b[k]);
  for (int off = 32; off > 0; off >>= 1) {
    cr += __shfl_xor(cr, off);
    ci += __shfl_xor(ci, off);
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { red[0][w] = cr; red[1][w] = ci; }
  __syncthreads();
  if (threadIdx.x == 0) {
    float r = 0.f, i = 0.f;
#pragma unroll
    for (int u = 0; u < NTH / 64; ++u) { r += red[0][u]; i += red[1][u]; }
    r *= unscale;
    i *= unscale;
    C[batch * sc + c_index(rn, m, n, N)] = make_float2(r, i);
    if (rn.c) atomicMax(amax_slot(rn.c), __float_as_uint(fmaxf(fabsf(r), fabsf(i))));
  }
}

template <int PREC, int WTM, int WTN>
static hipError_t launch_tiled(hipStream_t st, int64_t M, int64_t N, int64_t K, const float2* A, const float2* B, float2* C,
                         int64_t batch, int64_t sa, int64_t sb, int64_t sc, const uint32_t* amaxA,
                         const uint32_t* amaxB, const Renorm& rn, int split, float2* P, const OpMap& ma,
                         const OpMap& mb) {
  constexpr int BM = 32 * WTM, BN = 16 * WTN;
  const int64_t tiles = (M / BM) * (N / BN);
  if (!grid_takes(tiles * batch, kThreads)) return hipErrorInvalidConfiguration;
  auto run = [&](auto* kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)(tiles * batch), (unsigned)split), dim3(kThreads), 0, st, M, N, K, A, B, C,
                       sa, sb, sc, amaxA, amaxB, rn, K / split, P, batch, ma, mb);
    return hipGetLastError();
  };
  if constexpr (PREC == P_BF16X3) {
    if (ma.on == 1 && mb.on == 1) return run(cgemm_mfma<PREC, WTM, WTN, true, true>);
    if (ma.on == 1) return run(cgemm_mfma<PREC, WTM, WTN, true, false>);
    if (mb.on == 1) return run(cgemm_mfma<PREC, WTM, WTN, false, true>);
  }
  return run(cgemm_mfma<PREC, WTM, WTN, false, false>);
}

static bool pow2(int64_t x) { return x > 0 && (x & (x - 1)) == 0; }

bool cgemm_variant_fits(int precision, int64_t M, int64_t N, int64_t K, int variant) {
  const bool p2 = pow2(M) && pow2(N) && pow2(K);
  switch (variant) {
    case GEMM_TILED_4X4: return p2 && M >= 128 && N >= 64 && K >= kBK;
    case GEMM_TILED_2X2: return p2 && M >= 64 && N >= 32 && K >= kBK;
    case GEMM_TILED_1X2: return p2 && M >= 32 && N >= 32 && K >= kBK;
    case GEMM_LARGE: return p2 && M >= kV2BM && N >= kV2BN && K >= kV2BK;
    case GEMM_SKINNY: return N >= 4 && (N & 3) == 0 && N * K <= kSkinnyMaxB && K <= 64;
    case GEMM_SPLITK: return M * N <= 4096;
    case GEMM_SIMT:
    case GEMM_F32: return M >= 1 && N >= 1 && K >= 1;
    case GEMM_TALL: return cgemm_tall_fits(precision, M, N, K);
  }
  return false;
}

// FP16 products, sizes powers of two: the kernels and chunks of K of this rule, whatever is faster.  Another order
// of FP32 sums flips roundings to fp16 in every later step of a contraction: 1e-4 of the amplitudes of
// a 5x5 circuit of depth 30, 5e-4 with some products in FP32.
static int fp16_variant(int64_t M, int64_t N, int64_t K) {
  auto fits = [&](int v) { return cgemm_variant_fits(P_FP16, M, N, K, v); };
  if (fits(GEMM_LARGE)) return GEMM_LARGE;
  if (M >= 4096 && (N < 32 || K < kBK) && fits(GEMM_TALL)) return GEMM_TALL;
  if (fits(GEMM_TILED_1X2)) return M >= 128 && N >= 64 ? GEMM_TILED_4X4 : M >= 64 ? GEMM_TILED_2X2 : GEMM_TILED_1X2;
  if (fits(GEMM_SKINNY)) return GEMM_SKINNY;
  return M * N <= 4096 && K >= 256 ? GEMM_SPLITK : GEMM_SIMT;
}

static int fp16_split(int variant, int64_t M, int64_t N, int64_t K) {
  int64_t bm = 0, bn = 0, bk = kBK;
  if (variant == GEMM_LARGE) bm = kV2BM, bn = kV2BN, bk = kV2BK;
  else if (variant == GEMM_TILED_4X4) bm = 128, bn = 64;
  else if (variant == GEMM_TILED_2X2) bm = 64, bn = 32;
  else if (variant == GEMM_TILED_1X2) bm = 32, bn = 32;
  if (bm == 0 || (M / bm) * (N / bn) >= 256) return 1;
  int split = 1;
  while (split < 1024 && (M / bm) * (N / bn) * split * 2 <= 1024 && K / (split * 2) >= 4 * bk) split *= 2;
  return split;
}

// Every tile of one precision adds an output's products in the same order, so among the tiles the
// launch may pick by how many workgroups they give (batch included) without changing a result; the
// choice between the families below, and the cut of K, are functions of the shape alone, and a
// batched launch equals the launches of its elements bit by bit.
int cgemm_default_variant(int precision, int64_t M, int64_t N, int64_t K, int64_t blocks_per_tile) {
  if (precision == P_FP16 && pow2(M) && pow2(N) && pow2(K)) return fp16_variant(M, N, K);
  // HBM-bound tall-skinny products below the tiles' N and K (as fast as the 64 x 32 tiles where
  // those fit: 5.1 TB/s on 2^25 x 32 x 32 split-BF16)
  if (M >= 4096 && (N < 32 || K < kBK) && cgemm_variant_fits(precision, M, N, K, GEMM_TALL)) return GEMM_TALL;
  if (precision != P_FP32 && cgemm_variant_fits(precision, M, N, K, GEMM_TILED_1X2)) {
    // the largest tile that still yields a workgroup for each of 256 CUs (the 256 x 128 tile, the most
    // efficient per CU, from half as many)
    if (M >= kV2BM && N >= kV2BN && (M / kV2BM) * (N / kV2BN) * blocks_per_tile >= 128) return GEMM_LARGE;
    if (M >= 128 && N >= 64 && (M / 128) * (N / 64) * blocks_per_tile >= 256) return GEMM_TILED_4X4;
    if (M >= 64 && (M / 64) * (N / 32) * blocks_per_tile >= 256) return GEMM_TILED_2X2;
    return GEMM_TILED_1X2;
  }
  // K = 16 is half a K-tile of the smaller 16-bit tiles; few large tiles are slower than the FP32 tiles
  if (precision == P_BF16X3 && cgemm_variant_fits(precision, M, N, K, GEMM_LARGE) && (M / kV2BM) * (N / kV2BN) >= 128)
    return GEMM_LARGE;
  // a few dot products: a workgroup each; very long ones are spread further by the tiles' split K
  if (M * N <= 64 && K >= 32 && K <= (1 << 17)) return GEMM_SPLITK;
  // up to 256 thin ones, where a launch of many chains loses little by it: 16 x 16 x 256 4 us against 10 on tiles (32 of
  // them 8 / 11), x 1024 4 / 21 (14 / 22), x 4096 4 / 21 (38 / 22); 256 x 16 x 256 5 / 9 (88 / 9)
  if (M * N <= 256 && (M < 32 || N < 32) && K >= 256 && K <= 4096) return GEMM_SPLITK;
  // short K or N: the FP32 tiles would multiply zeros
  if ((K < 16 || (K < 32 && N < 32)) && cgemm_variant_fits(precision, M, N, K, GEMM_SKINNY)) return GEMM_SKINNY;
  if (K < 8 || M * N * K < 4096) return GEMM_SIMT;
  return GEMM_F32;
}

// A product of its own (qf_cgemm): dot products by a workgroup each while they are few and read less than the tiles
// take: 64 x 64 x 1024 7 us against 9 with K cut finely, x 2048 13 / 10; of thin ones, whose tiles multiply zeros,
// 2 x 1078 x 3529 12 / 33, 16 x 16 x 65536 19 / 29, 16 x 64 x 65536 82 / 26, 2048 x 2 x 8192 37 / 50.
static int direct_variant(int precision, int64_t M, int64_t N, int64_t K, int64_t batch) {
  const int v = cgemm_default_variant(precision, M, N, K);
  if (precision == P_FP16 && pow2(M) && pow2(N) && pow2(K)) return v;
  const int64_t outputs = batch * M * N, thin = std::min(M, N);
  const int64_t most = (int64_t)1 << (thin <= 2 ? 25 : thin < 32 ? 24 : 22);
  if (M * N <= 4096 && outputs <= 16384 && K >= 64 && outputs * K <= most) return GEMM_SPLITK;
  return v == GEMM_SPLITK && M * N > 64 ? GEMM_F32 : v;
}

template <int PREC>
static hipError_t launch_mfma(hipStream_t st, int variant, int64_t M, int64_t N, int64_t K, const float2* A,
                              const float2* B, float2* C, int64_t batch, int64_t sa, int64_t sb, int64_t sc,
                              const uint32_t* amaxA, const uint32_t* amaxB, const Renorm& rn, int split,
                              float2* P, const OpMap& ma, const OpMap& mb) {
  switch (variant) {
    case GEMM_LARGE:
      hipLaunchKernelGGL((cgemm_v2<PREC>), dim3((unsigned)((M / kV2BM) * (N / kV2BN)), (unsigned)split, (unsigned)batch),
                         dim3(kV2Threads), 0, st, M, N, K, A, B, C, sa, sb, sc, amaxA, amaxB, rn, K / split, P);
      return hipGetLastError();
    case GEMM_TILED_4X4:
      return launch_tiled<PREC, 4, 4>(st, M, N, K, A, B, C, batch, sa, sb, sc, amaxA, amaxB, rn, split, P, ma, mb);
    case GEMM_TILED_2X2:
      return launch_tiled<PREC, 2, 2>(st, M, N, K, A, B, C, batch, sa, sb, sc, amaxA, amaxB, rn, split, P, ma, mb);
    default:
      return launch_tiled<PREC, 1, 2>(st, M, N, K, A, B, C, batch, sa, sb, sc, amaxA, amaxB, rn, split, P, ma, mb);
  }
}

// K-chunks of an MFMA launch: K is cut (powers of two, chunks of at least 512) while the 64 x 32 tiles
// of one batch element number below 256 and the chunks' tiles stay within two per CU.  A chunk costs a
// write and a read of its partial tile and the reduction a launch, which K < 1024 does not repay: the
// 256 x 256 x 256 products of the 4 x 4 and 4 x 5 circuits took 332 us of split kernel and reduction per
// 64 chains, 100 us in one pass over K on smaller tiles.
// The few tiles of one product are cut finer: one 64 x 64 x 1024 18 us in chunks of 512, 12 of 256 (64 of them 33
// and 32).  batch > 0: a product of its own, with chunks down to 128 while the launch leaves CUs idle (9 us).
static int split_count(int precision, int variant, int64_t M, int64_t N, int64_t K, int64_t batch = 0) {
  if (precision == P_FP16 && variant != GEMM_F32) return fp16_split(variant, M, N, K);
  if (variant == GEMM_SKINNY || variant == GEMM_SPLITK || variant == GEMM_SIMT || variant == GEMM_TALL) return 1;
  const int64_t tiles = ((M + 63) / 64) * ((N + 31) / 32);
  if (tiles >= 256) return 1;
  const int64_t chunk = tiles <= 4 && K >= 1024 && K <= 2048 ? 256 : 512;
  int split = 1;
  while (tiles * split * 2 <= 512 && K / (split * 2) >= chunk) split *= 2;
  while (batch > 0 && K >= (tiles * batch <= 32 ? 512 : 1024) && tiles * batch * split * 2 <= 512 && split < 64 &&
         K / (split * 2) >= 128)
    split *= 2;
  return split;
}

size_t cgemm_split_scratch(int precision, int64_t M, int64_t N, int64_t K, int64_t batch, int variant, bool direct) {
  if (variant == GEMM_AUTO)
    variant = direct ? direct_variant(precision, M, N, K, batch) : cgemm_default_variant(precision, M, N, K);
  const int split = split_count(precision, variant, M, N, K, direct ? batch : 0);
  return split > 1 ? (size_t)split * (size_t)(batch * M * N) * sizeof(float2) : 0;
}

size_t env_gemm_scratch(int side, int64_t M, int64_t N, int64_t K, int64_t batch) {
  const int64_t rows = side ? N : M;
  const int split = split_count(P_FP32, GEMM_F32, rows, K, side ? M : N);
  return split > 1 ? (size_t)split * (size_t)(batch * rows * K) * sizeof(float2) : 0;
}

hipError_t launch_env_gemm(hipStream_t st, int side, int64_t M, int64_t N, int64_t K, const float2* env,
                           const float2* other, float2* out, int64_t batch, const Renorm& map, float2* scratch,
                           size_t scratch_bytes, bool plain) {
  const int64_t rows = side ? N : M;
  int split = scratch ? split_count(P_FP32, GEMM_F32, rows, K, side ? M : N) : 1;
  if (env_gemm_scratch(side, M, N, K, batch) > scratch_bytes) split = 1;
  const hipError_t e = launch_cgemm_f32_env(st, side, M, N, K, env, other, out, batch, map, &split, scratch, plain);
  if (e != hipSuccess || split == 1) return e;
  const unsigned blocks = (unsigned)std::min<int64_t>((batch * rows * K + kReduceOut - 1) / kReduceOut, 65536);
  hipLaunchKernelGGL(cgemm_split_reduce, dim3(blocks), dim3(256), 0, st, scratch, split, batch, rows * K, K, rows * K,
                     out, Renorm{});
  return hipGetLastError();
}

hipError_t launch_cgemm_ex(hipStream_t st, int precision, int64_t M, int64_t N, int64_t K, const float2* A,
                           const float2* B, float2* C, int64_t batch, int64_t sa, int64_t sb, int64_t sc,
                           const uint32_t* amaxA, const uint32_t* amaxB, const Renorm& rn, int variant,
                           float2* scratch, size_t scratch_bytes, const OpMap* ma, const OpMap* mb, int flags) {
  const bool direct = flags & GEMM_DIRECT, plain = flags & GEMM_PLAIN;
  if (rn.c && (!rn.a || !rn.b)) return hipErrorInvalidValue;
  if (M < 1 || N < 1 || K < 1 || batch < 1) return hipErrorInvalidValue;
  if (precision != P_FP32 && precision != P_BF16X3 && precision != P_FP16) return hipErrorInvalidValue;
  if ((ma || mb) && (variant != GEMM_AUTO || !cgemm_reads_maps(precision, M, N, K, batch))) return hipErrorInvalidValue;
  const OpMap a = ma ? *ma : OpMap{}, b = mb ? *mb : OpMap{};
  const bool chosen = variant != GEMM_AUTO && cgemm_variant_fits(precision, M, N, K, variant);
  int v = chosen ? variant : direct ? direct_variant(precision, M, N, K, batch) : cgemm_default_variant(precision, M, N, K);
  // split only when the caller's scratch holds every partial, otherwise one pass over K; where that leaves a few
  // outputs to a few workgroups (16 x 16 x 65536: 2 ms), a product of its own takes a workgroup per output (69 us)
  int split = scratch ? split_count(precision, v, M, N, K, direct ? batch : 0) : 1;
  if (split > 1 && (size_t)split * (size_t)(batch * M * N) * sizeof(float2) > scratch_bytes) split = 1;
  if (direct && !chosen && split == 1 && split_count(precision, v, M, N, K, batch) > 1 && M * N <= 4096 &&
      batch * M * N <= 16384 && !(precision == P_FP16 && pow2(M) && pow2(N) && pow2(K)))
    v = GEMM_SPLITK;
  if (rn.c && !rn.cleared) {
    const hipError_t e = launch_renorm_reset(st, rn, batch);
    if (e != hipSuccess) return e;
  }
  switch (v) {
    case GEMM_TALL:
      return launch_cgemm_tall(st, precision, M, N, K, A, B, C, batch, sa, sb, sc, amaxA, amaxB, rn, a, b);
    case GEMM_SKINNY: {
      const int64_t total = M * (N / 4);
      const unsigned blocks = (unsigned)std::min<int64_t>((total + 255) / 256, 65536);
      hipLaunchKernelGGL(cgemm_skinny, dim3(blocks, 1, (unsigned)batch), dim3(256), 0, st, M, N, K, A, B, C, sa, sb,
                         sc, rn, a, b);
      return hipGetLastError();
    }
    case GEMM_SPLITK:
      // a wave for the shortest sums, 16 waves from K = 16384 on (one output, K = 65536: 127 us with four), which many
      // outputs of K = 4096 would share out too finely (2048 of them 14 us with four waves each, 18 with 16)
      if (K < 256)
        hipLaunchKernelGGL(cgemm_splitk<64>, dim3((unsigned)(M * N), 1, (unsigned)batch), dim3(64), 0, st, M, N, K, A, B,
                           C, sa, sb, sc, rn);
      else if (K < 16384 || precision == P_FP16 || (direct && batch * M * N > 512))
        hipLaunchKernelGGL(cgemm_splitk<256>, dim3((unsigned)(M * N), 1, (unsigned)batch), dim3(256), 0, st, M, N, K, A,
                           B, C, sa, sb, sc, rn);
      else
        hipLaunchKernelGGL(cgemm_splitk<1024>, dim3((unsigned)(M * N), 1, (unsigned)batch), dim3(1024), 0, st, M, N, K,
                           A, B, C, sa, sb, sc, rn);
      return hipGetLastError();
    case GEMM_SIMT: {
      const unsigned blocks = (unsigned)std::min<int64_t>((M * N + 255) / 256, 65536);
      hipLaunchKernelGGL(cgemm_simt, dim3(blocks, 1, (unsigned)batch), dim3(256), 0, st, M, N, K, A, B, C, sa, sb, sc,
                         rn);
      return hipGetLastError();
    }
  }
  hipError_t e;
  if (precision == P_FP32 || v == GEMM_F32) {
    static const int tiles[] = {F32_AUTO, F32_64X64, F32_64X32, F32_32X32, F32_64X64};
    e = launch_cgemm_f32(st, M, N, K, A, B, C, batch, sa, sb, sc, rn, &split, scratch,
                         v != GEMM_F32 ? tiles[v] : plain ? F32_PLAIN : F32_AUTO, ma, mb);
  } else {
    if (!chosen) v = cgemm_default_variant(precision, M, N, K, batch * split);
    e = precision == P_BF16X3
            ? launch_mfma<P_BF16X3>(st, v, M, N, K, A, B, C, batch, sa, sb, sc, amaxA, amaxB, rn, split, scratch, a, b)
            : launch_mfma<P_FP16>(st, v, M, N, K, A, B, C, batch, sa, sb, sc, amaxA, amaxB, rn, split, scratch, a, b);
  }
  if (e == hipErrorInvalidConfiguration) {
    // more workgroups than a grid takes: the halves of the batch, or one product by the kernel that strides over outputs
    // (1 x 2^29 x 8 on tiles of 32 x 32)
    if (batch == 1) return launch_cgemm_ex(st, precision, M, N, K, A, B, C, 1, sa, sb, sc, amaxA, amaxB, rn, GEMM_SIMT);
    const int64_t half = batch / 2;
    e = launch_cgemm_ex(st, precision, M, N, K, A, B, C, half, sa, sb, sc, amaxA, amaxB, rn, variant, scratch, scratch_bytes,
                        ma, mb, flags);
    if (e != hipSuccess) return e;
    Renorm rest = rn;
    OpMap a2 = a, b2 = b;
    for (OpMap* m : {&a2, &b2})
      if (m->base_table) m->base_table += half * m->base_stride;
    if (rn.c) {
      rest.a += half * rn.a_step;
      rest.b += half * rn.b_step;
      rest.c += half * rn.c_step;
      rest.cleared = rn.cleared || rn.c_step == 0;
    }
    return launch_cgemm_ex(st, precision, M, N, K, a.base_table ? A : A + half * sa, b.base_table ? B : B + half * sb,
                           C + half * sc, batch - half, sa, sb, sc, amaxA, amaxB, rest, variant, scratch, scratch_bytes,
                           ma ? &a2 : nullptr, mb ? &b2 : nullptr, flags);
  }
  if (e != hipSuccess || split == 1) return e;
  const unsigned apart = rn.c_step ? (unsigned)batch : 1u;
  const unsigned blocks = (unsigned)std::min<int64_t>((batch / apart * M * N + kReduceOut - 1) / kReduceOut, 65536);
  hipLaunchKernelGGL(cgemm_split_reduce, dim3(blocks, 1, apart), dim3(256), 0, st, scratch, split, batch, M * N, N, sc, C,
                     rn);
  return hipGetLastError();
}

// The kernels of short sums, the FP32 tiles where they are whole, and the 16-bit tiles below the largest; FP16 keeps
// its copies.
bool cgemm_reads_maps(int precision, int64_t M, int64_t N, int64_t K, int64_t batch) {
  if (precision == P_FP16 || !pow2(M) || !pow2(N) || !pow2(K)) return false;
  int v = cgemm_default_variant(precision, M, N, K);
  if (v == GEMM_TALL || v == GEMM_SKINNY) return true;
  if (v == GEMM_F32) return M >= 32 && (N >= 32 || N == 16) && K >= 16;
  if (precision == P_FP32 || v == GEMM_SPLITK || v == GEMM_SIMT) return false;
  return cgemm_default_variant(precision, M, N, K, batch * split_count(precision, v, M, N, K)) != GEMM_LARGE;
}

// The tall kernel could too, but its scattered rows of results cost what the copy did (2^21 x 64 x 8).
bool cgemm_takes_row_order(int precision, int64_t M, int64_t N, int64_t K) {
  return precision != P_FP16 && pow2(M) && pow2(N) && pow2(K) &&
         cgemm_default_variant(precision, M, N, K) == GEMM_SKINNY;
}

hipError_t launch_cgemm(hipStream_t st, int precision, int64_t M, int64_t N, int64_t K, const float2* A,
                        const float2* B, float2* C, int64_t batch, int64_t sa, int64_t sb, int64_t sc) {
  return launch_cgemm_ex(st, precision, M, N, K, A, B, C, batch, sa, sb, sc, nullptr, nullptr, Renorm{});
}

// Max |re|, |im| of a complex64 array into *amax (as float bits; non-negative floats order
// like their bit patterns).  *amax must be zero before the launch.  One atomic per workgroup and at most
// 512 workgroups: atomics on one address are served about 10 ns apart, and one per wave over 2048
// workgroups cost 50 us for a 32 KiB operand.  Four 8-byte loads in flight per lane keep a large array
// at the card's read rate.
constexpr int kAmaxBlocks = 512, kAmaxUnroll = 4;

__global__ void __launch_bounds__(256)
amax_kernel(const float2* __restrict__ x, int64_t n, uint32_t* amax) {
  __shared__ float red[4];
  float m = 0.f;
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (; i + (kAmaxUnroll - 1) * step < n; i += kAmaxUnroll * step) {
    float2 v[kAmaxUnroll];
#pragma unroll
    for (int u = 0; u < kAmaxUnroll; ++u) v[u] = x[i + u * step];
#pragma unroll
    for (int u = 0; u < kAmaxUnroll; ++u) m = fmaxf(m, cmax(v[u]));
  }
  for (; i < n; i += step) m = fmaxf(m, cmax(x[i]));
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) atomicMax(amax, __float_as_uint(fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]))));
}

__global__ void zero_u32(uint32_t* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

hipError_t launch_amax(hipStream_t st, const float2* x, int64_t n, uint32_t* amax) {
  hipLaunchKernelGGL(zero_u32, dim3(1), dim3(64), 0, st, amax, 1);
  const unsigned blocks = (unsigned)std::min<int64_t>((n + 1023) / 1024, kAmaxBlocks);
  hipLaunchKernelGGL(amax_kernel, dim3(blocks), dim3(256), 0, st, x, n, amax);
  return hipGetLastError();
}

} // namespace qf
