// Parts shared by the kernels of FP32 products (cgemm_f32.hip: FP32 MFMAs; cgemm_f32s.hip: six bfloat16
// products): launch arguments, the loads of operand tiles, the tile order and the epilogue.
#pragma once
#include "cgemm_common.h"

namespace qf {

constexpr int kFBK = 16;       // complex k per K-tile

struct F32Args {
  int64_t M, N, K;
  const float2* A;
  const float2* B;
  float2* C;
  int64_t lda, ldb;      // elements between rows (k contiguous) or between k's (row index contiguous)
  int64_t batch, sa, sb, sc;  // batch strides
  int64_t kc;            // k per chunk
  float2* P;             // partial tiles [chunk][batch][M][N] when gridDim.y > 1
  Renorm amap;           // MAPA: A is another product's result under its output map (om_*)
  Renorm rn;
  OpMap ma, mb;          // gathered operands (whole tiles only)
};

// Whether a grid's x takes that many workgroups: fewer than 2^32 work-items.
inline bool grid_takes(int64_t blocks, int64_t threads) { return blocks * threads < ((int64_t)1 << 32); }

// cgemm_f32s.hip: products that it takes instead (by shape alone: a result does not depend on the batch), and
// their launches (plain, or side 0 / 1 of an environment).
bool f32s_takes(int64_t M, int64_t N, int64_t K);
hipError_t launch_f32s(hipStream_t st, const F32Args& g, int split, bool env, bool side);

// Loads of one operand tile (ROWS x 16 complex) into registers: pairs of neighbours along the
// contiguous index.  T = 0: k contiguous, 8 threads per row; T = 1: rows contiguous.
// MAP: the operand is a result X[x][y] under an output map (or plain, om_nh = 0), read with its y along k
// (T = 0) or along the rows (T = 1); the runs of y are at least 8 elements long, so a pair stays together.
template <int ROWS, int NTH, int T, bool EDGE, bool MAP>
struct F32Loader {
  static constexpr int pairs = ROWS * kFBK / 2;
  static constexpr int per = (pairs + NTH - 1) / NTH;
  static constexpr bool partial = pairs % NTH != 0;
  const float2* p[per];
  int row[per], k[per];   // of the pair's first element
  float4 r[per];
  const float2* mbase;    // MAP: the operand's start, the tile's first row and k
  int64_t mrow, mk;

  __device__ __forceinline__ void init_map(const float2* base, int64_t row0, int64_t k0) {
    mbase = base;
    mrow = row0;
    mk = k0;
    init(base, 0, 0);
  }
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
  __device__ __forceinline__ void load(int64_t kt, int64_t ld, int64_t rows_left, int64_t k_left, const Renorm& map) {
#pragma unroll
    for (int i = 0; i < per; ++i) {
      if (partial && (int)threadIdx.x + i * NTH >= pairs) continue;
      const float2* q;
      if constexpr (MAP) {
        const int64_t x = T == 0 ? mrow + row[i] : mk + kt + k[i], y = T == 0 ? mk + kt + k[i] : mrow + row[i];
        q = mbase + (c_row(map, x, ld) + c_col(map, y));
      } else {
        q = p[i] + (T == 0 ? kt : kt * ld);
      }
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
  // put(row, k, pair) for the thread's pairs.
  template <class Put>
  __device__ __forceinline__ void each(Put&& put) const {
#pragma unroll
    for (int i = 0; i < per; ++i)
      if (!partial || (int)threadIdx.x + i * NTH < pairs) put(row[i], k[i], r[i]);
  }
};

// The same loads of an operand that is read through an OpMap: two elements of one row each, from where the row
// and k are scattered to.  Rows or k's run over the lanes, whichever has the lower address bits; the plan
// checks that the lowest address bits belong to a tile's own rows and k's, so that lines are used whole.
// Twice the load instructions, but no launch and no pass to copy the operand: 16 chains of 256^3 split-BF16
// products 17.0 us with copies made, 6.7 us each, before; 20 us gathered.  The 4x5 path sum 938 -> 772 us, 4x4
// sampling 3.01 -> 2.63 ms.
template <int ROWS, int NTH>
struct F32Gather {
  static constexpr int pairs = ROWS * kFBK / 2;
  static constexpr int per = (pairs + NTH - 1) / NTH;
  static constexpr bool partial = pairs % NTH != 0;
  const float2* p[per];
  int row[per], k[per];
  float4 r[per];
  uint32_t second, kc0;

  __device__ __forceinline__ void init_gather(const float2* base, const OpMap& m, int64_t row0, int64_t k0) {
    const uint32_t r0 = map_row(m, (uint32_t)row0);
    second = 1u << (m.k & 31);
    kc0 = (uint32_t)k0;
#pragma unroll
    for (int i = 0; i < per; ++i) {
      const int id = (int)threadIdx.x + i * NTH;
      row[i] = m.row_fast ? id % ROWS : id / (kFBK / 2);
      k[i] = 2 * (m.row_fast ? id / ROWS : id % (kFBK / 2));
      p[i] = base + (r0 | map_bits<7>(row[i], m.row[0]) | map_bits<4>(k[i], m.k));
    }
  }
  __device__ __forceinline__ void load_gather(int64_t kt, const OpMap& m) {
    const uint32_t off = map_bits<12>(kc0 + (uint32_t)kt, m.k);
#pragma unroll
    for (int i = 0; i < per; ++i) {
      if (partial && (int)threadIdx.x + i * NTH >= pairs) continue;
      const float2* q = p[i] + off;
      const float2 a = q[0], b = q[second];
      r[i] = make_float4(a.x, a.y, b.x, b.y);
    }
  }
  template <class Put>
  __device__ __forceinline__ void each(Put&& put) const {
#pragma unroll
    for (int i = 0; i < per; ++i)
      if (!partial || (int)threadIdx.x + i * NTH < pairs) put(row[i], k[i], r[i]);
  }
};

// Stores a wave's 16 TM x 16 TN results whose first is (m, n), returns the largest magnitude.  c_row and
// c_col add over disjoint bits of their index (and m N over sums), so a lane's own part is computed once
// and the rest is uniform.
template <int TM, int TN, bool EDGE, class Acc>
__device__ __forceinline__ float f32_store(float2* C, const Renorm& rn, int64_t m, int64_t n, int64_t M, int64_t N,
                                           float unscale, const Acc (&acc)[TM][TN]) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4;
  float2* own = C + (c_row(rn, m, N) + c_col(rn, n)) + (c_row(rn, lg, N) + c_col(rn, l16));
  int64_t row[TM], step[4], col[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) row[i] = c_row(rn, 16 * i, N);
#pragma unroll
  for (int r = 0; r < 4; ++r) step[r] = c_row(rn, 4 * r, N);
#pragma unroll
  for (int j = 0; j < TN; ++j) col[j] = c_col(rn, 16 * j);
  float mx = 0.f;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float2* at = own + (row[i] + step[r]);
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const float2 v = acc[i][j].at(r), o = make_float2(v.x * unscale, v.y * unscale);
        if (!EDGE || (m + 16 * i + 4 * r + lg < M && n + 16 * j + l16 < N)) at[col[j]] = o;
        mx = fmaxf(mx, cmax(o));  // zeros past the edge
      }
    }
  return mx;
}

struct F32Place { int64_t m0, n0, batch; };

// Tile id of a launch (batch-major): consecutive tiles go to one XCD (8 XCDs, dealt round-robin) and are
// rasterised in groups of row tiles.  32 bits: a launch has fewer tiles than a grid's blocks.
__device__ __forceinline__ F32Place f32_place(uint32_t id, uint32_t tiles_m, uint32_t tiles_n, uint32_t total, int BM,
                                              int BN) {
  const uint32_t ntiles = tiles_m * tiles_n;
  if ((total & 7) == 0) id = (id & 7) * (total >> 3) + (id >> 3);
  const uint32_t batch = id / ntiles, bid = id - batch * ntiles;
  constexpr uint32_t group = 8;
  const uint32_t per_group = group * tiles_n;
  const uint32_t first_m = bid / per_group * group, in_group = bid % per_group;
  const uint32_t gsize = (tiles_m - first_m) < group ? (tiles_m - first_m) : group;
  F32Place p;
  p.batch = batch;
  p.m0 = (int64_t)(first_m + in_group % gsize) * BM;
  p.n0 = (int64_t)(in_group / gsize) * BN;
  return p;
}

} // namespace qf
