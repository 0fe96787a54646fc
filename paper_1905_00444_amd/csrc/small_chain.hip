// Whole contraction of one chain (bitstring x slice) in one workgroup, for plans whose tensors hold at
// most 2^11 elements (paper Sec. III-A: every slice of every bitstring is an independent network).
//
// Such a step computes for a microsecond, but a kernel launch per step and operand takes 3 to 6, so a
// chain of 20 steps was launch time throughout.  Here a workgroup runs all steps of its chain, forward and
// (backward plans) in reverse, with barriers between steps instead of launches; the chains of a launch
// run on different CUs.  Bound by latency, so a result that the next step reads stays in LDS, and the
// operands that are in memory before a step (world-lines; in reverse the forward results) are loaded
// during the step before it.
//
// Every index has dimension 2, so an operand element's address is the OR of bit scatters of its row,
// column and contracted indices: world-line slices, results and environments are read and written
// where they lie, without permuted copies.  All three products of a step
//   forward  C[m][n]    = sum_k A[m][k] B[n][k]
//   env of A E[m][k]    = sum_n env(C)[m][n] conj(B[n][k])
//   env of B E[n][k]    = sum_m env(C)[m][n] conj(A[m][k])
// are out[i][j] = sum_l X[i][l] Y[l][j] with other names: X and Y are gathered into LDS as [l][i] and
// [l][j], a thread takes 1 x 1 to 2 x 2 outputs, and where there are fewer outputs than threads, l is cut
// over the rest of them.  FP32 throughout.
//
// Measured (call to result): one 4x4 chain of depth 8, 15 steps, 109 us by launches, 33 here (of depth 16,
// 2^10 elements, 101 and 38), with gradient 309 and 91; 1000 chains 2014 and 83, with gradient 5930 and 224.
// Row and column scattered bit by bit in loops, and each step's scalars fetched on arrival: 40 (50), 99.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "cgemm_common.h"

namespace qf {

constexpr int kSmLog = 9;
constexpr int kSmThreads = 1 << kSmLog;
constexpr int kSmMax = 1 << kSmallMaxBits;
constexpr int kSmRegs = kSmMax / kSmThreads;

// Address of element i < 2^kSmallMaxBits: bits from b.n() on are zero in i.
template <int BITS = kSmallMaxBits>
__device__ __forceinline__ int scatter_bits(int i, SmallBits b) {
  int off = 0;
#pragma unroll
  for (int k = 0; k < BITS; ++k) off |= ((i >> k) & 1) << b.pos(k);
  return off;
}

struct SmallLds {
  float2 x[kSmMax];       // X[l][i]
  float2 y[kSmMax];       // Y[l][j]
  float2 c[kSmMax];       // the previous step's result (environment)
  float2 red[kSmThreads];
  uint32_t amax[2 * kSmallMaxSteps + 1];  // leaves, then results
  int e[2 * kSmallMaxSteps + 1];
  int base[kSmallMaxSteps + 1];           // fixed bits of the world-lines
};

// Orders LDS accesses only: loads and stores of global memory stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// This thread's elements of the operand p in the order of b.
__device__ __forceinline__ void fetch(float2 (&r)[kSmRegs], const float2* p, SmallBits b) {
  static_assert(kSmRegs == 4, "two bits above the thread's");
  const int at = scatter_bits<kSmLog>(threadIdx.x, b), size = 1 << b.n();
  const int hi[4] = {0, 1 << b.pos(kSmLog), 1 << b.pos(kSmLog + 1), 1 << b.pos(kSmLog) | 1 << b.pos(kSmLog + 1)};
#pragma unroll
  for (int q = 0; q < kSmRegs; ++q)
    if ((int)threadIdx.x + q * kSmThreads < size) r[q] = p[at | hi[q]];
}

__device__ __forceinline__ void stash(float2* dst, const float2 (&r)[kSmRegs], int bits, bool conj) {
#pragma unroll
  for (int q = 0; q < kSmRegs; ++q) {
    const int t = threadIdx.x + q * kSmThreads;
    if (t < 1 << bits) dst[t] = conj ? make_float2(r[q].x, -r[q].y) : r[q];
  }
}

__device__ __forceinline__ void cfma(float2& c, float2 a, float2 b) {
  c.x = fmaf(a.x, b.x, c.x);
  c.x = fmaf(-a.y, b.y, c.x);
  c.y = fmaf(a.x, b.y, c.y);
  c.y = fmaf(a.y, b.x, c.y);
}

// One TI x TJ tile of outputs per thread; they are 2^gi rows and 2^gj columns apart.
template <int TI, int TJ, class Out>
__device__ __forceinline__ void small_tile(const SmallLds& s, int ib, int jb, int L, Out&& out) {
  const int gi = ib - (TI - 1), gj = jb - (TJ - 1), t = threadIdx.x;
  const int i0 = t >> gj, j0 = t & ((1 << gj) - 1);
  float2 acc[TI][TJ];
#pragma unroll
  for (int u = 0; u < TI; ++u)
#pragma unroll
    for (int w = 0; w < TJ; ++w) acc[u][w] = make_float2(0.f, 0.f);
#pragma unroll 4
  for (int l = 0; l < L; ++l) {
    float2 a[TI], b[TJ];
#pragma unroll
    for (int u = 0; u < TI; ++u) a[u] = s.x[(l << ib) + i0 + (u << gi)];
#pragma unroll
    for (int w = 0; w < TJ; ++w) b[w] = s.y[(l << jb) + j0 + (w << gj)];
#pragma unroll
    for (int u = 0; u < TI; ++u)
#pragma unroll
      for (int w = 0; w < TJ; ++w) cfma(acc[u][w], a[u], b[w]);
  }
#pragma unroll
  for (int u = 0; u < TI; ++u)
#pragma unroll
    for (int w = 0; w < TJ; ++w) out(((i0 + (u << gi)) << jb) + j0 + (w << gj), acc[u][w]);
}

// out(i 2^jb + j, value) of all 2^(ib+jb) <= kSmMax outputs, from X and Y in LDS.
template <class Out>
__device__ __forceinline__ void small_product(SmallLds& s, int ib, int jb, int lb, Out&& out) {
  static_assert(kSmallMaxBits == kSmLog + 2, "tiles cover the outputs");
  const int tid = threadIdx.x, L = 1 << lb, ob = ib + jb;
  if (ob == kSmLog + 2 && ib >= 1 && jb >= 1) return small_tile<2, 2>(s, ib, jb, L, out);
  if (ob == kSmLog + 1 && jb >= 1) return small_tile<1, 2>(s, ib, jb, L, out);
  if (ob >= kSmLog) {  // also the rare single rows and columns of more outputs
    for (int t = tid; t < 1 << ob; t += kSmThreads) {
      const int i = t >> jb, j = t & ((1 << jb) - 1);
      float2 acc = make_float2(0.f, 0.f);
#pragma unroll 4
      for (int l = 0; l < L; ++l) cfma(acc, s.x[(l << ib) + i], s.y[(l << jb) + j]);
      out(t, acc);
    }
    return;
  }
  const int sb = min(kSmLog - ob, lb), seg = 1 << sb;  // l cut over 2^sb threads per output
  if (tid < 1 << (ob + sb)) {
    const int o = tid >> sb, i = o >> jb, j = o & ((1 << jb) - 1);
    float2 acc = make_float2(0.f, 0.f);
#pragma unroll 4
    for (int l = tid & (seg - 1); l < L; l += seg) cfma(acc, s.x[(l << ib) + i], s.y[(l << jb) + j]);
    if (sb == 0)
      out(o, acc);
    else
      s.red[tid] = acc;
  }
  if (sb > 0) {
    lds_barrier();
    if (tid < 1 << ob) {
      float2 v = make_float2(0.f, 0.f);
      for (int k = 0; k < seg; ++k) {  // in order
        const float2 r = s.red[(tid << sb) + k];
        v.x += r.x;
        v.y += r.y;
      }
      out(tid, v);
    }
  }
}

__device__ __forceinline__ int small_exp(uint32_t bits) {
  const float m = __uint_as_float(bits);
  if (!(m > 0.f) || !(m <= 3.0e38f)) return 0;
  int e;
  frexpf(m, &e);
  return e < -62 ? -62 : (e > 62 ? 62 : e);
}

// Bits of the largest m >= 0 of the wave: rows of 16 by DPP, then the four rows.
__device__ __forceinline__ uint32_t wave_max_bits(float m) {
  int v = __float_as_int(m);  // the order of non-negative floats
  v = max(v, __builtin_amdgcn_mov_dpp(v, 0xb1, 0xf, 0xf, true));   // lane ^ 1
  v = max(v, __builtin_amdgcn_mov_dpp(v, 0x4e, 0xf, 0xf, true));   // lane ^ 2
  v = max(v, __builtin_amdgcn_mov_dpp(v, 0x141, 0xf, 0xf, true));  // mirrored in 8
  v = max(v, __builtin_amdgcn_mov_dpp(v, 0x140, 0xf, 0xf, true));  // mirrored in 16
  const int a = max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16));
  return (uint32_t)max(a, max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

template <bool BACKWARD>
__global__ void __launch_bounds__(kSmThreads)
small_chain_kernel(SmallArgs a, const SmallStep* __restrict__ steps) {
  __shared__ SmallLds s;
  const int tid = threadIdx.x, g = blockIdx.x, S = a.n_steps, n = a.n_leaves;
  int64_t b, sl;
  chain_of(a.grp, g, b, sl);
  if (tid == 0) a.chain_b[g] = (int32_t)b;
  if (b < 0) return;  // idle chain (the whole workgroup)
  float2* mine = a.scratch + (int64_t)g * a.chain_elems;
  // leaves: magnitudes at most 1 (world-line entries), exponent 0
  for (int t = tid; t < n + S; t += kSmThreads) {
    s.amax[t] = t < n ? 0x3f800000u : 0u;
    s.e[t] = 0;
    if (t < n) s.base[t] = (int)leaf_base(a.grp, a.leaves[t], b, sl);
  }
  int warm = 0;  // the steps' lines into the scalar cache, together instead of one by one
#pragma unroll 8
  for (int i = 0; i < S; ++i) warm |= steps[i].mb;
  asm volatile("" ::"s"(warm));
  lds_barrier();
  // where operand r of a step lies in memory
  auto place = [&](const SmallStep& st, int r) -> const float2* {
    return st.leaf[r] >= 0 ? a.wl + st.off[r] + s.base[st.leaf[r]] : mine + st.off[r];
  };
  float2 ra[kSmRegs], rb[kSmRegs], re[kSmRegs];
  SmallStep st = steps[0];
  if (st.leaf[0] >= 0) fetch(ra, place(st, 0), st.a_km);
  if (st.leaf[1] >= 0) fetch(rb, place(st, 1), st.b_kn);
  for (int i = 0; i < S; ++i) {
    const SmallStep nx = steps[i + 1 < S ? i + 1 : i];
    const bool lds0 = i > 0 && st.node[0] == n + i - 1, lds1 = i > 0 && st.node[1] == n + i - 1;
    if ((st.leaf[0] < 0 && !lds0) || (st.leaf[1] < 0 && !lds1))
      __syncthreads();  // an earlier step's result in memory
    else
      lds_barrier();    // the previous step's result and magnitude
    if (lds0) fetch(ra, s.c, st.a_km);
    else if (st.leaf[0] < 0) fetch(ra, place(st, 0), st.a_km);
    if (lds1) fetch(rb, s.c, st.b_kn);
    else if (st.leaf[1] < 0) fetch(rb, place(st, 1), st.b_kn);
    const int mb = st.mb, nb = st.nb, kb = st.kb;
    stash(s.x, ra, mb + kb, false);
    stash(s.y, rb, nb + kb, false);
    if (i + 1 < S) {
      if (nx.leaf[0] >= 0) fetch(ra, place(nx, 0), nx.a_km);
      if (nx.leaf[1] >= 0) fetch(rb, place(nx, 1), nx.b_kn);
    }
    float unscale = 1.f;
    int e_ab = 0;
    if (a.renorm) {
      e_ab = small_exp(s.amax[st.node[0]]) + small_exp(s.amax[st.node[1]]);
      unscale = ldexpf(1.f, -e_ab);
      if (tid == 0) s.e[n + i] = s.e[st.node[0]] + s.e[st.node[1]] + e_ab;
    }
    lds_barrier();
    const bool next = i + 1 < S && (nx.node[0] == n + i || nx.node[1] == n + i);
    float2* C = mine + st.c;
    float mx = 0.f;
    small_product(s, mb, nb, kb, [&](int o, float2 v) {
      v = make_float2(v.x * unscale, v.y * unscale);
      const int at = scatter_bits(o, st.c_mn);
      if (next) s.c[at] = v;
      if (BACKWARD || !next) C[at] = v;
      mx = fmaxf(mx, cmax(v));
    });
    if (a.renorm) {
      const uint32_t top = wave_max_bits(mx);
      if ((tid & 63) == 0) atomicMax(&s.amax[n + i], top);
    }
    st = nx;
  }
  if constexpr (!BACKWARD) {
    if (tid == 0) a.chain_e[g] = s.e[n + S - 1];  // written by this thread
    return;
  }
  // reverse: environments lie behind the forward tensors, in their layouts
  __syncthreads();  // the forward results are in memory
  for (int j = tid; j < 1 << a.root.n(); j += kSmThreads) {
    const double2 c = a.cot[(b << a.root.n()) + j];
    s.c[scatter_bits(j, a.root)] = make_float2((float)c.x, (float)c.y);
  }
  fetch(ra, place(st, 0), st.a_mk);
  fetch(rb, place(st, 1), st.b_nk);
  bool in_lds = true;  // the environment of the step's result
  for (int i = S - 1; i >= 0; --i) {
    const SmallStep nx = steps[i > 0 ? i - 1 : 0];
    const int mb = st.mb, nb = st.nb, kb = st.kb;
    const float2* E = mine + a.env + st.c;
    // the environment that the next step reads comes second, over that of this step's result
    const bool next0 = i > 0 && st.node[0] == n + i - 1, next1 = i > 0 && st.node[1] == n + i - 1;
    if (in_lds)
      lds_barrier();
    else
      __syncthreads();  // written by an earlier step of this pass
    auto product = [&](bool of_a, bool last) {
      const SmallBits order = of_a ? st.c_nm : st.c_mn;
      if (in_lds)
        fetch(re, s.c, order);
      else
        fetch(re, E, order);
      stash(s.x, re, mb + nb, false);
      if (of_a)
        stash(s.y, rb, nb + kb, true);
      else
        stash(s.y, ra, mb + kb, true);
      if (last && i > 0) {
        fetch(ra, place(nx, 0), nx.a_mk);
        fetch(rb, place(nx, 1), nx.b_nk);
      }
      lds_barrier();
      const int r = of_a ? 0 : 1, leaf = st.leaf[r];
      const SmallBits to_order = of_a ? st.a_mk : st.b_nk;
      const bool next = of_a ? next0 : next1;
      float2* to = leaf >= 0 ? a.env_wl + st.off[r] + s.base[leaf] : mine + a.env + st.off[r];
      small_product(s, of_a ? mb : nb, kb, of_a ? nb : mb, [&](int o, float2 v) {
        const int at = scatter_bits(o, to_order);
        if (next) {
          s.c[at] = v;
        } else if (leaf >= 0) {  // gathers from all chains that fixed the same bits
          atomicAdd(&to[at].x, v.x);
          atomicAdd(&to[at].y, v.y);
        } else {
          to[at] = v;
        }
      });
      if (!last) lds_barrier();
    };
    product(next1, false);
    product(!next1, true);
    in_lds = next0 || next1;
    st = nx;
  }
}

hipError_t launch_small_chain(hipStream_t st, const SmallArgs& a, bool backward) {
  if (backward)
    hipLaunchKernelGGL(small_chain_kernel<true>, dim3((unsigned)a.grp.G), dim3(kSmThreads), 0, st, a, a.steps);
  else
    hipLaunchKernelGGL(small_chain_kernel<false>, dim3((unsigned)a.grp.G), dim3(kSmThreads), 0, st, a, a.steps);
  return hipGetLastError();
}

} // namespace qf
