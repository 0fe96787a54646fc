// Device helpers shared by the complex GEMM kernels (cgemm.hip, cgemm_presplit.hip): vector
// types, bfloat16 / fp16 packing, the power-of-two renormalisation of stored tensors, and the
// per-lane expansion of the B operand for the real embedding of complex products.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "qf_kernels.h"

namespace qf {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

enum { P_FP32 = 0, P_BF16X3 = 1, P_FP16 = 2 };

typedef float f2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));

// One v_cvt_pk_bf16_f32; two scalar conversions and an OR took three instructions.
__device__ __forceinline__ uint32_t pack_bf16x2(float re, float im) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f2v){re, im}, bf2));
}
__device__ __forceinline__ float bf16_lo_to_f32(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi_to_f32(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ uint32_t pack_f16x2(float re, float im) {
  _Float16 a = (_Float16)re, b = (_Float16)im;
  return (uint32_t)__builtin_bit_cast(uint16_t, a) | ((uint32_t)__builtin_bit_cast(uint16_t, b) << 16);
}

// Index of element (m, n) of a C[M][N] result under the epilogue's output map (Renorm::om_*):
// m * N + n, or with om_nh > 0 the top om_nh bits of n placed above the low om_q bits of m.
__device__ __forceinline__ int64_t c_index(const Renorm& rn, int64_t m, int64_t n, int64_t N) {
  if (rn.om_nh == 0) return m * N + n;
  const int q = rn.om_q, nl = rn.om_nl, nh = rn.om_nh;
  const int64_t mlo = m & (((int64_t)1 << q) - 1), nlo = n & (((int64_t)1 << nl) - 1);
  return ((((m >> q) << (nh + q)) | ((n >> nl) << q) | mlo) << nl) | nlo;
}

// The same index as a sum: c_index(m, n) = c_row(m) + c_col(n), so a kernel's epilogue computes the
// two parts once per row and column of a lane.
__device__ __forceinline__ int64_t c_row(const Renorm& rn, int64_t m, int64_t N) {
  if (rn.om_nh == 0) return m * N;
  const int64_t mlo = m & (((int64_t)1 << rn.om_q) - 1);
  return (((m >> rn.om_q) << (rn.om_nh + rn.om_q)) | mlo) << rn.om_nl;
}
__device__ __forceinline__ int64_t c_col(const Renorm& rn, int64_t n) {
  if (rn.om_nh == 0) return n;
  return ((n >> rn.om_nl) << (rn.om_q + rn.om_nl)) | (n & (((int64_t)1 << rn.om_nl) - 1));
}

// 4 x 4 transposition among the lanes of a quad: an MFMA tile leaves lane (l16, lg) with rows
// 4 lg .. 4 lg + 3 of real column l16; afterwards it has row 4 lg + (l16 & 3) of the real columns
// 4 (l16 / 4) .. + 3, which are two neighbouring complex results, one 16-byte store.  The exchanges are
// DPP moves (no LDS traffic), and one store instead of two halves the epilogue's address arithmetic:
// on 2^21 x 64 x 64 the former epilogue's 64-bit shifts per element took as long as a third of the MFMAs.
template <int CTRL>
__device__ __forceinline__ float quad_move(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ f4 quad_transpose(f4 v) {
  constexpr int kXor1 = 0xB1, kXor2 = 0x4E;  // quad_perm [1,0,3,2] and [2,3,0,1]
  const bool odd = threadIdx.x & 1, upper = threadIdx.x & 2;
  const float a = quad_move<kXor1>(odd ? v[0] : v[1]), b = quad_move<kXor1>(odd ? v[2] : v[3]);
  const f4 w = odd ? (f4){a, v[1], b, v[3]} : (f4){v[0], a, v[2], b};
  const float c = quad_move<kXor2>(upper ? w[0] : w[2]), d = quad_move<kXor2>(upper ? w[1] : w[3]);
  return upper ? (f4){c, d, w[2], w[3]} : (f4){w[0], w[1], c, d};
}
__device__ __forceinline__ float cmax4(f4 v) {
  return fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3])));
}

// Store of the result pair at index j (even) of the mapped order: complex64, or its split-BF16 planes
// (Renorm::so_*; so_kbits >= 4, so a pair never straddles a row of the planes).
__device__ __forceinline__ void store_c2(float2* C, const Renorm& rn, int64_t j, f4 o) {
  if (rn.so_ld == 0) {
    *reinterpret_cast<f4*>(C + j) = o;
    return;
  }
  uint32_t* w = reinterpret_cast<uint32_t*>(C);
  const int64_t idx = (j >> rn.so_kbits) * rn.so_ld + (j & (((int64_t)1 << rn.so_kbits) - 1));
  const uint32_t h0 = pack_bf16x2(o[0], o[1]), h1 = pack_bf16x2(o[2], o[3]);
  *reinterpret_cast<uint2*>(w + idx) = make_uint2(h0, h1);
  *reinterpret_cast<uint2*>(w + rn.so_plane + idx) =
      make_uint2(pack_bf16x2(o[0] - bf16_lo_to_f32(h0), o[1] - bf16_hi_to_f32(h0)),
                 pack_bf16x2(o[2] - bf16_lo_to_f32(h1), o[3] - bf16_hi_to_f32(h1)));
}

// Scale exponent that brings max|x| to about 2^14 (FP16 max is 65504 ~ 2^16).
__device__ __forceinline__ int fp16_shift(const uint32_t* amax) {
  if (!amax) return 0;
  const float m = __uint_as_float(*amax);
  if (!(m > 0.f)) return 0;
  int e;
  frexpf(m, &e);  // m = f * 2^e, f in [0.5, 1)
  return 14 - e;
}

// Binary exponent e of a stored tensor's max magnitude (amax = f 2^e, f in [0.5, 1)), clamped so
// that the epilogue factor 2^-(e_A + e_B) stays a normal float; 0 for an all-zero tensor.
__device__ __forceinline__ int renorm_exp(const NodeScale* n) {
  uint32_t bits = 0;
#pragma unroll
  for (int i = 0; i < kScaleSlots; ++i) {
    const uint32_t v = n->slot[i].amax;
    bits = v > bits ? v : bits;
  }
  const float m = __uint_as_float(bits);
  if (!(m > 0.f) || !(m <= 3.0e38f)) return 0;
  int e;
  frexpf(m, &e);
  return e < -62 ? -62 : (e > 62 ? 62 : e);
}

// The scales of one batch element.
__device__ __forceinline__ Renorm renorm_of(Renorm rn, int64_t batch) {
  if (rn.c) {
    rn.a += batch * rn.a_step;
    rn.b += batch * rn.b_step;
    rn.c += batch * rn.c_step;
  }
  return rn;
}

// Operand scales for staging (FP16 only) and the epilogue factor.  Renormalised: FP16 operands are
// brought to max ~2^14 from their exponents, the result is stored times 2^-(e_A + e_B), and
// thread 0 of a batch element's first workgroup writes the result's exponent.  Otherwise FP16 scales from
// the given max magnitudes and undoes them in the epilogue; FP32 / BF16 use no scaling.
template <int PREC>
__device__ __forceinline__ void renorm_begin(const Renorm& rn, const uint32_t* amaxA, const uint32_t* amaxB,
                                             bool first, float& scale_a, float& scale_b, float& unscale) {
  int s_a = 0, s_b = 0, e_ab = 0;
  if (rn.c) {
    const int ea = renorm_exp(rn.a), eb = renorm_exp(rn.b);
    e_ab = ea + eb;
    if constexpr (PREC == P_FP16) {
      s_a = 14 - ea;
      s_b = 14 - eb;
    }
    if (first && threadIdx.x == 0)
      rn.c->slot[0].e = rn.a->slot[0].e + rn.b->slot[0].e + e_ab;
  } else if constexpr (PREC == P_FP16) {
    s_a = fp16_shift(amaxA);
    s_b = fp16_shift(amaxB);
  }
  scale_a = ldexpf(1.f, s_a);
  scale_b = ldexpf(1.f, s_b);
  unscale = ldexpf(1.f, -(s_a + s_b + e_ab));
}

__device__ __forceinline__ float cmax(float2 v) { return fmaxf(fabsf(v.x), fabsf(v.y)); }

// Raises the workgroup's slot of c's amax to its largest m.  The atomics on one slot are served about 12 ns
// apart (two million waves on one slot cost 20 ms), so a workgroup first compares with a value read
// before and issues its atomic only if it holds a larger one: amax only grows during the launch, so any
// value read is a lower bound of the final one and skipping is exact.  seen_amax is called
// between the main loop and the epilogue, whose stores hide the read; a read before the main loop is
// too old (most workgroups then hold more: 2^21 x 8 x 64 took 308 us instead of 240).
__device__ __forceinline__ uint32_t* amax_slot(NodeScale* c) {
  return &c->slot[(blockIdx.x + blockIdx.z) % kScaleSlots].amax;
}
__device__ __forceinline__ uint32_t seen_amax(const Renorm& rn) {
  return rn.c ? __hip_atomic_load(amax_slot(rn.c), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
}
__device__ __forceinline__ float wave_max(float m) {
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  return m;
}
// One atomic per workgroup of WAVES waves; red: LDS that no wave reads any more (every thread calls).
template <int WAVES>
__device__ __forceinline__ void raise_amax(NodeScale* c, float m, uint32_t seen, float* red) {
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = red[0];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) t = fmaxf(t, red[w]);
    if (__float_as_uint(t) > seen) atomicMax(amax_slot(c), __float_as_uint(t));
  }
}
// One per wave, read and compared at the end (kernels whose load ring must stay alone in flight).
__device__ __forceinline__ void record_amax(NodeScale* c, float m) {
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) {
    const uint32_t v = __float_as_uint(m);
    if (v > __hip_atomic_load(amax_slot(c), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(amax_slot(c), v);
  }
}


// B operand for real column (n, q): q = 0 -> (br, -bi), q = 1 -> (bi, br), per packed complex.
// Branch-free with per-lane constants: rot = 16 q (rotate the two halves), flip = q ? 0 : sign
// bit of the upper half.
struct BExpand {
  uint32_t rot, flip;
  __device__ explicit BExpand(int q) : rot(q ? 16u : 0u), flip(q ? 0u : 0x80000000u) {}
  __device__ __forceinline__ uint32_t operator()(uint32_t w) const {
    return __builtin_amdgcn_alignbit(w, w, rot) ^ flip;
  }
};

// Bits of i scattered to N packed positions (OpMap).
template <int N>
__device__ __forceinline__ uint32_t map_bits(uint32_t i, uint64_t v) {
  uint32_t off = 0;
#pragma unroll
  for (int b = 0; b < N; ++b) off |= ((i >> b) & 1) << ((v >> (5 * b)) & 31);
  return off;
}
__device__ __forceinline__ uint32_t map_row(const OpMap& m, uint32_t row) {
  return map_bits<12>(row & 0xfff, m.row[0]) | map_bits<12>(row >> 12, m.row[1]);
}
__device__ __forceinline__ int64_t map_base(const OpMap& m, int64_t batch, int64_t stride) {
  int64_t at = m.src_base + (m.base_table ? m.base_table[batch * m.base_stride] : batch * stride);
  if (m.dyn_bits) at += (int64_t)(*m.dyn_bits & 1) * m.dyn_stride;
  return at;
}

// Bitstring b (-1: idle) and slice s of chain g.
__device__ __forceinline__ void chain_of(const ChainGroup& c, int g, int64_t& b, int64_t& s) {
  int64_t off;  // slice offset in the range
  if (c.gpb > 0) {
    const int64_t q = c.chain0 / c.G;
    b = q / c.gpb;
    off = (q - b * c.gpb) * c.G + g;
    if (b * c.s_range >= c.n_chains || off >= c.s_range) b = -1;
  } else {
    const int64_t k = c.chain0 + g;
    b = k < c.n_chains ? k / c.s_range : -1;
    off = k - b * c.s_range;
  }
  s = c.s_begin + off;
}

// World-line offset of the bits that chain (b, s) fixes; 0 for an idle chain.
__device__ __forceinline__ int64_t leaf_base(const ChainGroup& c, const LeafDesc& d, int64_t b, int64_t s) {
  if (b < 0) return 0;
  int64_t base = 0;
  for (int i = 0; i < d.n_cut; ++i) base |= ((s >> d.shift[i]) & 1) << d.pos[i];
  if (d.xpos >= 0) base |= (int64_t)(c.bits[b * c.n_qubits + d.qubit] & 1) << d.xpos;
  return base;
}

// Clears the results' amax before a renormalised GEMM raises them (cgemm.hip).
hipError_t launch_renorm_reset(hipStream_t st, const Renorm& rn, int64_t batch);

} // namespace qf
