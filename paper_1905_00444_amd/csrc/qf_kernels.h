// Host-side launchers of the HIP kernels (internal to the library).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qf {

// Power-of-two renormalisation state of one stored tensor: its true values are the stored values
// times 2^e; the largest |re| or |im| among the stored values is the largest of the slots' amax (float
// bits, which order like the values since they are non-negative).  The workgroups of a launch raise
// different slots, each in a 64-byte line of its own: atomics on one line are served 12 ns apart (1024
// workgroups that end together: 13 us on one slot, not measurable on 16).
constexpr int kScaleSlots = 16;
struct NodeScale {
  struct Slot { uint32_t amax; int32_t e; uint32_t pad[14]; } slot[kScaleSlots];  // e: slot 0 only
};

// Renormalised GEMM (all three null: off).  With e_A, e_B the binary exponents of the operands'
// amax (amax = f 2^e, f in [0.5, 1)), the GEMM stores C * 2^-(e_A + e_B), writes
// c's e = a's + b's + e_A + e_B from one thread, and raises c's amax to the stored result's largest
// magnitude (cleared by the launcher first).
struct Renorm {
  const NodeScale* a = nullptr;
  const NodeScale* b = nullptr;
  NodeScale* c = nullptr;
  // from one batch element's scale to the next one's: 0 where they share it, 1 where each keeps its own
  int a_step = 0, b_step = 0, c_step = 0;
  // Output map of the epilogue: with om_nh > 0, C[m][n] goes to index
  // ((m >> om_q) << (om_nh + om_q) | (n >> om_nl) << om_q | (m mod 2^om_q)) << om_nl | (n mod 2^om_nl),
  // i.e. the top om_nh bits of n sit above the low om_q bits of m (om_nl = log2 N - om_nh);
  // om_nh = 0: C[m][n] at m * N + n.
  int om_q = 0, om_nh = 0, om_nl = 0;
  // Split output (pre-split kernel, split-BF16): with so_ld > 0 the result goes out as the split
  // operand of its consumer instead of complex64: element j of the (mapped) order at word
  // (j >> so_kbits) * so_ld + (j mod 2^so_kbits) of a plane of bf16 hi pairs, its lo pair so_plane
  // words further (hi = bf16(x), lo = bf16(x - hi), as the splitting permute writes them).
  int so_kbits = 0;
  int64_t so_ld = 0, so_plane = 0;
  // c->amax has been cleared already (the start of the chain does it for all steps in one launch)
  bool cleared = false;
  // rows taken in another order (skinny products that read A through a map): bit i of a row is bit rp[i]
  // of the result's row, 5 bits per position, 12 to a word
  int rp_on = 0;
  uint64_t rp[2] = {0, 0};
};

// One instruction of a qubit's world-line program.
struct WlInstr {
  int32_t kind;   // 1: one-qubit gate; 2: bond from the q0 side of a diagonal gate (projector);
                  // 3: bond from the q1 side (diagonal entries)
  int32_t gate;   // index into the gate-value table
  int32_t bitpos; // bit position of the created bond in the world-line index (kinds 2, 3)
  int32_t out;    // index of the gate in the caller's order (gradient output row)
};

struct WlQubit {
  int64_t out_offset; // complex64 element offset of this qubit's tensor
  int32_t first;      // first instruction
  int32_t count;      // number of instructions
  int32_t nbond;      // number of bond bits m; tensor has 2^(m+1) elements, output bit on top
  int32_t pad;
};

// Build every world-line tensor: T_q[x][bonds] (x = output bit, most significant).
hipError_t launch_worldlines(hipStream_t st, const WlQubit* qubits, int n_qubits, int max_nbond,
                             const WlInstr* prog, const float2* gates, float2* out);

// Bit-permuting gather (see qf_permute in qfmi.h).  dyn_bits/dyn_stride: if dyn_bits != null,
// the source base gains dyn_bits[0] * dyn_stride (an output-bit value read on the device).
struct PermuteArgs {
  int nbits;
  int perm[64];
  int64_t src_base;
  float scale;
  const uint8_t* dyn_bits;
  int64_t dyn_stride;
  int conj;  // conjugate while copying
  // batched launches (grid z = batch): per-batch source/destination strides, and an optional
  // table of per-batch source base offsets base_table[z * base_stride]
  int batch = 1;
  int64_t src_bstride = 0, dst_bstride = 0;
  const int64_t* base_table = nullptr;
  int base_stride = 0;
  // split output: write bfloat16 hi = bf16(x) and lo = bf16(x - hi) of every complex number as
  // two planes of 2^nbits packed pairs (hi plane first) in the same 8 bytes per element
  int split = 0;
  // split output with padded rows: destination index j goes to word (j >> split_kbits) * split_ld
  // + (j & (2^split_kbits - 1)) of each plane, the lo plane 2^(nbits - split_kbits) * split_ld
  // words after the hi plane (split_ld = 0: dense planes)
  int split_kbits = 0;
  int64_t split_ld = 0;
  // split == 2: one plane of fp16 (re, im) pairs instead, each value times 2^(14 - e) where e is
  // the binary exponent of f16_scale->amax (the scale lands the tensor's largest entry near 2^14;
  // null: times 1), after `scale`
  const NodeScale* f16_scale = nullptr;
};
hipError_t launch_permute(hipStream_t st, const float2* src, float2* dst, const PermuteArgs& a);

// Adjoint of the gather: dst[src_base + sum_i bit_i(j) << perm[i]] += src[j] (same args).
hipError_t launch_scatter_add(hipStream_t st, const float2* src, float2* dst, const PermuteArgs& a);
// Batched over G chains: chain g's source at src + g * src_bstride, its extra base offset
// base_table[g * base_stride] (added to a.src_base); atomic additions; chains with chain_b < 0 skip.
hipError_t launch_scatter_add_batched(hipStream_t st, const float2* src, float2* dst, const PermuteArgs& a, int G,
                                      const int64_t* base_table, int base_stride, int64_t src_bstride,
                                      const int32_t* chain_b);

// Gradients of every gate from the world-line environments env (same layout as the
// world-lines): grad[out][e] += sum over tensor elements (complex64, 4 entries per gate).
hipError_t launch_worldline_grad(hipStream_t st, const WlQubit* qubits, int n_qubits, int max_nbond,
                                 const WlInstr* prog, const float2* gates, const float2* env, float2* grad);

// env_root[sum_t bit_t(j) << pos[t]] = cot[j] (complex128 -> complex64), j < 2^k.
hipError_t launch_seed_root(hipStream_t st, const double2* cot, int k, const int* pos, float2* env_root);
// Batched: env_root + g 2^k gets chain g's cotangent row cot + chain_b[g] 2^k (zeros if chain_b < 0).
hipError_t launch_seed_root_batched(hipStream_t st, const double2* cot, int k, const int* pos, int G,
                                    const int32_t* chain_b, float2* env_root);

// Measured ceilings (ceiling.hip): a register-only MFMA loop of `iters` trips over
// ceiling_mfma_blocks() workgroups (flops of one launch: ceiling_mfma_flops), and a streaming copy
// of `bytes` (a positive multiple of 16 KiB) from src to dst.
int64_t ceiling_mfma_blocks();
double ceiling_mfma_flops(int precision, int64_t iters);
hipError_t launch_ceiling_mfma(hipStream_t st, int precision, float* sink, int64_t iters);
hipError_t launch_stream_copy(hipStream_t st, const void* src, void* dst, int64_t bytes);

hipError_t launch_zero(hipStream_t st, void* p, size_t bytes);

// Per-leaf description of the bits fixed per chain (a chain is one bitstring x one slice).
constexpr int kMaxLeafCut = 24;
struct LeafDesc {
  int32_t n_cut;                 // fixed cut bits of this world-line
  int32_t xpos;                  // bit position of the output bit, -1 if the qubit is open
  int32_t qubit;
  int32_t pad;
  int32_t shift[kMaxLeafCut];    // bit of the slice id
  int32_t pos[kMaxLeafCut];      // bit position in the world-line
};

// Chains of a launch group.  gpb == 0: chain g is c = chain0 + g in bitstring-major order, b = c / s_range,
// s = s_begin + c % s_range, idle past n_chains.  gpb > 0 (groups per bitstring): group q = chain0 / G
// holds slices s_begin + (q mod gpb) G + g of bitstring b = q / gpb, idle past s_begin + s_range.
struct ChainGroup {
  int64_t chain0;
  int32_t G, n_qubits;
  const uint8_t* bits;  // device, n_qubits bytes per bitstring
  int64_t s_begin, s_range, n_chains, gpb;
};

// One world-line operand that is gathered at the start of a chain (or launch group) rather than by a
// permute of its own: element j of chain g's copy is src[base(g) + sum_i bit_i(j) << perm[i]], base from
// the world-line's LeafDesc, written as complex64 or in the forms of PermuteArgs::split.
constexpr int kGatherMaxBits = 14;
struct GatherJob {
  int64_t src;         // complex64 elements into the world-lines
  int64_t dst;         // bytes into the workspace
  int64_t dst_bstride; // complex64-sized elements between chains
  int32_t leaf, step;  // LeafDesc index; step that reads the copy
  int32_t batch;       // chains that have a copy of their own (1: shared)
  int32_t nbits, split, split_kbits;
  int64_t split_ld, split_plane;
  int32_t scale_node;  // split == 2: the NodeScale that gives the fp16 scale, else -1
  int8_t perm[kGatherMaxBits];
};
// A block of the launch: 1024 elements of one job from `first` on.
struct GatherBlock { int32_t job, first; };
constexpr int kGatherChunk = 1024;
constexpr int kMaxChainSteps = 256;
struct StepMask { uint64_t w[kMaxChainSteps / 64]; };

// Start of a chain group, in one launch: base_table[g * n_leaves + l] = offset of leaf l's fixed bits and
// chain_b[g] = bitstring (-1 for an idle chain) if base_table is given; the maxima of the steps i in `run`
// cleared if scales is given (steps' scales behind the leaves', chain_scales of them per step: 1, or the chains
// that the layout has room for); and the gathers of the jobs whose step is in `run`.
hipError_t launch_chain_begin(hipStream_t st, const ChainGroup& grp, int n_leaves, const LeafDesc* leaves,
                              int64_t* base_table, int32_t* chain_b, int n_steps, const StepMask& run, NodeScale* scales, int chain_scales,
                              const GatherJob* jobs, const GatherBlock* blocks, int n_blocks, const float2* wl, char* ws);
// out[chain_b[g]][j] += root[g root_stride + sum_t bit_t(j) << pos[t]] for g = 0..G-1 in order (FP64), times 2^e
// of root_scale[g root_scale_step], or of chain g's own exponent if chain_e is given.
hipError_t launch_slice_accumulate_batched(hipStream_t st, const float2* root, int64_t root_stride, int k, const int* pos,
                                           int G, const int32_t* chain_b, double2* out,
                                           const NodeScale* root_scale = nullptr, int root_scale_step = 0,
                                           const int32_t* chain_e = nullptr);

// Whole chains of small tensors, a workgroup each (small_chain.hip).
constexpr int kSmallMaxBits = 11;    // elements of any operand or result
constexpr int kSmallMaxSteps = 128;
// Bit i of an index goes to bit pos(i) < 32 of an address: up to 12 positions of 5 bits, and their number.
struct SmallBits {
  uint64_t v;
  __host__ __device__ int n() const { return (int)(v >> 60); }
  __host__ __device__ int pos(int i) const { return (int)(v >> (5 * i)) & 31; }
  void push(int p) { v = (v | (uint64_t)p << (5 * n())) + ((uint64_t)1 << 60); }
};
struct SmallStep {
  int64_t off[2], c;      // elements: A, B (into the world-lines for leaves, else the chain's scratch), C
  int32_t leaf[2];        // world-line index of A, B, or -1
  int32_t node[2];
  int32_t mb, nb, kb, pad;
  SmallBits a_km, a_mk, b_kn, b_nk, c_mn, c_nm;  // tensors as [k][m] (m the low bits), and so on
};
struct SmallArgs {
  ChainGroup grp;
  const SmallStep* steps;
  int n_steps, n_leaves;
  const LeafDesc* leaves;
  const float2* wl;
  float2* scratch;        // chain_elems per chain
  int64_t chain_elems;
  int renorm;
  int32_t *chain_b, *chain_e;
  // backward: cotangents, the root's output bits, environments (world-lines'; nodes' behind the tensors)
  const double2* cot;
  SmallBits root;
  float2* env_wl;
  int64_t env;
};
hipError_t launch_small_chain(hipStream_t st, const SmallArgs& a, bool backward);

// Split-BF16 GEMM on operands split by the permute (hi plane then lo plane per batch element), or
// FP16 GEMM on operands scaled and converted by the permute (one plane); precision P_BF16X3 / P_FP16
// (cgemm_common.h), 1 / 2 as qf_precision.
bool cgemm_presplit_fits(int64_t M, int64_t N, int64_t K, int precision = 1);
bool cgemm_presplit_pays(int64_t M, int64_t N, int64_t K, int precision);
hipError_t launch_cgemm_presplit(hipStream_t st, int64_t M, int64_t N, int64_t K, const void* A, const void* B,
                                 float2* C, int64_t batch, int64_t sa, int64_t sb, int64_t sc,
                                 const Renorm& rn = Renorm{}, int64_t lda = 0, int64_t ldb = 0, int precision = 1);

// Batched complex GEMM, C[m][n] = sum_k A[m][k] B[n][k].
hipError_t launch_cgemm(hipStream_t st, int precision, int64_t M, int64_t N, int64_t K,
                        const float2* A, const float2* B, float2* C, int64_t batch, int64_t sa,
                        int64_t sb, int64_t sc);
// GEMM kernel variants (GEMM_AUTO: chosen from the shape).
enum {
  GEMM_AUTO = 0,
  GEMM_TILED_4X4 = 1,  // 256 threads, 128 x 64 complex block tile (FP32: 64 x 64)
  GEMM_TILED_2X2 = 2,  // 64 x 32
  GEMM_TILED_1X2 = 3,  // 32 x 32
  GEMM_LARGE = 4,      // 512 threads, 256 x 128, double-buffered LDS (FP32: 64 x 64)
  GEMM_SKINNY = 5,     // B in LDS, SIMT FP32 (N K <= 4096, K <= 64)
  GEMM_SPLITK = 6,     // one workgroup per output (M N <= 4096), SIMT FP32
  GEMM_SIMT = 7,       // one thread per output, SIMT FP32
  GEMM_TALL = 8,       // M large, N and K <= 64: B in LDS, A streamed into registers (HBM-bound)
  GEMM_F32 = 9,        // FP32 MFMA tiles for any shape (the tile follows the launch)
  GEMM_N_VARIANTS = 10
};
// Tiles of the FP32 kernel (cgemm_f32.hip): by the launch, among them those of cgemm_f32s.hip or (plain) not, or given.
enum { F32_AUTO = 0, F32_PLAIN, F32_64X64, F32_64X32, F32_32X32, F32_128X16, F32_32X16 };
bool cgemm_variant_fits(int precision, int64_t M, int64_t N, int64_t K, int variant);
// blocks_per_tile: workgroups that a launch makes per output tile (batch x K-chunks).
int cgemm_default_variant(int precision, int64_t M, int64_t N, int64_t K, int64_t blocks_per_tile = 1);

// An operand that a product reads in another order than [row][k]: element (row, k) lies where the row's and k's
// bits are scattered to (5 bits per position, 12 to a word), from src_base + the dynamic output bit's
// offset + the chain's table entry (world-lines) or the chain's stride on.
struct OpMap {
  int on = 0;              // 2: [row][k] as it is, only elsewhere
  int row_fast = 0;        // the row's lowest bit is the lower one in memory
  uint64_t k = 0, row[2] = {0, 0};
  int64_t src_base = 0;
  const uint8_t* dyn_bits = nullptr;
  int64_t dyn_stride = 0;
  const int64_t* base_table = nullptr;
  int64_t base_stride = 0;
};
constexpr int kMapKBits = 12, kMapRowBits = 24;

// Same, with optional operand max magnitudes for FP16 scaling (ignored when rn is on: then the
// FP16 operands are scaled from rn.a / rn.b), optional renormalisation, and a kernel variant
// (one that does not fit the shape falls back to GEMM_AUTO).  flags: GEMM_DIRECT, a call of its own
// rather than a plan's step: the kernel and the cut of K then follow the batch and the scratch too; GEMM_PLAIN, FP32
// products on FP32 MFMAs only.
enum { GEMM_DIRECT = 1, GEMM_PLAIN = 2 };
hipError_t launch_cgemm_ex(hipStream_t st, int precision, int64_t M, int64_t N, int64_t K, const float2* A,
                           const float2* B, float2* C, int64_t batch, int64_t sa, int64_t sb, int64_t sc,
                           const uint32_t* amaxA, const uint32_t* amaxB, const Renorm& rn = Renorm{},
                           int variant = GEMM_AUTO, float2* scratch = nullptr, size_t scratch_bytes = 0,
                           const OpMap* ma = nullptr, const OpMap* mb = nullptr, int flags = 0);
// Whether that call (GEMM_AUTO) reads operands through maps.
bool cgemm_reads_maps(int precision, int64_t M, int64_t N, int64_t K, int64_t batch);
// ... and takes A's rows in any order (by shape alone).
bool cgemm_takes_row_order(int precision, int64_t M, int64_t N, int64_t K);
// FP32 MFMA product of any shape (cgemm_f32.hip).  *split: K-chunks wanted, set to those used (partials
// in P, summed by launch_split_reduce).
hipError_t launch_cgemm_f32(hipStream_t st, int64_t M, int64_t N, int64_t K, const float2* A, const float2* B,
                            float2* C, int64_t batch, int64_t sa, int64_t sb, int64_t sc, const Renorm& rn, int* split,
                            float2* P, int tile = F32_AUTO, const OpMap* ma = nullptr, const OpMap* mb = nullptr);
// Environments of a product C[M][N] = sum_K A[M][K] B[N][K] from that of C (env, under C's output map), in FP32
// without transposed copies: side 0: out[M][K] = sum_n env[m][n] conj(other[n][k]) with other = B; side 1:
// out[N][K] = sum_m env[m][n] conj(other[m][k]) with other = A.  Dense batch strides.
hipError_t launch_cgemm_f32_env(hipStream_t st, int side, int64_t M, int64_t N, int64_t K, const float2* env,
                                const float2* other, float2* out, int64_t batch, const Renorm& map, int* split,
                                float2* P, bool plain = false);
// The same with the split of K that the shape asks for, given the scratch (cgemm.hip).
hipError_t launch_env_gemm(hipStream_t st, int side, int64_t M, int64_t N, int64_t K, const float2* env,
                           const float2* other, float2* out, int64_t batch, const Renorm& map, float2* scratch,
                           size_t scratch_bytes, bool plain = false);
size_t env_gemm_scratch(int side, int64_t M, int64_t N, int64_t K, int64_t batch);
// Tall-skinny kernel (cgemm_tall.hip): powers of two, 8 <= N <= 64, 16 <= K <= 64.
bool cgemm_tall_fits(int precision, int64_t M, int64_t N, int64_t K);
hipError_t launch_cgemm_tall(hipStream_t st, int precision, int64_t M, int64_t N, int64_t K, const float2* A,
                             const float2* B, float2* C, int64_t batch, int64_t sa, int64_t sb, int64_t sc,
                             const uint32_t* amaxA, const uint32_t* amaxB, const Renorm& rn,
                             const OpMap& ma = OpMap{}, const OpMap& mb = OpMap{});
// Bytes of scratch that lets an MFMA launch of this shape split K over more workgroups (0: the
// launch fills the GPU without splitting, or its variant cannot split).
size_t cgemm_split_scratch(int precision, int64_t M, int64_t N, int64_t K, int64_t batch, int variant = GEMM_AUTO,
                           bool direct = false);

// p[i] = pseudo-random complex values, re and im uniform in [-1, 1) (hash of seed and i).
hipError_t launch_fill_random(hipStream_t st, float2* p, int64_t n, uint32_t seed);
// *amax = max |re|, |im| of x[0..n) (float bits).
hipError_t launch_amax(hipStream_t st, const float2* x, int64_t n, uint32_t* amax);

// out[j] += root[sum_t bit_t(j) << pos[t]] in complex128, j < 2^k.
hipError_t launch_slice_accumulate(hipStream_t st, const float2* root, int k, const int* pos,
                                   double2* out, const NodeScale* root_scale = nullptr);

} // namespace qf
