// What the projection kernels share: tile constants, the kernel argument block, and the epilogue
// that turns a finished 256 x 256 tile of logits (paper Sec. 3.3, Eq. 1) into the row's running
// softmax statistics, top-k list and target logit, or into the steering sweep's per-alpha
// statistics (Sec. 3.4).  The logits exist only in MFMA accumulators; everything here is private to
// the lane that owns the lens row.
#pragma once

#include "ll_common.h"

#include <limits.h>
#include <math.h>

#include <type_traits>

namespace ll {

struct GemmArgs {
  const uint16_t* A;        // [rows, lda] bf16 (this pass's rows)
  const float* inv_rms;     // [rows] or nullptr (rows already normalised)
  const uint16_t* gamma;    // [d] or nullptr
  const uint16_t* W;        // [V, d] bf16
  const int32_t* target;    // [rows] or nullptr
  const float* bias;        // [tiles * BM] fp32 (zero padded beyond V) or nullptr: the b of Eq. 1
  float4* stats;            // [rows, splits]     (m, S, T, z_target)
  uint2* top;               // [rows, splits, k]  (logit bits, id), sorted
  int64_t lda;              // row stride of A in elements
  int rows, d, V, k, splits, tiles, row_blocks;
  int last_row;             // of A, what is read for the rows past the end of a block: a row of zeros behind a panel, else the last row
  // steering sweep only (Sec. 3.4, Eq. 3 for several alpha in one pass):
  const float* u;           // [tiles * BM] fp32: W_U v, zero padded
  const float* eu;          // [2, tiles * BM / 16, 16, 16]: rows of e^(alpha u) and alpha u e^(alpha u) of 16 ids (see ll_epilogue_sweep.h)
  const float* shift_max;   // [tiles * BM / 16, 16]: per alpha the largest alpha u of 16 ids, with a margin; entry 15 the largest spread of any alpha u among them
  const float* shift_min;   // [tiles * BM / 16, 16]: per alpha the least
  const float* shift_tile;  // [tiles, 16]: per alpha the largest of a tile, with the margin
  const int* sweep_general; // nonzero: some |alpha u| is too large for the factored form; nullptr: the general form in any case
  float4* sweep_stats;      // [rows, n_alpha, splits]      (reference, S, T)
  float* sweep_ztgt;        // [rows, splits]               logit of the target id at alpha = 0
  uint2* sweep_top;         // [rows, n_alpha, splits, KS]  (logit bits, id), sorted
  int n_alpha, zero_alpha;  // zero_alpha: of nine, one that is zero, or -1
  float alphas[LL_SWEEP_MAX];
  // sharing top-k thresholds between the vocabulary splits of a row (nullptr: off)
  unsigned* bound;          // [rows] lower bounds on each row's k-th best logit, as ordered keys; zero at launch.  With classes: [classes, rows]
                            // the best logits of the row that each class of splits has seen (sweep: [k, n_alpha, rows])
  int classes;              // short calls: 0, or k, the classes that the splits are dealt into (see exchange_classes)
  int half_tiles;           // short calls: 0, or V in half tiles where the splits are cut between those
  int group_rows;           // row blocks that an XCD's workgroups share W_U's tiles between (see place_of)
  // sweeps that form u themselves (see ll_epilogue_sweep.h):
  float* u_out;             // u for the merge, [tiles * BM]
  int* exceeded;            // set once the factored form turns out not to do
  int* left_any;            // set once it leaves out a token, because of its |alpha u|, that the merge adds:
  float* left_z;            // [rows, splits, left_slots]: the logits of those tokens
  int* left_id;             // [row_blocks, splits, left_slots]: their ids
  int* left_n;              // [row_blocks, splits, 4]: how many (each wavefront's own count)
  const float* sampled;     // the largest |alpha u| of some vocabulary rows in SWEEP_SAMPLED parts
  const float* block_max;   // where u is given: the largest |u| of all, in SWEEP_BLOCK_MAX parts
  const float* direction;   // v
  const int* given;         // nonzero: u is there already (ll_unembed_direction_kernel), and is taken from there
  int only_general;         // the general form in any case
  int left_slots;           // most tokens that are left out of a split
  float alpha_most;         // largest |alpha|
};

using GemmKernel = void (*)(const GemmArgs);

// The direct-to-LDS kernels for a d that is not a multiple of 64 (ll_project_tail.hip); nullptr where there is none (the longest
// list with a bias).
GemmKernel tail_topk_kernel(int k, bool bias);
GemmKernel tail_sweep_kernel(bool lists);
// Those for calls of few tiles a workgroup, k <= 20 (ll_project_short.hip); ragged: d is not a multiple of 64.
GemmKernel short_topk_kernel(int k, bool bias, bool ragged);
// The general form of the steering sweep, for any d (see ll_epilogue_sweep.h).
GemmKernel general_sweep_kernel(bool lists);
// Both forms where the kernel forms u itself, any d (ll_project_sweep.hip).
GemmKernel whole_sweep_kernel(bool lists, bool general, bool ragged);

}  // namespace ll

namespace {

using namespace ll;

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

constexpr int BM = 256;          // vocabulary rows per tile (MFMA M side)
constexpr int BN = 256;          // lens rows per workgroup (MFMA N side)
constexpr int BK = 64;           // K step of the register-staged kernel
constexpr int NTHREADS = 256;    // 4 wavefronts, one per SIMD
constexpr int CHUNK_ROWS = 8192; // lens rows per pass
constexpr int MAX_SPLITS = 64;   // vocabulary splits per row block: one lane of the merging wavefront each
constexpr int MAX_PARTIALS = 256 * 256;   // rows of a pass x splits never exceeds rows per workgroup x workgroups
constexpr int NUM_XCD = 8;
constexpr int NUM_CU = 256;
constexpr float NEG_BIG = -3.0e38f;   // stands for "no logit" without the NaNs that -inf would breed
constexpr float LOG2E = 1.4426950408889634f;

// ---------------------------------------------------------------------------------------
// a3..a7: the fused kernels.
//
// One workgroup owns BN = 256 lens rows and one vocabulary split; it sweeps the split's 256-wide
// vocabulary tiles.  Per tile the logits Z^T[vocab, row] = W_tile . A^T are accumulated with bf16
// MFMAs, vocabulary on the M side, lens rows on the N side: wavefront w owns lens rows
// [64w, 64w+64) against all 256 vocabulary rows (8 x 2 accumulator tiles of 32 x 32 in the
// register-staged kernel, 16 x 4 tiles of 16 x 16 in the direct-to-LDS kernel).  In the
// accumulator layouts a lane holds vocabulary entries of ONE lens row per tile; after exchanging
// the row tiles between lane blocks (v_permlane32_swap, v_permlane16_swap) lane l of wavefront w
// holds all 256 logits of lens row 64w + l, so the whole epilogue is lane-private.
// ---------------------------------------------------------------------------------------
#define LL_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

typedef const float __attribute__((address_space(4)))* const_f32_ptr;   // read through scalar loads when the address is wave-uniform
typedef const int __attribute__((address_space(4)))* const_i32_ptr;

// Workgroup ids are dealt round-robin over the 8 XCDs; remap so that one XCD (one L2) gets an
// eighth of the numbers in a row.  Which row blocks and splits these are is place_of's matter (few
// rows: which parts), so that its CUs share A panels and W tiles.
__device__ __forceinline__ int xcd_logical_block() {
  const int per_xcd = gridDim.x / NUM_XCD;
  return (blockIdx.x % NUM_XCD) * per_xcd + blockIdx.x / NUM_XCD;
}

// The row block and the vocabulary split of a workgroup.  The 32 workgroups of an XCD are to be a rectangle that is near a square, R row
// blocks by 32 / R splits: per K stage R tiles of A and 32 / R of W come into its L2 from the fabric, 33 of 32 KB where they are of
// one row block (6.9 TB/s at 957 rows, d = 4096) and 12 at 4 by 8.  So the row blocks go in groups of four (up to seven: one group), of a
// group split after split, of a split block after block.  With at most eight splits an XCD has its four row blocks anyway.
// Whole calls, one row block after the other | so, in turn on one card: 957 rows, d = 4096, V = 128256 786 | 746 us; 777 rows, d = 1608, V = 50257 172 | 161;
// 4160 rows, d = 5120 4494 | 4471; sweeps of nine strengths whose u came from a pass of its own, 1500 rows, d = 4096 1454 | 1402, lists, 500 rows, d = 2560
// 555 | 547.
struct Place {
  int row_block, split;
};
inline int group_rows(int row_blocks, int splits) {   // row blocks of a group
  const int groups = splits <= NUM_XCD ? row_blocks : row_blocks <= 7 ? 1 : (row_blocks + 3) / 4;
  return (row_blocks + groups - 1) / groups;
}
__device__ __forceinline__ Place place_of(unsigned logical, const GemmArgs& p) {
  const unsigned rows = p.group_rows, of_group = rows * p.splits, g = logical / of_group, first = g * rows;
  const unsigned size = min(rows, p.row_blocks - first), at = logical - g * of_group, split = at / size;
  return {(int)(first + at - split * size), (int)split};
}

// ---------------------------------------------------------------------------------------
// Epilogue shared by both GEMM kernels.  State of one lens row, private to the lane that owns it.
// With m the running maximum: S = sum exp(z - m), T = sum exp(z - m) z.  Then
// logsumexp = m + log S and entropy = m + log S - T / S.
// The row's best KR logits (KR >= k) sit in registers, sorted: descending logit, and among equal
// logits ascending id.  A workgroup meets its vocabulary ids in increasing order, so a new
// candidate never outranks an equal logit already listed and a strict comparison is exact.
// ---------------------------------------------------------------------------------------
// Floats as unsigned keys of the same order, so that an integer atomic max is a float max.  Key 0
// is below every float's key: "nothing known yet".
__device__ __forceinline__ unsigned float_key(float f) {
  const unsigned b = __float_as_uint(f);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float key_float(unsigned k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}
constexpr unsigned KEY_NEG_INF = 0x007fffffu;   // float_key(-inf)
constexpr unsigned KEY_ZERO = 0x80000000u;      // float_key(+0); the key below it is -0's, an equal logit

// The largest float that ranks below a shared bound (-inf while there is none).  A logit EQUAL to the bound may still belong in
// the top k, since a smaller id wins a tie, so what is at or below the returned value, and no more, is out.
__device__ __forceinline__ float below_bound(unsigned key) {
  return key > KEY_NEG_INF ? key_float(key - (key == KEY_ZERO ? 2u : 1u)) : -INFINITY;
}

template <int KR>
struct RowState {
  float m = -INFINITY;
  float s = 0.f;
  float t = 0.f;
  float z_tgt = -INFINITY;  // logit of the target id, once its tile has passed
  int tgt = -1;             // target id of the row (-1: none)
  float shared_bound = -INFINITY;   // nothing at or below this can reach the row's final top k (see exchange_bound)
  int cls = -1;             // the split's class, if there are any
  bool first = true;        // no tile has been seen
  float lv[KR];             // top logits
  int li[KR];               // their ids
  // present: the lane has a lens row.  Nothing ever beats the list of one past the last row, which stands for a row of zeros.
  __device__ __forceinline__ void init(bool present) {
    const float lowest = present ? -INFINITY : INFINITY;
#pragma unroll
    for (int j = 0; j < KR; ++j) {
      lv[j] = lowest;
      li[j] = INT_MAX;
    }
  }
  __device__ __forceinline__ float tau() const { return lv[KR - 1]; }
  // A candidate has to beat both the row's own KR-th best and what the other splits report.
  __device__ __forceinline__ float threshold() const { return fmaxf(lv[KR - 1], shared_bound); }
  // Branch-free sorted insert: slot j takes its upper neighbour if the candidate goes above that
  // neighbour, the candidate if it goes exactly here, and keeps its entry otherwise.  For the
  // logits that is the median of (upper neighbour, own entry, candidate): one instruction.  Four
  // slots at a time, written as instructions: all comparisons of a block first, into four SGPR
  // pairs, then the medians, then the id selects.  Left to the compiler every comparison goes
  // through VCC with two wait states before the select that reads it (a VALU result in an SGPR
  // must not be read by the next two VALU instructions on this hardware).  The instructions are of
  // eight bytes and start at multiples of eight: from four bytes off, where a change anywhere before
  // may leave them, whole calls of lists of 24 take 3 to 4 % longer (1500 rows, d = 256, V = 20000: 133.4 us,
  // and 127.0 in place).
  __device__ __forceinline__ void insert(float z, int id) {
    static_assert(KR % 4 == 0, "blocks of four");
    unsigned long long above;   // lanes whose candidate ranks above the entry of the block's top slot
    asm("v_cmp_gt_f32_e64 %0, %1, %2" : "=s"(above) : "v"(z), "v"(lv[KR - 1]));
#pragma unroll
    for (int j = KR - 1; j >= 3; j -= 4) {
      const float up_v = j >= 4 ? lv[j >= 4 ? j - 4 : 0] : INFINITY;   // nothing ranks above slot 0's upper neighbour
      const int up_i = li[j >= 4 ? j - 4 : 0];
      unsigned long long m1, m2, m3, m4;
      asm(".p2align 3\n\t"                       // (see above)
          "v_cmp_gt_f32_e64 %9, %13, %2\n\t"     // above slot j-1
          "v_cmp_gt_f32_e64 %10, %13, %3\n\t"    // above slot j-2
          "v_cmp_gt_f32_e64 %11, %13, %4\n\t"    // above slot j-3
          "v_cmp_gt_f32_e64 %12, %13, %15\n\t"   // above slot j-4 (the next block's top slot)
          "v_med3_f32 %1, %2, %1, %13\n\t"       // new logits, top slot first: each reads its still old upper neighbour
          "v_med3_f32 %2, %3, %2, %13\n\t"
          "v_med3_f32 %3, %4, %3, %13\n\t"
          "v_med3_f32 %4, %15, %4, %13\n\t"
          "v_cndmask_b32_e64 %5, %5, %14, %0\n\t"    // id of slot j: the candidate's if it ranks above the old entry ...
          "v_cndmask_b32_e64 %5, %5, %6, %9\n\t"     // ... the upper neighbour's if it ranks above that one too
          "v_cndmask_b32_e64 %6, %6, %14, %9\n\t"
          "v_cndmask_b32_e64 %6, %6, %7, %10\n\t"
          "v_cndmask_b32_e64 %7, %7, %14, %10\n\t"
          "v_cndmask_b32_e64 %7, %7, %8, %11\n\t"
          "v_cndmask_b32_e64 %8, %8, %14, %11\n\t"
          "v_cndmask_b32_e64 %8, %8, %16, %12\n\t"
          "s_mov_b64 %0, %12"
          : "+s"(above), "+v"(lv[j]), "+v"(lv[j - 1]), "+v"(lv[j - 2]), "+v"(lv[j - 3]), "+v"(li[j]), "+v"(li[j - 1]),
            "+v"(li[j - 2]), "+v"(li[j - 3]), "=&s"(m1), "=&s"(m2), "=&s"(m3), "=&s"(m4)
          : "v"(z), "v"(id), "v"(up_v), "v"(up_i));
    }
  }
};

// The largest of three, as one instruction (the compiler's fmaxf first makes every operand that it can't trace a quiet number).
__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// Reads one accumulator element where it lives (an AGPR) at the point of use, so that the
// register allocator does not copy the whole 256-register tile into VGPRs ahead of the epilogue.
__device__ __forceinline__ float acc_read(float a) {
  float v;
  asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(a));
  return v;
}

// x[o] for a per-lane o in [0, 32): registers cannot be indexed by a lane-varying position, so
// pick through a binary tree of 31 selects.  The selects are written as instructions because the
// optimiser would otherwise fold the tree back into an indexed access and move the 32 values
// to scratch memory.
__device__ __forceinline__ float cndmask(float if_clear, float if_set, unsigned long long lanes) {
  float r;
  asm("v_cndmask_b32 %0, %1, %2, %3" : "=v"(r) : "v"(if_clear), "v"(if_set), "s"(lanes));
  return r;
}

__device__ __forceinline__ float select32(const float (&x)[32], int o) {
  const unsigned long long b0 = __builtin_amdgcn_ballot_w64((o & 1) != 0);
  const unsigned long long b1 = __builtin_amdgcn_ballot_w64((o & 2) != 0);
  const unsigned long long b2 = __builtin_amdgcn_ballot_w64((o & 4) != 0);
  const unsigned long long b3 = __builtin_amdgcn_ballot_w64((o & 8) != 0);
  const unsigned long long b4 = __builtin_amdgcn_ballot_w64((o & 16) != 0);
  // All five masks exist from here on, and two wait states have passed: on this hardware a VALU
  // result in an SGPR must not be read by a VALU instruction issued within the next two, and the
  // compiler, which would otherwise slide each comparison down to its first use, does not see
  // inside the select instructions below.
  unsigned long long m0_ = b0, m1_ = b1, m2_ = b2, m3_ = b3, m4_ = b4;
  asm volatile("s_nop 1" : "+s"(m0_), "+s"(m1_), "+s"(m2_), "+s"(m3_), "+s"(m4_));
  float a[16], b[8], c[4], e[2];
#pragma unroll
  for (int i = 0; i < 16; ++i) a[i] = cndmask(x[2 * i], x[2 * i + 1], m0_);
#pragma unroll
  for (int i = 0; i < 8; ++i) b[i] = cndmask(a[2 * i], a[2 * i + 1], m1_);
#pragma unroll
  for (int i = 0; i < 4; ++i) c[i] = cndmask(b[2 * i], b[2 * i + 1], m2_);
#pragma unroll
  for (int i = 0; i < 2; ++i) e[i] = cndmask(c[2 * i], c[2 * i + 1], m3_);
  return cndmask(e[0], e[1], m4_);
}

// x[o]: logit of vocabulary entry v0 + 32 I + o of the finished tile for this lane's row.  The swap
// hands the lower lane half the row tile j = 0 and the upper half j = 1, so that lane l owns row
// 64 w + l.
template <int I>
__device__ __forceinline__ void load_group(const f32x16 (&acc)[8][2], float (&x)[32]) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc_read(acc[I][0][r])),
                                               __float_as_uint(acc_read(acc[I][1][r])), false, false);
    const int o = 8 * (r >> 2) + (r & 3);
    x[o] = __uint_as_float(sw[0]);
    x[o + 4] = __uint_as_float(sw[1]);
  }
}

// The same for the accumulators of v_mfma_f32_16x16x32_bf16: 16 x 4 tiles of 16 x 16, where lane l
// holds, of tile (i, j), vocabulary rows 4 (l/16) + r (r = 0..3) of lens row 16 j + l%16.  Seen as
// blocks of 16 lanes, register j of lane block g has to go to register g of lane block j: a 4 x 4
// transpose, done by one round of v_permlane32_swap (blocks 2,3 of one register against blocks
// 0,1 of another) and one of v_permlane16_swap (odd blocks against even blocks).  Afterwards lane
// l owns lens row 64 w + l again, and register g holds vocabulary row 16 i + 4 g + r.
template <int I, int N>
__device__ __forceinline__ void load_group(const f32x4 (&acc)[N][4], float (&x)[32]) {
#pragma unroll
  for (int t = 0; t < 2; ++t) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      unsigned R0 = __float_as_uint(acc_read(acc[2 * I + t][0][r])), R1 = __float_as_uint(acc_read(acc[2 * I + t][1][r]));
      unsigned R2 = __float_as_uint(acc_read(acc[2 * I + t][2][r])), R3 = __float_as_uint(acc_read(acc[2 * I + t][3][r]));
      auto a = __builtin_amdgcn_permlane32_swap(R0, R2, false, false);
      auto b = __builtin_amdgcn_permlane32_swap(R1, R3, false, false);
      auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
      auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
      x[16 * t + r] = __uint_as_float(c[0]);
      x[16 * t + 4 + r] = __uint_as_float(c[1]);
      x[16 * t + 8 + r] = __uint_as_float(d[0]);
      x[16 * t + 12 + r] = __uint_as_float(d[1]);
    }
  }
}

// Bit o of the result: x[o] > tau0.  Two instructions per entry: the comparison, then the mask
// doubled plus the comparison's result as carry-in (entries taken from 31 down to 0).  Four
// entries at a time, comparisons first: a VALU result in an SGPR must not be read by the next two
// VALU instructions on this hardware.
__device__ __forceinline__ unsigned candidate_mask(const float (&x)[32], float tau0) {
  unsigned mask = 0;
#pragma unroll
  for (int o = 28; o >= 0; o -= 4) {
    unsigned long long c0, c1, c2, c3;
    asm("v_cmp_gt_f32_e64 %1, %5, %9\n\t"
        "v_cmp_gt_f32_e64 %2, %6, %9\n\t"
        "v_cmp_gt_f32_e64 %3, %7, %9\n\t"
        "v_cmp_gt_f32_e64 %4, %8, %9\n\t"
        "v_addc_co_u32_e64 %0, %1, %0, %0, %1\n\t"
        "v_addc_co_u32_e64 %0, %2, %0, %0, %2\n\t"
        "v_addc_co_u32_e64 %0, %3, %0, %0, %3\n\t"
        "v_addc_co_u32_e64 %0, %4, %0, %0, %4"
        : "+v"(mask), "=&s"(c0), "=&s"(c1), "=&s"(c2), "=&s"(c3)
        : "v"(x[o + 3]), "v"(x[o + 2]), "v"(x[o + 1]), "v"(x[o]), "v"(tau0));
  }
  return mask;
}

// Processes vocabulary entries [v0 + 32 I, v0 + 32 I + 32) of the finished tile for the lane's row.
template <int I, int KR, bool BIAS, class ACC>
__device__ __forceinline__ void epilogue_group(const ACC& acc, RowState<KR>& st, int v0, int V, bool partial,
                                               const float* __restrict__ bias) {
  float x[32];
  load_group<I>(acc, x);
  const int g0 = v0 + 32 * I;
  if (BIAS) {
    // The b of Eq. 1: the same 32 values for every lane, from a copy of the bias that is padded
    // to whole tiles.  Wave-uniform addresses through the constant address space: scalar loads,
    // which do not count against the vector-memory counter the operand rings are waited on.
    const_f32_ptr b = (const_f32_ptr)(uintptr_t)(bias + g0);
#pragma unroll
    for (int o = 0; o < 32; ++o) x[o] += b[o];
  }
  if (partial) {   // only the last tile of the vocabulary: a real branch (the empty asm keeps it one)
    asm volatile("");
#pragma unroll
    for (int o = 0; o < 32; ++o)
      if (g0 + o >= V) x[o] = NEG_BIG;
  }
  // a7: target gather
  const int tl = st.tgt - g0;
  if (__builtin_amdgcn_ballot_w64((unsigned)tl < 32u) != 0) {
#pragma unroll
    for (int o = 0; o < 32; ++o)
      if (tl == o) st.z_tgt = x[o];
  }
  // a5: online max / sum exp / sum exp * z
  float gmax = x[0];
#pragma unroll
  for (int o = 1; o < 32; ++o) gmax = fmaxf(gmax, x[o]);
  const float m_new = fmaxf(st.m, gmax);
  if (__builtin_amdgcn_ballot_w64(m_new > st.m) != 0) {
    const float sc = __builtin_amdgcn_exp2f((st.m - m_new) * LOG2E);   // first group: exp2(-inf) = 0
    st.s *= sc;
    st.t *= sc;
    st.m = m_new;
  }
  const float mb = st.m * LOG2E;
  float s4[4] = {0.f, 0.f, 0.f, 0.f}, t4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int o = 0; o < 32; ++o) {
    const float e = __builtin_amdgcn_exp2f(fmaf(x[o], LOG2E, -mb));
    s4[o & 3] += e;
    t4[o & 3] = fmaf(e, x[o], t4[o & 3]);
  }
  st.s += (s4[0] + s4[1]) + (s4[2] + s4[3]);
  st.t += (t4[0] + t4[1]) + (t4[2] + t4[3]);

  // a6: streaming top-k.  Only the lanes with a logit above their current KR-th best take part
  // (a divergent branch: the other lanes are masked off and cost no energy, which is what counts
  // on a power-limited chip): mark the candidates against that threshold, then insert them in
  // id order.
  if (gmax > st.threshold()) {
    const float tau0 = st.threshold();
    unsigned mask = candidate_mask(x, tau0);
    if (partial) mask &= (g0 + 32 <= V) ? 0xffffffffu : (g0 >= V ? 0u : (1u << (V - g0)) - 1u);
    while (mask != 0) {
      const int o = __builtin_ctz(mask);
      mask &= mask - 1;
      st.insert(select32(x, o), g0 + o);
    }
  }
}

// HALF: a tile of 128 entries (a short call's last tile).
template <int KR, bool BIAS, bool HALF, class ACC>
__device__ __forceinline__ void epilogue_tile(const ACC& acc, RowState<KR>& st, int v0, int V, const float* __restrict__ bias) {
  const bool partial = v0 + (HALF ? BM / 2 : BM) > V;
  // The accumulators are read below through inline asm, which the compiler's MFMA hazard
  // bookkeeping does not see: let the last MFMA of the tile drain first.
  asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");
  epilogue_group<0, KR, BIAS, ACC>(acc, st, v0, V, partial, bias);
  epilogue_group<1, KR, BIAS, ACC>(acc, st, v0, V, partial, bias);
  epilogue_group<2, KR, BIAS, ACC>(acc, st, v0, V, partial, bias);
  epilogue_group<3, KR, BIAS, ACC>(acc, st, v0, V, partial, bias);
  if constexpr (!HALF) {
    epilogue_group<4, KR, BIAS, ACC>(acc, st, v0, V, partial, bias);
    epilogue_group<5, KR, BIAS, ACC>(acc, st, v0, V, partial, bias);
    epilogue_group<6, KR, BIAS, ACC>(acc, st, v0, V, partial, bias);
    epilogue_group<7, KR, BIAS, ACC>(acc, st, v0, V, partial, bias);
  }
}

// The k-th best of a split's list (k <= KR, KR - k < 12).
// (Each entry goes through an empty asm statement: a plain chain of selects on k the optimiser
// folds into an indexed access and moves the whole list to scratch memory.)
template <int KR>
__device__ __forceinline__ float kth_best(const RowState<KR>& st, int k) {
  float best = st.lv[KR - 1];
#pragma unroll
  for (int j = KR - 2; j >= 0 && j >= KR - 12; --j) {
    float entry = st.lv[j];
    asm volatile("" : "+v"(entry));
    best = (k - 1 == j) ? entry : best;
  }
  return best;
}

// The workgroups that sweep other parts of the vocabulary for the same rows tell each other how
// good a logit has to be.  A split's k-th best logit so far is a lower bound on the row's k-th best
// overall, and nothing below the largest such bound can be in the final top k; without it every
// split collects candidates against its own slowly rising threshold (k (1 + ln(n/k)) insertions per
// row for n vocabulary entries: eight short streams cost far more than one long one).  After each
// tile a lane picks up the row's shared bound and publishes its own (atomic max on the key).  A
// logit EQUAL to the bound may still belong in the top k (a smaller id wins a tie), so the
// threshold is the next float below it (below_bound).  The final result does not depend on timing: a bound only
// removes entries that cannot be in the final top k; a split's own list may end up with fewer
// than k real entries, which the merge treats as absent.
// Placed at the END of the tile's epilogue: the operand loads in flight were sent before the
// epilogue began and have landed, so the wait for this one load costs one trip to the L2 and no
// more.  The publish needs no answer and is never waited for.
template <int KR>
__device__ __forceinline__ void exchange_bound(RowState<KR>& st, const GemmArgs& p, int my_row) {
  if (p.bound == nullptr) return;
  unsigned* const b = p.bound + min(my_row, p.rows - 1);
  asm volatile("" ::: "memory");
  const unsigned fresh = __hip_atomic_load(b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  st.shared_bound = below_bound(fresh);
  const float mine = kth_best(st, p.k);
  // (only what is news: the split whose bound it is, or any while all logits are equal, would send it after every tile)
  const unsigned key = float_key(mine);
  if (my_row < p.rows && key > fresh && key > KEY_NEG_INF) __hip_atomic_fetch_max(b, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("" ::: "memory");
}

// Short calls (ll_project_short.hip): where the splits are at least k, a better bound.  They are dealt into k classes, and a class's
// entry is the best logit that any of its splits has seen: k different ids, each at least the least of the k entries, which is
// the bound.  It ranks some k (1 + 1/2 + ... + 1/k) th of all ids seen by anyone, where the best k-th entry of one split of
// few tiles ranks several hundredth.

// The kernel's arguments that the exchange uses, read where it happens: kept in scalar registers through the epilogue they leave
// none to load a bias ahead.
typedef const GemmArgs __attribute__((address_space(4)))* const_args_ptr;
__device__ __forceinline__ const_args_ptr args_again() {
  auto args = (const_args_ptr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(args));
  return args;
}

template <int KR>
__device__ __forceinline__ unsigned least_of_classes(const RowState<KR>& st, unsigned* bound, int classes, int rows, int my_row, unsigned& own) {
  asm volatile("" : "+v"(my_row));   // (the address made anew each time rather than kept)
  const unsigned at = 4u * (unsigned)min(my_row, rows - 1);
  const unsigned char* b = reinterpret_cast<const unsigned char*>(bound);
  unsigned fresh[KR], least = 0xffffffffu;
#pragma unroll
  for (int c = 0; c < KR; ++c) {   // (all in flight together: past the last class the last one's again)
    fresh[c] = __hip_atomic_load(reinterpret_cast<const unsigned*>(b + at), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (c + 1 < classes) b += 4 * (int64_t)rows;
  }
  own = 0u;
#pragma unroll
  for (int c = 0; c < KR; ++c) {
    least = min(least, fresh[c]);
    own = c == st.cls ? fresh[c] : own;
  }
  return least;
}

// BIAS: and the next tile's biases, a word a line, into this XCD's L2, from where the epilogue's scalar loads come back in a third of
// the time.
template <int KR, bool BIAS>
__device__ __forceinline__ void exchange_classes(RowState<KR>& st, int v0, int my_row) {
  const const_args_ptr p = args_again();
  unsigned* const bound = p->bound;
  if (bound == nullptr) return;
  const int rows = p->rows;
  unsigned* b = bound + min(my_row, rows - 1);
  asm volatile("" ::: "memory");
  float warm = 0.f;
  if (BIAS) warm = p->bias[min(v0 + BM + 4 * (int)(threadIdx.x & 63), p->V - 1)];
  unsigned fresh;
  float mine;
  if (st.cls >= 0) {
    st.shared_bound = below_bound(least_of_classes(st, bound, p->classes, rows, my_row, fresh));
    b += (int64_t)st.cls * rows;
    mine = st.lv[0];
  } else {
    const int k = p->k;
    fresh = __hip_atomic_load(b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    st.shared_bound = below_bound(fresh);
    mine = kth_best(st, k);
  }
  if (BIAS) asm volatile("" : "+v"(warm));
  // (only what is news: the split whose bound it is, or any while all logits are equal, would send it after every tile)
  const unsigned key = float_key(mine);
  if (my_row < rows && key > fresh && key > KEY_NEG_INF) __hip_atomic_fetch_max(b, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("" ::: "memory");
}

// The largest of the tile's logits of the lane's own row.  (Vocabulary rows past the end are the last one's again, whose logit
// they repeat; with a bias the caller sees to it that there are none.)
template <bool BIAS, bool HALF, class ACC>
__device__ __forceinline__ float tile_max(const ACC& acc, int v0, const float* __restrict__ bias) {
  float q[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
  for (int i = 0; i < (HALF ? 8 : 16); ++i) {
    float4 b = make_float4(0.f, 0.f, 0.f, 0.f);
    if (BIAS) b = *reinterpret_cast<const float4*>(bias + v0 + 16 * i + 4 * ((threadIdx.x & 63) >> 4));
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float y0 = acc_read(acc[i][j][0]), y1 = acc_read(acc[i][j][1]), y2 = acc_read(acc[i][j][2]), y3 = acc_read(acc[i][j][3]);
      if (BIAS) {
        y0 += b.x;
        y1 += b.y;
        y2 += b.z;
        y3 += b.w;
      }
      q[j] = max3(max3(q[j], y0, y1), y2, y3);
    }
    LL_SCHED_FENCE();
  }
  // row block j's maxima are spread over the lane blocks: each lane block's own row block (see load_group)
  auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(q[0]), __float_as_uint(q[2]), false, false);
  auto c = __builtin_amdgcn_permlane32_swap(__float_as_uint(q[1]), __float_as_uint(q[3]), false, false);
  auto e = __builtin_amdgcn_permlane16_swap(a[0], c[0], false, false);
  auto f = __builtin_amdgcn_permlane16_swap(a[1], c[1], false, false);
  return max3(fmaxf(__uint_as_float(e[0]), __uint_as_float(e[1])), __uint_as_float(f[0]), __uint_as_float(f[1]));
}

// A split's first tile, whose list is empty: the splits tell each other their best logits before any of them builds its list.
// They come here at nearly the same time; a lane looks for the others' a few times (less than the insertions that it saves) and goes
// on with what there is.  Cycles of the epilogue of the first tile, without | with: 957 rows, d = 4096, V = 128256,
// k = 10: 66 800 | 31 000 (and 27 600 falling to 19 900 | 21 600 falling to 16 500 after that); 777 rows, d = 1608, V = 50257, k = 3
// with a bias: 39 900 | 31 400.
constexpr int FIRST_LOOKS = 8;
template <int KR, bool BIAS, bool HALF, class ACC>
__device__ __forceinline__ void first_bound(const ACC& acc, RowState<KR>& st, int v0, int my_row) {
  const const_args_ptr p = args_again();
  if (BIAS && v0 + (HALF ? BM / 2 : BM) > p->V) return;
  asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");   // as in epilogue_tile
  const float most = tile_max<BIAS, HALF>(acc, v0, p->bias);
  unsigned* const bound = p->bound;
  const int rows = p->rows, classes = p->classes;
  if (my_row < rows && most > -INFINITY)
    __hip_atomic_fetch_max(bound + (int64_t)st.cls * rows + my_row, float_key(most), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll 1
  for (int look = 0; look < FIRST_LOOKS; ++look) {
    asm volatile("" ::: "memory");
    unsigned own;
    const unsigned least = least_of_classes(st, bound, classes, rows, my_row, own);
    st.shared_bound = below_bound(least);
    if (__builtin_amdgcn_ballot_w64(least == 0u) == 0) break;
  }
  asm volatile("" ::: "memory");
}

// Per-(row, split) partial results: (m, S, T, z_target) and the k best (logit bits, id) pairs.
template <int KR>
__device__ __forceinline__ void epilogue_store(const GemmArgs& p, const RowState<KR>& st, int my_row, int split) {
  if (my_row >= p.rows) return;
  const int64_t o = (int64_t)my_row * p.splits + split;
  p.stats[o] = make_float4(st.m, st.s, st.t, st.z_tgt);
#pragma unroll
  for (int j = 0; j < KR; ++j)
    if (j < p.k) p.top[o * p.k + j] = make_uint2(__float_as_uint(st.lv[j]), (unsigned)st.li[j]);
}

// What a GEMM kernel does with a finished tile is a policy: the state of the lane's row, how a
// tile updates it, and what goes to the workspace at the end of the sweep.
// SHORT: with the classes of splits, and a last tile of half the width.
template <int KR, bool BIAS = false, bool SHORT = false>
struct TopKEpilogue {   // a5..a7: softmax statistics, k best logits, target logit (BIAS: Eq. 1's b added to every logit first)
  using State = RowState<KR>;
  static constexpr bool RELOAD_FRAGMENTS = false, OWN_U = false;
  static constexpr int ROWS = BN;
  static __device__ __forceinline__ bool skip(const GemmArgs&) { return false; }
  static __device__ __forceinline__ void init(State& st, const GemmArgs& p, int my_row, int split) {
    st.init(my_row < p.rows);
    if (SHORT && p.classes > 0) st.cls = split % p.classes;
    st.tgt = (p.target != nullptr && my_row < p.rows) ? p.target[my_row] : -1;
  }
  static __device__ __forceinline__ void settle(State& st) { asm volatile("" : "+v"(st.tgt)); }   // its loads have come back
  template <class ACC>
  static __device__ __forceinline__ void tile(const ACC& acc, State& st, int v0, const GemmArgs& p, int my_row) {
    epilogue_tile<KR, BIAS, false, ACC>(acc, st, v0, p.V, p.bias);
    // (the longest list together with a bias leaves no register for the exchange: that one kernel goes without)
    if (!(KR == 32 && BIAS)) exchange_bound(st, p, my_row);
  }
  template <bool HALF, class ACC>
  static __device__ __forceinline__ void short_tile(const ACC& acc, State& st, int v0, const GemmArgs& p, int my_row) {
    if (st.first && st.cls >= 0) first_bound<KR, BIAS, HALF>(acc, st, v0, my_row);
    st.first = false;
    epilogue_tile<KR, BIAS, HALF>(acc, st, v0, p.V, p.bias);
    exchange_classes<KR, BIAS>(st, v0, my_row);
  }
  static __device__ __forceinline__ void store(const GemmArgs& p, const State& st, int my_row, int split) {
    epilogue_store(p, st, my_row, split);
  }
};

// The top-k lists live in registers: the kernels are built for a few list lengths KR >= k.  pick(KR as a constant)
template <class F>
auto with_list_length(int k, F pick) {
  if (k <= 4) return pick(std::integral_constant<int, 4>{});
  if (k <= 12) return pick(std::integral_constant<int, 12>{});
  if (k <= 20) return pick(std::integral_constant<int, 20>{});
  return pick(std::integral_constant<int, 32>{});
}

}  // namespace
