// Epilogue policy of the steering sweep (Sec. 3.4, Eq. 3 read out for several alpha in one pass
// over W_U): the same GEMM kernels as the projection, with per-alpha row state.
#pragma once

#include "ll_epilogue.h"

#include <stddef.h>

#include <utility>

namespace {

// ---------------------------------------------------------------------------------------
// The logits of h' = norm(h) + alpha v are w = z + alpha u with u = W_U v, so one pass over W_U serves
// every alpha: per alpha the lane keeps softmax statistics and the KS best shifted logits.
//
// Done logit by logit and alpha by alpha this is ten vector instructions each, more than the contraction itself costs.
// The exponential is therefore taken out of the per-alpha work: with m a reference of the row,
//     e^(w - m) = e^(z - m) e^(alpha u),
// one exponential per logit and a factor E = e^(alpha u) that is the same for every row, and the sums
//     S = sum e E,   T1 = sum (e z) E,   T2 = sum e (alpha E u),        T = T1 + T2 = sum e^(w - m) w
// become products of small matrices, [alphas, ids] times [ids, rows], in fp32
// (v_mfma_f32_16x16x4_f32: full precision, fp32 accumulation; it runs on the vector ALU, but 1024 products an instruction).  The accumulator layout of the contraction is the
// operand layout of that instruction: register r of a 16 x 16 tile is, for lane l, id 4 (l / 16) + r of lens row
// l % 16, which is element (k = l / 16, n = l % 16) of the B operand, so the exponentials go in as they are, without the
// transpose that the projection's epilogue needs.  The table comes in A operand layout, loaded a group ahead.
//
// The arguments stay small: the form is used while |alpha u| <= SWEEP_SHIFT for every entry (then S >= e^-20 of its
// largest term, and no term that matters is near the smallest normal number), and the reference m, the same for the four
// lanes that hold a row, is any logit of the row from which none differs upwards by more than SWEEP_SHIFT; it moves
// rarely.  A sweep with larger shifts anywhere takes the general form, which exponentiates every shifted logit
// against the list's head, and so does one of few alphas: the products cost the same for any number up to eight.
//
// A tile goes in three passes over its accumulators, groups of 16 ids (one row of 16 x 16 accumulator tiles) each:
//   1. the largest logit of every group and of the tile (sweep_scan): which groups may hold a listed token, and whether the
//      references have to move, decided once a tile instead of beside every group's products;
//   2. the sums (sweep_sums): nothing but products and, between them, the exponentials of the next sixteen rows;
//   3. the shifted logits themselves (sweep_lists), only of the groups that pass 1 has marked.
// The lists know the other splits' logits (sweep_take_bounds), so past a split's first tile that is rare; and in a split's first
// tile, where every group would be marked, the splits tell each other their best logits between the passes (sweep_announce).
// The loops over groups are not unrolled where they are long, so that the code stays in the instruction cache.
//
// Bound by the vector ALU, on which the fp32 products run too: 32 of 32 cycles a group (48 with nine alphas none of which is zero)
// and some 120 other instructions.  Cycles of a tile's epilogue, with all of it in one pass | now: arg max, 1500 rows, d = 4096,
// V = 128256, nine alphas: first tile 89 900 | 74 600, the others 62 000 | 50 100 falling to 44 000 (sums 33 800, scan 3500; the
// contraction 145 000); lists of three, 500 rows, d = 2560, V = 151936: 184 700 | 96 400, then 103 000 falling to 78 900 | 69 700
// falling to 55 600 (contraction 100 000).  Whole calls: 1505 | 1444 us and 647 | 557 us.
//
// Where u comes from.  A pass of its own over W_U (ll_unembed_direction_kernel, and a kernel that makes the tables from u) costs what reading
// W_U costs, a tenth to a fifth of the calls above: 176 and 115 us.  The contraction reads the same W_U, and its blocks mostly have rows to
// spare: with OWN_U three rows of every block are v in three bf16 parts (ll_sweep_panel_kernel), and behind a tile's K loop
// the last wavefront's accumulators hold the tile's u.  The four wavefronts then make the tables in LDS, in the part of the ring that is free
// between two tiles.  Which form runs is not known before u is: a sample of W_U's rows says so where it is clear; where it is not
// (or where v is so long that the sums' rounding would show) the direction kernel does look at all of W_U, and u is taken from there.  A
// token that the sample has missed and whose shift is past SWEEP_SHIFT is left out, and added by the merge (SweepLeaveOut); should they be too many, or one
// be infinite, `exceeded` has the general form, launched behind the factored one, run over all.  Costs 2.6 us a tile (general form 0.4).
// Whole calls, u before | within: 1386 | 1233 us and 549 | 439 us.
// ---------------------------------------------------------------------------------------
constexpr int SWEEP_MAX = LL_SWEEP_MAX;
constexpr int SWEEP_KS = LL_SWEEP_KMAX;
constexpr float SWEEP_SHIFT = 20.0f;
constexpr float SWEEP_SHIFT_SURE = 0.7f * SWEEP_SHIFT;   // while a sample's largest shift is no more, the largest of all is taken to be below SWEEP_SHIFT
constexpr int SWEEP_SAMPLED = 256, SWEEP_BLOCK_MAX = NUM_CU * 4;   // parts of the sample, and of the largest |u|
constexpr float SWEEP_LONG = 0.1f;                         // longest alpha v, of the shortest row's length, whose u the contraction forms (see sweep_is_long)
constexpr float SWEEP_MARGIN = 2.0f * SWEEP_SHIFT * 0x1p-22f;   // more than the rounding of a shift up to SWEEP_SHIFT, and of a limit's own
constexpr int SWEEP_GROUP = 16;
constexpr unsigned SWEEP_NO_ID = 0xffffu;         // list entry that stands for "below the row's shared bound"
constexpr int SWEEP_MAX_TILES = 255;              // tiles per split: ids relative to the split's first fit 16 bits

// Table rows of a group of 16 ids, 16 floats each.  Up to eight alphas: E of alpha a in row a, alpha E u in row 8 + a.  Nine alphas
// one of which is zero: the same of the other eight; with E = 1 and alpha E u = 0 the zero one's sums are plain sums of e and e z.
// Nine others: alpha E u in row a, and E in row a of a second table behind the first.
constexpr int SWEEP_ROWS = 16;
constexpr int SWEEP_FEW = 4;          // code for all alphas is branched over past these
constexpr int SWEEP_SPLIT_ROWS = 8;   // most alphas with both factors in one operand
constexpr int SWEEP_PARTS = 3, SWEEP_OWN_ROWS = BN - SWEEP_PARTS;   // bf16 rows that are v, and the lens rows of a block that has them

// u of id g0 + l % 16 (the general form reads no more of the tables).
__device__ __forceinline__ float sweep_load_u(int g0, const GemmArgs& p) { return p.u[g0 + (threadIdx.x & 15)]; }

// Entry I of the lane's block of 16, as a DPP operand of the instruction that uses it.
template <int I>
__device__ __forceinline__ float bcast16(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x150 + I, 0xF, 0xF, true));
}
// x - (entry I of y) in one instruction (the compiler leaves the broadcast a move of its own).  y must not have been written by
// either of the two instructions before: the table is loaded a group ahead.
template <int I>
__device__ __forceinline__ float minus_bcast16(float x, float y) {
  float r;
  asm("v_subrev_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "=v"(r) : "v"(y), "v"(x), "n"(I));
  return r;
}
// f(o as a constant) for o = 0 .. 15
template <class F, int... O>
__device__ __forceinline__ void each16(F f, std::integer_sequence<int, O...>) {
  (f(std::integral_constant<int, O>{}), ...);
}
template <class F>
__device__ __forceinline__ void each16(F f) {
  each16(f, std::make_integer_sequence<int, 16>{});
}
template <class F>
__device__ __forceinline__ void each_alpha(F f) {
  each16(f, std::make_integer_sequence<int, SWEEP_MAX>{});
}

template <int KS, bool GENERAL>
struct SweepState {
  // Listed ids, relative to the split's first: 16 bits each, packed in pairs (entry j in half j % 2 of word j / 2) where the
  // registers are short.
  static constexpr int PER = GENERAL ? 1 : 2, IDS = (KS + PER - 1) / PER;
  __device__ __forceinline__ unsigned id(int a, int j) const { return (li[a][j / PER] >> (16 * (j % PER))) & 0xffffu; }
  // Factored form, per row block j of the wavefront (rows 16 j + l % 16): reference, and as D operands (rows 4 (l / 16) + r) S of alpha
  // a in row a and T in row 8 + a; of nine alphas that have a second table T in row a, and S in `more`.  Of nine of which one is
  // zero, more[j][0] and more[j][1] are the lane's share (ids 4 (l / 16) + r) of its S and T, the plain sums.
  float ref[4];
  f32x4 st[4], more[4];
  float next_shift;                          // of the tile that comes next (OWN_U: of this one), largest alpha u of alpha number l % 16
  // General form, of the lane's own row.
  float gs[SWEEP_MAX], gt[SWEEP_MAX];
  // Of the lane's own row (64 w + l):
  float lv[SWEEP_MAX][KS];                   // best shifted logits, sorted
  unsigned li[SWEEP_MAX][IDS];
  float z_tgt;
  int tgt, id0, split;                       // id0: first id of the split
  int given;                                 // OWN_U, general form: GemmArgs' given
};

// Register j of lane block g <-> register g of lane block j (see load_group).
__device__ __forceinline__ void transpose_blocks(float& r0, float& r1, float& r2, float& r3) {
  auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(r0), __float_as_uint(r2), false, false);
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(r1), __float_as_uint(r3), false, false);
  auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
  auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
  r0 = __uint_as_float(c[0]);
  r1 = __uint_as_float(c[1]);
  r2 = __uint_as_float(d[0]);
  r3 = __uint_as_float(d[1]);
}

// The group's logits of the lane's own row, from y[j][r] in accumulator layout.
__device__ __forceinline__ void own_row(const float (&y)[4][4], float (&x)[16]) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float q0 = y[0][r], q1 = y[1][r], q2 = y[2][r], q3 = y[3][r];
    transpose_blocks(q0, q1, q2, q3);
    x[r] = q0;
    x[4 + r] = q1;
    x[8 + r] = q2;
    x[12 + r] = q3;
  }
}

__device__ __forceinline__ float max16(const float (&x)[16]) {
  float m = x[0];
#pragma unroll
  for (int o = 1; o < 16; ++o) m = fmaxf(m, x[o]);
  return m;
}

// Sorted insert (descending logit; ids arrive in increasing order, so a strict comparison keeps the smaller id first
// among equal logits); a candidate that does not beat the last entry changes nothing.
template <int KS, bool GENERAL>
__device__ __forceinline__ void sweep_insert(SweepState<KS, GENERAL>& st, int a, float z, unsigned id) {
  using State = SweepState<KS, GENERAL>;
  float (&lv)[KS] = st.lv[a];
  unsigned ids[KS];
  bool above[KS];
#pragma unroll
  for (int j = 0; j < KS; ++j) {
    ids[j] = State::PER == 1 || KS == 1 ? st.li[a][j / State::PER] : st.id(a, j);
    above[j] = z > lv[j];
  }
#pragma unroll
  for (int j = KS - 1; j >= 0; --j) {   // from the bottom: each slot reads its still unchanged upper neighbour
    const int up = j > 0 ? j - 1 : 0;
    ids[j] = j > 0 && above[up] ? ids[up] : (above[j] ? id : ids[j]);
    lv[j] = j > 0 && above[up] ? lv[up] : (above[j] ? z : lv[j]);
  }
#pragma unroll
  for (int q = 0; q < State::IDS; ++q)
    st.li[a][q] = State::PER == 1 || KS == 1 ? ids[q] : ids[2 * q] | (ids[2 * q + 1 < KS ? 2 * q + 1 : 0] << 16);
}

// A select that stays one: the optimiser would otherwise fold a tree of them into an indexed access of an array in memory.
__device__ __forceinline__ float keep_select(bool c, float if_set, float if_clear) {
  float r = c ? if_set : if_clear;
  asm volatile("" : "+v"(r));
  return r;
}

// x[o] for a per-lane o in 0 .. 15.
__device__ __forceinline__ float pick16(const float (&x)[16], int o) {
  float half[8], quarter[4];
#pragma unroll
  for (int i = 0; i < 8; ++i) half[i] = keep_select((o & 1) != 0, x[2 * i + 1], x[2 * i]);
#pragma unroll
  for (int i = 0; i < 4; ++i) quarter[i] = keep_select((o & 2) != 0, half[2 * i + 1], half[2 * i]);
  const float lo = keep_select((o & 4) != 0, quarter[1], quarter[0]), hi = keep_select((o & 4) != 0, quarter[3], quarter[2]);
  return keep_select((o & 8) != 0, hi, lo);
}

// Bit o: x[o] > lim (see candidate_mask).
__device__ __forceinline__ unsigned above_mask16(const float (&x)[16], float lim) {
  unsigned mask = 0;
#pragma unroll
  for (int o = 12; o >= 0; o -= 4) {
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
        : "v"(x[o + 3]), "v"(x[o + 2]), "v"(x[o + 1]), "v"(x[o]), "v"(lim));
  }
  return mask;
}

// Lists the entries of w (ids first, first + 1, ..., the largest of them most) that beat the list's last one, in id order.
template <int KS>
__device__ __forceinline__ void sweep_collect(const float (&w)[16], float most, SweepState<KS, true>& st, int a, unsigned first) {
  if constexpr (KS == 1) {   // most beats the list: the lowest position that has it
    unsigned pos = 0;
#pragma unroll
    for (int o = 15; o >= 0; --o) pos = w[o] == most ? (unsigned)o : pos;
    st.lv[a][0] = most;
    st.li[a][0] = first + pos;
    return;
  }
  unsigned mask = above_mask16(w, st.lv[a][KS - 1]);
  while (mask != 0) {
    const int o = __builtin_ctz(mask);
    mask &= mask - 1;
    sweep_insert<KS, true>(st, a, pick16(w, o), first + (unsigned)o);
  }
}

// The kernel argument's alphas, to be read where they are used (held in scalar registers throughout they push others out).
__device__ __forceinline__ const_f32_ptr sweep_alphas() {
  auto args = (const unsigned char __attribute__((address_space(4)))*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(args));
  return (const_f32_ptr)(args + offsetof(GemmArgs, alphas));
}

// The general form: every shifted logit exponentiated against the list's head (which is at least every shifted logit seen).
template <int KS>
__device__ __forceinline__ void sweep_group_general(const float (&x)[16], SweepState<KS, true>& st, unsigned first, float u,
                                                    const GemmArgs& p) {
#pragma unroll
  for (int a = 0; a < SWEEP_MAX; ++a) {
    if (a < p.n_alpha) {
      float w[16];
      const float shift = p.alphas[a] * u;
      each16([&](auto o) { w[o] = x[o] + bcast16<o>(shift); });
      const float most = max16(w);
      if (most > st.lv[a][KS - 1]) {
        const float head = st.lv[a][0];
        sweep_collect<KS>(w, most, st, a, first);
        const float sc = __builtin_amdgcn_exp2f((head - st.lv[a][0]) * LOG2E);   // first group: exp2(-inf) = 0
        st.gs[a] *= sc;
        st.gt[a] *= sc;
      }
      const float mb = st.lv[a][0] * LOG2E;
      float s = 0.f, t = 0.f;
#pragma unroll
      for (int o = 0; o < 16; ++o) {
        const float e = __builtin_amdgcn_exp2f(fmaf(w[o], LOG2E, -mb));
        s += e;
        t = fmaf(e, w[o], t);
      }
      st.gs[a] += s;
      st.gt[a] += t;
      asm volatile("" : "+v"(st.gs[a]), "+v"(st.gt[a]));   // one alpha at a time
    }
  }
}

// The least of three (see max3), NaN once one of them is.
__device__ __forceinline__ float sticky_min3(float a, float b, float c) {
  float r;
  asm("v_minimum3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// The lane's number, made anew (what hangs on it would otherwise be kept in registers through the contraction).
__device__ __forceinline__ int fresh_lane() {
  int lane = threadIdx.x;
  asm volatile("" : "+v"(lane));
  return lane & 63;
}

// An argument, likewise (for comparisons with it).
__device__ __forceinline__ int fresh_scalar(int x) {
  asm volatile("" : "+s"(x));
  return x;
}

// (no instructions: without it the compiler copies the accumulators' elements out of a loop, into registers it does not have)
__device__ __forceinline__ void keep_in_accumulators(f32x4 (&acc)[16][4]) {
#pragma unroll
  for (int q = 0; q < 16; ++q)
#pragma unroll
    for (int j = 0; j < 4; ++j) asm volatile("" : "+a"(acc[q][j]));
}

// Group i of the tile: y[j][r] is id 4 (l / 16) + r of the group for row 16 j + l % 16.
__device__ __forceinline__ void sweep_read_group(f32x4 (&acc)[16][4], int i, float (&y)[4][4]) {
  keep_in_accumulators(acc);
  switch (i) {
#define LL_CASE(I)                                                                                        \
  case I:                                                                                                 \
    _Pragma("unroll") for (int j = 0; j < 4; ++j)                                                         \
        _Pragma("unroll") for (int r = 0; r < 4; ++r) y[j][r] = acc_read(acc[I][j][r]);                   \
    break;
    LL_CASE(0) LL_CASE(1) LL_CASE(2) LL_CASE(3) LL_CASE(4) LL_CASE(5) LL_CASE(6) LL_CASE(7)
    LL_CASE(8) LL_CASE(9) LL_CASE(10) LL_CASE(11) LL_CASE(12) LL_CASE(13) LL_CASE(14)
    default:
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) y[j][r] = acc_read(acc[15][j][r]);
#undef LL_CASE
  }
}

// Pass 1.  Bit g of the result: some lane holds, of group g, a logit above lim[j] in row 16 j + l % 16.  top: the tile's largest
// logits of those rows among the lane's ids.
__device__ __forceinline__ unsigned sweep_scan(f32x4 (&acc)[16][4], const float (&lim)[4], float (&top)[4]) {
  unsigned marked = 0;
  keep_in_accumulators(acc);
#pragma unroll
  for (int j = 0; j < 4; ++j) top[j] = -INFINITY;
  each16([&](auto g_) {
    constexpr int g = decltype(g_)::value;
    float most[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float y0 = acc_read(acc[g][j][0]), y1 = acc_read(acc[g][j][1]), y2 = acc_read(acc[g][j][2]), y3 = acc_read(acc[g][j][3]);
      most[j] = max3(max3(y0, y1, y2), y3, y3);
      top[j] = max3(top[j], most[j], most[j]);
    }
    const bool any = (most[0] > lim[0]) | (most[1] > lim[1]) | (most[2] > lim[2]) | (most[3] > lim[3]);
    if (__builtin_amdgcn_ballot_w64(any) != 0) marked |= 1u << g;
    LL_SCHED_FENCE();
  });
  return marked;
}

// References: each the same for the four lanes that hold a row.
template <int KS>
__device__ __forceinline__ void sweep_move_references(SweepState<KS, false>& st, const float (&top)[4]) {
  bool move = false;
#pragma unroll
  for (int j = 0; j < 4; ++j) move = move || top[j] > st.ref[j] + SWEEP_SHIFT;
  if (__builtin_amdgcn_ballot_w64(move) == 0) return;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const auto larger = [](uint32_t a, uint32_t b) { return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b))); };
    const float full = __uint_as_float(with_lane_xor<32>(with_lane_xor<16>(__float_as_uint(top[j]), larger), larger));
    const float ref = full > st.ref[j] + SWEEP_SHIFT ? full : st.ref[j];
    const float sc = ref == st.ref[j] ? 1.0f : __builtin_amdgcn_exp2f((st.ref[j] - ref) * LOG2E);   // first tile: exp2(-inf) = 0
    st.ref[j] = ref;
    st.st[j] *= sc;
    st.more[j] *= sc;
  }
}

// acc[alpha, row] += sum over lane blocks of a[alpha, id] b[id, row].  Written as an instruction: given the builtin the compiler
// wants the results in AGPRs, which the contraction fills.  So the waits are ours: two states between a vector instruction
// that writes an operand and the product that reads it, and 18 before a vector instruction reads a result.
__device__ __forceinline__ void sweep_product(f32x4& acc, float a, float b) {
  asm volatile("v_mfma_f32_16x16x4_f32 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}
__device__ __forceinline__ void sweep_first_product(f32x4& acc, float a, float b) {   // acc = 0 + ...
  asm volatile("v_mfma_f32_16x16x4_f32 %0, %1, %2, 0" : "=&v"(acc) : "v"(a), "v"(b));
}

// The products of one group and row block start from zero and are added to the row's sums behind the next block's products:
// the instruction does not round to nearest, and a chain of them over a split of 51 tiles left S too small by
// 1.1e-5 of itself and the entropy by 1e-4 (6000 rows, V = 128256).  A group's products and one addition a group have
// the error that a sum of exponentials in vector instructions has.
__device__ __forceinline__ void sweep_fold(f32x4& sum, f32x4& pending) {
  asm volatile("" : "+v"(pending));   // (here, not earlier)
  sum += pending;
  asm volatile("" : "+v"(sum));
}

// What a kernel that forms u itself keeps in LDS during a tile's epilogue: the upper half of each wavefront's 8 KB of the W slot whose
// stage is done (halves SWEEP_CHUNK apart, from SWEEP_HALF on).  First the three parts of the tile's u, in halves 0, 1 and 2; then the tables
// of four groups in each half.
constexpr int SWEEP_CHUNK = 64 * 128, SWEEP_HALF = 4096, SWEEP_TABLE = SWEEP_ROWS * SWEEP_GROUP * 4;
static_assert(4 * SWEEP_TABLE <= SWEEP_HALF && BM * 4 <= SWEEP_HALF, "a half");

// alphas[at] (0 past the last).
__device__ __forceinline__ float sweep_lane_alpha(int at) {
  const_f32_ptr alphas = sweep_alphas();
  float alpha = 0.f;
#pragma unroll
  for (int a = 0; a < SWEEP_MAX; ++a) alpha = at == a ? alphas[a] : alpha;
  return alpha;
}

// Pass 2.  Row block by row block: its eight products, then the exponentials that the next block's need, this block's plain sums
// and the last block's additions.  fp32 products run on the vector ALU: eight of them take 258 cycles alone, 485 with four
// vector instructions behind each, 449 with eight behind each pair, and 32 such instructions 200 (one wavefront, a bare loop).  So
// nothing is to be had from interleaving them, and what counts is their number: with S in the upper eight rows of the result and
// T in the lower ones, from the operand [E; alpha E u] times e and [0; E] times e z, a group takes 32.
template <int KS, bool OWN_U>
__device__ __forceinline__ void sweep_sums(f32x4 (&acc)[16][4], SweepState<KS, false>& st, int v0, const GemmArgs& p, const unsigned char* lds) {
  const int lane = fresh_lane();
  const bool nine = fresh_scalar(p.n_alpha) > SWEEP_SPLIT_ROWS, second = !OWN_U && nine && p.zero_alpha < 0, plain = nine && !second;
  const unsigned at = 4 * (lane & 15) + (lane >> 4);   // (row l % 16 of a group's table, ids 4 (l / 16) ..)
  const float4* tab = reinterpret_cast<const float4*>(p.eu + (int64_t)v0 * SWEEP_ROWS);
  const float4* const tab_end = tab + 15 * (SWEEP_GROUP * SWEEP_ROWS / 4);
  const int64_t to_second = second ? (int64_t)p.tiles * BM * SWEEP_ROWS / 4 : 0;
  float nref[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) nref[j] = -st.ref[j] * LOG2E;
  // OWN_U: the table is in LDS, four groups in each wavefront's half
  auto own = [&](int i) { return *reinterpret_cast<const float4*>(lds + SWEEP_HALF + SWEEP_CHUNK * (i >> 2) + SWEEP_TABLE * (i & 3) + 16 * at); };
  float4 next1, next2;
  if (OWN_U) {
    next1 = next2 = own(0);
  } else {
    next1 = tab[at];
    next2 = tab[at + to_second];
  }
  float y[4][4], e[2][4], ez[2][4];
  f32x4 pend[2], pend_more[2];
  pend[1] = pend_more[1] = f32x4{0.f, 0.f, 0.f, 0.f};
  sweep_read_group(acc, 0, y);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    e[0][r] = __builtin_amdgcn_exp2f(fmaf(y[0][r], LOG2E, nref[0]));
    ez[0][r] = e[0][r] * y[0][r];
  }
  // (The code's place: 500 to 4000 rows, lists and arg max, took up to 1.3 % longer where changes before it had moved it; of four places in
  // 32 bytes this is the best in the mean.)
  asm volatile(".p2align 5" ::: "memory");
#pragma unroll 1
  for (int i = 0; i < 16; ++i) {
    float a1[4] = {next1.x, next1.y, next1.z, next1.w}, a2[4] = {next2.x, next2.y, next2.z, next2.w};
    if (OWN_U) {
      next1 = next2 = own(min(i + 1, 15));
    } else {
      if (tab != tab_end) tab += SWEEP_GROUP * SWEEP_ROWS / 4;
      next1 = tab[at];
      next2 = tab[at + to_second];
    }
    if (!second) {   // [0; E] from [E; alpha E u]
#pragma unroll
      for (int r = 0; r < 4; ++r) a2[r] = __uint_as_float(dpp<0x118>(__float_as_uint(a1[r])));   // row_shr:8, zeros moved in
    }
    asm volatile("s_nop 1" : "+v"(a1[0]), "+v"(a1[1]), "+v"(a1[2]), "+v"(a1[3]), "+v"(a2[0]), "+v"(a2[1]), "+v"(a2[2]), "+v"(a2[3]));
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = j & 1, n = c ^ 1, jn = (j + 1) & 3, before = (j + 3) & 3;
      LL_SCHED_FENCE();
      sweep_first_product(pend[c], a1[0], e[c][0]);
      sweep_product(pend[c], a1[1], e[c][1]);
      sweep_product(pend[c], a1[2], e[c][2]);
      sweep_product(pend[c], a1[3], e[c][3]);
      sweep_product(pend[c], a2[0], ez[c][0]);
      sweep_product(pend[c], a2[1], ez[c][1]);
      sweep_product(pend[c], a2[2], ez[c][2]);
      sweep_product(pend[c], a2[3], ez[c][3]);
      if (second) {
        sweep_first_product(pend_more[c], a2[0], e[c][0]);
        sweep_product(pend_more[c], a2[1], e[c][1]);
        sweep_product(pend_more[c], a2[2], e[c][2]);
        sweep_product(pend_more[c], a2[3], e[c][3]);
        sweep_fold(st.more[before], pend_more[n]);
      }
      if (j == 3) sweep_read_group(acc, min(i + 1, 15), y);   // (the block that comes next is the next group's first)
      LL_SCHED_FENCE();
#pragma unroll
      for (int r = 0; r < 4; ++r) e[n][r] = __builtin_amdgcn_exp2f(fmaf(y[jn][r], LOG2E, nref[jn]));
#pragma unroll
      for (int r = 0; r < 4; ++r) ez[n][r] = e[n][r] * y[jn][r];
      if (plain) {
        st.more[j][0] += (e[c][0] + e[c][1]) + (e[c][2] + e[c][3]);
        st.more[j][1] += (ez[c][0] + ez[c][1]) + (ez[c][2] + ez[c][3]);
      }
      asm volatile("" : "+v"(e[n][0]), "+v"(e[n][1]), "+v"(e[n][2]), "+v"(e[n][3]), "+v"(ez[n][0]), "+v"(ez[n][1]), "+v"(ez[n][2]), "+v"(ez[n][3]));
      LL_SCHED_FENCE();
      sweep_fold(st.st[before], pend[n]);   // eight products since its last one
    }
  }
  asm volatile("s_nop 15\n\ts_nop 3" : "+v"(pend[1]), "+v"(pend_more[1]));
  sweep_fold(st.st[3], pend[1]);
  if (second) sweep_fold(st.more[3], pend_more[1]);
}

// Over the lane's block of 16.
__device__ __forceinline__ float largest_of_16(float x) {
  const auto larger = [](uint32_t a, uint32_t b) { return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b))); };
  return __uint_as_float(with_lane_xor<1>(with_lane_xor<2>(with_lane_xor<4>(with_lane_xor<8>(__float_as_uint(x), larger), larger), larger), larger));
}

// A tile's 256 entries in four registers, entry 64 q + l in lane l: the register that holds group i's, and of these the lane's l % 16 th.
__device__ __forceinline__ float sweep_group_register(const float (&x)[4], int i) {
  const float lo = keep_select((i & 4) != 0, x[1], x[0]), hi = keep_select((i & 4) != 0, x[3], x[2]);
  return keep_select((i & 8) != 0, hi, lo);
}
__device__ __forceinline__ float sweep_group_entry(const float (&x)[4], int i) {
  const int lane = 16 * (i & 3) + (fresh_lane() & 15);
  return __int_as_float(__builtin_amdgcn_ds_bpermute(4 * lane, __float_as_int(sweep_group_register(x, i))));
}

// The kernel's arguments that the factored form uses, likewise.
__device__ __forceinline__ GemmArgs sweep_args() {
  auto args = (const GemmArgs __attribute__((address_space(4)))*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(args));
  GemmArgs p = {};
  p.u = args->u;
  p.eu = args->eu;
  p.shift_max = args->shift_max;
  p.shift_min = args->shift_min;
  p.shift_tile = args->shift_tile;
  p.bound = args->bound;
  p.rows = args->rows;
  p.V = args->V;
  p.k = args->k;
  p.tiles = args->tiles;
  p.u_out = args->u_out;
  p.given = args->given;
  p.exceeded = args->exceeded;
  p.left_any = args->left_any;
  p.left_z = args->left_z;
  p.left_id = args->left_id;
  p.left_n = args->left_n;
  p.left_slots = args->left_slots;
  p.splits = args->splits;
  p.alpha_most = args->alpha_most;
  p.W = args->W;
  p.direction = args->direction;
  p.d = args->d;
  p.n_alpha = args->n_alpha;
  p.zero_alpha = args->zero_alpha;
  return p;
}

// Lists, for every alpha, those of the group's logits above lim that beat its list's last entry, in id order.  All alphas
// share one walk over the logits (their shifts are small: mostly the same ids), and all lanes stay on (a lane without a
// candidate left takes part with one that ranks nowhere).
template <int KS>
__device__ __forceinline__ void sweep_collect_all(const float (&x)[16], float lim, SweepState<KS, false>& st, float u, unsigned first,
                                                  const GemmArgs& p) {
  const_f32_ptr alphas = sweep_alphas();
  unsigned mask = above_mask16(x, lim);
  while (__builtin_amdgcn_ballot_w64(mask != 0) != 0) {
    const int o = mask != 0 ? __builtin_ctz(mask) : 0;
    const float z = mask != 0 ? pick16(x, o) : -INFINITY;
    const float uo = __int_as_float(__builtin_amdgcn_ds_bpermute(4 * o, __float_as_int(u)));   // (lanes 0 .. 15 hold the group's u)
    const unsigned id = first + (unsigned)o;
    mask &= mask - 1;
#pragma unroll
    for (int a = 0; a < SWEEP_MAX; ++a) {
      if (a == SWEEP_FEW && p.n_alpha <= SWEEP_FEW) break;
      sweep_insert<KS, false>(st, a, fmaf(alphas[a], uo, z), id);
      LL_SCHED_FENCE();
    }
  }
}

// Pass 3, the marked groups.  The group's largest logit of the lane's own row against the least unshifted logit that any alpha might
// list (its list's last entry less the group's largest shift; with a margin for the rounding of both, 2^-22 of either.  The
// shift's is in the table, none where all shifts are zero: rows of equal logits, which strength 0 leaves equal, would otherwise
// walk every group: 1500 rows, d = 4096, V = 128256, every 64th row zero: 2183 us, 1541 without the margin).
template <int KS>
__device__ __forceinline__ void sweep_lists(f32x4 (&acc)[16][4], SweepState<KS, false>& st, unsigned marked, const float (&u4)[4],
                                            const float (&shift4)[4], int v0, const GemmArgs& p) {
#pragma unroll 1
  while (marked != 0) {
    const int i = __builtin_ctz(marked);
    marked &= marked - 1;
    const int g0 = v0 + SWEEP_GROUP * i;
    float y[4][4], x[16];
    sweep_read_group(acc, i, y);
    float u = sweep_group_entry(u4, i), shift = sweep_group_entry(shift4, i);
    own_row(y, x);
    const int tl = st.tgt - g0;
    if (__builtin_amdgcn_ballot_w64((unsigned)tl < 16u) != 0) {
#pragma unroll
      for (int o = 0; o < 16; ++o)
        st.z_tgt = keep_select(tl == o, x[o], st.z_tgt);
    }
    const float gmax = max16(x);
    asm volatile("s_nop 1" : "+v"(shift), "+v"(u));   // (read by DPP instructions of ours from here on)
    float lim = INFINITY;   // (the lists of alphas that are not there end in infinity)
    each_alpha([&](auto a_) {
      constexpr int a = decltype(a_)::value;
      lim = fminf(lim, minus_bcast16<a>(st.lv[a][KS - 1], shift));
    });
    lim = fmaxf(lim - fabsf(lim) * 0x1p-22f, NEG_BIG);   // (entries past the vocabulary are NEG_BIG)
    if (__builtin_amdgcn_ballot_w64(gmax > lim) == 0) continue;
    // Nor is a logit listed that KS others of the group beat whatever the shifts: those KS at least as large as `least`, less the
    // spread of the group's shifts (table entry 15), with the same margin.
    float least = gmax;
    if (KS > 1) {
#pragma unroll
      for (int q = 0; q < 4; ++q) least = fminf(least, fmaxf(fmaxf(x[4 * q], x[4 * q + 1]), fmaxf(x[4 * q + 2], x[4 * q + 3])));
    }
    least = minus_bcast16<15>(least, shift);
    lim = fmaxf(lim, least - (fabsf(least) + 4.0f * SWEEP_SHIFT) * 0x1p-22f);
    sweep_collect_all<KS>(x, lim, st, u, (unsigned)(g0 - st.id0), p);
  }
}

// What the splits of a row tell each other, per alpha.  The splits are dealt into k classes, and a class's entry is the best
// shifted logit that any of its splits has seen: k different ids, each at least the least of the k entries, which therefore is a
// bound on the row's k-th best (for k = 1 the best so far).  It ranks some k (1 + 1/2 + ... + 1/k) th of all ids seen; the best
// k-th entry of any one split's list, of few ids each, ranks k + 1 to ten times lower: 500 rows, lists of three in 119 splits.
// Entries that are not above the bound cannot be in the row's top k: they give way to the largest float below it
// (below_bound: an equal logit with a smaller id still counts), which then is what a candidate has to beat.
template <int KS>
__device__ __forceinline__ unsigned* sweep_bound(const SweepState<KS, false>& st, const GemmArgs& p, int row, int cls, int a) {
  return reinterpret_cast<unsigned*>(reinterpret_cast<unsigned char*>(p.bound) + 4u * (unsigned)((cls * p.n_alpha + a) * p.rows + row));
}
// Takes the bounds over into the lists; PUBLISH: and sends the lists' heads where they are news.  (The loads first: a wait for one of them is also a
// wait for the atomics sent before it.)
template <int KS, bool PUBLISH>
__device__ __forceinline__ void sweep_take_bounds(SweepState<KS, false>& st, const GemmArgs& p, int my_row) {
  asm volatile("" : "+v"(my_row)::"memory");   // (the addresses made anew for every tile rather than kept)
  const int row = min(my_row, p.rows - 1), n_alpha = fresh_scalar(p.n_alpha), k = KS == 1 ? 1 : fresh_scalar(p.k), own = st.split % k;
  unsigned least[SWEEP_MAX], known[SWEEP_MAX], fresh[KS][SWEEP_MAX];
#pragma unroll
  for (int cls = 0; cls < KS; ++cls)   // (all loads in flight together, and no branch among them: past the last class or alpha the last one's again)
#pragma unroll
    for (int a = 0; a < SWEEP_MAX; ++a)
      fresh[cls][a] = __hip_atomic_load(sweep_bound(st, p, row, min(cls, k - 1), min(a, n_alpha - 1)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
  for (int a = 0; a < SWEEP_MAX; ++a) {
    least[a] = known[a] = fresh[0][a];
#pragma unroll
    for (int cls = 1; cls < KS; ++cls) {
      least[a] = min(least[a], fresh[cls][a]);
      known[a] = cls == own ? fresh[cls][a] : known[a];
    }
  }
#pragma unroll
  for (int a = 0; a < SWEEP_MAX; ++a) {
    if (a < n_alpha) {
      if (PUBLISH) {   // the list's head (the one of a list that holds none is below the bound)
        const unsigned key = float_key(st.lv[a][0]);
        if (my_row < p.rows && key > known[a] && key > KEY_NEG_INF)
          __hip_atomic_fetch_max(sweep_bound(st, p, my_row, own, a), key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      const float floor = below_bound(least[a]);
#pragma unroll
      for (int j = 0; j < KS; ++j) {
        const bool below = st.lv[a][j] <= floor;
        st.lv[a][j] = below ? floor : st.lv[a][j];
        st.li[a][j / 2] = below ? st.li[a][j / 2] | (SWEEP_NO_ID << (16 * (j % 2))) : st.li[a][j / 2];
      }
    }
  }
  asm volatile("" ::: "memory");
}
// In a split's first tile, ahead of its lists: the best shifted logits, from below (a group's largest logit with its least shift, and
// its least logit with its largest shift, which is the better one where a row's logits are nearly equal).  The second holds only while
// every logit of the group is a number: the id with the largest shift might be the one that has none.
template <int KS>
__device__ __forceinline__ void sweep_announce(f32x4 (&acc)[16][4], SweepState<KS, false>& st, const float (&least4)[4], const float (&most4)[4],
                                               const GemmArgs& p, int my_row) {
  float best[SWEEP_MAX];
#pragma unroll
  for (int a = 0; a < SWEEP_MAX; ++a) best[a] = -INFINITY;
#pragma unroll 1
  for (int i = 0; i < 16; ++i) {
    float y[4][4], q[4], l[4];
    sweep_read_group(acc, i, y);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      q[j] = max3(max3(y[j][0], y[j][1], y[j][2]), y[j][3], y[j][3]);
      l[j] = sticky_min3(sticky_min3(y[j][0], y[j][1], y[j][2]), y[j][3], y[j][3]);
    }
    transpose_blocks(q[0], q[1], q[2], q[3]);
    transpose_blocks(l[0], l[1], l[2], l[3]);
    const float gmax = max3(max3(q[0], q[1], q[2]), q[3], q[3]), gmin = sticky_min3(sticky_min3(l[0], l[1], l[2]), l[3], l[3]);
    const float least = sweep_group_entry(least4, i), most = sweep_group_entry(most4, i);
    each_alpha([&](auto a_) {
      constexpr int a = decltype(a_)::value;
      best[a] = max3(best[a], gmax + bcast16<a>(least), gmin + bcast16<a>(most));
    });
  }
#pragma unroll
  for (int a = 0; a < SWEEP_MAX; ++a) {   // (less what rounding, and the margin of the largest shifts, may have added)
    best[a] -= (fabsf(best[a]) + 4.0f * SWEEP_SHIFT) * 0x1p-22f;
    if (!(best[a] > NEG_BIG * 0.5f)) best[a] = -INFINITY;
  }
  const int n_alpha = fresh_scalar(p.n_alpha), cls = st.split % fresh_scalar(p.k);
#pragma unroll
  for (int a = 0; a < SWEEP_MAX; ++a)
    if (a < n_alpha && my_row < p.rows && best[a] > -INFINITY)
      __hip_atomic_fetch_max(sweep_bound(st, p, my_row, cls, a), float_key(best[a]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("" ::: "memory");
}

// What the contraction's sums leave of u is exact enough beside the logits' own sums, but not for a token whose unembedding row lies along the
// direction: its products have one sign, its u is many times the others', and every partial sum on the way rounds in that size (a token
// shifted by 13, d = 4096, |alpha v| a sixteenth of the rows' length: its log-probability was off by 2.0e-6 rms where u from the direction kernel
// leaves 1.1e-6, the entropy by 2.4e-6 | 1.2e-6).  So u of a token that has SWEEP_ODD times the mean |u| of its tile (six standard deviations of
// Gaussian ones; of a tile at most 34) is summed as the direction kernel sums it, to the same bits: one wavefront a token, 1.5 us.
constexpr float SWEEP_ODD = 7.5f;
__device__ __forceinline__ void sweep_exact_u(float (&u4)[4], int v0, const GemmArgs& p, unsigned char* lds) {
  const int lane = fresh_lane(), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const float there = (float)min(BM, p.V - v0), limit = SWEEP_ODD * wave_sum((fabsf(u4[0]) + fabsf(u4[1])) + (fabsf(u4[2]) + fabsf(u4[3])));
  const auto odd = [&](int q) { return there * fabsf(u4[q]) > limit; };   // (of an infinity, and in its tile, and of what is no number: never)
  const float most = max3(max3(fabsf(u4[0]), fabsf(u4[1]), fabsf(u4[2])), fabsf(u4[3]), 0.f);
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(there * most > limit) == 0, 1)) return;   // (the same in all four wavefronts)
  __syncthreads();   // the parts are read
  const float4* const v4 = reinterpret_cast<const float4*>(p.direction);
  int n = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    unsigned long long left = __builtin_amdgcn_ballot_w64(odd(q));
#pragma unroll 1
    for (; left != 0; left &= left - 1) {
      if ((n++ & 3) != wave) continue;
      const int id = 64 * q + __builtin_ctzll(left);
      const uint4* const row = reinterpret_cast<const uint4*>(p.W + (int64_t)(v0 + id) * p.d);
      float a = 0.f;
#pragma unroll 1
      for (int c = lane; c < p.d >> 3; c += 64) {
        const uint4 x = row[c];
        const float4 v0 = v4[2 * c], v1 = v4[2 * c + 1];
        a = fmaf(bf16_lo(x.x), v0.x, a);
        a = fmaf(bf16_hi(x.x), v0.y, a);
        a = fmaf(bf16_lo(x.y), v0.z, a);
        a = fmaf(bf16_hi(x.y), v0.w, a);
        a = fmaf(bf16_lo(x.z), v1.x, a);
        a = fmaf(bf16_hi(x.z), v1.y, a);
        a = fmaf(bf16_lo(x.w), v1.z, a);
        a = fmaf(bf16_hi(x.w), v1.w, a);
      }
      a = wave_sum(a);
      if (lane == 0) *reinterpret_cast<float*>(lds + SWEEP_HALF + 4 * id) = a;
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (odd(q)) {
      u4[q] = *reinterpret_cast<const float*>(lds + SWEEP_HALF + 4 * (64 * q + lane));
      asm volatile("" : "+v"(u4[q]));   // (or the compiler makes this load and the caller's from memory one that can do both)
    }
}

// u of the tile, entry 64 q + l in lane l, from the three rows of the direction in the last wavefront's accumulators.  v is the
// sum of three bf16 rows to the last bit (but for what is below the smallest normal number), so u = W v1 + W v2 + W v3 has the exact products that fp32 ones of W and v round.  An infinity of W
// against a zero of v2 or v3 would be no number: where the first part is not finite it is u.  given: u is there already.
__device__ __forceinline__ void sweep_own_u(f32x4 (&acc)[16][4], int v0, const GemmArgs& p, int my_row, bool given, unsigned char* lds, float (&u4)[4]) {
  const int lane = fresh_lane(), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if (__builtin_expect(given, 0)) {
#pragma unroll
    for (int q = 0; q < 4; ++q) u4[q] = p.u[v0 + 64 * q + lane];
    return;
  }
  const unsigned char* const in = lds + SWEEP_HALF;
  if (wave == 3) {
    const int part = (lane & 15) - (16 - SWEEP_PARTS);
    if (part >= 0) {
      unsigned char* const out = lds + SWEEP_HALF + SWEEP_CHUNK * part + 16 * (lane >> 4);
      each16([&](auto g_) {
        constexpr int g = decltype(g_)::value;
        *reinterpret_cast<float4*>(out + 4 * SWEEP_GROUP * g) =
            make_float4(acc_read(acc[g][3][0]), acc_read(acc[g][3][1]), acc_read(acc[g][3][2]), acc_read(acc[g][3][3]));
      });
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int id = 64 * q + lane;
    const float a = *reinterpret_cast<const float*>(in + 4 * id), b = *reinterpret_cast<const float*>(in + SWEEP_CHUNK + 4 * id),
                c = *reinterpret_cast<const float*>(in + 2 * SWEEP_CHUNK + 4 * id);
    const float whole = fabsf(a) < INFINITY ? a + (b + c) : a;
    u4[q] = v0 + id < p.V ? whole : 0.f;
  }
  sweep_exact_u(u4, v0, p, lds);
  if (__builtin_amdgcn_readfirstlane(my_row) == 64 * wave)   // the first row block's wavefronts: for the merge
    p.u_out[v0 + 64 * wave + lane] = sweep_group_register(u4, 4 * wave);
}

// The factored form leaves out tokens whose shift is too large for it, up to GemmArgs' left_slots a split: their logits (and u, for the others'
// limits and the tables) give way to what stands for none, and go to memory, from where the merge adds them to the row's sums and lists.  The sample
// mostly misses them where they are few: the token whose unembedding row the direction lies along, or some long rows.  Whole calls with such tokens, the
// general form over all of the call behind the factored one | left out | u and the largest shift from a pass of their own, us: 1500 rows, d = 4096, V = 128256: one
// 1790 to 2810 by its place | 1285 | 1770, sixty 1775 | 1283 | 1740, two hundred 1750 | 1331 | 1746; lists of three, 500 x 2560 x 151936: one 910 to 1145 | 462 | 830;
// 250 x 2048 x 50257: one 200 | 104 | 151.
template <int KS>
struct SweepLeaveOut {
  unsigned long long out[4];   // bit l of word q: entry 64 q + l is left out, or past the vocabulary
  int n, to;                   // left out, and how many of the split were before
  // u4 of what is left out becomes zero.  Too many, or one that is no number or infinite: `exceeded`, what the kernel makes of it is for nothing.
  __device__ __forceinline__ void look(float (&u4)[4], const SweepState<KS, false>& st, int v0, const GemmArgs& p, int my_row) {
    const int lane = fresh_lane();
    bool endless = false;
    n = to = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float shift = p.alpha_most * fabsf(u4[q]);
      const bool large = !(shift <= SWEEP_SHIFT);
      endless = endless || !(shift < INFINITY);
      out[q] = __builtin_amdgcn_ballot_w64(large);
      n += __builtin_popcountll(out[q]);
      u4[q] = large ? 0.f : u4[q];
      out[q] |= __builtin_amdgcn_ballot_w64(v0 + 64 * q + lane >= p.V);
    }
    if (__builtin_expect(n == 0, 1)) return;
    const GemmArgs more = sweep_args();   // (read here)
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), row0 = __builtin_amdgcn_readfirstlane(my_row);
    // (the count so far is in memory, each wavefront's by itself: all of its lanes have written what they read here)
    int* const count = more.left_n + 4 * ((row0 / SWEEP_OWN_ROWS) * more.splits + st.split) + wave;
    to = __builtin_amdgcn_readfirstlane(__hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    if (threadIdx.x == 0) *more.left_any = 1;
    if (__builtin_amdgcn_ballot_w64(endless) == 0 && to + n <= more.left_slots) {   // (all wavefronts alike)
      __hip_atomic_store(count, to + n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
    if (threadIdx.x == 0) *more.exceeded = 1;
    n = 0;
  }
  template <int G>
  __device__ __forceinline__ unsigned of_group() const { return (unsigned)(out[G / 4] >> (16 * (G % 4))) & 0xffffu; }
  __device__ __forceinline__ void save(f32x4 (&acc)[16][4], const SweepState<KS, false>& st, int v0, int my_row) const {
    const GemmArgs p = sweep_args();
    const int lane = fresh_lane(), row0 = __builtin_amdgcn_readfirstlane(my_row), of_block = (int)threadIdx.x & ~63;
    int at = to;
    each16([&](auto g_) {
      constexpr int g = decltype(g_)::value;
      unsigned bits = of_group<g>();
      if (bits == 0) return;
      float y[4][4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) y[j][r] = acc_read(acc[g][j][r]);
#pragma unroll 1
      for (; bits != 0; bits &= bits - 1) {
        const int o = __builtin_ctz(bits), id = v0 + SWEEP_GROUP * g + o;
        if (id >= p.V) break;
        if (threadIdx.x == 0) p.left_id[((int64_t)(row0 / SWEEP_OWN_ROWS) * p.splits + st.split) * p.left_slots + at] = id;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int of_wave = 16 * j + (lane & 15), row = row0 + of_wave;
          const float lo = keep_select((o & 1) != 0, y[j][1], y[j][0]), hi = keep_select((o & 1) != 0, y[j][3], y[j][2]);
          const float z = keep_select((o & 2) != 0, hi, lo);
          if (lane >> 4 == o >> 2 && of_block + of_wave < SWEEP_OWN_ROWS && row < p.rows)
            p.left_z[((int64_t)row * p.splits + st.split) * p.left_slots + at] = z;
        }
        ++at;
      }
    });
  }
};

// The tables of the wavefront's own 64 ids, for all (at most eight alphas besides a zero one).
__device__ __forceinline__ void sweep_put_tables(const float (&u4)[4], const GemmArgs& p, unsigned char* lds) {
  const int lane = fresh_lane(), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const float u = sweep_group_register(u4, 4 * wave);
  float* const at = reinterpret_cast<float*>(lds + SWEEP_HALF + SWEEP_CHUNK * wave + SWEEP_TABLE * (lane >> 4) + 4 * (lane & 15));
  const_f32_ptr alphas = sweep_alphas();
  const int n_alpha = fresh_scalar(p.n_alpha), left_out = n_alpha > SWEEP_SPLIT_ROWS ? p.zero_alpha : SWEEP_MAX;
  float alpha[SWEEP_MAX];
#pragma unroll
  for (int a = 0; a < SWEEP_MAX; ++a) alpha[a] = alphas[a];   // (all scalar loads at once)
#pragma unroll
  for (int r = 0; r < SWEEP_SPLIT_ROWS; ++r) {
    const float shift = (r >= left_out ? alpha[r + 1] : alpha[r]) * u, e = r < n_alpha ? expf(shift) : 0.f;
    at[SWEEP_GROUP * r] = e;
    at[SWEEP_GROUP * (SWEEP_SPLIT_ROWS + r)] = e * shift;
  }
}

// What GemmArgs' shift_tile holds, and its shift_max and shift_min of the tile's groups.  (Rounding keeps the order: the largest of alpha u
// is that of the largest or of the least u.)
__device__ __forceinline__ float sweep_tile_shift(const float (&u4)[4]) {
  const auto larger = [](uint32_t a, uint32_t b) { return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b))); };
  const auto of_all = [&](float x) {
    return __uint_as_float(with_lane_xor<32>(with_lane_xor<16>(__float_as_uint(largest_of_16(x)), larger), larger));
  };
  const float above = of_all(fmaxf(fmaxf(u4[0], u4[1]), fmaxf(u4[2], u4[3]))), below = -of_all(-fminf(fminf(u4[0], u4[1]), fminf(u4[2], u4[3])));
  const float alpha = sweep_lane_alpha(fresh_lane() & 15), most = fmaxf(alpha * above, alpha * below);
  return above == 0.f && below == 0.f ? 0.f : most + SWEEP_MARGIN;
}
__device__ __forceinline__ void sweep_group_shifts(const float (&u4)[4], float (&most4)[4], float (&least4)[4]) {
  const int at = fresh_lane() & 15;
  const float alpha = sweep_lane_alpha(at);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float x = alpha * largest_of_16(u4[q]), y = alpha * -largest_of_16(-u4[q]);
    const float most = fmaxf(x, y), least = fminf(x, y), spread = largest_of_16(most - least);
    most4[q] = at == 15 ? spread : most == 0.f && least == 0.f ? 0.f : most + SWEEP_MARGIN;
    least4[q] = least;
  }
}

// What a sample of the shifts says of all (for a wavefront; one load a lane, so that a kernel that is not the one returns soon).
enum { SWEEP_FITS, SWEEP_OPEN, SWEEP_TOO_LARGE };
__device__ __forceinline__ int sweep_sample_says(const float* sampled) {
  static_assert(SWEEP_SAMPLED == 256, "four a lane");
  const float4 x = reinterpret_cast<const float4*>(sampled)[threadIdx.x & 63];
  const bool large = !(x.x <= SWEEP_SHIFT && x.y <= SWEEP_SHIFT && x.z <= SWEEP_SHIFT && x.w <= SWEEP_SHIFT);
  const bool open = x.x > SWEEP_SHIFT_SURE || x.y > SWEEP_SHIFT_SURE || x.z > SWEEP_SHIFT_SURE || x.w > SWEEP_SHIFT_SURE;
  if (__builtin_amdgcn_ballot_w64(large) != 0) return SWEEP_TOO_LARGE;
  return __builtin_amdgcn_ballot_w64(open) != 0 ? SWEEP_OPEN : SWEEP_FITS;
}
// Whether the direction is long beside the shortest row (sampled[SWEEP_SAMPLED]: |alpha v|^2 of the largest alpha over SWEEP_LONG^2; row_sq: the rows'
// squares).  u as the contraction's accumulators sum it is off by 6e-7 of its root mean square, as their logits are of theirs, and the direction
// kernel's, of shorter sums, by a fifth of that.  Up to SWEEP_LONG the shifted logits are as exact as before, to what can be measured: rms errors of
// log-probabilities and entropies against 64 bits 0.994 to 1.003 times those with the direction kernel's u (d = 1024 and 4096, lengths of 0.03 to
// 0.1); at 0.19 up to 1.006, at twice the rows' length 1.8; rows of a twentieth of that length beside the same direction 1.015.
__device__ __forceinline__ bool sweep_is_long(const float* sampled, const float* row_sq, int rows) {
  const float length = sampled[SWEEP_SAMPLED];
  const int fours = (rows + 3) / 4;   // (behind the last row infinities)
  float shortest = INFINITY;          // (a row of what is no number has no say)
  for (int i = threadIdx.x & 63; i < fours; i += 512) {
    float4 x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = reinterpret_cast<const float4*>(row_sq)[min(i + 64 * j, fours - 1)];
#pragma unroll
    for (int j = 0; j < 8; ++j) shortest = fminf(fminf(fminf(shortest, x[j].x), fminf(x[j].y, x[j].z)), x[j].w);
  }
  shortest = -wave_max(-shortest);
  return !(length <= shortest);
}

// Two kernels per list length, of which the one that the table's flag does not ask for returns at once: both forms in one
// kernel do not fit the registers, and the host does not know the shifts.
template <int KS, bool GENERAL, bool OWN>
struct AnySweepEpilogue {
  using State = SweepState<KS, GENERAL>;
  static constexpr bool RELOAD_FRAGMENTS = true, OWN_U = OWN;
  static constexpr int ROWS = OWN_U ? SWEEP_OWN_ROWS : BN;
  static __device__ __forceinline__ bool skip(const GemmArgs& p) {
    if (OWN_U) {
      if (p.only_general) return false;   // (the host launches no other)
      const bool exceeded = GENERAL && *p.exceeded != 0;
      int says = sweep_sample_says(p.sampled);
      if (*(const_i32_ptr)(uintptr_t)p.given != 0) {   // the direction kernel has seen all
        bool large = false;
#pragma unroll
        for (int i = 0; i < SWEEP_BLOCK_MAX / 256; ++i) {
          const float4 x = reinterpret_cast<const float4*>(p.block_max)[64 * i + (threadIdx.x & 63)];
          large = large || !(p.alpha_most * x.x <= SWEEP_SHIFT && p.alpha_most * x.y <= SWEEP_SHIFT && p.alpha_most * x.z <= SWEEP_SHIFT &&
                             p.alpha_most * x.w <= SWEEP_SHIFT);
        }
        says = __builtin_amdgcn_ballot_w64(large) != 0 ? SWEEP_TOO_LARGE : SWEEP_FITS;
      }
      return (exceeded || says == SWEEP_TOO_LARGE) != GENERAL;
    }
    if (p.sweep_general == nullptr) return false;   // (the host launches one form only)
    return (*(const int __attribute__((address_space(4)))*)(uintptr_t)p.sweep_general != 0) != GENERAL;
  }
  static __device__ __forceinline__ void init(State& st, const GemmArgs& p, int my_row, int split) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      st.ref[j] = -INFINITY;
      st.st[j] = st.more[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int a = 0; a < SWEEP_MAX; ++a) {
      st.gs[a] = st.gt[a] = 0.f;
#pragma unroll
      // Nothing beats the lists of alphas that are not there, nor those of a lane past the last row: it holds the logits alpha u of a
      // row of zeros, which for all anyone knows grow with the id.  (The latter finite: limits are derived from them.)
      for (int j = 0; j < KS; ++j) st.lv[a][j] = a >= p.n_alpha ? INFINITY : my_row < p.rows ? -INFINITY : -NEG_BIG;
#pragma unroll
      for (int j = 0; j < State::IDS; ++j) st.li[a][j] = 0xffffffffu;
    }
    st.tgt = (p.target != nullptr && my_row < p.rows) ? p.target[my_row] : -1;
    st.z_tgt = -INFINITY;
    st.id0 = -1;
    st.split = split;
    st.next_shift = 0.f;
    if (OWN_U && GENERAL) st.given = *(const_i32_ptr)(uintptr_t)p.given;   // (ahead of its use: calls of one tile would wait for it)
  }
  static __device__ __forceinline__ void tile(f32x4 (&acc)[16][4], State& st, int v0, const GemmArgs& p, int my_row) {
    if constexpr (GENERAL)
      general_tile(acc, st, __builtin_amdgcn_readfirstlane(v0), p);
    else
      factored_tile(acc, st, __builtin_amdgcn_readfirstlane(v0), my_row);
  }
  static __device__ __forceinline__ void own_tile(f32x4 (&acc)[16][4], State& st, int v0, const GemmArgs& p, int my_row,
                                                  unsigned char* lds) {
    v0 = __builtin_amdgcn_readfirstlane(v0);
    if constexpr (GENERAL) {
      general_tile(acc, st, v0, p, my_row, lds);
    } else {
      factored_tile(acc, st, v0, my_row, lds);
    }
  }
  static __device__ __forceinline__ void factored_tile(f32x4 (&acc)[16][4], State& st, int v0, int my_row, unsigned char* lds = nullptr) {
    const int lane = fresh_lane();
    const GemmArgs p = sweep_args();
    const bool first = st.id0 < 0;
    if (first) st.id0 = v0;   // (the split's first tile)
    // of the sums' table (16 KB) one word a line, so that it is in this XCD's L2 by then
    float warm = 0.f;
    if (!OWN_U) warm = p.eu[(int64_t)v0 * SWEEP_ROWS + (64 * (threadIdx.x >> 6 & 1) + lane) * 32];
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");   // as in epilogue_tile: let the last MFMA drain
    float u4[4], shift4[4];
    SweepLeaveOut<KS> leave;
    if constexpr (OWN_U) {
      sweep_own_u(acc, v0, p, my_row, *(const_i32_ptr)(uintptr_t)p.given != 0, lds, u4);
      leave.look(u4, st, v0, p, my_row);
      leave.n = fresh_scalar(__builtin_amdgcn_readfirstlane(leave.n));   // (or the paths of it are told apart and the accumulators copied)
      leave.to = fresh_scalar(__builtin_amdgcn_readfirstlane(leave.to));
      __syncthreads();   // (the parts are read)
      sweep_put_tables(u4, p, lds);
      st.next_shift = sweep_tile_shift(u4);
    }
    // (rarely: a real branch, which the empty asm keeps it)
    if (OWN_U ? __builtin_expect((leave.out[0] | leave.out[1] | leave.out[2] | leave.out[3]) != 0, 0) : v0 + BM > p.V) {
      asm volatile("");
      if (OWN_U && leave.n != 0) leave.save(acc, st, v0, my_row);
      const int id = v0 + 4 * (lane >> 4);
      each16([&](auto g_) {
        constexpr int g = decltype(g_)::value;
        const unsigned mine = OWN_U ? leave.template of_group<g>() >> (4 * (lane >> 4)) : 0u;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            float x = acc_read(acc[g][j][r]);
            x = (OWN_U ? (mine >> r & 1) != 0 : id + 16 * g + r >= p.V) ? NEG_BIG : x;
            asm volatile("v_accvgpr_write_b32 %0, %1" : "=a"(acc[g][j][r]) : "v"(x));
          }
        LL_SCHED_FENCE();
      });
      asm volatile("s_nop 3" ::: "memory");
    }
    unsigned marked;
    if (OWN_U) __syncthreads();   // the tables of all four wavefronts
#pragma unroll 1
    for (bool again = false;; again = true) {
      // the least unshifted logit that any alpha might list, as in sweep_lists but with the tile's largest shifts
      float lim = INFINITY;
#pragma unroll
      for (int a = 0; a < SWEEP_MAX; ++a)
        lim = fminf(lim, st.lv[a][KS - 1] - __int_as_float(__builtin_amdgcn_readlane(__float_as_int(st.next_shift), a)));
      lim = fmaxf(lim - fabsf(lim) * 0x1p-22f, NEG_BIG);
      float lims[4], top[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) lims[j] = __int_as_float(__builtin_amdgcn_ds_bpermute(64 * j + 4 * (lane & 15), __float_as_int(lim)));
      marked = sweep_scan(acc, lims, top);
      if (again) break;
      sweep_move_references<KS>(st, top);
      if (first) {
        float least4[4];
        if constexpr (OWN_U) {
          sweep_group_shifts(u4, shift4, least4);
        } else {
          st.next_shift = p.shift_tile[v0 / BM * 16 + (lane & 15)];
          // (waited for here: at its use, which other tiles come to as well, the wait would be for the ring's loads too)
          asm volatile("" : "+v"(st.next_shift));
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            least4[q] = p.shift_min[v0 + 64 * q + lane];
            shift4[q] = p.shift_max[v0 + 64 * q + lane];
          }
        }
        sweep_announce<KS>(acc, st, least4, shift4, p, my_row);
      }
      asm volatile("" : "+v"(warm));
      sweep_sums<KS, OWN_U>(acc, st, v0, p, lds);
      if constexpr (OWN_U) {
        __syncthreads();   // (the tables are read: the LDS is the ring's again)
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          u4[q] = p.u[v0 + 64 * q + lane];
          shift4[q] = p.shift_max[v0 + 64 * q + lane];
        }
      }
      if (!first) break;
      sweep_take_bounds<KS, false>(st, p, my_row);   // and once more with what the others have announced meanwhile
    }
    const int tl = st.tgt - v0;
    unsigned long long targets = __builtin_amdgcn_ballot_w64((unsigned)tl < (unsigned)BM);
    while (targets != 0) {
      marked |= 1u << (__builtin_amdgcn_readlane(tl, __builtin_ctzll(targets)) >> 4);
      targets &= targets - 1;
    }
    if (OWN_U && marked != 0) {
      float least4[4];
      sweep_group_shifts(u4, shift4, least4);
    }
    sweep_lists<KS>(acc, st, marked, u4, shift4, v0, p);
    if (!OWN_U) {
      const int ahead = min(v0 / BM + 1, p.tiles - 1);
      st.next_shift = p.shift_tile[16 * ahead + (lane & 15)];
    }
    sweep_take_bounds<KS, true>(st, p, my_row);
    if (!OWN_U) asm volatile("" : "+v"(st.next_shift));   // (come back by now: as above)
  }
  static __device__ __forceinline__ void general_tile(f32x4 (&acc)[16][4], State& st, int v0, const GemmArgs& p, int my_row = 0,
                                                      unsigned char* lds = nullptr) {
    if (st.id0 < 0) st.id0 = v0;
    float u4[4], u_ahead = 0.f;
    if constexpr (OWN_U) {
      asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");
      sweep_own_u(acc, v0, p, my_row, st.given != 0, lds, u4);
      __syncthreads();   // the LDS is the ring's again
    } else {
      u_ahead = sweep_load_u(v0, p);
    }
    // As in epilogue_tile: let the last MFMA drain.  And the code's place: with what follows 20 bytes past a multiple of 32 the whole call takes
    // 1.0 % (arg max) to 1.8 % (lists) less than where the placed K loop leaves it, and as long as before that was placed; the
    // worst of eight places, four bytes apart, is 0 (the mean of five shapes each, two to six strengths, 60 to 1500 rows).
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15\n\t.p2align 5\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0" ::: "memory");
#pragma unroll 1
    for (int i = 0; i < 16; ++i) {
      float u = u_ahead;
      if constexpr (OWN_U)
        u = sweep_group_entry(u4, i);
      else
        u_ahead = sweep_load_u(__builtin_amdgcn_readfirstlane(v0 + SWEEP_GROUP * min(i + 1, 15)), p);
      LL_SCHED_FENCE();
      float y[4][4], x[16];
      sweep_read_group(acc, i, y);
      const int g0 = __builtin_amdgcn_readfirstlane(v0 + SWEEP_GROUP * i);
      if (g0 >= p.V) break;
      if (g0 + SWEEP_GROUP > p.V) {   // only the last group of the vocabulary: a real branch (the empty asm keeps it one)
        asm volatile("");
        const int id = g0 + 4 * ((threadIdx.x & 63) >> 4);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (id + r >= p.V) y[0][r] = y[1][r] = y[2][r] = y[3][r] = NEG_BIG;
      }
      own_row(y, x);
      const int tl = st.tgt - g0;
      if (__builtin_amdgcn_ballot_w64((unsigned)tl < 16u) != 0) {
#pragma unroll
        for (int o = 0; o < 16; ++o) {   // (lists: 477 us with selects that stay ones, 488 without; arg max 390 and 386)
          if constexpr (KS > 1)
            st.z_tgt = keep_select(tl == o, x[o], st.z_tgt);
          else if (tl == o)
            st.z_tgt = x[o];
        }
      }
      sweep_group_general<KS>(x, st, (unsigned)(g0 - st.id0), u, p);
    }
  }
  static __device__ __forceinline__ void store(const GemmArgs& p, const State& st, int my_row, int split) {
    if constexpr (!GENERAL) {   // statistics in accumulator layout: rows 16 j + l % 16 of the wavefront, table rows 4 (l / 16) + r
      const int lane = threadIdx.x & 63;
      const bool second = p.n_alpha > SWEEP_SPLIT_ROWS && p.zero_alpha < 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = OWN_U && (int)(threadIdx.x & ~63u) + 16 * j + (lane & 15) >= ROWS ? INT_MAX
                                                                                          : __builtin_amdgcn_readfirstlane(my_row) + 16 * j + (lane & 15);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float other = __shfl_xor(st.st[j][r], 32, kWave);   // row 8 + a
          int a = 4 * (lane >> 4) + r;
          const bool there = row < p.rows && a < (p.n_alpha > SWEEP_SPLIT_ROWS && !second ? SWEEP_SPLIT_ROWS : p.n_alpha);
          if (!second && p.n_alpha > SWEEP_SPLIT_ROWS && a >= p.zero_alpha) ++a;   // (the alphas but the one that is zero)
          if (there)
            p.sweep_stats[((int64_t)row * p.n_alpha + a) * p.splits + split] =
                make_float4(st.ref[j], second ? st.more[j][r] : st.st[j][r], second ? st.st[j][r] : other, 0.f);
        }
        if (!second && p.n_alpha > SWEEP_SPLIT_ROWS) {
          float s = st.more[j][0], t = st.more[j][1];
          s += __shfl_xor(s, 16, kWave);
          t += __shfl_xor(t, 16, kWave);
          s += __shfl_xor(s, 32, kWave);
          t += __shfl_xor(t, 32, kWave);
          if (row < p.rows && lane < 16)
            p.sweep_stats[((int64_t)row * p.n_alpha + p.zero_alpha) * p.splits + split] = make_float4(st.ref[j], s, t, 0.f);
        }
      }
    }
    if (my_row >= p.rows) return;
    p.sweep_ztgt[(int64_t)my_row * p.splits + split] = st.z_tgt;
#pragma unroll
    for (int a = 0; a < SWEEP_MAX; ++a)
      if (a < p.n_alpha) {
        const int64_t o = ((int64_t)my_row * p.n_alpha + a) * p.splits + split;
        if constexpr (GENERAL) p.sweep_stats[o] = make_float4(st.lv[a][0], st.gs[a], st.gt[a], 0.f);
#pragma unroll
        for (int j = 0; j < KS; ++j) {
          const unsigned id = st.id(a, j);
          const bool none = id == SWEEP_NO_ID;
          p.sweep_top[o * KS + j] =
              make_uint2(__float_as_uint(none ? -INFINITY : st.lv[a][j]), none ? (unsigned)INT_MAX : (unsigned)st.id0 + id);
        }
      }
  }
};
template <int KS, bool GENERAL>
struct SweepEpilogue : AnySweepEpilogue<KS, GENERAL, false> {};        // u and its tables from kernels before
template <int KS, bool GENERAL>
struct WholeSweepEpilogue : AnySweepEpilogue<KS, GENERAL, true> {};    // u formed by the contraction itself

}  // namespace
