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
// become products of small matrices, [alphas, ids] times [ids, rows], which the matrix pipe does in fp32
// (v_mfma_f32_16x16x4_f32: full precision, fp32 accumulation).  The accumulator layout of the contraction is the
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
// The shifted logits themselves are formed only where a group might hold a listed token: when its largest
// logit plus its largest shift (a table entry) beats the list's last entry for some lane.  The lists know the other
// splits' thresholds (sweep_exchange), so past a split's first tile that is rare.
//
// Groups of 16 ids (one row of 16 x 16 accumulator tiles) in a loop that is not unrolled, so that the code stays in the
// instruction cache.
//
// Measured, whole call, nine alphas: 1500 rows, d = 4096, V = 128256, arg max: 2.14 ms with nine exponentials a logit, 1.54 ms
// now (a plain projection of the rows takes 1.36 ms and u = W_U v 0.16 ms); 500 rows, d = 2560, V = 151936, lists of
// three: 2.09 ms (two passes of five and four alphas, over 64 splits), 0.65 ms now.  What is left above the projection is
// the unembedded direction, a read of W_U, and vector work beside the matrix pipe: an exponential a logit and its products.
// ---------------------------------------------------------------------------------------
constexpr int SWEEP_MAX = LL_SWEEP_MAX;
constexpr int SWEEP_KS = LL_SWEEP_KMAX;
constexpr float SWEEP_SHIFT = 20.0f;
constexpr float SWEEP_MARGIN = 2.0f * SWEEP_SHIFT * 0x1p-22f;   // more than the rounding of a shift up to SWEEP_SHIFT, and of a limit's own
constexpr int SWEEP_GROUP = 16;
constexpr unsigned SWEEP_NO_ID = 0xffffu;         // list entry that stands for "below the row's shared bound"
constexpr int SWEEP_MAX_TILES = 255;              // tiles per split: ids relative to the split's first fit 16 bits

// Table rows of a group of 16 ids, 16 floats each: rows 0 .. 15 are the first A operand, rows 16 .. 31 the second.
// Up to eight alphas: E of alpha a in row a, alpha E u in row 8 + a, and no second operand.  Nine: E in row a, alpha E u in row 16 + a.
constexpr int SWEEP_ROWS = 32;
constexpr int SWEEP_FEW = 4;          // code for all alphas is branched over past these
constexpr int SWEEP_SPLIT_ROWS = 8;   // most alphas with both factors in one operand

// What a lane reads for one group.
struct SweepTable {
  float4 a0, a1;   // its elements of the A operands: row l % 16, ids 4 (l / 16) ..
  float u;         // u of id l % 16
  float shift;     // largest alpha u of the group with a margin, of alpha number l % 16
};

template <bool GENERAL>
__device__ __forceinline__ void sweep_load_table(SweepTable& t, int g0, const GemmArgs& p) {
  const int lane = threadIdx.x & 63, l = lane & 15;
  t.u = p.u[g0 + l];
  if (GENERAL) return;
  t.shift = p.shift_max[g0 + l];
  const float4* const eu = reinterpret_cast<const float4*>(p.eu + (int64_t)(g0 / SWEEP_GROUP) * SWEEP_ROWS * SWEEP_GROUP) + (lane >> 4);
  t.a0 = eu[4 * l];
  t.a1 = eu[4 * l + SWEEP_ROWS * SWEEP_GROUP / 8];   // (unused with up to eight alphas; no branch around a load: the waits stay counted)
}

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
  // Factored form, per row block j of the wavefront (rows 16 j + l % 16): reference, and as D operands (alphas 4 (l / 16) + r) S, with
  // up to eight alphas T2 in the rows 8 + a of it, and T1, with nine alphas T.
  float ref[4];
  f32x4 s[4], t[4];
  // General form, of the lane's own row.
  float gs[SWEEP_MAX], gt[SWEEP_MAX];
  // Of the lane's own row (64 w + l):
  float lv[SWEEP_MAX][KS];                   // best shifted logits, sorted
  unsigned li[SWEEP_MAX][IDS];
  float z_tgt;
  int tgt, id0;                              // id0: first id of the split
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

// The general form: every shifted logit exponentiated against the list's head (which is at least every shifted logit seen).
template <int KS>
__device__ __forceinline__ void sweep_group_general(const float (&x)[16], SweepState<KS, true>& st, unsigned first, const SweepTable& tab,
                                                    const GemmArgs& p) {
#pragma unroll
  for (int a = 0; a < SWEEP_MAX; ++a) {
    if (a < p.n_alpha) {
      float w[16];
      const float shift = p.alphas[a] * tab.u;
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

// acc[alpha, row] += sum over lane blocks of a[alpha, id] b[id, row].  Written as an instruction: given the builtin the compiler
// wants the results in AGPRs, which the contraction fills.  So the waits are ours: two states between a vector instruction
// that writes an operand and the product that reads it, two more between products on one accumulator (there is always another
// one in between, or the s_nop here), and 18 before a vector instruction reads a result.
__device__ __forceinline__ void sweep_product(f32x4& acc, float a, float b) {
  asm volatile("s_nop 1\n\tv_mfma_f32_16x16x4_f32 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}
__device__ __forceinline__ void sweep_first_product(f32x4& acc, float a, float b) {   // acc = 0 + ...
  asm volatile("s_nop 1\n\tv_mfma_f32_16x16x4_f32 %0, %1, %2, 0" : "=&v"(acc) : "v"(a), "v"(b));
}

// The products of one group and row block, which start from zero and are added to the row's sums while the next block's
// products run: the instruction does not round to nearest, and a chain of them over a split of 51 tiles left S too small by
// 1.1e-5 of itself and the entropy by 1e-4 (6000 rows, V = 128256).  Four products of a group and one addition a group have
// the error that a sum of exponentials in vector instructions has.
struct SweepPending {
  f32x4 s[2], t[2];   // of row blocks of this parity
};
template <int KS>
__device__ __forceinline__ void sweep_fold(SweepState<KS, false>& st, SweepPending& pend, int block) {
  const int c = block & 1;
  asm volatile("" : "+v"(pend.s[c]), "+v"(pend.t[c]));   // (here, not earlier)
  st.s[block] += pend.s[c];
  st.t[block] += pend.t[c];
  asm volatile("" : "+v"(st.s[block]), "+v"(st.t[block]));
}
// The factored form (y as in sweep_group).
template <int KS>
__device__ __forceinline__ void sweep_group_factored(const float (&y)[4][4], SweepState<KS, false>& st, const SweepTable& tab,
                                                     unsigned first, const GemmArgs& p) {
  SweepPending pend;
  // references
  float most[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) most[j] = fmaxf(fmaxf(y[j][0], y[j][1]), fmaxf(y[j][2], y[j][3]));
  bool move = false;
#pragma unroll
  for (int j = 0; j < 4; ++j) move = move || most[j] > st.ref[j] + SWEEP_SHIFT;
  if (__builtin_amdgcn_ballot_w64(move) != 0) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float full = fmaxf(most[j], __shfl_xor(most[j], 16, kWave));
      full = fmaxf(full, __shfl_xor(full, 32, kWave));
      const float ref = full > st.ref[j] + SWEEP_SHIFT ? full : st.ref[j];
      const float sc = ref == st.ref[j] ? 1.0f : __builtin_amdgcn_exp2f((st.ref[j] - ref) * LOG2E);   // first group: exp2(-inf) = 0
      st.ref[j] = ref;
      st.s[j] *= sc;
      st.t[j] *= sc;
    }
  }
  const float a0[4] = {tab.a0.x, tab.a0.y, tab.a0.z, tab.a0.w}, a1[4] = {tab.a1.x, tab.a1.y, tab.a1.z, tab.a1.w};
  // Sums, row block by row block: the exponentials of the next one are made between the products of this one (a product
  // occupies the matrix pipe for 32 cycles).
  const bool second = p.n_alpha > SWEEP_SPLIT_ROWS;
  float e[2][4], ez[2][4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    e[0][r] = __builtin_amdgcn_exp2f(fmaf(y[0][r], LOG2E, -st.ref[0] * LOG2E));
    ez[0][r] = e[0][r] * y[0][r];
  }
  asm volatile("s_nop 1" : "+v"(e[0][0]), "+v"(e[0][1]), "+v"(e[0][2]), "+v"(e[0][3]), "+v"(ez[0][0]), "+v"(ez[0][1]), "+v"(ez[0][2]), "+v"(ez[0][3]));
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int c = j & 1, n = c ^ 1, jn = j < 3 ? j + 1 : 3;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      LL_SCHED_FENCE();
      if (r == 0) sweep_first_product(pend.s[c], a0[r], e[c][r]); else sweep_product(pend.s[c], a0[r], e[c][r]);
      if (j < 3) {
        e[n][r] = __builtin_amdgcn_exp2f(fmaf(y[jn][r], LOG2E, -st.ref[jn] * LOG2E));
        asm volatile("" : "+v"(e[n][r]));   // (here, not where it is used)
      }
      LL_SCHED_FENCE();
      if (r == 0) sweep_first_product(pend.t[c], a0[r], ez[c][r]); else sweep_product(pend.t[c], a0[r], ez[c][r]);
      if (j < 3) {
        ez[n][r] = e[n][r] * y[jn][r];
        asm volatile("" : "+v"(ez[n][r]));
      }
    }
    LL_SCHED_FENCE();
    if (j > 0) sweep_fold(st, pend, j - 1);   // eight products since
    LL_SCHED_FENCE();
    if (second) {
#pragma unroll
      for (int r = 0; r < 4; ++r) sweep_product(pend.t[c], a1[r], e[c][r]);
    }
    if (j < 3) asm volatile("s_nop 1" : "+v"(e[n][3]), "+v"(ez[n][3]));   // (the last of them was written just now)
  }
  LL_SCHED_FENCE();
  // Lists: the group's largest logit of the lane's own row against the least unshifted logit that any alpha might list (its
  // list's last entry less the group's largest shift; with a margin for the rounding of both, 2^-22 of either.  The shift's is in
  // the table, none where all shifts are zero: rows of equal logits, which strength 0 leaves equal, would otherwise walk every
  // group: 1500 rows, d = 4096, V = 128256, every 64th row zero: 2183 us, 1541 without the margin).
  float q0 = most[0], q1 = most[1], q2 = most[2], q3 = most[3];
  transpose_blocks(q0, q1, q2, q3);
  const float gmax = fmaxf(fmaxf(q0, q1), fmaxf(q2, q3));
  float lim = INFINITY;   // (the lists of alphas that are not there end in infinity)
  each_alpha([&](auto a_) {
    constexpr int a = decltype(a_)::value;
    if (a < SWEEP_FEW) lim = fminf(lim, minus_bcast16<a>(st.lv[a][KS - 1], tab.shift));
  });
  if (p.n_alpha > SWEEP_FEW)
    each_alpha([&](auto a_) {
      constexpr int a = decltype(a_)::value;
      if (a >= SWEEP_FEW) lim = fminf(lim, minus_bcast16<a>(st.lv[a][KS - 1], tab.shift));
    });
  lim = fmaxf(lim - fabsf(lim) * 0x1p-22f, NEG_BIG);   // (entries past the vocabulary are NEG_BIG)
  asm volatile("s_nop 15\n\ts_nop 3" : "+v"(lim), "+v"(pend.s[1]), "+v"(pend.t[1]));   // (behind the limit's dozen instructions)
  sweep_fold(st, pend, 3);
  if (__builtin_amdgcn_ballot_w64(gmax > lim) != 0) {
    float x[16];
    own_row(y, x);
    // Nor is a logit listed that KS others of the group beat whatever the shifts: those KS at least as large as `least`, less the
    // spread of the group's shifts (table entry 15), with the same margin.
    float least = gmax;
    if (KS > 1) {
#pragma unroll
      for (int i = 0; i < 4; ++i) least = fminf(least, fmaxf(fmaxf(x[4 * i], x[4 * i + 1]), fmaxf(x[4 * i + 2], x[4 * i + 3])));
    }
    least = minus_bcast16<15>(least, tab.shift);
    lim = fmaxf(lim, least - (fabsf(least) + 4.0f * SWEEP_SHIFT) * 0x1p-22f);
    sweep_collect_all<KS>(x, lim, st, tab.u, first, p);
  }
}

// One group of 16 ids: y[j][r] is id 4 (l / 16) + r of the group for row 16 j + l % 16.
template <int KS, bool GENERAL>
__device__ __forceinline__ void sweep_group(const float (&y)[4][4], SweepState<KS, GENERAL>& st, const SweepTable& tab, int g0, const GemmArgs& p) {
  const unsigned first = (unsigned)(g0 - st.id0);
  const int tl = st.tgt - g0;
  const bool has_target = __builtin_amdgcn_ballot_w64((unsigned)tl < 16u) != 0;
  if (GENERAL || has_target) {
    float x[16];
    own_row(y, x);
    if (has_target) {
#pragma unroll
      for (int o = 0; o < 16; ++o)
        if (tl == o) st.z_tgt = x[o];
    }
    if constexpr (GENERAL) sweep_group_general<KS>(x, st, first, tab, p);
  }
  if constexpr (!GENERAL) sweep_group_factored<KS>(y, st, tab, first, p);
}

// As exchange_bound of the projection, per alpha: publishes the k-th best of this split's list and picks up the row's
// best bound.  Entries below the bound cannot be in the row's top k: they give way to the largest float below it
// (below_bound: an equal logit with a smaller id still counts), which then is what a candidate has to beat.
template <int KS>
__device__ __forceinline__ void sweep_exchange(SweepState<KS, false>& st, const GemmArgs& p, int my_row) {
  asm volatile("" : "+v"(my_row));   // (the addresses made anew for every tile rather than kept)
  const int row = min(my_row, p.rows - 1);
  auto at = [&](int a) { return reinterpret_cast<unsigned*>(reinterpret_cast<unsigned char*>(p.bound) + 4u * (unsigned)(a * p.rows + row)); };
  unsigned fresh[SWEEP_MAX];
  asm volatile("" ::: "memory");
#pragma unroll
  for (int a = 0; a < SWEEP_MAX; ++a)
    fresh[a] = a < p.n_alpha ? __hip_atomic_load(at(a), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
#pragma unroll
  for (int a = 0; a < SWEEP_MAX; ++a) {
    if (a < p.n_alpha) {
      float kth = st.lv[a][KS - 1];
#pragma unroll
      for (int j = KS - 2; j >= 0; --j) kth = p.k - 1 == j ? st.lv[a][j] : kth;
      const unsigned key = float_key(kth);
      if (my_row < p.rows && key > fresh[a] && key > KEY_NEG_INF)
        __hip_atomic_fetch_max(at(a), key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const float floor = below_bound(fresh[a]);
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

// Two kernels per list length, of which the one that the table's flag does not ask for returns at once: both forms in one
// kernel do not fit the registers, and the host does not know the shifts.
template <int KS, bool GENERAL>
struct SweepEpilogue {
  using State = SweepState<KS, GENERAL>;
  static constexpr bool RELOAD_FRAGMENTS = true;
  static __device__ __forceinline__ bool skip(const GemmArgs& p) {
    if (p.sweep_general == nullptr) return false;   // (the host launches one form only)
    return (*(const int __attribute__((address_space(4)))*)(uintptr_t)p.sweep_general != 0) != GENERAL;
  }
  static __device__ __forceinline__ void init(State& st, const GemmArgs& p, int my_row) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      st.ref[j] = -INFINITY;
      st.s[j] = st.t[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int a = 0; a < SWEEP_MAX; ++a) {
      st.gs[a] = st.gt[a] = 0.f;
#pragma unroll
      for (int j = 0; j < KS; ++j) st.lv[a][j] = a < p.n_alpha ? -INFINITY : INFINITY;   // (nothing beats the lists of alphas that are not there)
#pragma unroll
      for (int j = 0; j < State::IDS; ++j) st.li[a][j] = 0xffffffffu;
    }
    st.tgt = (p.target != nullptr && my_row < p.rows) ? p.target[my_row] : -1;
    st.z_tgt = -INFINITY;
    st.id0 = -1;
  }
  static __device__ __forceinline__ void tile(f32x4 (&acc)[16][4], State& st, int v0, const GemmArgs& p, int my_row) {
    if (st.id0 < 0) st.id0 = __builtin_amdgcn_readfirstlane(v0);   // (the split's first tile)
    SweepTable ahead;
    sweep_load_table<GENERAL>(ahead, __builtin_amdgcn_readfirstlane(v0), p);
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");   // as in epilogue_tile: let the last MFMA drain
#pragma unroll 1
    for (int i = 0; i < 16; ++i) {
      // (no instructions: without it the compiler copies the accumulators' elements out of the loop, into registers it does not have)
#pragma unroll
      for (int q = 0; q < 16; ++q)
#pragma unroll
        for (int j = 0; j < 4; ++j) asm volatile("" : "+a"(acc[q][j]));
      const SweepTable tab = ahead;
      sweep_load_table<GENERAL>(ahead, __builtin_amdgcn_readfirstlane(v0 + SWEEP_GROUP * min(i + 1, 15)), p);
      LL_SCHED_FENCE();
      float y[4][4];
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
      const int g0 = __builtin_amdgcn_readfirstlane(v0 + SWEEP_GROUP * i);
      if (g0 >= p.V) break;
      if (g0 + SWEEP_GROUP > p.V) {   // only the last group of the vocabulary: a real branch (the empty asm keeps it one)
        asm volatile("");
        const int id = g0 + 4 * ((threadIdx.x & 63) >> 4);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (id + r >= p.V) y[0][r] = y[1][r] = y[2][r] = y[3][r] = NEG_BIG;
      }
      sweep_group<KS, GENERAL>(y, st, tab, g0, p);
    }
    if constexpr (!GENERAL) sweep_exchange<KS>(st, p, my_row);
  }
  static __device__ __forceinline__ void store(const GemmArgs& p, const State& st, int my_row, int split) {
    if constexpr (!GENERAL) {   // statistics in accumulator layout: rows 16 j + l % 16 of the wavefront, alphas 4 (l / 16) + r
      const int lane = threadIdx.x & 63;
      const bool second = p.n_alpha > SWEEP_SPLIT_ROWS;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = my_row - lane + 16 * j + (lane & 15);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float s = st.s[j][r], t = st.t[j][r];
          const float t2 = __shfl_xor(s, 32, kWave);   // row 8 + a
          const int a = 4 * (lane >> 4) + r;
          if (row < p.rows && a < p.n_alpha)
            p.sweep_stats[((int64_t)row * p.n_alpha + a) * p.splits + split] = make_float4(st.ref[j], s, second ? t : t + t2, 0.f);
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

}  // namespace
