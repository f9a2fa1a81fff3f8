// Epilogue policy of the steering sweep (Sec. 3.4, Eq. 3 read out for several alpha in one pass
// over W_U): the same GEMM kernels as the projection, with per-alpha row state.
#pragma once

#include "ll_epilogue.h"

namespace {

// ---------------------------------------------------------------------------------------
// The logits of h' = norm(h) + alpha v are w = z + alpha u with u = W_U v, so one pass over W_U serves
// every alpha: per alpha the lane keeps softmax statistics and the KS best shifted logits.
//
// What bounds it: vector instructions (the matrix pipe is idle meanwhile), so the exponential is taken
// out of the per-alpha work: with m the lane's running maximum of the UNshifted logits,
//     e^(w - m) = e^(z - m) e^(alpha u),
// one exponential per logit and a table factor E = e^(alpha u) that is the same for every row.  Then per
// alpha and logit
//     S += e E,   T1 += (e z) E,   T2 += e (E u),        T = T1 + alpha T2 = sum e^(w - m) w
// are three multiply-adds whose second factor is a scalar operand (the table rows of a group of 16 logits are
// read through the scalar cache while the group before is worked on).  fp32 throughout, e^(alpha u) as exact as the
// exponential it replaces; the arguments of both stay small: the form is used while |alpha u| <= SWEEP_SHIFT for
// every entry (then S >= e^-20, no term that matters is near the smallest normal number).  A sweep with larger shifts
// anywhere takes the general form, which exponentiates every shifted logit against the list's head.
//
// The shifted logits themselves are formed only where a group might hold a listed token: when its largest
// logit plus its largest shift (a table entry) beats the list's last entry for some lane.  The lists know the other
// splits' thresholds (sweep_exchange), so past a split's first tile that is rare.
//
// Groups of 16 logits (one 16 x 16 row of accumulator tiles) in a loop that is not unrolled: nine unrolled alphas times
// eight groups of 32 did not fit the instruction cache.
// Measured: SWEEP_MEASURED
// ---------------------------------------------------------------------------------------
constexpr int SWEEP_MAX = LL_SWEEP_MAX;
constexpr int SWEEP_KS = LL_SWEEP_KMAX;
constexpr float SWEEP_SHIFT = 20.0f;
constexpr int SWEEP_GROUP = 16;
constexpr int SWEEP_ROW = 2 * SWEEP_GROUP;        // table entries of a group and alpha: E[16], E u[16]
constexpr unsigned SWEEP_NO_ID = 0xffffu;         // list entry that stands for "below the row's shared bound"
constexpr int SWEEP_MAX_TILES = 255;              // tiles per split: ids relative to the split's first fit 16 bits

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float sgpr16;
typedef const sgpr16 __attribute__((address_space(4)))* const_sgpr16_ptr;

template <int KS>
struct SweepState {
  static constexpr int IDS = (KS + 1) / 2;   // ids in pairs: entry j in half j % 2 of word j / 2
  float m;                                   // running maximum of the unshifted logits (factored form)
  float s[SWEEP_MAX], t1[SWEEP_MAX], t2[SWEEP_MAX];
  float lv[SWEEP_MAX][KS];                   // best shifted logits, sorted
  unsigned li[SWEEP_MAX][IDS];
  float z_tgt;
  int tgt, id0;                              // id0: first id of the split
};

// The unshifted logits of group I of the finished tile: vocabulary rows 16 I .. 16 I + 15 for this lane's row (see load_group).
template <int I>
__device__ __forceinline__ void load_group16(const f32x4 (&acc)[16][4], float (&x)[16]) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    unsigned R0 = __float_as_uint(acc_read(acc[I][0][r])), R1 = __float_as_uint(acc_read(acc[I][1][r]));
    unsigned R2 = __float_as_uint(acc_read(acc[I][2][r])), R3 = __float_as_uint(acc_read(acc[I][3][r]));
    auto a = __builtin_amdgcn_permlane32_swap(R0, R2, false, false);
    auto b = __builtin_amdgcn_permlane32_swap(R1, R3, false, false);
    auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
    auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
    x[r] = __uint_as_float(c[0]);
    x[4 + r] = __uint_as_float(c[1]);
    x[8 + r] = __uint_as_float(d[0]);
    x[12 + r] = __uint_as_float(d[1]);
  }
}

__device__ __forceinline__ float max16(const float (&x)[16]) {
  float m = x[0];
#pragma unroll
  for (int o = 1; o < 16; ++o) m = fmaxf(m, x[o]);
  return m;
}

// Sorted insert (descending logit; ids arrive in increasing order, so a strict comparison keeps the smaller id first
// among equal logits) of a candidate that beats the last entry.
template <int KS>
__device__ __forceinline__ void sweep_insert(float (&lv)[KS], unsigned (&li)[(KS + 1) / 2], float z, unsigned id) {
  unsigned ids[KS];
#pragma unroll
  for (int j = 0; j < KS; ++j) ids[j] = (li[j / 2] >> (16 * (j % 2))) & 0xffffu;
#pragma unroll
  for (int j = KS - 1; j >= 1; --j) {   // from the bottom: each slot reads its still unchanged upper neighbour
    const bool above_upper = z > lv[j - 1], above_here = z > lv[j];
    ids[j] = above_upper ? ids[j - 1] : (above_here ? id : ids[j]);
    lv[j] = above_upper ? lv[j - 1] : (above_here ? z : lv[j]);
  }
  if (z > lv[0]) {
    lv[0] = z;
    ids[0] = id;
  }
#pragma unroll
  for (int q = 0; q < (KS + 1) / 2; ++q) li[q] = ids[2 * q] | ((2 * q + 1 < KS ? ids[2 * q + 1] : SWEEP_NO_ID) << 16);
}

// Lists the entries of w (ids first, first + 1, ...) that beat the list's last one, in id order.
template <int KS>
__device__ __forceinline__ void sweep_collect(const float (&w)[16], float (&lv)[KS], unsigned (&li)[(KS + 1) / 2], unsigned first) {
  unsigned mask = 0;
#pragma unroll
  for (int o = 15; o >= 0; --o) mask = (mask << 1) | (w[o] > lv[KS - 1] ? 1u : 0u);
  while (mask != 0) {
    const int o = __builtin_ctz(mask);
    mask &= mask - 1;
    float z = w[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) {
      float wi = w[i];
      asm volatile("" : "+v"(wi));   // (keeps the chain of selects from becoming an indexed array in memory)
      z = o == i ? wi : z;
    }
    if (z > lv[KS - 1]) sweep_insert<KS>(lv, li, z, first + (unsigned)o);
  }
}

// The general form: every shifted logit exponentiated against the list's head (which is at least every shifted logit seen).
template <int KS>
__device__ __forceinline__ void sweep_group_general(const float (&x)[16], SweepState<KS>& st, unsigned first, const sgpr16 u,
                                                    const GemmArgs& p) {
#pragma unroll
  for (int a = 0; a < SWEEP_MAX; ++a) {
    if (a < p.n_alpha) {
      float w[16];
      const float al = p.alphas[a];
#pragma unroll
      for (int o = 0; o < 16; ++o) w[o] = fmaf(al, u[o], x[o]);
      if (max16(w) > st.lv[a][KS - 1]) {
        const float head = st.lv[a][0];
        sweep_collect<KS>(w, st.lv[a], st.li[a], first);
        const float sc = __builtin_amdgcn_exp2f((head - st.lv[a][0]) * LOG2E);   // first group: exp2(-inf) = 0
        st.s[a] *= sc;
        st.t1[a] *= sc;
      }
      const float mb = st.lv[a][0] * LOG2E;
      float s = 0.f, t = 0.f;
#pragma unroll
      for (int o = 0; o < 16; ++o) {
        const float e = __builtin_amdgcn_exp2f(fmaf(w[o], LOG2E, -mb));
        s += e;
        t = fmaf(e, w[o], t);
      }
      st.s[a] += s;
      st.t1[a] += t;
      asm volatile("" : "+v"(st.s[a]), "+v"(st.t1[a]));   // one alpha at a time
    }
  }
}

// One group of 16 logits.
template <int KS, bool GENERAL>
__device__ __forceinline__ void sweep_group(const float (&x)[16], SweepState<KS>& st, int g0, const GemmArgs& p) {
  const unsigned first = (unsigned)(g0 - st.id0);
  const int tl = st.tgt - g0;
  if (__builtin_amdgcn_ballot_w64((unsigned)tl < 16u) != 0) {
#pragma unroll
    for (int o = 0; o < 16; ++o)
      if (tl == o) st.z_tgt = x[o];
  }
  const int64_t group = g0 / SWEEP_GROUP;
  const const_sgpr16_ptr u_row = (const_sgpr16_ptr)(uintptr_t)(p.u + g0);
  if constexpr (GENERAL) {
    sweep_group_general<KS>(x, st, first, *u_row, p);
    return;
  }
  // lists first: their shifted copy and the exponentials below need not be held at the same time
  const float gmax = max16(x);
  const const_f32_ptr shift = (const_f32_ptr)(uintptr_t)(p.shift_max + group * p.n_alpha);
#pragma unroll
  for (int a = 0; a < SWEEP_MAX; ++a) {
    if (a < p.n_alpha) {
      if (gmax + shift[a] > st.lv[a][KS - 1]) {
        const sgpr16 u = *u_row;
        float w[16];
        const float al = p.alphas[a];
#pragma unroll
        for (int o = 0; o < 16; ++o) w[o] = fmaf(al, u[o], x[o]);
        sweep_collect<KS>(w, st.lv[a], st.li[a], first);
      }
      LL_SCHED_FENCE();
    }
  }
  const float m_new = fmaxf(st.m, gmax);
  if (__builtin_amdgcn_ballot_w64(m_new > st.m) != 0) {
    const float sc = __builtin_amdgcn_exp2f((st.m - m_new) * LOG2E);   // first group: exp2(-inf) = 0
    st.m = m_new;
#pragma unroll
    for (int a = 0; a < SWEEP_MAX; ++a) {
      st.s[a] *= sc;
      st.t1[a] *= sc;
      st.t2[a] *= sc;
    }
  }
  const float mb = st.m * LOG2E;
  float e[16], ez[16];
#pragma unroll
  for (int o = 0; o < 16; ++o) {
    e[o] = __builtin_amdgcn_exp2f(fmaf(x[o], LOG2E, -mb));
    ez[o] = e[o] * x[o];
  }
  const const_sgpr16_ptr table = (const_sgpr16_ptr)(uintptr_t)(p.eu + group * p.n_alpha * SWEEP_ROW);
  sgpr16 E = table[0], EU = table[1];
#pragma unroll
  for (int a = 0; a < SWEEP_MAX; ++a) {
    if (a < p.n_alpha) {
      const sgpr16 cE = E, cEU = EU;
      if (a + 1 < SWEEP_MAX) {   // next alpha's rows on their way (past the last alpha: the next group's, never used)
        E = table[2 * a + 2];
        EU = table[2 * a + 3];
      }
      LL_SCHED_FENCE();
      float s0 = st.s[a], s1 = 0.f, t0 = st.t1[a], v0 = st.t2[a];
#pragma unroll
      for (int o = 0; o < 16; o += 2) {
        s0 = fmaf(e[o], cE[o], s0);
        t0 = fmaf(ez[o], cE[o], t0);
        v0 = fmaf(e[o], cEU[o], v0);
        s1 = fmaf(e[o + 1], cE[o + 1], s1);
        t0 = fmaf(ez[o + 1], cE[o + 1], t0);
        v0 = fmaf(e[o + 1], cEU[o + 1], v0);
      }
      st.s[a] = s0 + s1;
      st.t1[a] = t0;
      st.t2[a] = v0;
      asm volatile("" : "+v"(st.s[a]), "+v"(st.t1[a]), "+v"(st.t2[a]));   // one alpha at a time
      LL_SCHED_FENCE();
    }
  }
}

// As exchange_bound of the projection, per alpha: publishes the k-th best of this split's list and picks up the row's
// best bound.  Entries below the bound cannot be in the row's top k: they give way to the bound itself (the float just
// below it, since an equal logit with a smaller id still counts), which then is what a candidate has to beat.
template <int KS>
__device__ __forceinline__ void sweep_exchange(SweepState<KS>& st, const GemmArgs& p, int my_row) {
  const int row = min(my_row, p.rows - 1);
  unsigned fresh[SWEEP_MAX];
  asm volatile("" ::: "memory");
#pragma unroll
  for (int a = 0; a < SWEEP_MAX; ++a)
    fresh[a] = a < p.n_alpha ? __hip_atomic_load(p.bound + (unsigned)(a * p.rows + row), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
#pragma unroll
  for (int a = 0; a < SWEEP_MAX; ++a) {
    if (a < p.n_alpha) {
      float kth = st.lv[a][KS - 1];
#pragma unroll
      for (int j = KS - 2; j >= 0; --j) kth = p.k - 1 == j ? st.lv[a][j] : kth;
      const unsigned key = float_key(kth);
      if (my_row < p.rows && key > fresh[a] && key > KEY_NEG_INF)
        __hip_atomic_fetch_max(p.bound + (unsigned)(a * p.rows + row), key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const float floor = fresh[a] > KEY_NEG_INF ? key_float(fresh[a] - 1u) : -INFINITY;
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
  using State = SweepState<KS>;
  static constexpr bool RELOAD_FRAGMENTS = true;
  static __device__ __forceinline__ bool skip(const GemmArgs& p) {
    return (*(const int __attribute__((address_space(4)))*)(uintptr_t)p.sweep_general != 0) != GENERAL;
  }
  static __device__ __forceinline__ void init(State& st, const GemmArgs& p, int my_row) {
    st.m = -INFINITY;
#pragma unroll
    for (int a = 0; a < SWEEP_MAX; ++a) {
      st.s[a] = st.t1[a] = st.t2[a] = 0.f;
#pragma unroll
      for (int j = 0; j < KS; ++j) st.lv[a][j] = -INFINITY;
#pragma unroll
      for (int j = 0; j < State::IDS; ++j) st.li[a][j] = 0xffffffffu;
    }
    st.z_tgt = -INFINITY;
    st.tgt = (p.target != nullptr && my_row < p.rows) ? p.target[my_row] : -1;
    st.id0 = -1;
  }
  static __device__ __forceinline__ void tile(f32x4 (&acc)[16][4], State& st, int v0, const GemmArgs& p, int my_row) {
    if (st.id0 < 0) st.id0 = __builtin_amdgcn_readfirstlane(v0);   // (the split's first tile)
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");   // as in epilogue_tile: let the last MFMA drain
#pragma unroll 1
    for (int i = 0; i < 16; ++i) {
      // (no instructions: without it the compiler copies the accumulators' elements out of the loop, into registers it does not have)
#pragma unroll
      for (int q = 0; q < 16; ++q)
#pragma unroll
        for (int j = 0; j < 4; ++j) asm volatile("" : "+a"(acc[q][j]));
      float x[16];
      switch (i) {
#define LL_CASE(I)             \
  case I:                      \
    load_group16<I>(acc, x);   \
    break;
        LL_CASE(0) LL_CASE(1) LL_CASE(2) LL_CASE(3) LL_CASE(4) LL_CASE(5) LL_CASE(6) LL_CASE(7)
        LL_CASE(8) LL_CASE(9) LL_CASE(10) LL_CASE(11) LL_CASE(12) LL_CASE(13) LL_CASE(14)
        default: load_group16<15>(acc, x); break;
#undef LL_CASE
      }
      const int g0 = __builtin_amdgcn_readfirstlane(v0 + SWEEP_GROUP * i);
      if (g0 >= p.V) break;
      if (g0 + SWEEP_GROUP > p.V) {   // only the last group of the vocabulary: a real branch (the empty asm keeps it one)
        asm volatile("");
#pragma unroll
        for (int o = 0; o < 16; ++o)
          if (g0 + o >= p.V) x[o] = NEG_BIG;
      }
      sweep_group<KS, GENERAL>(x, st, g0, p);
    }
    if constexpr (!GENERAL) sweep_exchange<KS>(st, p, my_row);
  }
  static __device__ __forceinline__ void store(const GemmArgs& p, const State& st, int my_row, int split) {
    if (my_row >= p.rows) return;
    p.sweep_ztgt[(int64_t)my_row * p.splits + split] = st.z_tgt;
#pragma unroll
    for (int a = 0; a < SWEEP_MAX; ++a)
      if (a < p.n_alpha) {
        const int64_t o = ((int64_t)my_row * p.n_alpha + a) * p.splits + split;
        p.sweep_stats[o] = GENERAL ? make_float4(st.lv[a][0], st.s[a], st.t1[a], 0.f)
                                   : make_float4(st.m, st.s[a], fmaf(p.alphas[a], st.t2[a], st.t1[a]), 0.f);
#pragma unroll
        for (int j = 0; j < KS; ++j) {
          const unsigned id = (st.li[a][j / 2] >> (16 * (j % 2))) & 0xffffu;
          const bool none = id == SWEEP_NO_ID;
          p.sweep_top[o * KS + j] =
              make_uint2(__float_as_uint(none ? -INFINITY : st.lv[a][j]), none ? (unsigned)INT_MAX : (unsigned)st.id0 + id);
        }
      }
  }
};

}  // namespace
