// Projection of few lens rows (a decoding step's newest token, a handful of prompt positions): one
// read of W_U, streamed through registers at the rate memory gives it, and the merge of its parts.
#pragma once

#include "ll_epilogue.h"

namespace {

// ---------------------------------------------------------------------------------------
// With at most FEW_ROWS lens rows the contraction needs a fraction of the matrix pipe and the call
// is one read of W_U (2 V d bytes).  What counts is the load stream:
//   * W goes global -> registers, 8 rows x 128 B per instruction (whole cache lines), for a large W_U with the
//     non-temporal hint (every byte is used once, by one wavefront; the hint keeps the A panel in
//     L2), two K = 64 stages ahead;
//   * a wavefront owns its vocabulary rows outright (MU groups of 16), so nothing is waited for but
//     its own loads and the small A tile;
//   * the vocabulary is dealt in groups of 16 rows, so that 256 workgroups get equal shares of any V
//     (256-row tiles leave some compute units with three tiles and others with two).
// One workgroup of 8 wavefronts per compute unit; the A tile of a stage ([16 NJ rows][128 B], the
// normalised panel from L2) is shared through two LDS slots, one barrier per stage.
//
// W fragments: v_mfma_f32_16x16x32_bf16 wants lane l to hold row l%16, 16-byte chunk l/16 (+ 4 for
// the second K half).  A load instruction covers 8 rows: lane l fetches row l%8, chunk l/16 + 4
// ((l/8)%2), so lanes 0..7 of each block of 16 hold the first K half of rows 0..7 and lanes 8..15
// the second.  Two such registers (rows 0..7 and 8..15) exchange their halves by DPP rotations
// within the blocks and become the fragments of the two K halves.  K order and instruction are those
// of the direct-to-LDS kernel: the logits are the same bits.
//
// Bound by the read of W_U.  Kernel alone, W_U of 128256 x 8192 (2.1 GB), 81 rows, k = 20: 333 us =
// 6.3 TB/s, against 473 us on the 256-row tiles of the direct-to-LDS kernel; 151936 x 2560, 37 rows: 129 us
// = 6.0 TB/s against 212 us.  A loop that only loads W this way reaches 6.6 TB/s (without the
// non-temporal hint 5.9; W_U of 2.1 GB); loads of 16 rows x 64 B, which need no exchange of halves, 6.1.
// STREAM: with the hint (the caller chooses by W_U's size and by whether its rows are whole cache lines).
// ---------------------------------------------------------------------------------------
constexpr int FEW_WAVES = 8;
constexpr int FEW_THREADS = 64 * FEW_WAVES;
constexpr int FEW_ROWS = 128;        // lens rows of one workgroup
constexpr int FEW_CAP = 64;          // entries of a candidate list (>= LL_KMAX)
constexpr int FEW_MAX_SPLITS = 512;  // vocabulary parts of a call
constexpr int FEW_GROUPS = 4 * FEW_WAVES;   // partial maxima per row and part: (wavefront, lane block)
static_assert(FEW_GROUPS >= LL_KMAX, "the threshold is the k-th largest of the partial maxima");
static_assert(FEW_CAP >= LL_KMAX, "a list holds the top k");

struct FewArgs {
  const uint16_t* A;        // [rows, lda] bf16 normalised rows, zero padded from d to lda (a multiple of 64)
  const uint16_t* W;        // [V, d] bf16
  const int32_t* target;    // [rows] or nullptr
  const float* bias;        // [V] or nullptr
  float4* stats;            // [rows, splits]           (max, S, T, z_target)
  uint2* cand;              // [rows, splits, FEW_CAP]  (logit bits, id), unordered
  int* count;               // [rows, splits]           entries of the list
  int64_t lda;
  int rows, d, V, k, splits, units;   // splits: vocabulary parts; units: groups of 16 vocabulary rows
  int row_groups;           // workgroups of a part, 16 NJ rows each
};

typedef unsigned few_u32x4 __attribute__((ext_vector_type(4)));

// lanes 8..15 of every block of 16 from `from` rotated by 8, the others from `keep` (and vice versa)
__device__ __forceinline__ unsigned ror8_into_high(unsigned keep, unsigned from) {
  return (unsigned)__builtin_amdgcn_update_dpp((int)keep, (int)from, 0x128, 0xF, 0xC, false);
}
__device__ __forceinline__ unsigned ror8_into_low(unsigned keep, unsigned from) {
  return (unsigned)__builtin_amdgcn_update_dpp((int)keep, (int)from, 0x128, 0xF, 0x3, false);
}

// What stands in a lane's accumulators for an entry that is not there: past the wavefront's share or the vocabulary.  No entry
// of -inf is listed either; every other logit is, however low a bias has put it.
constexpr float FEW_ABSENT = -INFINITY;
constexpr float FEW_LOWEST = -3.402823466e38f;   // the lowest float that can be listed
constexpr float FEW_VOID = -2.0e38f;             // a maximum this low (its product with log2 e would not be finite): nothing that counts

// What the search for a row's threshold keeps (over the A tiles, which are done with).
template <int R>
struct FewSearch {
  float tau[R];              // the value on trial, then the threshold; NaN for rows that need none
  int count[R];              // entries at or above it
  int need[R];               // entries equal to the threshold that are listed, smallest ids first
  int ties[FEW_WAVES][R];    // such entries of each wavefront
};

template <int NJ, int MU, bool STREAM>
__global__ __launch_bounds__(FEW_THREADS) void ll_lens_few_kernel(FewArgs p) {
  constexpr int R = 16 * NJ;
  int part = blockIdx.x;
  if (p.row_groups > 1) {   // this workgroup's part, and its rows of it; those of one part side by side on one XCD, whose L2 they share W's lines in
    const int logical = xcd_logical_block();
    part = logical / p.row_groups;
    if (part >= p.splits) return;
    const int first = (logical - part * p.row_groups) * R;
    p.rows = min(p.rows - first, R);
    p.A += (int64_t)first * p.lda;
    p.target = p.target != nullptr ? p.target + first : nullptr;
    p.stats += (int64_t)first * p.splits;
    p.cand += (int64_t)first * p.splits * FEW_CAP;
    p.count += (int64_t)first * p.splits;
  }
  constexpr int A_CHUNKS = R * 8;                                              // 16-byte chunks of an A tile
  constexpr int A_PER = (A_CHUNKS + FEW_THREADS - 1) / FEW_THREADS;
  __shared__ __align__(16) unsigned char sA[2][R * 128];
  __shared__ __align__(16) float s_max[R][FEW_GROUPS];
  __shared__ float s_m[FEW_WAVES][R], s_s[FEW_WAVES][R], s_t[FEW_WAVES][R];
  __shared__ float s_zt[R], s_tau[R];
  __shared__ int s_cnt[R];
  __shared__ int s_over;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = lane >> 4, col = lane & 15;
  const int d = p.d, V = p.V;
  const int KT = (int)(p.lda >> 6);

  // A staging map: chunk q = tid + 512 i of the tile is row q / 8, chunk q % 8, kept at chunk ^ (row/2 % 8)
  unsigned a_off[A_PER];
  int a_dst[A_PER];
#pragma unroll
  for (int i = 0; i < A_PER; ++i) {
    const int q = min(tid + FEW_THREADS * i, A_CHUNKS - 1), r = q >> 3, c = q & 7;   // (threads past the tile repeat its last chunk)
    a_off[i] = (unsigned)((int64_t)min(r, p.rows - 1) * p.lda * 2) + c * 16;
    a_dst[i] = (r * 8 + (c ^ ((r >> 1) & 7))) * 16;
  }
  const unsigned char* const a_base = reinterpret_cast<const unsigned char*>(p.A);
  int f_off[2];
#pragma unroll
  for (int hk = 0; hk < 2; ++hk) f_off[hk] = (col * 8 + ((4 * hk + grp) ^ ((col >> 1) & 7))) * 16;

  // W map: lane fetches row lane % 8 of each half group, chunk w_chunk
  const int w_chunk = grp + 4 * ((lane >> 3) & 1);
  // last stage of a d that is not a multiple of 64: chunks past the row's end are read at chunk 0 and zeroed
  const bool ragged = (d & 63) != 0;
  const bool past_end = ragged && (KT - 1) * 64 + w_chunk * 8 >= d;

  // (one part per workgroup and no loop over parts: the compiler would keep the epilogue's addresses in registers through the
  // next part's main loop)
  const int ua = (int)((int64_t)part * p.units / p.splits);
  const int ub = (int)((int64_t)(part + 1) * p.units / p.splits);
  const int u0 = ua + (ub - ua) * wave / FEW_WAVES;                            // this wavefront's groups: u0 .. u0 + nu - 1
  const int nu = ua + (ub - ua) * (wave + 1) / FEW_WAVES - u0;                 // 0 .. MU
  const int row0 = min(u0 * 16, V - 1);
  const int row_max = min(nu > 0 ? (u0 + nu) * 16 - 1 : row0, V - 1);        // groups past nu re-read this row (one line) and are masked
  unsigned w_off[2 * MU];
#pragma unroll
  for (int h = 0; h < 2 * MU; ++h)
    w_off[h] = (unsigned)(min(row0 + 8 * h + (lane & 7), row_max) - row0) * (unsigned)(2 * d) + w_chunk * 16;
  const unsigned char* const w_base = reinterpret_cast<const unsigned char*>(p.W + (int64_t)row0 * d);

  f32x4 acc[MU][NJ];
#pragma unroll
  for (int u = 0; u < MU; ++u)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[u][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  few_u32x4 wb[2][2 * MU], ar[2][A_PER];
  auto load_a = [&](few_u32x4 (&q)[A_PER], int kt) {
#pragma unroll
    for (int i = 0; i < A_PER; ++i) q[i] = *reinterpret_cast<const few_u32x4*>(a_base + a_off[i] + (size_t)kt * 128);
  };
  auto store_a = [&](const few_u32x4 (&q)[A_PER], int slot) {
#pragma unroll
    for (int i = 0; i < A_PER; ++i) *reinterpret_cast<few_u32x4*>(sA[slot] + a_dst[i]) = q[i];
  };
  auto load_w = [&](few_u32x4 (&q)[2 * MU], int kt) {
    // Past the end all lanes fetch one line, never used: no branch around the loads, so that the compiler can count them.
    const unsigned keep = (unsigned)((kt - KT) >> 31);   // all ones while kt < KT
    const unsigned char* const base = w_base + (size_t)min(kt, KT - 1) * 128;
    const unsigned back = (past_end && kt == KT - 1) ? (unsigned)w_chunk * 16 : 0u;
#pragma unroll
    for (int h = 0; h < 2 * MU; ++h) {
      const few_u32x4* const src = reinterpret_cast<const few_u32x4*>(base + ((w_off[h] - back) & keep));
      q[h] = STREAM ? __builtin_nontemporal_load(src) : *src;
    }
  };
  // One K stage out of buffers B = kt % 2 of both operands; the loads of stage kt + 2 go out as the registers fall free.
  auto stage = [&](auto b_, int kt) {
    constexpr int B = decltype(b_)::value;
    store_a(ar[B ^ 1], B ^ 1);
    load_a(ar[B], min(kt + 2, KT - 1));
    LL_SCHED_FENCE();
    if (kt >= KT - 1) {   // (a branch without loads)
      if (past_end || kt == KT) {
#pragma unroll
        for (int h = 0; h < 2 * MU; ++h) wb[B][h] = few_u32x4{0u, 0u, 0u, 0u};
      }
    }
    // W fragments in place: first and second K half of group u
#pragma unroll
    for (int u = 0; u < MU; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const unsigned lo = wb[B][2 * u][i], hi = wb[B][2 * u + 1][i];
        wb[B][2 * u][i] = ror8_into_high(lo, hi);
        wb[B][2 * u + 1][i] = ror8_into_low(hi, lo);
      }
    bf16x8 fa[2][NJ];
#pragma unroll
    for (int hk = 0; hk < 2; ++hk)
#pragma unroll
      for (int j = 0; j < NJ; ++j) fa[hk][j] = *reinterpret_cast<const bf16x8*>(sA[B] + j * 16 * 128 + f_off[hk]);
#pragma unroll
    for (int u = 0; u < MU; ++u)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int hk = 0; hk < 2; ++hk)
          acc[u][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wb[B][2 * u + hk]), fa[hk][j], acc[u][j], 0, 0, 0);
    load_w(wb[B], kt + 2);
    LL_SCHED_FENCE();
    __syncthreads();
  };
  load_a(ar[0], 0);
  load_w(wb[0], 0);
  load_a(ar[1], min(1, KT - 1));
  load_w(wb[1], 1);
  store_a(ar[0], 0);
  if (tid < R) s_zt[tid] = -INFINITY;
  __syncthreads();
  // (an odd number of stages is filled up with one whose W is zero)
  for (int kt = 0; kt < KT; kt += 2) {
    stage(std::integral_constant<int, 0>{}, kt);
    stage(std::integral_constant<int, 1>{}, kt + 1);
  }

  // ---- epilogue: lane holds, of group u and row block j, vocabulary entries 16 (u0 + u) + 4 grp + r of lens row 16 j + col
  // (Row block by row block, fenced: otherwise the compiler interleaves them all and runs out of registers.)
  const int id0 = u0 * 16 + 4 * grp;
  const int id_end = min((u0 + nu) * 16, V);
#pragma unroll
  for (int u = 0; u < MU; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int id = id0 + 16 * u + r;
      const float b = p.bias != nullptr ? p.bias[min(id, V - 1)] : 0.f;
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[u][j][r] = id < id_end ? acc[u][j][r] + b : FEW_ABSENT;
    }
  LL_SCHED_FENCE();
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int n = 16 * j + col;
    const int tgt = (p.target != nullptr && n < p.rows) ? p.target[n] : -1;
    float mx = FEW_ABSENT;
#pragma unroll
    for (int u = 0; u < MU; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) mx = fmaxf(mx, acc[u][j][r]);
    s_max[n][wave * 4 + grp] = mx;
    if (tgt >= id0 && tgt < id_end) {
#pragma unroll
      for (int u = 0; u < MU; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (id0 + 16 * u + r == tgt) s_zt[n] = acc[u][j][r];
    }
    float m = fmaxf(mx, __shfl_xor(mx, 16, kWave));
    m = fmaxf(m, __shfl_xor(m, 32, kWave));
    const float mb = m <= FEW_VOID ? 0.f : m * LOG2E;   // (all terms are exp2(-inf))
    float s = 0.f, t = 0.f;
#pragma unroll
    for (int u = 0; u < MU; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float e = __builtin_amdgcn_exp2f(fmaf(acc[u][j][r], LOG2E, -mb));
        s += e;
        t = fmaf(e, id0 + 16 * u + r < id_end ? acc[u][j][r] : 0.f, t);
      }
    s += __shfl_xor(s, 16, kWave);
    t += __shfl_xor(t, 16, kWave);
    s += __shfl_xor(s, 32, kWave);
    t += __shfl_xor(t, 32, kWave);
    if (grp == 0) {
      s_m[wave][n] = m;
      s_s[wave][n] = s;
      s_t[wave][n] = t;
    }
    LL_SCHED_FENCE();
  }
  if (tid < R) {
    s_cnt[tid] = 0;
    s_tau[tid] = FEW_LOWEST;
  }
  if (tid == 0) s_over = 0;
  __syncthreads();
  // Threshold of a row: the k-th largest of its 32 partial maxima (the k entries that are those
  // maxima reach it, so nothing below it can be in the part's top k).  Up to k = 20 or so about 1.5 k of the part's
  // entries pass, as long as they lie anywhere and few are equal.  32 lanes a row, rank by counting.
  for (int n = tid >> 5; n < p.rows; n += FEW_THREADS / 32) {
    const int q = tid & 31;
    const float mine = s_max[n][q];
    int rank = 0;
#pragma unroll
    for (int i = 0; i < FEW_GROUPS; i += 4) {
      const float4 o = *reinterpret_cast<const float4*>(&s_max[n][i]);
      rank += (o.x > mine || (o.x == mine && i < q)) ? 1 : 0;
      rank += (o.y > mine || (o.y == mine && i + 1 < q)) ? 1 : 0;
      rank += (o.z > mine || (o.z == mine && i + 2 < q)) ? 1 : 0;
      rank += (o.w > mine || (o.w == mine && i + 3 < q)) ? 1 : 0;
    }
    // Equal logits all over (more than three quarters of the maxima are the first one): nothing is appended before the search below.
    const int first = __builtin_amdgcn_readlane(__float_as_int(mine), 0), second = __builtin_amdgcn_readlane(__float_as_int(mine), 32);
    const unsigned long long same = __builtin_amdgcn_ballot_w64(mine == __int_as_float(lane < 32 ? first : second));
    const bool flat = __builtin_popcount(lane < 32 ? (unsigned)same : (unsigned)(same >> 32)) > FEW_GROUPS / 4 * 3;
    if (rank == p.k - 1) {
      s_tau[n] = fmaxf(mine, FEW_LOWEST);
      if (flat && mine > FEW_ABSENT) s_cnt[n] = FEW_CAP + 1;
    }
  }
  // softmax statistics of the part: one thread a row
  if (tid < p.rows) {
    float m = s_m[0][tid];
#pragma unroll
    for (int w = 1; w < FEW_WAVES; ++w) m = fmaxf(m, s_m[w][tid]);
    float s = 0.f, t = 0.f;
#pragma unroll
    for (int w = 0; w < FEW_WAVES; ++w) {
      const float sc = m <= FEW_VOID ? 1.f : __builtin_amdgcn_exp2f((s_m[w][tid] - m) * LOG2E);   // (sums of 0 or NaN, whatever the scale)
      s = fmaf(sc, s_s[w][tid], s);
      t = fmaf(sc, s_t[w][tid], t);
    }
    p.stats[(int64_t)tid * p.splits + part] = make_float4(m, s, t, s_zt[tid]);
  }
  __syncthreads();
  // Append a lane's entries to the row's list, one counter update per lane and row.  passing(j): bit 4 u + r for entry (u, j, r).
  static_assert(MU * 4 <= 32, "a bit per entry");
  auto append = [&](auto passing) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int n = 16 * j + col;
      const unsigned bits = passing(j);
      const int c = __builtin_popcount(bits);
      if (c != 0 && n < p.rows) {
        const int at = atomicAdd(&s_cnt[n], c);
        if (at + c > FEW_CAP) {
          s_over = 1;
        } else {
          uint2* list = p.cand + ((int64_t)n * p.splits + part) * FEW_CAP + at;
#pragma unroll
          for (int u = 0; u < MU; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (bits & (1u << (4 * u + r))) *list++ = make_uint2(__float_as_uint(acc[u][j][r]), (unsigned)(id0 + 16 * u + r));
        }
      }
      LL_SCHED_FENCE();
    }
  };
  auto mask_of = [&](auto pass) {
    unsigned bits = 0;
#pragma unroll
    for (int u = 0; u < MU; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) bits |= pass(u, r) ? 1u << (4 * u + r) : 0u;
    return bits;
  };
  append([&](int j) {
    const float tau = s_tau[16 * j + col];
    return mask_of([&](int u, int r) { return acc[u][j][r] >= tau; });
  });
  __syncthreads();
  if (s_over != 0) {
    // Some lists do not hold all that passed: k is close to the number of partial maxima, the best entries sit together (like
    // tokens have neighbouring ids), or many are equal.  Those rows get a threshold that k to FEW_CAP entries reach, found by
    // bisection between the first one and the part's maximum; where that ends at a value which too many entries share, the
    // ones with the smallest ids make up the k.  The first trial is the next value up, so that equal logits (rows of zeros, masked
    // tokens) take one step; else a list ends after three to six, 32 at the most.
    // Whole calls, with the exact k-th best found bit by bit over all 42 bits of (value, position) | now, us: d = 256, k = 32,
    // 96 rows: V = 50257 157 | 54, V = 128256 277 | 67; k = 10, every 16th row zero: 96 rows, V = 50257 153 | 38.
    FewSearch<R>& f = *reinterpret_cast<FewSearch<R>*>(&sA[0][0]);
    static_assert(sizeof(FewSearch<R>) <= sizeof(sA), "over the A tiles");
    const bool mine = tid < R && s_cnt[min(tid, R - 1)] > FEW_CAP;   // thread n looks after row n
    unsigned lo = 0, hi = 0, trial = 0;   // keys: at least k entries reach lo, `above` < k of them hi
    int above = 0;
    if (mine) {
      float m = s_m[0][tid];
#pragma unroll
      for (int w = 1; w < FEW_WAVES; ++w) m = fmaxf(m, s_m[w][tid]);
      lo = float_key(s_tau[tid] + 0.f);
      hi = float_key(m + 0.f) + 1;
      trial = lo + 1;
      s_cnt[tid] = 0;
    }
    bool searching = mine;
    for (;;) {
      if (tid < R) {
        f.tau[tid] = searching ? key_float(trial) : __builtin_nanf("");
        f.count[tid] = 0;
      }
      __syncthreads();
      if (tid == 0) s_over = 0;   // (everyone has read it)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const float tau = f.tau[16 * j + col];
        if (__builtin_amdgcn_ballot_w64(tau == tau) != 0) {
          int c = 0;
#pragma unroll
          for (int u = 0; u < MU; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) c += acc[u][j][r] >= tau ? 1 : 0;
          if (c != 0) atomicAdd(&f.count[16 * j + col], c);
        }
        LL_SCHED_FENCE();
      }
      __syncthreads();
      if (searching) {
        const int c = f.count[tid];
        if (c >= p.k) {
          lo = trial;
        } else {
          hi = trial;
          above = c;
        }
        searching = !(c >= p.k && c <= FEW_CAP) && hi - lo > 1;
        trial = lo + (hi - lo) / 2;
        if (searching) s_over = 1;
      }
      __syncthreads();
      if (s_over == 0) break;
    }
    if (tid < R) {
      f.tau[tid] = mine ? key_float(lo) : __builtin_nanf("");
      f.need[tid] = hi - lo == 1 ? p.k - above : FEW_CAP;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const float tau = f.tau[16 * j + col];
      int c = 0;
#pragma unroll
      for (int u = 0; u < MU; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) c += acc[u][j][r] == tau ? 1 : 0;
      c += __shfl_xor(c, 16, kWave);
      c += __shfl_xor(c, 32, kWave);
      if (grp == 0) f.ties[wave][16 * j + col] = c;
      LL_SCHED_FENCE();
    }
    __syncthreads();
    append([&](int j) {
      const int n = 16 * j + col;
      const float tau = f.tau[n];
      unsigned bits = mask_of([&](int u, int r) { return acc[u][j][r] > tau; });
      int left = f.need[n];   // ties still to list, in the order of the ids: wavefront, group, lane block, entry
      for (int w = 0; w < wave; ++w) left -= f.ties[w][n];
#pragma unroll
      for (int u = 0; u < MU; ++u) {
        unsigned tie = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) tie |= acc[u][j][r] == tau ? 1u << r : 0u;
        const int c = __builtin_popcount(tie);
        const int beside = __shfl_xor(c, 16, kWave), pair = c + beside, other = __shfl_xor(pair, 32, kWave);
        int here = left - ((grp & 1) ? beside : 0) - ((grp & 2) ? other : 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if ((tie & (1u << r)) != 0 && here-- > 0) bits |= 1u << (4 * u + r);
        }
        left -= pair + other;
      }
      return bits;
    });
    __syncthreads();
  }
  if (tid < p.rows) p.count[(int64_t)tid * p.splits + part] = min(s_cnt[tid], FEW_CAP);
}

// ---------------------------------------------------------------------------------------
// Merge of the parts, one workgroup per row.  A list whose maximum is not among the k best maxima (by
// logit, then by part: ids grow with the part) holds nothing of the row's top k, and neither does an
// entry below the k-th best maximum: what is left of the k lists that matter, some tens of entries, is
// ranked by counting.  Bound by latency, so it has no chain of k dependent steps (k rounds of cross-lane
// exchanges over 256 sorted lists took 34 us for 81 rows at k = 20) and two trips to memory.
// Where many are left (few parts and a long k, many equal logits) they are bisected down to FEW_MERGE_RANKED
// first: counting takes the square of their number, 2048 entries 100 us.
// Order of entries as 64-bit keys: the logit's ordered bits, then the smaller part or id.
// ---------------------------------------------------------------------------------------
constexpr int FEW_MERGE_THREADS = 512;
constexpr int FEW_MERGE_MAX = LL_KMAX * FEW_CAP;   // entries of k lists
constexpr int FEW_MERGE_RANKED = 256;              // most entries ranked by counting (>= LL_KMAX)

__device__ __forceinline__ unsigned long long few_order(float z, unsigned id) {
  return ((unsigned long long)float_key(z + 0.f) << 32) | (unsigned)~id;
}

// Number of the first n keys above `mine` (n a multiple of 4, keys 16-byte aligned).
__device__ __forceinline__ int keys_above(const unsigned long long* keys, int n, unsigned long long mine) {
  int rank = 0;
  for (int o = 0; o < n; o += 4) {
    const ulonglong2 x = *reinterpret_cast<const ulonglong2*>(keys + o), y = *reinterpret_cast<const ulonglong2*>(keys + o + 2);
    rank += (x.x > mine ? 1 : 0) + (x.y > mine ? 1 : 0) + (y.x > mine ? 1 : 0) + (y.y > mine ? 1 : 0);
  }
  return rank;
}

__global__ __launch_bounds__(FEW_MERGE_THREADS) void ll_few_merge_kernel(
    const float4* __restrict__ stats, const uint2* __restrict__ cand, const int* __restrict__ count, int splits, int k, int V,
    int topk_softmax, const int32_t* __restrict__ target, int32_t* __restrict__ out_ids, float* __restrict__ out_p,
    float* __restrict__ out_logp, float* __restrict__ out_entropy) {
  constexpr int WAVES = FEW_MERGE_THREADS / 64;
  static_assert(FEW_MAX_SPLITS == FEW_MERGE_THREADS, "one part per thread");
  __shared__ __align__(16) unsigned long long s_part[FEW_MAX_SPLITS];
  __shared__ __align__(16) unsigned long long s_c[FEW_MERGE_MAX + 4];
  __shared__ float s_red[4][WAVES];
  __shared__ int2 s_list[LL_KMAX];   // (part, entries)
  __shared__ int s_above[FEW_MERGE_THREADS / 2];
  static_assert(LL_KMAX % WAVES == 0, "a list for each wavefront in every round");
  __shared__ float s_tau;
  __shared__ int s_n, s_count[2][WAVES];
  __shared__ float s_z[LL_KMAX];
  __shared__ int s_id[LL_KMAX];
  const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float4 q = make_float4(-INFINITY, 0.f, 0.f, -INFINITY);
  int entries = 0;
  if (tid < splits) {
    q = stats[(int64_t)row * splits + tid];
    entries = count[(int64_t)row * splits + tid];
  }
  const unsigned long long mine = tid < splits ? few_order(q.x, (unsigned)tid) : 0ull;
  s_part[tid] = mine;
  if (tid < LL_KMAX) {
    s_list[tid] = make_int2(0, 0);
    s_z[tid] = -INFINITY;
    s_id[tid] = INT_MAX;
  }
  if (tid == 0) {
    s_n = 0;
    s_tau = -INFINITY;
  }
  const float m_wave = wave_max(q.x), zt_wave = wave_max(q.w);
  if (lane == 0) {
    s_red[0][wave] = m_wave;
    s_red[1][wave] = zt_wave;
  }
  __syncthreads();
  float M = s_red[0][0], zt = s_red[1][0];
#pragma unroll
  for (int w = 1; w < WAVES; ++w) {
    M = fmaxf(M, s_red[0][w]);
    zt = fmaxf(zt, s_red[1][w]);
  }
  const float sc = tid < splits ? __builtin_amdgcn_exp2f((q.x - M) * LOG2E) : 0.f;
  const float s_wave = wave_sum(sc * q.y), t_wave = wave_sum(sc * q.z);
  if (lane == 0) {
    s_red[2][wave] = s_wave;
    s_red[3][wave] = t_wave;
  }
  // Ranks of the maxima.  Up to 256 parts: two threads a part, which count among half of them each (with that, and the loads of the
  // lists below all in flight, 37 rows, d = 2560, V = 151936, k = 10, whole call: 141.5 us, 139.6 now).
  const bool shared_count = splits > 64 && splits <= FEW_MERGE_THREADS / 2;   // (the same for all threads)
  int rank = 0;
  if (shared_count) {
    const int part = tid & (FEW_MERGE_THREADS / 2 - 1), half = (((splits + 1) / 2) + 3) & ~3;
    const bool upper = tid >= FEW_MERGE_THREADS / 2;   // (whole wavefronts)
    const unsigned long long of = s_part[part];
    rank = upper ? keys_above(s_part + half, ((splits + 3) & ~3) - half, of) : keys_above(s_part, half, of);
    if (upper) s_above[part] = rank;
  } else if (tid < splits) {
    rank = keys_above(s_part, (splits + 3) & ~3, mine);
  }
  if (shared_count) {
    __syncthreads();
    if (tid < splits) rank += s_above[tid];
  }
  if (tid < splits) {
    if (rank < k) s_list[rank] = make_int2(tid, entries);
    if (rank == k - 1) s_tau = q.x;
  }
  __syncthreads();
  const float tau = s_tau;
  constexpr int ROUNDS = (LL_KMAX + WAVES - 1) / WAVES;
  uint2 found[ROUNDS];
#pragma unroll
  for (int i = 0; i < ROUNDS; ++i) {   // (lists past the k-th have no entries: s_list)
    const int2 list = s_list[wave + WAVES * i];
    found[i] = make_uint2(0u, 0u);
    if (WAVES * i < k && lane < list.y) found[i] = cand[((int64_t)row * splits + list.x) * FEW_CAP + lane];
  }
#pragma unroll
  for (int i = 0; i < ROUNDS; ++i) {
    if (WAVES * i >= k) break;
    const uint2 e = found[i];
    const bool pass = lane < s_list[wave + WAVES * i].y && __uint_as_float(e.x) >= tau;
    const unsigned long long passing = __builtin_amdgcn_ballot_w64(pass);
    int at = 0;
    if (lane == 0 && passing != 0) at = atomicAdd(&s_n, __builtin_popcountll(passing));
    at = __builtin_amdgcn_readfirstlane(at);
    if (pass) s_c[at + __builtin_popcountll(passing & ((1ull << lane) - 1))] = few_order(__uint_as_float(e.x), e.y);
  }
  __syncthreads();
  int n = s_n;
  if (n > FEW_MERGE_RANKED) {   // (the same for all threads)
    constexpr int PER = FEW_MERGE_MAX / FEW_MERGE_THREADS;
    unsigned long long own[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) own[i] = tid + FEW_MERGE_THREADS * i < n ? s_c[tid + FEW_MERGE_THREADS * i] : 0ull;
    // keys differ: all n reach lo, none hi; each step halves the distance, and some step leaves k to FEW_MERGE_RANKED
    unsigned long long lo = few_order(tau, 0xffffffffu), hi = few_order(M, 0u) + 1;
    for (int step = 0;; ++step) {
      const unsigned long long trial = lo + (hi - lo) / 2;
      int c = 0;
#pragma unroll
      for (int i = 0; i < PER; ++i) c += __builtin_popcountll(__builtin_amdgcn_ballot_w64(own[i] >= trial));
      if (lane == 0) s_count[step & 1][wave] = c;
      __syncthreads();
      c = 0;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) c += s_count[step & 1][w];
      if (c >= k) lo = trial; else hi = trial;
      if ((c >= k && c <= FEW_MERGE_RANKED) || hi - lo <= 1) break;
    }
    if (tid == 0) s_n = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const bool pass = own[i] >= lo;
      const unsigned long long passing = __builtin_amdgcn_ballot_w64(pass);
      int at = 0;
      if (lane == 0 && passing != 0) at = atomicAdd(&s_n, __builtin_popcountll(passing));
      at = __builtin_amdgcn_readfirstlane(at);
      if (pass) s_c[at + __builtin_popcountll(passing & ((1ull << lane) - 1))] = own[i];
    }
    __syncthreads();
    n = s_n;
  }
  const int n4 = (n + 3) & ~3;
  if (tid < n4 - n) s_c[n + tid] = 0ull;
  __syncthreads();
  for (int i = tid; i < n; i += FEW_MERGE_THREADS) {
    const unsigned long long key = s_c[i];
    const int rank = keys_above(s_c, n4, key);
    if (rank < k) {
      s_z[rank] = key_float((unsigned)(key >> 32));
      s_id[rank] = (int)~(unsigned)key;
    }
  }
  __syncthreads();
  if (wave == 0) {
    float S = 0.f, T = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      S += s_red[2][w];
      T += s_red[3][w];
    }
    const float logS = logf(S);
    const float z = lane < k ? s_z[lane] : -INFINITY;
    const float z0 = s_z[0];
    const float sk = wave_sum(lane < k ? __builtin_amdgcn_exp2f((z - z0) * LOG2E) : 0.f);
    if (lane < k) {
      out_ids[(int64_t)row * k + lane] = s_id[lane];
      out_p[(int64_t)row * k + lane] = topk_softmax ? __builtin_amdgcn_exp2f((z - z0) * LOG2E) * (1.0f / sk)
                                                    : __builtin_amdgcn_exp2f(((z - M) - logS) * LOG2E);
    }
    if (lane == 0) {
      out_entropy[row] = (M - T / S) + logS;
      if (target != nullptr) {
        const int t = target[row];
        out_logp[row] = (t >= 0 && t < V) ? (zt - M) - logS : __builtin_nanf("");
      }
    }
  }
}

}  // namespace
