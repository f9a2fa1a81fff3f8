// Fused logit-lens projection for gfx950: RMS statistics / normalised panel, bf16 MFMA GEMM over
// the vocabulary with an online-softmax / top-k / target-gather epilogue, and the merge of the
// vocabulary splits.
//
// Follows the paper's Sec. 3.3 (Eq. 1 and "Top-k extraction") and Alg. 1 Phase 2; the logits of
// Eq. 1 live only in MFMA accumulators.
#include "ll_epilogue.h"
#include "ll_epilogue_sweep.h"
#include "ll_few_rows.h"
#include "ll_gemm_lds.h"
#include "ll_gemm_staged.h"

#include <atomic>
#include <climits>
#include <mutex>
#include <utility>
#include <vector>

namespace {

// ---------------------------------------------------------------------------------------
// a2: inv_rms[r] = 1 / sqrt(mean_j h[r,j]^2 + eps).  One wavefront per row, 16-byte loads.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void ll_rms_stats_kernel(const uint16_t* __restrict__ hidden, int64_t n_rows,
                                                           int d, float eps, float* __restrict__ inv_rms) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n_rows) return;
  const uint4* src = reinterpret_cast<const uint4*>(hidden + row * (int64_t)d);
  const int n16 = d >> 3;
  float acc0 = 0.f, acc1 = 0.f;
  for (int c = lane; c < n16; c += 64) {
    accum_sq(src[c], acc0, acc1);
  }
  const float ss = wave_sum(acc0 + acc1);
  if (lane == 0) inv_rms[row] = inv_rms_from_sumsq(ss, d, eps);
}

// The larger of two numbers, NaN once one of them is.
__device__ __forceinline__ float sticky_max(float a, float b) { return (a != a || a >= b) ? a : b; }

// ---------------------------------------------------------------------------------------
// a2 + a3 materialised: panel[r, :] = bf16((h[r, :] * inv_rms[r]) * gamma), zero padded to the
// panel's row stride; gamma == nullptr copies the rows unchanged.  One wavefront per row; the
// row stays in registers between the statistic and the write when it fits.
// ---------------------------------------------------------------------------------------
// SQUARES: and row_sq[row] the sum of the squares of what was written.
template <int NITER, bool SQUARES = false>
__device__ __forceinline__ void norm_panel_row(const uint16_t* __restrict__ hidden, const uint16_t* __restrict__ gamma,
                                               uint16_t* __restrict__ panel, int row, int rows, int d, int64_t lda, float eps,
                                               unsigned* __restrict__ bound, int bounds, float* __restrict__ row_sq = nullptr) {
  const int lane = threadIdx.x & 63;
  const int n16 = d >> 3;
  const int n16_pad = (int)(lda >> 3);
  uint4* dst = reinterpret_cast<uint4*>(panel + (int64_t)row * lda);
  if (row == rows) {   // one row of zeros behind them, what stands for the rows that are missing from a whole block
    for (int c = lane; c < n16_pad; c += 64) dst[c] = make_uint4(0, 0, 0, 0);
    return;
  }
  if (bound != nullptr && lane < bounds) bound[(int64_t)lane * rows + row] = 0u;   // the row's shared top-k bounds, before the pass that uses them
  const uint4* src = reinterpret_cast<const uint4*>(hidden + (int64_t)row * d);
  const uint4* g4 = reinterpret_cast<const uint4*>(gamma);
  float acc0 = 0.f, acc1 = 0.f, sq0 = 0.f, sq1 = 0.f;
  auto emit = [&](int c, const uint4 q, const uint4 g, float inv) {
    const uint32_t hw[4] = {q.x, q.y, q.z, q.w};
    const uint32_t gw[4] = {g.x, g.y, g.z, g.w};
    uint32_t ow[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      ow[i] = pack_bf16(bf16_lo(hw[i]) * inv * bf16_lo(gw[i]), bf16_hi(hw[i]) * inv * bf16_hi(gw[i]));
    const uint4 out = make_uint4(ow[0], ow[1], ow[2], ow[3]);
    dst[c] = out;
    if (SQUARES) accum_sq(out, sq0, sq1);
  };
  if (gamma == nullptr) {
    for (int c = lane; c < n16; c += 64) {
      const uint4 q = src[c];
      dst[c] = q;
      if (SQUARES) accum_sq(q, sq0, sq1);
    }
  } else if (NITER > 0) {
    // all loads of the row and of gamma before the first use, chunks past the end at the last one (their squares count as zero)
    uint4 cache[NITER > 0 ? NITER : 1], g[NITER > 0 ? NITER : 1];
#pragma unroll
    for (int it = 0; it < NITER; ++it) cache[it] = src[min(lane + 64 * it, n16 - 1)];
#pragma unroll
    for (int it = 0; it < NITER; ++it) g[it] = g4[min(lane + 64 * it, n16 - 1)];
#pragma unroll
    for (int it = 0; it < NITER; ++it)
      if (lane + 64 * it < n16) accum_sq(cache[it], acc0, acc1);
    const float inv = inv_rms_from_sumsq(wave_sum(acc0 + acc1), d, eps);
#pragma unroll
    for (int it = 0; it < NITER; ++it)
      if (lane + 64 * it < n16) emit(lane + 64 * it, cache[it], g[it], inv);
  } else {
    for (int c = lane; c < n16; c += 64) accum_sq(src[c], acc0, acc1);
    const float inv = inv_rms_from_sumsq(wave_sum(acc0 + acc1), d, eps);
    for (int c = lane; c < n16; c += 64) emit(c, src[c], g4[c], inv);
  }
  for (int c = n16 + lane; c < n16_pad; c += 64) dst[c] = make_uint4(0, 0, 0, 0);
  if (SQUARES) {
    const float sq = wave_sum(sq0 + sq1);
    if (lane == 0) row_sq[row] = sq;
  }
}

template <int NITER>
__global__ __launch_bounds__(256) void ll_norm_panel_kernel(const uint16_t* __restrict__ hidden,
                                                            const uint16_t* __restrict__ gamma, uint16_t* __restrict__ panel,
                                                            int rows, int zero_rows, int d, int64_t lda, float eps,
                                                            unsigned* __restrict__ bound, int bounds) {
  const int row = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (row >= rows + zero_rows) return;
  norm_panel_row<NITER>(hidden, gamma, panel, row, rows, d, lda, eps, bound, bounds);
}

// The same for a sweep whose kernel forms u itself.  Behind the row of zeros three rows whose sum is v: what is cut off it at 8, 16 and 24
// bits, so that nothing is lost (of an infinity or what is no number the first row has it, the others zero).  And the first
// n_waves wavefronts (SWEEP_SAMPLED, or none) look at `samples` rows of W_U, spread over the vocabulary, up to SAMPLE_ROWS each at once:
// sampled[w] is the largest |alpha u| of wavefront w's, NaN once one is.  What tells a long direction (see sweep_is_long): sampled[SWEEP_SAMPLED]
// from the direction, row_sq from the rows.
constexpr int SAMPLE_ROWS = 8;
__host__ __device__ inline int sweep_part_pieces(int64_t lda) { return (int)((lda / 8 + 63) / 64); }   // wavefronts of a part

template <int NITER>
__global__ __launch_bounds__(256) void ll_sweep_panel_kernel(const uint16_t* __restrict__ hidden, const uint16_t* __restrict__ gamma,
                                                             uint16_t* __restrict__ panel, int rows, int d, int64_t lda, float eps,
                                                             unsigned* __restrict__ bound, int bounds, const uint16_t* __restrict__ W, int V,
                                                             const float* __restrict__ v, float alpha_most, int n_waves, int samples,
                                                             float* __restrict__ sampled, float* __restrict__ row_sq,
                                                             int* __restrict__ flags, int n_flags) {
  const int lane = threadIdx.x & 63, n16 = d >> 3;
  int row = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  const float4* const v4 = reinterpret_cast<const float4*>(v);
  if (row < n_waves) {
    const uint4* w[SAMPLE_ROWS];
    float a[SAMPLE_ROWS], largest = 0.f;
#pragma unroll
    for (int i = 0; i < SAMPLE_ROWS; ++i) {   // (past the last the last one again)
      const int s = min(row + n_waves * i, samples - 1);
      w[i] = reinterpret_cast<const uint4*>(W + (int64_t)((int64_t)s * V / samples) * d);
      a[i] = 0.f;
    }
    for (int c = lane; c < n16; c += 64) {
      uint4 q[SAMPLE_ROWS];
#pragma unroll
      for (int i = 0; i < SAMPLE_ROWS; ++i) q[i] = w[i][c];
      const float4 v0 = v4[2 * c], v1 = v4[2 * c + 1];
#pragma unroll
      for (int i = 0; i < SAMPLE_ROWS; ++i) {
        a[i] = fmaf(bf16_lo(q[i].x), v0.x, a[i]);
        a[i] = fmaf(bf16_hi(q[i].x), v0.y, a[i]);
        a[i] = fmaf(bf16_lo(q[i].y), v0.z, a[i]);
        a[i] = fmaf(bf16_hi(q[i].y), v0.w, a[i]);
        a[i] = fmaf(bf16_lo(q[i].z), v1.x, a[i]);
        a[i] = fmaf(bf16_hi(q[i].z), v1.y, a[i]);
        a[i] = fmaf(bf16_lo(q[i].w), v1.z, a[i]);
        a[i] = fmaf(bf16_hi(q[i].w), v1.w, a[i]);
      }
    }
#pragma unroll
    for (int i = 0; i < SAMPLE_ROWS; ++i) largest = sticky_max(largest, fabsf(wave_sum(a[i])));
    if (lane == 0) sampled[row] = alpha_most * largest;
    return;
  }
  row -= n_waves;
  if (row <= rows) {
    if (row == rows) {
      for (int i = lane; i < n_flags; i += 64) flags[i] = 0;
      if (lane < 3) row_sq[rows + lane] = INFINITY;
    }
    norm_panel_row<NITER, true>(hidden, gamma, panel, row, rows, d, lda, eps, bound, bounds, row_sq);
    return;
  }
  row -= rows + 1;
  if (row == 0) {   // a wavefront of its own for the direction's length
    float vv = 0.f;
#pragma unroll 4
    for (int c = lane; c < 2 * n16; c += 64) {
      const float4 a = v4[c];
      vv += a.x * a.x + a.y * a.y + a.z * a.z + a.w * a.w;
    }
    vv = wave_sum(vv);
    if (lane == 0) sampled[SWEEP_SAMPLED] = alpha_most * alpha_most * vv * (1.0f / (SWEEP_LONG * SWEEP_LONG));
    return;
  }
  // and one for 64 chunks of each part
  const int pieces = sweep_part_pieces(lda), part = (row - 1) / pieces, c = (row - 1 - part * pieces) * 64 + lane;
  if (part >= SWEEP_PARTS || c >= (int)(lda >> 3)) return;
  const auto cut = [&](float x) -> uint32_t {
    const uint32_t first = __float_as_uint(x) & 0xffff0000u;
    if (!(fabsf(x) < INFINITY)) return part != 0 ? 0u : x != x ? 0x7fc0u : first >> 16;
    const float rest = x - __uint_as_float(first);
    const uint32_t second = __float_as_uint(rest) & 0xffff0000u;
    const uint32_t third = __float_as_uint(rest - __uint_as_float(second));
    return (part == 0 ? first : part == 1 ? second : third) >> 16;
  };
  uint4 q = make_uint4(0, 0, 0, 0);
  if (c < n16) {
    const float4 a = v4[2 * c], b = v4[2 * c + 1];
    q = make_uint4(cut(a.x) | cut(a.y) << 16, cut(a.z) | cut(a.w) << 16, cut(b.x) | cut(b.y) << 16, cut(b.z) | cut(b.w) << 16);
  }
  reinterpret_cast<uint4*>(panel + (int64_t)(rows + 1 + part) * lda)[c] = q;
}

// Copy of the bias of Eq. 1 padded with zeros to whole vocabulary tiles, so that the epilogue
// reads 32 entries per group without looking at V.
__global__ __launch_bounds__(256) void ll_pad_bias_kernel(const float* __restrict__ bias, int V, float* __restrict__ padded,
                                                          int n_padded) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n_padded; i += gridDim.x * blockDim.x)
    padded[i] = i < V ? bias[i] : 0.f;
}

__global__ __launch_bounds__(256) void ll_zero_u32_kernel(unsigned* __restrict__ p, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0u;
}

// ---------------------------------------------------------------------------------------
// Steering sweep, step 1: u = W_U v (one pass over W_U, HBM-bound: 2 V d bytes) and, per workgroup, the
// largest |u|.  One wavefront takes eight vocabulary rows at a time: a chunk of v read from LDS serves
// eight products, and eight 16-byte loads per lane are in flight.  STREAM: the loads carry the
// non-temporal hint, for a W_U that the Infinity Cache (256 MiB) would not keep for step 3 anyway.
// 151936 x 2560: 145 us without the hint, 118 us with it (6.6 TB/s); 128256 x 4096: 206 and 180 us (5.8 TB/s).
// ---------------------------------------------------------------------------------------
struct AlphaList {
  float a[SWEEP_MAX];
};

constexpr int UD_ROWS = 8;   // vocabulary rows a wavefront takes at a time
constexpr int UD_BLOCKS = SWEEP_BLOCK_MAX;
constexpr int64_t INFINITY_CACHE_BYTES = 256ll << 20, L2_BYTES = 32ll << 20;   // (the L2s of the eight XCDs together)

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

template <bool STREAM>
__global__ __launch_bounds__(256) void ll_unembed_direction_kernel(const uint16_t* __restrict__ W, const float* __restrict__ v,
                                                                   int V, int d, float scale, float* __restrict__ u, int n_padded,
                                                                   float* __restrict__ block_max, const float* __restrict__ sampled,
                                                                   const float* __restrict__ row_sq, int rows, bool only_general,
                                                                   int* __restrict__ given) {
  extern __shared__ __align__(16) float sv[];
  if (sampled != nullptr) {   // a look ahead of a kernel that forms u itself: only where it is asked for
    if (threadIdx.x < 64) {
      const bool wanted = sweep_is_long(sampled, row_sq, rows) || (!only_general && sweep_sample_says(sampled) == SWEEP_OPEN);
      if (threadIdx.x == 0) sv[0] = wanted ? 1.f : 0.f;   // (v may take all the LDS)
      if (blockIdx.x == 0 && threadIdx.x == 0) *given = wanted ? 1 : 0;
    }
    __syncthreads();
    if (sv[0] == 0.f) return;
    __syncthreads();
  }
  for (int j = threadIdx.x; j < d; j += blockDim.x) sv[j] = v[j];
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int n16 = d >> 3;
  if (blockIdx.x == 0 && V + (int)threadIdx.x < n_padded) u[V + threadIdx.x] = 0.f;   // (less than a tile)
  float largest = 0.f;   // (NaN once any u is)
  for (int r0 = (blockIdx.x * 4 + wave) * UD_ROWS; r0 < V; r0 += gridDim.x * 4 * UD_ROWS) {
    float acc[UD_ROWS];
    const u32x4* rows[UD_ROWS];
#pragma unroll
    for (int i = 0; i < UD_ROWS; ++i) {
      acc[i] = 0.f;
      rows[i] = reinterpret_cast<const u32x4*>(W + (int64_t)min(r0 + i, V - 1) * d);
    }
    for (int c = lane; c < n16; c += 64) {
      u32x4 q[UD_ROWS];
#pragma unroll
      for (int i = 0; i < UD_ROWS; ++i)   // all loads of the step in flight before the first use
        q[i] = STREAM ? __builtin_nontemporal_load(rows[i] + c) : rows[i][c];
      const float4 v0 = *reinterpret_cast<const float4*>(sv + 8 * c);
      const float4 v1 = *reinterpret_cast<const float4*>(sv + 8 * c + 4);
#pragma unroll
      for (int i = 0; i < UD_ROWS; ++i) {
        float a = acc[i];
        a = fmaf(bf16_lo(q[i].x), v0.x, a);
        a = fmaf(bf16_hi(q[i].x), v0.y, a);
        a = fmaf(bf16_lo(q[i].y), v0.z, a);
        a = fmaf(bf16_hi(q[i].y), v0.w, a);
        a = fmaf(bf16_lo(q[i].z), v1.x, a);
        a = fmaf(bf16_hi(q[i].z), v1.y, a);
        a = fmaf(bf16_lo(q[i].w), v1.z, a);
        a = fmaf(bf16_hi(q[i].w), v1.w, a);
        acc[i] = a;
      }
    }
#pragma unroll
    for (int i = 0; i < UD_ROWS; ++i) {
      const float x = wave_sum(acc[i]);
      if (r0 + i < V) {
        if (lane == 0) u[r0 + i] = scale * x;
        largest = sticky_max(largest, fabsf(x));
      }
    }
  }
  __syncthreads();   // v is done with: its LDS (all of it, at the largest d) takes the wavefronts' maxima
  if (lane == 0) sv[wave] = largest;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) largest = sticky_max(largest, sv[w]);
    block_max[blockIdx.x] = largest;
  }
}

// Step 2: what the sweep epilogue reads per group of 16 ids and per tile (see GemmArgs), the flag that says which form of the
// epilogue runs, and the zeroed bounds.  A block's turn is one tile.
__global__ __launch_bounds__(256) void ll_sweep_table_kernel(const float* __restrict__ block_max, int n_blocks, int n_padded,
                                                             AlphaList alphas, int n_alpha, int zero_alpha, const float* __restrict__ u,
                                                             float* __restrict__ eu, float* __restrict__ shift_max,
                                                             float* __restrict__ shift_min, float* __restrict__ shift_tile,
                                                             int* __restrict__ general, unsigned* __restrict__ bound, int n_bound) {
  __shared__ float s_most[SWEEP_MAX][16];
  static_assert(BM == 256, "a thread per id of a tile");
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n_bound; i += gridDim.x * blockDim.x) bound[i] = 0u;
  for (int id = blockIdx.x * blockDim.x + threadIdx.x; id < n_padded; id += gridDim.x * blockDim.x) {   // (whole tiles: n_padded is a multiple of 256)
    const float x = u[id];
    const int group = (threadIdx.x >> 4) & 15, at = id & 15;
    float* const rows = eu + (int64_t)(id >> 4) * (SWEEP_ROWS * SWEEP_GROUP) + at;
    const bool leave_zero = n_alpha > SWEEP_SPLIT_ROWS && zero_alpha >= 0;
    // (nine alphas none of which is zero: e^(alpha u) in a table of its own)
    const bool two = n_alpha > SWEEP_SPLIT_ROWS && !leave_zero;
    float* const factor = two ? rows + (int64_t)n_padded * SWEEP_ROWS : rows;
    float* const factor_u = two ? rows : rows + SWEEP_SPLIT_ROWS * SWEEP_GROUP;
    const int filled = two ? SWEEP_GROUP : SWEEP_SPLIT_ROWS;
    float spread = 0.f;
    int row = 0;
    for (int a = 0; a < n_alpha; ++a) {
      const float shift = alphas.a[a] * x;
      float most = shift, least = shift;
      most = largest_of_16(most);
      least = -largest_of_16(-least);
      spread = fmaxf(spread, most - least);
      // (with the margin for its rounding, SWEEP_MARGIN, unless no logit is shifted at all)
      most = most == 0.f && least == 0.f ? 0.f : most + SWEEP_MARGIN;
      if (at == a) {   // (alpha number a of the group: its first id + a)
        shift_max[id] = most;
        shift_min[id] = least;
        s_most[a][group] = most;
      }
      if (leave_zero && a == zero_alpha) continue;
      const float e = expf(shift);
      factor[row * SWEEP_GROUP] = e;
      factor_u[row * SWEEP_GROUP] = e * shift;
      ++row;
    }
    for (; row < filled; ++row) factor[row * SWEEP_GROUP] = factor_u[row * SWEEP_GROUP] = 0.f;
    if (at >= n_alpha) {
      shift_max[id] = at == 15 ? spread : 0.f;
      shift_min[id] = 0.f;
    }
    __syncthreads();
    if (threadIdx.x < 16) {
      float most = 0.f;
      if ((int)threadIdx.x < n_alpha) {
        most = s_most[threadIdx.x][0];
        for (int g = 1; g < 16; ++g) most = fmaxf(most, s_most[threadIdx.x][g]);
      }
      shift_tile[(id >> 8) * 16 + threadIdx.x] = most;
    }
    __syncthreads();
  }
  if (blockIdx.x != 0 || threadIdx.x >= 64) return;
  float largest = 0.f, alpha = 0.f;
  for (int i = threadIdx.x; i < n_blocks; i += 64) largest = sticky_max(largest, block_max[i]);
#pragma unroll
  for (int a = 0; a < SWEEP_MAX; ++a) alpha = fmaxf(alpha, fabsf(alphas.a[a]));
  const bool fine = alpha * largest <= SWEEP_SHIFT;
  const bool all_fine = __builtin_amdgcn_ballot_w64(!fine) == 0;
  if (threadIdx.x == 0) *general = all_fine ? 0 : 1;
}

// ---------------------------------------------------------------------------------------
// a8: merge the splits of each row and finalise.  One wavefront per row, one lane per split.
// ---------------------------------------------------------------------------------------
// One wavefront per row; lane s holds the lists of splits [s LPL, s LPL + LPL) (LPL = 1 while the splits fit one
// lane each; 4 when a pass of few rows cuts the vocabulary finer than that so as to fill the chip).  The row's
// lists (splits x k pairs, contiguous in the workspace) are first copied into LDS with coalesced loads: the k steps
// of the merge are a chain, each needing the next entry of whichever list won the step before, and from LDS that
// costs a fraction of a trip to memory.  At LPL = 1 a block is four wavefronts with a row each; at LPL = 4 a block
// has ONE row, all four wavefronts copy its lists (up to 64 KB: one wavefront alone would spend its time waiting for
// its own loads) and the first one merges.
// The chain's two reductions a step stay out of LDS (180 rows, 148 splits, k = 30, whole call: 125 us with exchanges through
// LDS, 107 now; 1500 rows, 37 splits, k = 5: 99 and 96).
// Dynamic LDS: rows of the block x splits x k x 8 bytes (at most 64 KB).
constexpr int MERGE_LPL = 4;                              // lists per lane of the merge when splits > 64
constexpr int MAX_PROJECT_SPLITS = MAX_SPLITS * MERGE_LPL;   // vocabulary splits per row block of the projection

template <int LPL>
__global__ __launch_bounds__(256) void ll_merge_kernel(const float4* __restrict__ stats, const uint2* __restrict__ top,
                                                       int rows, int splits, int k, int V, int topk_softmax,
                                                       const int32_t* __restrict__ target, int32_t* __restrict__ out_ids,
                                                       float* __restrict__ out_p, float* __restrict__ out_logp,
                                                       float* __restrict__ out_entropy, unsigned* __restrict__ bound, int bounds) {
  extern __shared__ __align__(8) uint2 lists[];
  const int wave = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63;
  const int row = LPL == 1 ? blockIdx.x * (blockDim.x >> 6) + wave : blockIdx.x;
  const bool valid = row < rows;          // (no early return: every wavefront reaches the barrier)
  const int n_entries = splits * k;
  uint2* mine = LPL == 1 ? lists + wave * n_entries : lists;
  if (valid) {
    const uint2* src = top + (int64_t)row * n_entries;
    if (LPL == 1)
      for (int i = lane; i < n_entries; i += 64) mine[i] = src[i];
    else
      for (int i = threadIdx.x; i < n_entries; i += blockDim.x) mine[i] = src[i];
  }
  __syncthreads();
  if (!valid || (LPL != 1 && wave != 0)) return;
  bool live[LPL];
  float4 q[LPL];
  float m_lane = -INFINITY, zt_lane = -INFINITY;
#pragma unroll
  for (int i = 0; i < LPL; ++i) {
    live[i] = lane * LPL + i < splits;
    q[i] = make_float4(-INFINITY, 0.f, 0.f, -INFINITY);
    if (live[i]) q[i] = stats[(int64_t)row * splits + lane * LPL + i];
    m_lane = fmaxf(m_lane, q[i].x);
    zt_lane = fmaxf(zt_lane, q[i].w);
  }
  const float M = wave_max(m_lane);
  float s_lane = 0.f, t_lane = 0.f;
#pragma unroll
  for (int i = 0; i < LPL; ++i) {
    const float sc = live[i] ? __builtin_amdgcn_exp2f((q[i].x - M) * LOG2E) : 0.f;
    s_lane += sc * q[i].y;
    t_lane += sc * q[i].z;
  }
  const float S = wave_sum(s_lane);
  const float T = wave_sum(t_lane);
  const float zt = wave_max(zt_lane);
  const float logS = logf(S);
  if (bound != nullptr && lane < bounds) bound[(int64_t)lane * rows + row] = 0u;   // the projection kernel of this pass is done with them: clear them for the next pass
  if (lane == 0) {
    out_entropy[row] = (M - T / S) + logS;
    if (target != nullptr) {
      const int t = target[row];
      out_logp[row] = (t >= 0 && t < V) ? (zt - M) - logS : __builtin_nanf("");
    }
  }
  // k-way merge of the per-split sorted lists (descending logit, ascending id): every lane holds the
  // heads of its lists; the wavefront's best head goes out and that list moves on.
  const uint2* tl = mine + lane * LPL * k;
  int head[LPL];
  float z[LPL];
  int id[LPL];
#pragma unroll
  for (int i = 0; i < LPL; ++i) {
    head[i] = 0;
    z[i] = -INFINITY;
    id[i] = INT_MAX;
    if (live[i]) {
      const uint2 e = tl[i * k];
      z[i] = __uint_as_float(e.x);
      id[i] = (int)e.y;
    }
  }
  float z0 = 0.f, sk = 0.f;   // top-k-only softmax: the largest selected logit and the sum over the selection
  float my_z = 0.f;           // lane j keeps the j-th selected logit and id, written out together at the end
  int my_id = 0;
  for (int j = 0; j < k; ++j) {
    float lz = z[0];   // this lane's best head: largest logit, smallest id among equals
    int li = id[0];
#pragma unroll
    for (int i = 1; i < LPL; ++i) {
      const bool better = z[i] > lz || (z[i] == lz && id[i] < li);
      lz = better ? z[i] : lz;
      li = better ? id[i] : li;
    }
    const float bz = wave_max(lz);
    const int bi = wave_min_int(lz == bz ? li : INT_MAX);
#pragma unroll
    for (int i = 0; i < LPL; ++i) {
      if (live[i] && z[i] == bz && id[i] == bi) {   // ids are distinct: exactly one list of one lane
        ++head[i];
        if (head[i] < k) {
          const uint2 e = tl[i * k + head[i]];
          z[i] = __uint_as_float(e.x);
          id[i] = (int)e.y;
        } else {
          z[i] = -INFINITY;
          id[i] = INT_MAX;
        }
      }
    }
    if (j == 0) z0 = bz;
    sk += __builtin_amdgcn_exp2f((bz - z0) * LOG2E);
    if (lane == j) {
      my_z = bz;
      my_id = bi;
    }
  }
  if (lane < k) {
    out_ids[(int64_t)row * k + lane] = my_id;
    // full-vocabulary probability, or the paper's own (Sec. 3.3): a softmax over the k selected logits only
    out_p[(int64_t)row * k + lane] = topk_softmax ? __builtin_amdgcn_exp2f((my_z - z0) * LOG2E) * (1.0f / sk)
                                                  : __builtin_amdgcn_exp2f(((my_z - M) - logS) * LOG2E);
  }
}

// e^(a - b), a and b of any distance that counts: what the rounding of a - b and of its product with log2 e leaves out is applied
// to the result.  (exp2f(rounded) alone is off by 2^-25 of the exponent: 1e-6 where two references are 20 apart.)
__device__ __forceinline__ float exp_difference(float a, float b) {
  constexpr float LOG2E_LOW = 1.92596299e-8f;   // log2 e - LOG2E
  const float d = a - b;
  if (!(fabsf(d) < 100.f)) return __builtin_amdgcn_exp2f(d * LOG2E);   // (0, infinity or NaN)
  const float back = d + b, lost = (a - back) + ((back - d) - b);      // a - b = d + lost
  const float x = d * LOG2E;
  const float rest = fmaf(d, LOG2E, -x) + (d * LOG2E_LOW + lost * LOG2E);
  return __builtin_amdgcn_exp2f(x) * fmaf(rest, 0.693147181f, 1.0f);
}

// Steering sweep, step 4: merge the splits of each (row, alpha) and finalise.  One wavefront each; lane l takes splits l,
// l + 64, ... (increasing ids), keeps their KS best, and the wavefront takes the best of its lanes' heads k times.
// The splits' references are any logits of the row, some of them far below its largest, so that M and log S are no small
// numbers that nearly cancel: the last steps are in 64 bits.
// LeftOut: of a sweep that forms u itself, the tokens that its factored form has left out (see ll_epilogue_sweep.h).
enum { FLAG_EXCEEDED, FLAG_GIVEN, FLAG_LEFT, FLAGS };   // flags; behind them GemmArgs' left_n
struct LeftOut {
  const int* flags;   // nullptr: none
  const float* z;
  const int* id;
  int slots;
  // f(id, logit, shifted logit) of the row's tokens in this lane's splits
  template <class F>
  __device__ __forceinline__ void each(int row, int splits, float alpha, const float* u, F f) const {
    const int block = row / SWEEP_OWN_ROWS * splits;
    for (int s = threadIdx.x & 63; s < splits; s += 64)
      for (int i = 0, n = flags[FLAGS + 4 * (block + s)]; i < n; ++i) {
        const int t = id[(block + s) * slots + i];
        const float x = z[((int64_t)row * splits + s) * slots + i];
        f(t, x, fmaf(alpha, u[t], x));
      }
  }
};
template <int KS>
__global__ __launch_bounds__(256) void ll_sweep_merge_kernel(const float4* __restrict__ stats, const uint2* __restrict__ top,
                                                             const float* __restrict__ ztgt, const float* __restrict__ u,
                                                             AlphaList alphas, int rows, int splits, int n_alpha, int k, int V,
                                                             const int32_t* __restrict__ target, int64_t out_stride,
                                                             int32_t* __restrict__ out_ids, float* __restrict__ out_p,
                                                             float* __restrict__ out_logp, float* __restrict__ out_entropy,
                                                             unsigned* __restrict__ bound, const LeftOut left) {
  const int item = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (item >= rows * n_alpha) return;
  const int lane = threadIdx.x & 63;
  const int row = item / n_alpha, a = item - row * n_alpha;
  const float4* const q = stats + (int64_t)item * splits;
  const uint2* const lists = top + (int64_t)item * splits * KS;
  float m = -INFINITY, zt = -INFINITY;
  float z[KS];
  int id[KS];
#pragma unroll
  for (int j = 0; j < KS; ++j) {
    z[j] = -INFINITY;
    id[j] = INT_MAX;
  }
  for (int s = lane; s < splits; s += 64) {
    m = fmaxf(m, q[s].x);
    if (target != nullptr) zt = fmaxf(zt, ztgt[(int64_t)row * splits + s]);
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      const uint2 e = lists[(int64_t)s * KS + i];
      float ze = __uint_as_float(e.x);
      int ie = (int)e.y;
#pragma unroll
      for (int j = 0; j < KS; ++j) {   // an entry that ranks above slot j takes it and pushes the slot's down (ids only grow: strictly greater)
        const bool above = ze > z[j];
        const float zo = z[j];
        const int io = id[j];
        z[j] = above ? ze : zo;
        id[j] = above ? ie : io;
        ze = above ? zo : ze;
        ie = above ? io : ie;
      }
    }
  }
  const bool some_left = left.flags != nullptr && left.flags[FLAG_LEFT] != 0 && left.flags[FLAG_EXCEEDED] == 0;
  if (some_left)
    left.each(row, splits, alphas.a[a], u, [&](int ie, float x, float ze) {
      if (target != nullptr && ie == target[row]) zt = x;
      m = fmaxf(m, ze);
#pragma unroll
      for (int j = 0; j < KS; ++j) {
        const bool above = ze > z[j] || (ze == z[j] && ie < id[j]);
        const float zo = z[j];
        const int io = id[j];
        z[j] = above ? ze : zo;
        id[j] = above ? ie : io;
        ze = above ? zo : ze;
        ie = above ? io : ie;
      }
    });
  const float M = wave_max(m);
  float s_lane = 0.f, t_lane = 0.f;
  for (int s = lane; s < splits; s += 64) {
    const float4 x = q[s];
    const float sc = exp_difference(x.x, M);
    s_lane = fmaf(sc, x.y, s_lane);
    t_lane = fmaf(sc, x.z, t_lane);
  }
  if (some_left)
    left.each(row, splits, alphas.a[a], u, [&](int, float, float w) {
      const float sc = exp_difference(w, M);
      s_lane += sc;
      t_lane = fmaf(sc, w, t_lane);
    });
  const float S = wave_sum(s_lane), T = wave_sum(t_lane);
  const double lse = (double)M + log((double)S);
  zt = wave_max(zt);
  const int64_t o = (int64_t)a * out_stride + row;
  // the projection kernel of this pass is done with the bounds, if it had any: clear them for the next pass
  if (bound != nullptr && lane < k) bound[(lane * n_alpha + a) * rows + row] = 0u;
  if (lane == 0) {
    out_entropy[o] = (float)(lse - (double)T / (double)S);
    if (target != nullptr) {
      const int t = target[row];
      out_logp[o] = t >= 0 && t < V ? (float)(((double)zt + (double)alphas.a[a] * u[t]) - lse) : __builtin_nanf("");
    }
  }
  float my_z = 0.f;   // lane j keeps the j-th
  int my_id = 0;
  for (int j = 0; j < k; ++j) {
    const float bz = wave_max(z[0]);
    const int bi = wave_min_int(z[0] == bz ? id[0] : INT_MAX);
    if (z[0] == bz && id[0] == bi) {   // ids are distinct: one lane
#pragma unroll
      for (int i = 0; i + 1 < KS; ++i) {
        z[i] = z[i + 1];
        id[i] = id[i + 1];
      }
      z[KS - 1] = -INFINITY;
      id[KS - 1] = INT_MAX;
    }
    if (lane == j) {
      my_z = bz;
      my_id = bi;
    }
  }
  if (lane < k) {
    out_ids[o * k + lane] = my_id;
    out_p[o * k + lane] = expf((float)((double)my_z - lse));
  }
}

// ---------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------
// The few-rows kernel: how the vocabulary is dealt.  One part per compute unit, or fewer when there are not eight groups of
// 16 vocabulary rows (one per wavefront) for each; a part has one workgroup, or several that share its rows (row_groups).  A wavefront holds the accumulators of MU
// groups against all the rows, so the register file bounds MU by the number of 16-row blocks; a larger share of the
// vocabulary goes in two or more rounds of workgroups.
struct FewPlan {
  bool ok, two_rounds;   // two_rounds: of more than 96 rows
  int nj, mu, units, splits;   // nj: 16-row blocks of the kernel instance; mu: groups per wavefront; units: groups in all
  int row_groups;              // workgroups that share a part, of nj blocks each
};

constexpr int SHORT_KMAX = 20, SHORT_KMAX_BIAS = 12;   // longest lists of the kernel of short calls

FewPlan make_few_plan(const ll_shape* s, int k) {
  FewPlan f = {};
  if (s->N < 1 || s->N > FEW_ROWS) return f;
  const int blocks = (int)((s->N + 15) / 16);
  f.nj = blocks <= 4 ? blocks : (blocks <= 6 ? 6 : 8);
  const int mu_max = f.nj <= 4 ? 5 : (f.nj == 6 ? 4 : 3);
  f.units = (int)(((int64_t)s->V + 15) / 16);
  int parts = (f.units + FEW_WAVES - 1) / FEW_WAVES;
  if (parts > NUM_CU) parts = NUM_CU;
  const int share = (f.units + parts - 1) / parts;
  const int rounds = (share + FEW_WAVES * mu_max - 1) / (FEW_WAVES * mu_max);
  f.splits = parts * rounds;
  if (f.splits > FEW_MAX_SPLITS) return f;   // V beyond some 200 000 to 330 000
  // More than 96 rows over more than one round (V past 98 000): a round's contraction and epilogue are no longer small beside
  // its share of W_U, and the 256-row tiles have few insertions left in a split's first tile (see exchange_classes), up to the
  // longest list that has classes without a bias and with one (project_impl); with the shortest where rows are not whole stages, which
  // those tiles pay more for (107 rows, d = 5096, V = 99168, k = 15: 280 | 305).  128 rows, here | 256-row kernels, us:
  // V = 128256: d = 64: k = 1 54 | 34, k = 8 56 | 41, k = 20 59 | 55, k = 24 76 | 126; d = 2560: k = 1 186 | 167, k = 8 187 | 153, k = 20 187 | 167,
  // k = 24 197 | 239; d = 8192: k = 1 432 | 427, k = 12 423 | 406, k = 20 421 | 416, k = 32 460 | 498; V = 151936, d = 1024: k = 1 113 | 100,
  // k = 20 119 | 116.
  f.two_rounds = rounds > 1 && f.nj == 8;
  if (f.two_rounds && k <= (s->d % DK == 0 ? SHORT_KMAX_BIAS : 4)) return f;
  f.mu = ((f.units + f.splits - 1) / f.splits + FEW_WAVES - 1) / FEW_WAVES;
  // A vocabulary of up to 16384 has no part for every second compute unit: the rows are then dealt to several workgroups a part, down to 16 each.
  // What that shortens is a part's epilogue, and the A tiles; W's lines come from memory once all the same (xcd_logical_block).  Whole
  // calls, one workgroup a part | several, us (rows, d, V, k): 64, 256, 4096, 5: 17.4 | 13.3; 128, 64, 4000, 5: 22.5 | 12.3; 81, 512, 8000, 10: 26.5 | 17.8;
  // 81, 1608, 6000, 5: 37.4 | 23.0; 100, 1024, 12000, 20: 31.7 | 25.8; 64, 2048, 16000, 10: 34.3 | 31.1; 128, 8192, 10000, 10: 114.6 | 91.7;
  // 20, 8192, 16000, 10: 94.9 | 89.1.  With W_U out of the caches: 64, 256, 4096, 5: 24.1 | 18.9; 81, 1608, 6000, 5: 48.7 | 36.2; 33, 5120, 8192, 10: 79.2 | 71.2;
  // 64, 2048, 16000, 10: 51.4 | 48.1; 128, 2560, 16000, 10: 75.1 | 59.9; 20, 8192, 16000, 10: 96.4 | 91.1.  The 256-row tiles take 0.98 to 1.4 times as long there (65, 96 and
  // 128 rows, d = 256 to 8192, lists of five); from V = 16385 to 20000, with one workgroup a part, 0.79 to 1.0 times.
  f.row_groups = 1;
  for (int nj = 1; nj < f.nj; ++nj) {
    const int groups = (blocks + nj - 1) / nj;
    if (nj != 5 && nj != 7 && f.splits * groups <= NUM_CU) {
      f.nj = nj;
      f.row_groups = groups;
      break;
    }
  }
  f.ok = true;
  return f;
}

struct Plan {
  size_t off_inv_rms, off_bound, off_bias, off_stats, off_top, off_panel, total;   // total: what a call cannot do without
  size_t roomy;   // with a row of zeros behind the panel and the bounds of the classes of splits (see classes_offset), never less for more rows:
                  // the least that is accepted, but in the static buffer
  int64_t lda;
  FewPlan few;
  size_t few_total, few_off_stats, few_off_cand, few_off_count, few_off_panel;
};

bool shape_ok(const ll_shape* s, int k) {
  if (s == nullptr) return false;
  if (s->N < 0 || s->d <= 0 || s->V <= 0 || (s->d & 7) != 0) return false;
  // rounding up to whole tiles (V) and whole K stages (d) stays inside 32 bits
  if (s->V > INT32_MAX - BM || s->d > INT32_MAX - 2 * DK) return false;
  if (k < 1 || k > LL_KMAX || k > s->V) return false;
  return true;
}

// Where the bounds of the classes of splits stand (one a row and class, k of them, in passes of at least k splits: rows x k never
// exceeds MAX_PARTIALS), and how much room they may want: behind what of the panel the pass fills, so that only the largest pass in
// the static buffer, where nothing is left behind its panel, has none for them.  Such a pass goes without classes, with the same results;
// reserving them there always would make the passes smaller (d = 3328, V = 128256, k = 20: 7936 rows).
size_t classes_offset(size_t off_panel, int64_t panel_rows, int64_t lda) {
  return align_up(off_panel + (size_t)panel_rows * (size_t)lda * sizeof(uint16_t), 256);
}
size_t classes_bytes(size_t rows, int k) {
  if (k > SHORT_KMAX) return 0;
  return (rows * k < (size_t)MAX_PARTIALS ? rows * k : (size_t)MAX_PARTIALS) * sizeof(unsigned);
}

Plan make_plan(const ll_shape* s, int k, int chunk_rows = CHUNK_ROWS) {
  Plan p = {};
  size_t off = 0;
  p.off_inv_rms = off;
  off = align_up(off + (size_t)s->N * sizeof(float), 256);
  const size_t rows = (size_t)(s->N < chunk_rows ? s->N : chunk_rows);
  p.off_bound = off;  // per-row top-k bounds shared between the splits of a pass
  off = align_up(off + rows * sizeof(unsigned), 256);
  p.off_bias = off;   // the bias padded to whole tiles (ll_project_ex)
  off = align_up(off + (size_t)((s->V + BM - 1) / BM) * BM * sizeof(float), 256);
  p.off_stats = off;
  const size_t partials = rows * MAX_PROJECT_SPLITS < (size_t)MAX_PARTIALS ? rows * MAX_PROJECT_SPLITS : (size_t)MAX_PARTIALS;
  off = align_up(off + partials * sizeof(float4), 256);
  p.off_top = off;
  off = align_up(off + partials * (size_t)k * sizeof(uint2), 256);
  p.lda = (s->d + DK - 1) / DK * DK;
  p.off_panel = off;
  p.total = classes_offset(off, (int64_t)rows, p.lda);
  p.roomy = align_up(classes_offset(off, (int64_t)rows + 1, p.lda) + classes_bytes(rows, k), 256);
  // The few-rows kernel's own layout of the same workspace, larger than what many more rows need above: 64 entries a row and part.
  // It is taken only where it fits the workspace that the caller handed over (one sized for a longer call need not hold it), and
  // where it also fits the library's static buffer, so that ll_project and ll_project_static run the same kernels.
  p.few = make_few_plan(s, k);
  if (p.few.ok) {
    const size_t lists = (size_t)s->N * p.few.splits;
    off = 0;
    p.few_off_stats = off;
    off = align_up(off + lists * sizeof(float4), 256);
    p.few_off_cand = off;
    off = align_up(off + lists * FEW_CAP * sizeof(uint2), 256);
    p.few_off_count = off;
    off = align_up(off + lists * sizeof(int), 256);
    p.few_off_panel = off;
    off = align_up(off + rows * (size_t)p.lda * sizeof(uint16_t), 256);
    p.few_total = off;
    p.few.ok = off <= (size_t)LL_STATIC_SCRATCH_BYTES;
  }
  return p;
}

// What a call is fastest with: room for the few-rows kernel's layout where that applies.
size_t wanted_bytes(const Plan& plan) { return plan.few.ok && plan.few_total > plan.roomy ? plan.few_total : plan.roomy; }

template <bool STREAM>
void (*few_kernel(int nj, int mu))(const FewArgs) {
#define LL_FEW(NJ, MU) \
  if (nj == NJ && mu <= MU) return ll_lens_few_kernel<NJ, MU, STREAM>
  LL_FEW(1, 1); LL_FEW(1, 3); LL_FEW(1, 5);
  LL_FEW(2, 1); LL_FEW(2, 3); LL_FEW(2, 5);
  LL_FEW(3, 1); LL_FEW(3, 3); LL_FEW(3, 5);
  LL_FEW(4, 1); LL_FEW(4, 3); LL_FEW(4, 5);
  LL_FEW(6, 2); LL_FEW(6, 3); LL_FEW(6, 4);
  LL_FEW(8, 1); LL_FEW(8, 2); LL_FEW(8, 3);
#undef LL_FEW
  return nullptr;
}

// A kernel that uses more than 64 KB of dynamic LDS has to be told so once per device; remembered
// here so that the hot path makes no attribute call.
int allow_dynamic_lds(const void* kern, size_t lds) {
  static std::mutex mu;
  static std::vector<std::pair<int, const void*>> done;
  int dev = -1;
  LL_HIP_CHECK(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lock(mu);
  for (const auto& e : done)
    if (e.first == dev && e.second == kern) return LL_OK;
  LL_HIP_CHECK(hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  done.emplace_back(dev, kern);
  return LL_OK;
}

// Most tiles a workgroup for which the kernel of short calls is taken, with the classes of splits and without (half tiles only).
// Whole calls, us, long | short (d, V, rows, k: tiles a workgroup).  With classes: 256, 4096, 1500, 10 (1, in halves): 50 | 30; 1608,
// 50257, 777, 3 with a bias (4): 197 | 187; 1024, 50257, 1500, 20 (5): 229 | 189; 4096, 128256, 957, 10 (8): 847 | 830; 1024,
// 128256, 4000, 10 (32): 949 | 920; 5120, 151936, 4160, 3 with a bias (40): no difference.  Without: 256, 4096, 4000, 20 (1): 78 | 77;
// 1608, 50257, 4000, 20 (13): 653 | 648; 256, 50257, 4000, 20 (13): 275 | 281; 256, 128256, 4000, 20 (32): 537 | 555; 4000 rows,
// k = 20 at d = 1024 with 3, 4 and 13 tiles: 155 | 150, 185 | 180, 460 | 460, and at d = 64 with 13 and 17: 226 | 230, 271 | 275.
constexpr int SHORT_TILES = 32, SHORT_TILES_WITHOUT = 8;

// The fewest vocabulary splits that give no workgroup more tiles than `most` splits would: the call takes as long as its
// busiest workgroup, and the others' lists cost the merge (197 tiles over 64 splits are four each at most; so they are over 50).
int even_splits(int tiles, int most) {
  if (most > tiles) most = tiles;
  if (most < 1) most = 1;
  const int each = (tiles + most - 1) / most;
  return (tiles + each - 1) / each;
}

// How a pass of `rows` rows deals the vocabulary.  One workgroup per compute unit: a pass of few rows cuts it finer (its cost is then the
// one read of W_U, spread over every compute unit's share of the memory system).
struct Deal {
  int row_blocks, splits;
  int half_tiles, classes;   // as in GemmArgs: of the kernel of short calls, where that is taken
  int tiles_each;            // whole tiles of the busiest workgroup, were there no half ones
};

// dear: the kernel of short calls costs more a tile than it saves in insertions, few in the shortest list (its bias comes late where
// the last K stage is ragged; of eight stages and more: in shorter ones the insertions weigh more).  Taken up to SHORT_TILES_WITHOUT
// tiles, for half a tile less up to twice those, for an arg max only for that.  Whole calls, long over short (N x V: tiles), k = 1 and
// 3 with a bias, d = 968: 300 x 128256 (4) 0.97, 1.04; 957 x 128256 (8) 0.96, 1.00; 2500 x 100000 (16) 0.95, 0.99; 4000 x 128256 (32)
// 0.96, 0.97; d = 1608: 300 x 128256 0.97, 1.00; 957 x 128256 0.99, 0.99; 1500 x 100000 (10, a half tile less) 1.01, 1.03; 4000 x
// 128256 0.98, 1.00; d = 200: 4000 x 128256 1.04, 1.05.  k = 10: 1.03 to 1.18.
Deal deal_vocabulary(int rows, int V, int k, bool short_kernel, bool dear) {
  const int tiles = (V + BM - 1) / BM;
  Deal l = {};
  l.row_blocks = (rows + BN - 1) / BN;
  const int most = NUM_CU / l.row_blocks < MAX_PROJECT_SPLITS ? NUM_CU / l.row_blocks : MAX_PROJECT_SPLITS;
  l.splits = even_splits(tiles, most);
  const int each = l.tiles_each = (tiles + l.splits - 1) / l.splits;
  if (!short_kernel || each > (dear ? SHORT_TILES / 2 : SHORT_TILES)) return l;
  // Few tiles a workgroup: the kernel that can end a split in half a tile, where that leaves the busiest workgroup half a tile less,
  // and that deals at least k splits into k classes (see exchange_classes).
  const int halves = (V + BM / 2 - 1) / (BM / 2), each_half = (halves + most - 1) / most;
  const int half_splits = (halves + each_half - 1) / each_half;
  if (each_half < 2 * each && (half_splits >= k || each <= SHORT_TILES_WITHOUT)) {
    l.half_tiles = halves;
    l.splits = half_splits;
  }
  if (l.splits >= k && !(dear && l.half_tiles == 0 && (k == 1 || each > SHORT_TILES_WITHOUT))) l.classes = k;
  return l;
}

// (few rows: one wavefront per block, so that they spread over the compute units)
void launch_norm_panel(const uint16_t* hidden, const uint16_t* gamma, uint16_t* panel, int rows, int zero_rows, int d, int64_t lda,
                       float eps, unsigned* bound, int bounds, hipStream_t stream) {
  const int per_block = rows <= 1024 ? 1 : 4;
  const dim3 grid((unsigned)((rows + zero_rows + per_block - 1) / per_block)), block(64 * per_block);
  if (d <= 64 * 8 * 4)
    hipLaunchKernelGGL(ll_norm_panel_kernel<4>, grid, block, 0, stream, hidden, gamma, panel, rows, zero_rows, d, lda, eps, bound, bounds);
  else if (d <= 64 * 8 * 8)
    hipLaunchKernelGGL(ll_norm_panel_kernel<8>, grid, block, 0, stream, hidden, gamma, panel, rows, zero_rows, d, lda, eps, bound, bounds);
  else if (d <= 64 * 8 * 16)
    hipLaunchKernelGGL(ll_norm_panel_kernel<16>, grid, block, 0, stream, hidden, gamma, panel, rows, zero_rows, d, lda, eps, bound, bounds);
  else
    hipLaunchKernelGGL(ll_norm_panel_kernel<0>, grid, block, 0, stream, hidden, gamma, panel, rows, zero_rows, d, lda, eps, bound, bounds);
}

void launch_sweep_panel(const uint16_t* hidden, const uint16_t* gamma, uint16_t* panel, int rows, int d, int64_t lda, float eps,
                        unsigned* bound, int bounds, const uint16_t* W, int V, const float* v, float alpha_most, int n_waves, int samples,
                        float* sampled, float* row_sq, int* flags, int n_flags, hipStream_t stream) {
  const int per_block = rows <= 1024 ? 1 : 4;
  const dim3 grid((unsigned)((n_waves + rows + 1 + 1 + SWEEP_PARTS * sweep_part_pieces(lda) + per_block - 1) / per_block)), block(64 * per_block);
  const auto kernel = d <= 64 * 8 * 4    ? ll_sweep_panel_kernel<4>
                      : d <= 64 * 8 * 8  ? ll_sweep_panel_kernel<8>
                      : d <= 64 * 8 * 16 ? ll_sweep_panel_kernel<16>
                                         : ll_sweep_panel_kernel<0>;
  hipLaunchKernelGGL(kernel, grid, block, 0, stream, hidden, gamma, panel, rows, d, lda, eps, bound, bounds, W, V, v, alpha_most, n_waves, samples,
                     sampled, row_sq, flags, n_flags);
}

int project_impl(const ll_shape* shape, void* workspace, size_t workspace_bytes, const void* hidden, const void* gamma,
                 const void* W_U, const float* bias, unsigned flags, float eps, int k, const int32_t* target_ids,
                 int32_t* out_topk_ids, float* out_topk_p,
                 float* out_target_logp, float* out_entropy, hipStream_t stream, float* phase_ms,
                 int chunk_rows = CHUNK_ROWS, bool static_buffer = false, int W_in_cache = -1) {   // W_in_cache: -1 by its size
  if (!shape_ok(shape, k)) return LL_EINVAL;
  if (shape->N == 0) {
    if (phase_ms) phase_ms[0] = phase_ms[1] = phase_ms[2] = 0.f;
    return LL_OK;
  }
  if (hidden == nullptr || W_U == nullptr || out_topk_ids == nullptr || out_topk_p == nullptr || out_entropy == nullptr)
    return LL_EINVAL;
  if (target_ids != nullptr && out_target_logp == nullptr) return LL_EINVAL;
  if (!(eps >= 0.f)) return LL_EINVAL;
  if ((flags & ~(unsigned)(LL_FLAG_TOPK_SOFTMAX | LL_FLAG_REGISTER_STAGED)) != 0 || ((uintptr_t)bias & 3)) return LL_EINVAL;
  const uintptr_t align_or = (uintptr_t)hidden | (uintptr_t)W_U | (uintptr_t)gamma;
  if (align_or & 15) return LL_EINVAL;
  const Plan plan = make_plan(shape, k, chunk_rows);
  if (workspace == nullptr || workspace_bytes < (static_buffer ? plan.total : plan.roomy) || ((uintptr_t)workspace & 255)) return LL_EWORKSPACE;

  unsigned char* ws = static_cast<unsigned char*>(workspace);
  float* inv_rms = reinterpret_cast<float*>(ws + plan.off_inv_rms);
  float4* stats = reinterpret_cast<float4*>(ws + plan.off_stats);
  uint2* top = reinterpret_cast<uint2*>(ws + plan.off_top);
  uint16_t* panel = reinterpret_cast<uint16_t*>(ws + plan.off_panel);

  const int64_t N = shape->N;
  const int d = shape->d, V = shape->V;
  const bool has_gamma = gamma != nullptr;
  const bool few_rows = plan.few.ok && workspace_bytes >= plan.few_total && !(flags & LL_FLAG_REGISTER_STAGED) &&
                        !(plan.few.two_rounds && d % DK == 0 && k <= SHORT_KMAX && bias == nullptr);
  // The direct-to-LDS kernel addresses rows with 32-bit byte offsets from a per-tile base.  It takes every other shape, a d
  // that is not a multiple of 64 in an instantiation of its own, which the longest list with a bias does not have.
  // 777 rows, d = 1608, V = 50257, k = 3 with a bias: 201 us, on the register-staged kernel 369
  // It needs the rows padded, which is a launch.  With classes of splits that always pays, unless there is a bias and no half tile; else
  // calls whose busiest workgroup has little to do are as fast or faster without.  Whole calls, direct-to-LDS over register-staged, by the
  // stages of 64 columns that the busiest workgroup has to do:
  //   classes, no bias (150 to 8192 rows, V = 1000 to 128256, k = 1, 10, 20): 1 stage 0.54-0.93, 20 stages 0.53-0.74
  //   k = 20 and 10 in fewer splits (2500 to 8192 rows): a norm  1 1.02-1.05, 2 0.99-1.02, 3 0.97-1.00;  none  1 1.05-1.08, 3 1.01-1.04, 5 0.99-1.02
  //   a bias (k = 3, 10) and half tiles: 0.63-0.90;  whole ones: a norm  1 0.98-1.09, 2 at most 1.04, 3 1.02, 4 1.02;  none  1 1.01-1.13,
  //     3 at most 1.07, 5 1.04, 7 1.03
  //   no kernel of short calls (k = 24, 32; 16 with a bias): a norm  1 0.99-1.05, 4 0.97-1.0, 5 0.97-1.01;  none  1 1.02-1.09, 4 0.97-1.06
  const int tiles = (V + BM - 1) / BM;
  const bool has_short = short_topk_kernel(k, bias != nullptr, d % DK != 0) != nullptr;
  const bool dear = bias != nullptr && d % DK != 0 && k <= 4 && plan.lda >= 8 * DK;
  const Deal first = deal_vocabulary((int)(N < CHUNK_ROWS ? N : CHUNK_ROWS), V, k, has_short, dear);   // (whatever the scratch: the same kernel)
  const int64_t stages = (int64_t)first.tiles_each * (plan.lda / DK);
  const bool worth_padding = (first.classes > 0 && (bias == nullptr || first.half_tiles > 0)) ||
                             stages >= (has_short ? (has_gamma ? 3 : 5) : (has_gamma ? 6 : 10));
  const GemmKernel tail_kern = d % DK != 0 && worth_padding ? tail_topk_kernel(k, bias != nullptr) : nullptr;
  const bool dma = !(flags & LL_FLAG_REGISTER_STAGED) && (d % DK == 0 || tail_kern != nullptr) &&
                   (int64_t)BM * plan.lda * 2 < (int64_t)1 << 31 && (int64_t)CHUNK_ROWS * plan.lda * 2 < (int64_t)1 << 31;
  const size_t lds = dma ? (size_t)SLOTS * SLOT_BYTES : (size_t)(BM + BN) * BK * 2;
  // A bias (rare: the paper's model families have none) selects a separate instantiation of the
  // kernel, so that calls without one carry no code or registers for it.
  const GemmKernel kern = dma && tail_kern != nullptr ? tail_kern : with_list_length(k, [&](auto kr) -> GemmKernel {
    constexpr int KR = decltype(kr)::value;
    if (dma) return bias ? ll_lens_gemm_dma_kernel<TopKEpilogue<KR, true>> : ll_lens_gemm_dma_kernel<TopKEpilogue<KR, false>>;
    return bias ? ll_lens_gemm_kernel<TopKEpilogue<KR, true>> : ll_lens_gemm_kernel<TopKEpilogue<KR, false>>;
  });
  if (const int rc = allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds); rc != LL_OK) return rc;
  const GemmKernel short_kern = dma ? short_topk_kernel(k, bias != nullptr, d % DK != 0) : nullptr;
  if (short_kern != nullptr)
    if (const int rc = allow_dynamic_lds(reinterpret_cast<const void*>(short_kern), lds); rc != LL_OK) return rc;
  // The direct-to-LDS kernel reads hidden in place when the rows need neither scaling nor padding.
  const bool need_panel = dma && (has_gamma || plan.lda != d);

  // Timing (ll_project_timed only): events are recorded in-stream around every kernel and read
  // after one synchronisation at the end, so the kernels run back to back as in ll_project.
  // (the events are created once per thread and kept: a timed call costs no event creation after the first)
  static thread_local std::vector<hipEvent_t> ev_pool;
  size_t n_ev = 0;
  auto mark = [&]() -> hipError_t {
    if (!phase_ms) return hipSuccess;
    if (n_ev == ev_pool.size()) {
      hipEvent_t e = nullptr;
      hipError_t rc = hipEventCreate(&e);
      if (rc != hipSuccess) return rc;
      ev_pool.push_back(e);
    }
    return hipEventRecord(ev_pool[n_ev++], stream);
  };
  auto finish = [&](int rc) { return rc; };
  const std::vector<hipEvent_t>& ev = ev_pool;
  auto read_phases = [&]() -> int {   // ll_project_timed: four marks per row pass
    if (!phase_ms) return LL_OK;
    LL_HIP_CHECK(hipStreamSynchronize(stream));
    phase_ms[0] = phase_ms[1] = phase_ms[2] = 0.f;
    for (size_t i = 0; i + 3 < n_ev; i += 4)
      for (int j = 0; j < 3; ++j) {
        float ms = 0.f;
        LL_HIP_CHECK(hipEventElapsedTime(&ms, ev[i + j], ev[i + j + 1]));
        phase_ms[j] += ms;
      }
    return LL_OK;
  };
#define LL_CHECK_F(expr)                                   \
  do {                                                     \
    hipError_t e__ = (expr);                               \
    if (e__ != hipSuccess) return finish(hip_failed(e__)); \
  } while (0)

  // Few rows: one read of W_U.  Whole call, us, here / on the 256-row tiles: d = 8192, V = 128256, k = 20: 1 row 331 / 480, 81 rows
  // 348 / 490, 97 to 128 rows (two rounds of workgroups) 460 / 495; d = 2560, V = 151936, k = 10: 37 rows 145 / 245, 128 rows 228 /
  // 275; 64 rows of d = 256, V = 4096: 13 / 49.  Past 128 rows the accumulators do not fit and the 256-row tiles are the better split.
  if (few_rows) {
    const FewPlan& few = plan.few;
    uint16_t* few_panel = reinterpret_cast<uint16_t*>(ws + plan.few_off_panel);
    const bool copy = has_gamma || plan.lda != d;
    LL_CHECK_F(mark());
    if (copy) {
      launch_norm_panel(static_cast<const uint16_t*>(hidden), static_cast<const uint16_t*>(gamma), few_panel, (int)N, 0, d, plan.lda, eps,
                        nullptr, 0, stream);
      LL_CHECK_F(hipGetLastError());
    }
    FewArgs a;
    a.A = copy ? few_panel : static_cast<const uint16_t*>(hidden);
    a.W = static_cast<const uint16_t*>(W_U);
    a.target = target_ids;
    a.bias = bias;
    a.stats = reinterpret_cast<float4*>(ws + plan.few_off_stats);
    a.cand = reinterpret_cast<uint2*>(ws + plan.few_off_cand);
    a.count = reinterpret_cast<int*>(ws + plan.few_off_count);
    a.lda = plan.lda;
    a.rows = (int)N;
    a.d = d;
    a.V = V;
    a.k = k;
    a.splits = few.splits;
    a.units = few.units;
    a.row_groups = few.row_groups;
    LL_CHECK_F(mark());
    // Whether the loads of W_U go past the caches: where its rows are whole lines of 128 bytes (others share lines between two stages,
    // and are faster through the caches whatever the size) and it is more than a third of the Infinity Cache.  Up to there it stays
    // in that cache from one call to the next beside twice its bytes of other weights, and the next call finds it there; a larger one read
    // that way only drives out what those would have found.  Whole calls, past the caches | through them, us: repeated on one
    // W_U, behind a read of twice its bytes (the read included), and on W_U that are not in the cache (d, MB, rows; k = 10, at
    // d = 576 16):
    //   2048, 30, 37: 31.6 | 31.2, 54.2 | 51.8, 33.6 | 34.4     1024, 34, 37: 24.1 | 23.8, 47.3 | 45.5, 25.0 | 25.6
    //   2560, 42, 37: 38.2 | 35.6, 63.2 | 59.2, 39.4 | 40.7     1024, 66, 37: 27.9 | 26.5, 58.9 | 57.4, 27.6 | 28.7
    //   4096, 66, 37: 51.7 | 47.6, 83.8 | 78.6, 52.5 | 53.2      768, 77, 64: 35.0 | 32.8, 69.1 | 67.5, 34.6 | 36.1
    //    576, 92, 36: 33.0 | 33.5, 72.8 | 83.1, 33.2 | 35.3     2048, 123, 37: 42.4 | 34.4, 92.2 | 118, 41.0 | 43.8
    //   4096, 123, 37: 55.5 | 48.3, 106 | 129, 54.6 | 56.4      and repeated, not in the cache: 4096, 240, 16: 63.3 | 50.4, 59.0 | 64.5
    //   4096, 400, 16: 99.9 | 109, 93.8 | 101      2560, 778, 37: 144 | 159, 139 | 154         8192, 1050, 81: 194 | 213, 204 | 226
    // and of rows that are not whole lines:
    //   1608, 60, 16: 32.3 | 26.3, 35.5 | 34.2     1608, 400, 81: 138 | 113, 137 | 112        4104, 1050, 16: 298 | 224, 300 | 226
    // (The scope bits of the loads, sc0 and sc1, make no difference either way.)
    const bool kept = W_in_cache < 0 ? (int64_t)V * d * 2 <= INFINITY_CACHE_BYTES / 3 : W_in_cache > 0;
    const bool stream_W = ((uintptr_t)W_U | (uintptr_t)d * 2) % 128 == 0 && !kept;
    hipLaunchKernelGGL(stream_W ? few_kernel<true>(few.nj, few.mu) : few_kernel<false>(few.nj, few.mu), dim3(few.row_groups > 1 ? (few.splits * few.row_groups + NUM_XCD - 1) / NUM_XCD * NUM_XCD : few.splits), dim3(FEW_THREADS), 0, stream, a);
    LL_CHECK_F(hipGetLastError());
    LL_CHECK_F(mark());
    hipLaunchKernelGGL(ll_few_merge_kernel, dim3((unsigned)N), dim3(FEW_MERGE_THREADS), 0, stream, (const float4*)a.stats, (const uint2*)a.cand,
                       (const int*)a.count, a.splits, k, V, (flags & LL_FLAG_TOPK_SOFTMAX) ? 1 : 0, target_ids, out_topk_ids,
                       out_topk_p, out_target_logp, out_entropy);
    LL_CHECK_F(hipGetLastError());
    LL_CHECK_F(mark());
    return finish(read_phases());
  }

  // A pass's deal, and where its shared bounds stand (off_bound; `bounds` of them a row).
  struct Pass : Deal {
    int bounds;
    size_t off_bound;
  };
  auto pass = [&](int rows) {
    Pass l = {deal_vocabulary(rows, V, k, short_kern != nullptr, dear), 1, plan.off_bound};
    const size_t at = classes_offset(plan.off_panel, need_panel ? rows + 1 : 0, plan.lda);
    if (l.classes > 0 && at + classes_bytes((size_t)rows, k) <= workspace_bytes) {
      l.bounds = k;
      l.off_bound = at;
    } else {
      l.classes = 0;
    }
    return l;
  };
  // Top-k bounds shared between the vocabulary splits of a row (direct-to-LDS kernel): zero at the start of a pass.  The panel
  // kernel clears them; where the rows are read in place a launch of its own does for the first pass, and the merge kernel of a pass
  // for the next one.  That launch clears what the passes use: all but the last are alike, and two kinds of them either share a place
  // or have each its own.
  if (dma && !need_panel) {
    const int full = (int)(N < chunk_rows ? N : chunk_rows), last = (int)(N % chunk_rows);
    const Pass a = pass(full), b = last > 0 ? pass(last) : a;
    int64_t n_a = (int64_t)full * a.bounds, n_b = (int64_t)last * b.bounds;
    if (a.off_bound == b.off_bound) {
      n_a = n_a > n_b ? n_a : n_b;
      n_b = 0;
    }
    hipLaunchKernelGGL(ll_zero_u32_kernel, dim3((unsigned)((n_a + 255) / 256)), dim3(256), 0, stream, reinterpret_cast<unsigned*>(ws + a.off_bound), (int)n_a);
    LL_CHECK_F(hipGetLastError());
    if (n_b > 0) {
      hipLaunchKernelGGL(ll_zero_u32_kernel, dim3((unsigned)((n_b + 255) / 256)), dim3(256), 0, stream, reinterpret_cast<unsigned*>(ws + b.off_bound), (int)n_b);
      LL_CHECK_F(hipGetLastError());
    }
  }
  float* bias_padded = nullptr;
  if (bias != nullptr) {
    bias_padded = reinterpret_cast<float*>(ws + plan.off_bias);
    hipLaunchKernelGGL(ll_pad_bias_kernel, dim3((tiles * BM + 1023) / 1024), dim3(256), 0, stream, bias, V, bias_padded, tiles * BM);
    LL_CHECK_F(hipGetLastError());
  }
  for (int64_t r0 = 0; r0 < N; r0 += chunk_rows) {
    const int rows = (int)((N - r0) < chunk_rows ? (N - r0) : chunk_rows);
    const uint16_t* h_rows = static_cast<const uint16_t*>(hidden) + r0 * d;
    const Pass l = pass(rows);
    const int row_blocks = l.row_blocks, splits = l.splits, bounds = l.bounds;
    unsigned* const bound = dma ? reinterpret_cast<unsigned*>(ws + l.off_bound) : nullptr;
    // (a row of zeros for the rows that the last block lacks, where the workspace has room for one)
    const int zero_rows = need_panel && rows % BN != 0 && plan.off_panel + (size_t)(rows + 1) * (size_t)plan.lda * sizeof(uint16_t) <= workspace_bytes ? 1 : 0;
    // a2 (+ a3 when the panel is used)
    LL_CHECK_F(mark());
    if (need_panel) {
      launch_norm_panel(h_rows, static_cast<const uint16_t*>(gamma), panel, rows, zero_rows, d, plan.lda, eps, bound, bounds, stream);
      LL_CHECK_F(hipGetLastError());
    } else if (!dma && has_gamma) {
      hipLaunchKernelGGL(ll_rms_stats_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, stream, h_rows, (int64_t)rows, d,
                         eps, inv_rms + r0);
      LL_CHECK_F(hipGetLastError());
    }
    GemmArgs a;
    a.A = need_panel ? panel : h_rows;
    a.lda = need_panel ? plan.lda : d;
    a.inv_rms = (!dma && has_gamma) ? inv_rms + r0 : nullptr;
    a.gamma = static_cast<const uint16_t*>(gamma);
    a.W = static_cast<const uint16_t*>(W_U);
    a.target = target_ids ? target_ids + r0 : nullptr;
    a.bias = bias_padded;
    a.stats = stats;
    a.top = top;
    a.rows = rows;
    a.last_row = rows - 1 + zero_rows;
    a.d = d;
    a.V = V;
    a.k = k;
    a.splits = splits;
    a.tiles = tiles;
    a.row_blocks = row_blocks;
    a.group_rows = group_rows(row_blocks, splits);
    a.bound = bound;
    a.classes = l.classes;
    a.half_tiles = l.half_tiles;
    const int grid = (row_blocks * splits + NUM_XCD - 1) / NUM_XCD * NUM_XCD;
    LL_CHECK_F(mark());
    hipLaunchKernelGGL(l.half_tiles > 0 || l.classes > 0 ? short_kern : kern, dim3(grid), dim3(NTHREADS), lds, stream, a);
    LL_CHECK_F(hipGetLastError());
    LL_CHECK_F(mark());
    if (splits <= MAX_SPLITS)
      hipLaunchKernelGGL(ll_merge_kernel<1>, dim3((rows + 3) / 4), dim3(256), (size_t)4 * splits * k * sizeof(uint2), stream,
                         (const float4*)stats, (const uint2*)top,
                         rows, splits, k, V, (flags & LL_FLAG_TOPK_SOFTMAX) ? 1 : 0, a.target, out_topk_ids + r0 * k,
                         out_topk_p + r0 * k,
                         out_target_logp ? out_target_logp + r0 : nullptr, out_entropy + r0, bound, bounds);
    else   // (only passes of at most three row blocks get here: one row per block keeps the lists within 64 KB of LDS)
      hipLaunchKernelGGL(ll_merge_kernel<MERGE_LPL>, dim3(rows), dim3(256), (size_t)splits * k * sizeof(uint2), stream,
                         (const float4*)stats, (const uint2*)top,
                         rows, splits, k, V, (flags & LL_FLAG_TOPK_SOFTMAX) ? 1 : 0, a.target, out_topk_ids + r0 * k,
                         out_topk_p + r0 * k,
                         out_target_logp ? out_target_logp + r0 : nullptr, out_entropy + r0, bound, bounds);
    LL_CHECK_F(hipGetLastError());
    LL_CHECK_F(mark());
  }
#undef LL_CHECK_F
  return finish(read_phases());
}

struct SweepPlan {
  size_t off_u, off_block_max, off_sampled, off_row_sq, off_eu, off_shift, off_shift_min, off_shift_tile, off_general, off_left_z, off_left_id, off_bound, off_stats, off_ztgt, off_top, off_panel, total;
  size_t off_project, wanted;   // the projection's workspace where one alpha is left to it; wanted: what the call is fastest with
  int64_t lda;
  int n_padded;   // V in whole tiles
  int flags;      // whole: FLAGS, and the counts of what is left out
};

// Vocabulary splits of a pass: one workgroup per compute unit, and ids within a split in 16 bits.
int sweep_splits(int rows, int tiles, int block_rows = BN) {
  const int row_blocks = (rows + block_rows - 1) / block_rows;
  const int splits = even_splits(tiles, NUM_CU / row_blocks);
  const int least = (tiles + SWEEP_MAX_TILES - 1) / SWEEP_MAX_TILES;
  return splits > least ? splits : least;
}

// whole: of a call whose kernel forms u itself (no tables; the direction's rows behind the panel; left_slots as in GemmArgs).  Callers bring the
// other's size.
SweepPlan make_sweep_plan(const ll_shape* s, int n_alpha, int k = 1, bool whole = false, int left_slots = 0) {
  SweepPlan p = {};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off = align_up(off + bytes, 256);
    return at;
  };
  const int tiles = (s->V + BM - 1) / BM;
  p.n_padded = tiles * BM;
  const size_t rows = (size_t)(s->N < CHUNK_ROWS ? s->N : CHUNK_ROWS);
  // rows x splits of a full pass and of a shorter last one
  size_t partials = rows * NUM_CU < (size_t)MAX_PARTIALS ? rows * NUM_CU : (size_t)MAX_PARTIALS;
  const size_t least = rows * ((tiles + SWEEP_MAX_TILES - 1) / SWEEP_MAX_TILES);
  if (partials < least) partials = least;
  if (whole) partials = rows * sweep_splits((int)rows, tiles, SWEEP_OWN_ROWS);   // (one pass)
  p.off_u = take((size_t)p.n_padded * sizeof(float));
  p.off_block_max = take(UD_BLOCKS * sizeof(float));
  p.off_project = off;
  if (whole) {
    p.off_sampled = take((SWEEP_SAMPLED + 1) * sizeof(float));
    p.off_row_sq = take((rows + 3) * sizeof(float));
    const size_t blocks = (rows + SWEEP_OWN_ROWS - 1) / SWEEP_OWN_ROWS * (partials / rows);
    p.flags = FLAGS + 4 * (int)blocks;
    p.off_left_z = take(partials * left_slots * sizeof(float));
    p.off_left_id = take(blocks * left_slots * sizeof(int));
  } else {
    p.off_eu = take((size_t)p.n_padded * 2 * SWEEP_ROWS * sizeof(float));
    p.off_shift = take((size_t)p.n_padded * sizeof(float));
    p.off_shift_min = take((size_t)p.n_padded * sizeof(float));
    p.off_shift_tile = take((size_t)tiles * 16 * sizeof(float));
  }
  p.off_general = take((whole ? p.flags : 1) * sizeof(int));
  p.off_bound = take(rows * n_alpha * k * sizeof(unsigned));
  p.off_stats = take(partials * n_alpha * sizeof(float4));
  p.off_ztgt = take(partials * sizeof(float));
  p.off_top = take(partials * n_alpha * (k > 1 ? SWEEP_KS : 1) * sizeof(uint2));
  p.lda = ((int64_t)s->d + DK - 1) / DK * DK;
  p.off_panel = take((rows + 1 + (whole ? SWEEP_PARTS : 0)) * (size_t)p.lda * sizeof(uint16_t));
  p.total = p.wanted = off;
  if (n_alpha == 1 && !whole) {
    const Plan project = make_plan(s, k);
    if (p.off_project + project.roomy > p.total) p.total = p.off_project + project.roomy;
    p.wanted = p.off_project + wanted_bytes(project);
    if (p.wanted < p.total) p.wanted = p.total;
  }
  return p;
}

// The direction kernel keeps v in LDS: 4 d bytes of the 160 KB.
constexpr int SWEEP_MAX_D = 40960;

bool sweep_shape_ok(const ll_shape* s, int n_alpha, int k = 1) {
  return shape_ok(s, k) && k <= SWEEP_KS && s->d <= SWEEP_MAX_D && n_alpha >= 1 && n_alpha <= SWEEP_MAX;
}

int sweep_impl(const ll_shape* shape, void* workspace, size_t workspace_bytes, const void* hidden, const void* gamma,
               const void* W_U, float eps, const float* v, const float* alphas, int n_alpha, int k, const int32_t* target_ids,
               int32_t* out_ids, float* out_p, float* out_logp, float* out_entropy, hipStream_t stream) {
  if (!sweep_shape_ok(shape, n_alpha, k)) return LL_EINVAL;
  if (shape->N == 0) return LL_OK;
  if (hidden == nullptr || W_U == nullptr || v == nullptr || alphas == nullptr || out_ids == nullptr || out_p == nullptr ||
      out_entropy == nullptr)
    return LL_EINVAL;
  if (target_ids != nullptr && out_logp == nullptr) return LL_EINVAL;
  if (!(eps >= 0.f)) return LL_EINVAL;
  if (((uintptr_t)hidden | (uintptr_t)W_U | (uintptr_t)gamma | (uintptr_t)v) & 15) return LL_EINVAL;
  AlphaList al;
  for (int a = 0; a < SWEEP_MAX; ++a) {
    al.a[a] = a < n_alpha ? alphas[a] : 0.f;
    if (!(al.a[a] == al.a[a]) || al.a[a] - al.a[a] != 0.f) return LL_EINVAL;   // NaN or infinite
  }
  SweepPlan plan = make_sweep_plan(shape, n_alpha, k);
  if (workspace == nullptr || workspace_bytes < plan.total || ((uintptr_t)workspace & 255)) return LL_EWORKSPACE;

  const int64_t N = shape->N;
  const int d = shape->d, V = shape->V;
  const int tiles = (V + BM - 1) / BM;
#define LL_CHECK_S(expr)                           \
  do {                                             \
    hipError_t e__ = (expr);                       \
    if (e__ != hipSuccess) return hip_failed(e__); \
  } while (0)

  const int first_rows = (int)(N < CHUNK_ROWS ? N : CHUNK_ROWS), first_splits = sweep_splits(first_rows, tiles);
  const int each = (tiles + first_splits - 1) / first_splits;
  // One strength is a projection whose bias is alpha u.  That is the faster call for lists, for few rows and for many tiles a split; the arg
  // max alone over few tiles costs less than the copy of the bias and the longer list.  Whole calls, projection | the sweep's own
  // kernel, us, d = 256 (N x V: tiles a split), arg max: 300 x 20000 (1) 39 | 34, 700 x 20000 (1) 43 | 34, 1500 x 4096 (1) 31 | 32, 300 x
  // 50257 (2) 60 | 53, 700 x 50257 (3) 69 | 68, 4000 x 20000 (5) 91 | 98, 4000 x 50257 (13) 181 | 217; lists of two: 300 x 20000 40 | 43,
  // 1500 x 4096 30 | 42, 300 x 50257 58 | 66, 700 x 50257 71 | 83, 4000 x 50257 185 | 254.
  const bool as_projection = n_alpha == 1 && (N <= FEW_ROWS || k > 1 || each > 4);
  // Few alphas: the general form alone, without the tables and the launch that fills them.  Its cost grows with every alpha, the
  // factored one's hardly does: the line moves up where a split has few tiles and there are no lists, and where the contraction is
  // short (what the factored form adds to it is the same, and the smaller share of the call).  Whole calls, general | factored, us
  // (N x V: tiles a split), arg max:
  //   d = 512:   300 x 20000 (1)   A = 7  75 | 80      A = 8  80 | 81        1500 x 4096 (1)     A = 7  76 | 86     A = 8  83 | 87
  //              300 x 50257 (2)   A = 5  107 | 120    A = 6  118 | 120      700 x 50257 (3)     A = 4  129 | 146   A = 5  146 | 149
  //              1500 x 50257 (5)  A = 4  204 | 221    A = 5  231 | 221      1500 x 80000 (8)    A = 4  305 | 307   A = 5  345 | 311
  //              1500 x 100000 (10)  A = 3  325 | 363  A = 4  374 | 367      4000 x 128256 (32)  A = 4  1043 | 977
  //   d = 128:   300 x 50257 (2)   A = 6  103 | 119    A = 7  114 | 117      700 x 50257 (3)     A = 5  124 | 143   A = 6  141 | 144
  //              1500 x 50257 (5)  A = 5  189 | 204    A = 6  215 | 204      1500 x 100000 (10)  A = 4  291 | 321   A = 5  341 | 329
  //   d = 2048:  300 x 50257 (2)   A = 5  178 | 177    A = 6  189 | 180      1500 x 80000 (8)    A = 4  592 | 575
  // and lists of three:
  //   d = 512:   300 x 50257 (2)   A = 3  121 | 133    A = 4  143 | 134      4000 x 128256 (32)  A = 3  1098 | 1152   A = 4  1291 | 1162
  //   d = 128:   300 x 50257 (2)   A = 4  128 | 129                          4000 x 128256 (32)  A = 3  865 | 1042    A = 4  1063 | 1053
  //   d = 2048:  300 x 50257 (2)   A = 3  192 | 193                          4000 x 128256 (32)  A = 3  2058 | 2028
  //   d = 64, A = 4, general over factored, lists of two and four: 60 x 20000 (1) 0.95, 0.90; 1500 x 50257 (5) 0.95, 0.90; 4000 x 50257 (13) 0.97, 0.91
  const bool lists = k > 1;
  const int most_general = lists ? (d <= 64 ? 4 : 3) : (each > 8 ? 3 : each > 2 ? 4 : each == 2 ? 5 : 7) + (d <= 256 ? 1 : 0);
  const bool only_general = n_alpha <= most_general;
  int zero_alpha = -1;   // of nine alphas one that is zero needs no place in the tables
  for (int a = 0; a < n_alpha; ++a)
    if (n_alpha > SWEEP_SPLIT_ROWS && al.a[a] == 0.f) zero_alpha = a;
  // Forming u in the contraction's own kernel saves the read of W_U before it (and the tables' kernel), takes three rows of every block, which
  // mostly are to spare, and time in every tile: 0.4 us in the general form, 2.6 in the factored one, whose wavefronts exchange parts
  // of u and tables and wait for each other four times.  So it is for calls of few tiles a workgroup on a large W_U, and never where the three rows give the
  // busiest workgroup a tile more: whether W_U is read all the same is only known on the device (see sweep_is_long; 256 rows, d = 5120, V = 148853, two
  // strengths, five tiles instead of three, u before | within: 648 | 591 us beside a short direction, but 628 | 786 beside a long one).  Whole calls, u before | u within, us, nine strengths, arg max (N x d x V: tiles a workgroup): 250 x 2048 x
  // 50257 (1) 133 | 98, 700 x 1024 x 50257 (3) 181 | 163, 1500 x 2048 x 50257 (5) 380 | 343, 1500 x 4096 x 128256 (12) 1386 | 1233, 4000 x 1024 x 50257 (13)
  // 602 | 614, 8000 x 2560 x 151936 (75) 5370 | 5440; lists of three: 500 x 2560 x 151936 (5) 549 | 439, 4000 x 512 x 128256 (34) 1267 | 1306; three strengths:
  // 1500 x 512 x 50257 (5) 169 | 160, 500 x 2560 x 151936 (5) 503 | 391.  A W_U of up to 64 MiB is read from the Infinity Cache
  // in some 10 us; the factored form then gains little (300 x 512 x 50257 (2) 121 | 115, 1500 x 512 x 50257 (5) 229 | 230) and keeps the kernels before it.
  // Beside a long direction, whose W_U the direction kernel reads all the same, u before | within (alpha v a quarter of the rows' length or more): nine strengths 1500 x 4096 x
  // 128256 1499 | 1466, 500 x 2560 x 151936, lists, 604 | 605, 250 x 2048 x 50257, lists, 164 | 164, 700 x 1024 x 50257 196 | 198; three 1200 x 4096 x 100000 997 | 958; seven 137 x 1792 x
  // 27710 101.8 | 103.0, 667 x 1792 x 9538 98.2 | 100.8 (short: 101.2 | 86.1 and 98.0 | 91.2); four 30 x 640 x 60000 66.2 | 67.6 (66.1 | 52.9).
  bool whole = !as_projection && N <= CHUNK_ROWS && (only_general || ((n_alpha <= SWEEP_SPLIT_ROWS || zero_alpha >= 0) && (int64_t)V * d * 2 > (64 << 20)));
  int left_slots = 0;
  if (whole) {
    const int own_splits = sweep_splits((int)N, tiles, SWEEP_OWN_ROWS);
    const int own_each = (tiles + own_splits - 1) / own_splits;
    const float more_us = (float)own_each * (only_general ? 0.4f : 2.6f);
    // (the tables' place takes some 32 tokens a split and row; few where the vocabulary is small beside the rows)
    left_slots = only_general ? 0 : 32;
    SweepPlan own = make_sweep_plan(shape, n_alpha, k, true, left_slots);
    for (; left_slots > 0 && own.total > plan.total; own = make_sweep_plan(shape, n_alpha, k, true, left_slots)) left_slots /= 2;
    whole = own_each <= each && more_us <= (float)V * (float)d * 2.0f / 6.0e6f + 5.0f && own.total <= plan.total;
    if (whole) plan = own;
  }

  unsigned char* ws = static_cast<unsigned char*>(workspace);
  float* const u = reinterpret_cast<float*>(ws + plan.off_u);
  float* eu = reinterpret_cast<float*>(ws + plan.off_eu);
  float* shift_max = reinterpret_cast<float*>(ws + plan.off_shift);
  float* shift_min = reinterpret_cast<float*>(ws + plan.off_shift_min);
  float* shift_tile = reinterpret_cast<float*>(ws + plan.off_shift_tile);
  float* block_max = reinterpret_cast<float*>(ws + plan.off_block_max);
  float* const sampled = reinterpret_cast<float*>(ws + plan.off_sampled);
  float* const row_sq = reinterpret_cast<float*>(ws + plan.off_row_sq);
  int* general = reinterpret_cast<int*>(ws + plan.off_general);
  float* const left_z = reinterpret_cast<float*>(ws + plan.off_left_z);
  int* const left_id = reinterpret_cast<int*>(ws + plan.off_left_id);
  unsigned* bound = reinterpret_cast<unsigned*>(ws + plan.off_bound);
  float4* stats = reinterpret_cast<float4*>(ws + plan.off_stats);
  float* ztgt = reinterpret_cast<float*>(ws + plan.off_ztgt);
  uint2* top = reinterpret_cast<uint2*>(ws + plan.off_top);
  uint16_t* panel = reinterpret_cast<uint16_t*>(ws + plan.off_panel);
  const auto direction = (int64_t)V * d * 2 >= INFINITY_CACHE_BYTES ? ll_unembed_direction_kernel<true> : ll_unembed_direction_kernel<false>;
  const size_t v_bytes = (size_t)d * sizeof(float);
  if (v_bytes > 64 * 1024)
    if (const int rc = allow_dynamic_lds(reinterpret_cast<const void*>(direction), (size_t)SWEEP_MAX_D * sizeof(float)); rc != LL_OK) return rc;
  if (!whole) {
    hipLaunchKernelGGL(direction, dim3(UD_BLOCKS), dim3(256), v_bytes, stream, static_cast<const uint16_t*>(W_U), v, V, d,
                       as_projection ? al.a[0] : 1.0f, u, plan.n_padded, block_max, (const float*)nullptr, (const float*)nullptr, 0, false, (int*)nullptr);
    LL_CHECK_S(hipGetLastError());
  }
  // (The few-rows kernel then reads W_U through the caches where the direction kernel has just left it in the Infinity Cache, with room
  // for what else is there; a W_U that the L2s hold together is left in them as that kernel has dealt it, for the next sweep's.  Whole
  // calls, past the caches | through them, us, 8 rows (d, V, MB): 2560, 4096, 21: 42.1 | 45.1; 2560, 8192, 42: 50.8 | 46.2; 4096, 8192, 67:
  // 72.7 | 68.8; 1024, 50257, 103: 54.2 | 49.3; 256, 128256, 66: no difference.)
  const bool W_in_cache = d >= 512 && (int64_t)V * d * 2 > L2_BYTES && (int64_t)V * d * 2 <= INFINITY_CACHE_BYTES / 2;
  if (as_projection)
    return project_impl(shape, ws + plan.off_project, workspace_bytes - plan.off_project, hidden, gamma, W_U, u, 0u, eps, k, target_ids, out_ids,
                        out_p, out_logp, out_entropy, stream, nullptr, CHUNK_ROWS, false, W_in_cache ? 1 : 0);
  if (!only_general && !whole) {
    const int n_bound = (int)(N < CHUNK_ROWS ? N : CHUNK_ROWS) * n_alpha * k;
    hipLaunchKernelGGL(ll_sweep_table_kernel, dim3(plan.n_padded / 256 < 2048 ? plan.n_padded / 256 : 2048), dim3(256), 0, stream,
                       (const float*)block_max, UD_BLOCKS, plan.n_padded, al, n_alpha, zero_alpha, (const float*)u, eu, shift_max,
                       shift_min, shift_tile, general, bound, n_bound);
    LL_CHECK_S(hipGetLastError());
  }
  // (d is at most SWEEP_MAX_D: the direct-to-LDS kernel's 32-bit row offsets always suffice)  Of two kernels one returns at once; where
  // they form u themselves the general one comes last, for the shifts that only then turn out too large.
  const GemmKernel general_kernel = whole ? whole_sweep_kernel(lists, true, true) : general_sweep_kernel(lists);
  const GemmKernel factored_kernel = only_general  ? nullptr
                                     : whole       ? whole_sweep_kernel(lists, false, d % DK != 0)
                                     : d % DK != 0 ? tail_sweep_kernel(lists)
                                     : lists       ? ll_lens_gemm_dma_kernel<SweepEpilogue<SWEEP_KS, false>>
                                                   : ll_lens_gemm_dma_kernel<SweepEpilogue<1, false>>;
  const GemmKernel kern[2] = {whole ? factored_kernel : general_kernel, whole ? general_kernel : factored_kernel};
  const size_t lds = (size_t)SLOTS * SLOT_BYTES;
  for (const GemmKernel g : kern)
    if (g != nullptr)
      if (const int rc = allow_dynamic_lds(reinterpret_cast<const void*>(g), lds); rc != LL_OK) return rc;

  // One vocabulary row in 32, up to 2048: of Gaussian shifts the sample's largest is then mostly within a quarter of the largest.
  const int samples = V < 32 * SAMPLE_ROWS * SWEEP_SAMPLED ? (V + 31) / 32 : SAMPLE_ROWS * SWEEP_SAMPLED;
  const int sample_waves = only_general ? 0 : SWEEP_SAMPLED;
  float alpha_most = 0.f;
  for (int a = 0; a < n_alpha; ++a) alpha_most = fmaxf(alpha_most, fabsf(al.a[a]));
  for (int64_t r0 = 0; r0 < N; r0 += CHUNK_ROWS) {
    const int rows = (int)((N - r0 < CHUNK_ROWS) ? (N - r0) : CHUNK_ROWS);
    const uint16_t* h_rows = static_cast<const uint16_t*>(hidden) + r0 * d;
    const bool need_panel = gamma != nullptr || plan.lda != d || whole;
    if (whole) {
      launch_sweep_panel(h_rows, static_cast<const uint16_t*>(gamma), panel, rows, d, plan.lda, eps, bound, only_general ? 0 : n_alpha * k,
                         static_cast<const uint16_t*>(W_U), V, v, alpha_most, sample_waves, samples, sampled, row_sq, general, plan.flags, stream);
      LL_CHECK_S(hipGetLastError());
      hipLaunchKernelGGL(direction, dim3(UD_BLOCKS), dim3(256), v_bytes, stream, static_cast<const uint16_t*>(W_U), v, V, d, 1.0f, u, plan.n_padded,
                         block_max, (const float*)sampled, (const float*)row_sq, rows, only_general, general + FLAG_GIVEN);
      LL_CHECK_S(hipGetLastError());
    } else if (need_panel) {
      launch_norm_panel(h_rows, static_cast<const uint16_t*>(gamma), panel, rows, 1, d, plan.lda, eps, nullptr, 0, stream);
      LL_CHECK_S(hipGetLastError());
    }
    GemmArgs a = {};
    a.A = need_panel ? panel : h_rows;
    a.lda = plan.lda;
    a.W = static_cast<const uint16_t*>(W_U);
    a.target = target_ids ? target_ids + r0 : nullptr;
    a.rows = rows;
    a.last_row = need_panel ? rows : rows - 1;
    a.d = d;
    a.V = V;
    a.k = k;
    a.tiles = tiles;
    const int block_rows = whole ? SWEEP_OWN_ROWS : BN;
    a.row_blocks = (rows + block_rows - 1) / block_rows;
    a.splits = sweep_splits(rows, tiles, block_rows);
    a.group_rows = group_rows(a.row_blocks, a.splits);
    a.u = a.u_out = u;
    a.direction = v;
    a.exceeded = general + FLAG_EXCEEDED;
    a.left_any = general + FLAG_LEFT;
    a.left_n = general + FLAGS;
    a.left_z = left_z;
    a.left_id = left_id;
    a.left_slots = left_slots;
    a.sampled = sampled;
    a.given = general + FLAG_GIVEN;
    a.only_general = only_general ? 1 : 0;
    a.block_max = block_max;
    a.alpha_most = alpha_most;
    a.eu = eu;
    a.shift_max = shift_max;
    a.shift_min = shift_min;
    a.shift_tile = shift_tile;
    a.sweep_general = only_general ? nullptr : general;
    a.sweep_stats = stats;
    a.sweep_ztgt = ztgt;
    a.sweep_top = top;
    a.bound = bound;
    a.n_alpha = n_alpha;
    a.zero_alpha = zero_alpha;
    for (int i = 0; i < SWEEP_MAX; ++i) a.alphas[i] = al.a[i];
    const int64_t blocks = ((int64_t)a.row_blocks * a.splits + NUM_XCD - 1) / NUM_XCD * NUM_XCD;
    for (const GemmKernel g : kern) {
      if (g == nullptr) continue;
      hipLaunchKernelGGL(g, dim3((unsigned)blocks), dim3(NTHREADS), lds, stream, a);
      LL_CHECK_S(hipGetLastError());
    }
    const auto merge = lists ? ll_sweep_merge_kernel<SWEEP_KS> : ll_sweep_merge_kernel<1>;
    hipLaunchKernelGGL(merge, dim3((unsigned)((rows * n_alpha + 3) / 4)), dim3(256), 0, stream, (const float4*)stats, (const uint2*)top,
                       (const float*)ztgt, (const float*)u, al, rows, a.splits, n_alpha, k, V, a.target, N, out_ids + r0 * k,
                       out_p + r0 * k, out_logp ? out_logp + r0 : nullptr, out_entropy + r0, only_general ? nullptr : bound,
                       LeftOut{whole && !only_general ? general : nullptr, left_z, left_id, left_slots});
    LL_CHECK_S(hipGetLastError());
  }
#undef LL_CHECK_S
  return LL_OK;
}

// ---------------------------------------------------------------------------------------
// Allocation-free variant: the workspace of ll_project in a device array of this library, for
// callers that cannot allocate.  The array's name is a host-side handle, not a device address:
// its address on the current device is looked up once per device and only that pointer is used
// from then on.  inv_rms, the partials, the lists and the panel are each written before they are
// read; the shared top-k bounds of the direct-to-LDS kernel, which have to start at zero, are cleared
// in every pass by the panel kernel, or where the rows are read in place by a fill kernel for the first
// pass and by each pass's merge for the next (the few-rows and the register-staged kernel have none):
// stale contents of an earlier call do not matter.
// ---------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char ll_static_scratch[LL_STATIC_SCRATCH_BYTES];
constexpr int MAX_DEVICES = 64;
std::atomic<void*> g_static_scratch_ptr[MAX_DEVICES];

int static_scratch_of_current_device(void** out) {
  int dev = -1;
  LL_HIP_CHECK(hipGetDevice(&dev));
  if (dev < 0 || dev >= MAX_DEVICES) return LL_EINVAL;
  void* ptr = g_static_scratch_ptr[dev].load(std::memory_order_acquire);
  if (ptr == nullptr) {
    LL_HIP_CHECK(hipGetSymbolAddress(&ptr, HIP_SYMBOL(ll_static_scratch)));
    if (ptr == nullptr || ((uintptr_t)ptr & 255)) return LL_EHIP;
    g_static_scratch_ptr[dev].store(ptr, std::memory_order_release);   // the same address whoever gets here first
  }
  *out = ptr;
  return LL_OK;
}

// Rows per pass for the static buffer: the usual 8192 when the plan fits, else the largest
// multiple of the row block that does; 0 when not even one row block fits.
int static_chunk_rows(const ll_shape* s, int k) {
  for (int rows = CHUNK_ROWS; rows >= BN; rows -= BN)
    if (make_plan(s, k, rows).total <= (size_t)LL_STATIC_SCRATCH_BYTES) return rows;
  return 0;
}

}  // namespace

extern "C" {

int ll_project_static(const ll_shape* shape, const void* hidden, const void* gamma, const void* W_U, float eps, int k,
                      const int32_t* target_ids, int32_t* out_topk_ids, float* out_topk_p, float* out_target_logp,
                      float* out_entropy, void* stream) {
  if (!shape_ok(shape, k)) return LL_EINVAL;
  if (shape->N == 0) return LL_OK;
  const int chunk = static_chunk_rows(shape, k);
  if (chunk == 0) return LL_ESCRATCH;
  void* ws = nullptr;
  if (const int rc = static_scratch_of_current_device(&ws); rc != LL_OK) return rc;
  return project_impl(shape, ws, (size_t)LL_STATIC_SCRATCH_BYTES, hidden, gamma, W_U, nullptr, 0u, eps, k, target_ids,
                      out_topk_ids, out_topk_p, out_target_logp, out_entropy, static_cast<hipStream_t>(stream), nullptr, chunk, true);
}

int64_t ll_project_static_pass_rows(const ll_shape* shape, int k) {
  if (!shape_ok(shape, k)) return 0;
  return static_chunk_rows(shape, k);
}

size_t ll_steer_sweep_workspace_bytes(const ll_shape* shape, int n_alpha) {
  if (!sweep_shape_ok(shape, n_alpha)) return 0;
  return make_sweep_plan(shape, n_alpha).wanted;
}

size_t ll_steer_sweep_topk_workspace_bytes(const ll_shape* shape, int n_alpha, int k) {
  if (!sweep_shape_ok(shape, n_alpha, k)) return 0;
  return make_sweep_plan(shape, n_alpha, k).wanted;
}

int ll_steer_sweep_topk(const ll_shape* shape, void* workspace, size_t workspace_bytes, const void* hidden, const void* gamma,
                        const void* W_U, float eps, const float* v, const float* alphas, int n_alpha, int k,
                        const int32_t* target_ids, int32_t* out_topk_ids, float* out_topk_p, float* out_target_logp,
                        float* out_entropy, void* stream) {
  return sweep_impl(shape, workspace, workspace_bytes, hidden, gamma, W_U, eps, v, alphas, n_alpha, k, target_ids, out_topk_ids,
                    out_topk_p, out_target_logp, out_entropy, static_cast<hipStream_t>(stream));
}

int ll_steer_sweep(const ll_shape* shape, void* workspace, size_t workspace_bytes, const void* hidden, const void* gamma,
                   const void* W_U, float eps, const float* v, const float* alphas, int n_alpha, const int32_t* target_ids,
                   int32_t* out_top1_ids, float* out_top1_p, float* out_target_logp, float* out_entropy, void* stream) {
  return sweep_impl(shape, workspace, workspace_bytes, hidden, gamma, W_U, eps, v, alphas, n_alpha, 1, target_ids, out_top1_ids,
                    out_top1_p, out_target_logp, out_entropy, static_cast<hipStream_t>(stream));
}

size_t ll_workspace_bytes(const ll_shape* shape, int k) {
  if (!shape_ok(shape, k)) return 0;
  if (shape->N == 0) return 256;
  return wanted_bytes(make_plan(shape, k));
}

int ll_project(const ll_shape* shape, void* workspace, size_t workspace_bytes, const void* hidden, const void* gamma,
               const void* W_U, float eps, int k, const int32_t* target_ids, int32_t* out_topk_ids, float* out_topk_p,
               float* out_target_logp, float* out_entropy, void* stream) {
  return project_impl(shape, workspace, workspace_bytes, hidden, gamma, W_U, nullptr, 0u, eps, k, target_ids, out_topk_ids,
                      out_topk_p, out_target_logp, out_entropy, static_cast<hipStream_t>(stream), nullptr);
}

int ll_project_ex(const ll_shape* shape, void* workspace, size_t workspace_bytes, const void* hidden, const void* gamma,
                  const void* W_U, const float* bias, unsigned flags, float eps, int k, const int32_t* target_ids,
                  int32_t* out_topk_ids, float* out_topk_p, float* out_target_logp, float* out_entropy, void* stream) {
  return project_impl(shape, workspace, workspace_bytes, hidden, gamma, W_U, bias, flags, eps, k, target_ids, out_topk_ids,
                      out_topk_p, out_target_logp, out_entropy, static_cast<hipStream_t>(stream), nullptr);
}

int ll_project_timed(const ll_shape* shape, void* workspace, size_t workspace_bytes, const void* hidden, const void* gamma,
                     const void* W_U, float eps, int k, const int32_t* target_ids, int32_t* out_topk_ids, float* out_topk_p,
                     float* out_target_logp, float* out_entropy, void* stream, float* phase_ms) {
  if (phase_ms == nullptr) return LL_EINVAL;
  return project_impl(shape, workspace, workspace_bytes, hidden, gamma, W_U, nullptr, 0u, eps, k, target_ids, out_topk_ids,
                      out_topk_p, out_target_logp, out_entropy, static_cast<hipStream_t>(stream), phase_ms);
}

}  // extern "C"
