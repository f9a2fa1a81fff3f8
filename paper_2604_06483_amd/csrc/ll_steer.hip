// Steering direction (paper Sec. 3.4, Eq. 2) and post-norm injection (Eq. 3) for gfx950.
// Both are bandwidth-bound: 16-byte loads, fp32 arithmetic, no atomics.
#include "ll_common.h"

#include <math.h>

namespace {

using namespace ll;

// ---------------------------------------------------------------------------------------
// Column sums.  Block (x, y): columns [64 x, 64 x + 64), row slice y.  A wavefront's load takes 128 bytes of eight rows,
// and both sets' next four loads are in flight together, so that what bounds the usual call (some hundred rows) is one trip
// to memory on as many CUs as there are column blocks.  One slice: writes mean(target) - mean(base) to `out` and the
// block's sum of squares to sq (unless null); several: the two partial sums to out[2][slices][d].
// Whole direction, normalised, d = 8192, before (512 columns a block, one workgroup that summed, normalised and scaled) | now:
// 64 + 64 rows 15.4 | 5.8 us, 400 + 600 rows 22 | 8.2 us, 4000 + 4000 rows 45 | 28 us, 32768 + 32768 rows 215 | 197 us (5.4 TB/s).
// ---------------------------------------------------------------------------------------
constexpr int SUM_COLS = 64;
constexpr int SUM_ROWS = 32;           // rows a workgroup loads at a time
constexpr int SUM_LOADS = 4;           // times in flight
constexpr int STEER_SLICES = 60;       // most slices of the rows
constexpr double STREAM_BYTES = 1 << 28;   // rows that the last-level cache (256 MB) can't hold are loaded past it
constexpr int STEER_WS_ROWS = 128;     // workspace, in units of d floats: two partial sums a slice, and the sums of squares

template <bool STREAM>
__device__ __forceinline__ uint4 load_row(const uint16_t* p) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  const u32x4* q = reinterpret_cast<const u32x4*>(p);
  const u32x4 x = STREAM ? __builtin_nontemporal_load(q) : *q;
  return make_uint4(x[0], x[1], x[2], x[3]);
}

// Sum over the lanes that differ in bits 3 to 5.
__device__ __forceinline__ float sum_rows8(float x) {
  const auto add = [](uint32_t a, uint32_t b) { return __float_as_uint(__uint_as_float(a) + __uint_as_float(b)); };
  return __uint_as_float(with_lane_xor<32>(with_lane_xor<16>(with_lane_xor<8>(__float_as_uint(x), add), add), add));
}

template <bool STREAM>
__global__ __launch_bounds__(256) void ll_steer_colsum_kernel(const uint16_t* __restrict__ base, int64_t n_base,
                                                              const uint16_t* __restrict__ target, int64_t n_target,
                                                              int d, int slices, int col_blocks, int neighbours,
                                                              float* __restrict__ out, float* __restrict__ sq) {
  __shared__ float red[2][4][SUM_COLS];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  // (workgroups are dealt round-robin over the 8 XCDs: `neighbours` column blocks in a row on one of them, or 0: as they come)
  const int block = neighbours != 0 ? (int)(blockIdx.x % 8) * neighbours + (int)(blockIdx.x / 8) : (int)blockIdx.x;
  if (block >= col_blocks) return;
  const int col0 = block * SUM_COLS + (lane & 7) * 8;
  const int64_t step = (int64_t)slices * SUM_ROWS;
  const int64_t n_max = n_base > n_target ? n_base : n_target;

  float sum[2][8];
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int i = 0; i < 8; ++i) sum[s][i] = 0.f;

  if (col0 < d) {
    for (int64_t r0 = (int64_t)blockIdx.y * SUM_ROWS + wave * 8 + (lane >> 3); r0 < n_max; r0 += SUM_LOADS * step) {
      uint4 q[2][SUM_LOADS];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const uint16_t* src = (s == 0 ? base : target) + col0;
        const int64_t n = s == 0 ? n_base : n_target;
#pragma unroll
        for (int i = 0; i < SUM_LOADS; ++i) {
          const int64_t r = r0 + i * step;
          q[s][i] = make_uint4(0, 0, 0, 0);
          if (r < n) q[s][i] = load_row<STREAM>(src + r * d);
        }
      }
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < SUM_LOADS; ++i) {
          const uint32_t w[4] = {q[s][i].x, q[s][i].y, q[s][i].z, q[s][i].w};
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            sum[s][2 * j] += bf16_lo(w[j]);
            sum[s][2 * j + 1] += bf16_hi(w[j]);
          }
        }
    }
  }
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      sum[s][i] = sum_rows8(sum[s][i]);
      if (lane < 8) red[s][wave][lane * 8 + i] = sum[s][i];
    }
  __syncthreads();
  if (wave != 0) return;
  const int col = block * SUM_COLS + lane;
  const float sb = (red[0][0][lane] + red[0][1][lane]) + (red[0][2][lane] + red[0][3][lane]);
  const float st = (red[1][0][lane] + red[1][1][lane]) + (red[1][2][lane] + red[1][3][lane]);
  if (slices > 1) {
    if (col < d) {
      out[(int64_t)blockIdx.y * d + col] = sb;
      out[((int64_t)slices + blockIdx.y) * d + col] = st;
    }
    return;
  }
  const float diff = col < d ? st / (float)n_target - sb / (float)n_base : 0.f;
  if (col < d) out[col] = diff;
  if (sq != nullptr) {
    const float ss = wave_sum(diff * diff);
    if (lane == 0) sq[block] = ss;
  }
}

// Several slices: sums them, four at a time, and writes the difference of means and every column block's sum of squares.
__global__ __launch_bounds__(256) void ll_steer_reduce_kernel(const float* __restrict__ part, int slices, int64_t n_base,
                                                              int64_t n_target, int d, float* __restrict__ out_v,
                                                              float* __restrict__ sq) {
  __shared__ float red[2][4][SUM_COLS];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int col = blockIdx.x * SUM_COLS + lane;
  float sb = 0.f, st = 0.f;
  if (col < d) {
#pragma unroll 4
    for (int s = wave; s < slices; s += 4) {
      sb += part[(int64_t)s * d + col];
      st += part[((int64_t)slices + s) * d + col];
    }
  }
  red[0][wave][lane] = sb;
  red[1][wave][lane] = st;
  __syncthreads();
  if (wave != 0) return;
  sb = (red[0][0][lane] + red[0][1][lane]) + (red[0][2][lane] + red[0][3][lane]);
  st = (red[1][0][lane] + red[1][1][lane]) + (red[1][2][lane] + red[1][3][lane]);
  const float diff = col < d ? st / (float)n_target - sb / (float)n_base : 0.f;
  if (col < d) out_v[col] = diff;
  const float ss = wave_sum(diff * diff);
  if (lane == 0) sq[blockIdx.x] = ss;
}

__device__ __forceinline__ float inv_length(float ss) { return ss > 0.f ? 1.0f / sqrtf(ss) : 0.f; }

// L2-normalises v: every workgroup adds the n_sq sums of squares in the same order and scales its 1024 columns.
__global__ __launch_bounds__(256) void ll_steer_scale_kernel(const float* __restrict__ sq, int n_sq, int d, float* __restrict__ out_v) {
  __shared__ float red[4];
  const int c = blockIdx.x * 1024 + threadIdx.x * 4;
  float4 x = c < d ? *reinterpret_cast<const float4*>(out_v + c) : make_float4(0.f, 0.f, 0.f, 0.f);
  float ss = 0.f;
  for (int i = threadIdx.x; i < n_sq; i += 256) ss += sq[i];
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float inv = inv_length((red[0] + red[1]) + (red[2] + red[3]));
  x.x *= inv;
  x.y *= inv;
  x.z *= inv;
  x.w *= inv;
  if (c < d) *reinterpret_cast<float4*>(out_v + c) = x;
}

// The whole direction in one workgroup: few rows of at most 1024 chunks of eight columns, one per thread.
__global__ __launch_bounds__(1024) void ll_steer_small_kernel(const uint16_t* __restrict__ base, int n_base,
                                                              const uint16_t* __restrict__ target, int n_target, int d,
                                                              int normalize, float* __restrict__ out_v) {
  __shared__ float red[16];
  const int col0 = threadIdx.x * 8;
  float sum[2][8], ss = 0.f;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
#pragma unroll
    for (int i = 0; i < 8; ++i) sum[s][i] = 0.f;
    if (col0 < d) {
      const uint16_t* src = (s == 0 ? base : target) + col0;
      const int n = s == 0 ? n_base : n_target;
#pragma unroll 4
      for (int r = 0; r < n; ++r) {
        const uint4 q = *reinterpret_cast<const uint4*>(src + (int64_t)r * d);
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          sum[s][2 * j] += bf16_lo(w[j]);
          sum[s][2 * j + 1] += bf16_hi(w[j]);
        }
      }
    }
  }
  float diff[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    diff[i] = sum[1][i] / (float)n_target - sum[0][i] / (float)n_base;
    ss = fmaf(diff[i], diff[i], ss);
  }
  float inv = 1.0f;
  if (normalize) {
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    float tot = 0.f;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) tot += red[w];
    inv = inv_length(tot);
  }
  if (col0 < d) {
#pragma unroll
    for (int i = 0; i < 8; i += 4)
      *reinterpret_cast<float4*>(out_v + col0 + i) =
          make_float4(diff[i] * inv, diff[i + 1] * inv, diff[i + 2] * inv, diff[i + 3] * inv);
  }
}

// The same without scratch memory for the sums of squares: one workgroup.
__global__ __launch_bounds__(1024) void ll_steer_finish_kernel(int d, float* __restrict__ out_v) {
  __shared__ float red[16];
  float ss = 0.f;
  for (int c = threadIdx.x; c < d; c += 1024) ss = fmaf(out_v[c], out_v[c], ss);
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < 16; ++w) tot += red[w];
  const float inv = inv_length(tot);
  for (int c = threadIdx.x; c < d; c += 1024) out_v[c] *= inv;   // each thread rescales what it read
}

// ---------------------------------------------------------------------------------------
// Injection: out = bf16(gamma * h * inv_rms + alpha * v).  One wavefront per row; the row is
// kept in registers between the statistic and the write when it fits (NITER 16-byte loads per
// lane), otherwise it is read twice.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ uint4 steered(const uint4 q, const uint4 g, const float4 va, const float4 vb, float inv, float alpha) {
  const uint32_t hw[4] = {q.x, q.y, q.z, q.w};
  const uint32_t gw[4] = {g.x, g.y, g.z, g.w};
  const float vv[8] = {va.x, va.y, va.z, va.w, vb.x, vb.y, vb.z, vb.w};
  uint32_t ow[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float lo = fmaf(alpha, vv[2 * i], bf16_lo(hw[i]) * inv * bf16_lo(gw[i]));
    const float hi = fmaf(alpha, vv[2 * i + 1], bf16_hi(hw[i]) * inv * bf16_hi(gw[i]));
    ow[i] = pack_bf16(lo, hi);
  }
  return make_uint4(ow[0], ow[1], ow[2], ow[3]);
}

template <int NITER>
__global__ __launch_bounds__(256) void ll_steer_inject_kernel(const uint16_t* hidden, const uint16_t* __restrict__ gamma,
                                                              const float* __restrict__ v, uint16_t* out, int64_t n_rows,
                                                              int d, float eps, float alpha) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n_rows) return;
  const uint4* src = reinterpret_cast<const uint4*>(hidden + row * (int64_t)d);
  uint4* dst = reinterpret_cast<uint4*>(out + row * (int64_t)d);
  const uint4* g4 = reinterpret_cast<const uint4*>(gamma);
  const float4* v4 = reinterpret_cast<const float4*>(v);
  const int n16 = d >> 3;

  float acc0 = 0.f, acc1 = 0.f;
  uint4 cache[NITER > 0 ? NITER : 1];
  if (NITER > 0) {
#pragma unroll
    for (int it = 0; it < NITER; ++it) {
      const int c = lane + 64 * it;
      if (c < n16) {
        cache[it] = src[c];
        accum_sq(cache[it], acc0, acc1);
      }
    }
  } else {
    for (int c = lane; c < n16; c += 64) accum_sq(src[c], acc0, acc1);
  }
  const float inv = inv_rms_from_sumsq(wave_sum(acc0 + acc1), d, eps);

  auto emit = [&](int c, const uint4 q) { dst[c] = steered(q, g4[c], v4[2 * c], v4[2 * c + 1], inv, alpha); };
  if (NITER > 0) {
#pragma unroll
    for (int it = 0; it < NITER; ++it) {
      const int c = lane + 64 * it;
      if (c < n16) emit(c, cache[it]);
    }
  } else {
    for (int c = lane; c < n16; c += 64) emit(c, src[c]);
  }
}

// The same with one workgroup per row: a few 16-byte loads per thread, gamma's and v's among them, all in flight at once, and
// the rows spread evenly over the chip.  The statistic is summed from LDS, by every wavefront, in the order of the kernel
// above and of the projection's norm, so that all of them have the same bits.
template <int NIT>
__global__ __launch_bounds__(256) void ll_steer_inject_row_kernel(const uint16_t* hidden, const uint16_t* __restrict__ gamma,
                                                                  const float* __restrict__ v, uint16_t* out, int d, float eps,
                                                                  float alpha) {
  __shared__ uint4 shared_row[NIT * 256];
  const int tid = threadIdx.x, lane = tid & 63, threads = blockDim.x;
  const int n16 = d >> 3;
  const uint4* src = reinterpret_cast<const uint4*>(hidden + blockIdx.x * (int64_t)d);
  uint4* dst = reinterpret_cast<uint4*>(out + blockIdx.x * (int64_t)d);
  uint4 h[NIT], g[NIT];
  float4 va[NIT], vb[NIT];
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int c = tid + threads * it;
    h[it] = c < n16 ? src[c] : make_uint4(0, 0, 0, 0);
    shared_row[c] = h[it];
  }
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int c = tid + threads * it < n16 ? tid + threads * it : 0;
    g[it] = reinterpret_cast<const uint4*>(gamma)[c];
    va[it] = reinterpret_cast<const float4*>(v)[2 * c];
    vb[it] = reinterpret_cast<const float4*>(v)[2 * c + 1];
  }
  __syncthreads();
  float acc0 = 0.f, acc1 = 0.f;
#pragma unroll
  for (int it = 0; it < NIT * 4; ++it)
    if (64 * it < n16) accum_sq(shared_row[lane + 64 * it], acc0, acc1);   // (padded with zeros to whole wavefronts)
  const float inv = inv_rms_from_sumsq(wave_sum(acc0 + acc1), d, eps);
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int c = tid + threads * it;
    if (c < n16) dst[c] = steered(h[it], g[it], va[it], vb[it], inv, alpha);
  }
}

// In-model injection with the two safeguards (Sec. 3.4, stability paragraph): out = bf16(h + beta v)
// with beta = s clipped in magnitude to clip_ratio times the row's L2 norm (s = alpha times the
// layer's scale; clip_ratio <= 0: no clipping).  Same shape as the kernel above, without the norm.
template <int NITER>
__global__ __launch_bounds__(256) void ll_steer_inject_raw_kernel(const uint16_t* hidden, const float* __restrict__ v,
                                                                  uint16_t* out, int64_t n_rows, int d, float s,
                                                                  float clip_ratio) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n_rows) return;
  const uint4* src = reinterpret_cast<const uint4*>(hidden + row * (int64_t)d);
  uint4* dst = reinterpret_cast<uint4*>(out + row * (int64_t)d);
  const float4* v4 = reinterpret_cast<const float4*>(v);
  const int n16 = d >> 3;

  float acc0 = 0.f, acc1 = 0.f;
  uint4 cache[NITER > 0 ? NITER : 1];
  if (NITER > 0) {
#pragma unroll
    for (int it = 0; it < NITER; ++it) {
      const int c = lane + 64 * it;
      if (c < n16) {
        cache[it] = src[c];
        accum_sq(cache[it], acc0, acc1);
      }
    }
  } else {
    for (int c = lane; c < n16; c += 64) accum_sq(src[c], acc0, acc1);
  }
  float beta = s;
  if (clip_ratio > 0.f) {
    const float cap = clip_ratio * sqrtf(wave_sum(acc0 + acc1));
    beta = copysignf(fminf(fabsf(s), cap), s);
  }

  auto emit = [&](int c, const uint4 q) {
    const float4 va = v4[2 * c], vb = v4[2 * c + 1];
    const uint32_t hw[4] = {q.x, q.y, q.z, q.w};
    const float vv[8] = {va.x, va.y, va.z, va.w, vb.x, vb.y, vb.z, vb.w};
    uint32_t ow[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      ow[i] = pack_bf16(fmaf(beta, vv[2 * i], bf16_lo(hw[i])), fmaf(beta, vv[2 * i + 1], bf16_hi(hw[i])));
    dst[c] = make_uint4(ow[0], ow[1], ow[2], ow[3]);
  };
  if (NITER > 0) {
#pragma unroll
    for (int it = 0; it < NITER; ++it) {
      const int c = lane + 64 * it;
      if (c < n16) emit(c, cache[it]);
    }
  } else {
    for (int c = lane; c < n16; c += 64) emit(c, src[c]);
  }
}

// one wavefront per row, four rows per workgroup, and the grid's x extent is a 31-bit number
constexpr int64_t kMaxInjectRows = (int64_t)4 * 0x7fffffff;

}  // namespace

extern "C" {

int ll_steer_inject_raw(const ll_shape* shape, const void* hidden, const float* v, float alpha, float layer_scale,
                        float clip_ratio, void* out_hidden, void* stream_) {
  if (shape == nullptr || shape->N < 0 || shape->d <= 0 || (shape->d & 7) != 0) return LL_EINVAL;
  if (shape->N > kMaxInjectRows) return LL_EINVAL;
  if (shape->N == 0) return LL_OK;
  if (hidden == nullptr || v == nullptr || out_hidden == nullptr) return LL_EINVAL;
  const float s = alpha * layer_scale;
  if (s - s != 0.f || clip_ratio - clip_ratio != 0.f) return LL_EINVAL;   // NaN or infinite
  if (((uintptr_t)hidden | (uintptr_t)v | (uintptr_t)out_hidden) & 15) return LL_EINVAL;
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  const int64_t N = shape->N;
  const int d = shape->d;
  const unsigned blocks = (unsigned)((N + 3) / 4);
  const uint16_t* h = static_cast<const uint16_t*>(hidden);
  uint16_t* o = static_cast<uint16_t*>(out_hidden);
  const int n16 = d >> 3;
#define LL_INJECT_RAW(NITER) \
  hipLaunchKernelGGL(ll_steer_inject_raw_kernel<NITER>, dim3(blocks), dim3(256), 0, stream, h, v, o, N, d, s, clip_ratio)
  if (n16 <= 64 * 2) {
    LL_INJECT_RAW(2);
  } else if (n16 <= 64 * 8) {
    LL_INJECT_RAW(8);
  } else if (n16 <= 64 * 16) {
    LL_INJECT_RAW(16);
  } else {
    LL_INJECT_RAW(0);
  }
#undef LL_INJECT_RAW
  LL_HIP_CHECK(hipGetLastError());
  return LL_OK;
}

size_t ll_steer_workspace_bytes(int32_t d) {
  if (d <= 0 || (d & 7) != 0) return 0;
  return (size_t)STEER_WS_ROWS * (size_t)d * sizeof(float);
}

int ll_steer_vector(const void* base, int64_t n_base, const void* target, int64_t n_target, int32_t d, int normalize,
                    float* out_v, void* workspace, size_t workspace_bytes, void* stream_) {
  if (base == nullptr || target == nullptr || out_v == nullptr) return LL_EINVAL;
  if (n_base < 1 || n_target < 1 || d <= 0 || (d & 7) != 0) return LL_EINVAL;
  if (((uintptr_t)base | (uintptr_t)target | (uintptr_t)out_v) & 15) return LL_EINVAL;
  if (workspace != nullptr && (workspace_bytes < ll_steer_workspace_bytes(d) || ((uintptr_t)workspace & 15)))
    return LL_EWORKSPACE;
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  const unsigned col_blocks = (unsigned)(((int64_t)d + SUM_COLS - 1) / SUM_COLS);
  const uint16_t* b = static_cast<const uint16_t*>(base);
  const uint16_t* t = static_cast<const uint16_t*>(target);
  const int64_t n_max = n_base > n_target ? n_base : n_target;
  // (d = 256: 1 + 1 rows 3.1 us, 10 + 16 rows 4.0, against 5.0 to 6 for the two launches below; d = 8192: 4.4 and 6.5 against
  // 6.6 and 6.7, and past 16 rows the one CU's share of the bandwidth is what counts)
  if (n_max <= 16 && d <= 8192) {
    hipLaunchKernelGGL(ll_steer_small_kernel, dim3(1), dim3((unsigned)((d + 511) / 512 * 64)), 0, stream, b, (int)n_base, t,
                       (int)n_target, d, normalize, out_v);
    LL_HIP_CHECK(hipGetLastError());
    return LL_OK;
  }
  float* part = static_cast<float*>(workspace);
  float* sq = workspace == nullptr ? nullptr : part + (size_t)2 * STEER_SLICES * d;
  // a slice for what the workgroup has in flight at once
  int64_t slices = workspace == nullptr ? 1 : (n_max + SUM_ROWS * SUM_LOADS - 1) / (SUM_ROWS * SUM_LOADS);
  if (slices > STEER_SLICES) slices = STEER_SLICES;
  // Rows that are not whole 128-byte lines: two column blocks share lines, so they go past no cache and next to each other on one
  // XCD, whose L2 then has the line for both.  20000 + 20000 rows of d = 8200, with the hint | without | neighbours, us: 190 | 175 | 130
  // (d = 1000, 40000 + 40000: 51 without, 42; d = 264, whose five blocks would leave three XCDs idle: 22, 30).
  const bool whole_lines = ((uintptr_t)base | (uintptr_t)target | (uintptr_t)d * 2) % 128 == 0;
  const bool stream_rows = whole_lines && (double)(n_base + n_target) * d * 2 > STREAM_BYTES;
  const unsigned neighbours = whole_lines || col_blocks < 16 ? 0 : (col_blocks + 7) / 8;
  hipLaunchKernelGGL(stream_rows ? ll_steer_colsum_kernel<true> : ll_steer_colsum_kernel<false>,
                     dim3(neighbours == 0 ? col_blocks : 8 * neighbours, (unsigned)slices), dim3(256), 0, stream, b, n_base, t, n_target, d, (int)slices,
                     (int)col_blocks, (int)neighbours, slices > 1 ? part : out_v, sq);
  LL_HIP_CHECK(hipGetLastError());
  if (slices > 1) {
    hipLaunchKernelGGL(ll_steer_reduce_kernel, dim3(col_blocks), dim3(256), 0, stream, (const float*)part, (int)slices, n_base,
                       n_target, d, out_v, sq);
    LL_HIP_CHECK(hipGetLastError());
  }
  if (!normalize) return LL_OK;
  if (sq != nullptr)
    hipLaunchKernelGGL(ll_steer_scale_kernel, dim3((unsigned)(((int64_t)d + 1023) / 1024)), dim3(256), 0, stream, (const float*)sq,
                       (int)col_blocks, d, out_v);
  else
    hipLaunchKernelGGL(ll_steer_finish_kernel, dim3(1), dim3(1024), 0, stream, d, out_v);
  LL_HIP_CHECK(hipGetLastError());
  return LL_OK;
}

int ll_steer_inject(const ll_shape* shape, const void* hidden, const void* gamma, float eps, const float* v, float alpha,
                    void* out_hidden, void* stream_) {
  if (shape == nullptr || shape->N < 0 || shape->d <= 0 || (shape->d & 7) != 0) return LL_EINVAL;
  if (shape->N > kMaxInjectRows) return LL_EINVAL;
  if (shape->N == 0) return LL_OK;
  if (hidden == nullptr || gamma == nullptr || v == nullptr || out_hidden == nullptr || !(eps >= 0.f)) return LL_EINVAL;
  if (((uintptr_t)hidden | (uintptr_t)gamma | (uintptr_t)v | (uintptr_t)out_hidden) & 15) return LL_EINVAL;
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  const int64_t N = shape->N;
  const int d = shape->d;
  const unsigned blocks = (unsigned)((N + 3) / 4);
  const uint16_t* h = static_cast<const uint16_t*>(hidden);
  const uint16_t* g = static_cast<const uint16_t*>(gamma);
  uint16_t* o = static_cast<uint16_t*>(out_hidden);
  const int n16 = d >> 3;
#define LL_INJECT(NITER) \
  hipLaunchKernelGGL(ll_steer_inject_kernel<NITER>, dim3(blocks), dim3(256), 0, stream, h, g, v, o, N, d, eps, alpha)
#define LL_INJECT_ROW(NIT)                                                                                                    \
  hipLaunchKernelGGL(ll_steer_inject_row_kernel<NIT>, dim3((unsigned)N), dim3((unsigned)((n16 + 64 * NIT - 1) / (64 * NIT) * 64)), \
                     0, stream, h, g, v, o, d, eps, alpha)
  // Up to six rows per CU one wavefront per row leaves the chip half empty and each of them waiting for its own row; with more
  // there are enough of them, and the workgroup's barrier costs more than it gives.  Workgroup | wavefront per row, us:
  //   d = 8192:  64 rows 4.7 | 8.1   1000 rows 8.5 | 11.7   1500 rows 12.0 | 14.8   2048 rows 15.5 | 15.4   4000 rows 25.6 | 22.8
  //   d = 5120:  64 rows 3.8 | 6.0   1000 rows 6.2 | 7.4    1500 rows 8.1 | 9.1     2048 rows 9.9 | 10.3    4000 rows 17.1 | 15.3
  //   d = 2560:  64 rows 3.1 | 4.1   1000 rows 4.3 | 4.8    1500 rows 5.1 | 5.2     2048 rows 5.9 | 5.6     4000 rows 9.4 | 8.9
  // Up to d = 1024 the row is two loads of a wavefront, which has nothing to gain.
  const bool few = N <= 1536;
  if (n16 <= 64 * 2) {
    LL_INJECT(2);
  } else if (few && n16 <= 256) {
    LL_INJECT_ROW(1);
  } else if (few && n16 <= 256 * 2) {
    LL_INJECT_ROW(2);
  } else if (few && n16 <= 256 * 4) {
    LL_INJECT_ROW(4);
  } else if (n16 <= 64 * 8) {
    LL_INJECT(8);
  } else if (n16 <= 64 * 16) {
    LL_INJECT(16);
  } else {
    LL_INJECT(0);
  }
#undef LL_INJECT_ROW
#undef LL_INJECT
  LL_HIP_CHECK(hipGetLastError());
  return LL_OK;
}

}  // extern "C"
