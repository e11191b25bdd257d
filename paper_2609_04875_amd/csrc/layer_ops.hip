// Elementwise steps of a full decoder layer around the projections: RMSNorm
// with a gain, rotary embedding of Q and K at absolute positions, and the
// SiLU-gated product of the MLP.  bf16 in and out, fp32 arithmetic, one
// rounding per stored value.  All three are HBM-bound streams: 16-byte loads
// and stores, fixed reduction order (results do not depend on timing).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "elementwise.h"
#include "internal.h"

namespace pgsr {

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ inline uint32_t pack(float a, float b) { return f32_to_bf16(a) | (f32_to_bf16(b) << 16); }

constexpr int kThreads = 256;

// y = x / sqrt(mean(x^2) + eps) * g, one workgroup per row; d_model % 8 == 0.
__global__ void __launch_bounds__(kThreads) rmsnorm_kernel(int32_t dm, const uint16_t* __restrict__ x,
                                                           const uint16_t* __restrict__ g, float eps,
                                                           uint16_t* __restrict__ y) {
  __shared__ float red[kThreads / 64];
  const int64_t row = blockIdx.x;
  const u32x4* xr = (const u32x4*)(x + row * dm);
  const u32x4* gr = (const u32x4*)g;
  u32x4* yr = (u32x4*)(y + row * dm);
  const int chunks = dm / 8;
  float ss = 0.f;
  for (int c = threadIdx.x; c < chunks; c += kThreads) {
    const u32x4 v = xr[c];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float a = lo_bf16(v[j]), b = hi_bf16(v[j]);
      ss = fmaf(a, a, ss);
      ss = fmaf(b, b, ss);
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) ss += __shfl_xor(ss, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float total = (red[0] + red[1]) + (red[2] + red[3]);
  const float inv = 1.f / sqrtf(total / (float)dm + eps);
  for (int c = threadIdx.x; c < chunks; c += kThreads) {
    const u32x4 v = xr[c], w = gr[c];
    u32x4 o;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      o[j] = pack(lo_bf16(v[j]) * inv * lo_bf16(w[j]), hi_bf16(v[j]) * inv * hi_bf16(w[j]));
    yr[c] = o;
  }
}

// Rotary embedding in place on x [n][heads][d]: for i < d/2 the pair
// (x_i, x_{i+d/2}) turns by pos * theta^(-2i/d).  The angle is formed and
// reduced to [-pi, pi] in fp64 (positions reach 10^5 radians), then sin and
// cos run in fp32 on the reduced angle.
__device__ inline void rope_angle(int32_t pos, int i, int d, double log2_theta, float& s, float& c) {
  const double inv = exp2(-2.0 * i / d * log2_theta);
  const double ang = (double)pos * inv;
  const double two_pi = 6.283185307179586476925287;
  const float r = (float)(ang - two_pi * rint(ang / two_pi));
  sincosf(r, &s, &c);
}
// The fused form is written out, so that every kernel rounds alike.
__device__ inline void rope_turn(float a, float b, float s, float c, uint32_t& x, uint32_t& y) {
  x = f32_to_bf16(fmaf(a, c, -(b * s)));
  y = f32_to_bf16(fmaf(b, c, a * s));
}

// Any even d, any alignment: one pair per thread.
__global__ void __launch_bounds__(kThreads) rope_kernel(int64_t n_pairs, int32_t heads, int32_t d,
                                                        uint16_t* __restrict__ x,
                                                        const int32_t* __restrict__ pos, double log2_theta) {
  const int half = d / 2;
  for (int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x; p < n_pairs;
       p += (int64_t)gridDim.x * kThreads) {
    const int i = (int)(p % half);
    const int64_t th = p / half;                  // token * heads + head
    float s, c;
    rope_angle(pos[th / heads], i, d, log2_theta, s, c);
    uint16_t* row = x + th * d;
    uint32_t lo, hi;
    rope_turn(lo_bf16(row[i]), lo_bf16(row[i + half]), s, c, lo, hi);
    row[i] = (uint16_t)lo;
    row[i + half] = (uint16_t)hi;
  }
}

// Two tensors (a layer's Q and K) of the same tokens in one launch, d a
// multiple of 16 up to 2 kRopeHalf, 16-byte boundaries.  The fp64 angle is what
// this step costs (about a hundred instructions against four per pair for the
// turn), so a workgroup forms a token's d/2 sines and cosines once, in LDS, and
// turns all its heads with them, 8 pairs per thread and access: 2048 tokens x
// 32 heads x 128: 23.4 -> 9.3 us, 8192 tokens 80.1 -> 23.2 us.  TPB tokens per
// workgroup: 4 fill the 256 threads of the angle step; few tokens take one each,
// for more workgroups.
constexpr int kRopeHalf = 128;

template <int TPB>
__global__ void __launch_bounds__(kThreads) rope_rows_kernel(int32_t n, int32_t heads0, int32_t heads1, int32_t d,
                                                             uint16_t* __restrict__ x0, uint16_t* __restrict__ x1,
                                                             const int32_t* __restrict__ pos, double log2_theta) {
  __shared__ __attribute__((aligned(16))) float cs[2][TPB][kRopeHalf];
  const int half = d / 2, t0 = blockIdx.x * TPB, nt = min(TPB, n - t0);
  for (int e = threadIdx.x; e < nt * half; e += kThreads) {
    const int t = e / half, i = e % half;
    rope_angle(pos[t0 + t], i, d, log2_theta, cs[0][t][i], cs[1][t][i]);
  }
  __syncthreads();
  const int per_row = half / 8, rows = heads0 + heads1;
  for (int e = threadIdx.x; e < nt * rows * per_row; e += kThreads) {
    const int i = (e % per_row) * 8, tr = e / per_row, t = tr / rows, h = tr % rows;
    uint16_t* row = h < heads0 ? x0 + ((int64_t)(t0 + t) * heads0 + h) * d
                               : x1 + ((int64_t)(t0 + t) * heads1 + (h - heads0)) * d;
    const u32x4 a = *(const u32x4*)(row + i), b = *(const u32x4*)(row + half + i);
    u32x4 lo, hi;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      uint32_t l0, h0, l1, h1;
      rope_turn(lo_bf16(a[k]), lo_bf16(b[k]), cs[0][t][i + 2 * k], cs[1][t][i + 2 * k], l0, h0);
      rope_turn(hi_bf16(a[k]), hi_bf16(b[k]), cs[0][t][i + 2 * k + 1], cs[1][t][i + 2 * k + 1], l1, h1);
      lo[k] = l0 | (l1 << 16);
      hi[k] = h0 | (h1 << 16);
    }
    *(u32x4*)(row + i) = lo;
    *(u32x4*)(row + half + i) = hi;
  }
}

// out[r][j] = SiLU(gu[r][j]) * gu[r][d_ff + j], SiLU(g) = g / (1 + e^-g).
__global__ void __launch_bounds__(kThreads) silu_mul_kernel(int64_t n_chunks, int32_t dff,
                                                            const uint16_t* __restrict__ gu,
                                                            uint16_t* __restrict__ out) {
  const int per_row = dff / 8;
  for (int64_t c = (int64_t)blockIdx.x * kThreads + threadIdx.x; c < n_chunks;
       c += (int64_t)gridDim.x * kThreads) {
    const int64_t r = c / per_row;
    const int j = (int)(c % per_row) * 8;
    const u32x4 g = *(const u32x4*)(gu + r * 2 * dff + j);
    const u32x4 u = *(const u32x4*)(gu + r * 2 * dff + dff + j);
    u32x4 o;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float g0 = lo_bf16(g[k]), g1 = hi_bf16(g[k]);
      o[k] = pack(silu_f32(g0) * lo_bf16(u[k]), silu_f32(g1) * hi_bf16(u[k]));
    }
    *(u32x4*)(out + r * dff + j) = o;
  }
}

int grid_for(int64_t work) {
  int64_t g = (work + kThreads - 1) / kThreads;
  return (int)(g < 1 ? 1 : (g > 65536 ? 65536 : g));
}

}  // namespace

hipError_t launch_rmsnorm(int32_t n, int32_t dm, const void* x, const void* g, float eps, void* y,
                          hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(rmsnorm_kernel, dim3(n), dim3(kThreads), 0, s, dm, (const uint16_t*)x,
                     (const uint16_t*)g, eps, (uint16_t*)y);
  return hipGetLastError();
}

hipError_t launch_rope(int32_t n, int32_t heads0, int32_t heads1, int32_t d, void* x0, void* x1,
                       const int32_t* pos, double theta, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const double log2_theta = log2(theta);
  // The row kernel shares a token's angles among its heads and takes Q and K in one
  // launch, but one workgroup walks all heads of a token, 256 accesses of 8 pairs at a
  // time (0.9 us each; us a call on the device, rows and a pair per thread).  One
  // tensor of up to 2^17 pairs or of one head has nothing to gain (1 token x 64
  // heads of 128: 4.0, 2.6; 100 x 8: 3.2, 2.6; 100 x 32: 3.3, 3.5), and past three
  // accesses a thread it takes a hundred tokens to win again (1 x 4096 heads: 131,
  // 3.5; 100 x 4096: 153, 131; 600 x 512: 31, 103).  A launch counts its threads in 32 bits.
  const int64_t heads = (int64_t)heads0 + heads1, per_token = heads * (d / 16);
  const bool share = heads1 > 0 || (heads > 1 && n * heads * (d / 2) > (1 << 17));
  if (d % 16 == 0 && d <= 2 * kRopeHalf && (((uintptr_t)x0 | (uintptr_t)x1) & 15) == 0 && share &&
      (per_token <= 768 || (n >= 128 && per_token < (1 << 28))) && n < (1 << 26)) {
    if (n >= 1024)
      hipLaunchKernelGGL(rope_rows_kernel<4>, dim3((n + 3) / 4), dim3(kThreads), 0, s, n, heads0, heads1, d,
                         (uint16_t*)x0, (uint16_t*)x1, pos, log2_theta);
    else
      hipLaunchKernelGGL(rope_rows_kernel<1>, dim3(n), dim3(kThreads), 0, s, n, heads0, heads1, d,
                         (uint16_t*)x0, (uint16_t*)x1, pos, log2_theta);
    return hipGetLastError();
  }
  for (int i = 0; i < 2; ++i) {
    const int32_t heads = i ? heads1 : heads0;
    const int64_t pairs = (int64_t)n * heads * (d / 2);
    if (pairs <= 0) continue;
    hipLaunchKernelGGL(rope_kernel, dim3(grid_for(pairs)), dim3(kThreads), 0, s, pairs, heads, d,
                       (uint16_t*)(i ? x1 : x0), pos, log2_theta);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  return hipSuccess;
}

hipError_t launch_silu_mul(int32_t n, int32_t dff, const void* gu, void* out, hipStream_t s) {
  const int64_t chunks = (int64_t)n * (dff / 8);
  if (chunks <= 0) return hipSuccess;
  hipLaunchKernelGGL(silu_mul_kernel, dim3(grid_for(chunks)), dim3(kThreads), 0, s, chunks, dff,
                     (const uint16_t*)gu, (uint16_t*)out);
  return hipGetLastError();
}

}  // namespace pgsr
