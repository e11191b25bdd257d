// Deterministic next-token sampling for re-decode: Gumbel-max over
// logits / T with noise from the counter-based generator Philox4x64-10
// (Salmon et al., SC 2011), so a (seed, stream, position) triple always picks
// the same token (assumption A1 of Theorem 1).  T = 0 is the greedy argmax.
//
// A row's vocabulary is cut into chunks of kChunk entries, one workgroup each;
// a thread draws one Philox block (4 words -> 4 entries) at a time.  Each
// candidate becomes a 64-bit key: the fp32 score mapped to an order-preserving
// unsigned integer in the high half, the complement of the vocabulary index in
// the low half.  The largest key is then the highest score with, among equal
// scores, the lowest index, whatever order the keys are reduced in, so the
// chunk partials (in a caller workspace) and the in-workgroup reductions are
// exact and deterministic.  NaN scores count as -inf.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.h"

namespace pgsr {

namespace {

constexpr int kThreads = 256;

struct Philox4 {
  uint64_t w[4];
};

// 64 x 64 -> 128-bit product from four 32-bit multiply-adds (the low and the
// high half asked for separately cost two multiplies more).
__device__ inline void mul128(uint64_t a, uint64_t b, uint64_t& hi, uint64_t& lo) {
  const uint32_t al = (uint32_t)a, ah = (uint32_t)(a >> 32), bl = (uint32_t)b, bh = (uint32_t)(b >> 32);
  const uint64_t p0 = (uint64_t)al * bl;
  const uint64_t p1 = (uint64_t)ah * bl + (p0 >> 32);
  const uint64_t p2 = (uint64_t)al * bh + (uint32_t)p1;
  hi = (uint64_t)ah * bh + (p1 >> 32) + (p2 >> 32);
  lo = (p2 << 32) | (uint32_t)p0;
}

// Ten Philox4x64 rounds on counter c with key k.
__device__ inline Philox4 philox4x64_10(uint64_t c0, uint64_t c1, uint64_t c2, uint64_t c3, uint64_t k0,
                                        uint64_t k1) {
  constexpr uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
  constexpr uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    uint64_t lo0, hi0, lo1, hi1;
    mul128(M0, c0, hi0, lo0);
    mul128(M1, c2, hi1, lo1);
    const uint64_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
    k0 += W0;
    k1 += W1;
  }
  return Philox4{{c0, c1, c2, c3}};
}

// Philox word -> the 23 bits that make u = (k + 1/2) / 2^23
__device__ inline uint32_t noise_bits(uint64_t w) { return (uint32_t)(w >> 41); }

// The score that decides: l / T - log(-log u) in fp32.
__device__ inline float exact_score(float l, float temperature, uint32_t k) {
  const float u = ((float)k + 0.5f) * (1.f / 8388608.f);
  return l / temperature - logf(-logf(u));
}

// The same to about 1e-5 (plus 2^-22 of |l / T|), in a fifth of the
// instructions: two hardware logarithms, a multiply for the division.  Near
// u = 1 the series of -ln(1 - t) replaces the first logarithm (t = 1 - u is
// exact; the tail left out is below 2e-5 of it).  NaN counts as -inf.
__device__ inline float rough_score(float l, float inv_temperature, uint32_t k) {
  constexpr float kLn2 = 0.69314718056f;
  const float kf = (float)k;
  const float t = (8388607.5f - kf) * (1.f / 8388608.f);
  const float near1 = t * fmaf(t, fmaf(t, fmaf(t, 0.25f, 1.f / 3.f), 0.5f), 1.f);
  const float away = -kLn2 * __builtin_amdgcn_logf((kf + 0.5f) * (1.f / 8388608.f));
  const float w = t < 0.1f ? near1 : away;
  return fmaxf(fmaf(l, inv_temperature, -kLn2 * __builtin_amdgcn_logf(w)), -INFINITY);
}

__device__ inline float load_logit(const float* p, int64_t i) { return p[i]; }
__device__ inline float load_logit(const uint16_t* p, int64_t i) {
  return __uint_as_float((uint32_t)p[i] << 16);
}

// Order-preserving key: larger score, then lower index, gives a larger key.
__device__ inline uint64_t make_key(float score, int32_t v) {
  if (!(score == score)) score = -INFINITY;   // NaN never wins
  score += 0.f;                                // -0 -> +0: equal scores tie
  const uint32_t b = __float_as_uint(score);
  const uint32_t mono = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
  return ((uint64_t)mono << 32) | (uint32_t)(0xFFFFFFFFu - (uint32_t)v);
}

__device__ inline uint64_t max_key_wave(uint64_t k) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const uint64_t o = __shfl_xor(k, off);
    k = o > k ? o : k;
  }
  return k;
}

// Four consecutive logits from v0 (a multiple of 4); entries at or past v_hi
// read as -inf.  VEC: rows start on the boundary of one wide load.
template <typename T, bool VEC>
__device__ inline void load4(const T* lr, int32_t v0, int32_t v_hi, float (&l)[4]) {
  if constexpr (VEC) {                              // vocab, so v_hi, is a multiple of 4
    if constexpr (sizeof(T) == 2) {
      const uint2 w = *(const uint2*)(lr + v0);
      l[0] = __uint_as_float(w.x << 16);
      l[1] = __uint_as_float(w.x & 0xFFFF0000u);
      l[2] = __uint_as_float(w.y << 16);
      l[3] = __uint_as_float(w.y & 0xFFFF0000u);
    } else {
      const float4 w = *(const float4*)(lr + v0);
      l[0] = w.x;
      l[1] = w.y;
      l[2] = w.z;
      l[3] = w.w;
    }
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) l[j] = v0 + j < v_hi ? load_logit(lr, v0 + j) : -INFINITY;
  }
}

// Best key over this thread's entries, every entry scored exactly.
template <typename T>
__device__ inline uint64_t scan_exact(const T* lr, const SampleArgs& a, uint64_t pos, uint64_t str, int32_t v_lo,
                                      int32_t v_hi) {
  const bool hot = a.temperature > 0.f;
  uint64_t best = 0;
  for (int32_t v0 = v_lo + 4 * (int32_t)threadIdx.x; v0 < v_hi; v0 += 4 * kThreads) {
    Philox4 r{};
    if (hot) r = philox4x64_10((uint64_t)(v0 / 4), pos, str, 0, a.seed, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int32_t v = v0 + j;
      if (v >= v_hi) break;
      float score = load_logit(lr, v);
      if (hot) score = exact_score(score, a.temperature, noise_bits(r.w[j]));
      const uint64_t k = make_key(score, v);
      best = k > best ? k : best;
    }
  }
  return best;
}

// Where the best l / T of the chunk is at least this far from 0, fp32 values lie 64
// apart and -log(-log u), between -2.9 and 16.7, rounds away: the scores there are
// l / T itself, and every entry below the best keeps its distance.
constexpr float kNoiseless = 6e8f;

// Best key over this thread's entries of l / T alone, and the best of that.
template <typename T, bool VEC>
__device__ inline uint64_t scan_noiseless(const T* lr, const SampleArgs& a, int32_t v_lo, int32_t v_hi, float& hi) {
  uint64_t best = 0;
  for (int32_t v0 = v_lo + 4 * (int32_t)threadIdx.x; v0 < v_hi; v0 += 4 * kThreads) {
    float l[4];
    load4<T, VEC>(lr, v0, v_hi, l);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float s = l[j] / a.temperature;
      hi = fmaxf(hi, s);                            // NaN counts as -inf
      const uint64_t k = make_key(s, v0 + j);
      if (v0 + j < v_hi) best = k > best ? k : best;
    }
  }
  return best;
}

// Best value over the workgroup's threads (red: one slot per wave, free again after
// the next barrier).
__device__ inline float max_block(float x, float* red) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) x = fmaxf(x, __shfl_xor(x, off));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kThreads / 64; ++w) x = fmaxf(x, red[w]);
  return x;
}

// Bound by ALU: ten Philox rounds of two 64 x 64-bit products per four
// entries, then the scores.  Scoring every entry exactly (two logf, a division)
// costs as much as the generator, and only the winner's score has to be exact:
// each thread keeps its best rough score with what made it (and its second
// best), the workgroup takes the best rough score of the chunk, and the threads
// within a margin of it score their candidate exactly (2e-3 and 2e-6 of the
// score, some hundred times what the rough one can be off).  A thread whose
// second best is within it too scans its entries again exactly.  32 rows x 128256
// bf16 logits: 21-22 -> 14.5 us with the reduction, where the calling program's own
// time per call is as long; 64 x 151936: 39.5 -> 28.5 us.
// Chunks without a likely entry (a mask of -inf, of the type's lowest value or of
// -1e9) have no margin that tells entries apart, but the noise rounds away in
// their scores: a scan of l / T alone, unless that is not so after all (a
// 1 / T that overflowed).  256 rows x 128256 with 50 entries left: 127 us with every
// entry scored exactly, 135 with the rough pass before it, 94 so; dense rows 84.
template <typename T, bool VEC>
__global__ void __launch_bounds__(kThreads) sample_chunk_kernel(SampleArgs a, const T* __restrict__ logits,
                                                                int32_t* __restrict__ tokens) {
  __shared__ uint64_t red[kThreads / 64];
  __shared__ float redf[kThreads / 64];
  const int row = blockIdx.x / a.n_chunks, chunk = blockIdx.x % a.n_chunks;
  const int64_t grow = (int64_t)a.row0 + row;
  const T* lr = logits + grow * a.vocab;
  const int32_t v_lo = chunk * a.chunk_len;
  const int32_t v_hi = min(a.vocab, v_lo + a.chunk_len);
  const uint64_t pos = (uint64_t)a.position[row], str = (uint64_t)a.stream[row];
  uint64_t best = 0;
  // Philox blocks of 4 entries; chunk_len is a multiple of 4, so blocks never
  // straddle two chunks.
  if (a.temperature > 0.f) {
    const float inv_t = 1.f / a.temperature;
    float top = -INFINITY, second = -INFINITY, top_l = 0.f;
    uint32_t top_k = 0;
    int32_t top_v = 0;
    for (int32_t v0 = v_lo + 4 * (int32_t)threadIdx.x; v0 < v_hi; v0 += 4 * kThreads) {
      float l[4];
      load4<T, VEC>(lr, v0, v_hi, l);
      const Philox4 r = philox4x64_10((uint64_t)(v0 / 4), pos, str, 0, a.seed, 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t k = noise_bits(r.w[j]);
        const float s = rough_score(l[j], inv_t, k);
        second = __builtin_amdgcn_fmed3f(s, top, second);   // second <= top: the middle one of the three
        const bool better = s > top;
        top = better ? s : top;
        top_l = better ? l[j] : top_l;
        top_k = better ? k : top_k;
        top_v = better ? v0 + j : top_v;
      }
    }
    const float m = max_block(top, redf);
    if (fabsf(m) < kNoiseless) {
      const float line = m - (2e-3f + 2e-6f * fabsf(m));
      if (!(second < line)) best = scan_exact(lr, a, pos, str, v_lo, v_hi);
      else if (!(top < line)) best = make_key(exact_score(top_l, a.temperature, top_k), top_v);
    } else {                                        // the whole workgroup, as m is
      float hi = -INFINITY;
      best = scan_noiseless<T, VEC>(lr, a, v_lo, v_hi, hi);
      __syncthreads();                              // every thread has read redf
      if (fabsf(max_block(hi, redf)) < kNoiseless) best = scan_exact(lr, a, pos, str, v_lo, v_hi);
    }
  } else {
    best = scan_exact(lr, a, pos, str, v_lo, v_hi);
  }
  best = max_key_wave(best);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = best;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t k = red[0];
#pragma unroll
    for (int w = 1; w < kThreads / 64; ++w) k = red[w] > k ? red[w] : k;
    if (a.n_chunks == 1)
      tokens[grow] = (int32_t)(0xFFFFFFFFu - (uint32_t)k);
    else
      a.partial[grow * a.n_chunks + chunk] = k;
  }
}

// One thread per row: the largest of its chunk keys.
__global__ void __launch_bounds__(kThreads) sample_reduce_kernel(int32_t n, int32_t n_chunks,
                                                                 const uint64_t* __restrict__ partial,
                                                                 int32_t* __restrict__ tokens) {
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  uint64_t k = 0;
  for (int c = 0; c < n_chunks; ++c) {
    const uint64_t p = partial[(int64_t)i * n_chunks + c];
    k = p > k ? p : k;
  }
  tokens[i] = (int32_t)(0xFFFFFFFFu - (uint32_t)k);
}

}  // namespace

hipError_t launch_sample(const SampleArgs& a, int dtype, const void* logits, int32_t* tokens,
                         hipStream_t s) {
  if (a.n <= 0) return hipSuccess;
  dim3 grid(a.n * a.n_chunks);
  // four logits per load where every row starts on its boundary
  const size_t eb = dtype == 1 ? 2 : 4;
  const bool vec = a.vocab % 4 == 0 && ((uintptr_t)logits & (4 * eb - 1)) == 0;
  if (dtype == 1 && vec)
    hipLaunchKernelGGL((sample_chunk_kernel<uint16_t, true>), grid, dim3(kThreads), 0, s, a, (const uint16_t*)logits, tokens);
  else if (dtype == 1)
    hipLaunchKernelGGL((sample_chunk_kernel<uint16_t, false>), grid, dim3(kThreads), 0, s, a, (const uint16_t*)logits, tokens);
  else if (vec)
    hipLaunchKernelGGL((sample_chunk_kernel<float, true>), grid, dim3(kThreads), 0, s, a, (const float*)logits, tokens);
  else
    hipLaunchKernelGGL((sample_chunk_kernel<float, false>), grid, dim3(kThreads), 0, s, a, (const float*)logits, tokens);
  return hipGetLastError();
}

hipError_t launch_sample_reduce(int32_t n, int32_t n_chunks, const uint64_t* partial, int32_t* tokens,
                                hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(sample_reduce_kernel, dim3((n + kThreads - 1) / kThreads), dim3(kThreads), 0, s, n,
                     n_chunks, partial, tokens);
  return hipGetLastError();
}

}  // namespace pgsr
