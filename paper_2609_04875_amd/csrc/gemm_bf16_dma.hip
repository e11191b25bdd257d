// Dense bf16 projection Y = X W^T (+ R) for every product with K a multiple of
// 128: X and W tiles brought to LDS by global->LDS loads through a ring of NST
// stages, tiles from 16 x 16 (one wave, a re-decoded token against a model's
// weights) to 256 x 128 (eight waves).
//
// What bounds it: few rows stream W from HBM once (1 x 4096 x 14336: 23 us,
// 5.1 TB/s; the register-staged kernel 134 us, because its two K steps in
// flight cover little of the load latency and each step pays an LDS store, a
// barrier and an LDS read in a row); a hundred rows are bound by LDS (each tile
// byte is written once and read by every wave that needs it; 102 x 4096 x
// 14336: 42.6 against 143 us, 33 us of it with W already in L2); from a few
// hundred rows on the matrix cores (2048 x 4096 x 4096: 62 against 86-91 us,
// 1110 TFLOP/s; 2048 x 1024 x 4096: 24.5 against 55 us).
//
// A stage is KSUB images of 64 k (128-byte rows of X, then of W).  A request
// is 8 rows x 128 bytes, 1 KB of contiguous LDS with lane l's 16 bytes at byte
// 16 l; chunk c of row j is fetched by the lane of slot c ^ ((j / 2) mod 8), so
// the 16 rows of an operand read fall on all 64 banks.  A request carries no
// register, so a workgroup keeps NST - 1 stages (28 to 96 KB) in flight.  Per
// stage a wave waits for its own requests of the next stage (s_waitcnt vmcnt,
// exact: the loop issues no other vector memory operation), meets the other
// waves at one barrier, reads the next operand group (GS k slices of 32) and
// refills the ring slot that the barrier freed, all ahead of the products of
// the operands already in registers.  Requests past the last stage are not
// issued; the waits of the last stages count what is left.
//
// Every output element takes the products of the register-staged and of the
// 256 x 256 kernel in the same order (A = W rows, B = X rows,
// v_mfma_f32_16x16x32_bf16, k slices of 32 from 0, then + R in fp32): the bits
// do not depend on the tile, and rows of Y not on which rows share the launch.
#include <hip/hip_runtime.h>

#include <cmath>
#include <utility>

#include "internal.h"

// The requests write M0 (the LDS address of a global->LDS load) from inline
// assembly that lists it as clobbered; nothing else in this file uses M0.
#pragma clang diagnostic ignored "-Winline-asm"

namespace pgsr {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kSub = 64;               // k per image row (128 bytes)
constexpr int kCus = 256;

__device__ inline float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

template <class F, int... I>
__device__ __forceinline__ void static_for(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}

// swizzle of the 16-byte chunk slot within a 128-byte image row
__device__ __forceinline__ int gsw(int row) { return (row >> 1) & 7; }

// all but this wave's latest N requests, and its LDS reads, complete
template <int N>
__device__ __forceinline__ void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}

template <int BM, int BN, int WGM, int WGN, int KSUB, int NST, int GS, int WPE, int GM>
__global__ void __launch_bounds__(WGM * WGN * 64, WPE)
gemm_bf16_dma_kernel(int M, int N, int K, const uint16_t* __restrict__ X, const uint16_t* __restrict__ W,
                     const uint16_t* R, uint16_t* Y) {
  constexpr int NW = WGM * WGN;
  constexpr int TM = BM / WGM / 16, TN = BN / WGN / 16;
  constexpr int XR = BM / 8 / NW, WR = BN / 8 / NW;       // 1 KB runs per wave and sub-image
  static_assert(XR * NW * 8 == BM && WR * NW * 8 == BN, "runs split evenly over the waves");
  constexpr int RPW = KSUB * (XR + WR);                    // requests per wave and stage
  static_assert(RPW * (NST - 1) <= 63, "vmcnt range");
  constexpr int SUBE = (BM + BN) * kSub, STE = KSUB * SUBE;   // elements of a sub-image pair, a stage
  constexpr int NKS = 2 * KSUB;                            // k slices of 32 per stage
  constexpr int NG = NKS / GS;                             // operand groups of GS slices per stage
  static_assert(NKS % GS == 0 && (NG == 1 || NG % 2 == 0), "operand groups");
  __shared__ __attribute__((aligned(16))) uint16_t lds[NST * STE];

  // output tile of this workgroup: XCD x = blockIdx % 8 takes tiles
  // [x * per_xcd, (x + 1) * per_xcd), in groups of GM tile rows (the tile rows
  // of one W panel run side by side on one XCD, so its L2 takes W once)
  const int n_tm = (M + BM - 1) / BM, n_tn = (N + BN - 1) / BN;
  const int per_xcd = (n_tm * n_tn + 7) / 8;
  const int t = (int)(blockIdx.x % 8) * per_xcd + (int)(blockIdx.x / 8);
  if (t >= n_tm * n_tn) return;
  const int grp = t / (GM * n_tn), first_m = grp * GM;
  const int gsize = min(n_tm - first_m, GM);
  const int idx = t - grp * GM * n_tn;
  const int m0 = (first_m + idx % gsize) * BM, n0 = (idx / gsize) * BN;

  const int tid = threadIdx.x;
  const int w = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, r16 = lane & 15, g4 = lane >> 4;
  const int wm = (w % WGM) * TM * 16, wn = (w / WGM) * TN * 16;

  // byte offsets of this lane's requests from the matrix start (m * k and n * k
  // are below 2^31); rows past M or N read row M-1 or N-1 (never stored)
  uint32_t xoff[XR], woff[WR];
#pragma unroll
  for (int j = 0; j < XR; ++j) {
    const int row = 8 * (w + NW * j) + lane / 8;
    xoff[j] = 2u * ((uint32_t)min(m0 + row, M - 1) * (uint32_t)K + 8u * ((lane & 7) ^ gsw(row)));
  }
#pragma unroll
  for (int j = 0; j < WR; ++j) {
    const int row = 8 * (w + NW * j) + lane / 8;
    woff[j] = 2u * ((uint32_t)min(n0 + row, N - 1) * (uint32_t)K + 8u * ((lane & 7) ^ gsw(row)));
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)&lds[0] + 1024u * w;
  const int nst = K / (kSub * KSUB);
  auto request = [&](int st, int slot) {
    const char* xs = (const char*)X + (int64_t)st * (2 * kSub * KSUB);
    const char* ws = (const char*)W + (int64_t)st * (2 * kSub * KSUB);
    const uint32_t img = lds0 + 2u * (uint32_t)(slot * STE);
#pragma unroll
    for (int sub = 0; sub < KSUB; ++sub) {
#pragma unroll
      for (int j = 0; j < WR; ++j)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                     ::"v"(woff[j]), "s"(ws + sub * 2 * kSub), "s"(img + 2u * (sub * SUBE + BM * kSub) + 1024u * NW * j)
                     : "memory", "m0");
#pragma unroll
      for (int j = 0; j < XR; ++j)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                     ::"v"(xoff[j]), "s"(xs + sub * 2 * kSub), "s"(img + 2u * (sub * SUBE) + 1024u * NW * j)
                     : "memory", "m0");
    }
  };
  // this wave's requests complete but for those of the latest `ahead` stages
  // (its LDS reads too), and every other wave's at the barrier
  auto landed = [&](int ahead) {
    if (ahead >= NST - 2) wait_loads<RPW * (NST - 2)>();
    else
      static_for([&](auto ic) { if (ahead == decltype(ic)::value) wait_loads<RPW * decltype(ic)::value>(); },
                 std::make_integer_sequence<int, (NST > 2 ? NST - 2 : 1)>{});
    if constexpr (NW > 1) asm volatile("s_barrier" ::: "memory");
  };

  // operand = 16 rows x 32 k: lane l -> row l % 16, k 8 (l / 16) .. +7 of the slice
  int soff[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) soff[h] = r16 * kSub + (((4 * h + g4) ^ gsw(r16)) << 3);
  bf16x8 wa[2][GS][TN], xb[2][GS][TM];
  auto read_ops = [&](int slot, int grp, auto set_c) {
    constexpr int set = decltype(set_c)::value;
#pragma unroll
    for (int h = 0; h < GS; ++h) {
      const int ks = grp * GS + h;
      const uint16_t* img = &lds[slot * STE + (ks / 2) * SUBE];
#pragma unroll
      for (int i = 0; i < TN; ++i)
        wa[set][h][i] = __builtin_bit_cast(bf16x8, *(const u32x4*)&img[(BM + wn + 16 * i) * kSub + soff[ks & 1]]);
#pragma unroll
      for (int j = 0; j < TM; ++j)
        xb[set][h][j] = __builtin_bit_cast(bf16x8, *(const u32x4*)&img[(wm + 16 * j) * kSub + soff[ks & 1]]);
    }
  };

  f32x4 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) acc[i][j] = f32x4{};

#pragma unroll
  for (int st = 0; st < NST - 1; ++st)
    if (st < nst) request(st, st);
  landed(min(NST - 1, nst) - 1);
  if (NST - 1 < nst) request(NST - 1, NST - 1);
  read_ops(0, 0, std::integral_constant<int, 0>{});

  int slot = 0;
  // stage s from ring slot `slot`, its first operand group in set par
  auto stage = [&](int s, auto par_c) {
    constexpr int par = decltype(par_c)::value;
    const int nslot = slot + 1 == NST ? 0 : slot + 1;
    static_for([&](auto gc) {
      constexpr int g = decltype(gc)::value, cur = (par + g) & 1;
      if constexpr (g < NG - 1) {
        read_ops(slot, g + 1, std::integral_constant<int, 1 - cur>{});
      } else if (s + 1 < nst) {
        landed(min(NST - 2, nst - 2 - s));
        read_ops(nslot, 0, std::integral_constant<int, 1 - cur>{});
        if (s + NST < nst) request(s + NST, slot);
      }
#pragma unroll
      for (int h = 0; h < GS; ++h)
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
          for (int j = 0; j < TM; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[cur][h][i], xb[cur][h][j], acc[i][j], 0, 0, 0);
    }, std::make_integer_sequence<int, NG>{});
    slot = nslot;
  };
  int s = 0;
  for (; s + 1 < nst; s += 2) {
    stage(s, std::integral_constant<int, 0>{});
    stage(s + 1, std::integral_constant<int, NG & 1>{});
  }
  if (s < nst) stage(s, std::integral_constant<int, 0>{});

  // acc[i][j] lane l, register q: n = wn + 16 i + 4 (l / 16) + q, m = wm + 16 j + l % 16
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    const int m = m0 + wm + 16 * j + r16;
    if (m >= M) continue;
#pragma unroll
    for (int i = 0; i < TN; ++i) {
      const int n = n0 + wn + 16 * i + 4 * g4;
      if (n >= N) continue;                        // N is a multiple of 8: whole group in or out
      const int64_t o = (int64_t)m * N + n;
      f32x4 v = acc[i][j];
      if (R) {
        const u32x2 rb = *(const u32x2*)(R + o);
        v[0] += bf16_to_f32((uint16_t)(rb[0] & 0xFFFF));
        v[1] += bf16_to_f32((uint16_t)(rb[0] >> 16));
        v[2] += bf16_to_f32((uint16_t)(rb[1] & 0xFFFF));
        v[3] += bf16_to_f32((uint16_t)(rb[1] >> 16));
      }
      *(bf16x4*)(Y + o) = __builtin_convertvector(v, bf16x4);
    }
  }
}

template <int BM, int BN, int WGM, int WGN, int KSUB, int NST, int GS, int WPE, int GM>
void launch_dma(int m, int n, int k, const void* x, const void* w, const void* r, void* y, hipStream_t s) {
  const int tiles = ((m + BM - 1) / BM) * ((n + BN - 1) / BN);
  hipLaunchKernelGGL((gemm_bf16_dma_kernel<BM, BN, WGM, WGN, KSUB, NST, GS, WPE, GM>), dim3(8 * ((tiles + 7) / 8)),
                     dim3(WGM * WGN * 64), 0, s, m, n, k, (const uint16_t*)x, (const uint16_t*)w,
                     (const uint16_t*)r, (uint16_t*)y);
}

// Tile choice: the time of a launch is close to
//   max(1, 0.36 r + 0.64 ceil(r)) * (K / 64) * step,   r = tiles / 256 CUs
// (a partly filled last round costs most of a whole one), with the measured
// time of one 64-k step of one tile per CU.  The steps below are the fit to
// 240 products (M 1 to 4096; N, K of three models' projections), where the
// tile it picks is on average 0.3% and at most 17% slower than the fastest of
// twelve; the last is the 256 x 256 kernel of gemm_bf16_wide.hip.
struct TileCost {
  int bm, bn;
  double step_ns;
};
constexpr TileCost kTiles[] = {{16, 16, 68},  {32, 16, 112},  {32, 32, 122},  {64, 32, 172},   {64, 64, 277},
                               {128, 64, 350}, {128, 128, 538}, {256, 128, 885}, {256, 256, 1450}};
constexpr int kWide = 8;

int pick_tile(int m, int n, int k, bool wide_ok) {
  int best = 0;
  double best_cost = 0;
  for (int i = 0; i <= kWide; ++i) {
    if (i == kWide && !wide_ok) break;
    const TileCost& t = kTiles[i];
    const double r = (double)((m + t.bm - 1) / t.bm) * ((n + t.bn - 1) / t.bn) / kCus;
    const double cost = t.step_ns * (r <= 1.0 ? 1.0 : 0.36 * r + 0.64 * ceil(r));
    if (i == 0 || cost < best_cost) {
      best = i;
      best_cost = cost;
    }
  }
  return best;
}

}  // namespace

bool gemm_bf16_dma_eligible(int m, int n, int k) {
  return k >= 128 && k % 128 == 0 && (int64_t)m * k < ((int64_t)1 << 31) && (int64_t)n * k < ((int64_t)1 << 31);
}

hipError_t launch_gemm_bf16_dma(int m, int n, int k, const void* x, const void* w, const void* r, void* y,
                                hipStream_t s) {
  if (!gemm_bf16_dma_eligible(m, n, k)) return hipErrorInvalidValue;
  switch (pick_tile(m, n, k, gemm_bf16_wide_eligible(m, n, k))) {
    case 0: launch_dma<16, 16, 1, 1, 2, 8, 4, 1, 8>(m, n, k, x, w, r, y, s); break;
    case 1: launch_dma<32, 16, 2, 1, 2, 8, 4, 1, 8>(m, n, k, x, w, r, y, s); break;
    case 2: launch_dma<32, 32, 2, 2, 2, 4, 4, 1, 8>(m, n, k, x, w, r, y, s); break;
    case 3: launch_dma<64, 32, 2, 2, 2, 6, 2, 1, 8>(m, n, k, x, w, r, y, s); break;
    case 4: launch_dma<64, 64, 2, 2, 2, 4, 2, 1, 8>(m, n, k, x, w, r, y, s); break;
    case 5: launch_dma<128, 64, 4, 2, 2, 3, 2, 1, 8>(m, n, k, x, w, r, y, s); break;
    case 6: launch_dma<128, 128, 4, 2, 1, 4, 1, 1, 8>(m, n, k, x, w, r, y, s); break;
    case 7: launch_dma<256, 128, 4, 2, 1, 3, 1, 1, 4>(m, n, k, x, w, r, y, s); break;
    default: return launch_gemm_bf16_wide(m, n, k, x, w, r, y, s);
  }
  return hipGetLastError();
}

}  // namespace pgsr
