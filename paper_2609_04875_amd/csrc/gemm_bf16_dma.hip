// Dense bf16 projection Y = X W^T (+ R) for every product with K a multiple of
// 128: X and W tiles brought to LDS by global->LDS loads through a ring of NST
// stages, tiles from 16 x 16 (one wave, a re-decoded token against a model's
// weights) to 256 x 128 (eight waves).
//
// What bounds it: few rows stream W from HBM once (1 x 4096 x 14336: 22 us,
// 5.3 TB/s; the register-staged kernel 134 us, because its two K steps in
// flight cover little of the load latency and each step pays an LDS store, a
// barrier and an LDS read in a row).  From a few tens of rows on it is the rate
// at which a CU takes lines that miss L2: the lines in flight are held in the
// 32 KB first-level cache, so at HBM's latency a CU takes about 59 B/ns, however
// many requests or waves wait (a copy of the kernel without LDS reads and
// products takes the same 43 us at 102 x 4096 x 14336, and 30 us with W and X
// in L2; waves that only load, other wave layouts and deeper rings move
// nothing).  2048 x 4096 x 4096: 62 against 86-91 us, 1110 TFLOP/s; 2048 x 1024
// x 4096: 24.5 against 55 us.
//
// A stage is KSUB images of 64 k (128-byte rows of X, then of W).  A request
// is 8 rows x 128 bytes, 1 KB of contiguous LDS with lane l's 16 bytes at byte
// 16 l; chunk c of row j is fetched by the lane of slot c ^ ((j / 2) mod 8), so
// the 16 rows of an operand read fall on all 64 banks.  A request carries no
// register, so a workgroup keeps NST - 1 stages (48 to 120 KB) in flight.  Per
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

#include "elementwise.h"
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

// Up to three products of the same X (W_s of n_s rows, Y_s [M][n_s]); their
// tile columns are numbered through.
struct DmaArgs {
  int m, k, count;
  const uint16_t* x;
  const uint16_t* w[kGemmMulti];
  const uint16_t* r[kGemmMulti];
  uint16_t* y[kGemmMulti];
  int n[kGemmMulti];
};

// ONCE: one tile row, so no other tile reads this W: non-temporal requests,
// which pass the first-level cache without taking lines of it (1 x 4096 x
// 14336: 22.2 against 24.5 us, the gate|up projection 1 x 28672 x 4096 41
// against 48, 102 x 28672 x 4096 in 128 x 128 tiles 52 against 56).  Where
// several tile rows share W they cost: the later readers miss L2 too (102 x
// 4096 x 14336 in 64 x 32 tiles: 49 against 44 us).
// SILU: W holds n gate rows, then n up rows; a tile takes BN / 2 of each in
// alternating groups of 16, so a lane holds gate and up of the same outputs
// (sub-tiles 2 i and 2 i + 1) and stores bf16(SiLU(bf16(gate)) * bf16(up)),
// the bits of the projection followed by the gated product.
template <int BM, int BN, int WGM, int WGN, int KSUB, int NST, int GS, int GM, bool SILU, bool ONCE>
__global__ void __launch_bounds__(WGM * WGN * 64, 1) gemm_bf16_dma_kernel(DmaArgs a) {
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
  constexpr int BNO = SILU ? BN / 2 : BN;                  // output columns of a tile
  const int M = a.m, K = a.k;
  const int n_tm = (M + BM - 1) / BM;
  int n_tn = 0;
#pragma unroll
  for (int i = 0; i < kGemmMulti; ++i) n_tn += i < a.count ? (a.n[i] + BNO - 1) / BNO : 0;
  const int per_xcd = (n_tm * n_tn + 7) / 8;
  const int t = (int)(blockIdx.x % 8) * per_xcd + (int)(blockIdx.x / 8);
  if (t >= n_tm * n_tn) return;
  const int grp = t / (GM * n_tn), first_m = grp * GM;
  const int gsize = min(n_tm - first_m, GM);
  const int idx = t - grp * GM * n_tn;
  const int m0 = (first_m + idx % gsize) * BM;
  int tn = idx / gsize;
  const uint16_t* __restrict__ X = a.x;
  const uint16_t* __restrict__ W = a.w[0];
  const uint16_t* R = a.r[0];
  uint16_t* Y = a.y[0];
  int N = a.n[0];
#pragma unroll
  for (int i = 1; i < kGemmMulti; ++i)
    if (i < a.count && tn >= (N + BNO - 1) / BNO) {
      tn -= (N + BNO - 1) / BNO;
      W = a.w[i];
      R = a.r[i];
      Y = a.y[i];
      N = a.n[i];
    }
  const int n0 = tn * BNO;

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
    const int wrow = SILU ? min(n0 + (row >> 5) * 16 + (row & 15), N - 1) + ((row >> 4) & 1) * N : min(n0 + row, N - 1);
    woff[j] = 2u * ((uint32_t)wrow * (uint32_t)K + 8u * ((lane & 7) ^ gsw(row)));
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
        if constexpr (ONCE)
          asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt"
                       ::"v"(woff[j]), "s"(ws + sub * 2 * kSub), "s"(img + 2u * (sub * SUBE + BM * kSub) + 1024u * NW * j)
                       : "memory", "m0");
        else
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
    if constexpr (SILU) {
#pragma unroll
      for (int i = 0; i < TN; i += 2) {
        const int n = n0 + wn / 2 + 8 * i + 4 * g4;
        if (n >= N) continue;                      // N is a multiple of 8: whole group in or out
        const bf16x4 gate = __builtin_convertvector(acc[i][j], bf16x4);
        const bf16x4 up = __builtin_convertvector(acc[i + 1][j], bf16x4);
        uint32_t o[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) o[q] = f32_to_bf16(silu_f32((float)gate[q]) * (float)up[q]);
        *(u32x2*)(Y + (int64_t)m * N + n) = u32x2{o[0] | (o[1] << 16), o[2] | (o[3] << 16)};
      }
    } else {
#pragma unroll
      for (int i = 0; i < TN; ++i) {
        const int n = n0 + wn + 16 * i + 4 * g4;
        if (n >= N) continue;                      // N is a multiple of 8: whole group in or out
        const int64_t o = (int64_t)m * N + n;
        f32x4 v = acc[i][j];
        if (R) {
          const u32x2 rb = *(const u32x2*)(R + o);
          v[0] += lo_bf16(rb[0]);
          v[1] += hi_bf16(rb[0]);
          v[2] += lo_bf16(rb[1]);
          v[3] += hi_bf16(rb[1]);
        }
        *(bf16x4*)(Y + o) = __builtin_convertvector(v, bf16x4);
      }
    }
  }
}

template <int BM, int BN, int WGM, int WGN, int KSUB, int NST, int GS, int GM, bool SILU = false>
void launch_dma(const DmaArgs& a, hipStream_t s) {
  constexpr int BNO = SILU ? BN / 2 : BN;
  int cols = 0;
  for (int i = 0; i < a.count; ++i) cols += (a.n[i] + BNO - 1) / BNO;
  const int tiles = ((a.m + BM - 1) / BM) * cols;
  const dim3 grid(8 * ((tiles + 7) / 8)), blk(WGM * WGN * 64);
  if (a.m <= BM)
    hipLaunchKernelGGL((gemm_bf16_dma_kernel<BM, BN, WGM, WGN, KSUB, NST, GS, GM, SILU, true>), grid, blk, 0, s, a);
  else
    hipLaunchKernelGGL((gemm_bf16_dma_kernel<BM, BN, WGM, WGN, KSUB, NST, GS, GM, SILU, false>), grid, blk, 0, s, a);
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

// the cheapest of tiles lo .. hi for the given products of one X
int pick_tile(int m, int count, const int* n, int lo, int hi) {
  int best = lo;
  double best_cost = 0;
  for (int i = lo; i <= hi; ++i) {
    const TileCost& t = kTiles[i];
    double cols = 0;
    for (int j = 0; j < count; ++j) cols += (n[j] + t.bn - 1) / t.bn;
    const double r = (double)((m + t.bm - 1) / t.bm) * cols / kCus;
    const double cost = t.step_ns * (r <= 1.0 ? 1.0 : 0.36 * r + 0.64 * ceil(r));
    if (i == lo || cost < best_cost) {
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

static hipError_t run_tile(int tile, const DmaArgs& a, hipStream_t s) {
  switch (tile) {
    case 0: launch_dma<16, 16, 1, 1, 2, 8, 4, 8>(a, s); break;
    case 1: launch_dma<32, 16, 2, 1, 2, 8, 4, 8>(a, s); break;
    case 2: launch_dma<32, 32, 2, 2, 2, 4, 4, 8>(a, s); break;
    case 3: launch_dma<64, 32, 2, 2, 2, 6, 2, 8>(a, s); break;
    case 4: launch_dma<64, 64, 2, 2, 2, 4, 2, 8>(a, s); break;
    case 5: launch_dma<128, 64, 4, 2, 2, 3, 2, 8>(a, s); break;
    case 6: launch_dma<128, 128, 4, 2, 1, 4, 1, 8>(a, s); break;
    case 7: launch_dma<256, 128, 4, 2, 1, 3, 1, 4>(a, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_gemm_bf16_dma(int m, int n, int k, const void* x, const void* w, const void* r, void* y,
                                hipStream_t s) {
  if (!gemm_bf16_dma_eligible(m, n, k)) return hipErrorInvalidValue;
  const int tile = pick_tile(m, 1, &n, 0, gemm_bf16_wide_eligible(m, n, k) ? kWide : kWide - 1);
  if (tile == kWide) return launch_gemm_bf16_wide(m, n, k, x, w, r, y, s);
  DmaArgs a{m, k, 1, (const uint16_t*)x, {(const uint16_t*)w}, {(const uint16_t*)r}, {(uint16_t*)y}, {n}};
  return run_tile(tile, a, s);
}

// One launch for the products unless the 256 x 256 kernel is the better one
// for them together: a launch less for each, and the short ones (n = 1024: 64
// tiles of 16 columns) fill the chip beside the long one (1 token x
// (4096 + 1024 + 1024) x 4096: 11.0 against 7.8 + 7.1 + 7.1 us, 102 tokens:
// 19.1 against 13.7 + 8.0 + 8.0 us).
bool gemm_bf16_multi_eligible(int m, int k, int count, const int* n) {
  if (count < 1 || count > kGemmMulti) return false;
  int64_t total = 0;
  for (int i = 0; i < count; ++i) {
    if (!gemm_bf16_dma_eligible(m, n[i], k)) return false;
    total += n[i];
  }
  if (total > INT32_MAX) return false;
  const int sum = (int)total;
  return !(gemm_bf16_wide_eligible(m, sum, k) && pick_tile(m, 1, &sum, 0, kWide) == kWide);
}

hipError_t launch_gemm_bf16_multi(int m, int k, int count, const int* n, const void* x, const void* const* w,
                                  void* const* y, hipStream_t s) {
  if (!gemm_bf16_multi_eligible(m, k, count, n)) return hipErrorInvalidValue;
  DmaArgs a{};
  a.m = m;
  a.k = k;
  a.count = count;
  a.x = (const uint16_t*)x;
  for (int i = 0; i < count; ++i) {
    a.w[i] = (const uint16_t*)w[i];
    a.y[i] = (uint16_t*)y[i];
    a.n[i] = n[i];
  }
  return run_tile(pick_tile(m, count, n, 0, kWide - 1), a, s);
}

// Gate|up projection with the gated product in the epilogue.  Two sub-tiles of
// 16 columns per wave are the least that hold a gate and an up group, so the
// narrowest tiles differ from those above.  The 256 x 256 kernel has no such
// epilogue: where it would be chosen the two launches stay.
bool gemm_bf16_silu_eligible(int m, int dff, int k) {
  if (dff % 8 != 0 || dff > (1 << 30) || !gemm_bf16_dma_eligible(m, 2 * dff, k)) return false;
  const int n = 2 * dff;
  return pick_tile(m, 1, &n, 0, gemm_bf16_wide_eligible(m, n, k) ? kWide : kWide - 1) != kWide;
}

hipError_t launch_gemm_bf16_silu(int m, int dff, int k, const void* x, const void* w, void* y, hipStream_t s) {
  if (!gemm_bf16_silu_eligible(m, dff, k)) return hipErrorInvalidValue;
  DmaArgs a{m, k, 1, (const uint16_t*)x, {(const uint16_t*)w}, {nullptr}, {(uint16_t*)y}, {dff}};
  const int n = 2 * dff;
  switch (pick_tile(m, 1, &n, 0, kWide - 1)) {
    case 0:
    case 1:
    case 2:
      // (14336 outputs x 4096: 42 against 49 us for 30 rows, 40.6 against 41.3
      // for one; fewer columns leave CUs without a tile of 64)
      if (n >= 64 * kCus) launch_dma<32, 64, 2, 2, 2, 3, 2, 8, true>(a, s);
      else if (m <= 16) launch_dma<16, 32, 1, 1, 2, 5, 2, 8, true>(a, s);
      else launch_dma<32, 32, 2, 1, 2, 4, 4, 8, true>(a, s);
      break;
    case 3: launch_dma<64, 32, 4, 1, 2, 6, 2, 8, true>(a, s); break;
    case 4: launch_dma<64, 64, 2, 2, 2, 4, 2, 8, true>(a, s); break;
    case 5: launch_dma<128, 64, 4, 2, 2, 3, 2, 8, true>(a, s); break;
    case 6: launch_dma<128, 128, 4, 2, 1, 4, 1, 8, true>(a, s); break;
    default: launch_dma<256, 128, 4, 2, 1, 3, 1, 4, true>(a, s); break;
  }
  return hipGetLastError();
}

}  // namespace pgsr
