// fp32 prefix + causal prefill attention over the paged cache, on the fp32
// matrix instructions (v_mfma_f32_16x16x4_f32: fp32 products and accumulation).
//
// A workgroup of four waves handles kRows consecutive query tokens of one query
// head.  Keys are visited in tiles of 16 at absolute positions 0, 16, 32, ...;
// wave w takes the tiles whose index is w mod 4 for all of the rows and keeps its
// own online softmax (running max m, running sum l, rescaled accumulator, base-2
// domain); the four states are merged at the end through LDS in the order 0, 1,
// 2, 3.  Tile ownership depends only on absolute positions, so a row's result
// depends only on its position and its keys: a selective replay and a full
// reset produce identical bits.
//
// Every matrix operand is loaded straight from memory into the registers that
// use it, 16 bytes a lane, one tile ahead; no LDS and no barrier in the loop:
//  * S^T = K Q^T (16 keys x 16 rows): any order of d serves as long as K and Q
//    share it, so lane group h = lane / 16 takes d in [h D/4, +D/4) and step j
//    multiplies element j of each: a lane's K row piece is contiguous;
//  * in the accumulator a lane then holds keys 4h .. 4h+3 of one row, and step r
//    of O^T += V^T P^T takes keys 4h + r (h = 0 .. 3): P is register r as it
//    stands and the V^T operand element r of the four slots 4h .. 4h+3 of one d
//    row of the [d][slot] block.
// Keys at or past the sequence length (always slots of the sequence's own last
// block) are masked by select and their V elements zeroed, so stale or NaN slots
// cannot leak into the result.
//
// Small calls are latency bound: the tiny episode (8 heads of 64, 128 tokens
// against 512 cached, split keys) takes
// 46.6 -> 21.5 us a call (34.5 us of it were this kernel on the vector units, one
// row per lane and LDS broadcasts of every key, 160 wave tiles of 32 keys on two
// of each workgroup's four waves).  Larger ones are bound by the matrix cores:
// 8 heads of 64, 2700 tokens against 300 cached, 687 -> 184 us; 8 / 2 heads of 128
// 2952 -> 331 us.
//
// Split-key mode (a call too small to fill the chip, with a workspace): split
// s of a query tile covers the keys [s * split_len, (s+1) * split_len) at
// absolute positions and writes its merged unnormalised state (m, l, acc) in
// fp32 for the split combine, which adds the splits in increasing order.
#include <hip/hip_runtime.h>

#include <cmath>

#include "attn_common.h"
#include "internal.h"

namespace pgsr {

namespace {

constexpr int kQB = 2;             // 16-row blocks per wave
constexpr int kRows = 16 * kQB;    // query tokens per workgroup
constexpr int kWaves = 4;
constexpr int kKT = 16;            // keys per tile

// max / sum over the four 16-lane groups: each swap leaves a lane its own value
// in one result and its partner group's in the other
template <class F>
__device__ inline float across_groups(float x, F f) {
  const int xi = __builtin_bit_cast(int, x);
  const auto p = __builtin_amdgcn_permlane16_swap(xi, xi, false, false);
  // through scalars: this compiler's bit cast of a vector element reads element 0
  const uint32_t p0 = p[0], p1 = p[1];
  const float y = f(__builtin_bit_cast(float, p0), __builtin_bit_cast(float, p1));
  const int yi = __builtin_bit_cast(int, y);
  const auto q = __builtin_amdgcn_permlane32_swap(yi, yi, false, false);
  const uint32_t q0 = q[0], q1 = q[1];
  return f(__builtin_bit_cast(float, q0), __builtin_bit_cast(float, q1));
}

template <int D>
__global__ void __launch_bounds__(kWaves * 64, 1) attn_f32_kernel(AttnArgs a) {
  constexpr int DL = D / 4;                       // d of one lane group
  constexpr int NDB = D / 16;                     // 16-row blocks of O^T
  constexpr int LD = D + 4;                       // LDS row of a published state (floats)
  __shared__ __attribute__((aligned(16))) float acc_lds[kWaves][kRows][LD];
  __shared__ float ml_lds[kWaves][kRows][2];

  const int tile = blockIdx.x / a.n_splits;
  const int split = blockIdx.x % a.n_splits;
  const int hq = blockIdx.y;
  int ei = 0;
  while (ei + 1 < a.n && a.e[ei + 1].tile_start <= tile) ++ei;
  const AttnEntry e = a.e[ei];
  const int lt = tile - e.tile_start;
  const int G = a.n_q_heads / a.n_kv_heads;
  const int g = hq / G;
  const int B = a.block_size;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r16 = lane & 15, h = lane >> 4;
  const int t0 = lt * kRows;
  int qpos[kQB];                                  // absolute position (-1: padding row)
#pragma unroll
  for (int b = 0; b < kQB; ++b) {
    const int t = t0 + 16 * b + r16;
    qpos[b] = t < e.q_len ? e.prefix + t : -1;
  }
  const int t_last = min(e.q_len, t0 + kRows) - 1;
  const int kv_len = e.prefix + e.q_len;
  // keys this workgroup visits: [key_lo, key_end), whole tiles at absolute
  // positions (split_len is a multiple of the tile)
  const int key_lo = a.n_splits > 1 ? split * a.split_len : 0;
  const int key_end = a.n_splits > 1 ? min(e.prefix + t_last + 1, key_lo + a.split_len) : e.prefix + t_last + 1;
  if (key_lo >= key_end) return;                  // the whole workgroup: no barrier is skipped
  const int kt0 = key_lo / kKT;
  const int n_kt = (key_end + kKT - 1) / kKT;

  // Q operand: lane (row r16, group h) holds d in [h D/4, +D/4)
  float q[kQB][DL];
#pragma unroll
  for (int b = 0; b < kQB; ++b) {
    const float* qp = (const float*)a.q +
                      ((int64_t)(e.q_off + (qpos[b] >= 0 ? t0 + 16 * b + r16 : 0)) * a.n_q_heads + hq) * D + h * DL;
#pragma unroll
    for (int c = 0; c < DL; c += 4) {
      const f32x4 v = qpos[b] >= 0 ? *(const f32x4*)(qp + c) : f32x4{0, 0, 0, 0};
#pragma unroll
      for (int i = 0; i < 4; ++i) q[b][c + i] = v[i];
    }
  }

  const int32_t* row = a.tables + (int64_t)e.seq * a.max_bps;
  const int64_t layer_off = (int64_t)a.layer * a.n_blocks * a.n_kv_heads;
  const float* kc = (const float*)a.k_cache;
  const float* vc = (const float*)a.v_cache;
  const int last_blk = (kv_len - 1) / B;
  auto block_of = [&](int kt) { return blk_id(row[min(kt * kKT / B, last_blk)], a.n_blocks, a.chk); };

  // a tile's operands: K row r16 (this group's d), V^T rows 16 db + r16 (slots 4h .. 4h+3)
  f32x4 kn[DL / 4], vn[NDB];
  auto load = [&](int kt, int32_t id) {
    const int slot = kt * kKT % B;
    const int64_t blk = layer_off + (int64_t)id * a.n_kv_heads + g;
    const float* kp = kc + (blk * B + slot + r16) * D + h * DL;
    const float* vp = vc + (blk * D + r16) * B + slot + 4 * h;
#pragma unroll
    for (int c = 0; c < DL / 4; ++c) kn[c] = *(const f32x4*)(kp + 4 * c);
#pragma unroll
    for (int db = 0; db < NDB; ++db) vn[db] = *(const f32x4*)(vp + (int64_t)db * 16 * B);
  };

  f32x4 acc[kQB][NDB];
  float m[kQB], l[kQB];
#pragma unroll
  for (int b = 0; b < kQB; ++b) {
    m[b] = -INFINITY;
    l[b] = 0.f;
#pragma unroll
    for (int db = 0; db < NDB; ++db) acc[b][db] = f32x4{0, 0, 0, 0};
  }
  const float c2 = a.scale_log2;

  int kt = kt0 + w;
  int32_t id_next = 0;
  if (kt < n_kt) {
    load(kt, block_of(kt));
    id_next = block_of(kt + kWaves);
  }
  for (; kt < n_kt; kt += kWaves) {
    f32x4 kk[DL / 4], vv[NDB];
#pragma unroll
    for (int c = 0; c < DL / 4; ++c) kk[c] = kn[c];
#pragma unroll
    for (int db = 0; db < NDB; ++db) vv[db] = vn[db];
    if (kt + kWaves < n_kt) {
      load(kt + kWaves, id_next);
      id_next = block_of(kt + 2 * kWaves);
    }
    const int key0 = kt * kKT + 4 * h;            // this lane's keys: key0 .. key0 + 3
    if (kt * kKT + kKT > kv_len) {
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int r = 0; r < 4; ++r) vv[db][r] = key0 + r < kv_len ? vv[db][r] : 0.f;
    }
    // four short chains instead of one of D/4 products: less rounding, and
    // products of one chain need not wait for each other
    f32x4 s[kQB], sp[kQB][4];
#pragma unroll
    for (int b = 0; b < kQB; ++b)
#pragma unroll
      for (int c = 0; c < 4; ++c) sp[b][c] = f32x4{0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < DL; ++j)
#pragma unroll
      for (int b = 0; b < kQB; ++b)
        sp[b][j % 4] = __builtin_amdgcn_mfma_f32_16x16x4f32(kk[j / 4][j % 4], q[b][j], sp[b][j % 4], 0, 0, 0);
#pragma unroll
    for (int b = 0; b < kQB; ++b) s[b] = (sp[b][0] + sp[b][1]) + (sp[b][2] + sp[b][3]);
#pragma unroll
    for (int b = 0; b < kQB; ++b) {
      float tmax = -INFINITY;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[b][r] = key0 + r <= qpos[b] && key0 + r < key_end ? s[b][r] * c2 : -INFINITY;
        tmax = fmaxf(tmax, s[b][r]);
      }
      tmax = across_groups(tmax, [](float x, float y) { return fmaxf(x, y); });
      const float m_new = fmaxf(m[b], tmax);
      const float m_use = m_new == -INFINITY ? 0.f : m_new;
      if (__ballot(m_new != m[b])) {
        const float alpha = exp2f(m[b] - m_use);  // 1 for a row whose max stays
        l[b] *= alpha;
#pragma unroll
        for (int db = 0; db < NDB; ++db) acc[b][db] *= alpha;
      }
      m[b] = m_new;
#pragma unroll
      for (int r = 0; r < 4; ++r) s[b][r] = exp2f(s[b][r] - m_use);
      l[b] += (s[b][0] + s[b][1]) + (s[b][2] + s[b][3]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int b = 0; b < kQB; ++b)
          acc[b][db] = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[db][r], s[b][r], acc[b][db], 0, 0, 0);
  }

  // Publish the four states (lane: row 16 b + r16, d 16 db + 4 h .. +3), then
  // every thread merges its part of the rows in the order 0, 1, 2, 3.
#pragma unroll
  for (int b = 0; b < kQB; ++b) {
    const float l_row = across_groups(l[b], [](float x, float y) { return x + y; });
#pragma unroll
    for (int db = 0; db < NDB; ++db) *(f32x4*)&acc_lds[w][16 * b + r16][16 * db + 4 * h] = acc[b][db];
    if (h == 0) {
      ml_lds[w][16 * b + r16][0] = m[b];
      ml_lds[w][16 * b + r16][1] = l_row;
    }
  }
  __syncthreads();
  constexpr int C4 = D / 4;                       // 16-byte chunks of a row
  for (int i = threadIdx.x; i < kRows * C4; i += kWaves * 64) {
    const int rr = i / C4, c = (i % C4) * 4, t = t0 + rr;
    if (t >= e.q_len) continue;
    float M = ml_lds[0][rr][0];
#pragma unroll
    for (int x = 1; x < kWaves; ++x) M = fmaxf(M, ml_lds[x][rr][0]);
    const float mu = M == -INFINITY ? 0.f : M;    // a split in which the row sees no key
    float L = 0.f;
    f32x4 o = {0, 0, 0, 0};
#pragma unroll
    for (int x = 0; x < kWaves; ++x) {
      const float wgt = exp2f(ml_lds[x][rr][0] - mu);
      L = fmaf(wgt, ml_lds[x][rr][1], L);
      o += wgt * *(const f32x4*)&acc_lds[x][rr][c];
    }
    const int64_t qrow = (int64_t)(e.q_off + t) * a.n_q_heads + hq;
    if (a.n_splits > 1) {                         // unnormalised partials
      const int64_t prow = (int64_t)split * a.n_rows + qrow;
      *(f32x4*)(a.ws_acc + prow * D + c) = o;
      if (c == 0) {
        a.ws_ml[2 * prow] = M;
        a.ws_ml[2 * prow + 1] = L;
      }
    } else {
      *(f32x4*)((float*)a.o + qrow * D + c) = o * (1.f / L);
    }
  }
}

}  // namespace

int attn_f32_tile_tokens(int, int) { return kRows; }

hipError_t launch_attn_f32(const AttnArgs& a, hipStream_t s) {
  if (a.n <= 0 || a.n_tiles <= 0) return hipSuccess;
  dim3 grid(a.n_tiles * a.n_splits, a.n_q_heads);
  if (a.head_dim == 64)
    hipLaunchKernelGGL(attn_f32_kernel<64>, grid, dim3(kWaves * 64), 0, s, a);
  else if (a.head_dim == 128)
    hipLaunchKernelGGL(attn_f32_kernel<128>, grid, dim3(kWaves * 64), 0, s, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace pgsr
