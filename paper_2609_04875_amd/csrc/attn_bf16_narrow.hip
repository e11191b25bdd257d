// bf16 prefix + causal prefill attention for head_dim 128 and 16-token cache
// blocks, for calls too small to fill the chip (gfx950): NW waves of 32 query
// rows, one per SIMD, tiles through global->LDS loads.
//
// What bounds it: such a call is a serial walk over the keys (its bits do not
// depend on the launch, so keys are not split), and the time is the number of
// 64-key tiles times the time of one.  The wide kernel's step carries 64 rows per
// wave (3000 cycles) and the register-gathering kernels wait for each tile's
// load latency; here a wave holds 32 rows, the tiles are requested three steps
// ahead and the other CUs stay idle.  32 query / 8 KV heads, us per call with
// the append (four-wave kernel, wide kernel, this one): 102 tokens against 1228
// cached 37, 44, 30; against 8189 181, 185, 139 (0.95 us a tile, of it 0.43 the
// 32 products at 2.4 GHz; the rest is one wave's softmax and LDS latency, which
// neither more waves per workgroup nor fewer change).  Two waves where every
// workgroup then still has a CU, else four; one wave measured 6-8% slower than
// two, its 32 requests a tile being issued in a row.
//
// Rows, key tiles and per-row arithmetic are those of the other three kernels
// (scores S^T = K Q^T and O^T += V^T P^T on v_mfma_f32_32x32x16_bf16, accumulators
// started at -m, 64-key row max with a lazy rescale, P rounded to bf16 and
// summed as rounded): the same bits.  The LDS images, the requests and the
// block table in LDS are the wide kernel's: K keeps [key][d] rows with chunk c
// of row j at slot c ^ j, V^T keeps [d][16 slots] with slots 0-7 and 8-15 of 32
// d rows in one half each; four 32 KB buffers rotate and the step on tile t
// requests tile t + 3.  The compute of a step is the pipelined kernel's and is
// scheduled by the compiler: S(t+1) with the exponentials of S(t)'s first 32
// keys, then O += V(t) P(t) with the others and the row max of S(t+1).  The
// requests carry no memory clobber, so the compiler may move LDS reads across
// them: they write the buffer of tile t - 1, which nothing reads between the
// barriers (which do clobber memory) of steps t and t + 2.
#include <hip/hip_runtime.h>

#include <cmath>

#include "attn_common.h"
#include "internal.h"

// The requests write M0 (the LDS address of a global->LDS load) from inline
// assembly that lists it as clobbered; nothing else in this file uses M0.
#pragma clang diagnostic ignored "-Winline-asm"

namespace pgsr {

namespace {

constexpr int kNKT = 64;              // keys per tile
constexpr int kNBufElems = 16384;     // elements per LDS tile buffer (K 8192, V^T 8192)
constexpr float kNSlack = 8.f;        // lazy rescale threshold, log2 units
constexpr int kNMaxIdt = 8192;        // block-table entries a workgroup keeps in LDS

template <int NW>
__global__ void __launch_bounds__(NW * 64, 1)
attn_bf16_narrow_kernel(AttnArgs a, const int32_t* __restrict__ tables, const uint16_t* __restrict__ qg_,
                        const uint16_t* __restrict__ kc, const uint16_t* __restrict__ vc,
                        uint16_t* __restrict__ og) {
  constexpr int B = 16, D = 128, KT = kNKT;
  constexpr int KB = KT / B;               // blocks per key tile
  constexpr int NDS = D / 16;              // reduction steps of S
  constexpr int NDB = D / 32;              // 32-row blocks of O^T
  constexpr int NKS = KT / 16;             // 16-key steps of PV
  constexpr int RPW = 4 / NW;              // 1 KB runs of a block image per wave
  constexpr int RPT = 8 * RPW;             // requests per wave and tile
  static_assert(KB == 4 && RPW * NW == 4, "request layout");
  __shared__ __attribute__((aligned(16))) uint16_t lds[4 * kNBufElems];
  __shared__ __attribute__((aligned(16))) uint32_t idt[kNMaxIdt];

  uint64_t clk0 = 0, rt0 = 0;
  if (a.clk) {
    clk0 = __builtin_amdgcn_s_memtime();
    rt0 = __builtin_amdgcn_s_memrealtime();
  }
  const int hkv = a.n_kv_heads;
  const int g = blockIdx.x % hkv;
  const int split = (blockIdx.x / hkv) % a.n_splits;
  const int tile = blockIdx.x / hkv / a.n_splits;
  int ei = 0;
  while (ei + 1 < a.n && a.e[ei + 1].tile_start <= tile) ++ei;
  const AttnEntry e = a.e[ei];
  const int G = a.n_q_heads / hkv;
  const int TPB = 32 / G;                           // tokens per 32-row block
  const int TW = NW * TPB;                          // tokens per tile
  const int n_tiles_e = (e.q_len + TW - 1) / TW;
  const int lt = n_tiles_e - 1 - (tile - e.tile_start);
  const int t0 = lt * TW;

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, r = lane & 31, hh = lane >> 5;
  const int hq = g * G + r % G;
  const int tok = t0 + w * TPB + r / G;
  const bool valid = r < TPB * G && tok < e.q_len;  // G not dividing 32: the last rows are padding
  const int qpos = valid ? e.prefix + tok : -1;
  const int t_last = min(e.q_len, t0 + TW) - 1;
  const int kv_len = e.prefix + e.q_len;
  const int first_q = e.prefix + t0;
  const int key_lo = split * a.split_len;
  const int key_end = min(e.prefix + t_last + 1, a.n_splits > 1 ? key_lo + a.split_len : INT32_MAX);
  if (key_lo >= key_end) return;                   // nothing of this tile in this split
  const int kt0 = key_lo / KT;
  const int n_kt = (key_end + KT - 1) / KT;
  // tiles [kt0, nu) hold only keys at or before every query of the workgroup
  const int nu = min(max((first_q + 1) / KT, kt0), n_kt);

  // Q rows (lane: Q[row][16*ds + 8*hh .. +7]), requested first, scaled below
  u32x4 qraw[NDS];
  {
    const uint16_t* qg = qg_ + ((int64_t)(e.q_off + tok) * a.n_q_heads + hq) * D + 8 * hh;
#pragma unroll
    for (int ds = 0; ds < NDS; ++ds) qraw[ds] = valid ? *(const u32x4*)(qg + 16 * ds) : u32x4{0, 0, 0, 0};
  }

  const int32_t* __restrict__ row = tables + (int64_t)e.seq * a.max_bps;
  const int64_t head_base = (int64_t)a.layer * a.n_blocks * hkv + g;
  const int last_blk = (kv_len - 1) / B;

  // A tile's blocks as byte offsets from block 0 of this layer and head (a
  // 32-bit range: the launcher takes only pools with n_blocks * n_kv_heads *
  // 4 KB < 4 GB); ids past the sequence's last block are clamped to it.  The
  // workgroup's part of the table sits in LDS: tiles up to n_kt + 3 are
  // requested.
  const uint32_t blk_bytes = (uint32_t)hkv * (B * D * 2);
  const int blk0 = kt0 * KB;
  for (int i = tid; i < (n_kt + 4 - kt0) * KB; i += NW * 64)
    idt[i] = (uint32_t)blk_id(row[min(blk0 + i, last_blk)], a.n_blocks, a.chk) * blk_bytes;
  __syncthreads();
  auto tile_ids = [&](int kt, int (&id)[KB]) {
    const u32x4 v = *(const u32x4*)&idt[(kt - kt0) * KB];
#pragma unroll
    for (int j = 0; j < KB; ++j) id[j] = __builtin_amdgcn_readfirstlane((int)v[j]);
  };
  const char* kc_h = (const char*)(kc + head_base * (B * D));
  const char* vc_h = (const char*)(vc + head_base * (B * D));
  const uint32_t lds0 = (uint32_t)(uintptr_t)&lds[0];
  // Wave w writes runs w, w + NW, .. of each block's K and V^T image.  K run q
  // = key rows 4q .. 4q+3; lane l -> row 4q + l / 16, LDS slot l % 16, so it
  // fetches chunk (l % 16) ^ row of that row.  V^T run q = d rows 32q ..
  // 32q+31; lane l -> d row 32q + l % 32, slots 8 (l / 32) .. +7.
  uint32_t kdma[RPW], vdma[RPW];
#pragma unroll
  for (int i = 0; i < RPW; ++i) {
    const int q = w + NW * i, krow = q * 4 + (lane >> 4);
    kdma[i] = 2u * (krow * D + ((lane & 15) ^ krow) * 8);
    vdma[i] = 2u * ((q * 32 + (lane & 31)) * B + (lane >> 5) * 8);
  }
  auto buf_of = [&](int x) { return ((x - kt0) & 3) * kNBufElems; };
  auto request_all = [&](int x, const int (&id)[KB]) {
    const int buf = buf_of(x);
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int i = 0; i < RPW; ++i) {
        const int blk = j & 3;
        const char* src = (j < 4 ? kc_h : vc_h) + (uint32_t)id[blk];
        const uint32_t img = lds0 + 2u * (buf + (j < 4 ? 0 : 8192) + blk * 2048) + 1024u * (w + NW * i);
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                     :: "v"(j < 4 ? kdma[i] : vdma[i]), "s"(src), "s"(img) : "m0");
      }
  };
  // Workgroup barrier once this wave's LDS traffic and all but its latest RPT
  // requests (the newest tile's) have completed.
  auto bar = [&]() { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(RPT) : "memory"); };

  f32x16 oacc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) oacc[db] = f32x16{};
  float m = -INFINITY, l = 0.f, alpha = 1.f, m_use = 0.f;
  f32x16 cinit = f32x16{};      // -m_use in every element: the start value of each S accumulator

  // Operand addresses (elements within a buffer).  K operand row i of a
  // 32-key half is key pi(i) (bits 2 and 3 of i swapped): block 2 kh + i / 16,
  // row pi(i) % 16, chunk 2 ds + hh at slot (2 ds + hh) ^ row.  V^T operand
  // (ks, db): block ks, d row 32 db + r, slots 8 hh .. +7 at 8 (r + 32 hh) of
  // group db.
  const int kr = (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1);
  const int krow_r = kr & 15;
  int kaddr[NDS];
#pragma unroll
  for (int ds = 0; ds < NDS; ++ds) kaddr[ds] = (r >> 4) * 2048 + krow_r * 128 + ((2 * ds + hh) ^ krow_r) * 8;
  const int vaddr = (r + 32 * hh) * 8;
  auto k_op = [&](int buf, int kh, int ds) {
    return __builtin_bit_cast(bf16x8, *(const u32x4*)&lds[buf + kh * 4096 + kaddr[ds]]);
  };
  auto v_op = [&](int buf, int ks, int db) {
    return __builtin_bit_cast(bf16x8, *(const u32x4*)&lds[buf + 8192 + ks * 2048 + db * 512 + vaddr]);
  };
  auto mfma = [](bf16x8 x, bf16x8 y, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, y, c, 0, 0, 0); };

  // Row max of a tile (log2 units) and the lazy-rescale decision; the wave
  // rescales O when any of its rows moved its reference max.
  auto update_max = [&](f32x16 (&s)[2]) {
    float x = -INFINITY;
#pragma unroll
    for (int kh = 0; kh < 2; ++kh)
#pragma unroll
      for (int i = 0; i < 16; ++i) x = fmaxf(x, s[kh][i]);
    const float mx = fmaxf(x, xor32(x)) + m_use;   // S holds s * c - m_use
    const bool bump = mx > m + kNSlack;
    const float m_new = bump ? mx : m;
    const float mu = m_new == -INFINITY ? 0.f : m_new;
    const float delta = mu - m_use;
    m_use = mu;
    alpha = bump ? __builtin_amdgcn_exp2f(m - m_use) : 1.f;
    m = m_new;
    if (__ballot(bump)) {
#pragma unroll
      for (int db = 0; db < NDB; ++db) oacc[db] *= alpha;
      s[0] -= delta;
      s[1] -= delta;
#pragma unroll
      for (int i = 0; i < 16; ++i) cinit[i] = -m_use;
    }
  };
  // P for 16 keys (registers o8 .. o8+7 of one 32-key half), rounded to bf16,
  // with the row-sum terms added in the fixed order.
  auto expo = [&](const f32x16& s, int o8, float& ps0, float& ps1) {
    f32x8 pv8;
#pragma unroll
    for (int j = 0; j < 8; ++j) pv8[j] = __builtin_amdgcn_exp2f(s[o8 + j]);
    const bf16x8 p = __builtin_convertvector(pv8, bf16x8);
    const bf16x2* p2 = (const bf16x2*)&p;
    ps0 = __builtin_amdgcn_fdot2_f32_bf16(p2[0], kOnes, ps0, false);
    ps1 = __builtin_amdgcn_fdot2_f32_bf16(p2[1], kOnes, ps1, false);
    ps0 = __builtin_amdgcn_fdot2_f32_bf16(p2[2], kOnes, ps0, false);
    ps1 = __builtin_amdgcn_fdot2_f32_bf16(p2[3], kOnes, ps1, false);
    return p;
  };

  // ---- prologue: tiles kt0 .. kt0+2 requested, kt0 and kt0+1 landed ---- //
#pragma unroll
  for (int x = 0; x < 3; ++x) {
    int id[KB];
    tile_ids(kt0 + x, id);
    request_all(kt0 + x, id);
  }
  // Q^T operands, Q scaled by scale * log2(e) and rounded once
  bf16x8 qf[NDS];
#pragma unroll
  for (int ds = 0; ds < NDS; ++ds) {
    asm volatile("" : "+v"(qraw[ds]));          // after the requests above
    const f32x8 qx = __builtin_convertvector(__builtin_bit_cast(bf16x8, qraw[ds]), f32x8) * a.scale_log2;
    qf[ds] = __builtin_convertvector(qx, bf16x8);
  }
  bar();

  auto qk = [&](int tb, f32x16 (&s)[2]) {
    s[0] = s[1] = cinit;
#pragma unroll
    for (int ds = 0; ds < NDS; ++ds)
#pragma unroll
      for (int kh = 0; kh < 2; ++kh) s[kh] = mfma(k_op(tb, kh, ds), qf[ds], s[kh]);
  };
  f32x16 sa[2], sb[2];
  if (nu > kt0) {
    qk(buf_of(kt0), sa);
    update_max(sa);
  }
  auto advance = [&](int x) {                   // request tile x + 3
    int ids[KB];
    tile_ids(x + 3, ids);
    request_all(x + 3, ids);
  };

  // ---- pipelined steps over unmasked tiles ----------------------------- //
  auto step = [&](int t, const f32x16 (&sc)[2], f32x16 (&sn)[2]) {
    bar();
    advance(t);
    const int tk = buf_of(t + 1), tv = buf_of(t);
    bf16x8 p[NKS];
    float ps0 = 0.f, ps1 = 0.f;
    sn[0] = sn[1] = cinit;
    // 16 products of S(t+1); exponentials of keys 0..31 of S(t)
#pragma unroll
    for (int ds = 0; ds < NDS; ++ds) {
#pragma unroll
      for (int kh = 0; kh < 2; ++kh) sn[kh] = mfma(k_op(tk, kh, ds), qf[ds], sn[kh]);
      if (ds % 4 == 0) p[ds / 4] = expo(sc[0], 8 * (ds / 4), ps0, ps1);
    }
    // 16 products of O; exponentials of keys 32..63, row max of S(t+1)
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
#pragma unroll
      for (int db = 0; db < NDB; ++db) oacc[db] = mfma(v_op(tv, ks, db), p[ks], oacc[db]);
      if (ks < 2) p[2 + ks] = expo(sc[1], 8 * ks, ps0, ps1);
    }
    l = fmaf(l, alpha, ps0 + ps1);
    asm volatile("" ::"v"(l));                  // this step's row sum in this step
    update_max(sn);
  };
  // exponentials of a whole tile, then O += V P
  auto pv_tile = [&](int tb, const f32x16 (&sc)[2]) {
    bf16x8 p[NKS];
    float ps0 = 0.f, ps1 = 0.f;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) p[ks] = expo(sc[ks / 2], 8 * (ks % 2), ps0, ps1);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
      for (int db = 0; db < NDB; ++db) oacc[db] = mfma(v_op(tb, ks, db), p[ks], oacc[db]);
    l = fmaf(l, alpha, ps0 + ps1);
  };

  int t = kt0;
  for (; t + 2 < nu; t += 2) {
    step(t, sa, sb);
    step(t + 1, sb, sa);
  }
  if (t + 1 < nu) {
    step(t, sa, sb);
    ++t;
    sa[0] = sb[0];
    sa[1] = sb[1];
  }
  if (nu > kt0) {                               // tile t's S is computed and its max taken
    bar();
    advance(t);
    pv_tile(buf_of(t), sa);
  }

  // ---- tiles on the diagonal: mask by select, unpipelined -------------- //
  for (int u = nu; u < n_kt; ++u) {
    bar();
    advance(u);
    const int tb = buf_of(u), kb = u * KT;
    if (kb + KT > kv_len) {
      // V^T slots at or past kv_len must read as 0 (P is 0 there; a stale or
      // poisoned slot need not be finite): 1024 runs of 8 slots
#pragma unroll
      for (int j = 0; j < 16 / NW; ++j) {
        const int c = tid + NW * 64 * j, blk = c >> 8, d = (c & 255) >> 1, half = c & 1;
        const int key0 = blk * B + half * 8;
        if (kb + key0 + 8 > kv_len) {
          u32x4* p = (u32x4*)&lds[tb + 8192 + blk * 2048 + (d >> 5) * 512 + ((d & 31) + 32 * half) * 8];
          *p = zero_tail(*p, kb + key0, kv_len);
        }
      }
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
    qk(tb, sa);
#pragma unroll
    for (int kh = 0; kh < 2; ++kh)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int key = kb + kh * 32 + 16 * (i >> 3) + 8 * hh + (i & 7);
        sa[kh][i] = key > qpos ? -INFINITY : sa[kh][i];
      }
    update_max(sa);
    pv_tile(tb, sa);
  }
  // requests past the last tile land in buffers nobody reads; they must
  // complete before the workgroup ends and its LDS is handed on
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

  // ---- epilogue: normalise and store (or write split partials) --------- //
  const float l_tot = l + xor32(l);
  if (valid && a.n_splits > 1) {
    const int64_t prow = (int64_t)split * a.n_rows + (int64_t)(e.q_off + tok) * a.n_q_heads + hq;
    float* acc = a.ws_acc + prow * D + 4 * hh;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4)
        *(f32x4*)(acc + db * 32 + 8 * i4) =
            f32x4{oacc[db][4 * i4 + 0], oacc[db][4 * i4 + 1], oacc[db][4 * i4 + 2], oacc[db][4 * i4 + 3]};
    if (hh == 0) *(f32x2*)(a.ws_ml + 2 * prow) = f32x2{m, l_tot};
  } else if (valid) {
    const float inv = a.o_scale / l_tot;
    uint16_t* op = og + ((int64_t)(e.q_off + tok) * a.n_q_heads + hq) * D + 4 * hh;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        f32x4 v4 = {oacc[db][4 * i4 + 0] * inv, oacc[db][4 * i4 + 1] * inv, oacc[db][4 * i4 + 2] * inv,
                    oacc[db][4 * i4 + 3] * inv};
        *(bf16x4*)(op + db * 32 + 8 * i4) = __builtin_convertvector(v4, bf16x4);
      }
  }
  if (a.clk && tid == 0 && (int)blockIdx.x < a.clk_n) {
    const uint64_t clk1 = __builtin_amdgcn_s_memtime(), rt1 = __builtin_amdgcn_s_memrealtime();
    uint64_t* c = a.clk + 4 * (int64_t)blockIdx.x;
    c[0] = clk0;
    c[1] = clk1;
    c[2] = rt0;
    c[3] = rt1;
  }
}

}  // namespace

int attn_bf16_narrow_tile_tokens(int group, int waves) { return waves * (32 / group); }

// Eligible where the wide kernel is (the same LDS images and block offsets).
hipError_t launch_attn_bf16_narrow(const AttnArgs& a, int waves, hipStream_t s) {
  if (a.n <= 0 || a.n_tiles <= 0) return hipSuccess;
  const int group = a.n_q_heads / a.n_kv_heads;
  int64_t max_kv = 0;
  for (int i = 0; i < a.n; ++i) max_kv = max(max_kv, (int64_t)a.e[i].prefix + a.e[i].q_len);
  if (!attn_bf16_wide_eligible(a.head_dim, group, a.block_size, a.n_blocks, a.n_kv_heads, max_kv))
    return hipErrorInvalidValue;
  const dim3 grid(a.n_tiles * a.n_kv_heads * a.n_splits), blk(waves * 64);
  const auto* q = (const uint16_t*)a.q;
  const auto* kc = (const uint16_t*)a.k_cache;
  const auto* vc = (const uint16_t*)a.v_cache;
  auto* o = (uint16_t*)a.o;
  if (waves == 4) hipLaunchKernelGGL(attn_bf16_narrow_kernel<4>, grid, blk, 0, s, a, a.tables, q, kc, vc, o);
  else if (waves == 2) hipLaunchKernelGGL(attn_bf16_narrow_kernel<2>, grid, blk, 0, s, a, a.tables, q, kc, vc, o);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace pgsr
