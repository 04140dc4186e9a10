// MoDA attention backward, bf16 inputs, fp32 accumulation, gfx950 MFMA.
//
// The paper gives no backward algorithm; this is the derivative of the forward
// definition (one softmax over causal sequence keys and same-position depth slots),
// evaluated by recomputation from Q, K, V, the depth tensors, O and LSE:
//   p_c = exp(scale <q_t, k_c> - LSE_t),  delta_t = <dO_t, O_t>,
//   dV_c += p_c dO_t,  e_c = p_c (<dO_t, v_c> - delta_t),
//   dQ_t = scale sum_c e_c k_c,  dK_c += scale e_c q_t.
// No atomics, every output element written exactly once:
//   delta  : LSE_t log2(e) and -delta_t for every row (row-parallel, vector ALUs).
//   grads  : dK, dV and dQ in ONE launch, whose workgroups each take a key tile or a query tile as the two
//            kernels below do; the depth slots go with the query tiles.  Calls of more than 16 positions
//            without depth slots, or with 1, 2 or 4 heads per group, whose workgroups fit one grid.  All others:
//   dkdv   : one workgroup per 128 sequence keys; Q / dO tiles stream through LDS;
//            S = Q K^T and dP = dO V^T are recomputed per 32x32 block on the MFMA
//            pipe, P and dS = P (dP - delta) are packed to bf16 straight out of the
//            accumulators and contracted over the queries into dV^T, dK^T.  The same
//            workgroup also takes the depth slots of its 128 positions (row-local: dKdepth,
//            dVdepth and the depth share of dQ, left in the workspace in fp32), before or
//            after its key-tile work: that part is bound by HBM, the rest by the matrix pipe.
//            (When there are too few key tiles to fill the chip, dkdv_short: one workgroup per 32
//            keys, whose waves deal out the queries; and dq_short likewise for dQ.)
//   dq     : one workgroup per 128 queries; K / V tiles stream through LDS; S^T, dP^T
//            are recomputed in the transposed orientation (a lane owns one query),
//            dQ^T += K^T dS^T on top of the depth share found in the workspace; every
//            element of dQ is rounded to bf16 once.
// Grouped-query attention (G = Hq / Hk query heads per key/value head, G <= 64): the
// gradients of the shared keys and values sum over the group.  dkdv walks the query
// tiles of all G heads; the depth-slot gradients hold the G heads of a position side by side, sum in
// fp32 and round every depth gradient once:
//   up to 4 heads  : inside grads (or dkdv, dkdv_short), on the vector ALUs (depth_gqa_row);
//   5 to 8 heads   : at d = 64 with blocks of 32 slots well filled, inside dkdv on the matrix pipe
//                    (depth_group_rows); otherwise a kernel of their own on the vector ALUs (depth_gqa);
//   9 heads and up : a kernel of their own on the matrix pipe (depth_group).
#include <algorithm>
#include <math.h>
#include <stdio.h>
#include <type_traits>

#include "moda_launch.h"
#include "moda_tile.h"

namespace moda {

constexpr float kLog2e = 1.4426950408889634f;

// ---------------------------------------------------------------- per-row scalars
// lse2[row] = LSE_row * log2(e) and minus_delta[row] = -<dO_row, O_row> for the other kernels: they
// exponentiate with exp2, and start the accumulators of dP = dO V^T from -delta, so that dP - delta
// comes out of the matrix pipe (a query tile's values are copied to LDS without passing through
// registers and read from there as accumulators).  The matrix kernels below are bound by power (on all-zero
// inputs they take the same cycles at 2.3 GHz instead of 1.5 to 1.7): a subtraction less per weight, one
// vector instruction in four, let the clock rise.  d = 64, B=1 Hq=64 Hk=8 T=16384: dK/dV 4.49 -> 4.25 ms, dQ
// 3.04 -> 2.93; d = 128, B=8 H=16 T=4096 without slots: whole call 1.87 -> 1.81 ms.
template <int D>
__global__ __launch_bounds__(256) void moda_bwd_delta_kernel(const void* dO, const void* O, const float* LSE,
                                                             float* lse2, float* minus_delta, long long rows) {
  constexpr int LPR = D / 8;  // lanes per row, 8 channels each
  const long long row = ((long long)blockIdx.x * 256 + threadIdx.x) / LPR;
  const int l = threadIdx.x % LPR;
  const long long rc = row < rows ? row : rows - 1;
  const u32x4 a = *(const u32x4*)((const char*)dO + (size_t)rc * D * 2 + l * 16);
  const u32x4 b = *(const u32x4*)((const char*)O + (size_t)rc * D * 2 + l * 16);
  float s = 0.f;
#pragma unroll
  for (int k = 0; k < 4; ++k) s = dot2_bf16(a[k], b[k], s);
  s = group_sum<LPR>(s);
  if (l == 0 && row < rows) {
    lse2[row] = LSE[row] * kLog2e;
    minus_delta[row] = -s;
  }
}

template <int D, int NW = 4>
struct BwdCfg {
  static constexpr int kXRow = D * 4 + 16;        // fp32 exchange row, padded
  static constexpr int kXWave = 32 * kXRow;       // 32 rows per wave
  static constexpr int kXBytes = NW * kXWave;
  static constexpr int kStageBytes = 2 * Tile<D>::kBytes;  // two tiles per stage
  static constexpr int kAux = 2 * 2 * 64 * 4;     // per stage: lse2, then -delta of 64 queries (dkdv only)
  static constexpr int kRing = 2 * kStageBytes;
  static constexpr int kLds = (kRing > kXBytes ? kRing : kXBytes) + kAux;
};

// 16 bytes per lane to a raw buffer (non-temporal), followed by two wait states in the same
// statement.  Measured on this chip: a vector-ALU instruction that overwrites the last data
// register of a 128-bit buffer store in the very next issue slot can still change what is
// stored (the last lanes of each row of 16 read their data last), also when the store takes its
// offset from a scalar register, the one case for which the compiler inserts no wait state.
__device__ __forceinline__ void buffer_store16_nt(const u32x4& v, const i32x4& rsrc, int voff, int soff) {
  asm volatile("buffer_store_dwordx4 %0, %1, %2, %3 offen nt\n\ts_nop 1" : : "v"(v), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}

// Eight channels of a finished dQ row: the depth share `acc` plus the sum over the sequence keys in LDS, in PARTS
// rows XPART bytes apart from `x` (the first channel of the first one) on; scaled and rounded once.
template <int PARTS, int XPART>
__device__ __forceinline__ void store_dq_row(const BwdParams& p, size_t row, int row_bytes, int l16, const float* acc, const unsigned char* x) {
  f32x4 a = *(const f32x4*)(x + l16 * 32), b = *(const f32x4*)(x + l16 * 32 + 16);
#pragma unroll
  for (int w = 1; w < PARTS; ++w) {
    a += *(const f32x4*)(x + w * XPART + l16 * 32);
    b += *(const f32x4*)(x + w * XPART + l16 * 32 + 16);
  }
  const float f = p.scale;
  *(u32x4*)((char*)p.dQ + row * row_bytes + l16 * 16) =
      (u32x4){pack_bf16((acc[0] + a[0]) * f, (acc[1] + a[1]) * f), pack_bf16((acc[2] + a[2]) * f, (acc[3] + a[3]) * f),
              pack_bf16((acc[4] + b[0]) * f, (acc[5] + b[1]) * f), pack_bf16((acc[6] + b[2]) * f, (acc[7] + b[3]) * f)};
}

// ---------------------------------------------------------------- depth-slot gradients (G = 1)
// The depth slots of ROWS consecutive positions (row0 ...) of one head, handled by one wave in a
// row-major mapping (d/8 lanes x 8 channels per row, 64 / (d/8) rows per wave step): dKdepth,
// dVdepth (row-local, written once) and the depth share of dQ, which is left in the workspace
// (fp32, not yet multiplied by the softmax scale) for the dQ kernel to start from.
// Work items (row step, chunk of kChunk slots) are walked with the loads of the next two
// items in flight (the phase is bound by memory latency).  Uses no LDS.
// With `xw` (dQ tiles that take their slots after their key tiles): the fp32 sums over the sequence keys in LDS, rows
// XROW bytes apart (see store_dq_row), are added and dQ is finished and stored.
template <int D, int ROWS, int CH = 5, int XROW = 0, int PARTS = 1, int XPART = 0>
__device__ __forceinline__ void depth_grad_rows(const BwdParams& p, int bh, int row0, int lane, const unsigned char* xw = nullptr) {
  using Tl = Tile<D>;
  constexpr int LPR = Tl::kChunks, RPS = 64 / LPR;
  static_assert(ROWS % RPS == 0, "whole row steps");
  constexpr int kChunk = CH;
  const int T = p.T, L = p.depth_count, La = p.depth_alloc;
  const int bg = bh, qw0 = row0;
  if (qw0 >= T) return;  // (wave-uniform)
  const int NIT = min(ROWS / RPS, (T - qw0 + RPS - 1) / RPS);
  const float c2 = p.scale_log2;
  const char* Qb = (const char*)p.Q + (size_t)bh * T * Tl::kRowBytes;
  const char* dOb = (const char*)p.dO + (size_t)bh * T * Tl::kRowBytes;
  const float* lseb = p.lse2 + (size_t)bh * T;
  const float* deltab = p.minus_delta + (size_t)bh * T;
  const int rg = lane / LPR, l16 = lane % LPR;
  const size_t drow = (size_t)La * Tl::kRowBytes;
  // (this phase only runs when every key/value head serves one query head: bg == bh)
  // The depth tensors are addressed from the first of the wave's positions (a 64-bit base)
  // with 32-bit offsets from there, so they may be of any size; `slab` is what is left of the
  // (batch, head) slab from that position on, clamped to what 32 bits hold.
  const int rbase = qw0;
  const size_t dbase = ((size_t)bg * T + rbase) * drow;
  const size_t left = (size_t)(T - rbase) * drow;
  const size_t slab = left < 0xffffffffull ? left : 0xffffffffull;
  const char* Kdb = (const char*)p.Kdepth + dbase;
  const char* Vdb = (const char*)p.Vdepth + dbase;
  char* dKdb = (char*)p.dKdepth + dbase;
  char* dVdb = (char*)p.dVdepth + dbase;
  float* dQd = p.dq_depth + (size_t)bh * T * D;
  const __amdgpu_buffer_rsrc_t kd_buf = __builtin_amdgcn_make_buffer_rsrc((void*)Kdb, 0, (int)(unsigned)slab, 0x00020000);
  const __amdgpu_buffer_rsrc_t vd_buf = __builtin_amdgcn_make_buffer_rsrc((void*)Vdb, 0, (int)(unsigned)slab, 0x00020000);
  const i32x4 dkd_buf = make_tile_buffer(dKdb, (unsigned)slab);
  const i32x4 dvd_buf = make_tile_buffer(dVdb, (unsigned)slab);
  const int nch = (L + kChunk - 1) / kChunk;

  struct Item {
    u32x4 q, g;   // the row's Q and dO channels of this lane
    float l2, md;  // LSE * log2(e), -delta
    u32x4 k[kChunk], v[kChunk];
  };
  float acc[8];
  auto begin_row = [&]() {
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] = 0.f;
  };
  auto end_row = [&](int row) {
    const int t = qw0 + row;
    if (t < T) {
      if constexpr (XROW > 0) {
        store_dq_row<PARTS, XPART>(p, (size_t)bh * T + t, Tl::kRowBytes, l16, acc, xw + row * XROW);
        return;
      }
      float* dst = dQd + (size_t)t * D + l16 * 8;
      *(f32x4*)dst = (f32x4){acc[0], acc[1], acc[2], acc[3]};
      *(f32x4*)(dst + 4) = (f32x4){acc[4], acc[5], acc[6], acc[7]};
    }
  };
  if (L == 0) {  // no attended slots: a zero share of dQ, zero gradients for allocated slots
    for (int it = 0; it < NIT; ++it) {
      const int row = it * RPS + rg, t = qw0 + row;
      begin_row();
      end_row(row);
      if (t < T) {
        const u32x4 z = {0u, 0u, 0u, 0u};
        for (int i = 0; i < La; ++i) {
          *(u32x4*)(dVdb + (size_t)(t - rbase) * drow + (size_t)i * Tl::kRowBytes + l16 * 16) = z;
          *(u32x4*)(dKdb + (size_t)(t - rbase) * drow + (size_t)i * Tl::kRowBytes + l16 * 16) = z;
        }
      }
    }
    return;
  }
  auto issue = [&](int it, int c, Item& b) {
    const int tc = min(qw0 + it * RPS + rg, T - 1);  // rows past the end use row T-1; nothing of them is stored
    b.q = *(const u32x4*)(Qb + (size_t)tc * Tl::kRowBytes + l16 * 16);
    b.g = *(const u32x4*)(dOb + (size_t)tc * Tl::kRowBytes + l16 * 16);
    b.l2 = lseb[tc];
    b.md = deltab[tc];
    const int voff = (int)((unsigned)(tc - rbase) * (unsigned)drow + (unsigned)l16 * 16u);  // 32 positions' slots: far below 4 GiB
    // slots of the chunk past depth_count re-read the last attended slot (a cache hit, ignored)
#pragma unroll
    for (int i = 0; i < kChunk; ++i)
      b.k[i] = __builtin_amdgcn_raw_buffer_load_b128(kd_buf, voff, min(c * kChunk + i, L - 1) * Tl::kRowBytes, 2);
#pragma unroll
    for (int i = 0; i < kChunk; ++i)
      b.v[i] = __builtin_amdgcn_raw_buffer_load_b128(vd_buf, voff, min(c * kChunk + i, L - 1) * Tl::kRowBytes, 2);
  };
  auto fold = [&](int it, int c, const Item& b) {
    // (rows past the end compute on row T-1; their stores lie outside the buffers, i.e. are not made)
    const int voff = (int)((unsigned)(it * RPS + rg) * (unsigned)drow + (unsigned)l16 * 16u);
    const int soff = c * kChunk * Tl::kRowBytes;
    float qx[8], gx[8];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      qx[2 * k] = bf16_lo(b.q[k]);
      qx[2 * k + 1] = bf16_hi(b.q[k]);
      gx[2 * k] = bf16_lo(b.g[k]);
      gx[2 * k + 1] = bf16_hi(b.g[k]);
    }
    // No branch per slot before the stores: the slots' chains of dependent instructions (dot products, lane sums,
    // exponential) overlap.  Slots past depth_count may hold anything (NaN included); here they repeat the last
    // attended one, with weight zero, and those that are allocated get zero gradients.
    float pe[kChunk], e[kChunk];
#pragma unroll
    for (int i = 0; i < kChunk; ++i) {
      float sdot = 0.f, gdot = 0.f;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        sdot = dot2_bf16(b.q[k], b.k[i][k], sdot);
        gdot = dot2_bf16(b.g[k], b.v[i][k], gdot);
      }
      sdot = group_sum<LPR>(sdot);
      gdot = group_sum<LPR>(gdot);
      pe[i] = fast_exp2(sdot * c2 - b.l2);
      e[i] = pe[i] * (gdot + b.md);
    }
    auto slot = [&](int i) {
      const float es = e[i] * p.scale;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        acc[2 * k] += e[i] * bf16_lo(b.k[i][k]);
        acc[2 * k + 1] += e[i] * bf16_hi(b.k[i][k]);
      }
      const u32x4 o1 = {pack_bf16(pe[i] * gx[0], pe[i] * gx[1]), pack_bf16(pe[i] * gx[2], pe[i] * gx[3]),
                        pack_bf16(pe[i] * gx[4], pe[i] * gx[5]), pack_bf16(pe[i] * gx[6], pe[i] * gx[7])};
      const u32x4 o2 = {pack_bf16(es * qx[0], es * qx[1]), pack_bf16(es * qx[2], es * qx[3]),
                        pack_bf16(es * qx[4], es * qx[5]), pack_bf16(es * qx[6], es * qx[7])};
      buffer_store16_nt(o1, dvd_buf, voff + i * Tl::kRowBytes, soff);
      buffer_store16_nt(o2, dkd_buf, voff + i * Tl::kRowBytes, soff);
    };
    if ((c + 1) * kChunk <= L) {  // (uniform)
#pragma unroll
      for (int i = 0; i < kChunk; ++i) slot(i);
      return;
    }
#pragma unroll
    for (int i = 0; i < kChunk; ++i) {
      if (c * kChunk + i < L) {
        slot(i);
      } else if (c * kChunk + i < La) {
        const u32x4 z = {0u, 0u, 0u, 0u};
        buffer_store16_nt(z, dvd_buf, voff + i * Tl::kRowBytes, soff);
        buffer_store16_nt(z, dkd_buf, voff + i * Tl::kRowBytes, soff);
      }
    }
  };
  int it = 0, c = 0, iti = 0, ci = 0;
  auto advance = [&](int& i_, int& c_) {
    if (++c_ == nch) {
      c_ = 0;
      ++i_;
    }
  };
  // (past the end the issue cursor stays on the last item: its loads are repeated and ignored)
  auto issue_next = [&](Item& b) {
    issue(iti, ci, b);
    int i2 = iti, c2n = ci;
    advance(i2, c2n);
    if (i2 < NIT) {
      iti = i2;
      ci = c2n;
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto one = [&](const Item& cur, Item& refill) -> bool {
    issue_next(refill);
    const int row = it * RPS + rg;
    if (c == 0) begin_row();
    fold(it, c, cur);
    if (c == nch - 1) {
      end_row(row);
      // allocated slots beyond the last chunk (depth_alloc > depth_count rounded up to a chunk)
      const int t = qw0 + row;
      if (t < T) {
        const u32x4 z = {0u, 0u, 0u, 0u};
        for (int i = nch * kChunk; i < La; ++i) {
          *(u32x4*)(dVdb + (size_t)(t - rbase) * drow + (size_t)i * Tl::kRowBytes + l16 * 16) = z;
          *(u32x4*)(dKdb + (size_t)(t - rbase) * drow + (size_t)i * Tl::kRowBytes + l16 * 16) = z;
        }
      }
    }
    advance(it, c);
    return it < NIT;
  };
  Item bufA, bufB, bufC;
  issue_next(bufA);
  issue_next(bufB);
  while (true) {
    if (!one(bufA, bufC)) break;
    if (!one(bufB, bufA)) break;
    if (!one(bufC, bufB)) break;
  }
}

// ---------------------------------------------------------------- depth-slot gradients, grouped queries (2 <= G <= 8)
// One row = one (batch, key/value head, position); d/8 lanes x 8 channels per row, `row` is
// (b * Hk + g) * T + t of this thread's row (rows that do not exist: `live` false, they compute on
// a clamped row and store nothing).  The GT (>= G) query heads of the group are resident (their Q
// and dO rows, LSE, delta, and their depth share of dQ); the row's slots stream by, the next ones
// prefetched.  Per slot i:
//   dVdepth_i = sum_h p_{h,i} dO_h,  dKdepth_i = scale sum_h e_{h,i} q_h  (summed in fp32, one
//                                    rounding each),
//   dQ_h     += e_{h,i} k_i          (left in the workspace, fp32, unscaled, for the dQ kernel).
// Groups of up to 4 heads: runs inside the kernel of dQ's tiles, for the positions of a tile, before or after
// its key tiles (3 heads: inside dK/dV): the phase is then bound by HBM (the slots read
// once, their gradients written once), the key tiles by the matrix pipe.
// XROW > 0: as for depth_grad_rows; `xw` is the row of the first head, the next head's XHEAD bytes further on.
template <int D, int GT, int AHEAD = 4, int XROW = 0, int XHEAD = 0, int PARTS = 1, int XPART = 0>
__device__ __forceinline__ void depth_gqa_row(const BwdParams& p, long long row, bool live, int l16, const unsigned char* xw = nullptr) {
  constexpr int LPR = D / 8, RB = D * 2;
  const int T = p.T, L = p.depth_count, La = p.depth_alloc, G = p.Hq / p.Hk;
  const long long rc = row;
  const int t = (int)(rc % T);
  const int bg = (int)(rc / T);
  const int bh0 = (bg / p.Hk) * p.Hq + (bg % p.Hk) * G;
  const float c2 = p.scale_log2;
  u32x4 q[GT], g[GT];
  float l2[GT], md[GT], dq[GT][8];
#pragma unroll
  for (int j = 0; j < GT; ++j) {
    const int bh = bh0 + min(j, G - 1);  // heads past the group repeat the last one with weight zero
    q[j] = *(const u32x4*)((const char*)p.Q + ((size_t)bh * T + t) * RB + l16 * 16);
    g[j] = *(const u32x4*)((const char*)p.dO + ((size_t)bh * T + t) * RB + l16 * 16);
    l2[j] = p.lse2[(size_t)bh * T + t];
    md[j] = p.minus_delta[(size_t)bh * T + t];
#pragma unroll
    for (int k = 0; k < 8; ++k) dq[j][k] = 0.f;
  }
  const size_t drow = (size_t)La * RB;
  const char* kd = (const char*)p.Kdepth + (size_t)rc * drow + l16 * 16;
  const char* vd = (const char*)p.Vdepth + (size_t)rc * drow + l16 * 16;
  char* dkd = (char*)p.dKdepth + (size_t)rc * drow + l16 * 16;
  char* dvd = (char*)p.dVdepth + (size_t)rc * drow + l16 * 16;

  // The next kAhead slots are in flight: each is only 2 KB of a wave's loads, and with one ahead a wave
  // of few heads waited out the memory latency at every slot.  (No load past the last slot, whose branch
  // is uniform.)  Backward call, one / four ahead: B=6 Hq=16 Hk=8 T=2048, 31 slots d=64 526 / 494 us, d=128
  // 1018 / 964; B=2 T=1000, 12 slots d=128 116 / 102.  At 8 heads the arithmetic is the longer part.
  constexpr int kAhead = GT > 4 ? 1 : AHEAD;
  u32x4 kn[kAhead], vn[kAhead];
  auto request = [&](int u, int i) {
    if (i < L) {
      kn[u] = __builtin_nontemporal_load((const u32x4*)(kd + (size_t)i * RB));
      vn[u] = __builtin_nontemporal_load((const u32x4*)(vd + (size_t)i * RB));
    }
  };
#pragma unroll
  for (int u = 0; u < kAhead; ++u) {
    kn[u] = vn[u] = (u32x4){0u, 0u, 0u, 0u};
    request(u, u);
  }
  auto slot = [&](int i, const u32x4& kv, const u32x4& vv) {
    float kx[8], ak[8], av[8];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      kx[2 * k] = bf16_lo(kv[k]);
      kx[2 * k + 1] = bf16_hi(kv[k]);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) ak[k] = av[k] = 0.f;
#pragma unroll
    for (int j = 0; j < GT; ++j) {
      float sdot = 0.f, gdot = 0.f;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        sdot = dot2_bf16(q[j][k], kv[k], sdot);
        gdot = dot2_bf16(g[j][k], vv[k], gdot);
      }
      sdot = group_sum<LPR>(sdot);
      gdot = group_sum<LPR>(gdot);
      const float pe = j < G ? fast_exp2(sdot * c2 - l2[j]) : 0.f;
      const float e = pe * (gdot + md[j]);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        av[2 * k] += pe * bf16_lo(g[j][k]);
        av[2 * k + 1] += pe * bf16_hi(g[j][k]);
        ak[2 * k] += e * bf16_lo(q[j][k]);
        ak[2 * k + 1] += e * bf16_hi(q[j][k]);
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) dq[j][k] += e * kx[k];
    }
    if (live) {
      const float f = p.scale;
      const u32x4 o1 = {pack_bf16(av[0], av[1]), pack_bf16(av[2], av[3]), pack_bf16(av[4], av[5]), pack_bf16(av[6], av[7])};
      const u32x4 o2 = {pack_bf16(ak[0] * f, ak[1] * f), pack_bf16(ak[2] * f, ak[3] * f),
                        pack_bf16(ak[4] * f, ak[5] * f), pack_bf16(ak[6] * f, ak[7] * f)};
      __builtin_nontemporal_store(o1, (u32x4*)(dvd + (size_t)i * RB));
      __builtin_nontemporal_store(o2, (u32x4*)(dkd + (size_t)i * RB));
    }
  };
  for (int i0 = 0; i0 < L; i0 += kAhead)
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int i = i0 + u;
      if (i >= L) break;  // (uniform)
      const u32x4 kv = kn[u], vv = vn[u];
      request(u, i + kAhead);
      slot(i, kv, vv);
    }
  if (live) {
    const u32x4 z = {0u, 0u, 0u, 0u};
    for (int i = L; i < La; ++i) {  // allocated but unattended slots get zero gradients
      *(u32x4*)(dvd + (size_t)i * RB) = z;
      *(u32x4*)(dkd + (size_t)i * RB) = z;
    }
#pragma unroll
    for (int j = 0; j < GT; ++j)
      if (j < G) {
        if constexpr (XROW > 0) {
          store_dq_row<PARTS, XPART>(p, (size_t)(bh0 + j) * T + t, RB, l16, dq[j], xw + j * XHEAD);
          continue;
        }
        float* dst = p.dq_depth + ((size_t)(bh0 + j) * T + t) * D + l16 * 8;
        *(f32x4*)dst = (f32x4){dq[j][0], dq[j][1], dq[j][2], dq[j][3]};
        *(f32x4*)(dst + 4) = (f32x4){dq[j][4], dq[j][5], dq[j][6], dq[j][7]};
      }
  }
}

// The same rows as a kernel of its own: groups of 5 to 8 heads (those that do not take
// depth_group_rows, see own_depth_kernel).  The arithmetic per fetched byte grows with the group, and on
// the vector ALUs the dK/dV kernel cannot hide it (measured at 8 heads: there it costs what it costs alone).
template <int D, int GT>
__global__ __launch_bounds__(256, 2) void moda_bwd_depth_gqa_kernel(BwdParams p) {
  constexpr int LPR = D / 8, ROWS = 256 / LPR;
  const long long row = (long long)blockIdx.x * ROWS + threadIdx.x / LPR;  // (b * Hk + g) * T + t
  const long long n_rows = (long long)p.B * p.Hk * p.T;
  depth_gqa_row<D, GT>(p, row < n_rows ? row : n_rows - 1, row < n_rows, threadIdx.x % LPR);
}

// Two fp32 as three pairs of bf16 whose sum they are: the differences are exact, and three times 8 bits
// hold the 24 of a float.  (x, y) become what the last pair leaves: zero for numbers whose third part
// is representable, NaN where x is infinite, NaN or rounds to an infinite bf16.
__device__ __forceinline__ void split2(float& x, float& y, uint32_t (&part)[3]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    part[k] = pack_bf16(x, y);
    x -= bf16_lo(part[k]);
    y -= bf16_hi(part[k]);
  }
}

// ---------------------------------------------------------------- depth-slot gradients of 5 to 8 heads, matrix pipe
// The depth slots of ROWS consecutive positions (row0 ...) of one key/value head, handled by one
// wave, for groups of up to 8 heads (G): per position and 32 slots, as for the larger groups below,
//   S^T, dP^T (slots x heads) -> E^T -> dQ_p += E Kd_p,   S, dP (heads x slots) -> P, E -> dVd_p, dKd_p.
// On the vector ALUs (depth_gqa_row) the sums over heads and channels take longer than the slots
// take to arrive at this group size, and inside the dK/dV kernel they cost what they cost alone;
// here the vector ALUs only exponentiate, so that the phase is HBM's and the key-tile work of the
// workgroup next door goes on beside it.  B=1 Hq=64 Hk=8 T=16384 d=64, 64 slots: 1.13 ms in a kernel of
// its own + 4.46 -> 5.16 ms together (0.9 would be the 4.3 GB alone at the rate of a large copy).
// Columns (or rows) of the products past the group repeat heads that exist and get weight zero
// (lse = +inf).  The weights P and E enter the products as the sum of three bf16 numbers, i.e. with all
// their 24 bits: the contractions over the heads have room for the second number in the 8 of their 16
// places that no head takes and take a second matrix instruction for the third, the one over the slots
// takes three.  A weight that is infinite or NaN has no such sum: the positions that show one (a logit
// gradient E covers its P, Q, dO, K and V) are left to the vector ALUs at the end (depth_gqa_row).
// LDS of one wave: tiles of 32 rows of Kd and Vd (later of their gradients, so that those are stored
// row by row, 16 bytes per lane), of 8 rows of Q and dO.  The next 32 slots, and the next position's
// Q and dO, are in flight in registers meanwhile.
template <int D>
struct DepthWave {
  static constexpr int kKV = 32 * D * 2, kQ = 8 * D * 2;
  static constexpr int kBytes = 2 * kKV + 2 * kQ;
};

template <int D, int ROWS>
__device__ __forceinline__ void depth_group_rows(const BwdParams& p, int bg, int row0, int lane, unsigned lds) {
  using Tl = Tile<D>;
  using W = DepthWave<D>;
  constexpr int RB = D * 2, kInst = W::kKV / 1024, kQInst = W::kQ / 1024;
  const int l32 = lane & 31, hi = lane >> 5;
  const int T = p.T, L = p.depth_count, La = p.depth_alloc, G = p.Hq / p.Hk;
  const int bh0 = (bg / p.Hk) * p.Hq + (bg % p.Hk) * G;
  const int n_pos = min(ROWS, T - row0);
  if (n_pos <= 0) return;  // (wave-uniform)
  const float c2 = p.scale_log2;
  const unsigned k_tile = lds, v_tile = lds + W::kKV, q_tile = lds + 2 * W::kKV, g_tile = q_tile + W::kQ;
  const size_t drow = (size_t)La * RB;
  const size_t dbase = ((size_t)bg * T + row0) * drow;
  FragAddr<D> fa;
  fa.init(lane);
  const int q_row = Tl::off(l32 & 7, hi);
  // this lane's 16 bytes of a 1 KB piece: row j, chunk position pc (the permutation of piece q differs
  // by piece_xor(q) from piece 0's)
  const int j = lane / Tl::kChunks, pc = lane % Tl::kChunks;
  const int g_off = j * RB + ((pc ^ Tl::swz(j)) << 4);
  auto lds_at = [](unsigned a) { return (u32x4 __attribute__((address_space(3)))*)(size_t)a; };

  const int nch = (L + 31) / 32;
  u32x4 kn[kInst], vn[kInst], qn[kQInst], gn[kQInst];
  f32x2 sn;
  auto issue_kv = [&](int pos, int c) {
    const size_t base = dbase + (size_t)pos * drow;
    const __amdgpu_buffer_rsrc_t kb =
        __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)p.Kdepth + base), 0, L * RB, 0x00020000);
    const __amdgpu_buffer_rsrc_t vb =
        __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)p.Vdepth + base), 0, L * RB, 0x00020000);
#pragma unroll
    for (int q = 0; q < kInst; ++q) {  // (slots past depth_count are not fetched: zeros)
      const int voff = xor_here(g_off, TileLoader<D>::piece_xor(q));
      kn[q] = __builtin_amdgcn_raw_buffer_load_b128(kb, voff, c * W::kKV + q * 1024, 2);
      vn[q] = __builtin_amdgcn_raw_buffer_load_b128(vb, voff, c * W::kKV + q * 1024, 2);
    }
  };
  auto issue_q = [&](int pos) {
    const int t = row0 + pos;
#pragma unroll
    for (int q = 0; q < kQInst; ++q) {
      const int r = q * (1024 / RB) + j;
      const size_t off = ((size_t)(bh0 + min(r, G - 1)) * T + t) * RB + ((pc ^ Tl::swz(r)) << 4);
      qn[q] = *(const u32x4*)((const char*)p.Q + off);
      gn[q] = *(const u32x4*)((const char*)p.dO + off);
    }
    const size_t row = (size_t)(bh0 + min(l32, G - 1)) * T + t;
    sn = (f32x2){p.lse2[row], p.minus_delta[row]};
  };
  if (nch > 0) {
    issue_q(0);
    issue_kv(0, 0);
  }
  static_assert(ROWS <= 32, "one bit per position");
  unsigned again = 0;  // positions with weights that are not finite
  for (int pos = 0; pos < n_pos; ++pos) {
    const int t = row0 + pos;
    float not_finite = 0.f;  // zero, or NaN
    const i32x4 dk_buf = make_tile_buffer((const char*)p.dKdepth + dbase + (size_t)pos * drow, (unsigned)(L * RB));
    const i32x4 dv_buf = make_tile_buffer((const char*)p.dVdepth + dbase + (size_t)pos * drow, (unsigned)(L * RB));
    f32x16 dqa[Tl::kDBlocks];  // dQ^T (depth share): lane = head, registers = channels
#pragma unroll
    for (int cb = 0; cb < Tl::kDBlocks; ++cb)
#pragma unroll
      for (int i = 0; i < 16; ++i) dqa[cb][i] = 0.f;
    float lse2 = INFINITY, m_delta = 0.f, l4[4], d4[4];  // d4, m_delta: -delta
    if (nch > 0) {
#pragma unroll
      for (int q = 0; q < kQInst; ++q) {
        *lds_at(q_tile + q * 1024 + lane * 16) = qn[q];
        *lds_at(g_tile + q * 1024 + lane * 16) = gn[q];
      }
      lse2 = l32 < G ? sn[0] : INFINITY;
      m_delta = sn[1];
#pragma unroll
      for (int r = 0; r < 4; ++r) {  // heads 4 hi + r
        l4[r] = __shfl(lse2, hi * 4 + r, 64);
        d4[r] = __shfl(m_delta, hi * 4 + r, 64);
      }
      issue_q(min(pos + 1, n_pos - 1));
    }
    for (int c = 0; c < nch; ++c) {
#pragma unroll
      for (int q = 0; q < kInst; ++q) {
        *lds_at(k_tile + q * 1024 + lane * 16) = kn[q];
        *lds_at(v_tile + q * 1024 + lane * 16) = vn[q];
      }
      const bool last = c == nch - 1;  // (past the last position: its last slots again, not used)
      issue_kv(last ? min(pos + 1, n_pos - 1) : pos, last ? (pos + 1 < n_pos ? 0 : c) : c + 1);
      asm volatile("" ::: "memory");
      const int c0 = c * 32;
      // ---- slots x heads: E^T, dQ^T += Kd^T E^T
      {
        f32x16 s, dp;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = dp[i] = 0.f;
#pragma unroll
        for (int st = 0; st < Tl::kDSteps; ++st) {
          const unsigned xk = (unsigned)xor_here(fa.row + (int)k_tile, st << 5), xq = (unsigned)xor_here(q_row + (int)q_tile, st << 5);
          s = mfma_bf16(FragAddr<D>::row_frag(xk, 0, 0), FragAddr<D>::row_frag(xq, 0, 0), s);
          dp = mfma_bf16(FragAddr<D>::row_frag(xk, 0, W::kKV), FragAddr<D>::row_frag(xq, 0, W::kQ), dp);
        }
        float ev[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int slot = c0 + (i >> 2) * 8 + hi * 4 + (i & 3);
          const float pe = slot < L ? fast_exp2(s[i] * c2 - lse2) : 0.f;
          ev[i] = pe * (dp[i] + m_delta);
        }
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          u32x4 e[3];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            float& x = ev[hf * 8 + 2 * k];
            float& y = ev[hf * 8 + 2 * k + 1];
            uint32_t part[3];
            split2(x, y, part);
            not_finite = fmaf(x, 0.f, fmaf(y, 0.f, not_finite));
#pragma unroll
            for (int n = 0; n < 3; ++n) e[n][k] = part[n];
          }
#pragma unroll
          for (int cb = 0; cb < Tl::kDBlocks; ++cb) {
            const bf16x8 kt = FragAddr<D>::tr_frag((unsigned)xor_here(fa.tr + (int)k_tile, cb << 6),
                                                   (unsigned)xor_here(fa.tr8 + (int)k_tile, cb << 6), hf, 0);
#pragma unroll
            for (int n = 0; n < 3; ++n) dqa[cb] = mfma_bf16(kt, __builtin_bit_cast(bf16x8, e[n]), dqa[cb]);
          }
        }
      }
      // ---- heads x slots (lane = slot, registers 0..3 = heads 4 hi ..): P, E
      u32x4 pw[2], ew[2];  // [0] places 0..3: first numbers, 4..7: second numbers of the four heads; [1] third numbers
      {
        f32x16 s, dp;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = dp[i] = 0.f;
#pragma unroll
        for (int st = 0; st < Tl::kDSteps; ++st) {
          const unsigned xk = (unsigned)xor_here(fa.row + (int)k_tile, st << 5), xq = (unsigned)xor_here(q_row + (int)q_tile, st << 5);
          s = mfma_bf16(FragAddr<D>::row_frag(xq, 0, 0), FragAddr<D>::row_frag(xk, 0, 0), s);
          dp = mfma_bf16(FragAddr<D>::row_frag(xq, 0, W::kQ), FragAddr<D>::row_frag(xk, 0, W::kKV), dp);
        }
        const bool live = c0 + l32 < L;
        pw[1] = ew[1] = (u32x4){0u, 0u, 0u, 0u};
#pragma unroll
        for (int r = 0; r < 4; r += 2) {
          float pv[2], ev[2];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            pv[u] = live ? fast_exp2(s[r + u] * c2 - l4[r + u]) : 0.f;
            ev[u] = pv[u] * (dp[r + u] + d4[r + u]);
          }
          uint32_t part[3];
          split2(pv[0], pv[1], part);
          pw[0][r / 2] = part[0];
          pw[0][2 + r / 2] = part[1];
          pw[1][r / 2] = part[2];
          split2(ev[0], ev[1], part);
          ew[0][r / 2] = part[0];
          ew[0][2 + r / 2] = part[1];
          ew[1][r / 2] = part[2];
        }
      }
      // ---- dVd^T = dO^T P, dKd^T = Q^T E (lane = slot), bf16 rows through the tiles, stored 16 bytes a lane
      asm volatile("" ::: "memory");
      auto gradient = [&](unsigned src, const u32x4 (&w)[2], float f, unsigned tile, const i32x4& buf) {
#pragma unroll
        for (int cb = 0; cb < Tl::kDBlocks; ++cb) {
          // (one transposing read: 8 heads, for the first and for the second numbers, and for the third)
          const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (s16x4 __attribute__((address_space(3)))*)(size_t)(unsigned)xor_here(fa.tr + (int)src, cb << 6));
          f32x16 acc;
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
          for (int n = 0; n < 2; ++n)
            acc = mfma_bf16(__builtin_bit_cast(bf16x8, __builtin_shufflevector(a, a, 0, 1, 2, 3, 0, 1, 2, 3)),
                            __builtin_bit_cast(bf16x8, w[n]), acc);
#pragma unroll
          for (int bq = 0; bq < 4; ++bq)
            *(u32x2 __attribute__((address_space(3)))*)(size_t)(tile + Tl::off(l32, cb * 4 + bq) + hi * 8) =
                (u32x2){pack_bf16(acc[4 * bq] * f, acc[4 * bq + 1] * f), pack_bf16(acc[4 * bq + 2] * f, acc[4 * bq + 3] * f)};
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int q = 0; q < kInst; ++q) {  // (slots past depth_count lie outside the buffer: not stored)
          const u32x4 x = *lds_at(tile + q * 1024 + lane * 16);
          buffer_store16_nt(x, buf, xor_here(g_off, TileLoader<D>::piece_xor(q)),
                            __builtin_amdgcn_readfirstlane(c * W::kKV + q * 1024));
        }
      };
      gradient(g_tile, pw, 1.0f, v_tile, dv_buf);
      gradient(q_tile, ew, p.scale, k_tile, dk_buf);
      asm volatile("" ::: "memory");
    }
    // allocated but unattended slots get zero gradients
    for (int i = L * (RB / 16) + lane; i < La * (RB / 16); i += 64) {
      const u32x4 z = {0u, 0u, 0u, 0u};
      *(u32x4*)((char*)p.dKdepth + dbase + (size_t)pos * drow + (size_t)i * 16) = z;
      *(u32x4*)((char*)p.dVdepth + dbase + (size_t)pos * drow + (size_t)i * 16) = z;
    }
    if (l32 < G) {
      float* dst = p.dq_depth + ((size_t)(bh0 + l32) * T + t) * D;
#pragma unroll
      for (int cb = 0; cb < Tl::kDBlocks; ++cb)
#pragma unroll
        for (int bq = 0; bq < 4; ++bq)
          *(f32x4*)(dst + cb * 32 + bq * 8 + hi * 4) =
              (f32x4){dqa[cb][4 * bq], dqa[cb][4 * bq + 1], dqa[cb][4 * bq + 2], dqa[cb][4 * bq + 3]};
    }
    if (__builtin_amdgcn_ballot_w64(not_finite != not_finite) != 0) again |= 1u << pos;
  }
  if (again != 0) {  // (wave-uniform)
    constexpr int LPR = D / 8, RPS = 64 / LPR;
    wait_own_copies<0>();  // (the stores that are replaced have been made)
    for (int r0 = 0; r0 < n_pos; r0 += RPS) {
      const int r = r0 + lane / LPR;
      if (((again >> r0) & ((1u << RPS) - 1)) != 0)
        depth_gqa_row<D, 8>(p, (long long)bg * T + row0 + min(r, n_pos - 1), r < n_pos && ((again >> r) & 1u) != 0, lane % LPR);
    }
  }
}

// ---------------------------------------------------------------- dK, dV
// Workgroup = 128 keys (4 waves x 32 keys).  Accumulators hold dK^T, dV^T
// ([channel][key]: a lane owns one key and 64 of its channels).
// GT: 4, 8 = the depth-slot gradients of a group of up to GT heads are taken here as well (4:
// depth_gqa_row; 8, at d = 64: depth_group_rows); 0 = none here.
template <int D, int GT>
__device__ __forceinline__ void dkdv_tile(const BwdParams& p, unsigned char* smem, int bg, int jt) {
  using Tl = Tile<D>;
  using C = BwdCfg<D>;
  float* aux = (float*)(smem + C::kLds - C::kAux);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hi = lane >> 5;
  const int T = p.T;
  const int j0 = jt * 128;
  const int kw0 = j0 + wave * 32;
  const int G = p.Hq / p.Hk;        // query heads per key/value head: their gradients add up here
  const int bh0 = (bg / p.Hk) * p.Hq + (bg % p.Hk) * G;  // first query head of the group

  const char* Kb = (const char*)p.Kseq + (size_t)bg * T * Tl::kRowBytes;
  const char* Vb = (const char*)p.Vseq + (size_t)bg * T * Tl::kRowBytes;

  // ---- Depth-slot gradients: row-local, bound by HBM (every depth slot read once, every gradient written
  // once), and independent of everything else this kernel does, which is bound by the matrix
  // pipe and leaves HBM idle.  Each workgroup takes the 128 positions of its key tile, before
  // its key-tile work (every other workgroup) or after it, so that at any time some compute
  // units stream while others compute.
  const bool depth_first = ((blockIdx.x >> 3) & 1) != 0;
  // (the workgroup's 128 positions, 256 / (d/8) at a time)
  auto group_depth = [&]() {
    if constexpr (GT == 8) {
      __syncthreads();  // (the waves' parts of LDS are other waves' before and after)
      depth_group_rows<D, 32>(p, bg, kw0, lane, (unsigned)(size_t)(lds_ptr)smem + wave * DepthWave<D>::kBytes);
      wait_own_reads();
      __syncthreads();
    } else if constexpr (GT > 0) {
      constexpr int LPR = D / 8, ROWS = 256 / LPR;
      for (int r0 = 0; r0 < 128; r0 += ROWS) {
        if (j0 + r0 + wave * (64 / LPR) >= T) break;  // (whole waves)
        const int t = j0 + r0 + tid / LPR;
        depth_gqa_row<D, GT>(p, (long long)bg * T + min(t, T - 1), t < T, tid % LPR);
      }
    }
  };
  if (GT > 0 && depth_first) group_depth();

  // resident K and V fragments of this wave's 32 keys (MFMA B operands: N = key, K = channels)
  bf16x8 kf[Tl::kDSteps], vf[Tl::kDSteps];
  {
    const int row = min(kw0 + l32, T - 1);
#pragma unroll
    for (int st = 0; st < Tl::kDSteps; ++st) {
      kf[st] = *(const bf16x8*)(Kb + (size_t)row * Tl::kRowBytes + st * 32 + hi * 16);
      vf[st] = *(const bf16x8*)(Vb + (size_t)row * Tl::kRowBytes + st * 32 + hi * 16);
    }
  }
  f32x16 dk[Tl::kDBlocks], dv[Tl::kDBlocks];
#pragma unroll
  for (int db = 0; db < Tl::kDBlocks; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) dk[db][i] = dv[db][i] = 0.f;

  const int nq = (T + 63) / 64;
  const int qt0 = p.causal ? j0 / 64 : 0;
  const int span = nq - qt0;   // query tiles that see this key tile, per query head
  const int n_items = G * span;  // work items: (query head of the group, query tile)
  const float c2 = p.scale_log2;
  const unsigned smem_addr = (unsigned)(size_t)(lds_ptr)smem;
  TileLoader<D> ld;
  ld.init(wave, lane);
  FragAddr<D> fa;
  fa.init(lane);

  // Work items are walked by counters (head, query tile): a division per tile, and the buffers built anew,
  // were 60 scalar instructions between a tile's barrier and its first copy.
  i32x4 q_buf, do_buf, st_buf;  // (st_buf: of waves 0 and 1)
  auto at_head = [&](int h) {
    const size_t row = (size_t)(bh0 + h) * T;
    q_buf = make_tile_buffer((const char*)p.Q + row * Tl::kRowBytes, (unsigned)T * Tl::kRowBytes);
    do_buf = make_tile_buffer((const char*)p.dO + row * Tl::kRowBytes, (unsigned)T * Tl::kRowBytes);
    st_buf = make_tile_buffer((wave == 0 ? p.lse2 : p.minus_delta) + row, (unsigned)T * 4);
  };
  int next_head = 0, next_qt = qt0;
  auto issue_next = [&](int stage) {
    ld.issue(q_buf, next_qt * 64, smem_addr + stage * C::kStageBytes);
    ld.issue(do_buf, next_qt * 64, smem_addr + stage * C::kStageBytes + Tl::kBytes);
    // lse2 and -delta of the tile's 64 queries: 256 contiguous bytes each, copied like the tiles (no
    // load whose result a wave would have to wait for while the tile copies are in flight:
    // memory operations complete in order) by waves 0 and 1
    if (wave < 2) copy4(st_buf, lane * 4, next_qt * 256, smem_addr + (unsigned)(C::kLds - C::kAux) + stage * 512 + wave * 256);
    if (++next_qt == nq) {
      next_qt = qt0;
      if (++next_head < G) at_head(next_head);
    }
  };

  int qt = qt0;  // of the item at hand
  if (n_items > 0) {
    at_head(0);
    issue_next(0);
  }
  for (int item = 0; item < n_items; ++item, qt = qt + 1 == nq ? qt0 : qt + 1) {
    const int stage = item & 1;
    wait_copies();
    __syncthreads();
    if (item + 1 < n_items) issue_next(stage ^ 1);

    const int q0 = qt * 64;
    if (p.causal && q0 + 63 < kw0) continue;  // every query of the tile precedes this wave's keys
    // per-lane fragment bases inside this stage (Q tile; the dO tile sits Tl::kBytes after it)
    const unsigned qtile = smem_addr + stage * C::kStageBytes;
    const unsigned b_row = fa.row + qtile, b_tr = fa.tr + qtile, b_tr8 = fa.tr8 + qtile;
    const float* lse_s = aux + stage * 128;  // of the tile's queries
    const float* delta_s = lse_s + 64;       // (-delta)
    // -delta of the lane's queries of a 32-query block, in the order of the accumulators
    auto minus_delta = [&](int qb) {
      f32x16 r;
#pragma unroll
      for (int b4 = 0; b4 < 4; ++b4) {
        const f32x4 x = *(const f32x4*)(delta_s + qb * 32 + b4 * 8 + hi * 4);
        r[4 * b4] = x[0]; r[4 * b4 + 1] = x[1]; r[4 * b4 + 2] = x[2]; r[4 * b4 + 3] = x[3];
      }
      return r;
    };

    const int key = kw0 + l32;
    // all 64 queries exist and (when causal) none precedes any of this wave's 32 keys
    const bool all_visible = q0 + 64 <= T && (!p.causal || q0 >= kw0 + 31);
    if constexpr (D == 64) {
      // Registers allow two 32-query blocks in flight: the exponentials of one are issued, four at a
      // time, between the matrix instructions of the other (its scores, then the first block's output
      // products), in whose shadow the vector ALUs then work.  The order is pinned step by step.
      // (Matrix and vector time of this kernel used to add up: 45 % matrix-pipe busy.  B=1 Hq=64 Hk=8
      // T=16384: 4.74 ms one block at a time; 4.61 so; 4.39 with the wave priority below, 1.0 PFLOP/s.)
      f32x16 s[2], dp[2];        // S, dP - delta
      u32x4 pb[2][2], ds[2][2];  // P and dS packed to bf16: [block][16-query half]
      auto mask = [&](int qb) {  // (a uniform branch around the comparisons, as below)
        if (!all_visible) {
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int q = q0 + qb * 32 + (i >> 2) * 8 + hi * 4 + (i & 3);
            const bool vis = q < T && (!p.causal || key <= q);
            s[qb][i] = vis ? s[qb][i] : -INFINITY;
          }
        }
      };
      // LSE log2 e of the lane's queries 4 b4 .. + 3 of a block
      f32x4 l4;
      auto read_stat = [&](int qb, int b4) { l4 = *(const f32x4*)(lse_s + qb * 32 + b4 * 8 + hi * 4); };
      // ... and their P and dS
      auto weights = [&](int qb, int b4) {
        float pv[4], dsv[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          pv[r] = fast_exp2(s[qb][b4 * 4 + r] * c2 - l4[r]);
          dsv[r] = pv[r] * dp[qb][b4 * 4 + r];
        }
        uint32_t o[4] = {pack_bf16(pv[0], pv[1]), pack_bf16(pv[2], pv[3]), pack_bf16(dsv[0], dsv[1]),
                         pack_bf16(dsv[2], dsv[3])};
        // (used here: else the computation sinks to the block of its products)
        asm volatile("" : "+v"(o[0]), "+v"(o[1]), "+v"(o[2]), "+v"(o[3]));
        pb[qb][b4 >> 1][(b4 & 1) * 2] = o[0];
        pb[qb][b4 >> 1][(b4 & 1) * 2 + 1] = o[1];
        ds[qb][b4 >> 1][(b4 & 1) * 2] = o[2];
        ds[qb][b4 >> 1][(b4 & 1) * 2 + 1] = o[3];
      };
      // Sixteen steps of two matrix instructions: 0..3 scores of block 0, 4..7 of block 1 (with the
      // weights of block 0), 8..11 products of block 0 (with the weights of block 1; 16-query half
      // (n - 8) / 2, channel block n % 2), 12..15 products of block 1.  Fragments are read two steps
      // ahead, the weights' row scalars one.
      bf16x8 fq[3], fg[3];
      auto read_frags = [&](int n) {
        if (n < 8) {
          const unsigned x = (unsigned)xor_here((int)b_row, (n & 3) << 5);
          fq[n % 3] = fa.row_frag(x, n >> 2, 0);
          fg[n % 3] = fa.row_frag(x, n >> 2, Tl::kBytes);
        } else {
          const int db = n & 1, ks = (n - 8) >> 1;
          const unsigned x0 = (unsigned)xor_here((int)b_tr, db << 6), x8 = (unsigned)xor_here((int)b_tr8, db << 6);
          fq[n % 3] = fa.tr_frag(x0, x8, ks, 0);
          fg[n % 3] = fa.tr_frag(x0, x8, ks, Tl::kBytes);
        }
      };
      dp[0] = minus_delta(0);
      read_frags(0);
      read_frags(1);
#pragma unroll
      for (int n = 0; n < 16; ++n) {
        if (n == 2) dp[1] = minus_delta(1);
        // (the wave whose instructions fill both pipes goes first; the other wave of the SIMD takes
        // what is left)
        if (n == 4) __builtin_amdgcn_s_setprio(1);
        if (n == 12) __builtin_amdgcn_s_setprio(0);
        if (n < 14) read_frags(n + 2);
        if (n < 8) {
          const int qb = n >> 2, st = n & 3;
          if (st == 0)
#pragma unroll
            for (int i = 0; i < 16; ++i) s[qb][i] = 0.f;
          s[qb] = mfma_bf16(fq[n % 3], kf[st], s[qb]);
          dp[qb] = mfma_bf16(fg[n % 3], vf[st], dp[qb]);
        } else {
          const int qb = (n - 8) >> 2, hf = ((n - 8) >> 1) & 1, db = n & 1;
          dv[db] = mfma_bf16(fg[n % 3], __builtin_bit_cast(bf16x8, pb[qb][hf]), dv[db]);
          dk[db] = mfma_bf16(fq[n % 3], __builtin_bit_cast(bf16x8, ds[qb][hf]), dk[db]);
        }
        if (n >= 4 && n < 12) weights((n - 4) >> 2, n & 3);
        if (n >= 3 && n < 11) read_stat((n - 3) >> 2, (n - 3) & 3);
        __builtin_amdgcn_sched_barrier(0);
        if (n == 3) mask(0);
        if (n == 7) mask(1);
      }
    } else {
      // one 32-query block at a time: S, dP (recomputed), P and dS for this lane's key and
      // 16 queries, then dV^T += dO^T P and dK^T += Q^T dS over those 32 queries
  #pragma unroll
      for (int qb = 0; qb < 2; ++qb) {
        f32x16 s, dp = minus_delta(qb);
  #pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = 0.f;
  #pragma unroll
        for (int st = 0; st < Tl::kDSteps; ++st) {
          const unsigned x = (unsigned)xor_here((int)b_row, st << 5);
          s = mfma_bf16(fa.row_frag(x, qb, 0), kf[st], s);
          dp = mfma_bf16(fa.row_frag(x, qb, Tl::kBytes), vf[st], dp);
        }
        // Order for the scheduler: LDS reads run one step (two fragments) ahead of the matrix
        // instructions that consume them, no further (the kernel has no registers to spare).
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
  #pragma unroll
        for (int st = 0; st < Tl::kDSteps - 2; ++st) {
          __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
        __builtin_amdgcn_sched_barrier(0);
        // Scores of (query, key) pairs that are not visible become -inf, i.e. weight zero.  Only
        // the diagonal tile and rows past the end have such pairs: everywhere else this block is
        // skipped (a uniform branch around the comparisons, not a second copy of the loop body).
        if (!all_visible) {
  #pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int q = q0 + qb * 32 + (i >> 2) * 8 + hi * 4 + (i & 3);
            const bool vis = q < T && (!p.causal || key <= q);
            s[i] = vis ? s[i] : -INFINITY;
          }
        }
        // one 16-query half at a time: P and dS packed to bf16, then straight into the products
        // that contract over those 16 queries (keeps few temporaries alive)
  #pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          float pv[8], dsv[8];
  #pragma unroll
          for (int b2 = 0; b2 < 2; ++b2) {
            const int b4 = hf * 2 + b2;
            const f32x4 l4 = *(const f32x4*)(lse_s + qb * 32 + b4 * 8 + hi * 4);
  #pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int i = b4 * 4 + r;
              const float pe = fast_exp2(s[i] * c2 - l4[r]);
              pv[b2 * 4 + r] = pe;
              dsv[b2 * 4 + r] = pe * dp[i];
            }
          }
          const bf16x8 pb = pack8(pv), dsb = pack8(dsv);
  #pragma unroll
          for (int db = 0; db < Tl::kDBlocks; ++db) {
            const unsigned x0 = (unsigned)xor_here((int)b_tr, db << 6), x8 = (unsigned)xor_here((int)b_tr8, db << 6);
            dv[db] = mfma_bf16(fa.tr_frag(x0, x8, qb * 2 + hf, Tl::kBytes), pb, dv[db]);
            dk[db] = mfma_bf16(fa.tr_frag(x0, x8, qb * 2 + hf, 0), dsb, dk[db]);
          }

        }
      }
    }
  }
  __syncthreads();

  // ---- write out: accumulator layout -> row-major through LDS, 16-byte stores
  unsigned char* xw = smem + wave * C::kXWave;
  constexpr int LPR = Tl::kChunks, RPS = 64 / LPR;
  const int rg = lane / LPR, l16 = lane % LPR;
#pragma unroll
  for (int which = 0; which < 2; ++which) {
#pragma unroll
    for (int db = 0; db < Tl::kDBlocks; ++db)
#pragma unroll
      for (int bq = 0; bq < 4; ++bq) {
        const f32x16& acc = which ? dv[db] : dk[db];
        f32x4 v = {acc[4 * bq], acc[4 * bq + 1], acc[4 * bq + 2], acc[4 * bq + 3]};
        *(f32x4*)(xw + l32 * C::kXRow + (db * 32 + bq * 8 + hi * 4) * 4) = v;
      }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    char* outb = (char*)(which ? p.dVseq : p.dKseq) + (size_t)bg * T * Tl::kRowBytes;
    const float f = which ? 1.0f : p.scale;
    for (int it = 0; it < 32 / RPS; ++it) {
      const int row = it * RPS + rg;
      const int key = kw0 + row;
      const f32x4 o0 = *(const f32x4*)(xw + row * C::kXRow + l16 * 32);
      const f32x4 o1 = *(const f32x4*)(xw + row * C::kXRow + l16 * 32 + 16);
      if (key < T) {
        u32x4 ov = {pack_bf16(o0[0] * f, o0[1] * f), pack_bf16(o0[2] * f, o0[3] * f),
                    pack_bf16(o1[0] * f, o1[1] * f), pack_bf16(o1[2] * f, o1[3] * f)};
        *(u32x4*)(outb + (size_t)key * Tl::kRowBytes + l16 * 16) = ov;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  if (GT > 0 && !depth_first) group_depth();
}

template <int D, int GT>
__global__ __launch_bounds__(256, 2) void moda_bwd_dkdv_kernel(BwdParams p) {
  using C = BwdCfg<D>;
  constexpr int kSmem = GT == 8 && 4 * DepthWave<D>::kBytes > C::kLds ? 4 * DepthWave<D>::kBytes : C::kLds;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kSmem];
  int bg, jt;  // (batch, key/value head); key tiles in natural order: the first ones see the most queries
  head_blocked_id(layered_id(p.causal, 2), p.B * p.Hk, (p.T + 127) / 128, bg, jt, p.head_group);
  dkdv_tile<D, GT>(p, smem, bg, jt);
}

// ---------------------------------------------------------------- dK, dV, few key tiles
// The kernel above needs B * Hk * T / 128 workgroups to fill the chip; below that most compute units
// idle while the first key tiles walk all query tiles of the group one after the other.  Here a
// workgroup = 32 keys and its 4 or 8 waves (NW) DEAL OUT THE QUERIES: item i, 32 queries of one head of the
// group, belongs to wave i % NW, which copies its Q / dO rows and their (LSE, delta) into LDS of its
// own (two stages, no workgroup barrier in the loop); their dK^T, dV^T are summed through LDS at
// the end, in wave order.  Four times the workgroups with a quarter of the steps each, for four
// times the reads of Q and dO, which the L2 serves.  The depth slots of the 32 positions are taken
// here as well.
// Bound by the latency of a wave's serial chain copy -> products -> exponentials -> products:
// B=2 Hq=16 Hk=8 T=1000 d=64, 12 slots: 82 -> 34 us; whole backward call at B=1 Hq=64 Hk=8 T=1024
// d=64, 64 slots: 293 -> 160 us, d=128: 530 -> 282 us.
// Eight waves (d = 64; the LDS of a unit holds one such workgroup, or two of four waves): the first key tiles,
// which see all queries of a large group, take half as long, where they are what the call waits for.  Backward
// call, 4 / 8 waves, us: B=1 Hq=8 Hk=1 T=16384 1404 / 1035; Hq=64 Hk=8 T=1000 75.5 / 60.8; Hq=32 Hk=4 T=3000, 24
// slots 260 / 220; but Hq=16 Hk=8 B=2 T=1000, 12 slots 46.1 / 50.9 (dkdv_waves draws the line).
template <int D, int NW = 4, int ST = 2>
struct BwdShortCfg {
  static constexpr int kStages = ST;
  static constexpr int kTile = 32 * D * 2;               // 32 rows of Q or dO
  static constexpr int kStage = 2 * kTile + 64 * 8;      // Q, dO, LSE log2 e, -delta (of 64 rows, 32 of them used)
  static constexpr int kPieces = kTile / 1024;           // copy instructions per tile
  static constexpr int kXRow = D + 4;                    // floats per row of the exchange buffer
  static constexpr int kXWave = 32 * kXRow;
  static constexpr int kRing = NW * ST * kStage;
  static constexpr int kLds = kRing > NW * kXWave * 4 ? kRing : NW * kXWave * 4;
};

// GT: 1, 2, 4 = the depth slots of the 32 positions are taken here as well, of groups of up to GT heads; 0 = not here.
// ST: stages of a wave's Q and dO tiles.  With one (in the launch with dQ, four waves, and eight at d = 128) Q's place is requested anew as soon as
// dK is formed and dO's after dV: half the LDS, so that at d = 128 two workgroups share a unit and at d = 64
// three.  (dK, dV and dQ in one launch, two stages / one, us: B=4 Hq=8 Hk=2 T=901 d=128 61 / 54; B=2 H=16 T=657 d=128 55 / 40;
// B=4 Hq=32 Hk=8 T=719 d=64, 4 slots 71 / 62.)
template <int D, int GT, int NW, int ST>
__device__ __forceinline__ void dkdv_short_tile(const BwdParams& p, unsigned char* smem, int bg, int jt) {
  using Tl = Tile<D>;
  using C = BwdShortCfg<D, NW, ST>;
  using Ld = TileLoader<D>;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hi = lane >> 5;
  const int T = p.T, G = p.Hq / p.Hk;
  const int j0 = jt * 32;
  const int bh0 = (bg / p.Hk) * p.Hq + (bg % p.Hk) * G;
  const float c2 = p.scale_log2;

  // depth slots of the 32 positions, before or after the key tile (alternating, as above)
  auto depth = [&]() {
    if constexpr (GT > 1) {
      constexpr int LPR = D / 8, ROWS = NW * 64 / LPR;
      for (int r0 = 0; r0 < 32; r0 += ROWS) {
        if (j0 + r0 + wave * (64 / LPR) >= T) break;  // (whole waves)
        const int t = j0 + r0 + tid / LPR;
        if (ROWS > 32 && t >= j0 + 32) break;  // (whole waves)
        depth_gqa_row<D, GT>(p, (long long)bg * T + min(t, T - 1), t < T, tid % LPR);
      }
    } else if constexpr (GT == 1) {
      if (wave < 4) depth_grad_rows<D, 8>(p, bg, j0 + wave * 8, lane);
    }
  };
  const bool depth_first = ((blockIdx.x >> 3) & 1) != 0;
  if (depth_first) depth();

  bf16x8 kf[Tl::kDSteps], vf[Tl::kDSteps];
  {
    const size_t row = ((size_t)bg * T + min(j0 + l32, T - 1)) * Tl::kRowBytes + hi * 16;
#pragma unroll
    for (int st = 0; st < Tl::kDSteps; ++st) {
      kf[st] = *(const bf16x8*)((const char*)p.Kseq + row + st * 32);
      vf[st] = *(const bf16x8*)((const char*)p.Vseq + row + st * 32);
    }
  }
  f32x16 dk[Tl::kDBlocks], dv[Tl::kDBlocks];
#pragma unroll
  for (int db = 0; db < Tl::kDBlocks; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) dk[db][i] = dv[db][i] = 0.f;

  const int qt0 = p.causal ? jt : 0;
  const int span = (T + 31) / 32 - qt0;
  const int n_items = G * span;
  const unsigned ring = (unsigned)(size_t)(lds_ptr)smem + wave * ST * C::kStage;
  FragAddr<D> fa;
  fa.init(lane);
  const int goff = (lane / Tl::kChunks) * Tl::kRowBytes + (((lane % Tl::kChunks) ^ Tl::swz(lane / Tl::kChunks)) << 4);
  // (items are walked by counters, as above: head and query tile, counted from qt0, of the next item to request)
  int head = 0, pos = wave;
  i32x4 q_buf, do_buf, l_buf, d_buf;
  auto at_head = [&]() {
    const size_t row = (size_t)(bh0 + head) * T;
    q_buf = make_tile_buffer((const char*)p.Q + row * Tl::kRowBytes, (unsigned)T * Tl::kRowBytes);
    do_buf = make_tile_buffer((const char*)p.dO + row * Tl::kRowBytes, (unsigned)T * Tl::kRowBytes);
    l_buf = make_tile_buffer(p.lse2 + row, (unsigned)T * 4);
    d_buf = make_tile_buffer(p.minus_delta + row, (unsigned)T * 4);
  };
  int next = 0;  // query tile of the next item
  auto advance = [&]() {
    if (pos >= span) {
      do {
        pos -= span;
        ++head;
      } while (pos >= span);
      at_head();
    }
    next = qt0 + pos;
    pos += NW;
  };
  auto issue_rows = [&](unsigned dst) {
    copy4(l_buf, lane * 4, next * 128, dst + 2 * C::kTile);
    copy4(d_buf, lane * 4, next * 128, dst + 2 * C::kTile + 256);
  };
  auto issue_tile = [&](const i32x4& buf, unsigned dst) {
#pragma unroll
    for (int q = 0; q < C::kPieces; ++q)
      tile_copy16(buf, xor_here(goff, Ld::piece_xor(q)), next * C::kTile + q * 1024, dst + q * 1024);
  };
  auto issue_q = [&]() {  // (one stage)
    issue_tile(q_buf, ring);
    issue_rows(ring);
  };
  auto issue_do = [&]() { issue_tile(do_buf, ring + C::kTile); };
  auto issue = [&](int stage) {
    if constexpr (ST == 1) {
      issue_q();
      issue_do();
    } else {  // (an offset serves both tiles)
      const unsigned dst = ring + stage * C::kStage;
#pragma unroll
      for (int q = 0; q < C::kPieces; ++q) {
        const int voff = xor_here(goff, Ld::piece_xor(q));
        tile_copy16(q_buf, voff, next * C::kTile + q * 1024, dst + q * 1024);
        tile_copy16(do_buf, voff, next * C::kTile + q * 1024, dst + C::kTile + q * 1024);
      }
      issue_rows(dst);
    }
  };
  if (wave < n_items) {
    at_head();
    advance();
    issue(0);
  }
  int stage = 0;
  for (int item = wave; item < n_items; item += NW, stage ^= ST - 1) {
    // (the wave's own copies into its own LDS: its wait publishes them, and the stage that the next
    // copies overwrite may be refilled as soon as the wave's reads of it have returned)
    const bool more = item + NW < n_items;
    const int q0 = next * 32;
    if constexpr (ST == 2) {
      wait_own_copies<0>();
      wait_own_reads();
      if (more) {
        advance();
        issue(stage ^ 1);
      }
    } else {
      wait_own_copies<C::kPieces>();  // (dO may still be on its way)
    }
    const unsigned qtile = ring + stage * C::kStage;
    const unsigned b_row = fa.row + qtile, b_tr = fa.tr + qtile, b_tr8 = fa.tr8 + qtile;
    const float* lse_s = (const float*)(smem + (qtile - (unsigned)(size_t)(lds_ptr)smem) + 2 * C::kTile);
    f32x16 s, dp;  // S, dP - delta
#pragma unroll
    for (int b4 = 0; b4 < 4; ++b4) {
      const f32x4 x = *(const f32x4*)(lse_s + 64 + b4 * 8 + hi * 4);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[4 * b4 + r] = 0.f;
        dp[4 * b4 + r] = x[r];
      }
    }
    if constexpr (ST == 1) {
#pragma unroll
      for (int st = 0; st < Tl::kDSteps; ++st)
        s = mfma_bf16(FragAddr<D>::row_frag((unsigned)xor_here((int)b_row, st << 5), 0, 0), kf[st], s);
      wait_own_copies<0>();
#pragma unroll
      for (int st = 0; st < Tl::kDSteps; ++st)
        dp = mfma_bf16(FragAddr<D>::row_frag((unsigned)xor_here((int)b_row, st << 5), 0, C::kTile), vf[st], dp);
    } else {
#pragma unroll
      for (int st = 0; st < Tl::kDSteps; ++st) {
        const unsigned x = (unsigned)xor_here((int)b_row, st << 5);
        s = mfma_bf16(FragAddr<D>::row_frag(x, 0, 0), kf[st], s);
        dp = mfma_bf16(FragAddr<D>::row_frag(x, 0, C::kTile), vf[st], dp);
      }
    }
    if (q0 + 32 > T || (p.causal && q0 < j0 + 31)) {  // (uniform) the diagonal, rows past the end
      const int key = j0 + l32;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int q = q0 + (i >> 2) * 8 + hi * 4 + (i & 3);
        s[i] = q < T && (!p.causal || key <= q) ? s[i] : -INFINITY;
      }
    }
    bf16x8 pb[2], dsb[2];
    auto weights = [&](int hf) {
      float pv[8], dsv[8];
#pragma unroll
      for (int b2 = 0; b2 < 2; ++b2) {
        const int b4 = hf * 2 + b2;
        const f32x4 l4 = *(const f32x4*)(lse_s + b4 * 8 + hi * 4);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = b4 * 4 + r;
          const float pe = fast_exp2(s[i] * c2 - l4[r]);
          pv[b2 * 4 + r] = pe;
          dsv[b2 * 4 + r] = pe * dp[i];
        }
      }
      pb[hf] = pack8(pv);
      dsb[hf] = pack8(dsv);
    };
    auto product = [&](int hf, int db, bool of_v, bool of_k) {
      const unsigned x0 = (unsigned)xor_here((int)b_tr, db << 6), x8 = (unsigned)xor_here((int)b_tr8, db << 6);
      if (of_v) dv[db] = mfma_bf16(FragAddr<D>::tr_frag(x0, x8, hf, C::kTile), pb[hf], dv[db]);
      if (of_k) dk[db] = mfma_bf16(FragAddr<D>::tr_frag(x0, x8, hf, 0), dsb[hf], dk[db]);
    };
    if constexpr (ST == 1) {  // Q's place is free, and requested anew, before dO's
      weights(0);
      weights(1);
#pragma unroll
      for (int n = 0; n < 2 * Tl::kDBlocks; ++n) product(n / Tl::kDBlocks, n % Tl::kDBlocks, false, true);
      wait_own_reads();
      if (more) {
        advance();
        issue_q();
      }
#pragma unroll
      for (int n = 0; n < 2 * Tl::kDBlocks; ++n) product(n / Tl::kDBlocks, n % Tl::kDBlocks, true, false);
      wait_own_reads();
      if (more) issue_do();
    } else {
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        weights(hf);
#pragma unroll
        for (int db = 0; db < Tl::kDBlocks; ++db) product(hf, db, true, true);
      }
    }
  }

  // ---- sum of the waves, row-major, 16-byte stores
  float* xb = (float*)smem;
  constexpr int LPR = Tl::kChunks;
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    __syncthreads();
#pragma unroll
    for (int db = 0; db < Tl::kDBlocks; ++db)
#pragma unroll
      for (int bq = 0; bq < 4; ++bq) {
        const f32x16& acc = which ? dv[db] : dk[db];
        *(f32x4*)(xb + wave * C::kXWave + l32 * C::kXRow + db * 32 + bq * 8 + hi * 4) =
            (f32x4){acc[4 * bq], acc[4 * bq + 1], acc[4 * bq + 2], acc[4 * bq + 3]};
      }
    __syncthreads();
    char* outb = (char*)(which ? p.dVseq : p.dKseq) + (size_t)bg * T * Tl::kRowBytes;
    const float f = which ? 1.0f : p.scale;
    for (int row = tid / LPR; row < 32; row += NW * 64 / LPR) {
      const float* x = xb + row * C::kXRow + (tid % LPR) * 8;
      f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        a += *(const f32x4*)(x + w * C::kXWave);
        b += *(const f32x4*)(x + w * C::kXWave + 4);
      }
      if (j0 + row < T)
        *(u32x4*)(outb + (size_t)(j0 + row) * Tl::kRowBytes + (tid % LPR) * 16) =
            (u32x4){pack_bf16(a[0] * f, a[1] * f), pack_bf16(a[2] * f, a[3] * f), pack_bf16(b[0] * f, b[1] * f),
                    pack_bf16(b[2] * f, b[3] * f)};
    }
  }
  if (!depth_first) depth();
}

template <int D, int GT, int NW>
__global__ __launch_bounds__(NW * 64, D == 64 ? 2 : 1) void moda_bwd_dkdv_short_kernel(BwdParams p) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[BwdShortCfg<D, NW>::kLds];
  int bg, jt;  // (batch, key/value head); key tiles in natural order: the first ones see the most queries
  head_blocked_id((int)blockIdx.x, p.B * p.Hk, (p.T + 31) / 32, bg, jt, p.head_group);
  dkdv_short_tile<D, GT, NW, 2>(p, smem, bg, jt);
}

// ---------------------------------------------------------------- dQ
// Workgroup = NW waves x 32 queries.  Accumulators hold dQ^T ([channel][query]: a lane owns
// one query).  Launched with NW = 4 (two workgroups per compute unit); NW = 8 (one workgroup
// per unit, a K/V tile serving twice as many queries) measured 6 % slower at B=8 H=16 T=4096.
// PS: workgroups per compute unit, i.e. waves per SIMD: 2, or at d = 64 3 (dq_per_unit draws the line).
// A tile is kQT / heads positions (from q0 on) of `heads` query heads (from bh0 on) of a group.
// GT: 1, 2, 4 = the depth slots of the tile's positions, which then has all heads of the group, are taken here,
// before the key tiles or (depth_first false) after them; 0 = their share of dQ, if there are any, is in the workspace.
template <int D, int NW, int PS, int GT>
__device__ __forceinline__ void dq_tile(const BwdParams& p, unsigned char* smem, int bg, int bh0, int heads, int q0, bool depth_first) {
  using Tl = Tile<D>;
  using C = BwdCfg<D, NW>;
  constexpr int kQT = NW * 32;  // queries per workgroup
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hi = lane >> 5;
  const int T = p.T;
  const int n_pos = kQT / heads;
  const int bh = bh0 + wave % heads;
  const int qw0 = q0 + wave / heads * 32;

  const char* Qb = (const char*)p.Q + (size_t)bh * T * Tl::kRowBytes;
  const char* Kb = (const char*)p.Kseq + (size_t)bg * T * Tl::kRowBytes;
  const char* Vb = (const char*)p.Vseq + (size_t)bg * T * Tl::kRowBytes;
  const char* dOb = (const char*)p.dO + (size_t)bh * T * Tl::kRowBytes;

  const int qi = qw0 + l32;
  const int qrow = min(qi, T - 1);

  const float c2 = p.scale_log2;
  unsigned char* xw = smem + wave * C::kXWave;  // this wave's fp32 exchange buffer (overlaps the ring)
  constexpr int LPR = Tl::kChunks, RPS = 64 / LPR, NIT = 32 / RPS;
  const int La = p.depth_alloc;

  // GT = 0: the depth-slot gradients and the depth share of dQ were computed before this kernel (by
  // the dK/dV kernel, or by the depth_gqa kernels with grouped queries).  GT > 0: they are computed here, the share
  // of a tile that takes its slots first through the workspace too: in fp32, not yet multiplied by the softmax scale.
  constexpr int kDepthRows = NW * 64 / LPR;  // rows of depth slots per pass
  if constexpr (GT > 0) {
    if (depth_first) {
      if constexpr (GT == 1) depth_grad_rows<D, 32>(p, bh, qw0, lane);
      else
        for (int r0 = 0; r0 < kQT / GT; r0 += kDepthRows) {
          if (q0 + r0 + wave * (64 / LPR) >= T) break;  // (whole waves)
          const int t = q0 + r0 + tid / LPR;
          depth_gqa_row<D, GT>(p, (long long)bg * T + min(t, T - 1), t < T, tid % LPR);
        }
      __syncthreads();
    }
  }
  f32x16 dq[Tl::kDBlocks];
  if (GT > 0 ? depth_first : La > 0) {
    const float* src = p.dq_depth + ((size_t)bh * T + qrow) * D;
#pragma unroll
    for (int db = 0; db < Tl::kDBlocks; ++db)
#pragma unroll
      for (int bq = 0; bq < 4; ++bq) {
        const f32x4 v = *(const f32x4*)(src + db * 32 + bq * 8 + hi * 4);
        dq[db][4 * bq] = v[0]; dq[db][4 * bq + 1] = v[1];
        dq[db][4 * bq + 2] = v[2]; dq[db][4 * bq + 3] = v[3];
      }
  } else {
#pragma unroll
    for (int db = 0; db < Tl::kDBlocks; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) dq[db][i] = 0.f;
  }

  // resident Q and dO fragments of this wave's 32 queries (MFMA B operands)
  bf16x8 qf[Tl::kDSteps], dof[Tl::kDSteps];
#pragma unroll
  for (int st = 0; st < Tl::kDSteps; ++st) {
    qf[st] = *(const bf16x8*)(Qb + (size_t)qrow * Tl::kRowBytes + st * 32 + hi * 16);
    dof[st] = *(const bf16x8*)(dOb + (size_t)qrow * Tl::kRowBytes + st * 32 + hi * 16);
  }
  const float lse2 = p.lse2[(size_t)bh * T + qrow], md = p.minus_delta[(size_t)bh * T + qrow];
  // dP - delta comes out of the matrix pipe: its accumulators start from here.  (Three waves per SIMD have no registers
  // to keep that: formed anew for every block.)
  auto minus_delta = [&]() {
    float x = md;
    if constexpr (PS > 2) asm volatile("" : "+v"(x));
    f32x16 r;
#pragma unroll
    for (int i = 0; i < 16; ++i) r[i] = x;
    return r;
  };

  const int n_keys = p.causal ? min(T, q0 + n_pos) : T;
  const int nt = (n_keys + 63) / 64;
  const int wave_last = p.causal ? min(nt - 1, (qw0 + 31) / 64) : nt - 1;
  const int lim = p.causal ? min(qi, T - 1) : T - 1;  // last visible key of this lane's query
  const int n_visible = p.causal ? min(T, qw0 + 1) : T;  // keys that exist and that every query of the wave sees
  const unsigned smem_addr = (unsigned)(size_t)(lds_ptr)smem;
  TileLoader<D, NW> ld;
  ld.init(wave, lane);
  FragAddr<D> fa;
  fa.init(lane);
  const i32x4 k_buf = make_tile_buffer(Kb, (unsigned)T * Tl::kRowBytes);
  const i32x4 v_buf = make_tile_buffer(Vb, (unsigned)T * Tl::kRowBytes);
  auto issue = [&](int kt, int stage) {
    ld.issue(k_buf, kt * 64, smem_addr + stage * C::kStageBytes);
    ld.issue(v_buf, kt * 64, smem_addr + stage * C::kStageBytes + Tl::kBytes);
  };

  // One key tile, or (BLOCKS = 1) its first 32 keys: S^T, dP^T, dS^T and dQ^T += K^T dS^T for this wave's 32 queries.
  auto tile = [&](int kt, int stage, auto blocks) {
    constexpr int BLOCKS = decltype(blocks)::value;
    // per-lane fragment bases inside this stage (K tile; the V tile sits Tl::kBytes after it)
    const unsigned ktile = smem_addr + stage * C::kStageBytes;
    const unsigned b_row = fa.row + ktile, b_tr = fa.tr + ktile, b_tr8 = fa.tr8 + ktile;

    f32x16 s[2], dp[2];  // S^T, dP^T - delta: [key block]; a lane holds 16 keys of its query
    u32x4 ds[2][2];      // dS^T packed to bf16: [key block][16-key half]
    const int k0 = kt * 64;
    const bool all_visible = k0 + 64 <= n_visible;
    auto mask = [&](int kb) {
      if (!all_visible) {  // (uniform) diagonal tile, keys past the end: invisible pairs get weight zero
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int key = k0 + kb * 32 + (i >> 2) * 8 + hi * 4 + (i & 3);
          s[kb][i] = key <= lim ? s[kb][i] : -INFINITY;
        }
      }
    };
    auto weights = [&](int kb, int b4) {  // dS of the lane's keys 4 b4 .. + 3 of a block
      float a[4];
#pragma unroll
      for (int r = 0; r < 4; ++r)
        a[r] = fast_exp2(s[kb][b4 * 4 + r] * c2 - lse2) * dp[kb][b4 * 4 + r];
      uint32_t o[2] = {pack_bf16(a[0], a[1]), pack_bf16(a[2], a[3])};
      asm volatile("" : "+v"(o[0]), "+v"(o[1]));  // (used here: else the computation sinks to its products)
      ds[kb][b4 >> 1][(b4 & 1) * 2] = o[0];
      ds[kb][b4 >> 1][(b4 & 1) * 2 + 1] = o[1];
    };
    // Steps: the scores of key block 0 (two matrix instructions each); those of block 1, with the
    // exponentials of block 0 between them; the products dQ^T += K^T dS^T of block 0 (one matrix
    // instruction each), with the exponentials of block 1; the products of block 1.  The vector ALUs
    // thus work in the shadow of the matrix pipe for half of the tile.  Fragments are read kAhead
    // steps ahead; the order is pinned step by step.  (Against scores, exponentials, products one
    // after the other: B=8 H=16 T=4096 d=128 0.88 -> 0.83 ms; B=1 Hq=64 Hk=8 T=16384 d=64 3.01 ->
    // 2.97 ms, where 1.11 PFLOP/s of matrix work hold the clock at 1.7 GHz.)
    constexpr int NS = Tl::kDSteps, NP = 2 * Tl::kDBlocks, kAhead = 2, kBuf = kAhead + 1, kScores = BLOCKS * NS, kSteps = kScores + BLOCKS * NP;
    bf16x8 fk[kBuf], fv[kBuf];
    auto read_frags = [&](int n) {
      if (n < kScores) {
        const unsigned x = (unsigned)xor_here((int)b_row, (n % NS) << 5);
        fk[n % kBuf] = fa.row_frag(x, n / NS, 0);
        fv[n % kBuf] = fa.row_frag(x, n / NS, Tl::kBytes);
      } else if (n < kSteps) {
        const int m = n - kScores, db = m % Tl::kDBlocks;
        fk[n % kBuf] = fa.tr_frag((unsigned)xor_here((int)b_tr, db << 6), (unsigned)xor_here((int)b_tr8, db << 6),
                                  m / Tl::kDBlocks, 0);
      }
    };
#pragma unroll
    for (int n = 0; n < kAhead; ++n) read_frags(n);
#pragma unroll
    for (int n = 0; n < kSteps; ++n) {
      if (BLOCKS == 2 && n == NS) __builtin_amdgcn_s_setprio(1);  // (as in the dK/dV kernel)
      if (BLOCKS == 2 && n == 2 * NS + NP) __builtin_amdgcn_s_setprio(0);
      read_frags(n + kAhead);
      if (n < kScores) {
        const int kb = n / NS, st = n % NS;
        if (st == 0)
#pragma unroll
          for (int i = 0; i < 16; ++i) s[kb][i] = 0.f;
        s[kb] = mfma_bf16(fk[n % kBuf], qf[st], s[kb]);
        dp[kb] = mfma_bf16(fv[n % kBuf], dof[st], st == 0 ? minus_delta() : dp[kb]);
        if (kb == 1 && st % (NS / 4) == 0) weights(0, st / (NS / 4));
      } else {
        const int m = n - kScores, ks = m / Tl::kDBlocks, db = m % Tl::kDBlocks;
        dq[db] = mfma_bf16(fk[n % kBuf], __builtin_bit_cast(bf16x8, ds[ks >> 1][ks & 1]), dq[db]);
        if (BLOCKS == 2 && m < NP && m % (NP / 4) == 0) weights(1, m / (NP / 4));
      }
      __builtin_amdgcn_sched_barrier(0);
      if (n == NS - 1) mask(0);
      if (BLOCKS == 1 && n == NS - 1) {
#pragma unroll
        for (int b4 = 0; b4 < 4; ++b4) weights(0, b4);
      }
      if (BLOCKS == 2 && n == 2 * NS - 1) mask(1);
    }
  };

  // Every wave takes part in the copies and barriers of all nt tiles, but computes only on the
  // tiles its queries see: first those (no branch around the products inside the loop, which
  // made the compiler copy the accumulators from one register block to another every tile),
  // then the rest.
  // Of the tile of its own positions a wave whose 32 queries are the first ones sees the first 32 keys only: the others stay out of
  // its products, where weights of zero would turn values that are not finite into NaN.
  const bool half = p.causal && (qw0 & 32) == 0;
  issue(0, 0);
  int kt = 0;
  auto next = [&]() {
    wait_copies();
    __syncthreads();
    if (kt + 1 < nt) issue(kt + 1, (kt & 1) ^ 1);
  };
  for (; kt <= wave_last - (half ? 1 : 0); ++kt) {
    next();
    tile(kt, kt & 1, std::integral_constant<int, 2>());
  }
  if (half && kt <= wave_last) {
    next();
    tile(kt, kt & 1, std::integral_constant<int, 1>());
    ++kt;
  }
  for (; kt < nt; ++kt) {
    wait_copies();
    __syncthreads();
    if (kt + 1 < nt) issue(kt + 1, (kt & 1) ^ 1);
  }
  __syncthreads();

  // ---- epilogue: accumulator layout -> row-major; depth slots (unless taken first); stores
#pragma unroll
  for (int db = 0; db < Tl::kDBlocks; ++db)
#pragma unroll
    for (int bq = 0; bq < 4; ++bq) {
      f32x4 v = {dq[db][4 * bq], dq[db][4 * bq + 1], dq[db][4 * bq + 2], dq[db][4 * bq + 3]};
      *(f32x4*)(xw + l32 * C::kXRow + (db * 32 + bq * 8 + hi * 4) * 4) = v;
    }
  if constexpr (GT > 0) {
    if (!depth_first) {
      __syncthreads();
      if constexpr (GT == 1) depth_grad_rows<D, 32, 5, C::kXRow>(p, bh, qw0, lane, xw);
      else
        for (int r0 = 0; r0 < kQT / GT; r0 += kDepthRows) {
          if (q0 + r0 + wave * (64 / LPR) >= T) break;
          const int r = r0 + tid / LPR, t = q0 + r;
          depth_gqa_row<D, GT, 4, C::kXRow, C::kXWave>(p, (long long)bg * T + min(t, T - 1), t < T, tid % LPR,
                                                    smem + r / 32 * GT * C::kXWave + r % 32 * C::kXRow);
        }
      return;
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  {
    const int rg = lane / LPR, l16 = lane % LPR;
    char* dQb = (char*)p.dQ + (size_t)bh * T * Tl::kRowBytes;
    for (int it = 0; it < NIT; ++it) {
      const int row = it * RPS + rg, t = qw0 + row;
      const f32x4 a0 = *(const f32x4*)(xw + row * C::kXRow + l16 * 32);
      const f32x4 a1 = *(const f32x4*)(xw + row * C::kXRow + l16 * 32 + 16);
      if (t < T) {
        const float f = p.scale;
        u32x4 ov = {pack_bf16(a0[0] * f, a0[1] * f), pack_bf16(a0[2] * f, a0[3] * f),
                    pack_bf16(a1[0] * f, a1[1] * f), pack_bf16(a1[2] * f, a1[3] * f)};
        *(u32x4*)(dQb + (size_t)t * Tl::kRowBytes + l16 * 16) = ov;
      }
    }
  }
}

template <int D, int NW, int PS>
__global__ __launch_bounds__(NW * 64, PS) void moda_bwd_dq_kernel(BwdParams p) {
  using C = BwdCfg<D, NW>;
  constexpr int kQT = NW * 32;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[C::kLds];
  const int n_qt = (p.T + kQT - 1) / kQT;
  // Ids are dealt to the dies by key/value head (see head_blocked_id): the G query heads of a
  // group stream the same K/V, so a die takes a group's heads one right after the other, query
  // tile by query tile (heavy, i.e. late, tiles first).
  const int G = p.Hq / p.Hk;
  int bg, tile_idx;  // (batch, key/value head); position in the walk over (query tile, head of the group)
  head_blocked_id(layered_id(p.causal, PS), p.B * p.Hk, n_qt * G, bg, tile_idx, p.head_group);
  dq_tile<D, NW, PS, 0>(p, smem, bg, (bg / p.Hk) * p.Hq + (bg % p.Hk) * G + tile_idx % G, 1, (n_qt - 1 - tile_idx / G) * kQT, false);
}

// ---------------------------------------------------------------- dQ, few query tiles
// The same change of split for dQ when the kernel above would have fewer workgroups than the chip
// takes: a workgroup = 32 queries, its 4 waves deal out the key tiles (32 keys, private LDS stages),
// the four dQ^T and the depth share are summed at the end.
// Whole backward call, B=1 H=8 T=2048, 4 slots: d=64 59 -> 46 us, d=128 97 -> 80 us; B=1 H=2
// T=16384: d=64 365 -> 320 us, d=128 712 -> 636 us.
// One LDS tile of K and one of V per wave (V is requested anew as soon as the scores are formed, K after
// the products): twice the workgroups fit a compute unit that did with two stages.
// A tile is 32 positions of `heads` (1, 2 or 4) query heads of a group: each has 4 / heads of the waves.  GT: as in dq_tile.
template <int D, int GT, int CH, int AHEAD, int NW = 4>
__device__ __forceinline__ void dq_short_tile(const BwdParams& p, unsigned char* smem, int bg, int bh0, int heads, int q0, bool depth_first) {
  using Tl = Tile<D>;
  using C = BwdShortCfg<D>;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hi = lane >> 5;
  const int T = p.T;
  const int bh = bh0 + wave % heads, wave0 = wave / heads, per_head = NW / heads;
  const float c2 = p.scale_log2;

  const int nt = ((p.causal ? min(T, q0 + 32) : T) + 31) / 32;
  const unsigned ktile = (unsigned)(size_t)(lds_ptr)smem + wave * 2 * C::kTile, vtile = ktile + C::kTile;
  FragAddr<D> fa;
  fa.init(lane);
  const i32x4 k_buf = make_tile_buffer((const char*)p.Kseq + (size_t)bg * T * Tl::kRowBytes, (unsigned)T * Tl::kRowBytes);
  const i32x4 v_buf = make_tile_buffer((const char*)p.Vseq + (size_t)bg * T * Tl::kRowBytes, (unsigned)T * Tl::kRowBytes);
  const int goff = (lane / Tl::kChunks) * Tl::kRowBytes + (((lane % Tl::kChunks) ^ Tl::swz(lane / Tl::kChunks)) << 4);
  auto issue = [&](const i32x4& buf, int kt, unsigned dst) {  // (tiles past the end: zeros)
#pragma unroll
    for (int q = 0; q < C::kPieces; ++q)
      tile_copy16(buf, xor_here(goff, TileLoader<D>::piece_xor(q)), (int)((unsigned)kt * (unsigned)C::kTile) + q * 1024,
                  dst + q * 1024);
  };
  constexpr int LPR = Tl::kChunks, ROWS = NW * 64 / LPR;
  constexpr int kRows = NW * 64 / LPR > 32 ? 64 / LPR : 32 / NW;  // rows of slots per wave
  if constexpr (GT > 0) {
    if (depth_first) {
      if constexpr (GT == 1) {
        if (wave * kRows < 32) depth_grad_rows<D, kRows, CH>(p, bh, q0 + wave * kRows, lane);
      }
      else
        for (int r0 = 0; r0 < 32; r0 += ROWS) {
          if (q0 + r0 + wave * (64 / LPR) >= T) break;  // (whole waves)
          const int t = q0 + r0 + tid / LPR;
          if (ROWS > 32 && r0 + tid / LPR >= 32) break;  // (whole waves)
          depth_gqa_row<D, GT, AHEAD>(p, (long long)bg * T + min(t, T - 1), t < T, tid % LPR);
        }
    }
  }
  if (wave0 < nt) {
    issue(k_buf, wave0, ktile);
    issue(v_buf, wave0, vtile);
  }

  const int qrow = min(q0 + l32, T - 1);
  bf16x8 qf[Tl::kDSteps], dof[Tl::kDSteps];
  {
    const size_t row = ((size_t)bh * T + qrow) * Tl::kRowBytes + hi * 16;
#pragma unroll
    for (int st = 0; st < Tl::kDSteps; ++st) {
      qf[st] = *(const bf16x8*)((const char*)p.Q + row + st * 32);
      dof[st] = *(const bf16x8*)((const char*)p.dO + row + st * 32);
    }
  }
  const float lse2 = p.lse2[(size_t)bh * T + qrow], md = p.minus_delta[(size_t)bh * T + qrow];
  f32x16 minus_delta;  // (as above)
#pragma unroll
  for (int i = 0; i < 16; ++i) minus_delta[i] = md;
  const int lim = p.causal ? qrow : T - 1;  // last visible key of this lane's query
  f32x16 dq[Tl::kDBlocks];
#pragma unroll
  for (int db = 0; db < Tl::kDBlocks; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) dq[db][i] = 0.f;

  const unsigned b_row = fa.row + ktile, b_tr = fa.tr + ktile, b_tr8 = fa.tr8 + ktile;
  for (int kt = wave0; kt < nt; kt += per_head) {
    wait_own_copies<0>();
    f32x16 s, dp = minus_delta;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
    for (int st = 0; st < Tl::kDSteps; ++st) {
      const unsigned x = (unsigned)xor_here((int)b_row, st << 5);
      s = mfma_bf16(FragAddr<D>::row_frag(x, 0, 0), qf[st], s);
      dp = mfma_bf16(FragAddr<D>::row_frag(x, 0, C::kTile), dof[st], dp);
    }
    wait_own_reads();
    if (kt + per_head < nt) issue(v_buf, kt + per_head, vtile);
    const int k0 = kt * 32;
    if (k0 + 32 > T || (p.causal && k0 + 31 > q0)) {  // (uniform) the diagonal, keys past the end
#pragma unroll
      for (int i = 0; i < 16; ++i)
        s[i] = k0 + (i >> 2) * 8 + hi * 4 + (i & 3) <= lim ? s[i] : -INFINITY;
    }
    float ds[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) ds[i] = fast_exp2(s[i] * c2 - lse2) * dp[i];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      float a[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) a[k] = ds[hf * 8 + k];
      const bf16x8 dsb = pack8(a);
#pragma unroll
      for (int db = 0; db < Tl::kDBlocks; ++db)
        dq[db] = mfma_bf16(FragAddr<D>::tr_frag((unsigned)xor_here((int)b_tr, db << 6), (unsigned)xor_here((int)b_tr8, db << 6),
                                                hf, 0), dsb, dq[db]);
    }
    wait_own_reads();
    if (kt + per_head < nt) issue(k_buf, kt + per_head, ktile);
  }

  // ---- depth share + the four waves, row-major, 16-byte stores
  __syncthreads();
  float* xb = (float*)smem;
#pragma unroll
  for (int db = 0; db < Tl::kDBlocks; ++db)
#pragma unroll
    for (int bq = 0; bq < 4; ++bq)
      *(f32x4*)(xb + wave * C::kXWave + l32 * C::kXRow + db * 32 + bq * 8 + hi * 4) =
          (f32x4){dq[db][4 * bq], dq[db][4 * bq + 1], dq[db][4 * bq + 2], dq[db][4 * bq + 3]};
  __syncthreads();
  if constexpr (GT > 0) {
    if (!depth_first) {
      constexpr int XROW = C::kXRow * 4, XWAVE = C::kXWave * 4;
      if constexpr (GT == 1) {
        if (wave * kRows < 32) depth_grad_rows<D, kRows, CH, XROW, NW, XWAVE>(p, bh, q0 + wave * kRows, lane, smem + wave * kRows * XROW);
      }
      else
        for (int r0 = 0; r0 < 32; r0 += ROWS) {
          if (q0 + r0 + wave * (64 / LPR) >= T) break;
          const int r = r0 + tid / LPR, t = q0 + r;
          if (ROWS > 32 && r >= 32) break;
          depth_gqa_row<D, GT, AHEAD, XROW, XWAVE, NW / GT, GT * XWAVE>(p, (long long)bg * T + min(t, T - 1), t < T, tid % LPR, smem + r * XROW);
        }
      return;
    }
  }
  for (int r = tid / LPR; r < 32 * heads; r += ROWS) {
    const int row = r % 32, h = r / 32, t = q0 + row, ch = (tid % LPR) * 8;
    if (t >= T) continue;
    const size_t at = (size_t)(bh0 + h) * T + t;
    f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
    if (p.depth_alloc > 0) {
      const float* share = p.dq_depth + at * D + ch;
      a = *(const f32x4*)share;
      b = *(const f32x4*)(share + 4);
    }
    const float* x = xb + row * C::kXRow + ch;
    for (int w = h; w < NW; w += heads) {
      a += *(const f32x4*)(x + w * C::kXWave);
      b += *(const f32x4*)(x + w * C::kXWave + 4);
    }
    const float f = p.scale;
    *(u32x4*)((char*)p.dQ + at * Tl::kRowBytes + ch * 2) =
        (u32x4){pack_bf16(a[0] * f, a[1] * f), pack_bf16(a[2] * f, a[3] * f), pack_bf16(b[0] * f, b[1] * f),
                pack_bf16(b[2] * f, b[3] * f)};
  }
}

template <int D, int NW = 4>
struct DqShortCfg {
  using C = BwdShortCfg<D>;
  static constexpr int kTiles = NW * 2 * C::kTile, kExchange = NW * C::kXWave * 4;
  static constexpr int kLds = kTiles > kExchange ? kTiles : kExchange;
};
template <int D>
__global__ __launch_bounds__(256, D == 64 ? 4 : 2) void moda_bwd_dq_short_kernel(BwdParams p) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[DqShortCfg<D>::kLds];
  const int G = p.Hq / p.Hk, n_qt = (p.T + 31) / 32;
  int bg, tile_idx;  // (as above: a group's heads one right after the other, late query tiles first)
  head_blocked_id((int)blockIdx.x, p.B * p.Hk, n_qt * G, bg, tile_idx, p.head_group);
  dq_short_tile<D, 0, 5, 4>(p, smem, bg, (bg / p.Hk) * p.Hq + (bg % p.Hk) * G + tile_idx % G, 1, (n_qt - 1 - tile_idx / G) * 32, false);
}

// ---------------------------------------------------------------- dK, dV and dQ in one launch
// One after the other, the two kernels each end with a last round that leaves units idle, and in grids of one
// round with their longest workgroups alone; and the depth slots, bound by HBM, ran beside the products of dK and dV only.
// Here a workgroup is a key tile (dK, dV; all of them first, the heaviest ones in front) or a query tile (dQ, late
// ones first), and the depth slots of a query tile's positions are taken by its workgroup, so that nothing passes
// between workgroups: a tile is 128 / G positions of all G heads of the group (few queries: 32 positions).  The first
// quarter of the query tiles takes its slots first, while key tiles keep the matrix pipe busy, the others after their keys,
// straight into the finished row.
// Key tiles of 128 keys or (KS) 32 dealt out to the waves, query tiles of 128 rows or (QS) 32 positions dealt out; eight
// waves instead of four (NW, with KS) where few tiles have long walks: grads_plan draws the lines.
// Backward call, two launches / one: B=8 H=16 T=4096 d=128, 15 slots 2.80 / 2.65 ms; B=2 Hq=16 Hk=8 T=1000 d=64, 12
// slots 58 / 45 us; B=2 H=16 T=1105 d=128, 1 slot 104 / 64; B=2 H=2 T=206 d=128, 12 slots 25 / 17; B=1 Hq=4 Hk=1 T=4026 d=128, 64
// slots 290 / 220; B=3 Hq=8 Hk=2 T=71 d=128, 1 slot 23.3 / 14.8.  0.80 (d = 64) and 0.72 (d = 128) on average of the 34800
// shapes that grads_plan is fitted to.
// All key tiles first / one every so often among the query tiles, largest share first: within 2 % of the best order;
// the first quarter / half / eighth / none of the query tiles with slots first 1.018 / 1.024 / 1.020 / 1.029 of the best.
// Three waves per SIMD (170 registers) also for four heads, whose slots then park 7 registers in scratch memory: with two waves
// 250 calls took 0.97 of the time on average, but 59 of them longer, up to 1.26.
constexpr int grads_waves_per_simd(int D, bool KS, bool QS, int NW) { return D == 64 && KS && QS && NW == 4 ? 3 : 2; }
template <int D, bool KS, bool QS, int NW>
struct GradsCfg {
  static constexpr int kPerSimd = grads_waves_per_simd(D, KS, QS, NW);
  static constexpr int kStages = NW == 8 && D == 64 ? 2 : 1;               // of a wave's Q and dO tiles (KS)
  static constexpr int kKeyLds = KS ? BwdShortCfg<D, NW, kStages>::kLds : BwdCfg<D>::kLds;
  static constexpr int kQueryLds = QS ? DqShortCfg<D, NW>::kLds : BwdCfg<D, NW>::kLds;
  static constexpr int kLds = kKeyLds > kQueryLds ? kKeyLds : kQueryLds;
};
template <int D, int GT, bool KS, bool QS, int NW>
__global__ __launch_bounds__(NW * 64, (grads_waves_per_simd(D, KS, QS, NW))) void moda_bwd_grads_kernel(BwdParams p, int heads, int spread) {
  using C = GradsCfg<D, KS, QS, NW>;
  constexpr int kKeys = KS ? 32 : 128;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[C::kLds];
  const int G = p.Hq / p.Hk, sub = G / heads, n_pos = QS ? 32 : NW * 32 / heads;
  const int n_kt = (p.T + kKeys - 1) / kKeys, n_qt = (p.T + n_pos - 1) / n_pos;
  int bg, w;
  // (a unit holds one workgroup of eight waves: LDS)
  head_walk_id(QS ? (int)blockIdx.x : layered_id(p.causal, NW == 8 ? 1 : 2), p.B * p.Hk, n_kt + n_qt * sub, bg, w, p.head_group);
  int kt = w, qi = w - n_kt;
  if (spread) {  // key tiles evenly among the query tiles
    const unsigned long long m = n_kt + (long long)n_qt * sub;
    kt = (int)((unsigned long long)(unsigned)w * n_kt / m);
    if ((int)((w + 1ull) * n_kt / m) == kt) {
      qi = w - kt;
      kt = n_kt;
    }
  }
  if (kt < n_kt) {
    if constexpr (KS) dkdv_short_tile<D, 0, NW, C::kStages>(p, smem, bg, kt);
    else dkdv_tile<D, 0>(p, smem, bg, kt);
    return;
  }
  const int bh0 = (bg / p.Hk) * p.Hq + (bg % p.Hk) * G + qi % sub * heads, q0 = (n_qt - 1 - qi / sub) * n_pos;
  const bool depth_first = qi * 4 < n_qt;
  if constexpr (QS) dq_short_tile<D, GT, C::kPerSimd == 3 ? 3 : 5, C::kPerSimd == 3 && GT == 4 ? 2 : 4, NW>(p, smem, bg, bh0, heads, q0, depth_first);
  else dq_tile<D, NW, 2, GT>(p, smem, bg, bh0, heads, q0, depth_first);
}

// ---------------------------------------------------------------- depth-slot gradients of a large group, matrix pipe
// Groups of more than 8 query heads (8 < G <= 64; the G * T rows of Q of a group must fit 32-bit
// byte offsets, else the call is rejected as unsupported).
// With that many heads per position the depth-slot gradients of ONE position are small dense
// products (the paper's group-aware depth calculation, here for the backward):
//   S  = Q_p Kd_p^T   [G x L]    dP = dO_p Vd_p^T
//   P  = exp2(S c2 - lse2_h),    E  = P (dP - delta_h)
//   dVd_p = P^T dO_p  [L x d],   dKd_p = scale E^T Q_p,   dQ_p (depth share) = E Kd_p  [G x d]
// One workgroup of ONE wave per (batch, key/value head, position).  The G heads' Q and dO rows
// of the position (rows of different heads, gathered) and 64 slots at a time of Kd_p, Vd_p are
// copied global -> LDS into four 64-row tiles of the layout the other backward kernels use;
// the score products are formed in both orientations (slots x heads for the product that
// contracts over slots, heads x slots for the two that contract over heads), exactly as the
// dK/dV and dQ kernels do for sequence keys.  Rows of the tiles beyond G heads / beyond
// depth_count slots are filled with zeros by the bounds-checked copies (unattended slots are
// never fetched) and get weight zero.  Sums in fp32 on the matrix pipe, one rounding per
// gradient element.  Several such workgroups share a compute unit (32 KB of LDS each at d = 64),
// which is what hides the latency of the copies.
template <int D, int NG>
__global__ __launch_bounds__(64) void moda_bwd_depth_group_kernel(BwdParams p) {
  using Tl = Tile<D>;
  constexpr int RB = D * 2;
  constexpr int kRowsPerInst = 1024 / RB;       // rows one copy instruction moves
  constexpr int kInst = 64 / kRowsPerInst;      // copy instructions per tile
  constexpr int kStatOff = 4 * Tl::kBytes;      // (lse2, -delta) per head row, after the four tiles
  __shared__ __attribute__((aligned(1024))) unsigned char smem[4 * Tl::kBytes + 64 * 8];
  const int lane = threadIdx.x, l32 = lane & 31, hi = lane >> 5;
  const int T = p.T, L = p.depth_count, La = p.depth_alloc, G = p.Hq / p.Hk;
  const long long row = blockIdx.x;  // (b * Hk + g) * T + t
  const int t = (int)(row % T);
  const int bg = (int)(row / T);
  const int bh0 = (bg / p.Hk) * p.Hq + (bg % p.Hk) * G;
  const float c2 = p.scale_log2;
  const unsigned smem_addr = (unsigned)(size_t)(lds_ptr)smem;
  const unsigned q_tile = smem_addr, g_tile = smem_addr + Tl::kBytes, k_tile = smem_addr + 2 * Tl::kBytes,
                 v_tile = smem_addr + 3 * Tl::kBytes;
  float* stat = (float*)(smem + kStatOff);
  FragAddr<D> fa;
  fa.init(lane);

  // ---- the heads' rows of this position: row h of the tile = head h of the group
  const int j = lane / Tl::kChunks, pc = lane % Tl::kChunks;  // this lane's row in a piece, chunk position
  {
    const size_t base = ((size_t)bh0 * T + t) * RB;
    const unsigned bytes = (unsigned)(((size_t)(G - 1) * T + 1) * RB);  // (< 0xffffff00, below the offset that stands for "no row": checked by the host)
    const i32x4 q_buf = make_tile_buffer((const char*)p.Q + base, bytes);
    const i32x4 g_buf = make_tile_buffer((const char*)p.dO + base, bytes);
#pragma unroll
    for (int q = 0; q < kInst; ++q) {
      const int h = q * kRowsPerInst + j;
      const int c = pc ^ Tl::swz(h);
      const int voff = h < G ? (int)((unsigned)h * (unsigned)T * (unsigned)RB + (unsigned)c * 16u) : (int)0xffffff80u;
      tile_copy16(q_buf, voff, 0, q_tile + q * 1024);
      tile_copy16(g_buf, voff, 0, g_tile + q * 1024);
    }
    // heads past the group get lse2 = +inf: weight zero
    const int h = lane;
    f32x2 st = {INFINITY, 0.f};
    const size_t row = (size_t)(bh0 + min(h, G - 1)) * T + t;
    if (h < G) st = (f32x2){p.lse2[row], p.minus_delta[row]};
    *(f32x2*)(stat + 2 * h) = st;
  }
  f32x16 dqa[NG][Tl::kDBlocks];  // dQ^T (depth share): [head block][channel block], lane = head
#pragma unroll
  for (int hb = 0; hb < NG; ++hb)
#pragma unroll
    for (int cb = 0; cb < Tl::kDBlocks; ++cb)
#pragma unroll
      for (int i = 0; i < 16; ++i) dqa[hb][cb][i] = 0.f;

  const size_t drow = (size_t)La * RB;
  const char* kd = (const char*)p.Kdepth + (size_t)row * drow;
  const char* vd = (const char*)p.Vdepth + (size_t)row * drow;
  char* dkd = (char*)p.dKdepth + (size_t)row * drow;
  char* dvd = (char*)p.dVdepth + (size_t)row * drow;

  for (int c0 = 0; c0 < L; c0 += 64) {
    // ---- 64 slots of this position (rows past depth_count: zeros)
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the fragment reads of the chunk before are complete
    __builtin_amdgcn_wave_barrier();
    {
      const unsigned bytes = (unsigned)(min(64, L - c0) * RB);
      const i32x4 k_buf = make_tile_buffer(kd + (size_t)c0 * RB, bytes);
      const i32x4 v_buf = make_tile_buffer(vd + (size_t)c0 * RB, bytes);
#pragma unroll
      for (int q = 0; q < kInst; ++q) {
        const int r = q * kRowsPerInst + j;
        const int voff = r * RB + ((pc ^ Tl::swz(r)) << 4);
        tile_copy16(k_buf, voff, 0, k_tile + q * 1024);
        tile_copy16(v_buf, voff, 0, v_tile + q * 1024);
      }
    }
    wait_copies();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const unsigned bq_row = fa.row + q_tile, bq_tr = fa.tr + q_tile, bq_tr8 = fa.tr8 + q_tile;
    const unsigned bk_row = fa.row + k_tile, bk_tr = fa.tr + k_tile, bk_tr8 = fa.tr8 + k_tile;
    constexpr int kGOff = Tl::kBytes;  // the dO tile follows the Q tile, the Vd tile the Kd tile

#pragma unroll
    for (int sb = 0; sb < 2; ++sb) {
      if (c0 + sb * 32 >= L) break;  // (uniform) no attended slot in this block
      // dVd^T, dKd^T of the block's 32 slots: [channel block], lane = slot
      f32x16 dva[Tl::kDBlocks], dka[Tl::kDBlocks];
#pragma unroll
      for (int cb = 0; cb < Tl::kDBlocks; ++cb)
#pragma unroll
        for (int i = 0; i < 16; ++i) dva[cb][i] = dka[cb][i] = 0.f;
#pragma unroll
      for (int hb = 0; hb < NG; ++hb) {
        if (hb * 32 >= G) break;  // (uniform)
        // ---- slots x heads: S^T, dP^T (lane = head, registers = slots) -> E^T -> dQ^T += Kd^T E^T
        {
          f32x16 s, dp;
#pragma unroll
          for (int i = 0; i < 16; ++i) s[i] = dp[i] = 0.f;
#pragma unroll
          for (int st = 0; st < Tl::kDSteps; ++st) {
            const unsigned xk = (unsigned)xor_here((int)bk_row, st << 5), xq = (unsigned)xor_here((int)bq_row, st << 5);
            s = mfma_bf16(FragAddr<D>::row_frag(xk, sb, 0), FragAddr<D>::row_frag(xq, hb, 0), s);
            dp = mfma_bf16(FragAddr<D>::row_frag(xk, sb, kGOff), FragAddr<D>::row_frag(xq, hb, kGOff), dp);
          }
          const f32x2 st_h = *(const f32x2*)(stat + 2 * (hb * 32 + l32));  // this lane's head
          float ev[16];
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int slot = c0 + sb * 32 + (i >> 2) * 8 + hi * 4 + (i & 3);
            const float pe = slot < L ? fast_exp2(s[i] * c2 - st_h[0]) : 0.f;
            ev[i] = pe * (dp[i] + st_h[1]);
          }
#pragma unroll
          for (int hf = 0; hf < 2; ++hf) {
            float a8[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) a8[k] = ev[hf * 8 + k];
            const bf16x8 eb = pack8(a8);
#pragma unroll
            for (int cb = 0; cb < Tl::kDBlocks; ++cb)
              dqa[hb][cb] = mfma_bf16(FragAddr<D>::tr_frag((unsigned)xor_here((int)bk_tr, cb << 6),
                                                           (unsigned)xor_here((int)bk_tr8, cb << 6), sb * 2 + hf, 0),
                                      eb, dqa[hb][cb]);
          }
        }
        // ---- heads x slots: S, dP (lane = slot, registers = heads) -> P, E -> dVd^T += dO^T P, dKd^T += Q^T E
        {
          f32x16 s, dp;
#pragma unroll
          for (int i = 0; i < 16; ++i) s[i] = dp[i] = 0.f;
#pragma unroll
          for (int st = 0; st < Tl::kDSteps; ++st) {
            const unsigned xk = (unsigned)xor_here((int)bk_row, st << 5), xq = (unsigned)xor_here((int)bq_row, st << 5);
            s = mfma_bf16(FragAddr<D>::row_frag(xq, hb, 0), FragAddr<D>::row_frag(xk, sb, 0), s);
            dp = mfma_bf16(FragAddr<D>::row_frag(xq, hb, kGOff), FragAddr<D>::row_frag(xk, sb, kGOff), dp);
          }
          const bool live = c0 + sb * 32 + l32 < L;  // this lane's slot is attended
#pragma unroll
          for (int hf = 0; hf < 2; ++hf) {
            float pv[8], evv[8];
#pragma unroll
            for (int b2 = 0; b2 < 2; ++b2) {
              const int b4 = hf * 2 + b2;
              const float* st4 = stat + (hb * 32 + b4 * 8 + hi * 4) * 2;
              const f32x4 ld01 = *(const f32x4*)st4, ld23 = *(const f32x4*)(st4 + 4);
              const float l4[4] = {ld01[0], ld01[2], ld23[0], ld23[2]};
              const float d4[4] = {ld01[1], ld01[3], ld23[1], ld23[3]};
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const int i = b4 * 4 + r;
                const float pe = live ? fast_exp2(s[i] * c2 - l4[r]) : 0.f;
                pv[b2 * 4 + r] = pe;
                evv[b2 * 4 + r] = pe * (dp[i] + d4[r]);  // (d4: -delta)
              }
            }
            const bf16x8 pb = pack8(pv), eb = pack8(evv);
#pragma unroll
            for (int cb = 0; cb < Tl::kDBlocks; ++cb) {
              const unsigned x0 = (unsigned)xor_here((int)bq_tr, cb << 6), x8 = (unsigned)xor_here((int)bq_tr8, cb << 6);
              dva[cb] = mfma_bf16(FragAddr<D>::tr_frag(x0, x8, hb * 2 + hf, kGOff), pb, dva[cb]);
              dka[cb] = mfma_bf16(FragAddr<D>::tr_frag(x0, x8, hb * 2 + hf, 0), eb, dka[cb]);
            }
          }
        }
      }
      // ---- store the block's dVdepth, dKdepth rows: lane = slot, 4 consecutive channels (8 bytes) at a time
      const int slot = c0 + sb * 32 + l32;
      if (slot < L) {
        const float f = p.scale;
#pragma unroll
        for (int cb = 0; cb < Tl::kDBlocks; ++cb)
#pragma unroll
          for (int bq = 0; bq < 4; ++bq) {
            const size_t off = (size_t)slot * RB + (cb * 32 + bq * 8 + hi * 4) * 2;
            *(u32x2*)(dvd + off) = (u32x2){pack_bf16(dva[cb][4 * bq], dva[cb][4 * bq + 1]),
                                           pack_bf16(dva[cb][4 * bq + 2], dva[cb][4 * bq + 3])};
            *(u32x2*)(dkd + off) = (u32x2){pack_bf16(dka[cb][4 * bq] * f, dka[cb][4 * bq + 1] * f),
                                           pack_bf16(dka[cb][4 * bq + 2] * f, dka[cb][4 * bq + 3] * f)};
          }
      }
    }
  }
  // allocated but unattended slots get zero gradients
  for (int i = L * (RB / 16) + lane; i < La * (RB / 16); i += 64) {
    *(u32x4*)(dvd + (size_t)i * 16) = (u32x4){0u, 0u, 0u, 0u};
    *(u32x4*)(dkd + (size_t)i * 16) = (u32x4){0u, 0u, 0u, 0u};
  }
  // the heads' depth share of dQ: lane = head, 4 consecutive channels (16 bytes of fp32) at a time
#pragma unroll
  for (int hb = 0; hb < NG; ++hb) {
    const int h = hb * 32 + l32;
    if (h < G) {
      float* dst = p.dq_depth + ((size_t)(bh0 + h) * T + t) * D;
#pragma unroll
      for (int cb = 0; cb < Tl::kDBlocks; ++cb)
#pragma unroll
        for (int bq = 0; bq < 4; ++bq)
          *(f32x4*)(dst + cb * 32 + bq * 8 + hi * 4) =
              (f32x4){dqa[hb][cb][4 * bq], dqa[hb][cb][4 * bq + 1], dqa[hb][cb][4 * bq + 2], dqa[hb][cb][4 * bq + 3]};
    }
  }
}

// ---------------------------------------------------------------- launchers
// Workspace: LSE log2 e, then -delta of every query row, then - when there are depth slots - the depth
// share of dQ in fp32, [B, Hq, T, d].
static size_t row_scalar_bytes(const BwdParams& p) {
  return (((size_t)p.B * p.Hq * p.T * 2 * sizeof(float)) + 255) / 256 * 256;
}
size_t bwd_bf16_workspace_bytes(const BwdParams& p, int d) {
  return row_scalar_bytes(p) + (p.depth_alloc > 0 ? (size_t)p.B * p.Hq * p.T * d * sizeof(float) : 0);
}

int bwd_bf16_max_group() { return 64; }

// Waves of the short dK/dV kernel that a call takes, 0: the other kernel; the one whose estimated time is shortest.
// Each is bound by the
// chain of its longest workgroup (few workgroups) or by what 256 compute units get done (many): a workgroup's
// steps (64 queries x 128 keys; short kernel: 32 x 32 per wave, its waves side by side), its two ends, and the
// depth slots of its positions, padding included.  The short kernel reads Q and dO four times as often, and
// pays `undealt` more where the heads cannot be dealt to the 8 dies (head_blocked_id) and every L2 sees
// them all.  Constants (us; per 256 units) fitted to both kernels' times at 7700 shapes, T = 2 to 16384, 1 to 2000
// heads, 1 to 16 per group, 0 to 64 slots: 0.4 % behind the better kernel on average, more than 10 % at 1 of 100.
// Eight waves: one workgroup per unit, whose ends (and halves of its waves in the depth slots) nothing hides;
// fitted to all three at 170 shapes of up to 3000 workgroups: 0.1 % behind the best on average, 4 % at most.
// Whole call without slots, workgroups of the short kernel: other / short, us:
//   d=64   causal      G=1 T=128: 512 16/15, 768 17/19;   T=512: 768 28/27, 1536 38/41;   T=2048: 1536 101/89, 2048 92/95
//                      G=8 T=128: 1024 72/63, 2048 115/129;   T=1000: 2048 361/331, undealt 1216 265/214, 2400 379/536
//          not causal  G=1 T=128: 512 15/15, 768 15/18;   T=1000: 512 42/34, 896 43/46;   T=4096: 768 133/126, 1280 192/194
//   d=128  causal      G=1 T=128: 256 23/18, 512 24/24, 768 26/32;   T=512: 640 47/46, 1024 50/57;   T=2048: 1024 147/131, 1536 176/179
//                      G=8 T=256: 1024 180/167, 1536 228/248;   T=1000: 1536 588/546, 2048 644/730
//          not causal  G=2 T=128: 256 27/20, 512 30/32;   T=512: 512 70/57, 768 81/84;   T=2048: 768 259/240, 1024 274/307
struct KeyCost {
  double step, step_unit, ends, short_step, short_unit, undealt, slot, slot_unit;
};
struct EightWaveCost {
  double step, unit, ends, slot, slot_unit, once;
};
static double fourth(double x) { return x * x * x * x; }
static double undealt_share(long long heads) {  // 0: a multiple of 8; 1: odd
  return (3 - (heads % 8 == 0 ? 3 : heads % 4 == 0 ? 2 : heads % 2 == 0 ? 1 : 0)) / 3.0;
}
static int dkdv_waves(const BwdParams& p, int d) {
  const KeyCost c = d == 64 ? KeyCost{1.26, 1.12, 1.2, 0.90, 0.66, 0.16, 0.18, 0.0043}
                            : KeyCost{2.7, 1.53, 3.9, 1.41, 1.58, 0.17, 0.36, 0.0076};
  const long long heads = (long long)p.B * p.Hk;
  const double G = p.Hq / p.Hk, n64 = (p.T + 63) / 64, n32 = (p.T + 31) / 32, n128 = (p.T + 127) / 128;
  const double L = G <= 4 ? p.depth_count : 0;  // (larger groups: a kernel of their own, or the same in both)
  const double slot = G > 1 ? 2 * c.slot : c.slot, odd = p.Hq / p.Hk % 4 ? 0.375 : 0.0;
  const double steps = G * n128 * (p.causal ? n64 - n128 + 1 : n64);
  const double short_steps = n32 * (G * (p.causal ? n32 + 1 : 2 * n32) / 8 + odd);
  const double chain = G * n64 * c.step + 4 * L * slot;
  const double load = heads * (steps * c.step_unit + n128 * (c.ends + 128 * L * c.slot_unit)) / 256;
  const double short_chain = (G * n32 / 4 + odd) * c.short_step + L * slot;
  const double short_load = heads * (short_steps * c.short_unit * (1 + c.undealt * undealt_share(heads)) +
                                     n32 * (c.ends + 32 * L * c.slot_unit)) / 256;
  const double other = fourth(chain) + fourth(load), four = fourth(short_chain) + fourth(short_load);  // (smooth maxima)
  if (d == 64) {
    const EightWaveCost e{1.25, 1.31, 3.65, 0.196, 0.0064, 0.82};
    const double odd8 = p.Hq / p.Hk % 8 ? 0.4375 : 0.0;
    const double steps8 = n32 * (G * (p.causal ? n32 + 1 : 2 * n32) / 16 + odd8);
    const double chain8 = (G * n32 / 8 + odd8) * e.step + (G > 1 ? 2 : 1) * L * e.slot + e.once;
    const double load8 = heads * (steps8 * e.unit * (1 + c.undealt * undealt_share(heads)) + n32 * (e.ends + 32 * L * e.slot_unit)) / 256;
    const double eight = fourth(chain8) + fourth(load8);
    if (eight < other && eight < four) return 8;
  }
  return four < other ? 4 : 0;
}
// The two dQ kernels likewise (32 queries against 128 per workgroup, key tiles dealt to the four waves; 3700
// shapes, 0.2 % behind the better one on average).  Whole call, one head, workgroups of the short kernel: other /
// short, us:
//   d=64   causal      T=128: 512 17/16, 1200 21/23;   T=512: 512 27/25, 896 29/31;   T=2048: 1216 79/74, 2048 90/93;   T=8192: 1536 285/264
//          not causal  T=128: 384 15/16;   T=512: 512 25/24, 896 27/30;   T=2048: 768 72/70, 1216 107/113
//   d=128  causal      T=128: 256 23/21, 576 25/27;   T=512: 576 47/46, 896 49/56;   T=2048: 1024 142/136, 1216 149/158
//          not causal  T=128: 256 21/21, 576 23/27;   T=512: 448 45/45, 576 46/54;   T=2048: 512 138/129, 768 140/153
struct QueryCost {
  double step, step_unit, ends, short_step, short_unit, undealt, short_ends;
};
static bool few_queries(const BwdParams& p, int d) {
  const QueryCost c = d == 64 ? QueryCost{0.49, 0.28, 0.94, 0.13, 0.23, 0.25, 0.56} : QueryCost{0.94, 0.66, 2.1, 0.67, 0.59, 0.21, 1.6};
  const double heads = (double)p.B * p.Hq, n64 = (p.T + 63) / 64, n32 = (p.T + 31) / 32, n128 = (p.T + 127) / 128;
  const double steps = n128 * (p.causal ? n64 - n128 + 1 : n64);
  const double short_steps = n32 * ((p.causal ? n32 + 1 : 2 * n32) / 8 + 0.375);
  const double chain = n64 * c.step, load = heads * (steps * c.step_unit + n128 * c.ends) / 256;
  const double short_chain = (n32 / 4 + 0.375) * c.short_step;
  const double short_load = heads * (short_steps * c.short_unit * (1 + c.undealt * undealt_share((long long)p.B * p.Hk)) +
                                     n32 * c.short_ends) / 256;
  return fourth(short_chain) + fourth(short_load) < fourth(chain) + fourth(load);
}
// Workgroups of the dQ kernel of 128 queries that share a compute unit.  At d = 64 three fit in registers: ahead where
// a workgroup's two ends weigh most, where three hold the grid and two do not (calls that are not causal; causal
// ones, whose third layer has few light tiles to go with the heavy ones, while they are short), and in larger
// grids of short sequences; otherwise two are as fast or faster, as the chip's power is what counts (three against
// two, whole call, workgroups: T=40: 1024 0.97, 2048 0.91;  not causal: T=300 768 0.98, T=1500 768 0.98, T=5789 736 0.95,
// T=2048 1024 1.02, 2048 1.00;  causal: T=300 768 0.97, T=700 768 0.97, T=1500 768 1.03, T=3000 768 1.05, T=512 1024 1.02,
// T=1000 2048 0.98, T=2048 4096 0.98, T=4096 2048 1.01, T=16384 2048 1.03).
static int dq_per_unit(const BwdParams& p, int d, long long workgroups) {
  if (d != 64 || workgroups <= 512) return 2;
  if (p.T <= 128) return 3;
  if (workgroups <= 768) return !p.causal || p.T <= 700 ? 3 : 2;
  return workgroups >= 2048 && p.T <= 2048 ? 3 : 2;
}
// Depth-slot gradients of 5 to 8 heads: inside dK/dV (depth_group_rows), or in a kernel of their own
// (depth_gqa).  The former takes 32 slots at a time whether they exist or not, and a wave takes 32
// positions one after the other: it needs mostly full blocks of slots, and enough key tiles.
// d = 64, backward call, inside / kernel of its own, 8 heads per group (5 heads the same within 3 %):
//   slots       16    18    20    22    24    28    32    36    44    48    56    64
//   T=1000    1.07  1.05  1.02  0.99  0.98  0.94  0.93  1.06  1.00  0.97  0.93  0.88
//   T=2048    1.05  1.03  1.01  0.99  0.98  0.95  0.92  1.02  0.98  0.97  0.92  0.90
//   T=16384   1.01  1.01  1.00  1.00  1.00  0.99  0.98  1.01  1.00  0.99  0.98  0.96
// d = 128 keeps the kernel of its own: beside the key tiles' registers the 32 slots and the next 32 do not
// fit (91 registers went to scratch memory, reloaded at every position), and the gain was 2 to 5 % at best
// (T=16384, 31 slots 14494 / 14205; T=2048, 64 slots 3073 / 2925) and a loss elsewhere (T=1000, 31 slots
// 1700 / 1724; B=116 Hq=32 Hk=4 T=84, 31 slots 503 / 530).
static bool own_depth_kernel(const BwdParams& p, int d) {
  const int G = p.Hq / p.Hk, L = p.depth_count, blocks = (L + 31) / 32;
  if (p.depth_alloc == 0 || G <= 4) return false;
  return G > 8 || d != 64 || dkdv_waves(p, d) != 0 || L * 16 < blocks * 32 * 11 || L == 0;
}
// Calls that take one kernel for dK, dV and dQ (moda_bwd_grads_kernel).  With depth slots the heads of a group have to fill the
// waves of a workgroup evenly, and up to 4 of them their gradients on the vector ALUs (5 to 8: their number of launches is fixed by
// tests of moda_kernels_per_call; one launch for them was not measured).  Up to 16 positions the launches stay apart for the same
// reason only: three are counted at 16 positions (H=1 T=16 d=128: 12.5 us, 8.2 in one launch).  So they do where the
// workgroups of both kinds, at 17 positions 2^24 of four waves, are too many for one grid.
// Key tiles of 32 keys with query tiles of 128 rows: not built for calls with slots that hardly ever are estimated to be fastest
// with them (9 of 25000 calls, whose next best kind takes 1.01 of the time).
constexpr bool grads_mixed(int d, int gt, int waves) { return gt == 0 || (waves == 8 ? gt == 4 && d == 128 : gt > 1 || d == 128); }
struct GradsPlan {
  bool few_keys, few_queries;
  int waves;
  int heads(const BwdParams& p) const {
    const int G = p.Hq / p.Hk;
    return p.depth_alloc > 0 ? G : few_queries ? 1 : G % 4 == 0 ? 4 : G % 2 == 0 ? 2 : 1;
  }
  long long key_tiles(const BwdParams& p) const { return ((long long)p.T + (few_keys ? 31 : 127)) / (few_keys ? 32 : 128); }
  long long query_tiles(const BwdParams& p) const {
    const int n = few_queries ? 32 : waves * 32 / heads(p);
    return ((long long)p.T + n - 1) / n;
  }
  long long workgroups(const BwdParams& p) const {
    return (long long)p.B * p.Hk * (key_tiles(p) + query_tiles(p) * (p.Hq / p.Hk / heads(p)));
  }
};
// Heads that a die walks together there (see head_walk_id): up to two rounds of workgroups all of them, so that the
// longest workgroups of all heads start first and neighbouring units do not all get one kind of tile (with one head of
// two key and two query tiles at a time every other unit had all the depth slots: B=72 H=1 T=37 d=128, 64 slots 101 -> 65 us);
// beyond, as many as have K and V in 512 KB of the L2, which their tiles then find there (256 KB / 512 KB / 1 MB / 2 MB / 4 MB, 70
// shapes: 0.894 / 0.890 / 0.892 / 0.894 / 0.899 of the time of two launches).  But all of them also where up to 1024 key tiles are
// most of the work: head by head the longest key tiles of a die's last heads start last, and the call ends with them alone.  One
// head at a time / all, us: d=64 B=2 Hq=16 Hk=8 T=3253, no slots 196 / 167; B=4 Hq=48 Hk=16 T=316, no slots, not causal 38.2 / 31.1;
// d=128 B=3 Hq=16 Hk=8 T=3816, 1 slot 702 / 587.  Slots as long as the key tiles keep the order head by head, which reads them
// between the key tiles: B=4 H=16 T=3979 d=64, 15 slots 684 / 708, B=1 H=16 T=4389 213 / 240.  90 shapes, up to 512 / 1024 / 2048 /
// any number of key tiles: 0.988 / 0.978 / 0.979 / 0.980 of the time head by head; with the line at 200 / 400 / 800 / 2000 positions
// of the group to a slot 0.981 / 0.978 / 0.981 / 0.985, and 0.981 without it.
static int grads_head_group(const BwdParams& p, int d, long long grid, long long key_tiles) {
  if (p.B * p.Hk % 8 != 0) return 0;
  const long long per_die = (long long)p.B * p.Hk / 8;
  if (grid <= 1024 || (key_tiles <= 1024 && (long long)p.T * (p.Hq / p.Hk) > 400ll * p.depth_count)) return (int)per_die;
  return (int)std::max(1ll, std::min(per_die, (512ll << 10) / (4ll * p.T * d)));
}
// The kind of tiles whose estimated time is shortest.  As for dkdv_waves: the chains of the longest key tile and of the longest
// query tile (a step: 64 queries x 128 keys, 128 x 64, or 32 x 32 per wave; chunks of slots one after the other), and what
// all tiles ask of 256 units (steps, ends, slots), in part rounded up to whole rounds of workgroups.  Constants (us; per 256
// units) fitted to the times of all kinds at 34800 shapes (T = 17 to 66000, 1 to 12000 heads, 1 to 16 per group, 0 to 64
// slots) so that the choice is right more than the time: the kind taken is 1.0 % (d = 64) and 1.1 % (d = 128) behind the best one on
// average, more than 10 % at 1 of 33; slower than two launches by more than 2 % at 16 and 4 of 1000.  (Without the rounds, and fitted
// to the times alone, 1.7 and 2.0 %, more than 10 % at 1 of 15; 24 and 11 of 1000; with two launches as a sixth kind, where they are
// ahead of the kind taken, 14 and 4: not worth it.)  Backward call, us, 128-row tiles / 32 keys and 32 positions / 32 keys, 128
// rows / the last two with eight waves:
//   d=64   G=1 T=216 32 heads, 64 slots  109 / 99 / 108 / 87 / -;   B=5 H=2 T=6284, 1 slot  207 / 282 / 262 / - / -
//          G=4 B=3 Hk=2 T=381, no slots  36 / 16.7 / 16.5 / 14.6 / -;   G=16 Hk=1 T=16817, no slots  4810 / 3130 / 2667 / 2654 / 2345
//   d=128  G=1 B=2 H=8 T=1351, 24 slots  153 / 161 / - / - / -;   B=2 H=4 T=564, 7 slots  41 / 22 / - / - / -
//          G=4 Hk=2 T=1099, 12 slots  170 / 63 / 52 / - / -;   Hk=4 T=8447, 31 slots  1440 / 1216 / - / - / -
//          G=1 H=1 T=5592, 15 slots not causal  205 / 93 / 159 / 107 / 247;   G=2 Hk=1 T=8526, 15 slots  623 / 449 / 320 / 393 / 450
// Heads that cannot be dealt to the dies are walked tile by tile, all heads at a time: with several rounds of workgroups all key
// tiles would come before all slots, which then only the products of dQ hide.  Where the slots are the longer part the key
// tiles go evenly among the query tiles instead (behind them / among them, us: B=89 Hq=4 Hk=2 T=997 d=128, 15 slots 887 / 802;
// B=41 H=1 T=7189 d=64, 15 slots 1280 / 1200; but B=99 H=1 T=5190 d=128, 7 slots 2810 / 2910, B=5 Hq=2 Hk=1 T=18303 d=64, 15
// slots 2782 / 3176.  Heads that can be dealt: 1.07 of the time on average.)
static int spread_key_tiles(const BwdParams& p, long long grid) {
  return p.head_group == 0 && grid > 1024 && p.depth_count >= 4 && (long long)p.T * (p.Hq / p.Hk) <= 600ll * p.depth_count;
}
struct GradsCost {
  GradsPlan plan;
  double key_step, query_step, key_unit, query_unit, key_ends, query_ends, slot, slot_unit, undealt, once;
  double group, last_round, key_step_all;  // (the last one: of calls that are not causal, of key_step)
};
static GradsPlan grads_plan(const BwdParams& p, int d) {
  static const GradsCost costs64[] = {{{false, false, 4}, 1.26, 0.0026, 0.861, 0.0562, 1.16, 4.19, 0.52, 0.359, 0.00497, 6.8, -0.0455, 0.293, 0.947},
                                      {{true, true, 4}, 1.13, 1, 0.545, 0.29, 1.83, 1.06, 0.512, 0.359, 0.223, 4.46, 0.0628, 0.214, 0.854},
                                      {{true, false, 4}, 0.998, 1.11, 0.812, 0.000684, 3.57, 2.59, 0.485, 0.416, 0.155, 5.11, -0.0733, 0.133, 0.759},
                                      {{true, true, 8}, 0.907, 0.518, 2.16, 0.00272, 5.1, 3.82, 0.409, 0.397, 0.000167, 7.26, -0.00562, 0.348, 0.866},
                                      {{true, false, 8}, 0.762, 2.35, 1.96, 0.000176, 4.97, 9.84, 0.645, 0.479, 0.000755, 5.21, -0.122, 0.422, 0.386}};
  static const GradsCost costs128[] = {{{false, false, 4}, 2.52, 0.000545, 1.63, 0.0982, 2.18, 6.48, 0.482, 0.355, 0.0209, 8.9, -0.0273, 0.187, 1.03},
                                       {{true, true, 4}, 1.62, 1.44, 1.77, 0.000563, 2.4, 3.67, 0.465, 0.325, 0.188, 6.45, 0.0939, 0.0721, 0.883},
                                       {{true, false, 4}, 1.53, 1.7, 1.39, 7.96e-05, 4.97, 4.66, 0.568, 0.427, 0.439, 7.29, -0.0669, 0.0125, 0.859},
                                       {{true, true, 8}, 1.69, 1.06, 2.79, 1.04, 11.7, 4.09, 0.549, 0.396, 0.000252, 8.6, -0.0337, 0.143, 1.03},
                                       {{true, false, 8}, 1.3, 3.42, 3.52, 9.13e-05, 7.73, 12.1, 0.779, 0.44, 0.00589, 7.5, -0.0691, 0.35, 0.93}};
  const double n32 = (p.T + 31) / 32, n64 = (p.T + 63) / 64, heads = (double)p.B * p.Hk / 256;
  const int G = p.Hq / p.Hk, per_step = 512 / d;  // (rows of slots that a wave takes at a time)
  const double walk32 = p.causal ? (n32 + 1) / 2 : n32;  // tiles of 32 that a tile of 32 sees on average
  GradsPlan best{};
  double least = 0;
  for (int i = 0; i < 5; ++i) {
    const GradsCost& c = d == 64 ? costs64[i] : costs128[i];
    if (p.depth_alloc > 0 && c.plan.few_keys && !c.plan.few_queries && !grads_mixed(d, G, c.plan.waves)) continue;
    const int nw = c.plan.waves, h = c.plan.heads(p), n_pos = c.plan.few_queries ? 32 : nw * 32 / h;
    const double kt = (double)c.plan.key_tiles(p), qt = (double)c.plan.query_tiles(p) * (G / h);
    double k_first, k_all, q_first, q_all;
    if (c.plan.few_keys) {
      k_first = G * n32 / nw;
      k_all = kt * (G * walk32 / nw + 0.5 - 0.5 / nw);
    } else {
      k_first = G * n64;
      k_all = kt * G * (p.causal ? n64 - kt + 1 : n64);
    }
    if (c.plan.few_queries) {
      q_first = n32 * h / nw;
      q_all = qt * (walk32 * h / nw + 0.5 - 0.5 * h / nw);
    } else {
      q_first = n64;
      q_all = qt * (p.causal ? (n64 + std::max(1.0, n_pos / 64.0)) / 2 : n64);
    }
    int passes = 0;
    if (p.depth_alloc > 0 && G == 1) passes = (std::min(p.T, c.plan.few_queries ? std::max(32 / nw, per_step) : 32) + per_step - 1) / per_step;
    else if (p.depth_alloc > 0) passes = (std::min(p.T, n_pos) + nw * per_step - 1) / (nw * per_step);
    double load = heads * ((k_all * c.key_unit + q_all * c.query_unit) * (1 + c.undealt * undealt_share((long long)p.B * p.Hk)) +
                           kt * c.key_ends + qt * c.query_ends + (double)p.T * p.depth_count * d / 1000 * c.slot_unit);
    // (rounds of workgroups that the chip holds at once: the last one lasts as long as a full one)
    const double rounds = heads * (kt + qt) / (nw == 8 ? 1 : d == 64 && c.plan.few_keys && c.plan.few_queries ? 3 : 2);
    if (rounds > 1) load *= 1 + c.last_round * (ceil(rounds) / rounds - 1);
    load *= pow(G, c.group);
    if (!p.causal) k_first *= c.key_step_all;
    const double time = c.once + sqrt(sqrt(fourth(k_first * c.key_step) + fourth(q_first * c.query_step + passes * p.depth_count * c.slot) + fourth(load)));
    if (i == 0 || time < least) {
      least = time;
      best = c.plan;
    }
  }
  return best;
}
// Whether a call takes one launch, and the plan of it.
static bool one_launch(const BwdParams& p, int d, GradsPlan& plan) {
  const int G = p.Hq / p.Hk;
  if (p.T <= 16 || (p.depth_alloc > 0 && G != 1 && G != 2 && G != 4)) return false;
  plan = grads_plan(p, d);
  return grid_ok(plan.workgroups(p), plan.waves * 64);
}
// The kernels of a call.
struct BwdRoute {
  bool one;        // moda_bwd_grads_kernel, as `plan` says; else
  GradsPlan plan;
  bool own_depth;  // a kernel for the depth-slot gradients,
  int waves;       // dK/dV (0: 128 keys to a workgroup) and
  bool few_queries;  // dQ
  int gt;          // heads per group whose depth slots the kernel of dQ (one launch) or of dK, dV takes, rounded up; 0: none
};
static BwdRoute bwd_route(const BwdParams& p, int d) {
  BwdRoute r{};
  const int G = p.Hq / p.Hk;
  r.one = one_launch(p, d, r.plan);
  r.own_depth = own_depth_kernel(p, d);
  // (up to 2 heads: up to 16 positions, where the estimate takes them too, or very many heads)
  r.waves = G <= 2 ? 4 : dkdv_waves(p, d);
  r.few_queries = few_queries(p, d);
  r.gt = p.depth_alloc == 0 || r.own_depth ? 0 : G <= 2 ? G : G <= 4 ? 4 : 8;
  return r;
}
int bwd_bf16_kernels(const BwdParams& p, int d) {
  const BwdRoute r = bwd_route(p, d);
  return r.one ? 2 : 3 + (r.own_depth ? 1 : 0);
}
int bwd_bf16_kernel_name(const BwdParams& p, int d, int which, char* name, size_t size) {
  const BwdRoute r = bwd_route(p, d);
  if (r.one)
    return snprintf(name, size, "moda_bwd_grads_kernel<%d, %d, %s, %s, %d>", d, r.gt, r.plan.few_keys ? "true" : "false",
                    r.plan.few_queries ? "true" : "false", r.plan.waves);
  if (which == 0 && r.waves == 0) return snprintf(name, size, "moda_bwd_dkdv_kernel<%d, %d>", d, r.gt);
  if (which == 0) return snprintf(name, size, "moda_bwd_dkdv_short_kernel<%d, %d, %d>", d, r.gt, r.waves);
  if (r.few_queries) return snprintf(name, size, "moda_bwd_dq_short_kernel<%d>", d);
  return snprintf(name, size, "moda_bwd_dq_kernel<%d, 4, %d>", d, dq_per_unit(p, d, (long long)p.B * p.Hq * (((long long)p.T + 127) / 128)));
}

template <int D>
static hipError_t launch_bwd_bf16_d(BwdParams p, hipStream_t stream) {
  const long long rows = (long long)p.B * p.Hq * p.T;
  const int G = p.Hq / p.Hk;
  const long long g_delta = (rows * (D / 8) + 255) / 256;
  const long long n_kt = (p.T + 127) / 128;
  const long long kv_rows = (long long)p.B * p.Hk * p.T;
  const long long g_depth = G <= 8 ? (kv_rows * (D / 8) + 255) / 256 : kv_rows;
  // every grid is checked before the first kernel is enqueued
  const BwdRoute r = bwd_route(p, D);
  const GradsPlan& plan = r.plan;
  const int few = r.waves;
  const long long g_grads = r.one ? plan.workgroups(p) : 0;
  const long long n32 = ((long long)p.T + 31) / 32;
  const long long g_dkdv = (long long)p.B * p.Hk * (few ? n32 : n_kt), g_dq = (long long)p.B * p.Hq * (r.few_queries ? n32 : n_kt);
  if (!grid_ok(g_delta, 256) || (!r.one && (!grid_ok(g_dkdv, few ? few * 64 : 256) || !grid_ok(g_dq, 256))) ||
      (r.own_depth && !grid_ok(g_depth, G <= 8 ? 256 : 64)))
    return kGridTooLarge;  // (own_depth: up to 8 heads 256 / (d/8) positions to a workgroup, above one, of one wave)
  if (G > bwd_bf16_max_group()) return hipErrorInvalidValue;
  // the group kernel gathers the G heads' rows of a position with 32-bit offsets from the first head
  if (G > 8 && p.depth_alloc > 0 && (unsigned long long)G * p.T * (D * 2) >= 0xffffff00ull) return kGridTooLarge;
  p.minus_delta = p.lse2 + rows;
  p.dq_depth = (float*)((char*)p.lse2 + row_scalar_bytes(p));
  hipError_t e = launch_kernel(moda_bwd_delta_kernel<D>, dim3((unsigned)g_delta), dim3(256), stream, p.dO, p.O, p.LSE,
                               p.lse2, p.minus_delta, rows);
  if (e != hipSuccess) return e;
  if (r.own_depth) {
    if (G <= 8) {
      e = launch_kernel(moda_bwd_depth_gqa_kernel<D, 8>, dim3((unsigned)g_depth), dim3(256), stream, p);
    } else {
      // large groups: one wave per position, the group's products on the matrix pipe
      const dim3 gw((unsigned)g_depth);
      if (G <= 32) e = launch_kernel(moda_bwd_depth_group_kernel<D, 1>, gw, dim3(64), stream, p);
      else e = launch_kernel(moda_bwd_depth_group_kernel<D, 2>, gw, dim3(64), stream, p);
    }
    if (e != hipSuccess) return e;
  }
  if (r.one) {
    const int heads = plan.heads(p);
    p.head_group = grads_head_group(p, D, g_grads, (long long)p.B * p.Hk * plan.key_tiles(p));
    const int spread = spread_key_tiles(p, g_grads);
    auto launch = [&](auto gt) {
      constexpr int GT = decltype(gt)::value;
      const auto kernel = plan.waves == 8 ? (plan.few_queries ? moda_bwd_grads_kernel<D, GT, true, true, 8> : moda_bwd_grads_kernel<D, GT, true, !grads_mixed(D, GT, 8), 8>)
                          : !plan.few_keys ? moda_bwd_grads_kernel<D, GT, false, false, 4>
                          : plan.few_queries ? moda_bwd_grads_kernel<D, GT, true, true, 4> : moda_bwd_grads_kernel<D, GT, true, !grads_mixed(D, GT, 4), 4>;
      return launch_kernel(kernel, dim3((unsigned)g_grads), dim3(plan.waves * 64), stream, p, heads, spread);
    };
    return r.gt == 0   ? launch(std::integral_constant<int, 0>())
           : r.gt == 1 ? launch(std::integral_constant<int, 1>())
           : r.gt == 2 ? launch(std::integral_constant<int, 2>())
                       : launch(std::integral_constant<int, 4>());
  }
  {
    constexpr int kEight = D == 64 ? 8 : 4;
    const dim3 gk((unsigned)g_dkdv), blk(few ? few * 64 : 256);
    auto pick = [few](auto other, auto four, auto eight) { return few == 0 ? other : few == 4 ? four : eight; };
    const auto kernel =
        r.gt == 1   ? moda_bwd_dkdv_short_kernel<D, 1, 4>
        : r.gt == 2 ? moda_bwd_dkdv_short_kernel<D, 2, 4>
        : r.gt == 0 ? pick(moda_bwd_dkdv_kernel<D, 0>, moda_bwd_dkdv_short_kernel<D, 0, 4>, moda_bwd_dkdv_short_kernel<D, 0, kEight>)
        : r.gt == 4 ? pick(moda_bwd_dkdv_kernel<D, 4>, moda_bwd_dkdv_short_kernel<D, 4, 4>, moda_bwd_dkdv_short_kernel<D, 4, kEight>)
                    : moda_bwd_dkdv_kernel<D, D == 64 ? 8 : 4>;  // (d = 128: never more than 4 here)
    e = launch_kernel(kernel, gk, blk, stream, p);
  }
  if (e != hipSuccess) return e;
  if (r.few_queries) return launch_kernel(moda_bwd_dq_short_kernel<D>, dim3((unsigned)g_dq), dim3(256), stream, p);
  return launch_kernel(dq_per_unit(p, D, g_dq) == 3 ? moda_bwd_dq_kernel<D, 4, D == 64 ? 3 : 2> : moda_bwd_dq_kernel<D, 4, 2>,
                       dim3((unsigned)g_dq), dim3(256), stream, p);
}

hipError_t launch_bwd_bf16(const BwdParams& p, int d, hipStream_t stream) {
  if (d == 128) return launch_bwd_bf16_d<128>(p, stream);
  if (d == 64) return launch_bwd_bf16_d<64>(p, stream);
  return hipErrorInvalidValue;
}

}  // namespace moda
