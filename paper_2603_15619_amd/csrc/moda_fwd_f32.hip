// MoDA attention forward, fp32 inputs, fp32 precision throughout, on the gfx950 matrix pipe.
//
// The accuracy path (max abs error 1e-5 against an fp64 evaluation is the target).  Its products
// run on the bf16 matrix instructions with every fp32 factor as the sum of THREE bf16 numbers, which hold
// its 24 bits: x y = x1 y1 + (x1 y2 + x2 y1 + x1 y3 + x3 y1 + x2 y2) + what is below 2^-24 of it.  bf16
// products are exact in fp32 and 16 of them are summed per instruction: six such instructions take 192
// cycles where the fp32 ones (64 FLOP per cycle and SIMD) take 512, and there are fewer roundings: error of
// O against 64 bits 2.05e-7 -> 1.70e-7 (T=700 d=64), 2.83e-7 -> 2.25e-7 (T=1500 d=128, 15 slots), with
// softmax scale 1 8.6e-7 -> 5.0e-7.  Factors that have no such parts take the fp32 instructions (see
// fold_tile).  The depth slots run on the vector ALUs at the memory rate.
//
// A workgroup = 32 queries of one head; its 4 (few tiles: 8) waves share the queries and DEAL OUT THE KEYS: key
// tile kt (32 keys) belongs to wave kt % NW, every wave keeps a running (max, normaliser, output) of
// its own, and all of them are folded into one softmax at the end, together with the partial result
// of the depth slots.  Dealing out keys instead of queries makes the unit of work 32 queries per
// 4 SIMDs: a few thousand rows of causal attention then fill 256 compute units evenly (32 queries
// per wave left the last query tiles of a T = 2000 call alone on the chip for twice the mean), and
// a call of a few hundred rows walks its longest row in a quarter of the steps.  (Sequences of a few
// positions, which this would pad to tiles of 32, go to the kernel of moda_fwd_f32_rows.hip.)
//
// What bounds it: the vector ALUs that form the parts (11 instructions per two numbers: 800 of a tile's
// 900 at d = 128) and the matrix pipe, of different waves, on the sequence keys; HBM on the depth slots (4 bytes
// per FLOP); every other workgroup takes its slots before its key tiles, the others after, so that both
// are busy.
//   B=1 H=16 T=2000 d=128, 15 slots: 0.168 ms, 99 TFLOP/s and 3.3 TB/s (fp32 matrix instructions: 0.211 ms; one
//                                    wave per query on the vector ALUs: 2.69 ms); no slots 0.162 -> 0.122
//   B=1 H=16 T=8000 d=128, no slots: 1.60 ms, 164 TFLOP/s (1.97; a library product of 8192^3 reaches 154)
//   B=1 H=2 T=256 d=64, 4 slots:     9.9 us (10.6), most of it latency from one end to the other
// (Splitting the next operand between the matrix instructions of one wave: no change; subtracting the
// parts with packed dot products, 7 instructions per two numbers instead of 11: 2 to 6 % slower.)
//
// Operand layouts.  S^T = K Q^T (keys on M, queries on N): the contraction may take the channels
// in any order that both operands share, so lane (l32, hi) holds channels 8 j + 4 hi .. + 3 of key
// l32 and two 128-bit loads make an operand; K comes straight from global memory
// (four consecutive loads use up a 128-byte line), Q from LDS.  A lane then owns 16 scores of one
// query, and registers 8 h .. 8 h + 7 of them are, as they stand, the B operand of O^T += V^T P^T for the keys
// 8 (i / 4) + i % 4 (lanes < 32) and 4 more (lanes >= 32).  Channels are dealt to the output blocks
// so that one load of a V row feeds them all: block cb, row r is channel r * (d / 32) + cb.
#include <type_traits>

#include "moda_launch.h"

namespace moda {

constexpr int kF32Rows = 32;   // queries per workgroup
constexpr int kF32Keys = 32;   // keys per tile (of one wave)
constexpr float kTiny = -100.f;       // (2^kTiny: weights below have not all of their bits in three parts either)
constexpr float kLargest = 0x1p120f;  // (the sums of first parts, rounded up, could overflow where those of the values do not)
// A minute value (below 2^-110) loses its last bits, 2^-134 of a number: nothing next to a value above kLeast whose
// weight is above 2^kWide, 2^-102 of an output.
constexpr float kWide = -50.f, kLeast = 0x1p-52f;
constexpr unsigned kLeastSplit = (127 - 100) << 23;  // numbers below 2^-100 are not split where they count by themselves

template <int D, int NW>
struct F32Cfg {
  static constexpr int kRow = D + 4;                 // floats per LDS row (16 consecutive rows hit 16 bank groups)
  static constexpr int kBlocks = D / 32;             // output blocks of 32 channels
  static constexpr int kFrags = D / 8;               // 128-bit K fragments per tile and lane
  static constexpr int kSteps = D / 16;              // bf16 matrix instructions per product of parts
  static constexpr int kRounds = D / 64;             // the waves' outputs are summed 64 channels at a time
  static constexpr int kXRow = 64 + 4;
  static constexpr int kXWave = kF32Rows * kXRow;    // floats of one wave's share in a round
  static constexpr int kQRow = D + 8;                // bf16 numbers per LDS row of a part of the queries
  static constexpr int kQPart = kF32Rows * kQRow;
  static constexpr int kShared = NW * kXWave; // floats: the queries (three parts), later the outputs
  static_assert(3 * kQPart * 2 <= kShared * 4, "the queries fit");
};

// Eight fp32 as three operands of packed bf16 whose sum they are: each part is the part before's remainder
// rounded to 8 bits, the remainders are exact, and three times 8 bits hold the 24 of a float.  (An
// infinite number, or one that rounds to an infinite bf16, leaves NaN in the second part.)
struct Parts {
  bf16x8 p[3];
};
__device__ __forceinline__ Parts split8(const float (&v)[8]) {
  Parts r;
  u32x4 w[3];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    float x = v[2 * k], y = v[2 * k + 1];
    asm volatile("" : "+v"(x), "+v"(y));  // (split here: else all operands of a loop are split at once)
#pragma unroll
    for (int n = 0; n < 3; ++n) {
      w[n][k] = pack_bf16(x, y);
      x -= bf16_lo(w[n][k]);
      y -= bf16_hi(w[n][k]);
    }
  }
#pragma unroll
  for (int n = 0; n < 3; ++n) r.p[n] = __builtin_bit_cast(bf16x8, w[n]);
  return r;
}
__device__ __forceinline__ f32x16 mfma_16(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// exp(scale * (a - b)) of raw scores a, b; the difference is formed before it is scaled, so that
// a large common part of the scores costs no precision.  b = -inf (an empty state) counts as 0.
// (exp2f, not the bare instruction, which returns zero for weights below 2^-126: a value of 2^127 still
// counts with them.)
__device__ __forceinline__ float weight(float a, float b, float c2) {
  return exp2f((a - (b == -INFINITY ? 0.f : b)) * c2);
}

template <int D, int NW>
__device__ __forceinline__ void fwd_f32_tile(const FwdParams& p) {
  using C = F32Cfg<D, NW>;
  // the queries, later the waves' outputs; the depth slots' partial outputs; (max, normaliser) of
  // each wave and of the depth slots; scratch for the rare path below
  __shared__ __attribute__((aligned(16))) float shared[C::kShared];
  __shared__ __attribute__((aligned(16))) float depth_o[kF32Rows * C::kRow];
  __shared__ float stat_m[NW + 1][kF32Rows], stat_l[NW + 1][kF32Rows];
  __shared__ float p_tile[kF32Keys][kF32Rows];

  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int bh, tile;
  head_blocked_id(layered_id(p.causal, NW == 8 ? 1 : D == 64 ? 3 : 2), p.B * p.Hq, p.n_qtiles, bh, tile, p.head_group);
  const int q0 = (p.n_qtiles - 1 - tile) * kF32Rows;  // heavy (late) tiles first
  const int b = bh / p.Hq, g = (bh - b * p.Hq) / (p.Hq / p.Hk);
  const size_t bg = (size_t)b * p.Hk + g;
  const int T = p.T, L = p.depth_count;
  const float c2 = p.scale_log2;

  // ---- queries -> LDS, as three parts of bf16 (rows past the end repeat the last one; nothing of them is
  // stored).  The 16 channels of a matrix instruction stand in the order in which a lane holds those of a
  // key: 4 hi .. + 3, then 8 + 4 hi .. + 3 at place 8 hi.
  // Where a query has a number that has not all of its 24 bits in three parts (below 2^-110 the last bits are none
  // of a bf16), or one so large that it would show what a minute key lacks, one number is replaced by NaN: the
  // tiles then take the fp32 matrix instructions (see fold_tile).  What is lost of the keys otherwise, 2^-134 of a
  // number, is below 2^-32 of an exponent.
  unsigned least_q = 0xffffffffu;
  float largest_q = 0.f;
  unsigned short *q_parts = (unsigned short*)shared, *dst;
  for (int i = tid; i < kF32Rows * (D / 4); i += NW * 64) {
    const int r = i / (D / 4), c = i % (D / 4);
    const f32x4 q = *(const f32x4*)((const float*)p.Q + ((size_t)bh * T + min(q0 + r, T - 1)) * D + c * 4);
    float x[4] = {q[0], q[1], q[2], q[3]};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      least_q = min(least_q, 2 * __builtin_bit_cast(unsigned, x[e]) - 1);  // (of zeros the largest number)
      largest_q = fmaxf(largest_q, fabsf(x[e]));
    }
    dst = q_parts + r * C::kQRow + (c >> 2) * 16 + (c & 1) * 8 + ((c >> 1) & 1) * 4;
#pragma unroll
    for (int n = 0; n < 3; ++n) {
      const u32x2 w = {pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3])};
      *(u32x2*)(dst + n * C::kQPart) = w;
      x[0] -= bf16_lo(w[0]);
      x[1] -= bf16_hi(w[0]);
      x[2] -= bf16_lo(w[1]);
      x[3] -= bf16_hi(w[1]);
    }
  }
  if (least_q < 2 * kLeastSplit - 1 || largest_q > (c2 <= 0x1p30f ? 0x1p64f : 0.f)) *dst = 0x7fc0;
  __syncthreads();

  // ---- depth slots: 16 lanes per row, 4 (d = 64) or 8 (d = 128) channels each; a wave takes 8 (of eight waves 4) of
  // the tile's rows, 4 at a time, kC slots at a time with the next kC in flight
  auto depth_rows = [&]() {
    constexpr int NV = D / 64, kC = D == 128 ? 3 : 6;
    const int rg = lane >> 4, l16 = lane & 15;
    const int nch = (L + kC - 1) / kC;
    struct Chunk {
      f32x4 k[kC][NV], v[kC][NV];
    };
    const size_t drow = (size_t)p.depth_alloc * D;
    constexpr int kRowSteps = kF32Rows / 4 / NW;
    auto row_of = [&](int it) { return (wave * kRowSteps + it) * 4 + rg; };
    auto issue = [&](int it, int c, Chunk& x) {
      const size_t base = (bg * T + min(q0 + row_of(it), T - 1)) * drow + l16 * 4;
#pragma unroll
      for (int u = 0; u < kC; ++u) {
        // (slots of the last chunk past depth_count re-read the last attended one: a cache hit)
        const size_t s = base + (size_t)min(c * kC + u, L - 1) * D;
#pragma unroll
        for (int n = 0; n < NV; ++n) {
          x.k[u][n] = __builtin_nontemporal_load((const f32x4*)((const float*)p.Kdepth + s + n * 64));
          x.v[u][n] = __builtin_nontemporal_load((const f32x4*)((const float*)p.Vdepth + s + n * 64));
        }
      }
    };
    f32x4 q[NV], o[NV];
    float m = -INFINITY, l = 0.f;
    auto fold = [&](int c, const Chunk& x) {
      float s[kC], mn = m, least = INFINITY;
#pragma unroll
      for (int u = 0; u < kC; ++u) {
        float a = 0.f;
#pragma unroll
        for (int n = 0; n < NV; ++n)
#pragma unroll
          for (int e = 0; e < 4; ++e) a = fmaf(q[n][e], x.k[u][n][e], a);
        a = group_sum<16>(a);
        s[u] = c * kC + u < L ? a : -INFINITY;
        mn = fmaxf(mn, s[u]);
        least = fminf(least, a);
      }
      const float al = weight(m, mn, c2);
      m = mn;
      l *= al;
#pragma unroll
      for (int n = 0; n < NV; ++n) o[n] *= al;
      const bool tiny = __builtin_amdgcn_ballot_w64((least - mn) * c2 < -126.f) != 0;  // (uniform; as for the key tiles)
      float w[kC];
      if (tiny) {
#pragma unroll
        for (int u = 0; u < kC; ++u) w[u] = weight(s[u], mn, c2);
      } else {
        const float ref = mn == -INFINITY ? 0.f : mn;
#pragma unroll
        for (int u = 0; u < kC; ++u) w[u] = fast_exp2((s[u] - ref) * c2);
      }
#pragma unroll
      for (int u = 0; u < kC; ++u) {
        if (c * kC + u >= L) break;  // (uniform)
        l += w[u];
#pragma unroll
        for (int n = 0; n < NV; ++n)
#pragma unroll
          for (int e = 0; e < 4; ++e) o[n][e] = fmaf(w[u], x.v[u][n][e], o[n][e]);
      }
    };
    int it = 0, c = 0, iti = 0, ci = 0;
    auto advance = [&](int& i_, int& c_) {
      if (++c_ == nch) {
        c_ = 0;
        ++i_;
      }
    };
    auto issue_next = [&](Chunk& x) {  // (past the end: the last chunk again, ignored)
      issue(min(iti, kRowSteps - 1), iti < kRowSteps ? ci : nch - 1, x);
      if (iti < kRowSteps) advance(iti, ci);
      __builtin_amdgcn_sched_barrier(0);
    };
    auto one = [&](const Chunk& cur, Chunk& refill) -> bool {
      issue_next(refill);
      const int r = row_of(it);
      if (c == 0) {
        m = -INFINITY;
        l = 0.f;
#pragma unroll
        for (int n = 0; n < NV; ++n) {
          o[n] = (f32x4){0.f, 0.f, 0.f, 0.f};
          q[n] = *(const f32x4*)((const float*)p.Q + ((size_t)bh * T + min(q0 + r, T - 1)) * D + l16 * 4 + n * 64);
        }
      }
      fold(c, cur);
      if (c == nch - 1) {
#pragma unroll
        for (int n = 0; n < NV; ++n) *(f32x4*)(depth_o + r * C::kRow + l16 * 4 + n * 64) = o[n];
        if (l16 == 0) {
          stat_m[NW][r] = m;
          stat_l[NW][r] = l;
        }
      }
      advance(it, c);
      return it < kRowSteps;
    };
    Chunk xa, xb;
    issue_next(xa);
    while (true) {
      if (!one(xa, xb)) break;
      if (!one(xb, xa)) break;
    }
  };
  const bool depth_first = L > 0 && ((blockIdx.x >> 3) & 1) != 0;
  if (depth_first) depth_rows();

  // ---- this wave's key tiles: wave, wave + NW, ...
  f32x16 o[C::kBlocks];
#pragma unroll
  for (int cb = 0; cb < C::kBlocks; ++cb)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[cb][i] = 0.f;
  float m = -INFINITY, l = 0.f;  // reference max of the raw scores; this lane's share of the normaliser
  const int n_keys = p.causal ? min(T, q0 + kF32Rows) : T;
  const int nt = (n_keys + kF32Keys - 1) / kF32Keys;
  // tiles that every query sees in full; at most one more (the diagonal, or the ragged end) follows
  const int n_full = p.causal ? q0 / kF32Keys : T / kF32Keys;
  const int lim = p.causal ? min(q0 + l32, T - 1) : T - 1;  // last key that this lane's query sees
  // (rows past the end of the tensor read as zeros: their scores are masked, their values weighted with 0)
  const float* Kb = (const float*)p.Kseq + bg * T * D;
  const float* Vb = (const float*)p.Vseq + bg * T * D;
  const unsigned bytes = (unsigned)T * (unsigned)(D * 4);
  const __amdgpu_buffer_rsrc_t k_buf = __builtin_amdgcn_make_buffer_rsrc((void*)Kb, 0, (int)bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t v_buf = __builtin_amdgcn_make_buffer_rsrc((void*)Vb, 0, (int)bytes, 0x00020000);
  const int k_off = l32 * D * 4 + hi * 16;
  const int v_off = hi * 4 * D * 4 + l32 * C::kBlocks * 4;
  f32x4 kf[C::kFrags];
  float vf[16][C::kBlocks];
  auto load_k = [&](int kt, int half) {
    const int soff = (int)((unsigned)kt * (unsigned)(kF32Keys * D * 4));
    int off = k_off;  // (opaque here, so that the sums below stay immediates of the loads instead of
    asm volatile("" : "+v"(off));  // being hoisted out of the key loop into a register each)
#pragma unroll
    for (int j = half * (C::kFrags / 2); j < (half + 1) * (C::kFrags / 2); ++j)
      kf[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(k_buf, off + j * 32, soff, 0));
  };
  auto load_v = [&](int kt, int half) {
    const unsigned soff = (unsigned)kt * (unsigned)(kF32Keys * D * 4);
#pragma unroll
    for (int i = half * 8; i < half * 8 + 8; ++i) {
      const int so = (int)(soff + ((i >> 2) * 8 + (i & 3)) * D * 4);
      if constexpr (D == 128) {
        const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(v_buf, v_off, so, 0));
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) vf[i][cb] = v[cb];
      } else {
        const f32x2 v = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(v_buf, v_off, so, 0));
        vf[i][0] = v[0];
        vf[i][1] = v[1];
      }
    }
  };
  if (wave < nt) {
    load_k(wave, 0);
    load_k(wave, 1);
  }
  auto fold_tile = [&](int kt, auto PARTIAL) {
    constexpr bool partial = decltype(PARTIAL)::value;
    // loads in flight: half of the tile's V during the scores; then its other half; half of the next
    // tile's K from the output products on, the rest from their middle (all of K and V at once do
    // not fit 256 registers)
    const int k_next = kt + NW;  // (past the last tile: rows that exist or zeros, not used)
    load_v(kt, 0);
    __builtin_amdgcn_sched_barrier(0);
    // S^T = K Q^T: the products of the first parts in one chain, the five others down to 2^-16 of them in
    // another (those left out are 2^-24 of a product)
    f32x16 s, s1;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = s1[i] = 0.f;
    const unsigned short* q_row = q_parts + l32 * C::kQRow + hi * 8;
    auto k_parts = [&](int st) {
      const float x[8] = {kf[2 * st][0], kf[2 * st][1], kf[2 * st][2], kf[2 * st][3],
                          kf[2 * st + 1][0], kf[2 * st + 1][1], kf[2 * st + 1][2], kf[2 * st + 1][3]};
      return split8(x);
    };
#pragma unroll
    for (int st = 0; st < C::kSteps; ++st) {
      bf16x8 q[3];
#pragma unroll
      for (int n = 0; n < 3; ++n) q[n] = *(const bf16x8*)(q_row + n * C::kQPart + st * 16);
      const Parts ka = k_parts(st);
      s = mfma_16(ka.p[0], q[0], s);
      s1 = mfma_16(ka.p[0], q[1], s1);
      s1 = mfma_16(ka.p[1], q[0], s1);
      s1 = mfma_16(ka.p[0], q[2], s1);
      s1 = mfma_16(ka.p[2], q[0], s1);
      s1 = mfma_16(ka.p[1], q[1], s1);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] += s1[i];
    // numbers that have no such parts (infinite, NaN, about to overflow; of the queries minute ones too) leave NaN or
    // infinity in the scores of their key or query: the tile is then taken on the fp32 matrix instructions
    float sum = s[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) sum += s[i];
    if (__builtin_amdgcn_ballot_w64(!(fabsf(sum) < INFINITY)) != 0) {
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] = 0.f;
      const float* q = (const float*)p.Q + ((size_t)bh * T + min(q0 + l32, T - 1)) * D + hi * 4;
#pragma unroll 1
      for (int j = 0; j < C::kFrags; ++j) {
        const f32x4 qj = *(const f32x4*)(q + j * 8);
        const f32x4 kj = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
            k_buf, k_off + j * 32, (int)((unsigned)kt * (unsigned)(kF32Keys * D * 4)), 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) s = mfma_f32(kj[e], qj[e], s);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    load_v(kt, 1);
    __builtin_amdgcn_sched_barrier(0);
    const int k0 = kt * kF32Keys;
    // exp2f takes four instructions more than the bare instruction, 3 to 8 % of the call if taken for every
    // weight: only tiles with a weight below 2^-126 take it (masked scores count as they are: their weights
    // are zero either way)
    float least = s[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) least = fminf(least, s[i]);
    if constexpr (partial) {
      int past = lim - k0 - hi * 4;  // (evaluated here: the loop has no registers for 16 constants)
      asm volatile("" : "+v"(past));
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if ((i >> 2) * 8 + (i & 3) > past) s[i] = -INFINITY;
    }
    float mx = s[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
    const float m_new = fmaxf(m, pair_max(mx));
    if (__builtin_amdgcn_ballot_w64(m_new > m) != 0) {
      const float al = weight(m, m_new, c2);
      m = m_new;
      l *= al;
#pragma unroll
      for (int cb = 0; cb < C::kBlocks; ++cb)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[cb][i] *= al;
    }
    const bool wide = __builtin_amdgcn_ballot_w64((least - m) * c2 < kWide) != 0;  // (uniform)
    const bool tiny = wide && __builtin_amdgcn_ballot_w64((least - m) * c2 < kTiny) != 0;
    if (tiny) {
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] = weight(s[i], m, c2);
    } else {
      const float ref = m == -INFINITY ? 0.f : m;
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] = fast_exp2((s[i] - ref) * c2);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) l += s[i];
    // O^T += V^T P^T.  Values that are infinite, NaN or about to overflow have no parts, and the last parts of the
    // smallest weights, or of minute values, would be lost: their tiles take the fp32 matrix instructions.
    // Minute values count by themselves where a channel has no others, or where
    // queries give the others no weight (looked for on tiles with such weights, or masked ones, only).
    // (Those tiles used to take both products, the smallest weights on one and the others on the other: T=2000 H=16,
    // softmax scale 2, where nearly all tiles are of that kind: d=64 99 -> 78 us, d=128 173 -> 147; on fp32
    // instructions throughout 84 and 165.)
    bool has_parts = true;
#pragma unroll
    for (int cb = 0; cb < C::kBlocks; ++cb) {  // (a lane's channels, one by one)
      float largest = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) largest = __builtin_elementwise_maximum(largest, fabsf(vf[i][cb]));
      has_parts = has_parts && largest < kLargest && (largest == 0.f || largest > kLeast);
    }
    if (partial || wide) {
      unsigned least_v = 0xffffffffu;
#pragma unroll
      for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int cb = 0; cb < C::kBlocks; ++cb)
          least_v = min(least_v, 2 * __builtin_bit_cast(unsigned, vf[i][cb]) - 1);  // (of zeros the largest number)
      has_parts = has_parts && least_v >= 2 * kLeastSplit - 1;
    }
    const bool plain = __builtin_amdgcn_ballot_w64(!has_parts) == 0;
    const bool by_parts = plain && !tiny;  // (uniform)
    if (!by_parts) {
      if (plain || !(partial && p.causal)) {  // (uniform)
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
          for (int cb = 0; cb < C::kBlocks; ++cb) o[cb] = mfma_f32(vf[i][cb], s[i], o[cb]);
      } else {
        // On a tile that the diagonal crosses a key's weight is zero for the queries before it, but zero times
        // an infinite or NaN value is not: the visible (key, query) pairs are taken one by one.  (One tile
        // per workgroup at most is crossed by the diagonal: one wave uses p_tile.)
        int h = hi, q = l32;  // (addresses formed here, not kept across the loop)
        asm volatile("" : "+v"(h), "+v"(q));
#pragma unroll
        for (int i = 0; i < 16; ++i) p_tile[(i >> 2) * 8 + h * 4 + (i & 3)][q] = s[i];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        for (int key = k0; key < min(T, k0 + kF32Keys); ++key) {
          const float wk = p_tile[key - k0][q];
          const float* vr = Vb + (size_t)key * D;
#pragma unroll
          for (int i = 0; i < 16; ++i)
#pragma unroll
            for (int cb = 0; cb < C::kBlocks; ++cb) {
              const float x = fmaf(wk, vr[((i >> 2) * 8 + h * 4 + (i & 3)) * C::kBlocks + cb], o[cb][i]);
              o[cb][i] = key <= lim ? x : o[cb][i];
            }
        }
      }
    }
    auto p_parts = [&](int hf) {
      const float x[8] = {s[8 * hf], s[8 * hf + 1], s[8 * hf + 2], s[8 * hf + 3],
                          s[8 * hf + 4], s[8 * hf + 5], s[8 * hf + 6], s[8 * hf + 7]};
      return split8(x);
    };
    auto v_parts = [&](int hf, int cb) {
      const float x[8] = {vf[8 * hf][cb], vf[8 * hf + 1][cb], vf[8 * hf + 2][cb], vf[8 * hf + 3][cb],
                          vf[8 * hf + 4][cb], vf[8 * hf + 5][cb], vf[8 * hf + 6][cb], vf[8 * hf + 7][cb]};
      return split8(x);
    };
    auto products = [&](int hf) {
      const Parts pp = p_parts(hf);
#pragma unroll
      for (int cb = 0; cb < C::kBlocks; ++cb) {
        const Parts va = v_parts(hf, cb);
        o[cb] = mfma_16(va.p[0], pp.p[0], o[cb]);
        o[cb] = mfma_16(va.p[0], pp.p[1], o[cb]);
        o[cb] = mfma_16(va.p[1], pp.p[0], o[cb]);
        o[cb] = mfma_16(va.p[0], pp.p[2], o[cb]);
        o[cb] = mfma_16(va.p[2], pp.p[0], o[cb]);
        o[cb] = mfma_16(va.p[1], pp.p[1], o[cb]);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    load_k(k_next, 0);
    if (by_parts) products(0);
    load_k(k_next, 1);
    __builtin_amdgcn_sched_barrier(0);
    if (by_parts) products(1);
  };
  int kt = wave;
  for (; kt < n_full; kt += NW) fold_tile(kt, std::false_type{});
  if (kt < nt) fold_tile(kt, std::true_type{});
  if (L > 0 && !depth_first) depth_rows();

  // ---- fold the partial softmaxes: (max, normaliser) of each wave, then the outputs, each scaled
  // to the common reference, summed 64 channels at a time
  l = pair_sum(l);
  if (hi == 0) {
    stat_m[wave][l32] = m;
    stat_l[wave][l32] = l;
  }
  __syncthreads();  // (also: every wave is done with the queries in LDS)
  const int n_part = NW + (L > 0 ? 1 : 0);
  {
    float mt = stat_m[0][l32];
    for (int w = 1; w < n_part; ++w) mt = fmaxf(mt, stat_m[w][l32]);
    const float f = weight(m, mt, c2);
#pragma unroll
    for (int cb = 0; cb < C::kBlocks; ++cb)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[cb][i] *= f;
  }
  // thread: a row, 8 (with eight waves 4) of the round's 64 channels
  constexpr int TPR = NW * 64 / kF32Rows, CPT = 64 / TPR;
  const int row = tid / TPR, ch = tid % TPR * CPT, t = q0 + row;
  float mt = stat_m[0][row];
  for (int w = 1; w < n_part; ++w) mt = fmaxf(mt, stat_m[w][row]);
  float lt = 0.f;
  for (int w = 0; w < n_part; ++w) lt += stat_l[w][row] * weight(stat_m[w][row], mt, c2);
  const float fd = L > 0 ? weight(stat_m[NW][row], mt, c2) : 0.f;
  const float inv = 1.0f / lt;
#pragma unroll
  for (int rd = 0; rd < C::kRounds; ++rd) {
    if (rd > 0) __syncthreads();
    float* xw = shared + wave * C::kXWave + l32 * C::kXRow;
    // output row r (of 32) of the blocks = channels r * kBlocks ..: 64 channels are 64 / kBlocks rows
#pragma unroll
    for (int i = rd * (16 / C::kRounds); i < (rd + 1) * (16 / C::kRounds); ++i) {
      const int c0 = ((i >> 2) * 8 + hi * 4 + (i & 3)) * C::kBlocks - rd * 64;
      if constexpr (D == 128) *(f32x4*)(xw + c0) = (f32x4){o[0][i], o[1][i], o[2][i], o[3][i]};
      else *(f32x2*)(xw + c0) = (f32x2){o[0][i], o[1][i]};
    }
    __syncthreads();
    f32x4 x[CPT / 4];
#pragma unroll
    for (int k = 0; k < CPT / 4; ++k) {
      x[k] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < NW; ++w) x[k] += *(const f32x4*)(shared + w * C::kXWave + row * C::kXRow + ch + 4 * k);
      if (L > 0) x[k] += *(const f32x4*)(depth_o + row * C::kRow + rd * 64 + ch + 4 * k) * fd;
      if (t < T) *(f32x4*)((float*)p.O + ((size_t)bh * T + t) * D + rd * 64 + ch + 4 * k) = x[k] * inv;
    }
  }
  if (tid % TPR == 0 && t < T) p.LSE[(size_t)bh * T + t] = mt * p.scale + logf(lt);
}

// Few tiles are bound by the chains of a wave's key tiles and slots, which eight waves to a workgroup halve.  (The kernel of
// few tiles has the plain name, by which the smallest call is known; the one of four waves had it while there was no other.)
template <int D>
__global__ __launch_bounds__(512, 2) void moda_fwd_f32_kernel(FwdParams p) {
  fwd_f32_tile<D, 8>(p);
}
template <int D>
__global__ __launch_bounds__(256, D == 64 ? 3 : 2) void moda_fwd_f32_four_kernel(FwdParams p) {
  fwd_f32_tile<D, 4>(p);
}

int fwd_f32_tile_rows() { return kF32Rows; }
// Eight waves while every workgroup has a unit of its own, unless there is no chain to halve (four / eight, us, tiles of
// 32 queries; d = 64: H=2 T=20, 31 slots 17.3 / 11.8;  B=2 H=16 T=112, 15 slots 14.9 / 12.0;  H=4 T=1669, 15 slots, 212 tiles 38.3 / 32.2;
// H=2 T=256, 4 slots 10.0 / 9.9;  288 tiles, T=548 21.3 / 21.0;  384 tiles 48.2 / 52.3;  no slots: H=8 T=56 6.2 / 6.8.
// d = 128: H=2 T=25, 31 slots 26.8 / 18.5;  160 tiles, T=141, 7 slots 19.3 / 17.1;  208 tiles, T=403, 24 slots 40.4 / 41.1;  256
// tiles, T=31, 4 slots 16.9 / 15.6;  416 tiles, T=404, 31 slots 94 / 106;  no slots: H=8 T=344 15.9 / 15.4, T=204 12.9 / 13.4.
// Three chunks of slots in flight instead of two: 1.03 of the time.)  One slot is no chain either at d = 128, where the fold
// is longer (T=107 11.9 / 12.4, T=246 15.2 / 15.9, 128 to 192 positions 0.98; d = 64: 0.96 to 0.99).
bool fwd_f32_eight_waves(const FwdParams& p, int d) {
  return (long long)p.B * p.Hq * ((p.T + kF32Rows - 1) / kF32Rows) <= 256 && (p.depth_count > (d == 128 ? 1 : 0) || p.T > 256);
}

hipError_t launch_fwd_f32(const FwdParams& p, int d, hipStream_t stream) {
  if (fwd_f32_by_rows(p)) return launch_fwd_f32_rows(p, d, stream);
  if (p.n_qtiles != (p.T + kF32Rows - 1) / kF32Rows) return hipErrorInvalidValue;
  const long long blocks = (long long)p.B * p.Hq * p.n_qtiles;
  const bool eight = fwd_f32_eight_waves(p, d);
  if (!grid_ok(blocks, eight ? 512 : 256)) return kGridTooLarge;
  dim3 grid((unsigned)blocks), block(eight ? 512 : 256);
  if (d == 128) return launch_kernel(eight ? moda_fwd_f32_kernel<128> : moda_fwd_f32_four_kernel<128>, grid, block, stream, p);
  if (d == 64) return launch_kernel(eight ? moda_fwd_f32_kernel<64> : moda_fwd_f32_four_kernel<64>, grid, block, stream, p);
  return hipErrorInvalidValue;
}

}  // namespace moda
