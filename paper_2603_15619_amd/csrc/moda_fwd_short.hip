// MoDA attention forward, bf16, for calls with few query tiles (gfx950 MFMA).
//
// The kernel of moda_fwd_bf16.hip walks the key tiles of 128 or 256 (position, head) pairs one after
// the other; a call of a few hundred such tiles leaves most of the chip waiting for the last ones.
// Here a workgroup = 32 pairs of one key/value head (32 / GT positions x GT heads of a group, as a
// wave there) and its 4 waves DEAL OUT THE KEYS: key tile i (32 keys) belongs to wave i % 4, which
// copies it into LDS of its own and keeps a running (max, normaliser, output) of its own; no
// workgroup barrier in the loop.  At the end the waves' states are folded into one softmax through
// LDS.  Four times the workgroups (eight times, against 256 pairs) with a quarter of the steps each;
// in return K and V are read from the L2 once per 32 pairs.
//
// Depth slots.  One head per tile: on the vector ALUs, d/8 lanes per row, 8 of the 32 rows per wave,
// before the key tiles in every other workgroup and after them in the others, as a fifth partial
// state that stays in registers meanwhile.  Several heads per tile: the slots of the tile's
// positions are 32-key blocks on the matrix pipe (key kk belongs to position kk / L), dealt out to
// the waves after the key tiles, or in every other workgroup before them (alternate_blocks).
//
// Bound by a wave's chain copy -> products -> exponentials -> products on the key tiles and by HBM on
// the depth slots.  B=1 H=8 T=2048, 4 slots: d=64 33 -> 17 us, d=128 43 -> 29 us;
// B=1 H=2 T=16384 d=64: 203 -> 123 us.
//
// K and V have one LDS tile each per wave; the next tile's K is requested as soon as the scores of
// this one are formed and its V as soon as the output product has read it, so that several
// workgroups fit a compute unit and cover each other's latency.
#include "moda_launch.h"
#include "moda_tile.h"

namespace moda {

constexpr int kShortCols = 32;  // (position, head) pairs per workgroup
constexpr int kShortWaves = 4;

// ROWS: depth slots of one head per tile are taken on the vector ALUs, as a fifth partial state.
template <int D, bool ROWS>
struct FwdShortCfg {
  static constexpr int kTile = 32 * D * 2;           // a K or V tile of 32 keys
  static constexpr int kPieces = kTile / 1024;       // copy instructions per tile
  static constexpr int kXRow = 64 + 4;               // states are exchanged 64 channels at a time
  static constexpr int kXPart = kShortCols * kXRow;  // floats of one partial state
  static constexpr int kTiles = kShortWaves * 2 * kTile;
  static constexpr int kExchange = (kShortWaves + (ROWS ? 1 : 0)) * kXPart * 4;
  static constexpr int kLds = kTiles > kExchange ? kTiles : kExchange;
};

// (at d = 64 without a fifth state four workgroups fit a compute unit)
template <int D, bool ROWS>
__global__ __launch_bounds__(kShortWaves * 64, D == 128 ? 2 : ROWS ? 3 : 4) void moda_fwd_short_kernel(FwdParams p) {
  using Tl = Tile<D>;
  using C = FwdShortCfg<D, ROWS>;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[C::kLds];
  __shared__ float stat_m[kShortWaves + 1][kShortCols], stat_l[kShortWaves + 1][kShortCols];

  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // ---- what this workgroup computes (heavy, i.e. late, tiles first; see moda_fwd_bf16.hip for the walk)
  const int G = p.Hq / p.Hk, GT = p.heads_per_tile, sub = G / GT;
  const int gt_shift = __builtin_ctz(GT), PW = kShortCols >> gt_shift;  // positions per tile
  int tbh, tile;
  head_blocked_id((int)blockIdx.x, p.B * p.Hk * sub, p.n_qtiles, tbh, tile, p.head_group);
  const int bg = tbh / sub, b = bg / p.Hk;
  const int hb = b * p.Hq + (bg - b * p.Hk) * G + (tbh - bg * sub) * GT;  // first head of the tile
  const int q0 = (p.n_qtiles - 1 - tile) * PW;
  const int T = p.T, L = p.depth_count;
  const float c2 = p.scale_log2;
  const size_t drow = (size_t)p.depth_alloc * Tl::kRowBytes;  // bytes of one position's slots

  // ---- depth slots, one head per tile: rows wave * 8 ... + 7, 64 / (d/8) at a time
  constexpr int LPR = Tl::kChunks, RPS = 64 / LPR, NIT = 8 / RPS;
  constexpr bool rows_on_valu = ROWS;
  float d_o[NIT][8], d_m[NIT], d_l[NIT];
  auto depth_rows = [&]() {
    constexpr int kC = 5;  // slots per step, the next step's in flight
    const int rg = lane / LPR, lc = lane % LPR;
    const int nch = (L + kC - 1) / kC;
    struct Chunk {
      u32x4 k[kC], v[kC];
    };
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int t = min(q0 + wave * 8 + it * RPS + rg, T - 1);  // rows past the end are never stored
      const u32x4 q = *(const u32x4*)((const char*)p.Q + ((size_t)hb * T + t) * Tl::kRowBytes + lc * 16);
      const char* kd = (const char*)p.Kdepth + ((size_t)bg * T + t) * drow + lc * 16;
      const char* vd = (const char*)p.Vdepth + ((size_t)bg * T + t) * drow + lc * 16;
      float m = -INFINITY, l = 0.f, o[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) o[k] = 0.f;
      auto issue = [&](int c, Chunk& x) {
#pragma unroll
        for (int u = 0; u < kC; ++u) {  // (past depth_count: the last attended slot again, ignored)
          const size_t off = (size_t)min(c * kC + u, L - 1) * Tl::kRowBytes;
          x.k[u] = __builtin_nontemporal_load((const u32x4*)(kd + off));
          x.v[u] = __builtin_nontemporal_load((const u32x4*)(vd + off));
        }
      };
      auto fold = [&](int c, const Chunk& x) {
        float s[kC], mn = m;
#pragma unroll
        for (int u = 0; u < kC; ++u) {
          float a = 0.f;
#pragma unroll
          for (int k = 0; k < 4; ++k) a = dot2_bf16(q[k], x.k[u][k], a);
          a = group_sum<LPR>(a);
          s[u] = c * kC + u < L ? a : -INFINITY;
          mn = fmaxf(mn, s[u]);
        }
        // (no slot of finite score so far: the state stays empty, the weights are exp2(-inf) = 0)
        const float al = mn == -INFINITY ? 0.f : fast_exp2((m - mn) * c2), mc = mn == -INFINITY ? 0.f : mn * c2;
        m = mn;
        l *= al;
#pragma unroll
        for (int k = 0; k < 8; ++k) o[k] *= al;
#pragma unroll
        for (int u = 0; u < kC; ++u) {
          if (c * kC + u >= L) break;  // (uniform)
          const float w = fast_exp2(s[u] * c2 - mc);
          l += w;
          // weight rounded to bf16, as for the sequence keys
          const uint32_t w_lo = pack_bf16(w, 0.f), w_hi = w_lo << 16;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            o[2 * k] = dot2_bf16(w_lo, x.v[u][k], o[2 * k]);
            o[2 * k + 1] = dot2_bf16(w_hi, x.v[u][k], o[2 * k + 1]);
          }
        }
      };
      Chunk xa, xb;
      issue(0, xa);
      for (int c = 0; c < nch; c += 2) {
        issue(min(c + 1, nch - 1), xb);
        fold(c, xa);
        if (c + 1 < nch) {
          issue(min(c + 2, nch - 1), xa);
          fold(c + 1, xb);
        }
      }
      d_m[it] = m;
      d_l[it] = l;
#pragma unroll
      for (int k = 0; k < 8; ++k) d_o[it][k] = o[k];
    }
  };
  const bool depth_first = rows_on_valu && ((blockIdx.x >> 3) & 1) != 0;

  // ---- tiles: sequence keys, then (several heads per tile) the blocks of depth slots
  const int n_keys = p.causal ? min(T, q0 + PW) : T;
  const int nt = (n_keys + 31) / 32;
  const int nd = L > 0 && GT > 1 ? PW * L : 0;  // depth slots of the tile's positions
  const int n_blocks = (nd + 31) / 32, n_tiles = nt + n_blocks;
  // the order in which they are dealt out: every other workgroup its blocks of slots first, where that pays
  const bool blocks_first = !ROWS && p.depth_mfma == 2 && ((blockIdx.x >> 3) & 1) != 0;
  auto tile_of = [&](int n) { return !blocks_first || n >= n_tiles ? n : n < n_blocks ? nt + n : n - n_blocks; };
  const unsigned k_tile = (unsigned)(size_t)(lds_ptr)smem + wave * 2 * C::kTile, v_tile = k_tile + C::kTile;
  FragAddr<D> fa;
  fa.init(lane);
  const i32x4 k_buf = make_tile_buffer((const char*)p.Kseq + (size_t)bg * T * Tl::kRowBytes, (unsigned)T * Tl::kRowBytes);
  const i32x4 v_buf = make_tile_buffer((const char*)p.Vseq + (size_t)bg * T * Tl::kRowBytes, (unsigned)T * Tl::kRowBytes);
  // (depth slots: buffers from the tile's first position to the end of the (batch, head) slab)
  const size_t left = (size_t)(T - q0) * drow;
  const unsigned recs = nd == 0 ? 0u : left < 0xffffff00ull ? (unsigned)left : 0xffffff00u;
  const i32x4 kd_buf = make_tile_buffer((const char*)p.Kdepth + ((size_t)bg * T + q0) * drow, recs);
  const i32x4 vd_buf = make_tile_buffer((const char*)p.Vdepth + ((size_t)bg * T + q0) * drow, recs);
  const int jr = lane / Tl::kChunks, pc = lane % Tl::kChunks;  // this lane's row and chunk position in a piece
  const int goff = jr * Tl::kRowBytes + ((pc ^ Tl::swz(jr)) << 4);
  // one K or V tile, global -> LDS; always kPieces operations (a tile past the last: none of its lanes
  // is in range, zeros arrive)
  auto copy = [&](const i32x4& seq, const i32x4& depth, unsigned dst, int n) {
    const int i = tile_of(n);
    if (i < nt) {
#pragma unroll
      for (int q = 0; q < C::kPieces; ++q)
        tile_copy16(seq, xor_here(goff, TileLoader<D>::piece_xor(q)), (int)((unsigned)i * (unsigned)C::kTile) + q * 1024,
                    dst + q * 1024);
    } else {
#pragma unroll
      for (int q = 0; q < C::kPieces; ++q) {
        const int r = q * (64 / Tl::kChunks) + jr;
        const unsigned kk = (unsigned)((i - nt) * 32 + r);
        const unsigned pos = L == 1 ? kk : __umulhi(kk, p.depth_magic);  // kk / L
        const unsigned slot = kk - pos * (unsigned)L;
        const unsigned off = (pos * (unsigned)p.depth_alloc + slot) * (unsigned)Tl::kRowBytes + ((pc ^ Tl::swz(r)) << 4);
        tile_copy16(depth, kk < (unsigned)nd ? (int)off : (int)0xffffff80u, 0, dst + q * 1024);
      }
    }
  };

  if (depth_first) depth_rows();

  // Q fragments (B operand: column l32 = position l32 / GT, head l32 % GT)
  bf16x8 qf[Tl::kDSteps];
  const int t_col = q0 + (l32 >> gt_shift);
  {
    const char* q = (const char*)p.Q + ((size_t)(hb + (l32 & (GT - 1))) * T + min(t_col, T - 1)) * Tl::kRowBytes + hi * 16;
#pragma unroll
    for (int st = 0; st < Tl::kDSteps; ++st) qf[st] = *(const bf16x8*)(q + st * 32);
  }
  f32x16 o[Tl::kDBlocks];
#pragma unroll
  for (int db = 0; db < Tl::kDBlocks; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[db][i] = 0.f;
  float m = -INFINITY, l = 0.f;
  const int lim = p.causal ? min(t_col, T - 1) : T - 1;  // last visible key of this lane's column

  if (wave < n_tiles) {
    copy(k_buf, kd_buf, k_tile, wave);
    copy(v_buf, vd_buf, v_tile, wave);
  }
  for (int n = wave; n < n_tiles; n += kShortWaves) {
    const int i = tile_of(n);
    wait_own_copies<C::kPieces>();  // this tile's K (its V was requested after it)
    const unsigned b_row = fa.row + k_tile, b_tr = fa.tr + v_tile, b_tr8 = fa.tr8 + v_tile;
    // two accumulation chains
    f32x16 s, s1;
#pragma unroll
    for (int k = 0; k < 16; ++k) s[k] = s1[k] = 0.f;
#pragma unroll
    for (int st = 0; st < Tl::kDSteps; st += 2) {
      s = mfma_bf16(FragAddr<D>::row_frag((unsigned)xor_here((int)b_row, st << 5), 0, 0), qf[st], s);
      s1 = mfma_bf16(FragAddr<D>::row_frag((unsigned)xor_here((int)b_row, (st + 1) << 5), 0, 0), qf[st + 1], s1);
    }
    wait_own_reads();  // the K tile has been read: it may be overwritten
    copy(k_buf, kd_buf, k_tile, n + kShortWaves);
#pragma unroll
    for (int k = 0; k < 16; ++k) s[k] += s1[k];
    if (i >= nt) {  // (uniform) slot r of the block is attended by the columns of its position
      const unsigned lo = (unsigned)((l32 >> gt_shift) * L - (i - nt) * 32);
#pragma unroll
      for (int k = 0; k < 16; ++k)
        s[k] = (unsigned)((k >> 2) * 8 + hi * 4 + (k & 3)) - lo < (unsigned)L ? s[k] : -INFINITY;
    } else if (i * 32 + 32 > T || (p.causal && i * 32 + 31 > q0)) {  // (uniform) the diagonal, keys past the end
      const int past = lim - i * 32 - hi * 4;
#pragma unroll
      for (int k = 0; k < 16; ++k) s[k] = (k >> 2) * 8 + (k & 3) <= past ? s[k] : -INFINITY;
    }
    float mx = s[0];
#pragma unroll
    for (int k = 1; k < 16; ++k) mx = fmaxf(mx, s[k]);
    mx = pair_max(mx);
    // the reference max is raised lazily: weights stay below 2^8 (see moda_fwd_bf16.hip)
    const bool raise = (mx - m) * c2 > 8.f;
    if (__builtin_amdgcn_ballot_w64(raise) != 0) {
      const float mn = fmaxf(m, mx);
      const float al = mn == m ? 1.f : fast_exp2((m - mn) * c2);  // (a column that has seen no key stays empty)
      m = mn;
      l *= al;
#pragma unroll
      for (int db = 0; db < Tl::kDBlocks; ++db)
#pragma unroll
        for (int k = 0; k < 16; ++k) o[db][k] *= al;
    }
    const float mc = m == -INFINITY ? 0.f : m * c2;
    bf16x8 pb[2];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      float e[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        e[k] = fast_exp2(s[hf * 8 + k] * c2 - mc);
        l += e[k];
      }
      pb[hf] = pack8(e);
    }
    wait_own_copies<C::kPieces>();  // this tile's V (the next tile's K was requested after it)
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int db = 0; db < Tl::kDBlocks; ++db)
        o[db] = mfma_bf16(FragAddr<D>::tr_frag((unsigned)xor_here((int)b_tr, db << 6), (unsigned)xor_here((int)b_tr8, db << 6),
                                               hf, 0), pb[hf], o[db]);
    wait_own_reads();
    copy(v_buf, vd_buf, v_tile, n + kShortWaves);
  }
  if (rows_on_valu && !depth_first) depth_rows();

  // ---- fold the partial states: references and normalisers, then the outputs, each scaled to the
  // common reference, summed 64 channels at a time
  l = pair_sum(l);
  if (hi == 0) {
    stat_m[wave][l32] = m;
    stat_l[wave][l32] = l;
  }
  const int n_part = kShortWaves + (rows_on_valu ? 1 : 0);
  if (rows_on_valu && lane % LPR == 0) {
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      stat_m[kShortWaves][wave * 8 + it * RPS + lane / LPR] = d_m[it];
      stat_l[kShortWaves][wave * 8 + it * RPS + lane / LPR] = d_l[it];
    }
  }
  wait_own_copies<0>();  // (copies requested past the last tile have landed)
  __syncthreads();  // the tiles become the exchange buffer
  auto common = [&](int col) {
    float x = stat_m[0][col];
    for (int w = 1; w < n_part; ++w) x = fmaxf(x, stat_m[w][col]);
    return x;
  };
  auto factor = [&](float ref, float x) { return x == -INFINITY ? 0.f : fast_exp2((x - ref) * c2); };
  const float f_col = factor(common(l32), m);
  const int row = tid >> 3, ch = (tid & 7) * 8;  // output: 8 threads per column, 8 channels each per round
  const float ref = common(row);
  float lt = 0.f;
  for (int w = 0; w < n_part; ++w) lt += stat_l[w][row] * factor(ref, stat_m[w][row]);
  const float inv = 1.0f / lt;
  const int t = q0 + (row >> gt_shift);
  const size_t orow = (size_t)(hb + (row & (GT - 1))) * T + t;
  float* xb = (float*)smem;
#pragma unroll
  for (int rd = 0; rd < D / 64; ++rd) {
    if (rd > 0) __syncthreads();
#pragma unroll
    for (int db = rd * 2; db < rd * 2 + 2; ++db)
#pragma unroll
      for (int bq = 0; bq < 4; ++bq)
        *(f32x4*)(xb + wave * C::kXPart + l32 * C::kXRow + (db - rd * 2) * 32 + bq * 8 + hi * 4) =
            (f32x4){o[db][4 * bq] * f_col, o[db][4 * bq + 1] * f_col, o[db][4 * bq + 2] * f_col, o[db][4 * bq + 3] * f_col};
    if (rows_on_valu && (lane % LPR) * 8 / 64 == rd) {
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const int r = wave * 8 + it * RPS + lane / LPR;
        const float f = factor(common(r), d_m[it]);
        float* dst = xb + kShortWaves * C::kXPart + r * C::kXRow + (lane % LPR) * 8 - rd * 64;
        *(f32x4*)dst = (f32x4){d_o[it][0] * f, d_o[it][1] * f, d_o[it][2] * f, d_o[it][3] * f};
        *(f32x4*)(dst + 4) = (f32x4){d_o[it][4] * f, d_o[it][5] * f, d_o[it][6] * f, d_o[it][7] * f};
      }
    }
    __syncthreads();
    f32x4 x0 = {0.f, 0.f, 0.f, 0.f}, x1 = x0;
    for (int w = 0; w < n_part; ++w) {
      x0 += *(const f32x4*)(xb + w * C::kXPart + row * C::kXRow + ch);
      x1 += *(const f32x4*)(xb + w * C::kXPart + row * C::kXRow + ch + 4);
    }
    if (t < T)
      *(u32x4*)((char*)p.O + orow * Tl::kRowBytes + (rd * 64 + ch) * 2) =
          (u32x4){pack_bf16(x0[0] * inv, x0[1] * inv), pack_bf16(x0[2] * inv, x0[3] * inv),
                  pack_bf16(x1[0] * inv, x1[1] * inv), pack_bf16(x1[2] * inv, x1[3] * inv)};
  }
  if ((tid & 7) == 0 && t < T) p.LSE[orow] = ref * p.scale + __logf(lt);
}

int fwd_short_tile_pairs() { return kShortCols; }

// Blocks of slots that all workgroups take last come all at once, and HBM idles before.  Every other workgroup takes them
// first where units hold several workgroups and the slots are a good part of the call (last / alternating, us, d = 64:
// B=2 Hq=16 Hk=8 T=1000, 12 slots 18.7 / 17.5;  1024 tiles, G=2 T=511, 15 slots 18.2 / 16.1;  760 tiles, G=4 T=593, 64 slots 23.9 / 21.0;
// 832, G=8 T=829, 64 slots 17.3 / 15.7;  but 720, G=8 T=1416, 4 slots 13.2 / 13.7;  528, G=4 T=2093, 4 slots 16.0 / 16.5;  744,
// G=2 T=2969, 7 slots 23.7 / 23.9;  336, G=4 T=238, 64 slots 8.8 / 9.5).  The lines, from 12700 calls (alternating, of the time of last):
// more than 512 workgroups (up to 512 1.00 to 1.05) and no second round of them (1024 at d = 64: 1.01 to 1.03); five slots to a head
// of the group, whose queries share what is read (d = 64: 0.97 from there on; two heads 8 / 9 / 10 / 11 / 12 slots 1.005 / 1.002 / 0.998 /
// 0.992 / 0.989, eight heads 15 to 31 1.01); up to 100 positions to a slot; heads in fours, as with an odd number of them neighbouring
// workgroups do not alternate (0.97 / 0.97 / 0.98 / 0.995 of multiples of 8, 4, 2 and odd numbers, B=15 Hq=2 T=1018, 64 slots 53 / 61).
// d = 128 the same: 0.96.
static bool alternate_blocks(const FwdParams& p, long long blocks) {
  const int G = p.Hq / p.Hk;
  return blocks > 512 && blocks <= 1024 && p.depth_count >= 5 * G && p.T <= 100ll * p.depth_count && (long long)p.B * p.Hk % 4 == 0;
}

hipError_t launch_fwd_short(const FwdParams& params, int d, hipStream_t stream) {
  FwdParams p = params;
  const int gt = p.heads_per_tile, pos = kShortCols / gt;
  if (gt < 1 || gt > kShortCols || (gt & (gt - 1)) != 0 || (p.Hq / p.Hk) % gt != 0) return hipErrorInvalidValue;
  if (p.n_qtiles != (p.T + pos - 1) / pos) return hipErrorInvalidValue;
  const long long blocks = (long long)p.B * (p.Hq / gt) * p.n_qtiles;
  if (!grid_ok(blocks, kShortWaves * 64)) return kGridTooLarge;
  if (p.depth_mfma && alternate_blocks(p, blocks)) p.depth_mfma = 2;
  dim3 grid((unsigned)blocks), block(kShortWaves * 64);
  if (d != 64 && d != 128) return hipErrorInvalidValue;
  const bool rows = p.depth_count > 0 && gt == 1;
  const auto kernel = d == 128 ? (rows ? moda_fwd_short_kernel<128, true> : moda_fwd_short_kernel<128, false>)
                               : (rows ? moda_fwd_short_kernel<64, true> : moda_fwd_short_kernel<64, false>);
  return launch_kernel(kernel, grid, block, stream, p);
}

}  // namespace moda
