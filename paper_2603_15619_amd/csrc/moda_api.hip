// libmoda C ABI: argument validation and kernel dispatch (host code only).
#include <algorithm>
#include <math.h>
#include <stdio.h>

#include "../../include/moda.h"
#include "moda_launch.h"

namespace {

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

constexpr int kMaxDepthAlloc = 8192;  // a tile's depth slots are addressed with 32-bit offsets

// Checks shared by every call: dimensions, dtype, head dimension, scale.
moda_status check_dims(const moda_shape* s) {
  if (!s) return MODA_ERR_NULL;
  if (s->B < 0 || s->T < 0 || s->Hq <= 0 || s->Hk <= 0 || s->d <= 0) return MODA_ERR_SHAPE;
  if (s->Hq % s->Hk != 0) return MODA_ERR_SHAPE;
  if (s->depth_count < 0 || s->depth_alloc < s->depth_count) return MODA_ERR_SHAPE;
  if (s->causal != 0 && s->causal != 1) return MODA_ERR_SHAPE;
  if (s->dtype != MODA_F32 && s->dtype != MODA_BF16) return MODA_ERR_UNSUPPORTED;
  if (s->d != 64 && s->d != 128) return MODA_ERR_UNSUPPORTED;
  if (!(s->scale == s->scale) || isinf(s->scale)) return MODA_ERR_SHAPE;  // NaN / inf
  if (s->depth_alloc > kMaxDepthAlloc) return MODA_ERR_UNSUPPORTED;
  // element counts that the kernels keep in 32-bit integers
  if ((long long)s->B * s->Hq > 0x7fffffffLL) return MODA_ERR_UNSUPPORTED;
  return MODA_OK;
}

// One (batch, head) slab of `rows` sequence rows must stay below 4 GiB: the kernels address a
// sequence tensor with 32-bit byte offsets inside a slab.  (The depth tensors are addressed
// from a 64-bit base per tile and have no such limit.)
bool slab_ok(const moda_shape* s, long long rows) {
  const unsigned long long esz = s->dtype == MODA_BF16 ? 2 : 4;
  return (unsigned long long)rows * (unsigned long long)s->d * esz < (1ull << 32);
}

// Shape checks of the calls that take [B, H, T, d] tensors (forward, backward, write step).
moda_status check_shape(const moda_shape* s) {
  const moda_status st = check_dims(s);
  if (st != MODA_OK) return st;
  return slab_ok(s, s->T) ? MODA_OK : MODA_ERR_UNSUPPORTED;
}

moda_status launch_status(hipError_t e) {
  if (e == hipSuccess) return MODA_OK;
  return e == moda::kGridTooLarge ? MODA_ERR_UNSUPPORTED : MODA_ERR_LAUNCH;
}

// Geometry of the bf16 forward kernel (see moda_fwd_bf16.hip): workgroups of 8 waves (256 (position, head)
// pairs) or of 4 (128 pairs), which copy every K/V tile from the L2 twice as often.
// d = 128: two waves per SIMD, so one workgroup of 8 or two of 4 per compute unit.  Long
// sequences in large grids take 8.  4 waves take
//   - grids that would leave compute units without work;
//   - sequences of up to 512 pairs, which 8 waves pad to 256, and whose ends weigh more than their copies
//     (4 / 8 waves, us, one head per tile: 12 slots T=128, 768 tiles of 128: 127 / 171, but with many slots and
//     little padding 8 take over where they fill the chip just once, or in two rounds and more (256 heads, 12 slots: T=256
//     84.6 / 82.3, T=200 71.2 / 71.9; 128 heads T=512 96.2 / 90.8;  1024 heads, 15 slots: T=200 324 / 326, T=239 382 / 372, T=400
//     745 / 738, T=512 892 / 863; 7 slots T=239 216 / 225; 256 heads, 31 slots T=512 376 / 366);
//   - one and a half rounds of workgroups of 8 waves, whose last half round 4 waves spread over all units
//     (768 tiles: 12 slots T=2000 not causal 168 / 187, causal T=1000 138 / 150; causal and longer 0.92 to 1.14:
//     not there).
// d = 64: four waves per SIMD, two workgroups of 8 or four of 4 per unit, and 4 waves up to one and a half rounds
//   of 8 (B=5 H=16 T=1020, 640 tiles, 15 slots 68 / 82 us; T=4720 32 heads on 4, 1184 tiles 108 / 114; T=11652 16 on 4, 1472
//   tiles 303 / 311; T=4570, 1728 tiles 143.3 / 143.7; B=8 H=16 T=2048, 2048 tiles 93 / 89) and for up to 1024 pairs
//   (B=16 H=16 T=1024, 2048 tiles 53.0 / 53.5; B=15 32 on 8 T=515 37 / 40).
int fwd_waves_per_workgroup(const moda_shape* s, int heads_per_tile) {
  const long long heads = (long long)s->B * s->Hq / heads_per_tile, pairs = (long long)s->T * heads_per_tile;
  const long long n = heads * ((pairs + 255) / 256);
  if (s->d == 64) return n <= 768 || pairs <= 1024 ? 4 : 8;
  if (n < 256) return 4;
  if (pairs <= 512) return heads_per_tile == 1 && s->depth_count >= 12 && (n == 256 || n >= 512) && 10 * heads * pairs > 9 * 256 * n ? 8 : 4;
  return n > 256 && n <= 448 && (!s->causal || s->T <= 1024) ? 4 : 8;
}

// Waves that share a SIMD in the bf16 forward kernel: four at d = 64, but two while two workgroups of 4 waves
// per unit hold the grid: a third and fourth wave are not there then, and the step for two, of a whole tile, is
// a little faster (two / four, us: T=1338, 352 tiles 19.1 / 20.4; T=13133, 412 tiles 143 / 147; T=900, 512 tiles 16.2 / 16.6;
// T=4096, 512 tiles 49 / 53; 640 tiles 25.4 / 25.3; with slots of one head per tile 440 tiles 96.6 / 101.5, 512 tiles 53.7 / 52.5, 640
// tiles 75.8 / 68.3).
int fwd_waves_per_simd(const moda_shape* s, int heads_per_tile, int waves) {
  if (s->d == 128) return 2;
  const long long n = (long long)s->B * s->Hq / heads_per_tile * (((long long)s->T * heads_per_tile + 127) / 128);
  return waves == 4 && n <= (heads_per_tile == 1 && s->depth_count > 0 ? 448 : 512) ? 2 : 4;
}

// Calls that take the kernel for few tiles (moda_fwd_short.hip): n = tiles of 128 (position, head)
// pairs; the short kernel has 4 n workgroups, of which the chip holds 512 at d = 128 and, at d = 64, 768
// with depth slots of one head per tile and 1024 otherwise.  It is ahead while they fit, on causal calls
// (half of whose tiles are short) somewhat longer, on others, whose workgroups all last equally long, mostly up to 192
// (short / other kernel, us, whole call; 12 slots where there are any):
//   d=64, no slots or several heads per tile, causal:  T=128 n=384 10/15;   T=512 n=256 10/13, n=384 16/15;
//                     T=4096: n=256 32/43, n=320 42/48, n=384 45/46, n=448 54/50;   T=8192: n=320 72/91, n=384 88/89, n=448 105/95
//     not causal:     T=512 n=256 13/13;   T=640: n=240 14/16;   T=768: n=192 13/16, n=240 17/16;   T=1024: n=192 15/16, n=208 19/16;
//                     T=2048: n=176 25/28, n=192 25/25, n=208 31/28;   two heads: T=1024 n=224 23/24, n=256 24/24;  T=1536 n=240 29/28
//   d=64, slots of one head, causal:  n=192: T=128 19/21, T=1024 28/28;   T=512 n=256 30/26;   T=4096: n=224 47/60, n=256 56/54;
//                     T=8000 n=252 73/92
//   d=128, causal:    n=128: T=100 8/13, T=512 11/15, T=900 15/19;   n=160: T=512 17/15, T=1024 18/20;
//                     n=192: T=1024 23/21, T=2048 30/32, T=4096 47/57;   T=8192 n=256 107/107;   T=9000 n=213 97/113
//     slots of one head:  n=128: T=512 28/35;   n=160: T=1024 47/41, T=4096 62/76;   n=192: T=4096 72/76;   T=9000 n=213 125/132;
//                     T=8192 n=256 131/127
//     not causal:     n=128: T=512 14/15, T=2048 32/34, T=4096 54/55 (12 slots 70/76), T=8192 102/104;   n=256: T=8192 192/134
bool fwd_few_tiles(const moda_shape* s, int heads_per_tile) {
  const long long n = (long long)s->B * s->Hq * ((s->T + 127) / 128);
  const bool rows = heads_per_tile == 1 && s->depth_count > 0;
  const int T = s->T;
  int most = 128;
  if (s->d == 64 && s->causal) most = rows ? (T >= 4096 ? 256 : 192) : T <= 256 || T >= 4096 ? 384 : 256;
  else if (s->d == 64 && rows) most = 192;
  else if (s->d == 64) most = T <= 512 || (heads_per_tile == 2 && T <= 1300) ? 256 : T <= 640 ? 240 : 192;
  else if (s->causal) most = rows ? (T >= 8192 ? 240 : T >= 4096 ? 192 : 128) : T >= 8192 ? 256 : T >= 2048 ? 192 : T >= 1024 ? 160 : 128;
  return n <= most;
}

// Heads that one die (workgroup ids equal mod 8) walks together, tile by tile: as many as have
// their streamed tensors (2 * T * d bf16 elements each: K and V, or Q and dO) in its 4 MB L2, at
// least one; a power of two that divides the heads of a die.  0: the ids cannot be dealt that way.
// Forward with four waves per SIMD (d = 64): a die holds twice the workgroups, and with few heads at a time its
// last rounds are the tiles of one head; two to eight heads in up to 8 MB (us, heads as for 4 MB / so: H=16
// T=16384 604 / 537; B=2 H=16 T=8192 305 / 272; B=8 H=16 T=4096 303 / 288; B=16 H=16 T=1024 56.0 / 53.5).
int heads_per_die_at_a_time(long long n_heads, int T, int d, bool four_per_simd = false) {
  if (n_heads % 8 != 0) return 0;
  const long long per_die = n_heads / 8;
  long long fit = (4ll << 20) / (4ll * T * d);
  if (four_per_simd) fit = std::min(8ll, std::max(2ll, 2 * fit));
  int hg = 1;
  while (hg * 2 <= fit && per_die % (hg * 2) == 0) hg *= 2;
  return hg;
}

// The forward kernel that a call takes.
struct FwdRoute {
  int heads_per_tile;
  bool few_tiles;       // moda_fwd_short.hip; else, bf16, moda_fwd_bf16.hip with
  int waves, per_simd;  // waves per workgroup, waves that share a SIMD
};
FwdRoute fwd_route(const moda_shape* s, const moda_fwd_tuning* tuning) {
  FwdRoute r;
  // grouped queries: as many heads of a group per tile (side by side in every wave) as divide the
  // group, up to 32
  const int G = s->Hq / s->Hk;
  r.heads_per_tile = 1;
  for (int gt = 32; gt > 1; gt /= 2)
    if (G % gt == 0) {
      r.heads_per_tile = gt;
      break;
    }
  // (without depth slots two heads per wave only halve the positions a tile covers: measured 10 %
  //  slower than one head per tile at G = 2, equal or faster from 4 heads on)
  if (s->depth_count == 0 && r.heads_per_tile < 4) r.heads_per_tile = 1;
  if (tuning && tuning->heads_per_tile > 0) r.heads_per_tile = tuning->heads_per_tile;
  r.waves = tuning && s->dtype == MODA_BF16 && tuning->waves != 0 ? tuning->waves : fwd_waves_per_workgroup(s, r.heads_per_tile);
  r.per_simd = fwd_waves_per_simd(s, r.heads_per_tile, r.waves);
  r.few_tiles = s->dtype == MODA_BF16 && !tuning && fwd_few_tiles(s, r.heads_per_tile);
  return r;
}

moda_status check_tuning(const moda_shape* s, const moda_fwd_tuning* tuning) {
  if (!tuning || s->dtype != MODA_BF16) return MODA_OK;
  if (tuning->waves != 0 && tuning->waves != 4 && tuning->waves != 8) return MODA_ERR_SHAPE;
  const int gt = tuning->heads_per_tile;
  if (gt < 0 || gt > 32 || (gt & (gt - 1)) != 0 || (gt > 0 && s->Hq / s->Hk % gt != 0)) return MODA_ERR_SHAPE;
  if (tuning->head_group < 0) return MODA_ERR_SHAPE;
  if (tuning->depth_path < 0 || tuning->depth_path > 2) return MODA_ERR_SHAPE;
  return MODA_OK;
}

float resolve_scale(const moda_shape* s) {
  return s->scale > 0.f ? s->scale : 1.0f / sqrtf((float)s->d);
}

moda::BwdParams bwd_dims(const moda_shape* s) {
  moda::BwdParams p{};
  p.B = s->B; p.Hq = s->Hq; p.Hk = s->Hk; p.T = s->T;
  p.depth_alloc = s->depth_alloc; p.depth_count = s->depth_count;
  p.causal = s->causal;
  return p;
}

}  // namespace

extern "C" {

const char* moda_status_string(moda_status st) {
  switch (st) {
    case MODA_OK: return "ok";
    case MODA_ERR_NULL: return "a required pointer is NULL";
    case MODA_ERR_SHAPE: return "invalid or inconsistent shape";
    case MODA_ERR_UNSUPPORTED: return "unsupported dtype, head dimension or size";
    case MODA_ERR_ALIGN: return "a base pointer is not 16-byte aligned";
    case MODA_ERR_LAUNCH: return "the HIP runtime refused a kernel launch";
    case MODA_ERR_WORKSPACE: return "workspace missing or too small";
  }
  return "unknown status";
}

int moda_version(void) { return 200; }

int moda_kernels_per_call(const moda_shape* s, int which) {
  if (check_shape(s) != MODA_OK || s->B == 0 || s->T == 0) return 0;
  if (which == 0) return 1;
  if (s->dtype != MODA_BF16 || s->Hq / s->Hk > moda::bwd_bf16_max_group()) return 0;
  return moda::bwd_bf16_kernels(bwd_dims(s), s->d);
}

int moda_fwd_kernel_name(const moda_shape* s, const moda_fwd_tuning* tuning, char* name, size_t size) {
  if (name && size > 0) name[0] = 0;
  if (check_shape(s) != MODA_OK || check_tuning(s, tuning) != MODA_OK || s->B == 0 || s->T == 0) return 0;
  const FwdRoute r = fwd_route(s, tuning);
  moda::FwdParams p;
  p.B = s->B; p.Hq = s->Hq; p.T = s->T; p.depth_count = s->depth_count;
  if (s->dtype == MODA_F32)
    return snprintf(name, size, "moda_fwd_f32_%skernel<%d>", moda::fwd_f32_by_rows(p) ? "rows_" : moda::fwd_f32_eight_waves(p, s->d) ? "" : "four_", s->d);
  if (r.few_tiles) return snprintf(name, size, "moda_fwd_short_kernel<%d, %s>", s->d, r.heads_per_tile == 1 && s->depth_count > 0 ? "true" : "false");
  return snprintf(name, size, "moda_fwd_bf16_kernel<%d, %d, %d>", s->d, r.waves, r.per_simd);
}

int moda_bwd_kernel_name(const moda_shape* s, int which, char* name, size_t size) {
  if (name && size > 0) name[0] = 0;
  if (check_shape(s) != MODA_OK || s->B == 0 || s->T == 0 || which < 0 || which > 1) return 0;
  if (s->dtype != MODA_BF16 || s->Hq / s->Hk > moda::bwd_bf16_max_group()) return 0;
  return moda::bwd_bf16_kernel_name(bwd_dims(s), s->d, which, name, size);
}

moda_status moda_attn_fwd_tuned(const void* Q, const void* Kseq, const void* Vseq, const void* Kdepth,
                                const void* Vdepth, void* O, float* LSE, const moda_shape* s,
                                const moda_fwd_tuning* tuning, void* hip_stream) {
  moda_status st = check_shape(s);
  if (st != MODA_OK) return st;
  const int G = s->Hq / s->Hk;
  st = check_tuning(s, tuning);
  if (st != MODA_OK) return st;
  if (s->B == 0 || s->T == 0) return MODA_OK;
  if (!Q || !Kseq || !Vseq || !O || !LSE) return MODA_ERR_NULL;
  if (s->depth_count > 0 && (!Kdepth || !Vdepth)) return MODA_ERR_NULL;
  if (!aligned16(Q) || !aligned16(Kseq) || !aligned16(Vseq) || !aligned16(O) || !aligned16(LSE) ||
      !aligned16(Kdepth) || !aligned16(Vdepth))
    return MODA_ERR_ALIGN;

  moda::FwdParams p;
  p.Q = Q; p.Kseq = Kseq; p.Vseq = Vseq; p.Kdepth = Kdepth; p.Vdepth = Vdepth;
  p.O = O; p.LSE = LSE;
  p.B = s->B; p.Hq = s->Hq; p.Hk = s->Hk; p.T = s->T;
  p.depth_alloc = s->depth_alloc; p.depth_count = s->depth_count;
  p.causal = s->causal;
  p.scale = resolve_scale(s);
  p.scale_log2 = p.scale * 1.4426950408889634f;
  const FwdRoute route = fwd_route(s, tuning);
  p.heads_per_tile = route.heads_per_tile;
  // depth slots: on the matrix pipe when several heads share a position's slots (the block
  // products are then dense enough to beat the vector ALUs), else on the vector ALUs, where the
  // phase already runs at the rate a compute unit can fetch
  p.depth_mfma = (p.heads_per_tile > 1 && s->depth_count > 0) ? 1 : 0;
  if (tuning && s->dtype == MODA_BF16 && tuning->depth_path != 0)
    p.depth_mfma = (tuning->depth_path == 2 && s->depth_count > 0) ? 1 : 0;
  p.depth_magic = s->depth_count > 1 ? (unsigned)((1ull << 32) / (unsigned)s->depth_count) + 1u : 0u;
  const int waves = route.waves, per_simd = route.per_simd;
  p.head_group = heads_per_die_at_a_time((long long)s->B * s->Hk * (G / p.heads_per_tile), s->T, s->d, per_simd == 4);
  if (tuning && tuning->head_group > 0) p.head_group = tuning->head_group;
  const int rows = moda::fwd_bf16_tile_rows(waves) / p.heads_per_tile;  // positions per tile
  p.n_qtiles = (s->T + rows - 1) / rows;

  if (s->dtype == MODA_F32) {  // one head per tile; a head streams twice the bytes of a bf16 one
    p.n_qtiles = (s->T + moda::fwd_f32_tile_rows() - 1) / moda::fwd_f32_tile_rows();
    p.head_group = heads_per_die_at_a_time((long long)s->B * s->Hq, s->T, 2 * s->d);
  }

  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  if (route.few_tiles) {
    const int pos = moda::fwd_short_tile_pairs() / p.heads_per_tile;
    p.n_qtiles = (s->T + pos - 1) / pos;
    return launch_status(moda::launch_fwd_short(p, s->d, stream));
  }
  return launch_status((s->dtype == MODA_BF16) ? moda::launch_fwd_bf16(p, s->d, waves, per_simd, stream)
                                               : moda::launch_fwd_f32(p, s->d, stream));
}

moda_status moda_attn_fwd(const void* Q, const void* Kseq, const void* Vseq, const void* Kdepth,
                          const void* Vdepth, void* O, float* LSE, const moda_shape* s,
                          void* hip_stream) {
  return moda_attn_fwd_tuned(Q, Kseq, Vseq, Kdepth, Vdepth, O, LSE, s, nullptr, hip_stream);
}

moda_status moda_depth_append(const void* K, const void* V, void* Kdepth, void* Vdepth, int32_t slot,
                              const moda_shape* s, void* hip_stream) {
  moda_status st = check_shape(s);
  if (st != MODA_OK) return st;
  if (slot < 0 || slot >= s->depth_alloc) return MODA_ERR_SHAPE;
  if (s->B == 0 || s->T == 0) return MODA_OK;
  if (!K || !V || !Kdepth || !Vdepth) return MODA_ERR_NULL;
  if (!aligned16(K) || !aligned16(V) || !aligned16(Kdepth) || !aligned16(Vdepth)) return MODA_ERR_ALIGN;
  const int esz = s->dtype == MODA_BF16 ? 2 : 4;
  return launch_status(moda::launch_depth_append(K, V, Kdepth, Vdepth, (long long)s->B * s->Hk * s->T, s->d * esz,
                                                 s->depth_alloc, slot, static_cast<hipStream_t>(hip_stream)));
}

// Shape checks of the decoding step: [B, H, d] queries, a sequence cache of kv_alloc rows per
// (batch, head), one position's depth slots.
static moda_status check_decode(const moda_shape* s, int32_t kv_alloc) {
  const moda_status st = check_dims(s);
  if (st != MODA_OK) return st;
  if (s->dtype != MODA_BF16) return MODA_ERR_UNSUPPORTED;
  if (s->T < 1 || kv_alloc < s->T) return MODA_ERR_SHAPE;  // the new token's own key is always attended
  return MODA_OK;  // (the decoding kernels address the caches with 64-bit pointers: no slab limit)
}

size_t moda_attn_decode_workspace_bytes(const moda_shape* s) {
  if (check_dims(s) != MODA_OK || s->dtype != MODA_BF16 || s->B == 0 || s->T < 1) return 0;
  return moda::decode_workspace_bytes(s->B, s->Hq, s->Hk, s->T, s->d);
}

// The least that the partial results of a (validated, not empty) decoding step take.
static size_t decode_least(const moda_shape* s) { return moda::decode_least_bytes(s->B, s->Hq, s->Hk, s->T, s->d); }

// The decoding step with the slices' partial results in `workspace` (already validated).
static moda_status decode_with(const void* Q, const void* Kseq, const void* Vseq, const void* Kdepth,
                               const void* Vdepth, void* O, float* LSE, int32_t kv_alloc, void* workspace,
                               size_t workspace_bytes, const moda_shape* s, void* hip_stream);

moda_status moda_attn_decode(const void* Q, const void* Kseq, const void* Vseq, const void* Kdepth,
                             const void* Vdepth, void* O, float* LSE, int32_t kv_alloc, void* workspace,
                             size_t workspace_bytes, const moda_shape* s, void* hip_stream) {
  moda_status st = check_decode(s, kv_alloc);
  if (st != MODA_OK) return st;
  if (s->B == 0) return MODA_OK;
  if (!Q || !Kseq || !Vseq || !O || !LSE) return MODA_ERR_NULL;
  if (s->depth_count > 0 && (!Kdepth || !Vdepth)) return MODA_ERR_NULL;
  const void* ptrs[] = {Q, Kseq, Vseq, Kdepth, Vdepth, O, LSE, workspace};
  for (const void* q : ptrs)
    if (!aligned16(q)) return MODA_ERR_ALIGN;
  if (!workspace || workspace_bytes < decode_least(s)) return MODA_ERR_WORKSPACE;
  return decode_with(Q, Kseq, Vseq, Kdepth, Vdepth, O, LSE, kv_alloc, workspace, workspace_bytes, s, hip_stream);
}

size_t moda_attn_decode_noalloc_max_bytes(void) { return moda::decode_static_scratch_bytes(); }

moda_status moda_attn_decode_noalloc(const void* Q, const void* Kseq, const void* Vseq, const void* Kdepth,
                                     const void* Vdepth, void* O, float* LSE, int32_t kv_alloc,
                                     const moda_shape* s, void* hip_stream) {
  moda_status st = check_decode(s, kv_alloc);
  if (st != MODA_OK) return st;
  if (s->B == 0) return MODA_OK;
  if (decode_least(s) > moda::decode_static_scratch_bytes()) return MODA_ERR_WORKSPACE;
  if (!Q || !Kseq || !Vseq || !O || !LSE) return MODA_ERR_NULL;
  if (s->depth_count > 0 && (!Kdepth || !Vdepth)) return MODA_ERR_NULL;
  const void* ptrs[] = {Q, Kseq, Vseq, Kdepth, Vdepth, O, LSE};
  for (const void* q : ptrs)
    if (!aligned16(q)) return MODA_ERR_ALIGN;
  void* ws = nullptr;  // this GPU's copy of the library's scratch array (device address)
  if (moda::decode_static_scratch(&ws) != hipSuccess) return MODA_ERR_LAUNCH;
  // Nothing in the scratch has to start at zero: the first kernel writes every partial result
  // that the second one reads.
  return decode_with(Q, Kseq, Vseq, Kdepth, Vdepth, O, LSE, kv_alloc, ws, moda::decode_static_scratch_bytes(), s,
                     hip_stream);
}

static moda_status decode_with(const void* Q, const void* Kseq, const void* Vseq, const void* Kdepth,
                               const void* Vdepth, void* O, float* LSE, int32_t kv_alloc, void* workspace,
                               size_t workspace_bytes, const moda_shape* s, void* hip_stream) {
  return launch_status(moda::launch_decode_bf16(Q, Kseq, Vseq, Kdepth, Vdepth, O, LSE, static_cast<float*>(workspace),
                                                workspace_bytes, s->B, s->Hq, s->Hk, s->T, kv_alloc, s->d, s->depth_alloc,
                                                s->depth_count, resolve_scale(s),
                                                static_cast<hipStream_t>(hip_stream)));
}

size_t moda_calibrate_mfma_operand_bytes(void) { return moda::calibrate_operand_bytes(); }
size_t moda_calibrate_mfma_sink_bytes(int32_t workgroups) {
  return workgroups > 0 ? moda::calibrate_sink_bytes(workgroups) : 0;
}
double moda_calibrate_mfma(const void* operands, float* sink, size_t sink_bytes, int32_t workgroups, int32_t iters,
                           void* hip_stream) {
  if (!operands || !sink || workgroups <= 0 || iters <= 0 || !aligned16(operands) || !aligned16(sink)) return 0.0;
  if (sink_bytes < moda::calibrate_sink_bytes(workgroups)) return 0.0;
  if (moda::launch_calibrate_mfma(operands, sink, workgroups, iters, static_cast<hipStream_t>(hip_stream)) != hipSuccess)
    return 0.0;
  return moda::calibrate_flops(workgroups, iters);
}

size_t moda_attn_bwd_workspace_bytes(const moda_shape* s) {
  if (check_shape(s) != MODA_OK) return 0;
  return moda::bwd_bf16_workspace_bytes(bwd_dims(s), s->d);
}

moda_status moda_attn_bwd(const void* Q, const void* Kseq, const void* Vseq, const void* Kdepth,
                          const void* Vdepth, const void* O, const float* LSE, const void* dO,
                          void* dQ, void* dKseq, void* dVseq, void* dKdepth, void* dVdepth,
                          void* workspace, size_t workspace_bytes, const moda_shape* s,
                          void* hip_stream) {
  moda_status st = check_shape(s);
  if (st != MODA_OK) return st;
  // this build's backward: bf16, at most bwd_bf16_max_group() query heads per key/value head
  if (s->dtype != MODA_BF16 || s->Hq / s->Hk > moda::bwd_bf16_max_group()) return MODA_ERR_UNSUPPORTED;
  if (s->B == 0 || s->T == 0) return MODA_OK;
  if (!Q || !Kseq || !Vseq || !O || !LSE || !dO || !dQ || !dKseq || !dVseq) return MODA_ERR_NULL;
  if (s->depth_count > 0 && (!Kdepth || !Vdepth)) return MODA_ERR_NULL;
  if (s->depth_alloc > 0 && (!dKdepth || !dVdepth)) return MODA_ERR_NULL;
  const void* ptrs[] = {Q, Kseq, Vseq, Kdepth, Vdepth, O, LSE, dO, dQ, dKseq, dVseq, dKdepth, dVdepth, workspace};
  for (const void* q : ptrs)
    if (!aligned16(q)) return MODA_ERR_ALIGN;
  if (!workspace || workspace_bytes < moda_attn_bwd_workspace_bytes(s)) return MODA_ERR_WORKSPACE;

  moda::BwdParams p = bwd_dims(s);
  p.Q = Q; p.Kseq = Kseq; p.Vseq = Vseq; p.Kdepth = Kdepth; p.Vdepth = Vdepth;
  p.O = O; p.LSE = LSE; p.dO = dO;
  p.dQ = dQ; p.dKseq = dKseq; p.dVseq = dVseq; p.dKdepth = dKdepth; p.dVdepth = dVdepth;
  p.lse2 = static_cast<float*>(workspace);
  p.causal = s->causal;
  p.scale = resolve_scale(s);
  p.scale_log2 = p.scale * 1.4426950408889634f;
  p.head_group = heads_per_die_at_a_time((long long)s->B * s->Hk, s->T, s->d);
  return launch_status(moda::launch_bwd_bf16(p, s->d, static_cast<hipStream_t>(hip_stream)));
}

}  // extern "C"
