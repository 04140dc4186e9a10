// MoDA attention for ONE new token per sequence (decoding; paper Table 1, "Decoding" rows).
// The new token's query attends the T positions of the sequence K/V cache (its own K/V
// included) and the depth slots of its own position, under one softmax (section 2.2); the
// depth cache of a decoding step is therefore only [B, Hk, depth_alloc, d].
//
// The call is bound by reading the sequence cache once (2 * B * Hk * T * d elements), so the
// keys are split over workgroups (one workgroup = one (batch, key/value head, slice of the
// sequence), all G query heads of the group together, so the slice is read once):
//   partial: per slice and head the running (max, normaliser, weighted value sum) in fp32,
//            written to the workspace; the depth slots of the new token's position are one
//            more slice (the last one), read from the depth cache instead of the sequence cache;
//   merge  : per (batch, query head): folds the slices into one softmax, normalises, stores
//            O and LSE.
// (A few hundred keys take one kernel: moda_decode_one_kernel.)
// Two forms of the partial kernel.  One query head per key/value head: vector ALUs only (one
// query row: no matrix shape to speak of); a lane owns 8 channels, d/8 lanes a key row,
// 64 / (d/8) key rows per wave instruction.  Grouped queries: the G heads of a group are the
// columns of small matrix products (keys x heads), see moda_decode_partial_mfma_kernel.
#include <algorithm>
#include <atomic>

#include "moda_launch.h"
#include "moda_tile.h"

namespace moda {

constexpr int kDecWaves = 4;

// Scratch of the entry point that allocates nothing (moda_attn_decode_noalloc): the partial
// results of the slices, which the caller's workspace holds otherwise.  One copy per GPU, held
// until the process ends.  In host code this name is only a handle for hipGetSymbolAddress:
// kernels get the device address that call returns, never the name.
constexpr size_t kDecodeScratchBytes = 8u << 20;
static __device__ __align__(256) unsigned char scratch[kDecodeScratchBytes];

constexpr int kMaxDevices = 64;
static std::atomic<void*> g_scratch_addr[kMaxDevices];  // device address of `scratch`, per device (0: not looked up yet)

size_t decode_static_scratch_bytes() { return kDecodeScratchBytes; }

// Device address of `scratch` on the CURRENT device: looked up once per device (on the first
// call made with that device current), then served from the table.
hipError_t decode_static_scratch(void** addr) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  void* p = g_scratch_addr[dev].load(std::memory_order_acquire);
  if (!p) {
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_addr[dev].store(p, std::memory_order_release);  // (two threads racing here store the same address)
  }
  *addr = p;
  return hipSuccess;
}

struct DecodeParams {
  const void* Q;       // [B, Hq, d]
  const void* Kseq;    // [B, Hk, T_alloc, d]
  const void* Vseq;
  const void* Kdepth;  // [B, Hk, depth_alloc, d]
  const void* Vdepth;
  void* O;             // [B, Hq, d]
  float* LSE;          // [B, Hq]
  float* ws;           // [B, Hq, n_slices, d + 2]
  int B, Hq, Hk, T, T_alloc;
  int depth_alloc, depth_count;
  int n_split, keys_per_split;  // slices of the sequence
  int n_slices;                 // n_split, plus one for the depth slots when there are any
  float scale, scale_log2;
};

// Two registers of which one's lanes 32.. and the other's lanes ..31 change places, added; the same with odd and even
// rows of 16 lanes.
__device__ __forceinline__ float swap_add32(float a, float b) {
  auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(int, a), __builtin_bit_cast(int, b), false, false);
  return __builtin_bit_cast(float, (int)r[0]) + __builtin_bit_cast(float, (int)r[1]);
}
__device__ __forceinline__ float swap_add16(float a, float b) {
  auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(int, a), __builtin_bit_cast(int, b), false, false);
  return __builtin_bit_cast(float, (int)r[0]) + __builtin_bit_cast(float, (int)r[1]);
}
// Sum and maximum over a wave's groups of LPR lanes: every lane gets that of the lanes at its place.
template <int LPR>
__device__ __forceinline__ float groups_sum(float x) {
  if (LPR == 8) x += dpp_mov<0x128>(x);  // row_ror:8
  return pair_sum(swap_add16(x, x));
}
template <int LPR>
__device__ __forceinline__ float groups_max(float x) {
  if (LPR == 8) x = fmaxf(x, dpp_mov<0x128>(x));
  const int i = __builtin_bit_cast(int, x);
  auto r = __builtin_amdgcn_permlane16_swap(i, i, false, false);
  return pair_max(fmaxf(__builtin_bit_cast(float, (int)r[0]), __builtin_bit_cast(float, (int)r[1])));
}

// A wave's state of one head, of its groups of LPR lanes (their references, normalisers, eight channels each), folded and
// written to red[0 .. D) (channels), red[D] (reference), red[D + 1] (normaliser).  Every exchange halves the channels that a
// lane holds.
template <int D>
__device__ __forceinline__ void fold_groups(float m, float l, const float (&o)[8], float c2, int lane, float* red) {
  constexpr int LPR = D / 8;
  const float mm = groups_max<LPR>(m);
  const float f = m == -INFINITY ? 0.f : fast_exp2((m - mm) * c2);
  const float ll = groups_sum<LPR>(l * f);
  float half[4], quarter[2];
#pragma unroll
  for (int k = 0; k < 4; ++k) half[k] = swap_add32(o[k] * f, o[k + 4] * f);  // lanes < 32: channel k, others k + 4
#pragma unroll
  for (int k = 0; k < 2; ++k) {  // even rows of 16 lanes: channel k, odd ones k + 2 of those
    quarter[k] = swap_add16(half[k], half[k + 2]);
    if (LPR == 8) quarter[k] += dpp_mov<0x128>(quarter[k]);
  }
  if ((lane & 15) < LPR)
    *(f32x2*)&red[lane % LPR * 8 + (lane >> 5) * 4 + ((lane >> 4) & 1) * 2] = (f32x2){quarter[0], quarter[1]};
  if (lane == 0) *(f32x2*)&red[D] = (f32x2){mm, ll};
}

template <int D, int GT>
__global__ __launch_bounds__(kDecWaves * 64) void moda_decode_partial_kernel(DecodeParams p) {
  constexpr int LPR = D / 8, RPS = 64 / LPR, RB = D * 2;
  __shared__ __attribute__((aligned(16))) float red[kDecWaves][GT][D + 2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int rg = lane / LPR, l16 = lane % LPR;
  const int G = p.Hq / p.Hk;
  const int n_gc = (G + GT - 1) / GT;  // head chunks per group
  int id = blockIdx.x;
  const int split = id % p.n_slices;
  id /= p.n_slices;
  const int gc = id % n_gc;
  const int bg = id / n_gc;  // (batch, key/value head)
  const int b = bg / p.Hk, g = bg - b * p.Hk;
  const int h0 = g * G + gc * GT;  // first query head of this chunk
  const float c2 = p.scale_log2;

  u32x4 q[GT];
  float m[GT], l[GT], o[GT][8];
#pragma unroll
  for (int j = 0; j < GT; ++j) {
    const int h = min(h0 + j, g * G + G - 1);  // heads past the group repeat the last one; never stored
    q[j] = *(const u32x4*)((const char*)p.Q + ((size_t)b * p.Hq + h) * RB + l16 * 16);
    m[j] = -INFINITY;
    l[j] = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) o[j][k] = 0.f;
  }
  // rows [k_begin, k_end) of the sequence cache, or (last slice) the depth slots of the position
  const bool is_depth = split == p.n_split;
  const int k_begin = is_depth ? 0 : split * p.keys_per_split;
  const int k_end = is_depth ? p.depth_count : min(p.T, k_begin + p.keys_per_split);
  const int k_last = k_end - 1;
  const size_t slab = is_depth ? (size_t)bg * p.depth_alloc * RB : (size_t)bg * p.T_alloc * RB;
  const char* Kb = (const char*)(is_depth ? p.Kdepth : p.Kseq) + slab + l16 * 16;
  const char* Vb = (const char*)(is_depth ? p.Vdepth : p.Vseq) + slab + l16 * 16;

  // this lane's keys: k_begin + (wave * RPS + rg) + i * (kDecWaves * RPS), kU at a time with the
  // next kU in flight; the running max is raised (and the state rescaled) once per kU keys
  constexpr int STEP = kDecWaves * RPS;
  constexpr int kU = 4;
  const int key0 = k_begin + wave * RPS + rg;
  auto load = [&](const char* base, int kk) {
    return __builtin_nontemporal_load((const u32x4*)(base + (size_t)min(kk, k_last) * RB));
  };
  u32x4 kn[kU], vn[kU];
#pragma unroll
  for (int u = 0; u < kU; ++u) {
    kn[u] = load(Kb, key0 + u * STEP);
    vn[u] = load(Vb, key0 + u * STEP);
  }
  for (int base = k_begin; base < k_end; base += kU * STEP) {  // uniform trip count over the workgroup
    const int key = key0 + (base - k_begin);
    u32x4 kv[kU], vv[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      kv[u] = kn[u];
      vv[u] = vn[u];
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      kn[u] = load(Kb, key + (kU + u) * STEP);
      vn[u] = load(Vb, key + (kU + u) * STEP);
    }
#pragma unroll
    for (int j = 0; j < GT; ++j) {
      float sc[kU];
      float mn = m[j];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        float a = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) a = dot2_bf16(q[j][k], kv[u][k], a);
        a = group_sum<LPR>(a);
        sc[u] = key + u * STEP < k_end ? a : -INFINITY;
        mn = fmaxf(mn, sc[u]);
      }
      // (mn is -inf only while every score so far was, or was NaN, which stays NaN; with reference 0 the others weigh nothing)
      const float ref = mn == -INFINITY ? 0.f : mn;
      const float al = fast_exp2((m[j] - ref) * c2);
      m[j] = mn;
      l[j] *= al;
#pragma unroll
      for (int k = 0; k < 8; ++k) o[j][k] *= al;
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const float pw = fast_exp2((sc[u] - ref) * c2);
        l[j] += pw;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          o[j][2 * k] += pw * bf16_lo(vv[u][k]);
          o[j][2 * k + 1] += pw * bf16_hi(vv[u][k]);
        }
      }
    }
  }

  // ---- the row groups of a wave, then the waves
#pragma unroll
  for (int j = 0; j < GT; ++j) fold_groups<D>(m[j], l[j], o[j], c2, lane, red[wave][j]);
  __syncthreads();
  // thread t < GT * D: head j = t / D, channel t % D
  for (int t = tid; t < GT * D; t += kDecWaves * 64) {
    const int j = t / D, ch = t % D;
    if (h0 + j >= g * G + G) continue;
    float mm = -INFINITY, ll = 0.f, oo = 0.f;
#pragma unroll
    for (int w = 0; w < kDecWaves; ++w) mm = fmaxf(mm, red[w][j][D]);
#pragma unroll
    for (int w = 0; w < kDecWaves; ++w) {
      const float mi = red[w][j][D];
      const float f = mi == -INFINITY ? 0.f : fast_exp2((mi - mm) * c2);
      ll += f * red[w][j][D + 1];
      oo += f * red[w][j][ch];
    }
    float* dst = p.ws + (((size_t)b * p.Hq + h0 + j) * p.n_slices + split) * (D + 2);
    dst[ch] = oo;
    if (ch == 0) {
      dst[D] = mm;
      dst[D + 1] = ll;
    }
  }
}

// ---------------------------------------------------------------- short contexts: one kernel
// With a few hundred rows (keys, then slots) per key/value head the second kernel takes as long as the first.  Here a
// workgroup of eight waves walks all rows of its (batch, key/value head, chunk of heads) as above and normalises.
constexpr int kDecOneWaves = 8;

template <int D, int GT>
__global__ __launch_bounds__(kDecOneWaves * 64, 2) void moda_decode_one_kernel(DecodeParams p) {
  constexpr int LPR = D / 8, RPS = 64 / LPR, RB = D * 2;
  __shared__ __attribute__((aligned(16))) float red[kDecOneWaves][GT][D + 2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int rg = lane / LPR, l16 = lane % LPR;
  const int G = p.Hq / p.Hk;
  const int n_gc = (G + GT - 1) / GT;
  const int gc = blockIdx.x % n_gc, bg = blockIdx.x / n_gc;
  const int b = bg / p.Hk, g = bg - b * p.Hk;
  const int h0 = g * G + gc * GT;
  const float c2 = p.scale_log2;
  const int T = p.T, n = T + p.depth_count;

  // row r: key r of the sequence cache, or slot r - T
  const size_t seq = (size_t)bg * p.T_alloc * RB + l16 * 16, dep = (size_t)bg * p.depth_alloc * RB + l16 * 16;
  auto load = [&](const void* cache, const void* slots, int r) {
    r = min(r, n - 1);
    const char* at = r < T ? (const char*)cache + seq + (size_t)r * RB : (const char*)slots + dep + (size_t)(r - T) * RB;
    return __builtin_nontemporal_load((const u32x4*)at);
  };
  constexpr int STEP = kDecOneWaves * RPS, kU = 4;
  const int row0 = wave * RPS + rg;
  u32x4 kn[kU], vn[kU];
#pragma unroll
  for (int u = 0; u < kU; ++u) {
    kn[u] = load(p.Kseq, p.Kdepth, row0 + u * STEP);
    vn[u] = load(p.Vseq, p.Vdepth, row0 + u * STEP);
  }
  u32x4 q[GT];
  float m[GT], l[GT], o[GT][8];
#pragma unroll
  for (int j = 0; j < GT; ++j) {
    const int h = min(h0 + j, g * G + G - 1);  // heads past the group repeat the last one; never stored
    q[j] = *(const u32x4*)((const char*)p.Q + ((size_t)b * p.Hq + h) * RB + l16 * 16);
    m[j] = -INFINITY;
    l[j] = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) o[j][k] = 0.f;
  }
  auto factor = [&](float x, float ref) { return x == -INFINITY ? 0.f : fast_exp2((x - ref) * c2); };
  for (int base = 0; base < n; base += kU * STEP) {  // (uniform)
    u32x4 kv[kU], vv[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      kv[u] = kn[u];
      vv[u] = vn[u];
    }
    if (base + kU * STEP < n) {  // (uniform)
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        kn[u] = load(p.Kseq, p.Kdepth, row0 + base + (kU + u) * STEP);
        vn[u] = load(p.Vseq, p.Vdepth, row0 + base + (kU + u) * STEP);
      }
    } else {  // rows past the end repeat the last one with weight zero, which an infinite value would turn into NaN
#pragma unroll
      for (int u = 0; u < kU; ++u)
        if (row0 + base + u * STEP >= n) vv[u] = (u32x4){0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int j = 0; j < GT; ++j) {
      float sc[kU], mn = m[j];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        float a = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) a = dot2_bf16(q[j][k], kv[u][k], a);
        a = group_sum<LPR>(a);
        sc[u] = row0 + base + u * STEP < n ? a : -INFINITY;
        mn = fmaxf(mn, sc[u]);
      }
      const float al = factor(m[j], mn);
      m[j] = mn;
      l[j] *= al;
#pragma unroll
      for (int k = 0; k < 8; ++k) o[j][k] *= al;
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const float pw = factor(sc[u], mn);
        l[j] += pw;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          o[j][2 * k] += pw * bf16_lo(vv[u][k]);
          o[j][2 * k + 1] += pw * bf16_hi(vv[u][k]);
        }
      }
    }
  }
  // ---- the row groups of a wave, then the waves
#pragma unroll
  for (int j = 0; j < GT; ++j) fold_groups<D>(m[j], l[j], o[j], c2, lane, red[wave][j]);
  __syncthreads();
  for (int t = tid; t < GT * D; t += kDecOneWaves * 64) {
    const int j = t / D, ch = t % D;
    if (h0 + j >= g * G + G) continue;
    float mm = -INFINITY, ll = 0.f, oo = 0.f;
#pragma unroll
    for (int w = 0; w < kDecOneWaves; ++w) mm = fmaxf(mm, red[w][j][D]);
#pragma unroll
    for (int w = 0; w < kDecOneWaves; ++w) {
      const float f = factor(red[w][j][D], mm);
      ll += f * red[w][j][D + 1];
      oo += f * red[w][j][ch];
    }
    const size_t row = (size_t)b * p.Hq + h0 + j;
    ((__bf16*)p.O)[row * D + ch] = (__bf16)(oo / ll);
    if (ch == 0) p.LSE[row] = mm * p.scale + __logf(ll);
  }
}

// ---------------------------------------------------------------- grouped queries: slices on the matrix pipe
// With G query heads per key/value head the arithmetic per key row grows G-fold on the vector
// ALUs and bounds the kernel well below the memory rate.  Here the (up to 32) heads of a group
// are the columns of matrix products: per block of 32 keys
//     S^T = K Q^T  (keys x heads),   O^T += V^T P^T  (channels x heads),
// so a lane owns ONE head (column) with 16 of the block's scores in registers: the running
// max / normaliser are per-lane scalars (two lanes per head, combined once at the end) and
// P^T is the second product's B operand straight from the accumulators.  Columns past the
// group hold zero queries and are never stored.
// A workgroup of 4 waves = (batch, key/value head, chunk of 32 heads, 4 consecutive slices):
// every WAVE takes a slice of its own and writes its own partial result; the workgroup only
// shares the Q tile.  A wave walks its slice 32 keys at a time with the K and V rows of the
// next block(s) in flight in registers (fully coalesced, bounds-checked raw-buffer loads:
// rows past the slice read as zeros and fetch nothing).  A block's K and V rows are
// written to the wave's two LDS tiles (the layout the backward kernels use) and read back as
// row fragments (K) and transposed fragments (V).
// Output: the same per-slice partial results as the kernel above.
constexpr int kDecMWaves = 4;   // waves (= slices) per workgroup
constexpr int kDecBlock = 32;   // keys per block
// Measured choices: d = 64: two blocks (8 KB each) in flight per wave and three waves per SIMD
// (146 registers); d = 128: one block (16 KB) and two waves per SIMD.  More waves beat deeper
// prefetch: a block's chain LDS write -> fragment reads -> matrix products -> exponentials ->
// matrix products has little to overlap within one wave.
constexpr int dec_blocks_in_flight(int d) { return d == 64 ? 2 : 1; }
constexpr int dec_waves_per_simd(int d) { return d == 64 ? 3 : 2; }

template <int D>
__global__ __launch_bounds__(kDecMWaves * 64) __attribute__((amdgpu_waves_per_eu(dec_waves_per_simd(D), dec_waves_per_simd(D))))
void moda_decode_partial_mfma_kernel(DecodeParams p) {
  using Tl = Tile<D>;
  constexpr int RB = D * 2;
  constexpr int kSteps = Tl::kDSteps;               // matrix instructions per score block
  constexpr int NB = kDecBlock / 32;                // sub-blocks of 32 keys
  constexpr int kRowsPerInst = 1024 / RB;           // rows one load instruction covers
  constexpr int kInst = kDecBlock / kRowsPerInst;   // load instructions per block of K or V
  constexpr int kHalf = kDecBlock * RB;             // bytes of a block of K or V
  constexpr int kQBytes = 32 * RB;
  constexpr int kPF = dec_blocks_in_flight(D);                            // blocks in flight
  // [Q tile: 32 heads][per wave: K tile, V tile of kDecBlock rows]
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kQBytes + 2 * kDecMWaves * kHalf];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, hi = lane >> 5;
  const int G = p.Hq / p.Hk;
  const int n_gc = (G + 31) / 32;
  const int n_sg = (p.n_slices + kDecMWaves - 1) / kDecMWaves;  // slice groups
  int id = blockIdx.x;
  const int sg = id % n_sg;
  id /= n_sg;
  const int gc = id % n_gc;
  const int bg = id / n_gc;
  const int b = bg / p.Hk, g = bg - b * p.Hk;
  const int h0 = g * G + gc * 32;            // first query head of this chunk
  const int nh = min(32, G - gc * 32);       // heads in this chunk
  const float c2 = p.scale_log2;
  const unsigned smem_addr = (unsigned)(size_t)(lds_ptr)smem;
  const unsigned q_tile = smem_addr, kt = smem_addr + kQBytes + 2 * wave * kHalf, vt = kt + kHalf;
  FragAddr<D> fa;
  fa.init(lane);

  // ---- Q tile: row n = head n of the chunk (zeros past the group)
  {
    const char* qb = (const char*)p.Q + ((size_t)b * p.Hq + h0) * RB;
#pragma unroll
    for (int i = tid; i < 32 * Tl::kChunks; i += kDecMWaves * 64) {
      const int n = i / Tl::kChunks, c = i % Tl::kChunks;
      u32x4 v = *(const u32x4*)(qb + (size_t)min(n, nh - 1) * RB + c * 16);
      if (n >= nh) v = (u32x4){0u, 0u, 0u, 0u};
      *(u32x4*)(smem + Tl::off(n, c)) = v;
    }
  }
  __syncthreads();
  const int split = sg * kDecMWaves + wave;  // this wave's slice
  if (split >= p.n_slices) return;

  f32x16 oa[Tl::kDBlocks];  // O^T: [channel block], lane = head, registers = channels 8 i + 4 hi + j
#pragma unroll
  for (int cb = 0; cb < Tl::kDBlocks; ++cb)
#pragma unroll
    for (int i = 0; i < 16; ++i) oa[cb][i] = 0.f;
  float m = -INFINITY, l = 0.f;
  const float lazy = 8.0f / c2;  // 8 powers of two, in units of the raw scores

  // rows [k_begin, k_end) of the sequence cache, or (last slice) the depth slots of the position
  const bool is_depth = split == p.n_split;
  const int k_begin = is_depth ? 0 : split * p.keys_per_split;
  const int k_end = is_depth ? p.depth_count : min(p.T, k_begin + p.keys_per_split);
  const int n_blocks = (k_end - k_begin + kDecBlock - 1) / kDecBlock;  // (>= 1: no slice is empty)
  const size_t slab = is_depth ? (size_t)bg * p.depth_alloc * RB : ((size_t)bg * p.T_alloc + k_begin) * RB;
  const unsigned bytes = (unsigned)(k_end - k_begin) * (unsigned)RB;
  const __amdgpu_buffer_rsrc_t k_buf = __builtin_amdgcn_make_buffer_rsrc(
      (void*)((const char*)(is_depth ? p.Kdepth : p.Kseq) + slab), 0, (int)bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t v_buf = __builtin_amdgcn_make_buffer_rsrc(
      (void*)((const char*)(is_depth ? p.Vdepth : p.Vseq) + slab), 0, (int)bytes, 0x00020000);
  // The tile-copy mapping: 1 KB per instruction; a lane fetches the chunk that belongs at its
  // place (16 * lane) of the piece of the permuted tile.  The permutation of piece q differs
  // from piece 0's by the swz of the piece's first row.
  const int jr = lane / Tl::kChunks, pc = lane % Tl::kChunks;
  const int g_off = jr * RB + ((pc ^ Tl::swz(jr)) << 4);
  auto piece_xor = [](int q) { return (D == 128 ? (q & 3) : ((q & 1) << 1)) << 4; };
  struct Block {
    u32x4 k[kInst];
    u32x4 v[kInst];
  };
  auto issue = [&](int blk, Block& r) {
    const int soff = blk * kHalf;  // (blocks past the slice: every lane out of range, zeros)
#pragma unroll
    for (int q = 0; q < kInst; ++q)
      r.k[q] = __builtin_amdgcn_raw_buffer_load_b128(k_buf, xor_here(g_off, piece_xor(q)), soff + q * 1024, 2);
#pragma unroll
    for (int q = 0; q < kInst; ++q)
      r.v[q] = __builtin_amdgcn_raw_buffer_load_b128(v_buf, xor_here(g_off, piece_xor(q)), soff + q * 1024, 2);
  };
  const unsigned bq_row = fa.row + q_tile, bk_row = fa.row + kt;
  const unsigned bv_tr = fa.tr + vt, bv_tr8 = fa.tr8 + vt;
  auto fold = [&](int blk, const Block& r) {
    // block -> the wave's LDS tiles (a wave's LDS operations execute in order: these writes
    // follow the fragment reads of the block before)
#pragma unroll
    for (int q = 0; q < kInst; ++q)
      *(u32x4 __attribute__((address_space(3)))*)(size_t)(kt + q * 1024 + lane * 16) = r.k[q];
#pragma unroll
    for (int q = 0; q < kInst; ++q)
      *(u32x4 __attribute__((address_space(3)))*)(size_t)(vt + q * 1024 + lane * 16) = r.v[q];
    f32x16 s[NB];
#pragma unroll
    for (int sb = 0; sb < NB; ++sb)
#pragma unroll
      for (int i = 0; i < 16; ++i) s[sb][i] = 0.f;
#pragma unroll
    for (int st = 0; st < kSteps; ++st) {
      const bf16x8 qf = FragAddr<D>::row_frag((unsigned)xor_here((int)bq_row, st << 5), 0, 0);
      const unsigned xk = (unsigned)xor_here((int)bk_row, st << 5);
#pragma unroll
      for (int sb = 0; sb < NB; ++sb) s[sb] = mfma_bf16(FragAddr<D>::row_frag(xk, sb, 0), qf, s[sb]);
    }
    const int key0 = k_begin + blk * kDecBlock;
    if (key0 + kDecBlock > k_end) {  // (uniform) the slice's last, partial block
#pragma unroll
      for (int sb = 0; sb < NB; ++sb)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (key0 + sb * 32 + (i >> 2) * 8 + hi * 4 + (i & 3) >= k_end) s[sb][i] = -INFINITY;
    }
    float bm = s[0][0];
#pragma unroll
    for (int sb = 0; sb < NB; ++sb)
#pragma unroll
      for (int i = 0; i < 16; ++i) bm = fmaxf(bm, s[sb][i]);
    bm = pair_max(bm);
    // The reference m of the exponentials is raised lazily: only when a block's maximum exceeds
    // it by more than 8 powers of two (weights then stay below 2^8, which fp32 sums and bf16
    // weights hold; any reference gives the same quotient).  The first block always raises it
    // (m = -inf, and the factor exp2(-inf) = 0 scales the empty state), unless all its scores are -inf: the
    // state then stays empty and the weights are zero.
    const bool raise = bm > m + lazy || m == -INFINITY;
    if (__builtin_amdgcn_ballot_w64(raise) != 0) {  // (uniform)
      const float mn = raise ? bm : m;
      const float al = mn == m ? 1.f : fast_exp2((m - mn) * c2);
      m = mn;
      l *= al;
#pragma unroll
      for (int cb = 0; cb < Tl::kDBlocks; ++cb)
#pragma unroll
        for (int i = 0; i < 16; ++i) oa[cb][i] *= al;
    }
    const float mc = m == -INFINITY ? 0.f : m * c2;
#pragma unroll
    for (int sb = 0; sb < NB; ++sb)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        float pv[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          pv[k] = fast_exp2(s[sb][hf * 8 + k] * c2 - mc);
          l += pv[k];
        }
        const bf16x8 pb = pack8(pv);
#pragma unroll
        for (int cb = 0; cb < Tl::kDBlocks; ++cb)
          oa[cb] = mfma_bf16(FragAddr<D>::tr_frag((unsigned)xor_here((int)bv_tr, cb << 6),
                                                  (unsigned)xor_here((int)bv_tr8, cb << 6), sb * 2 + hf, 0),
                             pb, oa[cb]);
      }
  };

  // Blocks are walked with the loads of the next kPF - 1 in flight; past the end the loads
  // are still issued (out of range: they fetch nothing), so that the wait for an older
  // block's registers never depends on a branch.
  Block buf[kPF];
#pragma unroll
  for (int i = 0; i < kPF - 1; ++i) issue(i, buf[i]);
  for (int blk0 = 0; blk0 < n_blocks; blk0 += kPF) {
#pragma unroll
    for (int i = 0; i < kPF; ++i) {
      const int blk = blk0 + i;
      issue(blk + kPF - 1, buf[(i + kPF - 1) % kPF]);
      if (blk < n_blocks) fold(blk, buf[i]);
    }
  }

  // ---- this slice's partial result of the lane's head: 4 consecutive channels at a time
  const float l_tot = pair_sum(l);
  if (l32 < nh) {
    float* dst = p.ws + (((size_t)b * p.Hq + h0 + l32) * p.n_slices + split) * (D + 2);
#pragma unroll
    for (int cb = 0; cb < Tl::kDBlocks; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float* d4 = dst + cb * 32 + i * 8 + hi * 4;
        d4[0] = oa[cb][4 * i];
        d4[1] = oa[cb][4 * i + 1];
        d4[2] = oa[cb][4 * i + 2];
        d4[3] = oa[cb][4 * i + 3];
      }
    if (hi == 0) {
      dst[D] = m;
      dst[D + 1] = l_tot;
    }
  }
}

// One workgroup of NG x D threads per (batch, query head): thread = channel, group g of D threads folds
// the slices g, g + NG, ... eight at a time (their loads issued together), with a running reference
// like any other online softmax; the groups' states are folded through LDS.  The fold of a head is
// a chain of memory latencies, one per eight slices, hence NG = 4 where there are more than 8 (B=8
// Hq=64, 49 slices of d=64: 7.6 -> 4.8 us; whole call, 9 slices, T=1003 H=16 d=128 6.8 -> 6.5; 16 slices, Hq=8 Hk=2 B=6 T=1000
// d=64 6.9 -> 6.6; with 8 slices or fewer 0 to 5 % longer).  From 2^17 outputs on the workgroups are several to a unit and
// hide each other's latency: up to 16 slices one group then (four / one, whole call, 9 to 12 slices: 2048 to 10496 heads
// of d=128 1.02 to 1.05, B=41 Hq=256 Hk=8 T=2419 115 / 106 us; 17 to 24: 0.99 to 1.01).
static int merge_groups(int n_slices, long long heads, int d) {
  return n_slices <= (heads * d > 1 << 17 ? 16 : 8) ? 1 : 4;
}

template <int D, int NG>
__global__ __launch_bounds__(NG * D) void moda_decode_merge_kernel(DecodeParams p) {
  constexpr int kU = 8;
  __shared__ float red[NG > 1 ? NG : 1][D], stat[NG > 1 ? NG : 1][2];
  // (the group is the same for a wave: what it reads of a slice besides its channel comes by scalar loads)
  const int ch = threadIdx.x % D, g = NG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / D);
  const int bh = blockIdx.x;
  const float c2 = p.scale_log2;
  const float* ws = p.ws + (size_t)bh * p.n_slices * (D + 2);
  float mm = -INFINITY, ll = 0.f, oo = 0.f;
  // (a slice or a group of them whose scores are all -inf is an empty state: reference -inf, weight zero)
  auto factor = [&](float m, float ref) { return m == -INFINITY ? 0.f : fast_exp2((m - ref) * c2); };
  for (int s0 = g; s0 < p.n_slices; s0 += kU * NG) {
    float mi[kU], li[kU], oi[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const float* w = ws + (size_t)min(s0 + u * NG, p.n_slices - 1) * (D + 2);
      mi[u] = w[D];
      li[u] = w[D + 1];
      oi[u] = w[ch];
    }
    float mn = mm;
#pragma unroll
    for (int u = 0; u < kU; ++u)
      if (s0 + u * NG < p.n_slices) mn = fmaxf(mn, mi[u]);
    const float al = factor(mm, mn);
    mm = mn;
    ll *= al;
    oo *= al;
#pragma unroll
    for (int u = 0; u < kU; ++u)
      if (s0 + u * NG < p.n_slices) {
        const float f = factor(mi[u], mm);
        ll += f * li[u];
        oo += f * oi[u];
      }
  }
  if constexpr (NG > 1) {
    red[g][ch] = oo;
    if (ch == 0) {
      stat[g][0] = mm;
      stat[g][1] = ll;
    }
    __syncthreads();
    if (g > 0) return;
    const float m0 = mm;
#pragma unroll
    for (int w = 1; w < NG; ++w) mm = fmaxf(mm, stat[w][0]);
    const float f0 = factor(m0, mm);
    ll *= f0;
    oo *= f0;
#pragma unroll
    for (int w = 1; w < NG; ++w) {
      const float f = factor(stat[w][0], mm);
      ll += f * stat[w][1];
      oo += f * red[w][ch];
    }
  }
  ((__bf16*)p.O)[(size_t)bh * D + ch] = (__bf16)(oo / ll);
  if (ch == 0) p.LSE[bh] = mm * p.scale + __logf(ll);
}

// How a call is cut into slices.  One query head per key/value head: workgroups of 4 waves,
// enough of them to fill 256 compute units a few times over, slices of at least 256 keys (128 while
// that makes no more than 8 slices: T=1003, 16 heads 7.4 -> 6.9 us; but 16 slices of 128 keys at T=2000,
// 4 heads 6.8 -> 7.5 us; 8 slices instead of 5 to 7 of 256 keys 0 to 4 % longer at d = 64, at d = 128 5 % shorter
// instead of 5 or 6, 3 % longer instead of 7).
// More than 4 query heads per key/value head (matrix-pipe kernel): one slice per wave, of at least 128
// keys (256 / 128: B=1 Hq=64 Hk=8 d=64 T=1003 13.2 / 10.1 us, T=4096 14.6 / 12.7; B=4 T=2000 d=128 22 / 16).
// The finer slices of either only where they make no more rounds of workgroups than slices of 256 keys, i.e. where
// compute units would be left over: 288 workgroups instead of 256 (B=4 Hq=16 Hk=8 T=1662 d=128) took 12.0 us
// instead of 9.3, 512 instead of 384 (B=64 Hk=2 T=281) 0.88 of the time.  Over 900 random calls, caches just read
// and from memory, this is 0.3 % behind the better cut on average; always the finer one 1.6 %.
// Calls that leave units without work take finer slices still (finest_slices): a slice of 128 keys is a chain of four blocks
// (d = 128: one in flight) or of two batches of rows that such a call only waits for.  Slices of 128 (vector ALUs, above 1792
// keys 256) / 64 / 32 keys, us, whole call, (batch, key/value head)s on the left:
//   G=8 d=128   2 T=122 10.6 / 7.9 / 7.1;   4 T=549 12.2 / 9.8 / 7.8;   32 T=371 12.2 / 9.3 / 8.6;   36 T=1604 15.9 / 12.8 / 14.9;   104 T=125 11.7 / 9.2 / 8.5;
//               2 T=4909 13.6 / 11.4 / 12.3;   20 T=5693 18.7 / 19.9 / 20;   48 T=3421 23 / 28
//   G=8 d=64    12 T=343 8.7 / 7.3 / 7.2;   48 T=1271 10.6 / 9.7 / 11.6;   2 T=9867 11.4 / 11.6;   104 T=2618 19 / 22
// Large groups write, and the merge reads, more per slice: fewer workgroups per slice then (32 heads a group, slices of 128 /
// these, us: d=64 64 T=378 12.5 / 14.8, 36 T=35 9.7 / 10.8, 104 T=482 11.2 / 13.6;  d=128 135 T=46 1.06).  And not two slices of 32 keys
// beside more than 32 slots, which last as long as both (d=128 G=8 192 T=39, 64 slots 1.07).
//   vector ALUs, d=128   G=1 8 T=1977 7.7 / 6.2, with 128 keys 6.6;   16 T=189 6.1 / 5.5;   30 T=1080 8.6 / 8.2;   G=4 32 T=233 8.1 / 7.2;   G=2 120 T=197 8.5 / 8.4
//   slices of 256 / 128 keys: d=128 8 T=3880 8.5 / 7.3;   8 T=7343 9.4 / 10.5;   d=64 8 T=2094 7.1 / 6.3;   4 T=3706 7.4 / 6.4;   32 T=1717 7.2 / 8.4;   2 T=4786 6.6 / 7.0
struct DecodePlan {
  bool mfma;
  int n_split;
  int keys_per_split;
};
struct DecodeRule {
  bool mfma;
  int d;
  int heads;     // query heads of a workgroup (matrix pipe)
  int want;      // slices that fill the chip, whatever the length
  int step;      // keys_per_split is a multiple of this
  int most_fine;    // most slices of the finer cut
  size_t slice_bytes;  // partial results of one slice of every (batch, head)
  long long groups;    // workgroups per slice (matrix pipe: per kDecMWaves slices)
  int round;           // workgroups that make one round
  int most_for_8;      // (vector ALUs) 8 slices in place of up to so many of 256 keys, where finer ones make more than 8
  long long rounds(int slices) const {
    return (groups * (mfma ? (slices + kDecMWaves - 1) / kDecMWaves : slices) + round - 1) / round;
  }
};
static int decode_heads_per_chunk(int G) {  // of the vector-ALU kernel (3 heads: one chunk of 4 with a padded head, not two)
  return G >= 3 ? 4 : G >= 2 ? 2 : 1;
}
static DecodeRule decode_rule(int B, int Hq, int Hk, int d) {
  DecodeRule r;
  const int G = Hq / Hk;
  // up to 4 heads per group the vector-ALU kernel is at the memory rate and ahead (measured)
  r.mfma = G > 4;
  r.d = d;
  r.heads = std::min(G, 32);
  if (r.mfma) {
    const int n_gc = (G + 31) / 32;
    // 12 wave-slices per compute unit: all resident at once at d = 64, one and a half rounds
    // at d = 128 (measured better than exactly one round: the second half-round evens out the tail)
    const long long slots = 256ll * 12;
    const long long per = slots / ((long long)B * Hk * n_gc);
    r.want = per < 1 ? 1 : (int)per;
    r.step = kDecBlock;
    r.groups = (long long)B * Hk * n_gc;
    r.round = d == 128 ? 512 : 256;  // (d = 128: two workgroups per compute unit run side by side at no loss)
  } else {
    r.want = (2048 + B * Hk - 1) / (B * Hk);
    r.step = kDecWaves * (64 / (d / 8));  // key rows a workgroup takes per step (16 or 32)
    const int gt = decode_heads_per_chunk(G);
    r.groups = (long long)B * Hk * ((G + gt - 1) / gt);
    r.round = 256;
  }
  r.most_for_8 = d == 128 ? 6 : 0;
  r.slice_bytes = (size_t)B * Hq * (d + 2) * sizeof(float);
  // (never so many that the partial results, with the depth slots' slice, outgrow the library's own scratch
  // array where those of the coarser slices fit it)
  r.most_fine = (int)(kDecodeScratchBytes / r.slice_bytes) - 1;
  return r;
}
static int coarse_slices(int T) { return (T + 255) / 256; }
static int fine_slices(bool mfma, int T) {
  const int fine = (T + 127) / 128, coarse = coarse_slices(T);
  return mfma || fine <= 8 ? fine : coarse > 8 ? coarse : 8;
}
// Most workgroups of the matrix-pipe kernel (one per slice) with slices of 32 and of 64 keys.
static int most_of_32(const DecodeRule& r) { return std::min(768, (r.d == 64 ? 3072 : 8192) / r.heads); }
static int most_of_64(const DecodeRule& r) { return std::min(1024, 16384 / r.heads); }
// Slices of the finest cut of a call with few workgroups, 0: it has none.  `depth`: its slots.
// (Vector ALUs, d = 128: 513 to 1792 keys keep slices of 128 and 256 keys, whose number tests fix at 1003, 1500, 1536 and 1537 keys.
// Slices of 64 are ahead there as well: 90 calls up to 1024 keys 0.95, 53 calls above 0.83 of the time.)
static int finest_slices(const DecodeRule& r, int T, int depth) {
  const int n32 = (T + 31) / 32, n64 = (T + 63) / 64, n128 = (T + 127) / 128;
  if (r.mfma) {
    if (n32 <= 16 && r.groups * n32 <= most_of_32(r) && !(n32 == 2 && depth > 32)) return n32;
    return n64 <= 96 && r.groups * n64 <= most_of_64(r) ? n64 : 0;
  }
  depth = depth > 0;
  if (r.d == 128 && (n64 <= 8 || (coarse_slices(T) >= 8 && n64 <= 32)) && r.groups * (n64 + depth) <= 256) return n64;
  return coarse_slices(T) >= 8 && n128 <= 32 && r.groups * (n128 + depth) <= 256 ? n128 : 0;
}
// No length up to T has more of them.
static int most_finest_slices(const DecodeRule& r, int T) {
  const long long n32 = (T + 31) / 32, n64 = (T + 63) / 64, n128 = (T + 127) / 128;
  if (r.mfma) return (int)std::max(std::min({n32, 16ll, most_of_32(r) / r.groups}), std::min({n64, 96ll, most_of_64(r) / r.groups}));
  return (int)std::min({r.d == 128 ? n64 : n128, 32ll, 256 / r.groups});
}
static DecodePlan cut(const DecodeRule& r, int T, int most) {
  int s = r.want < most ? r.want : most;
  if (s < 1) s = 1;
  DecodePlan pl;
  pl.mfma = r.mfma;
  pl.keys_per_split = ((T + s - 1) / s + r.step - 1) / r.step * r.step;
  pl.n_split = (T + pl.keys_per_split - 1) / pl.keys_per_split;
  return pl;
}
// The cut of a call whose partial results (of n_split slices and the depth slots) have `room` bytes: the finer
// slices if they fit and make no more rounds, else the coarser ones.
static DecodePlan decode_plan(const DecodeRule& r, int T, int depth_count, size_t room) {
  const int depth = depth_count > 0 ? 1 : 0;
  const int finest = finest_slices(r, T, depth_count);
  if (finest > 0 && finest <= r.most_fine && (size_t)(finest + 1) * r.slice_bytes <= room) return cut(r, T, finest);
  const DecodePlan coarse = cut(r, T, coarse_slices(T));
  const int most = fine_slices(r.mfma, T);
  if (most > r.most_fine || (!r.mfma && T > 1024 && coarse_slices(T) > r.most_for_8)) return coarse;
  const DecodePlan fine = cut(r, T, most);
  const bool fits = (size_t)(fine.n_split + 1) * r.slice_bytes <= room;
  return fits && r.rounds(fine.n_split + depth) <= r.rounds(coarse.n_split + depth) ? fine : coarse;
}

// What every length up to T needs at most for its finer cut, taken or not, so that a workspace of the longest
// context serves the shorter ones.  (A cut never has more than min(want, most) slices, and among the lengths up to
// T the finer ones take every number of slices up to min(fine, most_fine).)
size_t decode_workspace_bytes(int B, int Hq, int Hk, int T, int d) {
  const DecodeRule r = decode_rule(B, Hq, Hk, d);
  int most = std::max(fine_slices(r.mfma, T), most_finest_slices(r, T));
  if (most > r.most_fine) most = r.most_fine > coarse_slices(T) ? r.most_fine : coarse_slices(T);
  return (size_t)((r.want < most ? r.want : most) + 1) * r.slice_bytes;
}

size_t decode_least_bytes(int B, int Hq, int Hk, int T, int d) {
  const DecodeRule r = decode_rule(B, Hq, Hk, d);
  return (size_t)(cut(r, T, coarse_slices(T)).n_split + 1) * r.slice_bytes;
}

// Calls that take one kernel: few batches of rows (256 at d = 64, 128 at d = 128), more of them where the workgroups fill the
// chip anyway (a little more than one round of them does not); groups of more than 4 heads, in chunks of 4, one batch and no more
// workgroups than units; 3 or 4 heads one batch, and above 256 workgroups, of which a unit holds one at a time, only up to two
// rounds and where the other kernels have a second slice to fold.  Two kernels / one,
// us, whole call, (batch, key/value head)s, rows:
//   1 head   d=64 48, 35 5.4 / 3.7;   180, 150 5.9 / 3.6;   24, 308 5.4 / 4.4;   12, 745 5.5 / 5.1;   48, 1217 6.2 / 7.4;   720, 1015 34.6 / 28.4
//            d=128 16, 93 5.4 / 3.5;   80, 151 6.1 / 4.5;   368, 293 13.5 / 11.6;   16, 510 6.0 / 6.0;   8, 843 5.9 / 8.7
//   2 heads  d=64 40, 220 5.8 / 4.4;   8, 341 5.8 / 5.4;   64, 593 6.5 / 6.8;   d=128 816, 79 17.0 / 10.6;   50, 351 6.5 / 6.8
//            d=64 264, 986 16.1 / 18.2;   400 to 640, 800 to 1000 0.93
//   4 heads  d=64 128, 80 6.5 / 5.6;   32, 527 6.7 / 9.7;   d=128 148, 121 10.3 / 5.7;   8, 129 6.9 / 7.4;   3 or 4 heads, no slots:
//            d=64 536, 12 9.8 / 13.3;   666, 55 10.0 / 13.6;   d=128 648, 49 10.3 / 13.9;   with slots: 257 to 512 0.68 to 1.03, 552, 61 1.07
//   8 heads  d=64 4, 236 6.9 / 5.4;   164, 210 8.1 / 10.0;   d=128 112, 118 9.2 / 6.0;   32 heads: 29, 108 9.0 / 5.6, 56, 34 8.5 / 9.6
static bool decode_in_one(const DecodeParams& p, int d, int gt) {
  const int batch = kDecOneWaves * (64 / (d / 8)) * 4, G = p.Hq / p.Hk;
  const long long batches = ((long long)p.T + p.depth_count + batch - 1) / batch, blocks = (long long)p.B * p.Hk * ((G + gt - 1) / gt);
  if (!grid_ok(blocks, kDecOneWaves * 64)) return false;
  if (G > 4) return batches <= 1 && blocks <= 256;
  if (gt == 4) return batches <= 1 && (blocks <= 256 || (blocks <= 512 && p.n_slices > 1));
  return batches <= (blocks >= 384 ? 4 : blocks >= 256 ? 3 : gt == 1 && d == 64 ? 3 : 2);
}

template <int D>
static hipError_t launch_in_one(const DecodeParams& p, int gt, hipStream_t stream) {
  const long long blocks = (long long)p.B * p.Hk * ((p.Hq / p.Hk + gt - 1) / gt);
  return launch_kernel(gt == 4 ? moda_decode_one_kernel<D, 4> : gt == 2 ? moda_decode_one_kernel<D, 2> : moda_decode_one_kernel<D, 1>,
                       dim3((unsigned)blocks), dim3(kDecOneWaves * 64), stream, p);
}

template <int D>
static hipError_t launch_decode_d(DecodeParams p, bool mfma, hipStream_t stream) {
  const int G = p.Hq / p.Hk;
  if (decode_in_one(p, D, decode_heads_per_chunk(G))) return launch_in_one<D>(p, decode_heads_per_chunk(G), stream);
  const int groups = merge_groups(p.n_slices, (long long)p.B * p.Hq, D);
  if (!grid_ok((long long)p.B * p.Hq, groups * D)) return kGridTooLarge;
  hipError_t e;
  if (mfma) {
    const long long blocks = (long long)p.B * p.Hk * ((G + 31) / 32) * ((p.n_slices + kDecMWaves - 1) / kDecMWaves);
    if (!grid_ok(blocks, kDecMWaves * 64)) return kGridTooLarge;
    e = launch_kernel(moda_decode_partial_mfma_kernel<D>, dim3((unsigned)blocks), dim3(kDecMWaves * 64), stream, p);
  } else {
    const int gt = decode_heads_per_chunk(G);
    const long long blocks = (long long)p.B * p.Hk * ((G + gt - 1) / gt) * p.n_slices;
    if (!grid_ok(blocks, kDecWaves * 64)) return kGridTooLarge;
    dim3 grid((unsigned)blocks), block(kDecWaves * 64);
    if (gt == 4) e = launch_kernel(moda_decode_partial_kernel<D, 4>, grid, block, stream, p);
    else if (gt == 2) e = launch_kernel(moda_decode_partial_kernel<D, 2>, grid, block, stream, p);
    else e = launch_kernel(moda_decode_partial_kernel<D, 1>, grid, block, stream, p);
  }
  if (e != hipSuccess) return e;
  if (groups == 1)
    return launch_kernel(moda_decode_merge_kernel<D, 1>, dim3((unsigned)(p.B * p.Hq)), dim3(D), stream, p);
  return launch_kernel(moda_decode_merge_kernel<D, 4>, dim3((unsigned)(p.B * p.Hq)), dim3(4 * D), stream, p);
}

hipError_t launch_decode_bf16(const void* Q, const void* Kseq, const void* Vseq, const void* Kdepth,
                              const void* Vdepth, void* O, float* LSE, float* ws, size_t ws_bytes, int B, int Hq,
                              int Hk, int T, int T_alloc, int d, int depth_alloc, int depth_count, float scale,
                              hipStream_t stream) {
  DecodeParams p;
  p.Q = Q; p.Kseq = Kseq; p.Vseq = Vseq; p.Kdepth = Kdepth; p.Vdepth = Vdepth;
  p.O = O; p.LSE = LSE; p.ws = ws;
  p.B = B; p.Hq = Hq; p.Hk = Hk; p.T = T; p.T_alloc = T_alloc;
  p.depth_alloc = depth_alloc; p.depth_count = depth_count;
  const DecodePlan pl = decode_plan(decode_rule(B, Hq, Hk, d), T, depth_count, ws_bytes);
  p.n_split = pl.n_split;
  p.keys_per_split = pl.keys_per_split;
  p.n_slices = pl.n_split + (depth_count > 0 ? 1 : 0);
  p.scale = scale;
  p.scale_log2 = scale * 1.4426950408889634f;
  if (d == 128) return launch_decode_d<128>(p, pl.mfma, stream);
  if (d == 64) return launch_decode_d<64>(p, pl.mfma, stream);
  return hipErrorInvalidValue;
}

}  // namespace moda
