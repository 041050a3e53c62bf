// Internal declarations shared by the translation units of libstarattn.
// Nothing here is part of the public ABI (see include/star_attn.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

namespace star {

// Division by a number that is the same for a whole launch, for numerators below 2^31: the kernels
// that a short call waits for would otherwise spend a chain of twenty instructions on each.
// (n / d = (mulhi(n, m) + n) >> s with s = ceil(log2 d), m = floor(2^32 (2^s - d) / d) + 1.)
struct Div {
  uint32_t d, m, s;
};
inline Div make_div(uint32_t d) {
  Div x = {d, 0, 0};
  while (x.s < 31 && ((uint32_t)1 << x.s) < d) ++x.s;
  x.m = (uint32_t)((((uint64_t)1 << 32) * (((uint64_t)1 << x.s) - d)) / d + 1);
  return x;
}
__device__ inline uint32_t quotient(uint32_t n, const Div& x) { return (__umulhi(n, x.m) + n) >> x.s; }
__device__ inline Div div_of(uint32_t d, uint32_t m) { return Div{d, m, d > 1 ? 32u - (uint32_t)__builtin_clz(d - 1) : 0u}; }

// What a launch costs the host grows with its arguments beyond 112 bytes (96 / 128 / 192 / 288 bytes 2.8 / 3.2 / 3.6 / 4.0 us, where the
// host is at its slower pace; 2.3 to 2.5 at its faster one), and a wavefront waits for them at its start.  The decode, fp32 and
// merge kernels of a call under a flat plan, two launches that a short call consists of, take theirs packed (FlatCall, FlatMerge) and
// unpack them into what the others are handed.  Nine fp32 calls, 1024 keys: enqueueing 69 to 83 -> 62 to 65 us (54 to 56 at the faster
// pace); one token, us, at the faster pace: fp32 on 1024 keys 6.81 -> 6.60, bf16, 32 / 8 heads, on 2000 7.52 -> 7.34, four sequences of
// 8000 (64 / 8 heads) 28.4 -> 27.9.  (The row-tiled bf16 kernels would spill more, and their calls are longer.)

// ---------------------------------------------------------------------------
// Phase-2 split plan: every part of the cache (one per context block, plus the
// tail) is cut into `splits of split_len keys`; a split never straddles a part
// boundary, so per-part results can be rebuilt from whole splits.
// Split index s in [0, n_blocks * spb) is context block s / spb, piece s % spb;
// indices from n_blocks * spb on are pieces of the tail.
// ---------------------------------------------------------------------------
//
// A "flat" plan ignores part boundaries; it is used by calls that do not ask for
// per-part outputs, where equal splits matter more than part boundaries.  For the
// streaming decode kernel, with S = s_total splits, split s is the comb of 32-key
// steps s, s + S, s + 2S, ... of everything the call may see (split_len only sizes
// S), so that one split per resident workgroup sweeps the cache together with the
// others.  For the row-tiled kernels split s is the run [s, s + 1) * split_len; with one
// split the fp32 kernel writes the call's results itself and nothing is merged.
struct SplitPlan {
  int64_t split_len;   // keys per split (multiple of 32)
  int32_t spb;         // splits per context block
  int32_t st;          // splits for the tail [L, cache_capacity)
  int32_t n_blocks;    // n = ceil(L / b)
  int32_t s_total;     // n_blocks * spb + st  (flat: number of splits)
  int32_t decode;      // 1: streaming split-KV kernel, 0: row-tiled kernel
  int32_t flat;        // 1: splits ignore part boundaries
  int32_t tile_rows;   // row-tiled kernels: rows per workgroup (bf16 256 or 128, fp32 32 or 16)
  int32_t waves;       // decode kernel: wavefronts that share a split (more than one: flat plans only), taking
                       // its steps in turn: wavefront w of split s the steps s * waves + w, + S * waves, ...
                       // fp32 kernel: wavefronts that share a 16-row tile (4; anything else: 8)
};

// Geometry every kernel needs.  Strides are in elements.
struct Geom {
  int32_t B, Hq, Hkv, G, d;
  int64_t L, b, a, cap;
  float scale;          // softmax scale (natural units)
};

// What prefixes a context block after the first (values of the public
// STAR_ATTN_ANCHOR_* constants).
enum AnchorMode {
  ANCHOR_FIRST = 0, ANCHOR_PREVIOUS = 1, ANCHOR_EXTERNAL = 2, ANCHOR_PER_BLOCK = 3,
  ANCHOR_ALL_BLOCKS = 4   // the call is a host's share: its first block is prefixed too
};

struct Phase1Args {
  Geom g;
  const void* Q;        // [B, L, Hq, d]
  void* O;              // [B, L, Hq, d]
  float* LSE;           // [B, Hq, L] or null
  const void* Kc;       // caches [B, Hkv, cap, d], already holding the context
  const void* Vc;
  int32_t anchor_mode;  // AnchorMode
  const void* Ka;       // ANCHOR_EXTERNAL / ALL_BLOCKS / PER_BLOCK: anchor keys / values of n_anchor
  const void* Va;       // = 1 / 1 / n anchors, token-major [B, n_anchor, a, Hkv, d]
  const void* Kin;      // the token-major inputs [B, L, Hkv, d] to read keys / values from (and to
  const void* Vin;      // file in the caches); null: read the caches
  unsigned int* tickets;  // bf16 kernel: this launch's eight work-queue counters (device memory)
  int32_t tickets_clear;  // bf16 kernel: a preceding kernel of the call has zeroed them
  int32_t n_cu;           // bf16 kernel: compute units of the device the call runs on
};

// Anchor key rows [*lo, *hi) of 0-based block i, and whether they index the
// external anchor buffers (true; rows counted over all of a batch's anchors) or
// the context keys (false).  Block 0 has none, unless the call's context is a
// host's share that starts after the global first block (ANCHOR_ALL_BLOCKS).
__host__ __device__ inline bool anchor_range(const Geom& g, int mode, int64_t i, int64_t* lo,
                                             int64_t* hi) {
  if (g.a == 0 || (i == 0 && mode != ANCHOR_ALL_BLOCKS)) { *lo = 0; *hi = 0; return false; }
  if (mode == ANCHOR_PREVIOUS) { *lo = i * g.b - g.a; *hi = i * g.b; return false; }
  if (mode == ANCHOR_PER_BLOCK) { *lo = i * g.a; *hi = (i + 1) * g.a; return true; }
  *lo = 0; *hi = g.a;
  return mode == ANCHOR_EXTERNAL || mode == ANCHOR_ALL_BLOCKS;
}

// Rotary embedding a kernel applies on the way; log2_theta == 0: none.
struct Rotary {
  double log2_theta;
  int64_t pos0;         // position of the call's first new token
};

struct Phase2Args {
  Geom g;
  SplitPlan plan;
  int64_t cache_len;    // tokens cached before this call
  int32_t q_len;
  int32_t causal;       // 1: the new tokens are appended and token j sees rows [0, cache_len + j];
                        // 0: nothing is appended and every token sees rows [0, cache_len)
  const void* Qq;       // [B, q_len, Hq, d]
  const void* Kn;       // new tokens' K, V [B, q_len, Hkv, d], which the kernel appends; null: the
  const void* Vn;       // caches already hold them, or there are none
  void* Kc;
  void* Vc;
  float* O_sub;         // [B, s_total, Hq, q_len, d]   per-split local attention
  float* LSE_sub;       // [B, s_total, Hq, q_len]      per-split log-sum-exp
  void* O;              // fp32 kernel, flat plan of one split: the call's own results (MergeArgs'
  float* A;             // O, A, LSE) instead of O_sub / LSE_sub; else all null
  float* LSE;
  Rotary rotary;        // decode kernel: Qq and Kn as given are unrotated (log2_theta != 0), token j at pos0 + j
};

// Cache rows a phase-2 call may see in all, and new token j's exclusive bound.
__host__ __device__ inline int64_t visible_total(const Phase2Args& a) {
  return a.cache_len + (a.causal ? a.q_len : 0);
}
__host__ __device__ inline int64_t visible_limit(const Phase2Args& a, int j) {
  return a.causal ? a.cache_len + j + 1 : a.cache_len;
}

struct RowGrid {        // workgroups of the row-tiled phase-2 kernels: kv head fastest, row tile, split, batch
  Div Hkv, tiles, splits, G;
};
// A phase-2 call under a flat plan.
struct FlatCall {
  const void *Qq, *Kn, *Vn;
  void *Kc, *Vc;
  float *out, *lse;      // `kind`: 0 O_sub and LSE_sub, 1 O, 2 A and LSE
  int32_t cache_len, cap, q_len, split_len, s_total;
  uint32_t heads;        // G << 16 | Hkv
  float scale;
  int16_t causal, kind;
  uint32_t m[4];         // the divisors' (RowGrid)
  int32_t first_wg;
};
static_assert(sizeof(FlatCall) <= 112, "see above");
inline FlatCall pack(const Phase2Args& a, const RowGrid& by) {
  const Geom& g = a.g;
  FlatCall c = {a.Qq, a.Kn, a.Vn, a.Kc, a.Vc, nullptr, nullptr, (int32_t)a.cache_len, (int32_t)g.cap, a.q_len, (int32_t)a.plan.split_len,
                a.plan.s_total, (uint32_t)g.G << 16 | (uint32_t)g.Hkv, g.scale, (int16_t)a.causal, 0, {by.Hkv.m, by.tiles.m, by.splits.m, by.G.m}, 0};
  if (a.O) { c.kind = 1; c.out = (float*)a.O; }
  else if (a.A) { c.kind = 2; c.out = a.A; c.lse = a.LSE; }
  else { c.out = a.O_sub; c.lse = a.LSE_sub; }
  return c;
}
// (B, L, b and what a plan along blocks has stay unset: no kernel asks for them under a flat plan)
__device__ inline void unpack(const FlatCall& c, int d, Phase2Args* a) {
  Geom& g = a->g;
  g.G = c.heads >> 16; g.Hkv = c.heads & 0xffff; g.Hq = g.G * g.Hkv; g.d = d; g.cap = c.cap; g.scale = c.scale;
  g.B = 0; g.L = g.b = g.a = 0;
  a->plan = SplitPlan{c.split_len, 0, 0, 0, c.s_total, 0, 1, 0, 0};
  a->cache_len = c.cache_len; a->q_len = c.q_len; a->causal = c.causal;
  a->Qq = c.Qq; a->Kn = c.Kn; a->Vn = c.Vn; a->Kc = c.Kc; a->Vc = c.Vc;
  a->O_sub = c.out; a->LSE_sub = c.lse;
  a->O = c.kind == 1 ? c.out : nullptr; a->A = c.kind == 2 ? c.out : nullptr; a->LSE = c.kind == 2 ? c.lse : nullptr;
  a->rotary = Rotary{0.0, 0};
}

// Split s of (batch beta, head h, token j) is row
//   beta * batch_stride + s * split_stride + h * q_len + j
// of O_sub (d floats per row) and LSE_sub.
struct MergeArgs {
  Geom g;
  SplitPlan plan;
  int32_t q_len;
  int32_t out_bf16;
  const float* O_sub;
  const float* LSE_sub;
  int64_t batch_stride;
  int64_t split_stride;
  float* O_part;        // [B, n+1, Hq, q_len, d] or null
  float* LSE_part;      // [B, n+1, Hq, q_len] or null
  void* O;              // [B, q_len, Hq, d] in the storage dtype, or null
  float* A;             // the same result in fp32, [B, Hq, q_len, d] (Eq. 1 of everything
  float* LSE;           // merged), and its log-sum-exp [B, Hq, q_len]; each may be null
  void* Qq;             // with rotary.log2_theta != 0: the call's queries [B, q_len, Hq, 128] in bf16, to be
  Rotary rotary;        // rotated in place (flat plans; the kernels in front have read them as they were)
  int32_t wide;         // 1: the sums of a flat plan in 64 bits
};

// The streaming decode kernel runs in two set-ups.  K and V of a call that fit
// the 256 MB last-level cache with room to spare are found there by the next
// decode step: ordinary loads, four single-wavefront workgroups per CU.  Larger ones are
// used once per step and gone before the next: non-temporal loads, three per CU.
// (131072 tokens of eight heads: 82.6 us with three, 83.2 with four, 85.6 with six, 83.0 with two; 32768 of them, resident:
// 29.4 with four, 30.0 with six, 29.5 with eight.)
__host__ __device__ inline bool decode_cache_resident(const Geom& g, int64_t total_keys) {
  return 2 * (int64_t)g.B * g.Hkv * total_keys * g.d * 2 <= ((int64_t)192 << 20);
}
// Tokens of a call on unrotated projections up to which the decode kernel and the merge rotate them,
// instead of a kernel in front: every wavefront evaluates their angles.  us, front / here: 1 token on 8191 (32 / 8
// heads) 14.4 / 12.4, 4 tokens 15.9 / 13.8, 5 on 3000 (12 / 4) 12.3 / 10.1, 8 on 8191 (16 / 16) 18.6 / 18.7, 16 tokens
// 19.9 / 22.2.
constexpr int DECODE_ROPE_TOKENS = 8;
inline int decode_wavefronts_per_cu(bool resident) { return resident ? 4 : 3; }

// Key range [lo, hi) of split s of a plan other than the decode kernel's flat one (hi
// clipped to what exists for this call).
__host__ __device__ inline void split_range(const SplitPlan& p, int64_t L, int64_t b,
                                            int64_t total_keys, int s, int64_t* lo, int64_t* hi) {
  if (p.flat) {
    int64_t x = (int64_t)s * p.split_len, y = x + p.split_len;
    *lo = x < total_keys ? x : total_keys;
    *hi = y < total_keys ? y : total_keys;
    return;
  }
  int n_ctx = p.n_blocks * p.spb;
  if (s < n_ctx) {
    int64_t m = s / p.spb, piece = s % p.spb;
    int64_t blo = m * b, bhi = (m + 1) * b < L ? (m + 1) * b : L;
    int64_t x = blo + piece * p.split_len;
    int64_t y = x + p.split_len;
    *lo = x < bhi ? x : bhi;
    *hi = y < bhi ? y : bhi;
  } else {
    int64_t x = L + (int64_t)(s - n_ctx) * p.split_len;
    int64_t y = x + p.split_len;
    *lo = x < total_keys ? x : total_keys;
    *hi = y < total_keys ? y : total_keys;
  }
}

// Row tiling of the bf16 phase-1 kernel: heads of one KV group that share a workgroup,
// and tokens per workgroup.
int flash_heads_per_workgroup(int G);
int flash_tokens_per_workgroup(int G);

// Compute units of the current device (cached per device; 0 if the runtime refuses).
int device_cu_count();

// A launch counts work-items in 32 bits, and the runtime keeps the low 32 bits of a larger
// grid without an error: 8454015 workgroups of 512 threads run as 65407.  More workgroups than
// fit are therefore launched in pieces; launch(first, n) enqueues workgroups [first, first + n).
template <typename Launch>
inline hipError_t launch_in_pieces(int64_t workgroups, int threads, Launch launch) {
  const int64_t most = (int64_t)0xffffffffu / threads;
  for (int64_t first = 0; first < workgroups; first += most) {
    launch((unsigned)first, (unsigned)(workgroups - first < most ? workgroups - first : most));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Whether the nx bytes at x and the ny bytes at y have any in common.
inline bool overlap(const void* x, size_t nx, const void* y, size_t ny) {
  return (uintptr_t)x < (uintptr_t)y + ny && (uintptr_t)y < (uintptr_t)x + nx;
}

// What a phase-1 call launches: row tiles of `rows` rows shared by `waves` wavefronts, one
// workgroup each, or (queued) drawn from the work queues.
struct Phase1Plan {
  int32_t queued, rows, waves, group;
  int64_t tiles;
  int32_t split;       // fp32: products of bf16 parts
  int32_t pieces;      // fp32: workgroups that share a tile's columns of d (one if the results are stored over Q)
};
Phase1Plan phase1_plan_bf16(const Geom& g, int anchor_mode, int n_cu);
Phase1Plan phase1_plan_f32(const Geom& g);

// Host-side launchers (each returns the hipError_t of its launch).
// X [B, n_tokens, H, d] rotated into Y (same layout; Y may be X), token t at pos0 + t; with
// K and V (null: neither) [B, n_tokens, Hkv, d], rotated K and V as it is into cache rows
// [dst_row, dst_row + n_tokens).  `clear`: eight counters to zero on the way, or null.
hipError_t launch_rope(int dtype, const Geom& g, int H, const void* X, void* Y, const void* K, const void* V,
                       void* Kc, void* Vc, int64_t n_tokens, int64_t dst_row, int64_t pos0, double theta,
                       unsigned int* clear, hipStream_t st);
hipError_t launch_phase1_f32(const Phase1Args& a, hipStream_t st);
hipError_t launch_phase2_f32(const Phase2Args& a, hipStream_t st);
hipError_t launch_phase1_bf16(const Phase1Args& a, hipStream_t st);
hipError_t launch_phase2_rows_bf16(const Phase2Args& a, hipStream_t st);
hipError_t launch_phase2_decode_bf16(const Phase2Args& a, hipStream_t st);
hipError_t launch_merge(const MergeArgs& a, hipStream_t st);

}  // namespace star
