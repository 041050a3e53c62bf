// bf16 split-KV partial attention for decode-sized phase-2 calls (head_dim 128,
// G * q_len <= 16 rows per KV head, up to 32 or 64 without per-part outputs): Eq. 1-2
// evaluated per split of the cache, with Algorithm 2's "append, then attend" fused in.
//
// A decode step reads every cached K and V byte exactly once and does 4-8 flops
// per byte, so the kernel is built as an HBM stream:
//   * a wavefront walks its keys with no barriers; without per-part outputs the
//     N wavefronts of a KV head that are resident at once take the comb of 32-key steps
//     w, w + N, w + 2N, ... so that at any moment they
//     read one contiguous window of its cache (every memory channel busy, none
//     hot); with per-part outputs a split is a contiguous run inside one part;
//   * a split is one wavefront's keys and a workgroup one wavefront, or (SplitPlan::waves) four or two
//     wavefronts share one and meet in LDS behind the key loop, where the pairs of more splits would cost
//     more to store and merge (streams() and make_plan() in api.hip, with both sides measured);
//   * a 32-key step is loaded into registers with plain 16-byte loads: K (8 KiB) straight in the
//     layout the MFMA wants -- lane (i, j4) takes key i, bytes 64t + 16 j4 .. +15 of its row for
//     t = 0..3; V (8 KiB) as 1 KiB-contiguous bursts.  As soon as its scores are taken and its V is in
//     LDS the next step is requested into the same registers, ahead of the softmax and the products.
//     All waits are the compiler's (straight-line code, static register indices; steps that are not
//     cached as a whole have a loop of their own behind the others').  Measured against batches of two steps consumed before the next two are requested
//     (the resident set-up: one step, whose V the compiler requested only once its K was there), whole
//     calls: 131072 tokens of eight heads 84.8 -> 82.4 us, four sequences of 32768 84.5 -> 83.0, 32768 tokens 30.5 -> 29.4;
//     two steps per batch requested early: 84.1;
//   * a cache too large to stay in the 256 MB last-level cache between steps is
//     read with non-temporal loads (every byte is used once: leaving it out of
//     the caches is worth 9-16 % of the step at 0.5-4 GB); a smaller one with
//     ordinary loads, so that the next step finds it there;
//   * all G query heads of the KV group (and up to 16/G new tokens) form the 16
//     columns of v_mfma_f32_16x16x32_bf16, so K and V are read once per KV head; more rows are up to four
//     such column blocks (RB), every K and V^T fragment feeding all of them: 32 rows leave room for two wavefronts
//     on a SIMD (252 registers; three blocks would spill 70), 48 and 64 for one;
//     S^T = K Q^T leaves each lane with keys of one query column, and the
//     exponentiated tile is directly the B operand of O^T += V^T P^T; V goes
//     through an 8 KiB LDS buffer (one wavefront's LDS accesses are in order) only to be
//     read back transposed, 16-byte chunks rotated-XOR swizzled so that writes
//     and transposing reads are conflict-free;
//   * rows at or beyond cache_len are the new tokens: they are read from the
//     call's Kq/Vq and written to the cache by the workgroup whose split holds
//     them, so no separate append kernel runs before a decode step (PIPED and EARLY, in the kernel, say when);
//   * unrotated projections of a few tokens are rotated on the way: every wavefront turns its query
//     rows while its first step is under way, the one that files a new key its row (and the merge
//     kernel, behind all readers, the queries in memory).  A kernel in front of this one that did it
//     took 2.3 us and a launch.
// Each workgroup writes its split's normalised output rows and their
// log-sum-exp; the merge kernel folds the splits (Eq. 3-4).
#include "rotary.h"

namespace star {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) int i32x4;

constexpr int D = 128;
constexpr int ROWB = D * 2;
constexpr int STEP = 32;                 // keys per pipeline step
constexpr int STEPB = STEP * ROWB;       // 8 KiB of K (and of V) per step
constexpr int ROPE_TOKENS = DECODE_ROPE_TOKENS;
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

#define LDS_AS __attribute__((address_space(3)))

typedef const __attribute__((address_space(1))) char* GlobalBytes;
typedef const __attribute__((address_space(1))) i32x4* GlobalVec;

// chunk c of key row r sits in slot c ^ swz(r)
__device__ __forceinline__ int swz(int r) { return ((r << 1) & 15) | ((r >> 3) & 1); }

__device__ __forceinline__ float xor16(float x) {
  return __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(x), 0x401F));
}
__device__ __forceinline__ float xor32_max(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float xor32_sum(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// RB blocks of 16 rows: the lane's columns.
template <int RB>
struct DecState {
  bf16x8 q[RB][4];     // Q^T fragments: q[.][t] = Q[column lane%16][32t + 8*(lane/16) .. +7]
  f32x4 o[RB][8];      // O^T: o[.][dt][v] = O[column][16dt + 4*(lane/16) + v]
  float m[RB], l[RB];  // running maximum (raw logits; uniform over a column's four lanes), this lane's share of the sum
  float neg_mc[RB];    // -m * c (0 while nothing was visible)
};

// One 32-key step in registers.
struct StepRegs {
  i32x4 k[8];      // k[4kt + t]: key 16kt + lane%16, bytes 64t + 16*(lane/16) .. +15 (MFMA A operand)
  i32x4 v[8];      // v[it]: key 4it + lane/16, bytes 16*(lane%16) .. +15
};
template <int RB>
struct Scores {
  f32x4 s[RB][2];
};

// Where a split's rows come from: cache rows below `cache_len`, the call's new
// tokens (token-major, `new_stride` bytes between tokens) from there on.
struct Source {
  GlobalBytes Kb;      // cache base of this (batch, kv head)
  GlobalBytes Vb;
  GlobalBytes Kn;      // new-token base of this (batch, kv head)
  GlobalBytes Vn;
  int cache_len;
  int new_stride;
};

// Load the step [key0, key0 + 32), all of it cached.
template <bool NT>
__device__ __forceinline__ void load_step(StepRegs& r, const Source& src, int key0, unsigned koff, unsigned voff) {
  GlobalBytes kp = src.Kb + (size_t)key0 * ROWB, vp = src.Vb + (size_t)key0 * ROWB;
#pragma unroll
  for (int it = 0; it < 8; ++it) {
    GlobalVec ka = (GlobalVec)(kp + (it >> 2) * 16 * ROWB + (it & 3) * 64 + koff);
    r.k[it] = NT ? __builtin_nontemporal_load(ka) : *ka;
  }
#pragma unroll
  for (int it = 0; it < 8; ++it) {
    GlobalVec va = (GlobalVec)(vp + it * 4 * ROWB + voff);
    r.v[it] = NT ? __builtin_nontemporal_load(va) : *va;
  }
}
// cos and sin of the call's tokens, for a call on unrotated projections.
struct Angles {
  float cs[ROPE_TOKENS][D / 2], sn[ROPE_TOKENS][D / 2];
};
// One row of Q or K as the MFMA operands hold it (lane group j4: elements 32 t + 8 j4 .. +7 in x[t]).
template <typename T>
__device__ __forceinline__ void rotate(T* x, const Angles& angles, int token, int j4) {
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    bf16x8 lo = __builtin_bit_cast(bf16x8, x[t]), hi = __builtin_bit_cast(bf16x8, x[t + 2]);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float a = (float)lo[e], b = (float)hi[e];
      const float cs = angles.cs[token][32 * t + 8 * j4 + e], sn = angles.sn[token][32 * t + 8 * j4 + e];
      lo[e] = (__bf16)rotary_lo(a, b, cs, sn);
      hi[e] = (__bf16)rotary_hi(a, b, cs, sn);
    }
    x[t] = __builtin_bit_cast(T, lo);
    x[t + 2] = __builtin_bit_cast(T, hi);
  }
}

// The same for a step that ends past `hi` or among the call's tokens.  Rows at or past `hi`
// re-read the last valid row (they are masked in the score tile).
__device__ __forceinline__ void load_last(StepRegs& r, const Source& src, int key0, int hi, int lane) {
  const int col = lane & 15, j4 = lane >> 4;
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) {
    int kk = key0 + 16 * kt + col;
    kk = kk < hi ? kk : hi - 1;
    GlobalBytes kp = kk < src.cache_len ? src.Kb + (size_t)kk * ROWB : src.Kn + (size_t)(kk - src.cache_len) * src.new_stride;
#pragma unroll
    for (int t = 0; t < 4; ++t) r.k[4 * kt + t] = *(GlobalVec)(kp + t * 64 + j4 * 16);
  }
#pragma unroll
  for (int it = 0; it < 8; ++it) {
    int vk = key0 + 4 * it + j4;
    vk = vk < hi ? vk : hi - 1;
    GlobalBytes vp = vk < src.cache_len ? src.Vb + (size_t)vk * ROWB : src.Vn + (size_t)(vk - src.cache_len) * src.new_stride;
    r.v[it] = *(GlobalVec)(vp + col * 16);
  }
}
// Such a step's keys that are the call's join the cache from the registers (turned, if they are unrotated).
template <bool ROPE>
__device__ __forceinline__ void file_last(StepRegs& r, const Source& src, char* Kc, char* Vc, int key0, int hi, int lane, const Angles* angles) {
  const int col = lane & 15, j4 = lane >> 4;
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) {
    const int kk = key0 + 16 * kt + col;
    if (kk < src.cache_len || kk >= hi) continue;
    if (ROPE) rotate(&r.k[4 * kt], *angles, kk - src.cache_len, j4);
#pragma unroll
    for (int t = 0; t < 4; ++t) *(i32x4*)(Kc + (size_t)kk * ROWB + t * 64 + j4 * 16) = r.k[4 * kt + t];
  }
#pragma unroll
  for (int it = 0; it < 8; ++it) {
    const int vk = key0 + 4 * it + j4;
    if (vk >= src.cache_len && vk < hi) *(i32x4*)(Vc + (size_t)vk * ROWB + col * 16) = r.v[it];
  }
}

// A step in two halves.  First its scores, and V into LDS (row 4it + lane/16, swizzled chunk
// lane%16): the step's registers are then free.
template <int RB>
__device__ __forceinline__ void score_step(const DecState<RB>& w, const StepRegs& r, const unsigned (&vw)[4],
                                           Scores<RB>& x) {
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int b = 0; b < RB; ++b) {
        const f32x4 acc = t == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : x.s[b][kt];
        x.s[b][kt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, r.k[4 * kt + t]), w.q[b][t], acc, 0, 0, 0);
      }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int it = 0; it < 8; ++it)
    *(LDS_AS i32x4*)(size_t)(vw[it & 3] + (it >> 2) * 16 * ROWB) = r.v[it];
}
template <int RB>
__device__ __forceinline__ void mask_step(Scores<RB>& x, int key0, const int (&lim)[RB], int j4) {
#pragma unroll
  for (int b = 0; b < RB; ++b) {
    const int n = lim[b] - key0 - 4 * j4;     // element (kt, v) is key key0 + 16kt + 4*j4 + v
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int v = 0; v < 4; ++v) x.s[b][kt][v] = (16 * kt + v) < n ? x.s[b][kt][v] : -INFINITY;
  }
}
// Then softmax and products.
template <int RB>
__device__ __forceinline__ void attend_step(DecState<RB>& w, const Scores<RB>& x, const unsigned (&vaddr)[8], float c) {
  // B operand slot e of lane group j4 is key 16(e/4) + 4*j4 + e%4; the A operand
  // (V^T, d-row lane%16) takes keys 4*j4..+3 and 16 + 4*j4..+3 from two
  // transposing reads.
  s16x4 lo[8], hi[8];
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) {
    lo[dt] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(size_t)(vaddr[dt]));
    hi[dt] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(size_t)(vaddr[dt] + 16 * ROWB));
  }
  __builtin_amdgcn_sched_barrier(0);
  bf16x8 p[RB];
#pragma unroll
  for (int b = 0; b < RB; ++b) {
    const f32x4(&s)[2] = x.s[b];
    const float tmax = fmaxf(fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3])),
                             fmaxf(fmaxf(s[1][0], s[1][1]), fmaxf(s[1][2], s[1][3])));
    // Lanes exchange their maxima only where some column's moves.  (The largest weight is exactly one this
    // way; a reference that moves later costs less and 6 % of precision.)
    if (__builtin_amdgcn_ballot_w64(tmax > w.m[b]) != 0) {
      const float m = fmaxf(w.m[b], xor32_max(fmaxf(tmax, xor16(tmax)))), mm = m == -INFINITY ? 0.f : m;
      const float alpha = __builtin_amdgcn_exp2f((w.m[b] - mm) * c);
      w.l[b] *= alpha;
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) w.o[b][dt] *= alpha;
      w.m[b] = m;
      w.neg_mc[b] = mm * -c;
    }
    float lsum = 0.f;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float e = __builtin_amdgcn_exp2f(__builtin_fmaf(s[kt][v], c, w.neg_mc[b]));
        lsum += e;
        p[b][4 * kt + v] = (__bf16)e;
      }
    w.l[b] += lsum;
  }
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) {
    bf16x8 a = __builtin_shufflevector(__builtin_bit_cast(bf16x4, lo[dt]), __builtin_bit_cast(bf16x4, hi[dt]), 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
    for (int b = 0; b < RB; ++b) w.o[b][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, p[b], w.o[b][dt], 0, 0, 0);
  }
}

// LDS of a workgroup of KW wavefronts: a step's V of each; behind the key loop, a half of d at a time (a quarter where
// that would pass 64 KiB), their results: row 16 b + lane % 16, 16-byte chunk of the piece XORed with the row's low bits.
template <int RB, int KW>
struct Meeting {
  union {
    char v[KW][STEPB];
    float o[KW][16 * RB][D / (RB > 2 ? 4 : 2)];
  };
  float m[KW][16 * RB], l[KW][16 * RB], scale[KW][16 * RB];
};
// KW wavefronts have walked different keys of the same rows: their sum goes to O_sub / LSE_sub, `to(row)`
// being a row's number there.  The order is fixed.
template <int RB, int KW, typename To>
__device__ __forceinline__ void meet(const Phase2Args& a, Meeting<RB, KW>& x, const DecState<RB>& w, int n_rows, float c, To to) {
  constexpr int ROWS = 16 * RB;
  constexpr int PIECES = RB > 2 ? 4 : 2, CHUNKS = 32 / PIECES;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, col = lane & 15, j4 = lane >> 4;
#pragma unroll
  for (int b = 0; b < RB; ++b) {
    const float l = xor32_sum(w.l[b] + xor16(w.l[b]));
    if (j4 == 0) { x.m[wave][16 * b + col] = w.m[b]; x.l[wave][16 * b + col] = l; }
  }
  __syncthreads();
  for (int i = tid; i < KW * ROWS; i += 64 * KW) {
    const int k = i / ROWS, row = i % ROWS;
    float m = -INFINITY;
#pragma unroll
    for (int n = 0; n < KW; ++n) m = fmaxf(m, x.m[n][row]);
    const float mm = m == -INFINITY ? 0.f : m;
    float l = 0.f;
#pragma unroll
    for (int n = 0; n < KW; ++n) l += x.l[n][row] * __builtin_amdgcn_exp2f((x.m[n][row] - mm) * c);
    x.scale[k][row] = l > 0.f ? __builtin_amdgcn_exp2f((x.m[k][row] - mm) * c) * (1.f / l) : 0.f;
    if (k == 0 && row < n_rows) a.LSE_sub[to(row)] = l > 0.f ? (m * c + __builtin_amdgcn_logf(l)) * LN2 : -INFINITY;
  }
#pragma unroll
  for (int h = 0; h < PIECES; ++h) {
    if (h > 0) __syncthreads();
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
      for (int dt = 0; dt < 8 / PIECES; ++dt)
        *(f32x4*)&x.o[wave][16 * b + col][((4 * dt + j4) ^ (col & (CHUNKS - 1))) * 4] = w.o[b][8 / PIECES * h + dt];
    __syncthreads();
    for (int i = tid; i < ROWS * CHUNKS; i += 64 * KW) {
      const int row = i / CHUNKS, chunk = i % CHUNKS;
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < KW; ++k) acc += *(const f32x4*)&x.o[k][row][(chunk ^ (row & (CHUNKS - 1))) * 4] * x.scale[k][row];
      if (row < n_rows) *(f32x4*)(a.O_sub + to(row) * D + D / PIECES * h + 4 * chunk) = acc;
    }
  }
}

// grid: x = split, y = kv head, z = batch; KW wavefronts, which take the split's steps in turn.  NT = non-temporal
// loads; ROPE = Qq and Kn are unrotated (at most ROPE_TOKENS tokens).  KW > 1: flat plans only.
struct DecodeDiv {
  Div steps, G;        // steps between two of a wavefront's (flat plans): splits times KW
};
// What a launch is handed: packed under a flat plan (m[0] and m[3] the divisors'), else as it is.
struct Call {
  Phase2Args a;
  DecodeDiv by;
};
struct FlatTurnedCall {
  FlatCall call;
  Rotary rotary;
};
template <int KW>
__device__ __forceinline__ Call unpacked(const Call& c) { return c; }
template <int KW>
__device__ __forceinline__ Call unpacked(const FlatCall& c) {
  Call x;
  unpack(c, D, &x.a);
  x.by = DecodeDiv{div_of(c.s_total * KW, c.m[0]), div_of(x.a.g.G, c.m[3])};
  return x;
}
template <int KW>
__device__ __forceinline__ Call unpacked(const FlatTurnedCall& c) {
  Call x = unpacked<KW>(c.call);
  x.a.rotary = c.rotary;
  return x;
}
template <bool NT, bool ROPE, int RB, int KW, typename C>
__global__ __launch_bounds__(64 * KW, RB > 2 ? 1 : 2) void decode_bf16_kernel(C call) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  const Call from = unpacked<KW>(call);
  const Phase2Args& a = from.a;
  const DecodeDiv& by = from.by;
  Meeting<RB, KW>& meeting = *(Meeting<RB, KW>*)lds;
  const Geom& g = a.g;
  const int wave = KW == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = KW == 1 ? threadIdx.x : threadIdx.x & 63;
  Angles* angles = (Angles*)(lds + sizeof(Meeting<RB, KW>)) + wave;      // each wavefront its own: no barrier
  const int qc = lane & 15, j4 = lane >> 4;
  const int sp = blockIdx.x, kvh = blockIdx.y, beta = blockIdx.z;
  const int R = g.G * a.q_len;                 // <= 16 RB live columns
  int head[RB], j[RB];
  bool live[RB];
#pragma unroll
  for (int b = 0; b < RB; ++b) {
    const int row = 16 * b + qc, token = quotient(row, by.G);
    live[b] = row < R;
    head[b] = kvh * g.G + row - token * g.G;
    j[b] = live[b] ? token : 0;
  }

  const int cache_len = (int)a.cache_len;
  const int total = (int)visible_total(a);
  // without new-token tensors the caches already hold the appended rows
  const bool fused_append = a.Kn != nullptr;
  const int cached = fused_append ? cache_len : total;
  // step `cur` of this wavefront covers keys [base + cur * stride, +32) below hi; the first n_whole of
  // them lie in the cache as a whole and are visible to every token
  const int first_lim = (int)visible_limit(a, 0), free_hi = cached < first_lim ? cached : first_lim;
  int base, stride, nsteps, n_whole, hi;
  const int first_step = sp * KW + wave, all_steps = a.plan.s_total * KW;      // (flat)
  if (KW > 1 || a.plan.flat) {
    const int T = (total + STEP - 1) / STEP, whole = free_hi / STEP;
    base = first_step * STEP;
    stride = all_steps * STEP;
    nsteps = first_step < T ? (int)quotient(T - first_step + all_steps - 1, by.steps) : 0;
    n_whole = first_step < whole ? (int)quotient(whole - first_step + all_steps - 1, by.steps) : 0;
    hi = total;
  } else {
    int64_t lo64, hi64;
    split_range(a.plan, g.L, g.b, total, sp, &lo64, &hi64);
    base = (int)lo64;
    stride = STEP;
    hi = (int)hi64;
    nsteps = hi > base ? (hi - base + STEP - 1) / STEP : 0;
    const int room = (free_hi < hi ? free_hi : hi) - base;
    n_whole = room > 0 ? room / STEP : 0;
  }
  const size_t out0 = ((size_t)beta * a.plan.s_total + sp) * g.Hq * a.q_len;
  if (KW == 1 && nsteps == 0) {                // empty split (short block, unused tail)
#pragma unroll
    for (int b = 0; b < RB; ++b)
      if (live[b] && j4 == 0) a.LSE_sub[out0 + (size_t)head[b] * a.q_len + j[b]] = -INFINITY;
    return;
  }

  Source src;
  const size_t cache0 = ((size_t)beta * g.Hkv + kvh) * (size_t)g.cap * ROWB, new0 = ((size_t)beta * a.q_len * g.Hkv + kvh) * ROWB;
  src.Kb = (GlobalBytes)a.Kc + cache0;
  src.Vb = (GlobalBytes)a.Vc + cache0;
  src.Kn = (GlobalBytes)a.Kn + new0;
  src.Vn = (GlobalBytes)a.Vn + new0;
  src.cache_len = cached;
  src.new_stride = g.Hkv * ROWB;

  // the query rows and the first step are requested before anything waits
  DecState<RB> w;
#pragma unroll
  for (int b = 0; b < RB; ++b) {
    GlobalBytes qrow = (GlobalBytes)a.Qq + (((size_t)beta * a.q_len + j[b]) * g.Hq + (live[b] ? head[b] : kvh * g.G)) * ROWB;
#pragma unroll
    for (int t = 0; t < 4; ++t) w.q[b][t] = __builtin_bit_cast(bf16x8, *(GlobalVec)(qrow + (32 * t + 8 * j4) * 2));
  }
  const unsigned koff = qc * ROWB + j4 * 16, voff = j4 * ROWB + qc * 16;
  StepRegs r;
  // The steps that hold the call's tokens are a wavefront's last, and the longest chain of a call where they are requested when the others are
  // done.  Caches read from HBM (NT): requested like the others, the tokens filed from the registers.  us: one token on 131072 (32 / 8 heads) 82.4 ->
  // 80.8, four sequences of 32768 (64 / 8) 82.7 -> 81.1, 300000 180.3 -> 176.8, 64 rows on 131072 90.6 -> 89.4.  Two tiles of 16 rows fill the
  // registers, and rotated keys are worth filing from them: there a first step only is requested early (32 rows on 8191 13.4 -> 12.4,
  // unrotated 10000 tokens (12 / 4) 10.7 -> 10.4; 32 rows on 20000 without / with the rest 19.3 / 19.9).  Other calls file the tokens from loads of their
  // own in front of the loop: stores late in a short call are waited for at its end (600 keys 7.3 / 7.5, 3000 of sixteen heads 9.15 / 9.4).
  constexpr bool PIPED = NT && RB != 2, EARLY = NT || ROPE || RB > 1;
  const auto request = [&](int s) {
    if (s < n_whole) load_step<NT>(r, src, base + s * stride, koff, voff);
    else if (EARLY && s < nsteps) load_last(r, src, base + s * stride, hi, lane);
  };
  request(0);
  __builtin_amdgcn_sched_barrier(0);
  if (ROPE) {
    static_assert(!ROPE || RB == 1, "a row per column");
    static_assert(D / 2 == 64, "a lane per pair");
    const double freq = rotary_frequency(lane, D, a.rotary.log2_theta);
    for (int t = 0; t < a.q_len; ++t)
      rotary_angle(a.rotary.pos0 + t, freq, &angles->cs[t][lane], &angles->sn[t][lane]);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    rotate(w.q[0], *angles, j[0], j4);
  }
#pragma unroll
  for (int b = 0; b < RB; ++b) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (!live[b]) w.q[b][t] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};     // dead columns contribute zeros
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) w.o[b][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    w.m[b] = -INFINITY;
    w.neg_mc[b] = 0.f;
    w.l[b] = 0.f;
  }

  // Algorithm 2, append: the new tokens whose rows fall into this wavefront's steps
  // join the cache (16 lanes move one 256-byte row of K and of V).
  if (!EARLY && fused_append && hi > cache_len) {
    for (int key = cache_len + j4; key < hi; key += 4) {
      const int step = key / STEP;                          // another split's step?
      if (KW > 1 || a.plan.flat ? step - (int)quotient(step, by.steps) * all_steps != first_step : key < base) continue;
      const size_t so = (size_t)(key - cache_len) * src.new_stride, dof = cache0 + (size_t)key * ROWB + qc * 16;
      const i32x4 k = *(GlobalVec)(src.Kn + so + qc * 16), v = *(GlobalVec)(src.Vn + so + qc * 16);
      *(i32x4*)((char*)a.Kc + dof) = k;
      *(i32x4*)((char*)a.Vc + dof) = v;
    }
  }

  const unsigned lds0 = (unsigned)(size_t)(LDS_AS char*)lds + wave * STEPB;
  // V rows into LDS: lane writes row 4it + lane/16, chunk lane%16 (swizzled)
  unsigned vw[4];
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    int row = 4 * it + j4;
    vw[it] = lds0 + row * ROWB + ((qc ^ swz(row)) << 4);
  }
  // V^T operand: source lane addresses row 4*j4 + (lane%16)/4 (+16 for the second
  // read), columns 16dt + 4*(lane%4) .. +3
  unsigned vaddr[8];
  {
    int rr = 4 * j4 + (qc >> 2);
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
      vaddr[dt] = lds0 + rr * ROWB + (((2 * dt + ((lane & 3) >> 1)) ^ swz(rr)) << 4) + 8 * (lane & 1);
  }

  const float c = g.scale * LOG2E;
  // Once a step's scores are there and its V is in LDS its registers are free, and the next step
  // is requested into them: it arrives behind this one's softmax and products, and those of the
  // other wavefronts of the CU.
  for (int s = 0; s < n_whole; ++s) {
    Scores<RB> x;
    score_step(w, r, vw, x);
    if (PIPED) request(s + 1);
    else if (s + 1 < n_whole) load_step<NT>(r, src, base + (s + 1) * stride, koff, voff);
    __builtin_amdgcn_sched_barrier(0);
    attend_step(w, x, vaddr, c);
  }
  int lim[RB];
#pragma unroll
  for (int b = 0; b < RB; ++b) {
    const int row_lim = live[b] ? (int)visible_limit(a, j[b]) : 0;
    lim[b] = row_lim < hi ? row_lim : hi;
  }
  for (int s = n_whole; s < nsteps; ++s) {
    Scores<RB> x;
    if (!PIPED && (!EARLY || s > 0)) load_last(r, src, base + s * stride, hi, lane);
    if (EARLY) file_last<ROPE>(r, src, (char*)a.Kc + cache0, (char*)a.Vc + cache0, base + s * stride, hi, lane, angles);
    score_step(w, r, vw, x);
    if (PIPED) request(s + 1);
    __builtin_amdgcn_sched_barrier(0);
    mask_step(x, base + s * stride, lim, j4);
    attend_step(w, x, vaddr, c);
  }

  if (KW > 1) {
    meet<RB, KW>(a, meeting, w, R, c, [&](int row) {
      const int token = quotient(row, by.G);
      return out0 + (size_t)(kvh * g.G + row - token * g.G) * a.q_len + token;
    });
    return;
  }
#pragma unroll
  for (int b = 0; b < RB; ++b) {
    const float l_tot = xor32_sum(w.l[b] + xor16(w.l[b]));
    if (!live[b]) continue;
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
    const size_t out = out0 + (size_t)head[b] * a.q_len + j[b];
    float* orow = a.O_sub + out * D;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) *(f32x4*)(orow + 16 * dt + 4 * j4) = w.o[b][dt] * inv;
    if (j4 == 0)
      a.LSE_sub[out] = l_tot > 0.f ? (w.m[b] * c + __builtin_amdgcn_logf(l_tot)) * LN2 : -INFINITY;
  }
}

template <bool NT, bool ROPE, int RB, int KW>
hipError_t launch(const Phase2Args& a, hipStream_t st) {
  const Geom& g = a.g;
  const dim3 grid((unsigned)a.plan.s_total, (unsigned)g.Hkv, (unsigned)g.B);
  const DecodeDiv by = {make_div((uint32_t)a.plan.s_total * KW), make_div(g.G)};
  const size_t lds = sizeof(Meeting<RB, KW>) + (ROPE ? KW * sizeof(Angles) : 0);
  if (a.plan.flat) {
    const FlatCall c = pack(a, RowGrid{by.steps, by.steps, by.steps, by.G});
    if constexpr (ROPE) decode_bf16_kernel<NT, ROPE, RB, KW, FlatTurnedCall><<<grid, 64 * KW, lds, st>>>(FlatTurnedCall{c, a.rotary});
    else decode_bf16_kernel<NT, ROPE, RB, KW, FlatCall><<<grid, 64 * KW, lds, st>>>(c);
  } else if constexpr (!ROPE && RB == 1 && KW == 1) {
    decode_bf16_kernel<NT, ROPE, RB, KW, Call><<<grid, 64 * KW, lds, st>>>(Call{a, by});
  } else {
    return hipErrorInvalidValue;      // (flat plans only)
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_phase2_decode_bf16(const Phase2Args& a, hipStream_t st) {
  const Geom& g = a.g;
  const int64_t rows = (int64_t)g.G * a.q_len;
  const int waves = a.plan.waves;
  if (g.Hkv > 65535 || g.B > 65535 || rows > 64 || (waves > 1 && !a.plan.flat)) return hipErrorInvalidValue;
  const bool resident = decode_cache_resident(g, visible_total(a));
  // what make_plan() gives, and nothing else: set-ups that share their splits are not told apart by their results
  if (rows <= 16 ? waves != 1 && (waves != 4 || !resident) : rows <= 32 ? waves != 4 && (waves != 2 || !resident) : waves != 4 || resident)
    return hipErrorInvalidValue;
  if (a.rotary.log2_theta != 0) {
    if (rows > 16 || a.q_len > ROPE_TOKENS) return hipErrorInvalidValue;
    if (waves == 4) return launch<false, true, 1, 4>(a, st);
    return resident ? launch<false, true, 1, 1>(a, st) : launch<true, true, 1, 1>(a, st);
  }
  if (rows <= 16) {
    if (waves == 4) return launch<false, false, 1, 4>(a, st);
    return resident ? launch<false, false, 1, 1>(a, st) : launch<true, false, 1, 1>(a, st);
  }
  if (rows <= 32) {
    if (waves == 2) return launch<false, false, 2, 2>(a, st);
    return resident ? launch<false, false, 2, 4>(a, st) : launch<true, false, 2, 4>(a, st);
  }
  return rows <= 48 ? launch<true, false, 3, 4>(a, st) : launch<true, false, 4, 4>(a, st);
}

}  // namespace star
