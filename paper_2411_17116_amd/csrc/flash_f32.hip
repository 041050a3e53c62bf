// fp32 path (head_dim 64 or 128): row-tiled attention on the fp32 matrix
// instructions, fp32 storage, products, sums and softmax throughout, so the result
// stays within 1e-5 of an fp64 evaluation at the sizes this path is meant for.
//
// What bounds it: the fp32 MFMA rate (157 TFLOP/s, 32 cycles for the 2048 flops of
// v_mfma_f32_16x16x4_f32) for long key ranges, latency for short ones.  Both are
// served by the same split:
//   * A workgroup owns a tile of 16 NB query rows of one KV group, and its KW
//     wavefronts share the tile's KEYS: wavefront w takes the 16-key units
//     w, w + KW, ...  Nothing crosses wavefronts until the end, so there is no LDS
//     and no barrier in the key loop, and a tile of few rows still has KW
//     wavefronts' worth of loads and MFMAs in flight.
//   * Rows are packed over the heads of a KV group (row = token * G + head in
//     group), so that a K/V unit is read once for all of them.
//   * S^T = K Q^T: lane (col = lane % 16, j4 = lane / 16) supplies K[col][16 t + 4 j4 + e]
//     straight from a 16-byte global load (any assignment of d to (MFMA step, lane
//     group) works as long as Q uses the same one) and receives keys 4 j4 + v of
//     query row col.  Those are exactly the lanes that have to supply P^T in MFMA
//     step v of O^T += V^T P^T, whose four keys are 4 j4 + v; V is loaded as
//     256-byte row pieces, element e of a lane's 16 bytes being output row
//     d = 64 h + 4 (lane % 16) + e of MFMA e.  So neither K, V nor P moves between lanes.
//   * K of the next unit is requested once the scores of this one are done, V once
//     its products are done: each load has half a unit of MFMAs (2048 cycles at
//     NB = 2, d = 128) to arrive.
//   * Softmax runs against a reference per row and wavefront that moves only when a score leaves its
//     headroom, so that a unit has no maximum search over lanes and no rescaling of O.
//   * The KW partial results (O, m, l) of a row meet in LDS once, at the end.
// Phase 1 reads K and V where the caller left them and files its own tokens' rows in
// the caches; phase 2 reads the new tokens from the call's Kq / Vq and appends them.
// Measured, whole calls, against a kernel of one thread per row: 8 / 2 heads, d = 128,
// L = 4099, b = 1024, a = 512: 3390 -> 151 us (100 TFLOP/s; 119 at 8192 tokens in blocks of
// 2048, where a library fp32 matrix product reaches 152); 1 head, d = 64, L = 1024,
// b = a = 256: 274 -> 9.9 us.
#include "star_internal.h"

namespace star {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

typedef const __attribute__((address_space(1))) char* GlobalBytes;
typedef const __attribute__((address_space(1))) f32x4* GlobalVec;

constexpr int UNIT = 16;   // keys per step of a wavefront
// How far (log2 units) a score may rise above its row's reference before the reference moves.
// O / l does not depend on the reference, and 2^8 times the largest numerator is as far from overflow
// as it was, so nothing is lost; scores of N(0, 1) inputs stay within it of the first unit's, and a
// unit then costs no exchange between lanes and no rescaling of O.  Against moving it to every new maximum, us
// (8 / 2 heads): d = 128: L = 4099 (b = 1024, a = 512) 152 -> 142, 8192 (b = a = 2048) 706 -> 663, L = 3001 53.7 ->
// 52.2; d = 64: 8192 375 -> 352, 4099 117.5 -> 107.7; 1 head, 1024 10.2 -> 9.8.
constexpr float HEADROOM = 8.f;
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

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

// The keys a row tile walks: rows [a_lo, a_hi) of Ka / Va, visible to every row of
// the tile, then keys [l_lo, l_hi), of which a row sees those below its own bound;
// key k of the second range is row k - l_off of Kl / Vl.  Consecutive rows are
// a_stride / l_stride bytes apart.
// Everything here is uniform over a wavefront, so that a unit's address is a scalar
// base plus a 32-bit offset per lane.
struct KeySeq {
  GlobalBytes Ka, Va, Kl, Vl;
  unsigned a_stride, l_stride;
  int a_lo, a_hi, l_lo, l_hi, l_off;
  int n_a, n_units;
  __device__ __forceinline__ void count() {
    n_a = (a_hi - a_lo + UNIT - 1) / UNIT;
    n_units = n_a + (l_hi - l_lo + UNIT - 1) / UNIT;
  }
};

// A wavefront's state.  Lane (col, j4) belongs to row col of each of NB 16-row blocks.
template <int D, int NB>
struct RowState {
  f32x4 q[NB][D / 16];        // q[.][t][e] = Q[row][16 t + 4 j4 + e] * scale * log2(e)
  f32x4 o[NB][D / 64][4];     // o[.][h][e][w] = O[row][64 h + 16 j4 + 4 w + e]
  float m[NB], top[NB];       // reference (log2 units; uniform over a row's four lanes; 0 until a key is
                              // visible) and the score beyond which it moves (-inf until then)
  float l[NB];                // this lane's share of the sum of 2^(s - m)
};

template <int D>
struct Unit {
  f32x4 k[D / 16];
  f32x4 v[4][D / 64];
};

// Unit u: its first row in K / V, how many rows of the range are left from there on,
// and its first key.
struct UnitAt {
  GlobalBytes K, V;
  unsigned stride;
  int n_rows;
  int key0;
  bool local;
};
__device__ __forceinline__ UnitAt unit_at(const KeySeq& seq, int u) {
  // the four bases as scalars of their own: chosen between as struct members, the
  // compiler would keep the struct in scratch memory and index it
  GlobalBytes Ka = seq.Ka, Va = seq.Va, Kl = seq.Kl, Vl = seq.Vl;
  asm("" : "+s"(Ka), "+s"(Va), "+s"(Kl), "+s"(Vl));
  UnitAt x;
  x.local = u >= seq.n_a;
  x.key0 = x.local ? seq.l_lo + (u - seq.n_a) * UNIT : seq.a_lo + u * UNIT;
  x.n_rows = (x.local ? seq.l_hi : seq.a_hi) - x.key0;
  x.stride = x.local ? seq.l_stride : seq.a_stride;
  const size_t off = (size_t)(x.local ? x.key0 - seq.l_off : x.key0) * x.stride;
  x.K = (x.local ? Kl : Ka) + off;
  x.V = (x.local ? Vl : Va) + off;
  return x;
}

// Rows past the range's end re-read its last row (their scores are masked).
template <int D>
__device__ __forceinline__ void load_k(Unit<D>& r, const UnitAt& x, int lane) {
  int i = lane & 15;
  if (x.n_rows < UNIT) i = i < x.n_rows ? i : x.n_rows - 1;
  const unsigned off = (unsigned)i * x.stride + 16 * (lane >> 4);
#pragma unroll
  for (int t = 0; t < D / 16; ++t) r.k[t] = *(GlobalVec)(x.K + off + 64 * t);
}
template <int D>
__device__ __forceinline__ void load_v(Unit<D>& r, const UnitAt& x, int lane) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    int i = 4 * (lane >> 4) + v;
    if (x.n_rows < UNIT) i = i < x.n_rows ? i : x.n_rows - 1;
    const unsigned off = (unsigned)i * x.stride + 16 * (lane & 15);
#pragma unroll
    for (int h = 0; h < D / 64; ++h) r.v[v][h] = *(GlobalVec)(x.V + off + 256 * h);
  }
}

// One unit: scores, softmax, products.  MORE: K and V of unit `nxt` are requested as soon
// as this unit's are used up -- without a branch, so that the compiler's waits for V
// need not include them.
template <int D, int NB, bool MORE>
__device__ __forceinline__ void attend_unit(RowState<D, NB>& w, Unit<D>& r, const UnitAt& cur, const UnitAt& nxt,
                                            const int (&row_lim)[NB], int wave_lim, int lane) {
  const int j4 = lane >> 4;
  // four chains per score tile (element e of every 16-byte piece has its own; two where the
  // registers are used up): a quarter of the terms, and of the partial sums' size, per chain
  // keeps the rounding of a large logit down
  constexpr int CH = NB == 2 && D == 128 ? 2 : 4;
  f32x4 s[NB], part[NB][CH];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int k = 0; k < CH; ++k) part[b][k] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < D / 16; ++t)
#pragma unroll
    for (int e = 0; e < 4; e += 2)
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int k = e; k < e + 2; ++k)
          part[b][k % CH] = __builtin_amdgcn_mfma_f32_16x16x4f32(r.k[t][k], w.q[b][t][k], part[b][k % CH], 0, 0, 0);
  if (MORE) load_k<D>(r, nxt, lane);
#pragma unroll
  for (int b = 0; b < NB; ++b)
    s[b] = CH == 2 ? part[b][0] + part[b][1] : (part[b][0] + part[b][1]) + (part[b][CH - 2] + part[b][CH - 1]);
  if (cur.n_rows < UNIT || (cur.local && cur.key0 + UNIT > wave_lim)) {
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int room = row_lim[b] - cur.key0;
      const int n = (cur.local && room < cur.n_rows ? room : cur.n_rows) - 4 * j4;
#pragma unroll
      for (int v = 0; v < 4; ++v) s[b][v] = v < n ? s[b][v] : -INFINITY;
    }
  }
  float t[NB];
  bool beyond = false;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    t[b] = fmaxf(fmaxf(s[b][0], s[b][1]), fmaxf(s[b][2], s[b][3]));
    beyond |= t[b] > w.top[b];
  }
  if (__builtin_amdgcn_ballot_w64(beyond) != 0) {      // some row's reference moves
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const float row = xor32_max(fmaxf(t[b], xor16(t[b])));
      const float m_old = w.top[b] == -INFINITY ? -INFINITY : w.m[b], m_new = fmaxf(m_old, row);
      const float m = m_new == -INFINITY ? 0.f : m_new;
      const float alpha = __builtin_amdgcn_exp2f(m_old - m);   // 0 while nothing was visible
      w.m[b] = m;
      w.top[b] = m_new + HEADROOM;
      w.l[b] *= alpha;
#pragma unroll
      for (int h = 0; h < D / 64; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) w.o[b][h][e] *= alpha;
    }
  }
#pragma unroll
  for (int b = 0; b < NB; ++b) {
#pragma unroll
    for (int v = 0; v < 4; ++v) s[b][v] = __builtin_amdgcn_exp2f(s[b][v] - w.m[b]);
    w.l[b] += (s[b][0] + s[b][1]) + (s[b][2] + s[b][3]);
  }
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int h = 0; h < D / 64; ++h)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          w.o[b][h][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(r.v[v][h][e], s[b][v], w.o[b][h][e], 0, 0, 0);
  if (MORE) load_v<D>(r, nxt, lane);
}

// The lane's query row of row block b, as it is in memory (scale_rows() follows once the
// first keys have been requested, so that both round trips overlap).
template <int D, int NB>
__device__ __forceinline__ void load_row(RowState<D, NB>& w, int b, const float* q, int j4) {
#pragma unroll
  for (int t = 0; t < D / 16; ++t) w.q[b][t] = *(const f32x4*)(q + 16 * t + 4 * j4);
#pragma unroll
  for (int h = 0; h < D / 64; ++h)
#pragma unroll
    for (int e = 0; e < 4; ++e) w.o[b][h][e] = f32x4{0.f, 0.f, 0.f, 0.f};
  w.m[b] = 0.f;
  w.top[b] = -INFINITY;
  w.l[b] = 0.f;
}
template <int D, int NB>
__device__ __forceinline__ void scale_rows(RowState<D, NB>& w, float qk_scale) {
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int t = 0; t < D / 16; ++t) w.q[b][t] *= qk_scale;
}

// Attend the wavefront's rows to units first, first + step, ... of the sequence.
//   row_lim   this lane's exclusive bound on keys of the second range, per row block
//   wave_lim  smallest bound of the wavefront's live rows
template <int D, int NB>
__device__ __forceinline__ void attend(RowState<D, NB>& w, const KeySeq& seq, int first, int step,
                                       const int (&row_lim)[NB], int wave_lim, float qk_scale, int lane) {
  if (first >= seq.n_units) return;
  Unit<D> r;
  UnitAt cur = unit_at(seq, first);
  load_k<D>(r, cur, lane);
  load_v<D>(r, cur, lane);
  scale_rows<D, NB>(w, qk_scale);
  for (int u = first + step; u < seq.n_units; u += step) {
    const UnitAt nxt = unit_at(seq, u);
    attend_unit<D, NB, true>(w, r, cur, nxt, row_lim, wave_lim, lane);
    cur = nxt;
  }
  attend_unit<D, NB, false>(w, r, cur, cur, row_lim, wave_lim, lane);
}

// LDS in which the KW wavefronts' results of a tile meet, 64 columns of d at a time.
// The pitch of 68 floats spreads the 16 rows of a 16-byte write over all banks.
template <int NB, int KW>
struct Meet {
  float o[KW][16 * NB][68];
  float m[KW][16 * NB], l[KW][16 * NB];
  float scale[KW][16 * NB];
};

// Fold the wavefronts' partial results; `store(row, col, f32x4)` takes the normalised
// output of tile row `row`, columns col .. col + 3, and `store_lse(row, lse)` its
// natural-log denominator (-inf, output 0, for a row that saw no key).
template <int D, int NB, int KW, typename Store, typename StoreLse>
__device__ __forceinline__ void meet(RowState<D, NB>& w, Meet<NB, KW>& x, Store store, StoreLse store_lse) {
  constexpr int ROWS = 16 * NB;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, col = lane & 15, j4 = lane >> 4;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    float l = w.l[b] + xor16(w.l[b]);
    l = xor32_sum(l);
    if (j4 == 0) { x.m[wave][16 * b + col] = w.top[b] == -INFINITY ? -INFINITY : w.m[b]; x.l[wave][16 * b + col] = l; }
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
    for (int n = 0; n < KW; ++n) l += x.l[n][row] * __builtin_amdgcn_exp2f(x.m[n][row] - mm);
    x.scale[k][row] = l > 0.f ? __builtin_amdgcn_exp2f(x.m[k][row] - mm) * (1.f / l) : 0.f;
    if (k == 0) store_lse(row, l > 0.f ? (m + log2f(l)) * LN2 : -INFINITY);
  }
#pragma unroll
  for (int h = 0; h < D / 64; ++h) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        *(f32x4*)&x.o[wave][16 * b + col][16 * j4 + 4 * c] =
            f32x4{w.o[b][h][0][c], w.o[b][h][1][c], w.o[b][h][2][c], w.o[b][h][3][c]};
    __syncthreads();
    for (int i = tid; i < ROWS * 16; i += 64 * KW) {
      const int row = i >> 4, c = 4 * (i & 15);
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < KW; ++k) acc += *(const f32x4*)&x.o[k][row][c] * x.scale[k][row];
      store(row, 64 * h + c, acc);
    }
    if (h + 1 < D / 64) __syncthreads();
  }
}

// Copy `n` rows of d floats (K and V) into cache rows: 16 bytes per thread and step, the
// calling thread being `thread` of `n_threads`.
template <int D>
__device__ __forceinline__ void file_rows(const float* K, const float* V, int64_t stride, float* Kc, float* Vc,
                                          int n, int thread, int n_threads) {
  for (int i = thread; i < n * (D / 4); i += n_threads) {
    const int row = i / (D / 4), c = 4 * (i % (D / 4));
    const f32x4 k = *(const f32x4*)(K + row * stride + c), v = *(const f32x4*)(V + row * stride + c);
    *(f32x4*)(Kc + (int64_t)row * D + c) = k;
    *(f32x4*)(Vc + (int64_t)row * D + c) = v;
  }
}

// ------------------------------------------------------------------ phase 1
// Workgroups are numbered (kv head fastest, batch, block in group -- block 0, which has no anchor,
// last --, tile in block -- late, i.e. heavy, first --, group of blocks).  Inside a group
// the tiles come in descending weight, so that those that share a CU, or come last,
// even out.
template <int D, int NB, int KW>
__global__ __launch_bounds__(64 * KW, 2) void phase1_f32_kernel(Phase1Args a, int group, int tiles_per_block,
                                                                int first_wg) {
  __shared__ Meet<NB, KW> x;
  constexpr int ROWS = 16 * NB;
  const Geom& g = a.g;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, col = lane & 15, j4 = lane >> 4;
  int id = first_wg + (int)blockIdx.x;
  const int kvh = id % g.Hkv; id /= g.Hkv;
  const int beta = id % g.B; id /= g.B;
  const int n = (int)((g.L + g.b - 1) / g.b), first = id / (group * tiles_per_block) * group;
  id -= first * tiles_per_block;
  const int in_group = n - first < group ? n - first : group;
  const int i = first + id % in_group + 1 == n ? 0 : first + id % in_group + 1;
  const int t = tiles_per_block - 1 - id / in_group;
  const int s = (int)(i * g.b);
  const int e = (int)(s + g.b < g.L ? s + g.b : g.L);
  const int r0 = t * ROWS, n_rows = (e - s) * g.G;    // rows of this block
  if (r0 >= n_rows) return;                           // tile beyond a short block
  const int live_rows = n_rows - r0 < ROWS ? n_rows - r0 : ROWS;
  const int tok0 = s + r0 / g.G, head0 = r0 % g.G;    // the tile's first row; row rr is rr rows on

  // K / V rows from the token-major inputs when they are handed over as they are
  // (then this kernel also files them in the caches), else from the filled caches
  const bool from_input = a.Kin != nullptr;
  const int64_t stride = from_input ? (int64_t)g.Hkv * D : D;      // floats between rows
  const int64_t in0 = ((int64_t)beta * g.L * g.Hkv + kvh) * D, cache0 = ((int64_t)beta * g.Hkv + kvh) * g.cap * D;
  const float* Kb = from_input ? (const float*)a.Kin + in0 : (const float*)a.Kc + cache0;
  const float* Vb = from_input ? (const float*)a.Vin + in0 : (const float*)a.Vc + cache0;

  RowState<D, NB> w;
  int row_lim[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int rr = 16 * b + col;
    const unsigned r = head0 + (rr < live_rows ? rr : 0);     // rows past the block repeat the first
    const int tok = tok0 + (int)(r / (unsigned)g.G), head = kvh * g.G + (int)(r % (unsigned)g.G);
    row_lim[b] = tok + 1;
    load_row<D, NB>(w, b, (const float*)a.Q + (((int64_t)beta * g.L + tok) * g.Hq + head) * D, j4);
  }
  const int wave_lim = tok0 + 1;                      // the tile's first row sees least

  KeySeq seq;
  int64_t a_lo, a_hi;
  const bool ext = anchor_range(g, a.anchor_mode, i, &a_lo, &a_hi);
  seq.a_lo = (int)a_lo; seq.a_hi = (int)a_hi;
  // separately given anchors: token-major, n_anchor * a rows per batch
  const int64_t anchor_rows = (int64_t)(a.anchor_mode == ANCHOR_PER_BLOCK ? n : 1) * g.a;
  const int64_t anchor0 = ((int64_t)beta * anchor_rows * g.Hkv + kvh) * D;
  seq.Ka = (GlobalBytes)(ext ? (const float*)a.Ka + anchor0 : Kb);
  seq.Va = (GlobalBytes)(ext ? (const float*)a.Va + anchor0 : Vb);
  seq.a_stride = (unsigned)(ext ? (int64_t)g.Hkv * D : stride) * 4;
  seq.Kl = (GlobalBytes)Kb; seq.Vl = (GlobalBytes)Vb; seq.l_stride = (unsigned)stride * 4; seq.l_off = 0;
  seq.l_lo = s;
  seq.l_hi = tok0 + (head0 + live_rows - 1) / g.G + 1;
  seq.count();
  attend<D, NB>(w, seq, wave, KW, row_lim, wave_lim, g.scale * LOG2E, lane);

  meet<D, NB, KW>(w, x,
      [&](int row, int c, f32x4 v) {
        if (row >= live_rows) return;
        const unsigned r = head0 + row;
        const int tok = tok0 + (int)(r / (unsigned)g.G), head = kvh * g.G + (int)(r % (unsigned)g.G);
        *(f32x4*)((float*)a.O + (((int64_t)beta * g.L + tok) * g.Hq + head) * D + c) = v;
      },
      [&](int row, float lse) {
        if (row >= live_rows || !a.LSE) return;
        const unsigned r = head0 + row;
        const int tok = tok0 + (int)(r / (unsigned)g.G), head = kvh * g.G + (int)(r % (unsigned)g.G);
        a.LSE[((int64_t)beta * g.Hq + head) * g.L + tok] = lse;
      });

  // Algorithm 1, "keep the block's K/V": a token is filed by the tile that holds its first row
  if (from_input) {
    const int t0 = tok0 + (head0 + g.G - 1) / g.G, t1 = tok0 + (head0 + live_rows + g.G - 1) / g.G;
    file_rows<D>(Kb + (int64_t)t0 * stride, Vb + (int64_t)t0 * stride, stride,
                 (float*)a.Kc + cache0 + (int64_t)t0 * D, (float*)a.Vc + cache0 + (int64_t)t0 * D, t1 - t0, threadIdx.x,
                 64 * KW);
  }
}

// ------------------------------------------------------------------ phase 2
// Workgroups are numbered (kv head fastest, row tile, split, batch).
template <int D, int NB, int KW>
__global__ __launch_bounds__(64 * KW, 2) void phase2_f32_kernel(Phase2Args a, int row_tiles, int first_wg) {
  __shared__ Meet<NB, KW> x;
  constexpr int ROWS = 16 * NB;
  const Geom& g = a.g;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, col = lane & 15, j4 = lane >> 4;
  int id = first_wg + (int)blockIdx.x;
  const int kvh = id % g.Hkv; id /= g.Hkv;
  const int tile = id % row_tiles; id /= row_tiles;
  const int sp = id % a.plan.s_total;
  const int beta = id / a.plan.s_total;
  const int r0 = tile * ROWS, n_rows = g.G * a.q_len;  // row = token * G + head in group
  const int live_rows = n_rows - r0 < ROWS ? n_rows - r0 : ROWS;

  const int total = (int)visible_total(a), cache_len = (int)a.cache_len;
  int64_t lo, hi;
  split_range(a.plan, g.L, g.b, total, sp, &lo, &hi);

  RowState<D, NB> w;
  int row_lim[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int rr = 16 * b + col, r = r0 + (rr < live_rows ? rr : 0);   // rows past the last repeat the first
    const int j = r / g.G, head = kvh * g.G + r % g.G;
    row_lim[b] = (int)visible_limit(a, j);
    load_row<D, NB>(w, b, (const float*)a.Qq + (((int64_t)beta * a.q_len + j) * g.Hq + head) * D, j4);
  }
  const int wave_lim = (int)visible_limit(a, r0 / g.G);

  // rows below cache_len are cached and visible to every token; the rest are the
  // call's own tokens, read where the caller left them (or from the caches, if a
  // preceding kernel has put them there)
  const int64_t cache0 = ((int64_t)beta * g.Hkv + kvh) * g.cap * D;
  const bool fused_append = a.Kn != nullptr;
  KeySeq seq;
  const float* Kb = (const float*)a.Kc + cache0;
  const float* Vb = (const float*)a.Vc + cache0;
  seq.Ka = (GlobalBytes)Kb; seq.Va = (GlobalBytes)Vb; seq.a_stride = 4 * D;
  seq.a_lo = (int)lo;
  seq.a_hi = (int)(hi < cache_len ? hi : cache_len);
  if (seq.a_hi < seq.a_lo) seq.a_hi = seq.a_lo;
  seq.l_lo = lo > cache_len ? (int)lo : cache_len;
  seq.l_hi = (int)hi;
  if (seq.l_hi < seq.l_lo) seq.l_hi = seq.l_lo;
  const int64_t new0 = ((int64_t)beta * a.q_len * g.Hkv + kvh) * D;
  const float* Kl = fused_append ? (const float*)a.Kn + new0 : Kb;
  const float* Vl = fused_append ? (const float*)a.Vn + new0 : Vb;
  seq.Kl = (GlobalBytes)Kl; seq.Vl = (GlobalBytes)Vl;
  seq.l_stride = (unsigned)(fused_append ? g.Hkv * D : D) * 4;
  seq.l_off = fused_append ? cache_len : 0;
  seq.count();
  attend<D, NB>(w, seq, wave, KW, row_lim, wave_lim, g.scale * LOG2E, lane);

  const bool direct = a.O != nullptr || a.A != nullptr;      // one split: nothing to merge
  meet<D, NB, KW>(w, x,
      [&](int row, int c, f32x4 v) {
        if (row >= live_rows) return;
        const int r = r0 + row, j = r / g.G, head = kvh * g.G + r % g.G;
        float* dst = a.O ? (float*)a.O + (((int64_t)beta * a.q_len + j) * g.Hq + head) * D
                   : a.A ? a.A + (((int64_t)beta * g.Hq + head) * a.q_len + j) * D
                         : a.O_sub + ((((int64_t)beta * a.plan.s_total + sp) * g.Hq + head) * a.q_len + j) * D;
        *(f32x4*)(dst + c) = v;
      },
      [&](int row, float lse) {
        if (row >= live_rows) return;
        const int r = r0 + row, j = r / g.G, head = kvh * g.G + r % g.G;
        if (!direct) a.LSE_sub[(((int64_t)beta * a.plan.s_total + sp) * g.Hq + head) * a.q_len + j] = lse;
        else if (a.LSE) a.LSE[((int64_t)beta * g.Hq + head) * a.q_len + j] = lse;
      });

  // Algorithm 2, append: the split that holds a new token files its row, its row tiles
  // in turn (as in phase2_rows_bf16_kernel)
  const int filers = row_tiles < 64 ? row_tiles : 64;
  if (fused_append && tile < filers && seq.l_hi > seq.l_lo) {
    const int64_t stride = (int64_t)g.Hkv * D, src = (int64_t)(seq.l_lo - cache_len) * stride;
    file_rows<D>(Kl + src, Vl + src, stride, (float*)a.Kc + cache0 + (int64_t)seq.l_lo * D,
                 (float*)a.Vc + cache0 + (int64_t)seq.l_lo * D, seq.l_hi - seq.l_lo,
                 tile * 64 * KW + threadIdx.x, filers * 64 * KW);
  }
}

template <int D, int NB, int KW>
hipError_t launch_phase1(const Phase1Args& a, hipStream_t st) {
  const Geom& g = a.g;
  const int64_t n = (g.L + g.b - 1) / g.b, bmax = g.b < g.L ? g.b : g.L;
  const int64_t tpb = (bmax * g.G + 16 * NB - 1) / (16 * NB), wgs = n * tpb * g.B * g.Hkv;
  // (a block of 2^31 rows would be 550 GB of queries)
  if (wgs > 0x7fffffff || bmax * g.G > 0x7fffffff - 64) return hipErrorInvalidValue;
  // All blocks in one group where the tiles start at once (two workgroups per CU and more), so that
  // heavy and light ones share CUs, else block by block: with several rounds of them a group of
  // few blocks leaves the XCDs that get the light blocks idle.  us, in one group / block by
  // block, 8 / 2 heads, blocks of L / 4, b = a: d = 128: L = 1024 (512 tiles) 24.2 / 26.5, 2048 (1024) 79 / 70,
  // 4099 (1032) 256 / 209, 8192 (2048) 813 / 705; d = 64: 4099 135 / 118, 6000 (1504) 246 / 216.
  // Over 350 drawn shapes, time lost against the better of the two: to 512 tiles 0.9 % and 1.1 %, from
  // 513 to 1536 4.4 % and 3.4 %, beyond 3.8 % and 3.4 %.
  const int64_t group = wgs <= 512 ? n : 1;
  return launch_in_pieces(wgs, 64 * KW, [&](unsigned first, unsigned n_wgs) {
    phase1_f32_kernel<D, NB, KW><<<dim3(n_wgs), 64 * KW, 0, st>>>(a, (int)group, (int)tpb, (int)first);
  });
}

template <int D, int NB, int KW>
hipError_t launch_phase2(const Phase2Args& a, hipStream_t st) {
  const Geom& g = a.g;
  const int64_t tiles = ((int64_t)g.G * a.q_len + 16 * NB - 1) / (16 * NB);
  const int64_t wgs = tiles * g.B * g.Hkv * a.plan.s_total;
  if (wgs > 0x7fffffff || (int64_t)g.G * a.q_len > 0x7fffffff - 64) return hipErrorInvalidValue;
  return launch_in_pieces(wgs, 64 * KW, [&](unsigned first, unsigned n_wgs) {
    phase2_f32_kernel<D, NB, KW><<<dim3(n_wgs), 64 * KW, 0, st>>>(a, (int)tiles, (int)first);
  });
}

}  // namespace

// 32-row tiles shared by four wavefronts (two workgroups per CU) once there are four such
// tiles per CU; down to one 16-row tile per CU, 16-row tiles shared by four (three per CU);
// fewer rows than that are bound by the latency of a tile: eight wavefronts share it.
// Measured (32 x 4 / 16 x 4 / 16 x 8, us; 8 / 2 heads except the last): d = 128: L = 8192
// (2048 32-row tiles) 705 / 740 / 819, L = 4099 (1025) 151 / 156 / 193, L = 1024 (256)
// 26.3 / 23.7 / 29.2; d = 64: L = 8192 369 / 375 / 395, L = 2048 (512) 39.0 / 37.3 / 39.4;
// 1 head, d = 64, L = 1024 (32) 16.0 / 10.0 / 9.9.
// Blocks of at most two units of keys have nothing to share: one wavefront per tile.  Against
// the set-up above (and one thread per row), us, 8 / 8 heads: d = 64, 100000 tokens: b = 1, a = 0
// 4790 -> 975 (3336), b = 4, a = 0 1245 -> 274 (1000), b = 4, a = 4 1379 -> 368 (1495); 50000 tokens,
// d = 128: b = a = 16 474 -> 251 (2262); three units and more: 146 -> 144 (b = 32, a = 0), 165 -> 169 (64).
Phase1Plan phase1_plan_f32(const Geom& g) {
  const int64_t bmax = g.b < g.L ? g.b : g.L, n = (g.L + g.b - 1) / g.b, rows = g.L * g.G * g.Hkv * g.B;
  Phase1Plan p = {0, 16, 8, 0, 0};
  if ((g.a + UNIT - 1) / UNIT + (bmax + UNIT - 1) / UNIT <= 2) p.waves = 1;
  else if (rows >= 1024 * 32) { p.rows = 32; p.waves = 4; }
  else if (rows >= 256 * 16) p.waves = 4;
  p.tiles = n * ((bmax * g.G + p.rows - 1) / p.rows) * g.B * g.Hkv;
  return p;
}

hipError_t launch_phase1_f32(const Phase1Args& a, hipStream_t st) {
  const Phase1Plan p = phase1_plan_f32(a.g);
  if (p.waves == 1) return a.g.d == 64 ? launch_phase1<64, 1, 1>(a, st) : launch_phase1<128, 1, 1>(a, st);
  if (p.rows == 32) return a.g.d == 64 ? launch_phase1<64, 2, 4>(a, st) : launch_phase1<128, 2, 4>(a, st);
  if (p.waves == 4) return a.g.d == 64 ? launch_phase1<64, 1, 4>(a, st) : launch_phase1<128, 1, 4>(a, st);
  return a.g.d == 64 ? launch_phase1<64, 1, 8>(a, st) : launch_phase1<128, 1, 8>(a, st);
}

// Per-part outputs over short blocks make splits of at most four units: one wavefront per
// 32-row tile.  Against four (and one thread per row), us: 114 tokens on 54 keys in blocks of
// 2, three sequences of 120 / 6 heads 418 -> 277 (373), 395 on 600 in blocks of 40, 7 heads
// 58.8 -> 52.1 (91.6); splits of 128 keys and more lose by it (1000 on 1000 53.8 -> 59.3).
hipError_t launch_phase2_f32(const Phase2Args& a, hipStream_t st) {
  if (a.plan.tile_rows == 32 && !a.plan.flat && a.plan.split_len <= 4 * UNIT)
    return a.g.d == 64 ? launch_phase2<64, 2, 1>(a, st) : launch_phase2<128, 2, 1>(a, st);
  if (a.plan.tile_rows == 32) return a.g.d == 64 ? launch_phase2<64, 2, 4>(a, st) : launch_phase2<128, 2, 4>(a, st);
  return a.g.d == 64 ? launch_phase2<64, 1, 8>(a, st) : launch_phase2<128, 1, 8>(a, st);
}

}  // namespace star
