// fp32 path (head_dim 64 or 128): row-tiled attention, fp32 storage, sums and softmax throughout and products good to 24 bits, so
// the result stays within 1e-5 of an fp64 evaluation at the sizes this path is meant for.  Tiles of 16 rows take their products on the
// fp32 matrix instructions, tiles of 32 rows in parts on the bf16 ones ("split products" below), but on short key ranges.
//
// What bounds it: the fp32 MFMA rate (157 TFLOP/s, 32 cycles for the 2048 flops of
// v_mfma_f32_16x16x4_f32) for long key ranges of 16-row tiles, latency for short ones.  Both are
// served by the same split:
//   * A workgroup owns a tile of 16 NB query rows of one KV group, and its KW
//     wavefronts share the tile's KEYS: wavefront w takes the 16-key units
//     w, w + KW, ...  Nothing crosses wavefronts until the end, so there is no
//     barrier in the key loop (LDS only for a wavefront's own K), and a tile of few rows
//     still has KW wavefronts' worth of loads and MFMAs in flight.
//   * Rows are packed over the heads of a KV group (row = token * G + head in
//     group), so that a K/V unit is read once for all of them.
//   * S^T = K Q^T: lane (col = lane % 16, j4 = lane / 16) supplies K[col][16 t + 4 j4 + e]
//     from a 16-byte global load, or from LDS (any assignment of d to (MFMA step, lane
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
// Measured, whole calls, against a kernel of one thread per row and fp32 products throughout: 8 / 2 heads, d = 128,
// L = 4099, b = 1024, a = 512: 3390 -> 134 -> 102.5 us (147 TFLOP/s; 174 at 8192 tokens in blocks of 2048, 129 with fp32 products;
// a library fp32 matrix product reaches 152); 1 head, d = 64, L = 1024, b = a = 256: 274 -> 9.2 -> 7.6 us.
#include "star_internal.h"

namespace star {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

typedef const __attribute__((address_space(1))) char* GlobalBytes;
typedef const __attribute__((address_space(1))) f32x4* GlobalVec;

constexpr int UNIT = 16;   // keys per step of a wavefront
// How a kernel takes its products: in fp32 from K as it is loaded, in fp32 from K turned through LDS, in bf16 parts.
enum { PLAIN, TURNED, SPLIT };
// How far (log2 units) a score may rise above its row's reference before the reference moves.
// O / l does not depend on the reference.  Scores of N(0, 1) inputs stay within it of the first unit's, and a
// unit then costs no exchange between lanes and no rescaling of O.  Against moving it to every new maximum, us
// (8 / 2 heads): d = 128: L = 4099 (b = 1024, a = 512) 140.3 -> 134.1, 8192 (b = a = 2048) 704 -> 673; d = 64: 4099
// (b = a = 1024) 103.1 -> 99.8; 1 head, 1024 10.2 -> 9.9.
// The weights in O are held 2^-HEADROOM as large, so that none is above one and sums of V overflow no earlier than
// with the maximum itself as reference (products with V below 1e-35 go denormal 8 bits earlier).  Without that
// sums of |V| beyond 1e36 could overflow; it costs, us, without / with: the three prefills 131.8 / 134.3, 664 / 666 and 95.9 /
// 98.3, d = 64, 8192 353 / 353, 1 head, 1024 9.1 / 9.2.
constexpr float HEADROOM = 8.f, HELD = 1.f / 256;
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
  int n_a, n_units;            // in units of KEYS keys
  template <int KEYS>
  __device__ __forceinline__ void count() {
    n_a = (a_hi - a_lo + KEYS - 1) / KEYS;
    n_units = n_a + (l_hi - l_lo + KEYS - 1) / KEYS;
  }
};

// The columns of d a workgroup computes: one of P pieces, H times 16 E of them (E adjacent ones a lane).
template <int D, int P>
struct Piece {
  static constexpr int C = D / P, E = C < 64 ? C / 16 : 4, H = C / (16 * E);
  typedef __attribute__((ext_vector_type(E))) float vec;
  typedef const __attribute__((address_space(1))) vec* Vec;
};

// A wavefront's state.  Lane (col, j4) belongs to row col of each of NB 16-row blocks.
template <int D, int NB, int P = 1>
struct RowState {
  typedef Piece<D, P> Cols;
  f32x4 q[NB][D / 16];        // q[.][t][e] = Q[row][16 t + 4 j4 + e] * scale * log2(e)
  f32x4 o[NB][Cols::H][Cols::E];      // o[.][h][e][w] = HELD O[row][E (16 h + 4 j4 + w) + e] of the piece
  float m[NB], top[NB];       // reference (log2 units; uniform over a row's four lanes; 0 until a key is
                              // visible) and the score beyond which it moves (-inf until then)
  float l[NB];                // this lane's share of the sum of 2^(s - m)
};

template <int D, int P = 1>
struct Unit {
  f32x4 k[D / 16];
  typename Piece<D, P>::vec v[4][Piece<D, P>::H];
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
template <int KEYS>
__device__ __forceinline__ UnitAt unit_at(const KeySeq& seq, int u) {
  // the four bases as scalars of their own: chosen between as struct members, the
  // compiler would keep the struct in scratch memory and index it
  GlobalBytes Ka = seq.Ka, Va = seq.Va, Kl = seq.Kl, Vl = seq.Vl;
  asm("" : "+s"(Ka), "+s"(Va), "+s"(Kl), "+s"(Vl));
  UnitAt x;
  x.local = u >= seq.n_a;
  x.key0 = x.local ? seq.l_lo + (u - seq.n_a) * KEYS : seq.a_lo + u * KEYS;
  x.n_rows = (x.local ? seq.l_hi : seq.a_hi) - x.key0;
  x.stride = x.local ? seq.l_stride : seq.a_stride;
  const size_t off = (size_t)(x.local ? x.key0 - seq.l_off : x.key0) * x.stride;
  x.K = (x.local ? Kl : Ka) + off;
  x.V = (x.local ? Vl : Va) + off;
  return x;
}

// Rows past the range's end re-read its last row (their scores are masked).
// A matrix operand has a lane per key, and four neighbouring lanes that read from four rows take four times as long as four that read
// 64 bytes of one.  Where few wavefronts or short ranges leave nothing to hide that (TURN; the launches say where), K is loaded four
// lanes to a row and turned through LDS (turn_k(), a wavefront's own 16 rows: no barrier).
template <int D, bool TURN, int P>
__device__ __forceinline__ void load_k(Unit<D, P>& r, const UnitAt& x, int lane) {
  int i = TURN ? (lane >> 4) + (lane & 12) : lane & 15;
  if (x.n_rows < UNIT) i = i < x.n_rows ? i : x.n_rows - 1;
  const unsigned off = (unsigned)i * x.stride + 16 * (TURN ? lane & 3 : lane >> 4);
#pragma unroll
  for (int t = 0; t < D / 16; ++t) r.k[t] = *(GlobalVec)(x.K + off + 64 * t);
}
// Chunk c (16 bytes) of row i sits in slot c ^ i of its row (low four bits): neither the 16 lanes of a write, four rows that differ
// in their upper bits, nor those of a read meet in a bank.
template <int D, int P>
__device__ __forceinline__ void turn_k(Unit<D, P>& r, f32x4* rows, int lane) {
  const int i = (lane >> 4) + (lane & 12), p = lane & 3, col = lane & 15, j4 = lane >> 4;
#pragma unroll
  for (int t = 0; t < D / 16; ++t) rows[i * (D / 4) + ((4 * t + p) ^ i)] = r.k[t];
#pragma unroll
  for (int t = 0; t < D / 16; ++t) r.k[t] = rows[col * (D / 4) + ((4 * t + j4) ^ col)];
}
template <int D, int P>
__device__ __forceinline__ void load_v(Unit<D, P>& r, const UnitAt& x, int lane) {
  typedef Piece<D, P> Cols;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    int i = 4 * (lane >> 4) + v;
    if (x.n_rows < UNIT) i = i < x.n_rows ? i : x.n_rows - 1;
    const unsigned off = (unsigned)i * x.stride + 4 * Cols::E * (lane & 15);
#pragma unroll
    for (int h = 0; h < Cols::H; ++h) r.v[v][h] = *(typename Cols::Vec)(x.V + off + 64 * Cols::E * h);
  }
}

// Moves the references that a score of the unit leaves; t: the lane's largest.
template <int D, int NB, int P>
__device__ __forceinline__ void move_references(RowState<D, NB, P>& w, const float (&t)[NB]) {
  bool beyond = false;
#pragma unroll
  for (int b = 0; b < NB; ++b) beyond |= t[b] > w.top[b];
  if (__builtin_amdgcn_ballot_w64(beyond) == 0) return;
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
    for (int h = 0; h < Piece<D, P>::H; ++h)
#pragma unroll
      for (int e = 0; e < Piece<D, P>::E; ++e) w.o[b][h][e] *= alpha;
  }
}

// One unit: scores, softmax, products.  MORE: K and V of unit `nxt` are requested as soon
// as this unit's are used up -- without a branch, so that the compiler's waits for V
// need not include them.
template <int D, int NB, bool MORE, bool TURN, int P>
__device__ __forceinline__ void attend_unit(RowState<D, NB, P>& w, Unit<D, P>& r, f32x4* rows, const UnitAt& cur, const UnitAt& nxt,
                                            const int (&row_lim)[NB], int wave_lim, int lane) {
  const int j4 = lane >> 4;
  if (TURN) turn_k<D, P>(r, rows, lane);
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
  if (MORE) load_k<D, TURN, P>(r, nxt, lane);
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
#pragma unroll
  for (int b = 0; b < NB; ++b) t[b] = fmaxf(fmaxf(s[b][0], s[b][1]), fmaxf(s[b][2], s[b][3]));
  move_references<D, NB, P>(w, t);
#pragma unroll
  for (int b = 0; b < NB; ++b) {
#pragma unroll
    for (int v = 0; v < 4; ++v) s[b][v] = __builtin_amdgcn_exp2f(s[b][v] - w.m[b]);
    w.l[b] += (s[b][0] + s[b][1]) + (s[b][2] + s[b][3]);
#pragma unroll
    for (int v = 0; v < 4; ++v) s[b][v] *= HELD;
  }
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int h = 0; h < Piece<D, P>::H; ++h)
#pragma unroll
      for (int e = 0; e < Piece<D, P>::E; ++e)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          w.o[b][h][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(r.v[v][h][e], s[b][v], w.o[b][h][e], 0, 0, 0);
  if (MORE) load_v<D, P>(r, nxt, lane);
}

// The lane's query row of row block b, as it is in memory (scale_rows() follows once the
// first keys have been requested, so that both round trips overlap).
template <int D, int NB, int P>
__device__ __forceinline__ void load_row(RowState<D, NB, P>& w, int b, const float* q, int j4) {
#pragma unroll
  for (int t = 0; t < D / 16; ++t) w.q[b][t] = *(const f32x4*)(q + 16 * t + 4 * j4);
#pragma unroll
  for (int h = 0; h < Piece<D, P>::H; ++h)
#pragma unroll
    for (int e = 0; e < Piece<D, P>::E; ++e) w.o[b][h][e] = f32x4{0.f, 0.f, 0.f, 0.f};
  w.m[b] = 0.f;
  w.top[b] = -INFINITY;
  w.l[b] = 0.f;
}
template <int D, int NB, int P>
__device__ __forceinline__ void scale_rows(RowState<D, NB, P>& w, float qk_scale) {
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int t = 0; t < D / 16; ++t) w.q[b][t] *= qk_scale;
}

// Attend the wavefront's rows to units first, first + step, ... of the sequence.
//   row_lim   this lane's exclusive bound on keys of the second range, per row block
//   wave_lim  smallest bound of the wavefront's live rows
template <int D, int NB, bool TURN, int P>
__device__ __forceinline__ void attend(RowState<D, NB, P>& w, f32x4* rows, const KeySeq& seq, int first, int step,
                                       const int (&row_lim)[NB], int wave_lim, float qk_scale, int lane) {
  if (first >= seq.n_units) return;
  Unit<D, P> r;
  UnitAt cur = unit_at<UNIT>(seq, first);
  load_k<D, TURN, P>(r, cur, lane);
  load_v<D, P>(r, cur, lane);
  scale_rows<D, NB, P>(w, qk_scale);
  for (int u = first + step; u < seq.n_units; u += step) {
    const UnitAt nxt = unit_at<UNIT>(seq, u);
    attend_unit<D, NB, true, TURN, P>(w, r, rows, cur, nxt, row_lim, wave_lim, lane);
    cur = nxt;
  }
  attend_unit<D, NB, false, TURN, P>(w, r, rows, cur, cur, row_lim, wave_lim, lane);
}

// ------------------------------------------------------------------ split products
// 32-row tiles take both products on the bf16 matrix instructions, which do sixteen times the work: an fp32 number is three bf16
// parts of 8 bits, x = h + m + l, and a product the sum of the six products of parts that reach its 24 bits (what is left out is
// below 2^-24 of it), summed in fp32, 32 products at a time where an fp32 instruction adds four.  Error against 64 bits, rms over 16 seeds,
// fp32 products / split: prefill, 8 / 2 heads, 4099 tokens: d = 128 2.75 / 1.84e-7 (log-sum-exp 1.79 / 1.57e-7), d = 64 2.79 / 2.08e-7
// (1.81 / 1.80e-7); 100 tokens on 4000 keys 1.78 / 1.58e-7.  With queries 4 to 16 times as large, split over fp32 products (2099 tokens):
// d = 128 0.78 to 0.80 (log-sum-exp 0.83 to 0.87), d = 64 0.84 to 0.88 (0.91 to 0.93).
// What bounds this loop is the sum of 192 MFMAs (3072 cycles) and 640 VALU instructions per 32 keys and 32 rows, two thirds of them
// to split K and V (a dot product and an MFMA do not overlap; split with shifts and subtractions, which do, they are 960, and the
// prefill above takes 114 us); with one row block to a wavefront (16-row tiles) that outweighs what the MFMAs save.  Tiles whose
// wavefronts share the split of K and V through LDS, two barriers per 32 keys, took 116 to 126 us.
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
constexpr int SPLIT_UNIT = 32;
// Which values they hold: a part is a multiple of 2^-133 (denormals are kept), so that a number of 2^-110 and more is the sum of its
// parts and a smaller one off by up to 2^-134, and from 3.39e38 on it is infinite.
//   * Weights are held 2^16 times as large, the smallest that exp2 gives (2^-126) then in full.  2^112 is what a row's sum of
//     weighted values may then come to.
//   * K is off by 2^-134: by 2^-39 in a score, if no query element is above 2^88.  Rows with one above that, or below 2^-110 and not
//     zero, are taken in fp32 products (held()).
//   * V is off by 2^-134: a wavefront's results below 2^-108 are taken again in fp32 products, as are those that are not finite, in
//     which an infinite part or sum shows (unsafe()).  (Values below 2^-134 count as zero.)
// The two checks and the weights' scale, 8 / 2 heads, d = 128, 4099 tokens: 103.2 -> 103.4 us.  What a second walk costs there, where
// fp32 products alone took 134 us: all V, or one column of it, below 3e-33, or sums above 5e33: 224; a NaN or an infinity in V, in half of
// the blocks 157, in the anchor 170; queries that are taken in fp32 products from the start 147.  8192 tokens (666): 1120, 650, 777 and
// 690; d = 64 (97.5): 177, 115, 134 and 107; 100 tokens on 16000 keys (69.6): 113, 83, 77 and 75.  One look at a part of the results behind a
// wavefront's first unit brings values that are small throughout to 160, and the ordinary call to 103.9: not kept.
constexpr float SPLIT_HELD = 0x1p16f, Q_MOST = 0x1p88f, Q_LEAST = 0x1p-110f, O_LEAST = 0x1p-108f;

struct Parts {                 // of eight elements
  u32x4 h, m, l;
};
__device__ __forceinline__ uint32_t rounded(float x, float y) { return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)x, (__bf16)y}); }
__device__ __forceinline__ float left(float x, uint32_t pair, uint32_t minus) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pair), __builtin_bit_cast(bf16x2, minus), x, false);
}
// Elements 2 i and 2 i + 1: the rounded pair and, by a product with (-1, 0) or (0, -1), what it leaves of each (exact).
__device__ __forceinline__ void split_pair(Parts& p, int i, float x, float y) {
  // (in registers: as a literal the second would be taken for the inline constant -1.0, which is another pair)
  uint32_t first = 0x0000bf80u, second = 0xbf800000u;
  asm("" : "+s"(first), "+s"(second));
  p.h[i] = rounded(x, y);
  x = left(x, p.h[i], first); y = left(y, p.h[i], second);
  p.m[i] = rounded(x, y);
  x = left(x, p.m[i], first); y = left(y, p.m[i], second);
  p.l[i] = rounded(x, y);
}
__device__ __forceinline__ f32x4 multiply(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// The query rows' parts: step t of the scores takes Q[row][32 t + 4 j4 .. +3] and Q[row][32 t + 16 + 4 j4 .. +3].  At d = 128 the two
// smaller ones are in LDS, for all wavefronts of the tile (they hold the same rows).
template <int D>
struct SharedRows {
  u32x4 m[2][D / 32][64], l[2][D / 32][64];
};
template <int D>
struct SplitRows {
  static constexpr bool SHARED = D == 128;
  u32x4 h[2][D / 32], m[2][SHARED ? 1 : D / 32], l[2][SHARED ? 1 : D / 32];
};

// Two 16-key pieces c of K, and V in pieces h of 64 columns.
template <int D>
struct SplitUnit {
  f32x4 k[2][D / 16];
  f32x4 v[D / 64][2][4];
};
template <int D>
__device__ __forceinline__ void load_k(SplitUnit<D>& r, const UnitAt& x, int c, int lane) {
  int i = 16 * c + (lane & 15);
  if (x.n_rows < SPLIT_UNIT) i = i < x.n_rows ? i : x.n_rows - 1;
  const unsigned off = (unsigned)i * x.stride + 16 * (lane >> 4);
#pragma unroll
  for (int t = 0; t < D / 16; ++t) r.k[c][t] = *(GlobalVec)(x.K + off + 64 * t);
}
template <int D>
__device__ __forceinline__ void load_v(SplitUnit<D>& r, const UnitAt& x, int h, int lane) {
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      int i = 16 * c + 4 * (lane >> 4) + v;
      if (x.n_rows < SPLIT_UNIT) i = i < x.n_rows ? i : x.n_rows - 1;
      r.v[h][c][v] = *(GlobalVec)(x.V + (unsigned)i * x.stride + 16 * (lane & 15) + 256 * h);
    }
}

// One unit, as attend_unit().  At d = 128 there are registers for half of K and of V: V is requested where K has been used up,
// and the next unit's K where V has; at d = 64 each a whole unit ahead.
template <int D, bool MORE>
__device__ __forceinline__ void attend_split_unit(RowState<D, 2>& w, const SplitRows<D>& q, const SharedRows<D>* shared, SplitUnit<D>& r,
                                                  const UnitAt& cur, const UnitAt& nxt, const int (&row_lim)[2], int wave_lim, int lane) {
  constexpr bool SHARED = SplitRows<D>::SHARED, LATE = D == 128;
  const int j4 = lane >> 4;
  f32x4 s[2][2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    // sums of their own for large and small products, and two of the large, which keeps the rounding of a large logit below the fp32
    // products' (the ratios above; with one at d = 128 0.94 to 0.98, the log-sum-exp 1.01, and 102.7 us where two take 102.9)
    f32x4 sum[2][2], small[2], least[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) sum[b][0] = sum[b][1] = small[b] = least[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < D / 32; ++t) {
      Parts k;
#pragma unroll
      for (int e = 0; e < 4; ++e) split_pair(k, e, r.k[c][2 * t + e / 2][2 * (e & 1)], r.k[c][2 * t + e / 2][2 * (e & 1) + 1]);
      u32x4 qm[2], ql[2];
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        qm[b] = SHARED ? shared->m[b][t][lane] : q.m[b][SHARED ? 0 : t];
        ql[b] = SHARED ? shared->l[b][t][lane] : q.l[b][SHARED ? 0 : t];
      }
#pragma unroll
      for (int b = 0; b < 2; ++b) sum[b][t % 2] = multiply(k.h, q.h[b][t], sum[b][t % 2]);
#pragma unroll
      for (int b = 0; b < 2; ++b) small[b] = multiply(k.m, q.h[b][t], small[b]);
#pragma unroll
      for (int b = 0; b < 2; ++b) least[b] = multiply(k.l, q.h[b][t], least[b]);
#pragma unroll
      for (int b = 0; b < 2; ++b) small[b] = multiply(k.h, qm[b], small[b]);
#pragma unroll
      for (int b = 0; b < 2; ++b) least[b] = multiply(k.m, qm[b], least[b]);
#pragma unroll
      for (int b = 0; b < 2; ++b) least[b] = multiply(k.h, ql[b], least[b]);
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) s[b][c] = (sum[b][0] + sum[b][1]) + (small[b] + least[b]);
    __builtin_amdgcn_sched_barrier(0);
    if (LATE) load_v<D>(r, cur, c, lane);
    else if (MORE) load_k<D>(r, nxt, c, lane);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (cur.n_rows < SPLIT_UNIT || (cur.local && cur.key0 + SPLIT_UNIT > wave_lim)) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int room = row_lim[b] - cur.key0;
      const int n = (cur.local && room < cur.n_rows ? room : cur.n_rows) - 4 * j4;
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) s[b][c][v] = 16 * c + v < n ? s[b][c][v] : -INFINITY;
    }
  }
  float top[2];
#pragma unroll
  for (int b = 0; b < 2; ++b)
    top[b] = fmaxf(fmaxf(fmaxf(s[b][0][0], s[b][0][1]), fmaxf(s[b][0][2], s[b][0][3])),
                   fmaxf(fmaxf(s[b][1][0], s[b][1][1]), fmaxf(s[b][1][2], s[b][1][3])));
  move_references<D, 2, 1>(w, top);
  Parts p[2];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) s[b][c][v] = __builtin_amdgcn_exp2f(s[b][c][v] - w.m[b]);
    w.l[b] += ((s[b][0][0] + s[b][0][1]) + (s[b][0][2] + s[b][0][3])) + ((s[b][1][0] + s[b][1][1]) + (s[b][1][2] + s[b][1][3]));
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      s[b][c] *= SPLIT_HELD;
      split_pair(p[b], 2 * c, s[b][c][0], s[b][c][1]);
      split_pair(p[b], 2 * c + 1, s[b][c][2], s[b][c][3]);
    }
  }
#pragma unroll
  for (int h = 0; h < D / 64; ++h) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      Parts v;
#pragma unroll
      for (int i = 0; i < 4; ++i) split_pair(v, i, r.v[h][i / 2][2 * (i & 1)][e], r.v[h][i / 2][2 * (i & 1) + 1][e]);
#pragma unroll
      for (int b = 0; b < 2; ++b) w.o[b][h][e] = multiply(v.l, p[b].h, w.o[b][h][e]);
#pragma unroll
      for (int b = 0; b < 2; ++b) w.o[b][h][e] = multiply(v.m, p[b].m, w.o[b][h][e]);
#pragma unroll
      for (int b = 0; b < 2; ++b) w.o[b][h][e] = multiply(v.h, p[b].l, w.o[b][h][e]);
#pragma unroll
      for (int b = 0; b < 2; ++b) w.o[b][h][e] = multiply(v.m, p[b].h, w.o[b][h][e]);
#pragma unroll
      for (int b = 0; b < 2; ++b) w.o[b][h][e] = multiply(v.h, p[b].m, w.o[b][h][e]);
#pragma unroll
      for (int b = 0; b < 2; ++b) w.o[b][h][e] = multiply(v.h, p[b].h, w.o[b][h][e]);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (MORE) {
      if (LATE) load_k<D>(r, nxt, h, lane);
      else load_v<D>(r, nxt, h, lane);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Whether the parts hold the wavefront's (scaled) queries.  (Zeros are told from other small ones only where there are any, here and below.)
template <int D>
__device__ __forceinline__ bool held(const RowState<D, 2>& w) {
  const auto outside = [&](bool zeros) {
    float most = 0.f, least = INFINITY;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int t = 0; t < D / 16; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float size = fabsf(w.q[b][t][e]);
          most = fmaxf(most, size);
          least = fminf(least, zeros && size == 0.f ? INFINITY : size);
        }
    return __builtin_amdgcn_ballot_w64(most > Q_MOST || least < Q_LEAST) != 0;
  };
  return !outside(false) || !outside(true);
}
// Whether they may have gone wrong.
template <int D>
__device__ __forceinline__ bool unsafe(const RowState<D, 2>& w) {
  const auto outside = [&](bool zeros) {
    bool any = false;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const float l = xor32_sum(w.l[b] + xor16(w.l[b]));
      float most = l, least = INFINITY;
#pragma unroll
      for (int h = 0; h < D / 64; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const float size = fabsf(w.o[b][h][e][v]);
            most = __builtin_elementwise_maximum(most, size);      // (NaN if any is)
            least = fminf(least, zeros && size == 0.f ? INFINITY : size);
          }
      any |= !(most < INFINITY) || least < O_LEAST * HELD * l;
    }
    return __builtin_amdgcn_ballot_w64(any) != 0;
  };
  return outside(false) && outside(true);
}

// As attend() for wavefront `wave` of KW, all of which call it (`w` holds the rows); `again()` loads the rows once more.
template <int D, int KW, typename Again>
__device__ __forceinline__ void attend_split(RowState<D, 2>& w, SharedRows<D>* shared, KeySeq& seq, int wave, const int (&row_lim)[2],
                                             int wave_lim, float qk_scale, int lane, Again again) {
  constexpr bool SHARED = SplitRows<D>::SHARED, LATE = D == 128;
  seq.count<SPLIT_UNIT>();
  const bool any = wave < seq.n_units;
  SplitUnit<D> r;
  UnitAt cur;
  if (any) {
    cur = unit_at<SPLIT_UNIT>(seq, wave);
#pragma unroll
    for (int c = 0; c < 2; ++c) load_k<D>(r, cur, c, lane);
    if (!LATE)
#pragma unroll
      for (int h = 0; h < D / 64; ++h) load_v<D>(r, cur, h, lane);
  }
  scale_rows<D, 2, 1>(w, qk_scale);
  const bool in_parts = held<D>(w);
  SplitRows<D> q;
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int t = 0; t < D / 32; ++t) {
      Parts x;
#pragma unroll
      for (int e = 0; e < 4; ++e) split_pair(x, e, w.q[b][2 * t + e / 2][2 * (e & 1)], w.q[b][2 * t + e / 2][2 * (e & 1) + 1]);
      q.h[b][t] = x.h;
      if (!SHARED) {
        q.m[b][SHARED ? 0 : t] = x.m;
        q.l[b][SHARED ? 0 : t] = x.l;
      } else if ((b * (D / 32) + t) % KW == wave) {
        shared->m[b][t][lane] = x.m;
        shared->l[b][t][lane] = x.l;
      }
    }
  if (SHARED) __syncthreads();
  if (!any) return;
  if (__builtin_expect(in_parts, 1)) {
    for (int u = wave + KW; u < seq.n_units; u += KW) {
      const UnitAt nxt = unit_at<SPLIT_UNIT>(seq, u);
      attend_split_unit<D, true>(w, q, shared, r, cur, nxt, row_lim, wave_lim, lane);
      cur = nxt;
    }
    attend_split_unit<D, false>(w, q, shared, r, cur, cur, row_lim, wave_lim, lane);
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int h = 0; h < D / 64; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) w.o[b][h][e] *= HELD / SPLIT_HELD;
    if (__builtin_expect(!unsafe<D>(w), 1)) return;
  }
  // the same keys in fp32 products, which take every value, as attend() takes them
  again();
  cur = unit_at<SPLIT_UNIT>(seq, wave);
  Unit<D> one;
  load_k<D, false, 1>(one, cur, lane);
  load_v<D, 1>(one, cur, lane);
  scale_rows<D, 2, 1>(w, qk_scale);
  for (int u = wave, half = 0;;) {
    UnitAt nxt = cur;
    half = half == 0 && cur.n_rows > UNIT;
    if (half) {
      nxt.K += (size_t)UNIT * cur.stride;
      nxt.V += (size_t)UNIT * cur.stride;
      nxt.key0 += UNIT;
      nxt.n_rows -= UNIT;
    } else {
      u += KW;
      if (u >= seq.n_units) break;
      nxt = unit_at<SPLIT_UNIT>(seq, u);
    }
    attend_unit<D, 2, true, false, 1>(w, one, nullptr, cur, nxt, row_lim, wave_lim, lane);
    cur = nxt;
  }
  attend_unit<D, 2, false, false, 1>(w, one, nullptr, cur, cur, row_lim, wave_lim, lane);
}

// log(l 2^m) for l > 0: the exponent of l joins m without a rounding lost, so that l may be a large sum
// (the reference m can lie HEADROOM below the row's maximum) or a small one.
__device__ __forceinline__ float log_sum(float m, float l) {
  const float e = (float)__builtin_amdgcn_frexp_expf(l), t = m + e, back = t - m, lost = (m - (t - back)) + (e - back);
  return fmaf(t, LN2, (log2f(__builtin_amdgcn_frexp_mantf(l)) + lost) * LN2);
}

template <bool A, typename X, typename Y> struct Either { typedef X type; };
template <typename X, typename Y> struct Either<false, X, Y> { typedef Y type; };
// LDS in which the KW wavefronts' results of a tile meet, 64 columns of d at a time.
// The pitch of 68 floats spreads the 16 rows of a 16-byte write over all banks.
template <int D, int NB, int KW, int HOW>
struct Meet {
  struct None {};
  union {
    // until the key loop ends:
    typename Either<HOW == SPLIT && D == 128, SharedRows<D>, None>::type rows;      // split products
    typename Either<HOW == TURNED, f32x4[KW][4 * D], None>::type k;          // turn_k()
    float o[KW][16 * NB][68];
  };
  float m[KW][16 * NB], l[KW][16 * NB];
  float scale[KW][16 * NB];
};

// Fold the wavefronts' partial results; `store(row, col, f32x4)` takes the normalised
// output of tile row `row`, columns col .. col + 3, and `store_lse(row, lse)` its
// natural-log denominator (-inf, output 0, for a row that saw no key).
template <int D, int NB, int KW, int HOW, int P, typename Store, typename StoreLse>
__device__ __forceinline__ void meet(RowState<D, NB, P>& w, Meet<D, NB, KW, HOW>& x, Store store, StoreLse store_lse) {
  constexpr int ROWS = 16 * NB, E = Piece<D, P>::E, H = Piece<D, P>::H;
  typedef typename Piece<D, P>::vec vec;
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
    x.scale[k][row] = l > 0.f ? __builtin_amdgcn_exp2f(x.m[k][row] - mm) * (1.f / l) * (1.f / HELD) : 0.f;
    if (k == 0) store_lse(row, l > 0.f ? log_sum(m, l) : -INFINITY);
  }
#pragma unroll
  for (int h = 0; h < H; ++h) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        vec v;
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = w.o[b][h][e][c];
        *(vec*)&x.o[wave][16 * b + col][E * (4 * j4 + c)] = v;
      }
    __syncthreads();
    for (int i = tid; i < ROWS * 4 * E; i += 64 * KW) {
      const int row = i / (4 * E), c = 4 * (i % (4 * E));
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < KW; ++k) acc += *(const f32x4*)&x.o[k][row][c] * x.scale[k][row];
      store(row, 16 * E * h + c, acc);
    }
    if (h + 1 < H) __syncthreads();
  }
}

// The key loop of wavefront `wave`.
template <int D, int NB, int KW, int HOW, int P, typename Again>
__device__ __forceinline__ void attend_rows(RowState<D, NB, P>& w, Meet<D, NB, KW, HOW>& x, KeySeq& seq, int wave, const int (&row_lim)[NB],
                                            int wave_lim, float qk_scale, int lane, Again again) {
  if constexpr (HOW == SPLIT) {
    attend_split<D, KW>(w, (SharedRows<D>*)&x.rows, seq, wave, row_lim, wave_lim, qk_scale, lane, again);
  } else {
    seq.count<UNIT>();
    attend<D, NB, HOW == TURNED, P>(w, (f32x4*)&x.k + wave * (4 * D), seq, wave, KW, row_lim, wave_lim, qk_scale, lane);
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
// Workgroups are numbered (kv head fastest, batch, tile), tiles in descending weight over all blocks.
// A workgroup goes to the XCD of its number mod 8 and there to the four shader engines
// strictly in turn, so numbers 32 apart share eight CUs, and none starts before those in front
// of it have: tiles of one weight next to each other keep all engines in step, whereas
// heavy tiles behind light ones, or numbers without a tile (a short last block's), leave engines idle.
// Against block by block, heavy tiles of each first, us (8 / 2 heads): d = 128: L = 4099 (b = 1024, a = 512) 142.4 ->
// 133.4, L = 3001 (b = 375, a = 93) 52.2 -> 46.5, 8192 (b = a = 2048) 662 -> 668; d = 64: 4099 (b = a = 1024) 107.5 ->
// 97.2; two sequences of 6000, 4 / 2 heads 125.5 -> 118.0; 300 workgroups and fewer the same.  Divisions by
// multiplication (struct Div) in place of the compiler's chains: another 1-2 us, 0.9 of 10 us at 1024 tokens of one head.
// Class c holds the tiles that walk c + 1 tiles' worth of keys: tile c - anchor_tiles of the
// blocks behind an anchor, tile c of a block without one (the first, unless there are no anchors or it
// has one too).  Runs of classes with the same number of tiles:
struct TileOrder {
  int first[4];        // first tile of the run
  int top[4];          // its highest class
  Div per[4];          // tiles per class
  int full[4];         // of which full-length blocks behind an anchor
  int last[4];         // 1: and the short last block
  int anchor_tiles, plain, n_blocks;      // plain: first block behind an anchor
  int turn_from, turn;                    // workgroups from the one on: turn - number
  Div Hkv, B, G;
};
struct Tile {
  int kvh, beta, i, t;                    // t: tile within block i
};
__device__ __forceinline__ Tile tile_at(const TileOrder& p, int wg) {
  uint32_t id = wg >= p.turn_from ? p.turn - wg : wg, q = quotient(id, p.Hkv);
  const int kvh = id - q * p.Hkv.d;
  id = q;
  q = quotient(id, p.B);
  const int beta = id - q * p.B.d;
  id = q;
  int first = p.first[0], top = p.top[0], full = p.full[0], last = p.last[0];
  Div per = p.per[0];
#pragma unroll
  for (int k = 1; k < 4; ++k) {
    // values of their own: chosen between as array elements, they would be put into scratch memory
    int f = p.first[k], c = p.top[k], n = p.full[k], l = p.last[k];
    Div x = p.per[k];
    asm("" : "+s"(f), "+s"(c), "+s"(n), "+s"(l), "+s"(x.d), "+s"(x.m), "+s"(x.s));
    if ((int)id >= f) { first = f; top = c; per = x; full = n; last = l; }
  }
  id -= first;
  q = quotient(id, per);
  const int c = top - (int)q, e = id - q * per.d;
  const bool anchored = e < full + last;
  const int i = e < full ? p.plain + e : anchored ? p.n_blocks - 1 : 0, t = anchored ? c - p.anchor_tiles : c;
  return {__builtin_amdgcn_readfirstlane(kvh), __builtin_amdgcn_readfirstlane(beta), __builtin_amdgcn_readfirstlane(i),
          __builtin_amdgcn_readfirstlane(t)};
}
template <int D, int NB, int KW, int HOW, int P>
__global__ __launch_bounds__(64 * KW, 2) void phase1_f32_kernel(Phase1Args a, TileOrder order, int first_wg) {
  __shared__ Meet<D, NB, KW, HOW> x;
  constexpr int ROWS = 16 * NB;
  const Geom& g = a.g;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, col = lane & 15, j4 = lane >> 4;
  const int wg = first_wg + (int)blockIdx.x, piece = wg % P;
  const Tile tile = tile_at(order, wg / P);
  const int kvh = tile.kvh, beta = tile.beta, i = tile.i, t = tile.t;
  const int s = (int)(i * g.b);
  const int e = (int)(s + g.b < g.L ? s + g.b : g.L);
  const int r0 = t * ROWS, n_rows = (e - s) * g.G;    // rows of this block
  const int live_rows = n_rows - r0 < ROWS ? n_rows - r0 : ROWS;
  const int row0_tok = (int)quotient(r0, order.G);
  const int tok0 = s + row0_tok, head0 = r0 - row0_tok * g.G;      // the tile's first row; row rr is rr rows on

  // K / V rows from the token-major inputs when they are handed over as they are
  // (then this kernel also files them in the caches), else from the filled caches
  const bool from_input = a.Kin != nullptr;
  const int64_t stride = from_input ? (int64_t)g.Hkv * D : D;      // floats between rows
  const int64_t in0 = ((int64_t)beta * g.L * g.Hkv + kvh) * D, cache0 = ((int64_t)beta * g.Hkv + kvh) * g.cap * D;
  const float* Kb = from_input ? (const float*)a.Kin + in0 : (const float*)a.Kc + cache0;
  const float* Vb = from_input ? (const float*)a.Vin + in0 : (const float*)a.Vc + cache0;

  RowState<D, NB, P> w;
  int row_lim[NB];
  const auto load_rows = [&]() {
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int rr = 16 * b + col;
      const unsigned r = head0 + (rr < live_rows ? rr : 0);     // rows past the block repeat the first
      const unsigned j = quotient(r, order.G);
      const int tok = tok0 + (int)j, head = kvh * g.G + (int)(r - j * g.G);
      row_lim[b] = tok + 1;
      load_row<D, NB, P>(w, b, (const float*)a.Q + (((int64_t)beta * g.L + tok) * g.Hq + head) * D, j4);
    }
  };
  load_rows();
  const int wave_lim = tok0 + 1;                      // the tile's first row sees least

  KeySeq seq;
  int64_t a_lo, a_hi;
  const bool ext = anchor_range(g, a.anchor_mode, i, &a_lo, &a_hi);
  seq.a_lo = (int)a_lo; seq.a_hi = (int)a_hi;
  // separately given anchors: token-major, n_anchor * a rows per batch
  const int64_t anchor_rows = (int64_t)(a.anchor_mode == ANCHOR_PER_BLOCK ? order.n_blocks : 1) * g.a;
  const int64_t anchor0 = ((int64_t)beta * anchor_rows * g.Hkv + kvh) * D;
  seq.Ka = (GlobalBytes)(ext ? (const float*)a.Ka + anchor0 : Kb);
  constexpr int C = Piece<D, P>::C;
  seq.Va = (GlobalBytes)((ext ? (const float*)a.Va + anchor0 : Vb) + piece * C);
  seq.a_stride = (unsigned)(ext ? (int64_t)g.Hkv * D : stride) * 4;
  seq.Kl = (GlobalBytes)Kb; seq.Vl = (GlobalBytes)(Vb + piece * C); seq.l_stride = (unsigned)stride * 4; seq.l_off = 0;
  seq.l_lo = s;
  seq.l_hi = tok0 + (int)quotient(head0 + live_rows - 1, order.G) + 1;
  attend_rows<D, NB, KW, HOW, P>(w, x, seq, wave, row_lim, wave_lim, g.scale * LOG2E, lane, load_rows);

  meet<D, NB, KW, HOW, P>(w, x,
      [&](int row, int c, f32x4 v) {
        if (row >= live_rows) return;
        const unsigned r = head0 + row, j = quotient(r, order.G);
        const int tok = tok0 + (int)j, head = kvh * g.G + (int)(r - j * g.G);
        *(f32x4*)((float*)a.O + (((int64_t)beta * g.L + tok) * g.Hq + head) * D + piece * C + c) = v;
      },
      [&](int row, float lse) {
        if (row >= live_rows || !a.LSE || piece != 0) return;
        const unsigned r = head0 + row, j = quotient(r, order.G);
        const int tok = tok0 + (int)j, head = kvh * g.G + (int)(r - j * g.G);
        a.LSE[((int64_t)beta * g.Hq + head) * g.L + tok] = lse;
      });

  // Algorithm 1, "keep the block's K/V": a token is filed by the tile that holds its first row
  if (from_input) {
    const int t0 = tok0 + (head0 > 0 ? 1 : 0), t1 = tok0 + (int)quotient(head0 + live_rows + g.G - 1, order.G);
    file_rows<D>(Kb + (int64_t)t0 * stride, Vb + (int64_t)t0 * stride, stride,
                 (float*)a.Kc + cache0 + (int64_t)t0 * D, (float*)a.Vc + cache0 + (int64_t)t0 * D, t1 - t0,
                 piece * 64 * KW + threadIdx.x, P * 64 * KW);
  }
}

// ------------------------------------------------------------------ phase 2
// What a launch is handed: packed under a flat plan, else as it is.
struct Call {
  Phase2Args a;
  RowGrid grid;
  int first_wg;
};
template <int ROWS>
__device__ __forceinline__ Call unpacked(const Call& c) { return c; }
template <int ROWS>
__device__ __forceinline__ Call unpacked(const FlatCall& c) {
  Call x;
  unpack(c, 0, &x.a);
  const Geom& g = x.a.g;
  x.grid = RowGrid{div_of(g.Hkv, c.m[0]), div_of(((unsigned)g.G * c.q_len + ROWS - 1) / ROWS, c.m[1]), div_of(c.s_total, c.m[2]), div_of(g.G, c.m[3])};
  x.first_wg = c.first_wg;
  return x;
}
template <int D, int NB, int KW, int HOW, int P, typename C>
__global__ __launch_bounds__(64 * KW, 2) void phase2_f32_kernel(C call) {
  __shared__ Meet<D, NB, KW, HOW> x;
  constexpr int ROWS = 16 * NB;
  const Call from = unpacked<ROWS>(call);
  const Phase2Args& a = from.a;
  const RowGrid& grid = from.grid;
  const int first_wg = from.first_wg;
  const Geom& g = a.g;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, col = lane & 15, j4 = lane >> 4;
  const uint32_t wg = first_wg + blockIdx.x, id = wg / P, of_head = quotient(id, grid.Hkv), of_tile = quotient(of_head, grid.tiles);
  const int kvh = id - of_head * grid.Hkv.d, tile = of_head - of_tile * grid.tiles.d, beta = quotient(of_tile, grid.splits);
  const int sp = of_tile - beta * grid.splits.d, row_tiles = grid.tiles.d;
  const int r0 = tile * ROWS, n_rows = g.G * a.q_len;  // row = token * G + head in group
  const int live_rows = n_rows - r0 < ROWS ? n_rows - r0 : ROWS;

  const int total = (int)visible_total(a), cache_len = (int)a.cache_len;
  int64_t lo, hi;
  split_range(a.plan, g.L, g.b, total, sp, &lo, &hi);

  const int piece = wg % P, first_d = piece * Piece<D, P>::C;      // (P > 1: calls of one split)
  RowState<D, NB, P> w;
  int row_lim[NB];
  const auto load_rows = [&]() {
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int rr = 16 * b + col, r = r0 + (rr < live_rows ? rr : 0);   // rows past the last repeat the first
      const int j = quotient(r, grid.G), head = kvh * g.G + r - j * g.G;
      row_lim[b] = (int)visible_limit(a, j);
      load_row<D, NB, P>(w, b, (const float*)a.Qq + (((int64_t)beta * a.q_len + j) * g.Hq + head) * D, j4);
    }
  };
  load_rows();
  const int wave_lim = (int)visible_limit(a, quotient(r0, grid.G));

  // rows below cache_len are cached and visible to every token; the rest are the
  // call's own tokens, read where the caller left them (or from the caches, if a
  // preceding kernel has put them there)
  const int64_t cache0 = ((int64_t)beta * g.Hkv + kvh) * g.cap * D;
  const bool fused_append = a.Kn != nullptr;
  KeySeq seq;
  const float* Kb = (const float*)a.Kc + cache0;
  const float* Vb = (const float*)a.Vc + cache0;
  seq.Ka = (GlobalBytes)Kb; seq.Va = (GlobalBytes)(Vb + first_d); seq.a_stride = 4 * D;
  seq.a_lo = (int)lo;
  seq.a_hi = (int)(hi < cache_len ? hi : cache_len);
  if (seq.a_hi < seq.a_lo) seq.a_hi = seq.a_lo;
  seq.l_lo = lo > cache_len ? (int)lo : cache_len;
  seq.l_hi = (int)hi;
  if (seq.l_hi < seq.l_lo) seq.l_hi = seq.l_lo;
  const int64_t new0 = ((int64_t)beta * a.q_len * g.Hkv + kvh) * D;
  const float* Kl = fused_append ? (const float*)a.Kn + new0 : Kb;
  const float* Vl = fused_append ? (const float*)a.Vn + new0 : Vb;
  seq.Kl = (GlobalBytes)Kl; seq.Vl = (GlobalBytes)(Vl + first_d);
  seq.l_stride = (unsigned)(fused_append ? g.Hkv * D : D) * 4;
  seq.l_off = fused_append ? cache_len : 0;
  attend_rows<D, NB, KW, HOW, P>(w, x, seq, wave, row_lim, wave_lim, g.scale * LOG2E, lane, load_rows);

  const bool direct = a.O != nullptr || a.A != nullptr;      // one split: nothing to merge
  meet<D, NB, KW, HOW, P>(w, x,
      [&](int row, int c, f32x4 v) {
        if (row >= live_rows) return;
        const int r = r0 + row, j = quotient(r, grid.G), head = kvh * g.G + r - j * g.G;
        float* dst = a.O ? (float*)a.O + (((int64_t)beta * a.q_len + j) * g.Hq + head) * D
                   : a.A ? a.A + (((int64_t)beta * g.Hq + head) * a.q_len + j) * D
                         : a.O_sub + ((((int64_t)beta * a.plan.s_total + sp) * g.Hq + head) * a.q_len + j) * D;
        *(f32x4*)(dst + first_d + c) = v;
      },
      [&](int row, float lse) {
        if (row >= live_rows || piece != 0) return;
        const int r = r0 + row, j = quotient(r, grid.G), head = kvh * g.G + r - j * g.G;
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
                 (tile * P + piece) * 64 * KW + threadIdx.x, filers * P * 64 * KW);
  }
}

// The order of a call's tiles of `rows` rows; returns their number (of one KV head and batch), or -1 if
// there are too many.
int64_t tile_order(const Phase1Args& a, int rows, TileOrder* o) {
  const Geom& g = a.g;
  const int64_t n = (g.L + g.b - 1) / g.b, bmax = g.b < g.L ? g.b : g.L;
  if (bmax * g.G > 0x7fffffff - 64) return -1;
  const bool alike = g.a == 0 || a.anchor_mode == ANCHOR_ALL_BLOCKS || n == 1;      // no first block by itself
  const int64_t per_block = (bmax * g.G + rows - 1) / rows, rest = g.L - (n - 1) * g.b;
  const int64_t of_last = n > 1 && rest < g.b ? (rest * g.G + rows - 1) / rows : 0;
  const int64_t most = 1 << 28, wide = (g.a * g.G + rows / 2) / rows, anchor = alike ? 0 : wide < most ? wide : most;
  const int64_t n_full = n - (alike ? 0 : 1) - (of_last > 0 ? 1 : 0);
  o->plain = alike ? 0 : 1; o->n_blocks = (int)n; o->anchor_tiles = (int)anchor;
  // between two of these classes the same blocks have a tile in each
  int64_t bound[5] = {anchor + per_block, anchor + of_last, alike ? 0 : per_block, anchor, 0}, tiles = 0;
  for (int i = 1; i < 5; ++i)
    for (int k = i; k > 0 && bound[k] > bound[k - 1]; --k) { const int64_t x = bound[k]; bound[k] = bound[k - 1]; bound[k - 1] = x; }
  for (int k = 0; k < 4; ++k) {
    const int64_t hi = bound[k], lo = bound[k + 1];
    o->full[k] = (int)(lo >= anchor ? n_full : 0);
    o->last[k] = lo >= anchor && hi <= anchor + of_last ? 1 : 0;
    const int64_t per = o->full[k] + o->last[k] + (!alike && hi <= per_block ? 1 : 0);
    o->per[k] = make_div((uint32_t)(per > 0 ? per : 1));
    o->top[k] = (int)(hi - 1);
    o->first[k] = per > 0 && hi > lo ? (int)tiles : 0x7fffffff;      // (a run of none is passed over)
    tiles += per * (hi - lo);
    if (tiles * g.B * g.Hkv > 0x7fffffff) return -1;
  }
  o->Hkv = make_div(g.Hkv); o->B = make_div(g.B); o->G = make_div(g.G);
  return tiles;
}

template <int D, int NB, int KW, int HOW, int P = 1>
hipError_t launch_phase1(const Phase1Args& a, hipStream_t st) {
  TileOrder o;
  const int64_t tiles = tile_order(a, 16 * NB, &o);
  if (tiles < 0) return hipErrorInvalidValue;
  const int64_t wgs = tiles * a.g.B * a.g.Hkv;
  // Where all tiles start at once, two to a CU at most, the lighter half comes in reverse, so that a CU
  // holds a heavy one and a light one: 8 / 2 heads, d = 128, L = 1024 (512 tiles) 23.6 -> 21.9 us.
  const int64_t cus = 256;
  o.turn_from = 0x7fffffff; o.turn = 0;
  if (wgs > cus && wgs <= 2 * cus) { o.turn_from = (int)cus; o.turn = (int)(cus + wgs - 1); }
  return launch_in_pieces(wgs * P, 64 * KW, [&](unsigned first, unsigned n_wgs) {
    phase1_f32_kernel<D, NB, KW, HOW, P><<<dim3(n_wgs), 64 * KW, 0, st>>>(a, o, (int)first);
  });
}

template <int D, int NB, int KW, int HOW, int P = 1>
hipError_t launch_phase2(const Phase2Args& a, hipStream_t st) {
  const Geom& g = a.g;
  const int64_t tiles = ((int64_t)g.G * a.q_len + 16 * NB - 1) / (16 * NB);
  const int64_t wgs = tiles * g.B * g.Hkv * a.plan.s_total;
  if (wgs > 0x7fffffff || (int64_t)g.G * a.q_len > 0x7fffffff - 64) return hipErrorInvalidValue;
  const RowGrid grid = {make_div(g.Hkv), make_div((uint32_t)tiles), make_div(a.plan.s_total), make_div(g.G)};
  if constexpr (KW > 1) {
    if (a.plan.flat) {
      FlatCall call = pack(a, grid);
      return launch_in_pieces(wgs * P, 64 * KW, [&](unsigned first, unsigned n_wgs) {
        call.first_wg = (int)first;
        phase2_f32_kernel<D, NB, KW, HOW, P, FlatCall><<<dim3(n_wgs), 64 * KW, 0, st>>>(call);
      });
    }
  }
  if constexpr (P == 1 && (KW != 4 || NB == 2)) {
    return launch_in_pieces(wgs, 64 * KW, [&](unsigned first, unsigned n_wgs) {
      phase2_f32_kernel<D, NB, KW, HOW, P, Call><<<dim3(n_wgs), 64 * KW, 0, st>>>(Call{a, grid, (int)first});
    });
  }
  return hipErrorInvalidValue;      // (flat plans only)
}

}  // namespace

// Workgroups that share a tile's columns of d read all of its query rows and store a part of each, in any order: one workgroup
// takes whole tiles, reading before it stores, where a call's results (`rows` rows of O or A and their LSE) lie over its queries.
static bool over_queries(const void* O, const void* LSE, const void* Q, int64_t rows, int d) {
  const size_t bytes = (size_t)rows * d * sizeof(float);
  return overlap(O, bytes, Q, bytes) || overlap(LSE, (size_t)rows * sizeof(float), Q, bytes);
}

// Blocks of at most two units of keys have nothing to share: one wavefront per tile.  Against the set-ups below (and one thread
// per row), us, 8 / 8 heads: d = 64, 100000 tokens: b = 1, a = 0 4790 -> 975 (3336), b = 4, a = 0 1245 -> 274 (1000), b = 4, a = 4
// 1379 -> 368 (1495); 50000 tokens, d = 128: b = a = 16 474 -> 251 (2262); three units and more: 146 -> 144 (b = 32, a = 0), 165 -> 169
// (64).
// 32-row tiles shared by four wavefronts (two workgroups per CU) from more than one such tile per CU on, if their rows see keys enough;
// down to one 16-row tile per CU, 16-row tiles shared by four (three per CU); fewer rows than that are bound by the latency of a tile:
// eight wavefronts share it, and where a tile and CUs for it are left over, two or four workgroups compute a half or a quarter of its
// columns of d each: every one takes all scores, but the products with V, the other half of a tile's MFMAs, are shared (one head, b = a = L / 4,
// us, whole tiles / halves / quarters: d = 64: L = 500 (32 tiles) 6.9 / 6.5 / 6.3, 1024 (64) 9.25 / 8.45 / 8.0, 1500 (96) 11.6 / 10.6
// / 14.1; d = 128: 500 11.8 / 9.7 / 9.1, 1000 16.3 / 13.5 / 13.4, 2000 (128) 25.2 / 22.0 / 33.8; sixteen wavefronts to a tile 11.3
// where eight take 9.25).  Eight wavefronts: one head, d = 64, L = 1024 (32) 10.0 (four) / 9.9, d = 64, 8 / 2 heads, 2048 37.3 / 39.4.
// What decides between the tiles is how many keys a row sees on average (`seen`; less by the square of the padding that 32 rows add to 16): a
// 32-row tile has the longer start (the parts of its queries) and end, and units of 32 keys for four wavefronts leave some idle on short ranges.
// 16-row tiles that all run at once (768, and some that start as the shortest end) are hard to beat; so is one round (512) of 32-row tiles that
// 16-row ones need two for.
// Below the lines 16-row tiles, but for more than 32768 rows of d = 64, which take 32-row tiles in fp32 products there.
// us, 16-row tiles / 32-row tiles in fp32 products / in split products, from 350 calls drawn over 4096 to 200000 rows and 33 to 5800 keys:
//   d = 128, up to 850 16-row tiles: seen 82 15.3 / 18.8 / 18.5, 114 16.8 / 20.6 / 18.7, 141 19.7 / - / 22.7, 185 22.0 / 25.9 / 22.4, 196 22.2 / 24.8 / 21.6, 209
//   23.4 / - / 26.5, 244 25.9 / 28.8 / 23.9, 1366 86.4 / 114.0 / 84.7 (of 8192 rows and fewer none, 917 40.4 / 65.8 / 52.3).  960 / 496 tiles: 108 23.5 /
//   - / 20.3.  More: 26 15.2 / 20.0 / 21.6, 73 23.2 / 26.2 / 24.7, 111 19.0 /
//   21.4 / 19.4, 115 26.2 / 28.9 / 27.3, 125 26.6 / 29.9 / 26.5, 136 21.7 / 23.3 / 21.5, 151 33.6 / 36.8 / 34.3, 214 35.9 / 36.4 / 31.8, 1154 87.5 / 86.0 / 65.0;
//   100000 rows: 38 111 / 131 / 143, 49 72 / 91 / 86, 100 71.3 / 79.8 / 74.6, 146 84.4 / 88.7 / 78.0, 227 162 / 136 / 126, 764 398 / 366 / 302.
//   d = 64, up to 768 16-row tiles: 356 18.4 / 20.0 / 18.9, 410 20.8 / 25.3 / 22.4, 680 26.8 / - / 24.8, 853 33.3 / 39.1 / 31.5.  Up to 512 32-row tiles: 109 11.3 / 12.1 / 12.6,
//   114 11.9 / 12.1 / 13.2, 234 17.4 / - / 16.4, 264 19.6 / 17.8 / 17.4.  More: 44 9.9 / 11.2 / 14.0, 154 16.9 / 17.9 / 17.2, 257 20.9 / 22.6 / 22.7, 328 26.2 /
//   28.2 / 24.1, 771 67.4 / 67.1 / 56.6.  More than 32768 rows: 163 85.8 / 70.2 / 79.4, 200 56.5 / 52.0 / 57.4, 344 46.2 / 45.2 / 45.9, 362 - /
//   84.1 / 79.7, 386 67.5 / 64.7 / 62.0, 802 192 / 183 / 161.
Phase1Plan phase1_plan_f32(const Geom& g) {
  const int64_t bmax = g.b < g.L ? g.b : g.L, rows = g.L * g.G * g.Hkv * g.B;
  const int64_t full = g.L / g.b, rest = g.L - full * g.b;      // (the short last block has fewer)
  const auto tiles = [&](int64_t r) { return (full * ((g.b * g.G + r - 1) / r) + (rest * g.G + r - 1) / r) * g.B * g.Hkv; };
  const int64_t t16 = tiles(16), t32 = tiles(32);
  const double pad = 2.0 * t32 / t16, seen = (double)(full * g.b * (g.b + 1) / 2 + rest * (rest + 1) / 2 + g.a * (g.L - bmax)) / g.L / (pad * pad);
  const double line = g.d == 128 ? t16 <= 850 ? 230 : t16 > 900 && t32 <= 512 ? 100 : 120 : t16 <= 768 ? 600 : t32 <= 512 ? 200 : 280;
  Phase1Plan p = {0, 16, 8, 0, 0, 0, 1};
  if ((g.a + UNIT - 1) / UNIT + (bmax + UNIT - 1) / UNIT <= 2) p.waves = 1;
  else if (rows > 256 * 32 && (seen >= line || (g.d == 64 && rows >= 1024 * 32))) {
    p.rows = 32; p.waves = 4;
    p.split = seen >= line;
  } else if (rows >= 256 * 16) p.waves = 4;
  p.tiles = tiles(p.rows);
  if (p.waves == 8) p.pieces = p.tiles <= 64 ? 4 : p.tiles <= 128 ? 2 : 1;
  return p;
}

hipError_t launch_phase1_f32(const Phase1Args& a, hipStream_t st) {
  const Phase1Plan p = phase1_plan_f32(a.g);
  if (p.waves == 1) return a.g.d == 64 ? launch_phase1<64, 1, 1, PLAIN>(a, st) : launch_phase1<128, 1, 1, PLAIN>(a, st);
  if (p.rows == 32 && a.g.d == 128) return launch_phase1<128, 2, 4, SPLIT>(a, st);
  if (p.rows == 32) return p.split ? launch_phase1<64, 2, 4, SPLIT>(a, st) : launch_phase1<64, 2, 4, PLAIN>(a, st);
  if (p.waves == 4) return a.g.d == 64 ? launch_phase1<64, 1, 4, PLAIN>(a, st) : launch_phase1<128, 1, 4, PLAIN>(a, st);
  // K is turned but for long ranges at d = 64 on more than 128 tiles and where four wavefronts share a tile.  us, as loaded / turned: one
  // head, b = a = L / 4: d = 64: 300 (quarters) 5.6 / 4.9, 1024 7.8 / 7.55, 2000 (halves) 12.8 / 12.0, 3000 (whole) 18.7 / 19.0, 4 / 2 heads,
  // 1000, b = 250 7.7 / 7.3; d = 128: 500 9.1 / 8.3, 1000 13.4 / 11.5, 4000 42.3 / 40.2; four wavefronts: one head, 4096, d = 64 26.3 / 29.7,
  // d = 128 28.0 / 30.3, 8 / 2 heads, 1024, d = 128 20.9 / 19.6.
  const int pieces = over_queries(a.O, a.LSE, a.Q, (int64_t)a.g.B * a.g.L * a.g.Hq, a.g.d) ? 1 : p.pieces;
  if (pieces == 4) return a.g.d == 64 ? launch_phase1<64, 1, 8, TURNED, 4>(a, st) : launch_phase1<128, 1, 8, TURNED, 4>(a, st);
  if (pieces == 2) return a.g.d == 64 ? launch_phase1<64, 1, 8, TURNED, 2>(a, st) : launch_phase1<128, 1, 8, TURNED, 2>(a, st);
  if (a.g.d == 128) return launch_phase1<128, 1, 8, TURNED>(a, st);
  return a.g.a + (a.g.b < a.g.L ? a.g.b : a.g.L) <= 512 ? launch_phase1<64, 1, 8, TURNED>(a, st) : launch_phase1<64, 1, 8, PLAIN>(a, st);
}

// Per-part outputs over short blocks make splits of at most four units: one wavefront per
// 32-row tile.  Against four (and one thread per row), us: 114 tokens on 54 keys in blocks of
// 2, three sequences of 120 / 6 heads 418 -> 277 (373), 395 on 600 in blocks of 40, 7 heads
// 58.8 -> 52.1 (91.6); splits of 128 keys and more lose by it (1000 on 1000 53.8 -> 59.3).
// 16-row tiles turn K (as in phase 1), us, as loaded / turned: 4000 keys (8 / 2 heads, d = 128) 8.5 / 8.3, 16000 11.8 / 11.5, 300 (one head, d = 64)
// 5.5 / 5.3, 50000 10.6 / 10.7, 33 tokens on 2000 13.6 / 12.7.
// Split products (as in phase 1), fp32 / split, us: d = 128: 100 tokens on 16000 keys (8 / 2 heads) 69.6 / 54.0, on 4000 31.1 / 26.5, 20 on
// 4000 15.0 / 14.8; d = 64: 100 on 16000 40.1 / 33.3 (runs of 864 keys), but 40 on 16000 20.7 / 21.3 (320), 20 on 16000 16.7 / 19.0 (192).
constexpr int SPLIT_RUN_64 = 512;       // longest splits that d = 64 takes in fp32 products in phase 2
hipError_t launch_phase2_f32(const Phase2Args& a, hipStream_t st) {
  if (a.plan.tile_rows == 32 && !a.plan.flat && a.plan.split_len <= 4 * UNIT)
    return a.g.d == 64 ? launch_phase2<64, 2, 1, PLAIN>(a, st) : launch_phase2<128, 2, 1, PLAIN>(a, st);
  if (a.plan.tile_rows == 32 && a.g.d == 128) return launch_phase2<128, 2, 4, SPLIT>(a, st);
  if (a.plan.tile_rows == 32) return a.plan.split_len > SPLIT_RUN_64 ? launch_phase2<64, 2, 4, SPLIT>(a, st) : launch_phase2<64, 2, 4, PLAIN>(a, st);
  if (a.plan.waves == 4) return a.g.d == 64 ? launch_phase2<64, 1, 4, TURNED>(a, st) : launch_phase2<128, 1, 4, TURNED>(a, st);
  // One split: few tiles share their columns of d, as in phase 1.  us, one token, one head: d = 64: 500 keys 8.7 -> 7.5, 250 6.3 -> 5.8;
  // d = 128: 250 10.6 -> 8.1; two sequences of 20 tokens on 200 (8 / 2 heads) 11.8 -> 9.4.
  if ((a.O || a.A) && !over_queries(a.O ? a.O : a.A, a.LSE, a.Qq, (int64_t)a.g.B * a.q_len * a.g.Hq, a.g.d)) {
    const int64_t tiles = (int64_t)a.g.B * a.g.Hkv * (((int64_t)a.g.G * a.q_len + 15) / 16);
    if (tiles <= 64) return a.g.d == 64 ? launch_phase2<64, 1, 8, TURNED, 4>(a, st) : launch_phase2<128, 1, 8, TURNED, 4>(a, st);
    if (tiles <= 128) return a.g.d == 64 ? launch_phase2<64, 1, 8, TURNED, 2>(a, st) : launch_phase2<128, 1, 8, TURNED, 2>(a, st);
  }
  return a.g.d == 64 ? launch_phase2<64, 1, 8, TURNED>(a, st) : launch_phase2<128, 1, 8, TURNED>(a, st);
}

}  // namespace star
