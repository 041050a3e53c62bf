// LSE merge (Eq. 3-4; Algorithm 2's running update): combines the per-split
// local attention outputs A_s and log-sum-exps lse_s of one query row into the
// global attention output,
//     lse = log sum_s exp(lse_s),   O = sum_s exp(lse_s - lse) A_s.
// Splits are first folded into their part (context block or tail) so that the
// per-part pair (A_m, lse_m) the paper's hosts would exchange can be written
// out; the parts are then folded in index order with the online-softmax update
//     lse' = logaddexp(lse, lse_m),  O' = exp(lse - lse') O + exp(lse_m - lse') A_m,
// which is what Eq. 3-4 evaluate to.  An empty split or part has lse = -inf and
// weight 0.  Under a flat split plan everything is one part.  The order of every
// fold is fixed, so results are deterministic.  The same kernel is the query
// host's aggregation of the pairs gathered from other hosts (Algorithm 2): the
// hosts' pairs are the splits of one part.  Besides the output in the storage
// dtype it can leave the merged pair itself, (A, lse) in fp32 -- what a host
// sends when its cache is one share of a larger one.
//
// Two sets of kernels:
//   * merge_flat_kernel / merge_flat_rows_kernel for calls of one part (a flat split plan,
//     pairs gathered from hosts), which is every call of a serving loop.  What bounds them
//     is latency: a decode step has few rows of 24 to 512 splits, so the rows are spread
//     over many workgroups (a piece of d each) and the weights of the splits in flight are
//     taken against their common maximum, with no chain from split to split.
//   * merge_kernel / merge_rows_kernel for calls with several parts: the per-part pairs are
//     written out on the way.  merge_kernel: one workgroup per (batch, head, row), 8 groups
//     of 32 lanes walk the splits of a part, each lane owning d/32 output elements and each
//     group folding its splits with a running maximum (4 in flight); the partial results
//     are combined through LDS.
// Traffic is s_total * (d + 1) floats per row -- negligible next to the cache.
//
// The fold over parts keeps a compensation term per accumulator (Kahan
// summation; 64-bit sums where all splits are folded at once): a context cut into hundreds of small blocks is hundreds of
// sequential additions, and in fp32 their rounding errors would otherwise add up
// to the 1e-5 the fp32 path is held to.
#include "rotary.h"

namespace star {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

// sum += x with the rounding error of the addition carried in `comp`
__device__ __forceinline__ void add_compensated(float& sum, float& comp, float x) {
  const float y = x - comp;
  const float t = sum + y;
  comp = (t - sum) - y;
  sum = t;
}

__device__ __forceinline__ unsigned short f32_to_bf16_rne(float f) {
  unsigned int u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x40u);  // NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}

template <int D, int GROUPS, int INFL>
__global__ __launch_bounds__(32 * GROUPS) void merge_kernel(MergeArgs a, unsigned first_wg) {
  constexpr int E = D / 32;                  // output elements per lane
  __shared__ float red_max[GROUPS];
  __shared__ float red_w[GROUPS];
  __shared__ float red_acc[GROUPS][D];
  const Geom& g = a.g;
  const int tid = threadIdx.x, grp = tid >> 5, li = tid & 31;
  int64_t row = first_wg + blockIdx.x;      // (beta, h, j), j fastest
  int j = (int)(row % a.q_len);
  int h = (int)((row / a.q_len) % g.Hq);
  int beta = (int)(row / ((int64_t)a.q_len * g.Hq));
  const SplitPlan& p = a.plan;
  const int64_t sub_stride = a.split_stride;                                 // rows between splits
  const int64_t base = (int64_t)beta * a.batch_stride + (int64_t)h * a.q_len + j;   // split 0
  const int n_parts = p.n_blocks + 1;

  float m_g = -INFINITY, l_g = 0.f, l_c = 0.f;
  float acc_g[E], acc_c[E];
#pragma unroll
  for (int e = 0; e < E; ++e) acc_g[e] = acc_c[e] = 0.f;

  for (int m = 0; m < n_parts; ++m) {
    int s_lo, s_hi;
    if (m < p.n_blocks) { s_lo = m * p.spb; s_hi = s_lo + p.spb; }
    else { s_lo = p.n_blocks * p.spb; s_hi = p.s_total; }

    // Each group folds its splits (s_lo + grp, + GROUPS, ...) with a running maximum;
    // LSE and output loads of a split are independent of the fold, so several
    // splits are in flight at once.
    float pm = -INFINITY, wsum = 0.f;
    float acc[E];
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = 0.f;
    for (int s0 = s_lo + grp; s0 < s_hi; s0 += INFL * GROUPS) {
      float ls[INFL];
      float v[INFL][E];
#pragma unroll
      for (int u = 0; u < INFL; ++u) {
        int s = s0 + u * GROUPS;
        ls[u] = -INFINITY;
        if (s < s_hi) {
          ls[u] = a.LSE_sub[base + s * sub_stride];
          const float* src = a.O_sub + (base + s * sub_stride) * D + li * E;
#pragma unroll
          for (int e = 0; e < E; ++e) v[u][e] = src[e];
        }
      }
#pragma unroll
      for (int u = 0; u < INFL; ++u) {
        if (ls[u] == -INFINITY) continue;        // empty split: weight 0, output unset
        float m_new = fmaxf(pm, ls[u]);
        float sc_old = expf(pm - m_new);         // 0 for the first non-empty split
        float w = expf(ls[u] - m_new);
        wsum = wsum * sc_old + w;
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] = acc[e] * sc_old + w * v[u][e];
        pm = m_new;
      }
    }
    // combine the groups: bring every group to the common maximum
    __syncthreads();                         // previous part's reads of red_* are done
    if (li == 0) red_max[grp] = pm;
    __syncthreads();
    float pmax = red_max[0];
#pragma unroll
    for (int k = 1; k < GROUPS; ++k) pmax = fmaxf(pmax, red_max[k]);
    float adj = pm > -INFINITY ? expf(pm - pmax) : 0.f;
    if (li == 0) red_w[grp] = wsum * adj;
#pragma unroll
    for (int e = 0; e < E; ++e) red_acc[grp][li * E + e] = acc[e] * adj;
    __syncthreads();
    pm = pmax;

    if (grp == 0) {
      float wtot = 0.f;
#pragma unroll
      for (int k = 0; k < GROUPS; ++k) wtot += red_w[k];
      float A_m[E];
      float lse_m = -INFINITY;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        float t = 0.f;
#pragma unroll
        for (int k = 0; k < GROUPS; ++k) t += red_acc[k][li * E + e];
        A_m[e] = wtot > 0.f ? t / wtot : 0.f;
      }
      if (wtot > 0.f) lse_m = pm + logf(wtot);
      if (a.O_part) {
        int64_t pr = (((int64_t)beta * n_parts + m) * g.Hq + h) * a.q_len + j;
#pragma unroll
        for (int e = 0; e < E; ++e) a.O_part[pr * D + li * E + e] = A_m[e];
        if (li == 0) a.LSE_part[pr] = lse_m;
      }
      if (lse_m > -INFINITY) {
        float m_new = fmaxf(m_g, lse_m);
        float sc_old = expf(m_g - m_new);     // 0 on the first non-empty part
        float sc_new = expf(lse_m - m_new);
        if (sc_old != 1.f) {                  // the maximum moved: rescale sums and compensations
#pragma unroll
          for (int e = 0; e < E; ++e) { acc_g[e] *= sc_old; acc_c[e] *= sc_old; }
          l_g *= sc_old;
          l_c *= sc_old;
        }
#pragma unroll
        for (int e = 0; e < E; ++e) add_compensated(acc_g[e], acc_c[e], sc_new * A_m[e]);
        add_compensated(l_g, l_c, sc_new);
        m_g = m_new;
      }
    }
  }
  if (grp == 0) {
    int64_t orow = ((int64_t)beta * a.q_len + j) * g.Hq + h;
    int64_t arow = ((int64_t)beta * g.Hq + h) * a.q_len + j;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      float out = l_g > 0.f ? acc_g[e] / l_g : 0.f;
      if (a.A) a.A[arow * D + li * E + e] = out;
      if (!a.O) continue;
      if (a.out_bf16) ((unsigned short*)a.O)[orow * D + li * E + e] = f32_to_bf16_rne(out);
      else ((float*)a.O)[orow * D + li * E + e] = out;
    }
    if (a.LSE && li == 0) a.LSE[arow] = l_g > 0.f ? m_g + logf(l_g) : -INFINITY;
  }
}

// The same merge for calls with many rows and few splits per part (query
// encoding: thousands of rows, one to a few splits per context block; a handful
// of gathered host pairs): 32 lanes own a row, eight rows share a workgroup, and
// nothing crosses lanes -- no LDS, no barriers.  A part's splits are folded in
// index order with INFL loads in flight, the parts in index order after them.
template <int D, int INFL>
__global__ __launch_bounds__(256) void merge_rows_kernel(MergeArgs a, int64_t n_rows, unsigned first_wg) {
  constexpr int E = D / 32;
  const Geom& g = a.g;
  const int li = threadIdx.x & 31;
  const int64_t row = (int64_t)(first_wg + blockIdx.x) * 8 + (threadIdx.x >> 5);      // (beta, h, j), j fastest
  if (row >= n_rows) return;
  const int j = (int)(row % a.q_len);
  const int h = (int)((row / a.q_len) % g.Hq);
  const int beta = (int)(row / ((int64_t)a.q_len * g.Hq));
  const SplitPlan& p = a.plan;
  const int64_t base = (int64_t)beta * a.batch_stride + (int64_t)h * a.q_len + j;
  const int n_parts = p.n_blocks + 1;

  float m_g = -INFINITY, l_g = 0.f, l_c = 0.f;
  float acc_g[E], acc_c[E];
#pragma unroll
  for (int e = 0; e < E; ++e) acc_g[e] = acc_c[e] = 0.f;
  for (int m = 0; m < n_parts; ++m) {
    int s_lo, s_hi;
    if (m < p.n_blocks) { s_lo = m * p.spb; s_hi = s_lo + p.spb; }
    else { s_lo = p.n_blocks * p.spb; s_hi = p.s_total; }
    float pm = -INFINITY, wsum = 0.f;
    float acc[E];
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = 0.f;
    for (int s0 = s_lo; s0 < s_hi; s0 += INFL) {
      float ls[INFL];
      float v[INFL][E];
#pragma unroll
      for (int u = 0; u < INFL; ++u) {
        const int s = s0 + u;
        ls[u] = -INFINITY;
        if (s < s_hi) {
          ls[u] = a.LSE_sub[base + s * a.split_stride];
          const float* src = a.O_sub + (base + s * a.split_stride) * D + li * E;
#pragma unroll
          for (int e = 0; e < E; ++e) v[u][e] = src[e];
        }
      }
#pragma unroll
      for (int u = 0; u < INFL; ++u) {
        if (ls[u] == -INFINITY) continue;        // empty split: weight 0, output unset
        float m_new = fmaxf(pm, ls[u]);
        float sc_old = expf(pm - m_new);         // 0 for the first non-empty split
        float w = expf(ls[u] - m_new);
        wsum = wsum * sc_old + w;
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] = acc[e] * sc_old + w * v[u][e];
        pm = m_new;
      }
    }
    float A_m[E];
#pragma unroll
    for (int e = 0; e < E; ++e) A_m[e] = wsum > 0.f ? acc[e] / wsum : 0.f;
    const float lse_m = wsum > 0.f ? pm + logf(wsum) : -INFINITY;
    if (a.O_part) {
      int64_t pr = (((int64_t)beta * n_parts + m) * g.Hq + h) * a.q_len + j;
#pragma unroll
      for (int e = 0; e < E; ++e) a.O_part[pr * D + li * E + e] = A_m[e];
      if (li == 0) a.LSE_part[pr] = lse_m;
    }
    if (lse_m > -INFINITY) {
      float m_new = fmaxf(m_g, lse_m);
      float sc_old = expf(m_g - m_new);          // 0 on the first non-empty part
      float sc_new = expf(lse_m - m_new);
      if (sc_old != 1.f) {                       // the maximum moved: rescale sums and compensations
#pragma unroll
        for (int e = 0; e < E; ++e) { acc_g[e] *= sc_old; acc_c[e] *= sc_old; }
        l_g *= sc_old;
        l_c *= sc_old;
      }
#pragma unroll
      for (int e = 0; e < E; ++e) add_compensated(acc_g[e], acc_c[e], sc_new * A_m[e]);
      add_compensated(l_g, l_c, sc_new);
      m_g = m_new;
    }
  }
  const int64_t orow = ((int64_t)beta * a.q_len + j) * g.Hq + h;
  const int64_t arow = ((int64_t)beta * g.Hq + h) * a.q_len + j;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    float out = l_g > 0.f ? acc_g[e] / l_g : 0.f;
    if (a.A) a.A[arow * D + li * E + e] = out;
    if (!a.O) continue;
    if (a.out_bf16) ((unsigned short*)a.O)[orow * D + li * E + e] = f32_to_bf16_rne(out);
    else ((float*)a.O)[orow * D + li * E + e] = out;
  }
  if (a.LSE && li == 0) a.LSE[arow] = l_g > 0.f ? m_g + logf(l_g) : -INFINITY;
}

// ------------------------------------------------------------------ one part
// Weight of a split, e^x for x <= 0 (0 for -inf, NaN for NaN): exp2 of the product's fraction in two parts,
// so that the product's rounding does not show.  This, one rounding per product and addition
// and a division in store_merged() hold an fp32 merge to the error its roundings leave: rms
// against 64 bits for 2 / 4 / 8 pairs 4.2 / 4.8 / 5.3e-8; with exp2 of a rounded product and a
// rounded reciprocal it was 4.6 / 5.2 / 5.6e-8.  expf() is as exact and costs more where many
// rows have 9 to 64 splits (20480 rows of 16, d = 64: 26 us with the short forms, 33 like this, 37
// with expf(); 29 since the groups of a wavefront meet without a weight).
__device__ __forceinline__ float weight(float x) {
  constexpr float HI = 1.4426950408889634f, LO = 1.925963e-8f;     // log2(e)
  x = x < -200.f ? -200.f : x;
  const float n = __builtin_rintf(x * HI);
  return __builtin_ldexpf(__builtin_amdgcn_exp2f(fmaf(x, LO, fmaf(x, HI, -n))), (int)fmaxf(n, -300.f));
}

// A call of one part as a launch is handed it.
struct FlatMerge {
  const float *O_sub, *LSE_sub;
  void* O;
  float *A, *LSE;
  int64_t batch_stride, split_stride;
  int32_t Hq, q_len, S;
  int16_t d, out_bf16;
  void* Qq;
  Rotary rotary;
};
static_assert(sizeof(FlatMerge) + 16 <= 112, "(and what merge_flat_rows_kernel takes besides)");
inline FlatMerge pack(const MergeArgs& a) {
  return FlatMerge{a.O_sub, a.LSE_sub, a.O, a.A, a.LSE, a.batch_stride, a.split_stride, a.g.Hq, a.q_len, a.plan.s_total,
                   (int16_t)a.g.d, (int16_t)a.out_bf16, a.Qq, a.rotary};
}

// What one lane gathers: the weighted sum of its four elements of the splits' outputs, the
// sum of weights, both relative to exp(m).  Sum is double where the splits follow blocks (MergeArgs::wide),
// of which there may be hundreds: float sums of 64 and 128 of them were off by up to 1.3 and 1.6e-7, these round twice.
template <typename Sum>
struct Fold {
  typedef __attribute__((ext_vector_type(4))) Sum Sum4;
  float m;
  Sum w;
  Sum4 acc;
};
template <typename Sum>
__device__ __forceinline__ Fold<Sum> empty_fold() {
  typedef typename Fold<Sum>::Sum4 Sum4;
  return Fold<Sum>{-INFINITY, Sum(0), Sum4{Sum(0), Sum(0), Sum(0), Sum(0)}};
}
__device__ __forceinline__ float finite(float m) { return m == -INFINITY ? 0.f : m; }

template <int N>
__device__ __forceinline__ float largest(const float (&ls)[N]) {
  float m = ls[0];
#pragma unroll
  for (int u = 1; u < N; ++u) m = fmaxf(m, ls[u]);
  return m;
}
// N splits at once: `ls` their log-sum-exps (-inf: empty, `v` unset), none above `m`.
template <typename Sum, int N>
__device__ __forceinline__ void fold_splits(Fold<Sum>& f, const float (&ls)[N], const f32x4 (&v)[N], float m) {
  m = fmaxf(m, f.m);
  const float mm = finite(m);
  const Sum old = weight(f.m - mm);
  f.w *= old;
  f.acc *= old;
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const Sum w = weight(ls[u] - mm);
    f.w += w;
    const f32x4 x = ls[u] == -INFINITY ? f32x4{0.f, 0.f, 0.f, 0.f} : v[u];
    f.acc += __builtin_convertvector(x, typename Fold<Sum>::Sum4) * w;      // (one rounding: the product must not pass a select)
  }
  f.m = m;
}
template <typename Sum>
__device__ __forceinline__ void store_merged(const FlatMerge& a, int beta, int h, int64_t j, int d0, const Fold<Sum>& f) {
  const f32x4 out = f.w > 0 ? __builtin_convertvector(f.acc / f.w, f32x4) : f32x4{0.f, 0.f, 0.f, 0.f};
  const int64_t orow = ((int64_t)beta * a.q_len + j) * a.Hq + h, arow = ((int64_t)beta * a.Hq + h) * a.q_len + j;
  if (a.A) *(f32x4*)(a.A + arow * a.d + d0) = out;
  if (a.O) {
    if (a.out_bf16) {
      unsigned short* o = (unsigned short*)a.O + orow * a.d + d0;
      const uint32_t lo = f32_to_bf16_rne(out[0]) | (uint32_t)f32_to_bf16_rne(out[1]) << 16;
      const uint32_t hi = f32_to_bf16_rne(out[2]) | (uint32_t)f32_to_bf16_rne(out[3]) << 16;
      *(uint2*)o = make_uint2(lo, hi);
    } else {
      *(f32x4*)((float*)a.O + orow * a.d + d0) = out;
    }
  }
  if (a.LSE && d0 == 0) a.LSE[arow] = f.w > 0 ? f.m + logf((float)f.w) : -INFINITY;
}

// A wavefront turns row (beta, h, j) of the call's queries, a lane per pair (bf16, d = 128).  Workgroups
// behind the merge's own do this: the kernel in front has read the queries as they were.
__device__ __forceinline__ void rotate_query(const FlatMerge& a, int beta, int h, int j, int lane) {
  __bf16* row = (__bf16*)a.Qq + (((int64_t)beta * a.q_len + j) * a.Hq + h) * 128;
  const float x = (float)row[lane], y = (float)row[lane + 64];
  float cs, sn;
  rotary_angle(a.rotary.pos0 + j, rotary_frequency(lane, 128, a.rotary.log2_theta), &cs, &sn);
  row[lane] = (__bf16)rotary_lo(x, y, cs, sn);
  row[lane + 64] = (__bf16)rotary_hi(x, y, cs, sn);
}

// One workgroup per (row, piece of 4 LPS elements of d): LPS lanes per split, the others
// walk the splits, INFL in flight per lane.  grid: x = token * pieces + piece (and, behind them, a token
// each to rotate), y = head, z = batch.
template <int LPS, int THREADS, int INFL, typename Sum>
__global__ __launch_bounds__(THREADS) void merge_flat_kernel(FlatMerge a) {
  constexpr int GROUPS = THREADS / LPS, WAVES = THREADS / 64;
  __shared__ float red_m[WAVES];
  __shared__ Sum red_w[WAVES];
  __shared__ typename Fold<Sum>::Sum4 red_acc[WAVES][LPS];
  const int tid = threadIdx.x, li = tid % LPS, grp = tid / LPS;
  const int h = blockIdx.y, beta = blockIdx.z, S = a.S;
  const int log2_pieces = __builtin_ctz(a.d / (4 * LPS)), j = blockIdx.x >> log2_pieces;      // (d is 64 or 128)
  if (j >= a.q_len) {
    if (tid < 64) rotate_query(a, beta, h, blockIdx.x - (a.q_len << log2_pieces), tid);
    return;
  }
  const int d0 = (blockIdx.x & ((1 << log2_pieces) - 1)) * (4 * LPS) + 4 * li;
  const int64_t base = (int64_t)beta * a.batch_stride + (int64_t)h * a.q_len + j;

  // the weights of a step are taken against the maximum of its splits over the whole wavefront:
  // the groups' sums then meet without another weight
  Fold<Sum> f = empty_fold<Sum>();
  for (int s0 = 0; s0 < S; s0 += INFL * GROUPS) {
    float ls[INFL];
    f32x4 v[INFL];
#pragma unroll
    for (int u = 0; u < INFL; ++u) {
      const int s = s0 + grp + u * GROUPS;
      const int64_t r = base + (int64_t)(s < S ? s : S - 1) * a.split_stride;
      ls[u] = a.LSE_sub[r];
      v[u] = *(const f32x4*)(a.O_sub + r * a.d + d0);
      if (s >= S) ls[u] = -INFINITY;
    }
    float m = largest<INFL>(ls);
#pragma unroll
    for (int x = LPS; x < 64; x <<= 1) m = fmaxf(m, __shfl_xor(m, x));
    fold_splits<Sum, INFL>(f, ls, v, m);
  }
  // the groups of a wavefront, then the wavefronts
#pragma unroll
  for (int x = LPS; x < 64; x <<= 1) {
    f.w += __shfl_xor(f.w, x);
#pragma unroll
    for (int e = 0; e < 4; ++e) f.acc[e] += __shfl_xor(f.acc[e], x);
  }
  if ((tid & 63) < LPS) {
    if (li == 0) { red_m[tid >> 6] = f.m; red_w[tid >> 6] = f.w; }
    red_acc[tid >> 6][li] = f.acc;
  }
  __syncthreads();
  if (tid >= LPS) return;
  f = empty_fold<Sum>();
#pragma unroll
  for (int k = 0; k < WAVES; ++k) f.m = fmaxf(f.m, red_m[k]);
  const float mm = finite(f.m);
#pragma unroll
  for (int k = 0; k < WAVES; ++k) {
    const Sum w = weight(red_m[k] - mm);
    f.w += red_w[k] * w;
    f.acc += red_acc[k][li] * w;
  }
  store_merged(a, beta, h, j, d0, f);
}

// Many rows of a few splits each (query encoding, pairs of other hosts): d / 4 lanes own a
// row, INFL splits in flight, nothing crosses lanes.
template <int D, int INFL, typename Sum>
__global__ __launch_bounds__(256) void merge_flat_rows_kernel(FlatMerge a, uint32_t m_q_len, uint32_t m_Hq, unsigned n_rows, unsigned first_wg) {
  constexpr int LPR = D / 4;
  const struct { Div q_len, Hq; } by = {div_of(a.q_len, m_q_len), div_of(a.Hq, m_Hq)};
  const unsigned n_wgs = (n_rows + 256 / LPR - 1) / (256 / LPR), wg = first_wg + blockIdx.x, tid = threadIdx.x;
  const bool turn = wg >= n_wgs;                                         // a wavefront per row to rotate
  const unsigned row = turn ? (wg - n_wgs) * 4 + tid / 64 : wg * (256 / LPR) + tid / LPR;      // (beta, h, j), j fastest
  if (row >= n_rows) return;
  const unsigned bh = quotient(row, by.q_len), j = row - bh * by.q_len.d, beta = quotient(bh, by.Hq), h = bh - beta * by.Hq.d;
  if (turn) {
    rotate_query(a, (int)beta, (int)h, (int)j, tid & 63);
    return;
  }
  const int d0 = 4 * (tid % LPR), S = a.S;
  const int64_t base = (int64_t)beta * a.batch_stride + (int64_t)h * a.q_len + j;
  Fold<Sum> f = empty_fold<Sum>();
  for (int s0 = 0; s0 < S; s0 += INFL) {
    float ls[INFL];
    f32x4 v[INFL];
#pragma unroll
    for (int u = 0; u < INFL; ++u) {
      const int64_t r = base + (int64_t)(s0 + u < S ? s0 + u : s0) * a.split_stride;
      ls[u] = a.LSE_sub[r];
      v[u] = *(const f32x4*)(a.O_sub + r * D + d0);
      if (s0 + u >= S) ls[u] = -INFINITY;
    }
    fold_splits<Sum, INFL>(f, ls, v, largest<INFL>(ls));
  }
  store_merged(a, (int)beta, (int)h, j, d0, f);
}

template <int LPS, int THREADS, int INFL, typename Sum>
hipError_t launch_flat(const MergeArgs& a, hipStream_t st) {
  const int turn = a.rotary.log2_theta != 0 ? a.q_len : 0;
  const dim3 grid((unsigned)(a.q_len * (a.g.d / (4 * LPS)) + turn), (unsigned)a.g.Hq, (unsigned)a.g.B);
  merge_flat_kernel<LPS, THREADS, INFL, Sum><<<grid, THREADS, 0, st>>>(pack(a));
  return hipGetLastError();
}

template <typename Sum>
hipError_t merge_one_part(const MergeArgs& a, int64_t rows, hipStream_t st) {
  const int S = a.plan.s_total;
  if (S <= 8 && rows >= 64) {
    const int64_t wgs = a.g.d == 64 ? (rows + 15) / 16 : (rows + 7) / 8, turn = a.rotary.log2_theta != 0 ? (rows + 3) / 4 : 0;
    const FlatMerge c = pack(a);
    const uint32_t m_q_len = make_div(a.q_len).m, m_Hq = make_div(a.g.Hq).m;
    return launch_in_pieces(wgs + turn, 256, [&](unsigned first, unsigned n_wgs) {
      // (a split past the last costs as much as one)
      if (a.g.d == 64 && S <= 4) merge_flat_rows_kernel<64, 4, Sum><<<dim3(n_wgs), 256, 0, st>>>(c, m_q_len, m_Hq, (unsigned)rows, first);
      else if (a.g.d == 64) merge_flat_rows_kernel<64, 8, Sum><<<dim3(n_wgs), 256, 0, st>>>(c, m_q_len, m_Hq, (unsigned)rows, first);
      else if (S <= 4) merge_flat_rows_kernel<128, 4, Sum><<<dim3(n_wgs), 256, 0, st>>>(c, m_q_len, m_Hq, (unsigned)rows, first);
      else merge_flat_rows_kernel<128, 8, Sum><<<dim3(n_wgs), 256, 0, st>>>(c, m_q_len, m_Hq, (unsigned)rows, first);
    });
  }
  // Few rows: pieces of d, so that the row's splits are in flight at once over more
  // workgroups and wavefronts; many rows fill the GPU as they are.  Measured, us, for
  // (rows x splits) against the kernel with the chain from split to split and a workgroup
  // per row: 8 x 384 10.8 -> 4.3, 32 x 128 5.7 -> 3.9, 32 x 96 6.0 -> 4.7, 672 x 29
  // 7.4 -> 4.0 (pieces of 32: 6.2-8.2), 8 x 32 (d = 64) 8.6 -> 3.3.  65 to 128 splits of few rows in one
  // step instead of two: whole decode calls of 8191 tokens (128 splits) 12.4 -> 11.8, 131072 (96) 82.6 -> 82.4.
  // A result merged into one of its own slabs: another piece's workgroup may not have read the
  // row's log-sum-exps yet when the first piece stores the new one, so a row stays whole.
  const bool in_place = a.LSE >= a.LSE_sub && a.LSE < a.LSE_sub + rows * S;
  if (in_place) return a.g.d == 64 ? launch_flat<16, 256, 4, Sum>(a, st) : launch_flat<32, 256, 4, Sum>(a, st);
  if (rows < 256) return S > 64 ? launch_flat<8, 512, 2, Sum>(a, st) : launch_flat<16, 256, 4, Sum>(a, st);
  if (S > 64) return launch_flat<16, 512, 4, Sum>(a, st);
  return a.g.d == 64 ? launch_flat<16, 256, 4, Sum>(a, st) : launch_flat<32, 256, 4, Sum>(a, st);
}

}  // namespace

hipError_t launch_merge(const MergeArgs& a, hipStream_t st) {
  const int64_t rows = (int64_t)a.g.B * a.g.Hq * a.q_len;
  if (rows > 0x7fffffff) return hipErrorInvalidValue;
  const SplitPlan& p = a.plan;
  if (p.flat) return a.wide ? merge_one_part<double>(a, rows, st) : merge_one_part<float>(a, rows, st);
  // splits the largest part is made of
  const int per_part = p.spb > p.st ? p.spb : p.st;
  const bool many = per_part <= 8 && rows >= 64;      // many rows, few splits each: a row per 32 lanes
  return launch_in_pieces(many ? (rows + 7) / 8 : rows, 256, [&](unsigned first, unsigned n_wgs) {
    const dim3 grid(n_wgs);
    if (many && a.g.d == 64) merge_rows_kernel<64, 4><<<grid, 256, 0, st>>>(a, rows, first);
    else if (many) merge_rows_kernel<128, 4><<<grid, 256, 0, st>>>(a, rows, first);
    else if (a.g.d == 64) merge_kernel<64, 8, 4><<<grid, 256, 0, st>>>(a, first);
    else merge_kernel<128, 8, 4><<<grid, 256, 0, st>>>(a, first);
  });
}

}  // namespace star
