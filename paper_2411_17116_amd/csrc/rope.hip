// Rotary position embedding for projections that arrive unrotated.
//
// Section 2.1 fixes the position every token carries (a context token keeps its
// index, the anchor keeps 0..a-1, a new token of phase 2 sits behind the cache),
// so the rotated key of an anchor token is the rotated key of that context token
// and one rotated K serves both roles.  The embedding itself is the one of the
// Llama family the paper evaluates: dimension i < d/2 pairs with i + d/2 and the
// pair is turned by pos * theta^(-2i/d).
//
// One kernel does everything a call needs before it can attend: Q is rotated (in
// place, or X -> Y for the rotation alone), K is rotated on its way from
// [B, T, Hkv, d] into the head-major cache [B, Hkv, cap, d], and V goes there as it
// is.  It is bound by HBM for a prefill and by latency for a decode step:
//   * A workgroup owns TT tokens.  Their d/2 angles each are evaluated once into LDS
//     (a thread's angles share the frequency) -- in double precision, because
//     pos * frequency reaches 1e6 rad and fp32 cannot hold its fractional turn -- and
//     serve all heads.
//   * Then every thread keeps one (token, pair of 16-byte chunks) and walks the
//     token's rows (query heads, key heads, value heads), BATCH rows requested before
//     the first is stored: rows rotated in place would otherwise be a chain of round
//     trips (nothing may be loaded ahead of a store that could alias it).
// Measured: a decode token of the 32 / 8-head shape (48 rows) 2.6 us, where two kernels
// that walked the heads in turn and a copy took 15 + 6 + 2.8 (and two more launch gaps).
#include "rotary.h"

namespace star {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;

template <typename T> struct Chunk;
template <> struct Chunk<float> {
  static constexpr int N = 4;
  typedef f32x4 vec;
  static __device__ __forceinline__ vec pack(const float (&x)[4]) { return f32x4{x[0], x[1], x[2], x[3]}; }
};
template <> struct Chunk<__bf16> {
  static constexpr int N = 8;
  typedef bf16x8 vec;
  static __device__ __forceinline__ vec pack(const float (&x)[8]) {
    bf16x8 v;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (__bf16)x[e];      // round to nearest even
    return v;
  }
};

constexpr int THREADS = 256;
constexpr int BATCH = 3;

struct RopeArgs {
  const void* X;          // [B, T, H, d] -> Y, same layout (Y may be X)
  void* Y;
  const void* K;          // [B, T, Hkv, d] -> rows [dst_row, dst_row + T) of Kc [B, Hkv, cap, d],
  const void* V;          // rotated, and V -> Vc as it is (Hkv = 0: neither)
  void* Kc;
  void* Vc;
  int32_t H, Hkv;
  uint32_t n_tokens, total;   // T, B T
  uint32_t first;         // first token of the launch
  int64_t cap, dst_row, pos0;
  double log2_theta;
  unsigned int* clear;    // eight counters to zero for the launch behind this one, or null
};

template <typename T, int half, int TT>
__global__ __launch_bounds__(THREADS) void rope_kernel(RopeArgs a) {
  constexpr int N = Chunk<T>::N;
  typedef typename Chunk<T>::vec vec;
  __shared__ float cs_all[TT][half], sn_all[TT][half];
  const int tid = threadIdx.x;
  const uint32_t tok0 = a.first + blockIdx.x * TT;
  if (a.clear && blockIdx.x == 0 && tid < 8) a.clear[tid] = 0u;
  {
    static_assert(THREADS % half == 0, "a thread's angles share their frequency");
    const int i = tid % half;
    const double inv_freq = rotary_frequency(i, 2 * half, a.log2_theta);
#pragma unroll
    for (int k0 = 0; k0 < TT; k0 += THREADS / half) {
      const int k = k0 + tid / half;
      if (k < TT)                                  // tokens past the last: angles nobody reads
        rotary_angle(a.pos0 + (tok0 + k) % a.n_tokens, inv_freq, &cs_all[k][i], &sn_all[k][i]);
    }
  }
  __syncthreads();

  constexpr int cpr = half / N;                    // chunk pairs per row: 8 or 16
  const int c = (tid % cpr) * N, k = (tid / cpr) % TT, slot = tid / (cpr * TT), n_slots = THREADS / (cpr * TT);
  const uint32_t tok = tok0 + k;
  if (tok >= a.total) return;
  float cs[N], sn[N];
#pragma unroll
  for (int e = 0; e < N; ++e) { cs[e] = cs_all[k][c + e]; sn[e] = sn_all[k][c + e]; }
  const uint32_t beta = tok / a.n_tokens, t = tok % a.n_tokens;
  constexpr size_t d = 2 * half;
  const size_t cache0 = ((size_t)beta * a.Hkv * a.cap + a.dst_row + t) * d + c;
  const int n_rows = a.H + 2 * a.Hkv;
  for (int h0 = slot; h0 < n_rows; h0 += BATCH * n_slots) {
    vec lo[BATCH], hi[BATCH];
    T* dst[BATCH];
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      int h = h0 + u * n_slots;
      if (h >= n_rows) h = h0;                     // past the last: row h0 again, not stored
      const T* src;
      if (h < a.H) {
        src = (const T*)a.X + ((size_t)tok * a.H + h) * d + c;
        dst[u] = (T*)a.Y + ((size_t)tok * a.H + h) * d + c;
      } else {
        const bool v = h >= a.H + a.Hkv;
        const int g = h - a.H - (v ? a.Hkv : 0);
        src = (const T*)(v ? a.V : a.K) + ((size_t)tok * a.Hkv + g) * d + c;
        dst[u] = (T*)(v ? a.Vc : a.Kc) + cache0 + (size_t)g * a.cap * d;
      }
      lo[u] = *(const vec*)src;
      hi[u] = *(const vec*)(src + half);
    }
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const int h = h0 + u * n_slots;
      if (h >= n_rows) break;
      if (h < a.H + a.Hkv) {
        float ylo[N], yhi[N];
#pragma unroll
        for (int e = 0; e < N; ++e) {
          const float x = (float)lo[u][e], y = (float)hi[u][e];
          ylo[e] = rotary_lo(x, y, cs[e], sn[e]);
          yhi[e] = rotary_hi(x, y, cs[e], sn[e]);
        }
        lo[u] = Chunk<T>::pack(ylo);
        hi[u] = Chunk<T>::pack(yhi);
      }
      *(vec*)dst[u] = lo[u];
      *(vec*)(dst[u] + half) = hi[u];
    }
  }
}

template <typename T, int half, int TT>
hipError_t launch(RopeArgs a, hipStream_t st) {
  return launch_in_pieces(((int64_t)a.total + TT - 1) / TT, THREADS, [&](unsigned first, unsigned n_wgs) {
    a.first = first * TT;
    rope_kernel<T, half, TT><<<dim3(n_wgs), THREADS, 0, st>>>(a);
    a.clear = nullptr;
  });
}

// Tokens per workgroup.  One where a token's rows keep 256 threads busy, or where there
// are too few tokens to fill the GPU otherwise; four for fewer rows; sixteen where the
// angles outweigh the rows.  Measured on 131072 tokens, d = 128, bf16, us with 1 / 4 / 16
// tokens (a kernel that gave a thread all heads of its chunk, before): 32 rows 376 / 390 /
// 413 (469), 16 rows 177 / 190 / 212 (240), 8 rows 92 / 76 / 81 (86), 4 rows 87 / 50 / 41
// (44), 1 row 79 / 40 / 30 (35); 4000 tokens of 8 rows 8.6 / 7.5 / 7.6 (8.8).
template <typename T, int half>
hipError_t launch(const RopeArgs& a, hipStream_t st) {
  const int64_t rows = (int64_t)a.H + 2 * a.Hkv;
  if (rows >= 16 || a.total < 1024) return launch<T, half, 1>(a, st);
  if (rows > 4 || a.total < 4096) return launch<T, half, 4>(a, st);
  return launch<T, half, 16>(a, st);
}

}  // namespace

hipError_t launch_rope(int dtype, const Geom& g, int H, const void* X, void* Y, const void* K, const void* V,
                       void* Kc, void* Vc, int64_t n_tokens, int64_t dst_row, int64_t pos0, double theta,
                       unsigned int* clear, hipStream_t st) {
  const int64_t total = (int64_t)g.B * n_tokens;
  if (total == 0) return hipSuccess;
  if (total > 0x7fffffff) return hipErrorInvalidValue;      // (550 GB and more of one tensor)
  RopeArgs a;
  a.X = X; a.Y = Y; a.K = K; a.V = V; a.Kc = Kc; a.Vc = Vc;
  a.H = H; a.Hkv = K ? g.Hkv : 0;
  a.n_tokens = (uint32_t)n_tokens; a.total = (uint32_t)total;
  a.cap = g.cap; a.dst_row = dst_row; a.pos0 = pos0; a.log2_theta = log2(theta);
  a.clear = clear;
  if (dtype != 0) return launch<__bf16, 64>(a, st);
  return g.d == 64 ? launch<float, 32>(a, st) : launch<float, 64>(a, st);
}

}  // namespace star
