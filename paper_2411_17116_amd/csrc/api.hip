// C-ABI entry points of libstarattn: argument validation, the phase-2 split
// plan, and kernel dispatch.  All checks run on the host before anything is
// enqueued; no exception or HIP error state leaves these functions.
#include "../../include/star_attn.h"
#include "star_internal.h"

#include <math.h>

#include <mutex>

namespace star {

// ---------------------------------------------------------------------------
// Per-device facts and the library's only state: static device memory that
// serves callers who hand in no workspace.
// ---------------------------------------------------------------------------
constexpr int MAX_DEVICES = 64;
constexpr int TICKET_SLOTS = 64;      // fallback sets of phase-1 work-queue counters

// Fallback work-queue counters of the bf16 phase-1 kernel (eight per launch),
// used only when star_attn_phase1* gets no workspace.  In host code the name is
// a stand-in: the device address comes from hipGetSymbolAddress, once per device
// (see device_state()).
static __device__ __align__(256) unsigned int phase1_ticket_slots[TICKET_SLOTS][8];

// Scratch of star_attn_phase2_static (per-split outputs and log-sum-exps), for
// callers that cannot bring a workspace.  Every GPU the library runs on holds
// its own copy until the process ends.  As above, host code uses the address
// hipGetSymbolAddress returns, never the name.
static __device__ __align__(256) unsigned char scratch[STAR_ATTN_STATIC_SCRATCH_BYTES];

struct DeviceState {
  bool ready = false;
  int n_cu = 0;
  unsigned int* tickets = nullptr;          // device address of phase1_ticket_slots on this device
  unsigned char* scratch_ptr = nullptr;     // device address of scratch on this device
  hipEvent_t slot_done[TICKET_SLOTS] = {};  // recorded behind the launch that last used a slot
  bool slot_used[TICKET_SLOTS] = {};
  bool slot_pending[TICKET_SLOTS] = {};     // taken by a call that has not recorded its event yet
  unsigned next_slot = 0;
};
static DeviceState g_dev[MAX_DEVICES];
static std::mutex g_dev_mu;

// State of the current device (looked up once per device), or null if the HIP
// runtime refuses.  Holds g_dev_mu only while it fills an entry.
static DeviceState* device_state() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return nullptr;
  DeviceState* d = &g_dev[dev];
  std::lock_guard<std::mutex> lock(g_dev_mu);
  if (d->ready) return d;
  if (hipDeviceGetAttribute(&d->n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      d->n_cu <= 0)
    return nullptr;
  if (hipGetSymbolAddress((void**)&d->tickets, HIP_SYMBOL(phase1_ticket_slots)) != hipSuccess ||
      hipGetSymbolAddress((void**)&d->scratch_ptr, HIP_SYMBOL(scratch)) != hipSuccess ||
      !d->tickets || !d->scratch_ptr)
    return nullptr;
  d->ready = true;
  return d;
}

// Compute units of the current device; the MI355X's 256 when no device can be
// asked (size queries still answer on a machine without a GPU).
int device_cu_count() {
  DeviceState* d = device_state();
  return d ? d->n_cu : 256;
}

// A free set of fallback counters of the current device: one whose last launch
// has finished.  -1 when all TICKET_SLOTS sets belong to launches still in flight.
static int acquire_ticket_slot(DeviceState* d) {
  std::lock_guard<std::mutex> lock(g_dev_mu);
  for (int k = 0; k < TICKET_SLOTS; ++k) {
    const int slot = (int)((d->next_slot + k) % TICKET_SLOTS);
    if (d->slot_pending[slot]) continue;       // another thread is between taking it and its launch
    if (d->slot_used[slot] && hipEventQuery(d->slot_done[slot]) != hipSuccess) {
      (void)hipGetLastError();          // hipErrorNotReady is an answer, not a failure
      continue;
    }
    if (!d->slot_done[slot] &&
        hipEventCreateWithFlags(&d->slot_done[slot], hipEventDisableTiming) != hipSuccess)
      return -1;
    d->slot_used[slot] = true;
    d->slot_pending[slot] = true;
    d->next_slot = (unsigned)(slot + 1);
    return slot;
  }
  return -1;
}

static int validate_shape(const star_attn_shape* s) {
  if (!s) return STAR_ATTN_ERR_NULL_POINTER;
  if (s->dtype != STAR_ATTN_F32 && s->dtype != STAR_ATTN_BF16) return STAR_ATTN_ERR_UNSUPPORTED_DTYPE;
  if (s->batch <= 0 || s->n_q_heads <= 0 || s->n_kv_heads <= 0 || s->head_dim <= 0 ||
      s->ctx_len <= 0 || s->block <= 0 || s->cache_capacity <= 0)
    return STAR_ATTN_ERR_INVALID_SHAPE;
  if (s->n_q_heads % s->n_kv_heads != 0) return STAR_ATTN_ERR_INVALID_SHAPE;
  if (s->n_q_heads > 65535 || s->batch > 65535) return STAR_ATTN_ERR_INVALID_SHAPE;
  // the kernels index tokens with 32-bit integers
  if (s->cache_capacity > (int64_t)0x7ff00000 || s->block > (int64_t)0x7ff00000)
    return STAR_ATTN_ERR_INVALID_SHAPE;
  if (s->dtype == STAR_ATTN_F32) {
    if (s->head_dim != 64 && s->head_dim != 128) return STAR_ATTN_ERR_UNSUPPORTED_HEAD_DIM;
  } else {
    if (s->head_dim != 128) return STAR_ATTN_ERR_UNSUPPORTED_HEAD_DIM;
  }
  if (s->anchor < 0 || s->anchor > s->block) return STAR_ATTN_ERR_ANCHOR_GT_BLOCK;
  if (s->cache_capacity < s->ctx_len) return STAR_ATTN_ERR_CACHE_OVERFLOW;
  if (!(s->softmax_scale >= 0.f) || isinf(s->softmax_scale)) return STAR_ATTN_ERR_INVALID_SHAPE;
  return STAR_ATTN_OK;
}

static Geom make_geom(const star_attn_shape* s) {
  Geom g;
  g.B = s->batch; g.Hq = s->n_q_heads; g.Hkv = s->n_kv_heads; g.G = g.Hq / g.Hkv; g.d = s->head_dim;
  g.L = s->ctx_len; g.b = s->block; g.a = s->anchor; g.cap = s->cache_capacity;
  g.scale = s->softmax_scale > 0.f ? s->softmax_scale : 1.0f / sqrtf((float)s->head_dim);
  return g;
}

static int64_t ceil_div(int64_t x, int64_t y) { return (x + y - 1) / y; }
static int64_t round_up(int64_t x, int64_t y) { return ceil_div(x, y) * y; }

// Wavefronts of the decode kernel that are resident at once on the current
// device (256 CUs on an MI355X): one split each under a flat plan of up to 16 rows.
static int64_t decode_slots(const Geom& g, int64_t total) {
  return device_cu_count() * (int64_t)decode_wavefronts_per_cu(decode_cache_resident(g, total));
}
static int64_t decode_slots_max() { return device_cu_count() * (int64_t)4; }

// Calls of 17 to 64 rows per KV head without per-part outputs that stream the cache through the decode kernel.
// More than 16 rows (a block of columns each 16) leave one wavefront too many pairs, so four share a split (two
// where a short cache gives none of them more than one step) and meet in LDS, one workgroup per CU. us, row-tiled
// (128 rows) / streamed, 32 / 8 heads: 20 rows on 600 keys 11.7 / 9.6, 32 on 2000 15.0 / 11.5, on 20000 24.7 / 20.8, on 131072
// 100.5 / 88.0; four sequences (32 KV heads) 20 on 1000 15.6 / 12.2, 32 on 2000 18.2 / 14.6; eight 17.9 / 14.9, 22.4 / 18.6.
// (With up to two workgroups per CU and a step to every wavefront it was slower than row-tiled at 300 to 800 keys of 32 to 96
// KV heads: 32 rows on 800 keys of 48 15.1 / 18.5.)
//   * 33 to 64 rows take all registers of a SIMD for one wavefront, which pays where a long cache comes from HBM: 48 on
//     131072 102.5 / 90.6, 64 104.2 / 90.8, 48 on 60000 55.9 / 50.2; resident 36.3 / 37.5 on 32768, 22.8 / 21.0 on 16384, 64 rows
//     26.4 / 21.6; 64 on 9000 of 44 KV heads 48.9 / 51.5, of 64 67.2 / 69.0.
//   * Where KV heads leave CUs idle, the row-tiled kernel is cut into as many splits as fill them: streaming has to keep four
//     fifths of the CUs busy once there is more than a launch's time to lose. 20000 keys: 132 KV heads (52 %) 264 / 331,
//     264 (52 % of two rounds) 558 / 651, 128 (all) 261 / 233; 60000: 96 (75 %) 521 / 548; 3000: 132 54.8 / 59.3; 2000 47.6 / 40.3.
// A single key tile has nothing to stream.
constexpr int64_t STREAM_WGS = 256;                  // one per CU
constexpr int64_t STREAM_PAIRED_KEYS = 64 * 32;      // most for two wavefronts to a split
constexpr int64_t STREAM_WIDE_KEYS = 16384;          // fewest for 33 rows and more
constexpr int64_t STREAM_ANY_KEYS = 2560;            // most that stream however few CUs they keep busy
static int64_t stream_slots(const Geom& g) {
  const int64_t slots = STREAM_WGS / ((int64_t)g.B * g.Hkv);
  return slots > 1 ? slots : 1;
}
// A bf16 call of few rows, too many for one block of columns.
static bool few_rows(const Geom& g, int64_t rows, int64_t total) {
  return total > 64 && rows > 16 && rows <= (decode_cache_resident(g, total) ? 32 : 64);
}
// Whether a call streams; if so, into how many splits and how many wavefronts share one.
static bool streams(const Geom& g, int64_t rows, int64_t total, int* waves, int64_t* splits) {
  if (!few_rows(g, rows, total) || (rows > 32 && total < STREAM_WIDE_KEYS)) return false;
  const int64_t pairs = (int64_t)g.B * g.Hkv, slots = stream_slots(g), steps = ceil_div(total, 32);
  *waves = steps <= 2 * slots && total <= STREAM_PAIRED_KEYS ? 2 : 4;
  const int64_t worth = ceil_div(steps, *waves);
  *splits = slots < worth ? slots : worth;
  if (total <= STREAM_PAIRED_KEYS)         // no more than the longest chain of steps asks for: fewer pairs to merge
    *splits = ceil_div(steps, ceil_div(steps, *splits * *waves) * *waves);
  const int64_t wgs = pairs * slots;
  return total <= STREAM_ANY_KEYS || slots >= worth || 5 * wgs >= 4 * STREAM_WGS * ceil_div(wgs, STREAM_WGS);
}

// ---- fp32 kernel: tiles of 16 rows shared by eight wavefronts (one workgroup per CU) or, for short runs of
// one tile per KV head, by four, or of 32 rows shared by four (two per CU).
// Most splits: what the resident workgroups can take at once, and never more than
// 4096 / (B Hq ceil(q / 64)), which bounds the per-split pairs a call keeps.
static int64_t f32_splits_max(const Geom& g, int64_t q_len, int tile) {
  const int64_t tiles = (int64_t)g.B * g.Hkv * ceil_div((int64_t)g.G * q_len, tile);
  const int64_t fill = (tile == 16 ? 256 : 512) / tiles, bound = ceil_div(4096, (int64_t)g.B * g.Hq * ceil_div(q_len, 64));
  return fill < 1 ? 1 : fill < bound ? fill : bound;
}
constexpr int64_t F32_SPLIT_MIN = 128;     // keys: one or two 16-key units for each wavefront
// Runs of 64 keys, one unit for each of four wavefronts, where a KV head's rows are one tile and all the runs start at
// once: what counts is the chain of units a wavefront walks.  More than 128 runs cost more to merge than
// they save, so beyond 8192 keys the runs grow.  us per call of one row, eight wavefronts and 128 keys / this: 1000 keys (2
// heads, d = 64) 8.6 / 7.7, 4000 (8 / 2 heads, d = 128) 11.8 / 9.8, 16000 14.2 / 13.3, 65000 31.1 / 30.6.  One KV head leaves half
// the CUs idle with them, which pays up to five units for each wavefront: d = 64, 32000 11.8 / 11.4, 40000 12.2 / 12.1,
// 50000 13.0 / 13.4, 131000 17.9 / 19.4, 262000 30.3 / 37.2.  With more runs than start at once they
// lose: two sequences of 9000 (8 / 2, d = 128), five tokens and one, 34.7 / 35.9.  0: not such a call.
static int64_t f32_short_runs(const Geom& g, int64_t q_len, int64_t total) {
  const int64_t worth = ceil_div(total, 64), runs = worth < 128 ? worth : 128, wgs = (int64_t)g.B * g.Hkv * runs;
  return (int64_t)g.G * q_len <= 16 && wgs <= 256 && (wgs > 128 || total <= 128 * 5 * 64) &&
                 runs <= ceil_div(4096, (int64_t)g.B * g.Hq * ceil_div(q_len, 64)) ? runs : 0;
}
// Rows per tile: 16 while those tiles with splits of that size leave CUs idle or fill them
// about twice (a unit of 16 keys then takes half as long), 32 beyond.  Measured, us, against
// 32-row tiles shared by eight wavefronts, one workgroup per CU (8 / 2 heads, d = 128):
// 33 tokens on 300 keys 18.2 -> 12.6, on 4000 26.0 -> 22.9; 100 on 4000 50.0 -> 32.7, on
// 16000 124 -> 74.  (Of 32-row tiles in fp32 products; in split products the last two take 26.9 and 54.7.)
// d = 128 without per-part outputs: runs of 128 keys have one unit of split products for each wavefront, whose start then counts, and
// 16-row tiles of longer runs are faster up to 850 tiles times runs, if all of one run start at once (750 if they are few and the runs to merge many).  us, 32-row tiles in fp32
// products / in split products / 16-row tiles: 111 tokens on 2309 keys (4 / 1 heads, 532) 22.9 / 24.9 / 15.2, 72 on 368 (three of 10 / 2, 552) 22.0 / 23.6 /
// 13.9, 100 on 2000 (8 / 2, 850) 24.6 / 25.9 / 17.4, 4 on 13722 (20 / 4, 864) 22.8 / 21.5 / 23.4; few tiles: 11 on 7137 (16 / 4, 672) 23.2 / 24.5 / 19.1, 6 on
// 25655 (two of 4 / 1, 804) - / 21.4 / 23.1; 336 tiles of two runs 14.0 / 15.2 / 17.4.
static int f32_tile_rows(const Geom& g, int64_t q_len, int64_t total, bool want_parts) {
  const int64_t rows = (int64_t)g.G * q_len, tiles = (int64_t)g.B * g.Hkv * ceil_div(rows, 16);
  const int64_t most = g.d == 128 && !want_parts && tiles <= 256 ? tiles < 16 ? 750 : 850 : 512;
  return rows <= 16 || (double)tiles * ceil_div(total, F32_SPLIT_MIN) <= most ? 16 : 32;
}
// Up to these bytes of K and V per KV head one workgroup walks all keys of its rows and
// there is nothing to merge.  us from a graph, one workgroup (or the two or four that share its columns) / splits and their merge: one
// row of one head, d = 64: 250 keys (125 KiB) 5.2 / 7.0, 487 6.7 / 6.2, 700 8.3 / 6.8, 1034 10.3 / 6.2; 32 rows on 487 7.1 / 8.2, on 1024 10.7 /
// 7.8; 8 / 2 heads, d = 128: 250 (250 KiB) 7.5 / 9.0, 400 8.9 / 7.8.  (Enqueued one by one, splits are a launch more.)
constexpr int64_t F32_DIRECT_BYTES = 256 << 10;

// ---- bf16 row-tiled kernel: one workgroup per CU is resident, 256 on the whole chip.  (The costs
// below and the fp32 split counts are for the whole chip; on a partition of it calls are cut
// finer than they need be, with the same results.)
constexpr int64_t ROW_WGS = 256;

// Workgroups of one split with tiles of `tile` rows.
static int64_t rows_wgs(const Geom& g, int64_t q_len, int tile) {
  return (int64_t)g.B * g.Hkv * ceil_div((int64_t)g.G * q_len, tile);
}
// Time of `splits` splits of `len` keys, in hundredths of a key tile's time (1.65 us): rounds
// of resident workgroups, each of them its key tiles -- 64 keys for 256 rows, or 128 keys
// for 128 rows, whose halves share them, 15 % dearer: twice the L2 -> LDS bytes -- and some
// 6 tiles' time to start, fill the pipeline and store; then the per-split pairs, written
// and read back at the rate of a copy (8 MB per tile's time).  Measured (32 / 8 heads, us
// with 256 / 128 rows): 64 tokens on 1000 keys 24.3 / 20.2, 8000 34.8 / 23.9, 32768 56 /
// 53, 131072 156 / 166; 33 tokens on 32768 49 / 51; 256 tokens on 131072 487 / 550.
static double rows_cost(const Geom& g, int64_t q_len, int tile, int64_t splits, int64_t len) {
  const double keys = tile == 128 ? 115.0 * ceil_div(len, 128) : 100.0 * ceil_div(len, 64);
  const double pairs = 8.0 * splits * g.B * g.Hq * q_len * (g.d + 1);
  return ceil((double)splits * rows_wgs(g, q_len, tile) / ROW_WGS) * (keys + 600) + pairs / 80000;
}
// The same for splits of every part, which need not be equal nor full: runs of up to `len` keys
// of n - 1 blocks, of the last block and of what lies behind the context.  Longest first, the
// resident workgroups take them in rounds; shorter runs fit into a round that is not full.  A
// workgroup's start and end cost less with fewer rows to store, and the halves' meeting something
// of its own.  The four figures minimise the time lost to the wrong tile over 400 drawn shapes
// timed with both: 0.3 % on average (17 shapes by over 3 %); 1.3 % (55) if every split counts
// as a full one: 256 tokens on 131072 in blocks of 16384 (32 / 8 heads), whose tail split
// then starts a second round of 256-row tiles: 573 us with 128 rows, 521 with 256.
static double parts_cost(const Geom& g, int64_t q_len, int64_t total, int tile, int64_t len) {
  const int64_t n = ceil_div(g.L, g.b), wgs = rows_wgs(g, q_len, tile), rows = (int64_t)g.G * q_len;
  const double fixed = tile == 128 ? 500 : 600 - (rows < 256 ? 256.0 - rows : 0);
  const int64_t part[3] = {n > 1 ? g.b : 0, g.L - (n - 1) * g.b, total - g.L}, count[3] = {n - 1, 1, 1};
  int64_t runs[4] = {0, 0, 0, 0}, keys[4] = {len, 0, 0, 0};      // full ones, and each part's last
  for (int i = 0; i < 3; ++i) {
    runs[0] += count[i] * (part[i] / len);
    keys[i + 1] = part[i] % len;
    runs[i + 1] = keys[i + 1] ? count[i] : 0;
  }
  double cost = 0;
  int64_t room = 0;                                              // workgroups the last round still takes
  for (int64_t last = len + 1;;) {
    int i = -1;
    for (int k = 0; k < 4; ++k)
      if (runs[k] && keys[k] < last && (i < 0 || keys[k] > keys[i])) i = k;
    if (i < 0) return cost;
    last = keys[i];
    int64_t w = -room;
    for (int k = 0; k < 4; ++k) w += keys[k] == last ? runs[k] * wgs : 0;
    if (w <= 0) { room = -w; continue; }
    const int64_t rounds = ceil_div(w, ROW_WGS);
    cost += (double)rounds * ((tile == 128 ? 120.0 * ceil_div(last, 128) : 100.0 * ceil_div(last, 64)) + fixed);
    room = rounds * ROW_WGS - w;
  }
}
// Splits whose per-split pairs fit `bytes` of workspace.
static int64_t splits_that_fit(const Geom& g, int64_t q_len, int64_t bytes) {
  return bytes / 256 * 256 / ((int64_t)g.B * g.Hq * q_len * (g.d + 1) * 4);
}
// Largest number of splits whose per-split pairs a call may keep: what
// star_attn_phase2_static's scratch holds, and at least `aligned`.
static int64_t rows_splits_cap(const Geom& g, int64_t q_len, int64_t aligned) {
  const int64_t fit = splits_that_fit(g, q_len, STAR_ATTN_STATIC_SCRATCH_BYTES);
  return fit > aligned ? fit : aligned;
}
// Equal runs of keys for a call without per-part outputs: with either tile, the number of
// splits that fills the resident workgroups once, or, where a split's workgroups do not
// divide them, up to four times.
struct RowsChoice {
  int tile;
  int64_t splits, len;
  double cost;
};
static RowsChoice rows_flat(const Geom& g, int64_t q_len, int64_t total, int64_t cap) {
  RowsChoice best = {0, 0, 0, 0.0};
  for (int tile = 256; tile >= 128; tile -= 128)
    for (int64_t k = 0; k <= 4; ++k) {
      int64_t s = k == 0 ? 1 : k * ROW_WGS / rows_wgs(g, q_len, tile);
      if (s > ceil_div(total, 256)) s = ceil_div(total, 256);     // keys worth a split
      if (s > cap) s = cap;
      if (s < 1) continue;
      const int64_t len = round_up(ceil_div(total, s), 64);
      s = ceil_div(total, len);
      const double cost = rows_cost(g, q_len, tile, s, len);
      if (best.tile == 0 || cost < best.cost) best = {tile, s, len, cost};
    }
  return best;
}

// Split plan for a phase-2 call with q_len new tokens that can see `total`
// cache rows.  Decode-sized calls (G * q_len rows fit one 16-column MFMA tile)
// stream the cache: without per-part outputs the keys of each (batch, KV head)
// are cut into equal splits, one per resident workgroup; with per-part outputs
// the splits respect block boundaries.  Larger calls are compute-bound and use
// as few splits as still fill the GPU; fp32 calls ditto, in equal runs of keys when
// no per-part outputs are asked for.  The number of equal runs depends on `total`: a
// caller whose workspace was sized for a shorter cache gets as many as fit
// `max_bytes` (at least one), so that a call it could make does not become one it cannot.
static bool make_plan(const star_attn_shape* s, int64_t q_len, int64_t total, bool want_parts,
                      SplitPlan* p, int64_t max_bytes = INT64_MAX) {
  Geom g = make_geom(s);
  int64_t n = ceil_div(g.L, g.b);
  int64_t bmax = g.b < g.L ? g.b : g.L;
  int64_t tail_cap = g.cap - g.L;
  int64_t rows = (int64_t)g.G * q_len;
  int64_t fit = splits_that_fit(g, q_len, max_bytes);
  if (fit < 1) fit = 1;
  int waves = 1;
  int64_t splits = 0;
  p->decode = s->dtype == STAR_ATTN_BF16 && (rows <= 16 || (!want_parts && streams(g, rows, total, &waves, &splits))) ? 1 : 0;
  p->flat = 0;
  p->tile_rows = 0;
  p->waves = 1;
  p->n_blocks = (int32_t)n;
  if (n > (1 << 24)) return false;
  int64_t split_len;
  if (p->decode && rows > 16) {
    p->waves = waves;
    if (splits > fit) splits = fit;
    p->flat = 1;
    p->split_len = round_up(ceil_div(total, splits), 32);
    p->spb = 0;
    p->st = 0;
    p->s_total = (int32_t)splits;
    return true;
  }
  if (p->decode && !want_parts) {
    int64_t pairs = (int64_t)g.B * g.Hkv;
    int64_t slots = decode_slots(g, total);
    if (slots <= 0) return false;                  // no usable device
    int64_t s0 = slots / pairs > 1 ? slots / pairs : 1;
    split_len = round_up(ceil_div(total, s0), 32);
    if (split_len < 64) split_len = 64;
    p->flat = 1;
    p->split_len = split_len;
    p->spb = 0;
    p->st = 0;
    p->s_total = (int32_t)ceil_div(total, split_len);
    // More than 64 splits of a resident cache: four wavefronts share one, and a quarter or half of them is left
    // to merge.  Two such workgroups per CU, one where there are fewer than eight KV heads and four times the
    // splits per head.  us, one wavefront / four: 8191 tokens of eight heads 11.1 / 10.4, 13900 15.3 / 15.1; 27800 of two 12.0 /
    // 10.3, 131000 26.6 / 25.1; up to 64 splits the meeting costs more than the merge saves (2000 of eight 7.5 / 7.9,
    // 16000 of sixteen 26.7 / 27.2), and caches read from HBM gain nothing (131072 of eight 82.3 / 82.2, four
    // sequences of 32768 83.1 / 83.8).  Eight heads and more have two wavefronts on a SIMD: where a sixth and more of
    // the last round's have no step (a quarter with more than eight rows, whose pairs weigh more), the others' take longer
    // than one wavefront with more steps: 8400 tokens of eight 10.9 / 12.6, 10600 13.2 / 14.2, 16800 17.0 / 18.2, 25400 21.5 / 22.4;
    // twelve rows 12.8 / 13.4, 14.8 / 15.0, 18.3 / 19.0, 22.7 / 22.7, but 12283 16.2 / 15.2 (four rows 14.4 / 14.6).
    if (p->s_total > 64 && decode_cache_resident(g, total)) {
      const int64_t wgs = device_cu_count() * (int64_t)(pairs < 8 ? 1 : 2), steps = ceil_div(total, 32), most = ceil_div(steps, 4);
      int64_t splits = wgs / pairs < most ? wgs / pairs : most;
      if (splits < 1) splits = 1;
      const int64_t room = ceil_div(steps, 4 * splits) * 4 * splits;      // steps of as many rounds
      if (pairs < 8 || 12 * steps >= (rows > 8 ? 9 : 10) * room) {
        p->waves = 4;
        p->split_len = round_up(ceil_div(total, splits), 32);
        p->s_total = (int32_t)splits;
      }
    }
    return true;
  }
  if (s->dtype == STAR_ATTN_F32 && !want_parts) {
    p->tile_rows = f32_tile_rows(g, q_len, total, want_parts);
    int64_t splits = f32_short_runs(g, q_len, total);
    p->waves = splits > 0 ? 4 : 8;
    if (splits == 0) {
      splits = f32_splits_max(g, q_len, p->tile_rows);
      if (splits > ceil_div(total, F32_SPLIT_MIN)) splits = ceil_div(total, F32_SPLIT_MIN);
    }
    if (total * g.d * 8 <= F32_DIRECT_BYTES) splits = 1;
    if (splits > fit) splits = fit;
    if (splits == 1) p->waves = 8;
    p->flat = 1;
    p->split_len = round_up(ceil_div(total, splits), 32);
    p->spb = 0;
    p->st = 0;
    p->s_total = (int32_t)ceil_div(total, p->split_len);
    return true;
  }
  if (p->decode) {
    int64_t key_heads = g.cap * g.B * g.Hkv;
    int64_t want = ceil_div(key_heads, 2048);
    split_len = 256;
    while (split_len < want && split_len < 4096) split_len *= 2;
  } else {
    // splits over all blocks that fill the GPU; keys worth a split.  (bf16: counted with tiles
    // whose heads are not packed, fewer splits than packed rows would need for odd groups.)
    int64_t want, min_len;
    if (s->dtype == STAR_ATTN_F32) {
      // (the same splits for every length of the cache)
      p->tile_rows = f32_tile_rows(g, q_len, total, want_parts);
      want = f32_splits_max(g, q_len, f32_tile_rows(g, q_len, g.cap, want_parts));
      min_len = F32_SPLIT_MIN;
    } else {
      const int64_t wgs = (int64_t)g.B * g.Hkv * (g.G / flash_heads_per_workgroup(g.G)) *
                          ceil_div(q_len, flash_tokens_per_workgroup(g.G));
      want = ceil_div(ROW_WGS, wgs);
      min_len = 256;
    }
    int64_t spb = ceil_div(want, n);
    int64_t spb_max = bmax / min_len > 1 ? bmax / min_len : 1;
    if (spb > spb_max) spb = spb_max;
    if (spb < 1) spb = 1;
    split_len = round_up(ceil_div(bmax, spb), s->dtype == STAR_ATTN_F32 ? 32 : 64);
  }
  int64_t spb = ceil_div(bmax, split_len);
  int64_t st = tail_cap > 0 ? ceil_div(tail_cap, split_len) : 1;
  int64_t s_total = n * spb + st;
  if (s_total > (1 << 24)) return false;
  if (s->dtype == STAR_ATTN_BF16 && !p->decode) {
    const double c256 = rows_cost(g, q_len, 256, s_total, split_len), c128 = rows_cost(g, q_len, 128, s_total, split_len);
    p->tile_rows = c128 < c256 ? 128 : 256;
    if (want_parts)
      p->tile_rows = parts_cost(g, q_len, total, 128, split_len) < parts_cost(g, q_len, total, 256, split_len) ? 128 : 256;
    // equal runs of keys instead of splits of every part, if they take less time
    if (!want_parts) {
      const int64_t cap = rows_splits_cap(g, q_len, s_total);
      const RowsChoice f = rows_flat(g, q_len, total, cap < fit ? cap : fit);
      if (s_total > fit || f.cost < (c128 < c256 ? c128 : c256)) {
        p->flat = 1;
        p->tile_rows = f.tile;
        p->split_len = f.len;
        p->spb = 0;
        p->st = 0;
        p->s_total = (int32_t)f.splits;
        return true;
      }
    }
  }
  p->split_len = split_len;
  p->spb = (int32_t)spb;
  p->st = (int32_t)st;
  p->s_total = (int32_t)s_total;
  return true;
}

static size_t plan_bytes(const star_attn_shape* s, const SplitPlan& p, int64_t q_len) {
  size_t rows = (size_t)s->batch * (size_t)p.s_total * (size_t)s->n_q_heads * (size_t)q_len;
  size_t bytes = rows * (size_t)(s->head_dim + 1) * sizeof(float);
  return (bytes + 255) & ~(size_t)255;
}

static bool misaligned(const void* p) { return ((uintptr_t)p & 15u) != 0; }

// Rotary embedding requested by the *_rope entry points (theta == 0: none).
struct Rope {
  double theta;
  int64_t pos0;
};

static int validate_rope(const star_attn_shape* s, double theta, int64_t pos0) {
  if (!(theta > 1.0) || isinf(theta) || pos0 < 0 || pos0 > ((int64_t)1 << 40))
    return STAR_ATTN_ERR_INVALID_SHAPE;
  (void)s;    // every supported head_dim is even
  return STAR_ATTN_OK;
}

// Bytes of the separately given anchors (K or V), 256-byte padded.
static size_t anchor_bytes(const star_attn_shape* s, int anchor_mode) {
  size_t es = s->dtype == STAR_ATTN_F32 ? 4 : 2;
  size_t anchors = anchor_mode == STAR_ATTN_ANCHOR_PER_BLOCK
                       ? (size_t)((s->ctx_len + s->block - 1) / s->block) : 1;
  size_t n = (size_t)s->batch * (size_t)s->n_kv_heads * anchors * (size_t)s->anchor *
             (size_t)s->head_dim * es;
  return (n + 255) & ~(size_t)255;
}

// Bytes the bf16 phase-1 kernel's eight work-queue counters take in a workspace.
constexpr size_t TICKET_BYTES = 256;

}  // namespace star

using namespace star;

extern "C" {

size_t star_attn_workspace_bytes(const star_attn_shape* shape, int64_t max_q_len) {
  if (validate_shape(shape) != STAR_ATTN_OK || max_q_len <= 0) return 0;
  // The plan depends on q_len only through the number of row tiles, so the largest
  // requirement is found at tile boundaries and at max_q_len itself.
  const Geom g = make_geom(shape);
  size_t best = 0;
  auto need = [&](int64_t splits, int64_t q) {
    SplitPlan p = {};
    p.s_total = (int32_t)splits;
    size_t b = plan_bytes(shape, p, q);
    if (b > best) best = b;
  };
  auto consider = [&](int64_t q) {
    if (q < 1 || q > max_q_len) return;
    SplitPlan p;
    // the number of part-aligned splits never exceeds what the full cache needs
    const bool ok = make_plan(shape, q, shape->cache_capacity, true, &p);
    const int64_t aligned = ok ? p.s_total : 0;
    need(aligned, q);
    // a shorter cache may be cut into more equal runs than the full one; bound them
    if (p.decode) {
      int64_t pairs = (int64_t)g.B * g.Hkv;
      int64_t s0 = decode_slots_max() / pairs > 1 ? decode_slots_max() / pairs : 1;
      SplitPlan f;
      if (make_plan(shape, q, shape->cache_capacity, false, &f)) need(f.s_total > s0 ? f.s_total : s0, q);
    } else if (shape->dtype == STAR_ATTN_F32) {
      const int64_t worth = ceil_div(g.cap, F32_SPLIT_MIN);
      if ((int64_t)g.G * q <= 16) {       // the most short runs of any length of the cache
        const int64_t all = 256 / ((int64_t)g.B * g.Hkv), most = all < 128 ? all : 128, short_worth = ceil_div(g.cap, 64);
        if (most > 0) need(most < short_worth ? most : short_worth, q);
      }
      for (int tile = 16; tile <= 32; tile += 16) {
        const int64_t most = f32_splits_max(g, q, tile);
        need(most < worth ? most : worth, q);
      }
    } else if (ok) {
      if ((int64_t)g.G * q <= 64) {
        const int64_t worth = ceil_div(ceil_div(g.cap, 32), 2), slots = stream_slots(g);
        need(slots < worth ? slots : worth, q);
      }
      int64_t most = 4 * ROW_WGS / rows_wgs(g, q, 256), worth = ceil_div(g.cap, 256);
      if (most > worth) most = worth;
      if (most < 1) most = 1;
      SplitPlan f = {};
      f.s_total = (int32_t)most;
      if (plan_bytes(shape, f, q) <= STAR_ATTN_STATIC_SCRATCH_BYTES) need(most, q);
      else if (best < STAR_ATTN_STATIC_SCRATCH_BYTES) best = STAR_ATTN_STATIC_SCRATCH_BYTES;   // rows_splits_cap
      need(1, q);
    }
  };
  for (int64_t q = 1; q <= max_q_len && q <= 64; ++q) consider(q);
  if (shape->dtype == STAR_ATTN_F32) {
    // tiles hold 32 / G tokens, not a whole number: every q_len up to where one split
    // per part fills the GPU
    for (int64_t q = 65; q <= max_q_len && q <= 256 * 32; ++q) consider(q);
  } else {
    for (int64_t q = 64; q <= max_q_len; q += 32) { consider(q); consider(q + 1); }
    // the equal runs' tiles end elsewhere (256 / G or 128 / G tokens)
    for (int64_t q = 65; q < max_q_len && q <= 4096; ++q)
      if (rows_wgs(g, q + 1, 128) != rows_wgs(g, q, 128)) consider(q);
    if (max_q_len > 4096 && best < STAR_ATTN_STATIC_SCRATCH_BYTES) best = STAR_ATTN_STATIC_SCRATCH_BYTES;
  }
  consider(max_q_len);
  return best;
}

size_t star_attn_phase1_workspace_bytes(const star_attn_shape* shape, int anchor_mode) {
  if (validate_shape(shape) != STAR_ATTN_OK) return 0;
  if (shape->dtype == STAR_ATTN_BF16) return TICKET_BYTES;     // the launch's work-queue counters
  const bool given = anchor_mode == STAR_ATTN_ANCHOR_EXTERNAL ||
                     anchor_mode == STAR_ATTN_ANCHOR_PER_BLOCK ||
                     anchor_mode == STAR_ATTN_ANCHOR_ALL_BLOCKS;
  return given ? 2 * anchor_bytes(shape, anchor_mode) : 0;
}

}  // extern "C"

static bool known_mode(int anchor_mode) {
  return anchor_mode == STAR_ATTN_ANCHOR_FIRST || anchor_mode == STAR_ATTN_ANCHOR_PREVIOUS ||
         anchor_mode == STAR_ATTN_ANCHOR_EXTERNAL || anchor_mode == STAR_ATTN_ANCHOR_PER_BLOCK ||
         anchor_mode == STAR_ATTN_ANCHOR_ALL_BLOCKS;
}

// Phase 1 behind every public variant.  With `rope`, Q is rotated in place and K
// on its way into the cache.
static int phase1_impl(const star_attn_shape* shape, int anchor_mode, const Rope* rope, void* Q,
                       const void* K, const void* V, const void* K_anchor, const void* V_anchor,
                       void* O_ctx, float* LSE_ctx, void* K_cache, void* V_cache, void* workspace,
                       size_t workspace_bytes, void* hip_stream) {
  int rc = validate_shape(shape);
  if (rc != STAR_ATTN_OK) return rc;
  if (rope && (rc = validate_rope(shape, rope->theta, rope->pos0)) != STAR_ATTN_OK) return rc;
  if (!known_mode(anchor_mode)) return STAR_ATTN_ERR_INVALID_MODE;
  if (!Q || !K || !V || !O_ctx || !K_cache || !V_cache) return STAR_ATTN_ERR_NULL_POINTER;
  if (misaligned(Q) || misaligned(K) || misaligned(V) || misaligned(O_ctx) ||
      misaligned(K_cache) || misaligned(V_cache) || ((uintptr_t)LSE_ctx & 3u))
    return STAR_ATTN_ERR_MISALIGNED;
  const bool ext = (anchor_mode == STAR_ATTN_ANCHOR_EXTERNAL ||
                    anchor_mode == STAR_ATTN_ANCHOR_PER_BLOCK ||
                    anchor_mode == STAR_ATTN_ANCHOR_ALL_BLOCKS) && shape->anchor > 0;
  // separately given anchors are read where the caller left them; the fp32 workspace
  // stays a requirement of the call (star_attn_phase1_workspace_bytes) all the same
  const bool ext_workspace = ext && shape->dtype == STAR_ATTN_F32;
  if (ext) {
    if (!K_anchor || !V_anchor) return STAR_ATTN_ERR_NULL_POINTER;
    if (misaligned(K_anchor) || misaligned(V_anchor)) return STAR_ATTN_ERR_MISALIGNED;
  }
  if (ext_workspace) {
    if (!workspace) return STAR_ATTN_ERR_NULL_POINTER;
    if ((uintptr_t)workspace & 255u) return STAR_ATTN_ERR_MISALIGNED;
    if (workspace_bytes < 2 * anchor_bytes(shape, anchor_mode))
      return STAR_ATTN_ERR_WORKSPACE_TOO_SMALL;
  }
  Geom g = make_geom(shape);
  hipStream_t st = (hipStream_t)hip_stream;
  // The bf16 kernel's workgroups draw their row tiles from eight counters: the
  // caller's workspace if there is one, else a free set of the library's own.
  DeviceState* ds = nullptr;
  unsigned int* tickets = nullptr;
  int slot = -1;
  if (shape->dtype == STAR_ATTN_BF16) {
    if (workspace) {
      if ((uintptr_t)workspace & 15u) return STAR_ATTN_ERR_MISALIGNED;
      if (workspace_bytes < TICKET_BYTES) return STAR_ATTN_ERR_WORKSPACE_TOO_SMALL;
    }
    if (!(ds = device_state())) return STAR_ATTN_ERR_LAUNCH_FAILED;
    if (workspace) {
      tickets = (unsigned int*)workspace;
    } else {
      // a captured launch would carry its set into every replay of the graph
      hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
      if (hipStreamIsCapturing(st, &cap) != hipSuccess) (void)hipGetLastError();
      if (cap != hipStreamCaptureStatusNone) return STAR_ATTN_ERR_BUSY;
      if ((slot = acquire_ticket_slot(ds)) < 0) return STAR_ATTN_ERR_BUSY;
      tickets = ds->tickets + 8 * slot;
    }
  }
  // On every way out: the set is free again once everything enqueued so far is
  // done.  A set whose event could not be recorded is never handed out again.
  struct SlotRelease {
    DeviceState* ds; int slot; hipStream_t st;
    ~SlotRelease() {
      if (slot < 0) return;
      if (hipEventRecord(ds->slot_done[slot], st) != hipSuccess) { (void)hipGetLastError(); return; }
      std::lock_guard<std::mutex> lock(g_dev_mu);
      ds->slot_pending[slot] = false;
    }
  } slot_release{ds, slot, st};
  // Algorithm 1: keep the K/V of every block once (anchor copies never exist here).
  // The attention kernels read plain inputs where they are and file them in the
  // caches themselves; rotated keys go through the caches.
  if (rope && launch_rope(shape->dtype, g, g.Hq, Q, Q, K, V, K_cache, V_cache, g.L, 0, rope->pos0, rope->theta,
                          tickets, st) != hipSuccess)
    return STAR_ATTN_ERR_LAUNCH_FAILED;
  Phase1Args a;
  a.g = g; a.Q = Q; a.O = O_ctx; a.LSE = LSE_ctx; a.Kc = K_cache; a.Vc = V_cache;
  a.anchor_mode = anchor_mode; a.Ka = K_anchor; a.Va = V_anchor;
  a.Kin = rope ? nullptr : K;
  a.Vin = rope ? nullptr : V;
  a.tickets = tickets;
  a.tickets_clear = rope ? 1 : 0;
  a.n_cu = ds ? ds->n_cu : 0;
  hipError_t e = shape->dtype == STAR_ATTN_F32 ? launch_phase1_f32(a, st) : launch_phase1_bf16(a, st);
  return e == hipSuccess ? STAR_ATTN_OK : STAR_ATTN_ERR_LAUNCH_FAILED;
}

extern "C" {

int star_attn_phase1_anchor(const star_attn_shape* shape, int anchor_mode, const void* Q,
                            const void* K, const void* V, const void* K_anchor,
                            const void* V_anchor, void* O_ctx, float* LSE_ctx, void* K_cache,
                            void* V_cache, void* workspace, size_t workspace_bytes,
                            void* hip_stream) {
  return phase1_impl(shape, anchor_mode, nullptr, const_cast<void*>(Q), K, V, K_anchor, V_anchor,
                     O_ctx, LSE_ctx, K_cache, V_cache, workspace, workspace_bytes, hip_stream);
}

int star_attn_phase1(const star_attn_shape* shape, const void* Q, const void* K, const void* V,
                     void* O_ctx, float* LSE_ctx, void* K_cache, void* V_cache,
                     void* workspace, size_t workspace_bytes, void* hip_stream) {
  return phase1_impl(shape, STAR_ATTN_ANCHOR_FIRST, nullptr, const_cast<void*>(Q), K, V, nullptr,
                     nullptr, O_ctx, LSE_ctx, K_cache, V_cache, workspace, workspace_bytes,
                     hip_stream);
}

int star_attn_phase1_rope(const star_attn_shape* shape, double rope_theta, int64_t pos0, void* Q,
                          const void* K, const void* V, void* O_ctx, float* LSE_ctx,
                          void* K_cache, void* V_cache, void* workspace, size_t workspace_bytes,
                          void* hip_stream) {
  Rope rope = {rope_theta, pos0};
  return phase1_impl(shape, STAR_ATTN_ANCHOR_FIRST, &rope, Q, K, V, nullptr, nullptr, O_ctx,
                     LSE_ctx, K_cache, V_cache, workspace, workspace_bytes, hip_stream);
}

int star_attn_rope(const star_attn_shape* shape, int32_t n_heads, int64_t n_tokens, int64_t pos0,
                   double rope_theta, const void* X, void* Y, void* hip_stream) {
  int rc = validate_shape(shape);
  if (rc != STAR_ATTN_OK) return rc;
  if ((rc = validate_rope(shape, rope_theta, pos0)) != STAR_ATTN_OK) return rc;
  if (n_heads <= 0 || n_tokens <= 0) return STAR_ATTN_ERR_INVALID_SHAPE;
  if (!X || !Y) return STAR_ATTN_ERR_NULL_POINTER;
  if (misaligned(X) || misaligned(Y)) return STAR_ATTN_ERR_MISALIGNED;
  hipError_t e = launch_rope(shape->dtype, make_geom(shape), n_heads, X, Y, nullptr, nullptr, nullptr, nullptr,
                             n_tokens, 0, pos0, rope_theta, nullptr, (hipStream_t)hip_stream);
  return e == hipSuccess ? STAR_ATTN_OK : STAR_ATTN_ERR_LAUNCH_FAILED;
}

}  // extern "C"

// Phase 2 behind every public variant.  With `rope`, Qq is rotated in place and
// Kq on its way into the cache (new token j sits at pos0 + cache_len + j).
// `pair` (a host's share of a call): the result is left as the fp32 pair
// (A, LSE) instead of O, and Kq == Vq == NULL means "append nothing, every new
// token sees cache rows [0, cache_len)".
static int phase2_impl(const star_attn_shape* shape, const Rope* rope, int64_t cache_len,
                       int64_t q_len, void* Qq, const void* Kq, const void* Vq, void* K_cache,
                       void* V_cache, float* O_part, float* LSE_part, void* O, bool pair, float* A,
                       float* LSE, void* workspace, size_t workspace_bytes, void* hip_stream,
                       bool static_scratch = false) {
  int rc = validate_shape(shape);
  if (rc != STAR_ATTN_OK) return rc;
  if (rope && (rc = validate_rope(shape, rope->theta, rope->pos0)) != STAR_ATTN_OK) return rc;
  if (q_len <= 0 || q_len > (1 << 20) || cache_len < shape->ctx_len) return STAR_ATTN_ERR_INVALID_SHAPE;
  const bool append = !(pair && !Kq && !Vq);
  const int64_t total = cache_len + (append ? q_len : 0);
  if (total > shape->cache_capacity) return STAR_ATTN_ERR_CACHE_OVERFLOW;
  if (static_scratch) workspace_bytes = STAR_ATTN_STATIC_SCRATCH_BYTES;
  if (!Qq || !K_cache || !V_cache || (!workspace && !static_scratch)) return STAR_ATTN_ERR_NULL_POINTER;
  if (append && (!Kq || !Vq)) return STAR_ATTN_ERR_NULL_POINTER;
  if (pair ? (!A || !LSE) : !O) return STAR_ATTN_ERR_NULL_POINTER;
  if ((O_part == nullptr) != (LSE_part == nullptr)) return STAR_ATTN_ERR_NULL_POINTER;
  if (misaligned(Qq) || misaligned(Kq) || misaligned(Vq) || misaligned(K_cache) ||
      misaligned(V_cache) || misaligned(O) || misaligned(O_part) || ((uintptr_t)LSE_part & 3u) ||
      misaligned(A) || ((uintptr_t)LSE & 3u) || ((uintptr_t)workspace & 255u))
    return STAR_ATTN_ERR_MISALIGNED;
  SplitPlan plan;
  if (!make_plan(shape, q_len, total, O_part != nullptr, &plan))
    return STAR_ATTN_ERR_INVALID_SHAPE;
  // (A call of few rows makes do with the static scratch too: whether it streams, in few splits, or is row-tiled, in
  // more, is a matter of the CUs that it keeps busy.)
  Geom g = make_geom(shape);
  const bool makes_do = !static_scratch || (shape->dtype == STAR_ATTN_BF16 && few_rows(g, (int64_t)g.G * q_len, total));
  if (makes_do && workspace_bytes < plan_bytes(shape, plan, q_len) &&
      !make_plan(shape, q_len, total, O_part != nullptr, &plan, (int64_t)workspace_bytes))
    return STAR_ATTN_ERR_INVALID_SHAPE;
  if (workspace_bytes < plan_bytes(shape, plan, q_len)) return STAR_ATTN_ERR_WORKSPACE_TOO_SMALL;
  if ((int64_t)g.B * plan.s_total * ((q_len + 31) / 32) * g.Hq > (int64_t)0x7fffffff)
    return STAR_ATTN_ERR_INVALID_SHAPE;
  if (static_scratch) {
    // the current device's copy of the static array (its address was looked up
    // once, with that device current)
    DeviceState* ds = device_state();
    if (!ds) return STAR_ATTN_ERR_LAUNCH_FAILED;
    workspace = ds->scratch_ptr;
  }
  hipStream_t st = (hipStream_t)hip_stream;

  // Algorithm 2: the new tokens' K/V join the cache before they attend.  The
  // attention kernels append them themselves (they read the new rows from Kq/Vq and
  // write them to the cache).  Unrotated keys are rotated into the cache first.
  // (A few rotated tokens on the decode kernel's equal runs are turned there, and by the merge.  Not where O is
  // stored over Qq, which one launch would both merge into and rotate, nor where Kq are rows of the cache, which
  // would be read behind their rotation.)
  const size_t q_bytes = (size_t)g.B * q_len * g.Hq * g.d * 2, k_bytes = (size_t)g.B * q_len * g.Hkv * g.d * 2;
  const bool turn = append && rope && plan.decode && plan.flat && g.G * q_len <= 16 && q_len <= DECODE_ROPE_TOKENS &&
                    (int64_t)g.B * g.Hq * q_len <= (1 << 20) && !overlap(O, q_bytes, Qq, q_bytes) &&
                    !overlap(Kq, k_bytes, K_cache, (size_t)g.B * g.Hkv * g.cap * g.d * 2);
  const bool fused_append = append && (!rope || turn);
  if (append && rope && !turn &&
      launch_rope(shape->dtype, g, g.Hq, Qq, Qq, Kq, Vq, K_cache, V_cache, q_len, cache_len,
                  rope->pos0 + cache_len, rope->theta, nullptr, st) != hipSuccess)
    return STAR_ATTN_ERR_LAUNCH_FAILED;

  size_t rows = (size_t)g.B * plan.s_total * g.Hq * (size_t)q_len;
  Phase2Args a;
  a.g = g; a.plan = plan; a.cache_len = cache_len; a.q_len = (int32_t)q_len;
  a.causal = append ? 1 : 0;
  a.Qq = Qq; a.Kc = K_cache; a.Vc = V_cache;
  a.Kn = fused_append ? Kq : nullptr;
  a.Vn = fused_append ? Vq : nullptr;
  a.O_sub = (float*)workspace;
  a.LSE_sub = (float*)workspace + rows * g.d;
  const bool direct = shape->dtype == STAR_ATTN_F32 && plan.flat && plan.s_total == 1;
  a.O = direct && !pair ? O : nullptr;
  a.A = direct && pair ? A : nullptr;
  a.LSE = direct && pair ? LSE : nullptr;
  a.rotary = Rotary{turn ? log2(rope->theta) : 0.0, turn ? rope->pos0 + cache_len : 0};
  hipError_t e;
  if (shape->dtype == STAR_ATTN_F32) e = launch_phase2_f32(a, st);
  else if (plan.decode) e = launch_phase2_decode_bf16(a, st);
  else e = launch_phase2_rows_bf16(a, st);
  if (e != hipSuccess) return STAR_ATTN_ERR_LAUNCH_FAILED;
  if (direct) return STAR_ATTN_OK;

  MergeArgs m;
  m.g = g; m.plan = plan;
  // Without per-part outputs the splits of all parts are merged at once, whatever they were cut along: part
  // by part it is a chain of round trips.  us (8 / 2 heads), part by part / at once: 21 tokens on 16384 keys in blocks of
  // 2048 34.7 / 19.4, of 256 73.4 / 19.7, 84 on 4096 in blocks of 1024 23.7 / 18.6, 64 on 1024 in blocks of 256 18.5 / 14.8;
  // 23 on 2048 (32 / 8 heads) 20.2 / 16.2.  The sums are held in 64 bits, as merge part by part compensates its own (in
  // 32 bits: 18.3, 18.4, 18.1, 14.4, 15.7).  (The kernels of one part number a row's pieces in one launch.)
  m.wide = 0;
  if (!O_part && !plan.flat && (int64_t)g.B * g.Hq * q_len < (1 << 22)) { m.plan.flat = 1; m.wide = 1; }
  m.q_len = (int32_t)q_len; m.out_bf16 = shape->dtype == STAR_ATTN_BF16;
  m.O_sub = a.O_sub; m.LSE_sub = a.LSE_sub; m.O_part = O_part; m.LSE_part = LSE_part;
  m.batch_stride = (int64_t)plan.s_total * g.Hq * q_len;
  m.split_stride = (int64_t)g.Hq * q_len;
  m.O = pair ? nullptr : O;
  m.A = pair ? A : nullptr;
  m.LSE = pair ? LSE : nullptr;
  m.Qq = Qq;
  m.rotary = a.rotary;
  return launch_merge(m, st) == hipSuccess ? STAR_ATTN_OK : STAR_ATTN_ERR_LAUNCH_FAILED;
}

extern "C" {

int star_attn_phase2(const star_attn_shape* shape, int64_t cache_len, int64_t q_len,
                     const void* Qq, const void* Kq, const void* Vq,
                     void* K_cache, void* V_cache, float* O_part, float* LSE_part, void* O,
                     void* workspace, size_t workspace_bytes, void* hip_stream) {
  return phase2_impl(shape, nullptr, cache_len, q_len, const_cast<void*>(Qq), Kq, Vq, K_cache,
                     V_cache, O_part, LSE_part, O, false, nullptr, nullptr, workspace,
                     workspace_bytes, hip_stream);
}

int star_attn_phase2_static(const star_attn_shape* shape, int64_t cache_len, int64_t q_len,
                            const void* Qq, const void* Kq, const void* Vq, void* K_cache,
                            void* V_cache, void* O, void* hip_stream) {
  return phase2_impl(shape, nullptr, cache_len, q_len, const_cast<void*>(Qq), Kq, Vq, K_cache,
                     V_cache, nullptr, nullptr, O, false, nullptr, nullptr, nullptr, 0, hip_stream,
                     /*static_scratch=*/true);
}

int star_attn_phase2_partial(const star_attn_shape* shape, int64_t cache_len, int64_t q_len,
                             const void* Qq, const void* Kq, const void* Vq, void* K_cache,
                             void* V_cache, float* A, float* LSE, void* workspace,
                             size_t workspace_bytes, void* hip_stream) {
  if ((Kq == nullptr) != (Vq == nullptr)) return STAR_ATTN_ERR_NULL_POINTER;
  return phase2_impl(shape, nullptr, cache_len, q_len, const_cast<void*>(Qq), Kq, Vq, K_cache,
                     V_cache, nullptr, nullptr, nullptr, true, A, LSE, workspace, workspace_bytes,
                     hip_stream);
}

int star_attn_merge(const star_attn_shape* shape, int64_t n_parts, int64_t q_len,
                    const float* A_parts, const float* LSE_parts, void* O, float* A, float* LSE,
                    void* hip_stream) {
  int rc = validate_shape(shape);
  if (rc != STAR_ATTN_OK) return rc;
  if (n_parts <= 0 || n_parts > (1 << 20) || q_len <= 0 || q_len > (1 << 20))
    return STAR_ATTN_ERR_INVALID_SHAPE;
  if (!A_parts || !LSE_parts || (!O && !A)) return STAR_ATTN_ERR_NULL_POINTER;
  if (misaligned(A_parts) || ((uintptr_t)LSE_parts & 3u) || misaligned(O) || misaligned(A) ||
      ((uintptr_t)LSE & 3u))
    return STAR_ATTN_ERR_MISALIGNED;
  Geom g = make_geom(shape);
  const int64_t rows = (int64_t)g.B * g.Hq * q_len;
  if (rows > (int64_t)0x7fffffff || rows * n_parts > ((int64_t)1 << 40)) return STAR_ATTN_ERR_INVALID_SHAPE;
  MergeArgs m;
  m.g = g;
  m.plan = SplitPlan{0, 0, 0, 0, (int32_t)n_parts, 0, 1, 0, 0};    // one part made of n_parts splits
  m.q_len = (int32_t)q_len;
  m.out_bf16 = shape->dtype == STAR_ATTN_BF16;
  m.O_sub = A_parts; m.LSE_sub = LSE_parts;
  m.batch_stride = (int64_t)g.Hq * q_len;                    // [n_parts, B, Hq, q_len, d]
  m.split_stride = rows;
  m.O_part = nullptr; m.LSE_part = nullptr;
  m.O = O; m.A = A; m.LSE = LSE;
  m.Qq = nullptr; m.rotary = Rotary{0.0, 0}; m.wide = 0;
  return launch_merge(m, (hipStream_t)hip_stream) == hipSuccess ? STAR_ATTN_OK
                                                                : STAR_ATTN_ERR_LAUNCH_FAILED;
}

int star_attn_phase2_rope(const star_attn_shape* shape, double rope_theta, int64_t pos0,
                          int64_t cache_len, int64_t q_len, void* Qq, const void* Kq,
                          const void* Vq, void* K_cache, void* V_cache, float* O_part,
                          float* LSE_part, void* O, void* workspace, size_t workspace_bytes,
                          void* hip_stream) {
  Rope rope = {rope_theta, pos0};
  return phase2_impl(shape, &rope, cache_len, q_len, Qq, Kq, Vq, K_cache, V_cache, O_part,
                     LSE_part, O, false, nullptr, nullptr, workspace, workspace_bytes, hip_stream);
}

const char* star_attn_status_string(int status) {
  switch (status) {
    case STAR_ATTN_OK: return "ok";
    case STAR_ATTN_ERR_INVALID_SHAPE: return "invalid shape";
    case STAR_ATTN_ERR_NULL_POINTER: return "required pointer is NULL";
    case STAR_ATTN_ERR_UNSUPPORTED_HEAD_DIM: return "unsupported head_dim";
    case STAR_ATTN_ERR_UNSUPPORTED_DTYPE: return "unsupported dtype";
    case STAR_ATTN_ERR_ANCHOR_GT_BLOCK: return "anchor outside [0, block]";
    case STAR_ATTN_ERR_CACHE_OVERFLOW: return "cache capacity exceeded";
    case STAR_ATTN_ERR_WORKSPACE_TOO_SMALL:
      return "workspace too small (star_attn_phase2_static: the call needs more than the static scratch)";
    case STAR_ATTN_ERR_LAUNCH_FAILED: return "kernel launch failed";
    case STAR_ATTN_ERR_MISALIGNED: return "pointer not sufficiently aligned";
    case STAR_ATTN_ERR_INVALID_MODE: return "unknown anchor mode";
    case STAR_ATTN_ERR_BUSY:
      return "no workspace given and the library's own work-queue counters are all in flight "
             "(or the stream is being captured)";
    default: return "unknown status";
  }
}

int star_attn_phase2_plan(const star_attn_shape* shape, int64_t cache_len, int64_t q_len,
                          int want_parts, star_attn_plan_info* out) {
  int rc = validate_shape(shape);
  if (rc != STAR_ATTN_OK) return rc;
  if (!out) return STAR_ATTN_ERR_NULL_POINTER;
  if (q_len <= 0 || q_len > (1 << 20) || cache_len < shape->ctx_len) return STAR_ATTN_ERR_INVALID_SHAPE;
  const int64_t total = cache_len + q_len;
  if (total > shape->cache_capacity) return STAR_ATTN_ERR_CACHE_OVERFLOW;
  SplitPlan plan;
  if (!make_plan(shape, q_len, total, want_parts != 0, &plan)) return STAR_ATTN_ERR_INVALID_SHAPE;
  const bool resident = decode_cache_resident(make_geom(shape), total);
  out->decode = plan.decode;
  out->flat = plan.flat;
  out->n_splits = plan.s_total;
  out->non_temporal = plan.decode && !resident ? 1 : 0;
  out->steps_per_batch = plan.decode ? (resident ? 1 : 2) : 0;
  out->tile_rows = plan.tile_rows;
  out->split_len = plan.split_len;
  out->workspace_bytes = (int64_t)plan_bytes(shape, plan, q_len);
  return STAR_ATTN_OK;
}

int star_attn_phase1_plan(const star_attn_shape* shape, int anchor_mode, star_attn_phase1_plan_info* out) {
  int rc = validate_shape(shape);
  if (rc != STAR_ATTN_OK) return rc;
  if (!known_mode(anchor_mode)) return STAR_ATTN_ERR_INVALID_MODE;
  if (!out) return STAR_ATTN_ERR_NULL_POINTER;
  const Geom g = make_geom(shape);
  const Phase1Plan p = shape->dtype == STAR_ATTN_F32 ? phase1_plan_f32(g) : phase1_plan_bf16(g, anchor_mode, device_cu_count());
  out->queued = p.queued;
  out->tile_rows = p.rows;
  out->wavefronts = p.waves;
  out->group = p.group;
  out->n_tiles = p.tiles;
  return STAR_ATTN_OK;
}

const char* star_attn_kernel_path(const star_attn_shape* shape) {
  if (validate_shape(shape) != STAR_ATTN_OK) return nullptr;
  return shape->dtype == STAR_ATTN_F32 ? "f32-valu" : "bf16-mfma";
}

}  // extern "C"
