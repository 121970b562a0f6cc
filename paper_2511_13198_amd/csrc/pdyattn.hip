// C-ABI of the pdyattn library: argument validation, workspace carving and
// kernel launches.  Declarations and the contract live in include/pdyattn.h.
#include "../../include/pdyattn.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <vector>

#include "bwd.hpp"
#include "fwd.hpp"
#include "plan.hpp"

namespace {

thread_local char g_err[512] = "";

pdy_status fail(pdy_status st, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return st;
}

pdy_status hip_fail(hipError_t e, const char* what) {
  return fail(PDY_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

// Smallest tile of a launch that can be large, which bounds the work items (the
// 64-row tiles of four key groups are only for launches of under kManyItems
// workgroups of larger ones).
constexpr int kTile = 128;

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

struct Sizes {
  int64_t T, N, maxlen, hq, hkv, d;
};

int tiles_of(const Sizes& s, int tile) {
  const int64_t n = (s.maxlen + tile - 1) / tile;
  return n < 1 ? 1 : (int)n;
}

// forward and dQ workgroup size: 8 waves (256 query rows, 128-key tiles, one
// workgroup per CU) unless every segment has at most kShortSeg tokens; then
// 4 waves (128 rows, 64-key tiles, two workgroups per CU), whose smaller
// items and diagonal tiles outweigh their extra barriers there (measured
// fwd+bwd: 1K-2K tokens 7-12 % faster, 4K and longer 3-15 % slower)
#ifndef PDY_WAVES_LONG
#define PDY_WAVES_LONG 8
#endif
constexpr int64_t kShortSeg = 2048;
int fwd_waves(const Sizes& s) { return s.maxlen > kShortSeg ? PDY_WAVES_LONG : 4; }

// How a launch's workgroups are made up: nw waves in `groups` key groups (forward
// and dQ, 32 * nw / groups query rows each) or query groups (dK/dV, as many keys).
struct Shape {
  int nw;
  int groups;
  int tile() const { return 32 * nw / groups; }
};

pdy_status check_sizes(int32_t T, int32_t N, int32_t maxlen, int32_t hq, int32_t hkv, int32_t d,
                       Sizes* out) {
  if (T < 0) return fail(PDY_ERR_INVALID_ARG, "total_tokens must be >= 0 (got %d)", T);
  if (N < 1) return fail(PDY_ERR_INVALID_ARG, "num_seqs must be >= 1 (got %d)", N);
  if (maxlen < 0 || maxlen > T)
    return fail(PDY_ERR_INVALID_ARG, "max_seqlen must be in [0, total_tokens] (got %d, T=%d)",
                maxlen, T);
  if (T > 0 && maxlen < 1)
    return fail(PDY_ERR_INVALID_ARG, "max_seqlen must be >= 1 when total_tokens > 0");
  // one segment spans [0, T) by the contract, and a single-segment call
  // builds no tile schedule but sizes its grid from max_seqlen: anything
  // other than T would leave rows unwritten (or visit rows past the end)
  if (N == 1 && maxlen != T)
    return fail(PDY_ERR_INVALID_ARG,
                "with num_seqs = 1 max_seqlen must equal total_tokens (got %d, T=%d)", maxlen, T);
  if (hq < 1 || hkv < 1)
    return fail(PDY_ERR_INVALID_ARG, "head counts must be >= 1 (got Hq=%d, Hkv=%d)", hq, hkv);
  if (hq % hkv != 0)
    return fail(PDY_ERR_INVALID_ARG, "num_heads_q (%d) must be a multiple of num_heads_kv (%d)",
                hq, hkv);
  if (d != 64 && d != 128)
    return fail(PDY_ERR_UNSUPPORTED, "head_dim %d not supported (64 or 128)", d);
  // element offsets are computed in 64 bits; keep T*H*d well inside that and
  // the grid (items x heads) inside 2^31 blocks
  const int64_t items = (int64_t)T / kTile + N;
  if (items * hq >= (int64_t)1 << 31)
    return fail(PDY_ERR_INVALID_ARG, "problem too large for one launch");
  out->T = T;
  out->N = N;
  out->maxlen = maxlen;
  out->hq = hq;
  out->hkv = hkv;
  out->d = d;
  return PDY_OK;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// ---------------------------------------------------------------------------
// Optional per-thread kernel timing: while enabled, every launch is bracketed
// by two events on its own stream; pdy_profile_stop reduces them per kernel.
// ---------------------------------------------------------------------------
enum KernelId { K_PLAN = 0, K_FWD, K_DKDV, K_DQ, K_SPLIT_MERGE, K_SPLIT_SUM, K_COUNT };
const char* const kKernelNames[K_COUNT] = {"plan_kernel",     "fwd_kernel",
                                           "bwd_dkdv_kernel", "bwd_dq_kernel",
                                           "split_merge_kernel", "split_sum_kernel"};
struct ProfRec {
  int kid;
  hipEvent_t a, b;
};
thread_local bool g_prof_on = false;
thread_local std::vector<ProfRec> g_prof_recs;
thread_local std::vector<hipEvent_t> g_prof_pool;

hipError_t prof_event(hipEvent_t* ev) {
  if (!g_prof_pool.empty()) {
    *ev = g_prof_pool.back();
    g_prof_pool.pop_back();
    return hipSuccess;
  }
  return hipEventCreate(ev);
}

// Launch through `fn` (which enqueues exactly one kernel on `st`), timing it
// when profiling is on.  Returns the launch error, if any.
template <typename F>
hipError_t launch_timed(int kid, hipStream_t st, F fn) {
  if (!g_prof_on) {
    fn();
    return hipGetLastError();
  }
  ProfRec r;
  r.kid = kid;
  hipError_t e = prof_event(&r.a);
  if (e == hipSuccess) e = prof_event(&r.b);
  if (e == hipSuccess) e = hipEventRecord(r.a, st);
  if (e != hipSuccess) return e;
  fn();
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = hipEventRecord(r.b, st);
  if (e == hipSuccess) g_prof_recs.push_back(r);
  return e;
}

size_t plan_bytes(const Sizes& s, int tile) {
  return align256(pdy::plan_ints((int)s.N, tiles_of(s, tile)) * 4);
}

size_t dd_bytes(const Sizes& s) { return align256((size_t)s.hq * (size_t)s.T * 4); }

// upper bound on sum_i ceil(len_i / tile) (the number of work items)
int64_t grid_items(const Sizes& s, int tile) {
  const int64_t bound1 = s.T / tile + s.N;
  const int64_t bound2 = s.N * (int64_t)tiles_of(s, tile);
  return bound1 < bound2 ? bound1 : bound2;
}

// Split-K.  A launch whose work items cannot fill the chip (fewer than
// kFillItems workgroups, two per CU) can cut every item's inner loop -- the
// key tiles of a query tile (forward, dQ) or the query steps of a key tile
// (dK/dV) -- into 2 or 4 parts, one workgroup each; the parts' fp32 partial
// results are then combined.  Otherwise the heaviest item alone sets the
// launch's time (a 16K-token sequence over 4 heads has 256 forward items, the
// last of which visits every key).  Splitting shortens the heaviest item by
// (inner - inner/p) tiles but writes and reads back p partial results, so it
// is taken only while that saves time by the estimate below: a tile's time
// from the kernels' measured throughput per CU (≈ 4.5 TFLOP/s forward and
// dK/dV, ≈ 5 dQ), the partial traffic at ≈ 4 TB/s, plus one launch.  The
// decision depends on the sizes alone (balanced_split below also on the
// causal flag), so the workspace queries reproduce it; partial buffers exist
// only for launches this small (parts x items < 2 kFillItems, or at most
// kMaxParts slices of a balanced split of fewer than kCUs workgroups).
constexpr int64_t kFillItems = 512;
constexpr int kMaxSplit = 4;
constexpr double kPartBytesPerUs = 4.0e6;  // partial results written + read back
constexpr double kLaunchUs = 4.0;          // the combining kernel

// inner: tiles of the heaviest item; tile_us: time of one tile; part_bytes:
// bytes of one part's partial results
int split_parts(int64_t items, int64_t inner, double tile_us, double part_bytes) {
  auto saved = [&](int p) {  // estimated time saved by p parts (p = 1: none)
    if (p == 1) return 0.0;
    const int64_t left = (inner + p - 1) / p;
    return (double)(inner - left) * tile_us - (2.0 * p * part_bytes / kPartBytesPerUs + kLaunchUs);
  };
  int p = 1;
  while (p < kMaxSplit && items * p < kFillItems && inner >= 4 * p && saved(2 * p) > saved(p))
    p *= 2;
  return p;
}

int fwd_key_tile(const Sizes& s, const Shape& sh) {
  if (sh.groups > 1) return pdy::FwdCfg<128, 8, 2>::BK;
  if (s.d == 64) return sh.nw == 8 ? pdy::FwdCfg<64, 8>::BK : pdy::FwdCfg<64, 4>::BK;
  return sh.nw == 8 ? pdy::FwdCfg<128, 8>::BK : pdy::FwdCfg<128, 4>::BK;
}

int dq_key_tile(const Sizes& s, const Shape& sh) {
  if (s.d == 64) return sh.nw == 8 ? pdy::DqCfg<64, 8>::BK : pdy::DqCfg<64, 4>::BK;
  return sh.nw == 8 ? pdy::DqCfg<128, 8>::BK : pdy::DqCfg<128, 4>::BK;
}

// microseconds for one CU to process `pairs` (query, key) pairs of one head
// with `flops_per_pair_d` x d FLOPs each at `tflops` per CU
double tile_us(double pairs, const Sizes& s, double flops_per_pair_d, double tflops) {
  return pairs * flops_per_pair_d * (double)s.d / (tflops * 1e6);
}

// A split of `p` parts per item (p = 1: none).
pdy::Split uniform_split(int p) {
  pdy::Split sp{};
  sp.parts = p;
  sp.cap = 0;
  sp.rows = sp.keys = sp.group = 1;
  return sp;
}

constexpr int64_t kCUs = 256;  // compute units of the chip
constexpr int kMaxParts = 16;  // partial slices of a balanced split at most

// Balanced split-K of a causal single-segment launch whose uniform split
// takes p > 1 parts per item.  Under the causal mask the items' units range
// from one to the heaviest item's, so equal part counts leave the heaviest
// item's parts (which set the launch's time) several times the mean part; a
// balanced split gives the heaviest items more parts and light items fewer.
// It is taken only when the uniform split's workgroups fit one round on the
// chip (one per CU): over two rounds the uniform parts, dealt heaviest first,
// already pair a heavy part with a light one on each CU, which balanced parts
// (ordered by item, not by size) do not (8K tokens x 4 heads: 607 against 567
// TFLOP/s).  For a budget of workgroups (over the heads) the smallest cap
// (units per part) that fits it is found by bisection (O(items log units) on
// the host; items < 256 here), with at most kMaxParts slices.  Two budgets
// are tried, the uniform split's workgroup count and one workgroup per CU,
// and the one with the lower estimated time is kept: the heaviest part or the
// mean load per CU, whichever is larger, at unit_us per unit, plus the
// partial results written and read back (slice_bytes for all items of all
// heads) at the rate the uniform split assumes.  `shape` gives kind, nitems,
// total, causal, rows, keys and group.
pdy::Split balanced_split(pdy::Split shape, int p, int64_t heads, double unit_us,
                          double slice_bytes) {
  if ((int64_t)p * shape.nitems * heads > kCUs) return uniform_split(p);
  int units[kCUs];  // (nitems <= kCUs by the line above)
  int64_t total_units = 0;
  for (int i = 0; i < shape.nitems; ++i) total_units += units[i] = shape.units(i);
  const int umax = units[0];  // item 0 is the heaviest
  const double mean_load = (double)total_units * heads / kCUs;
  auto entries = [&](int cap) {
    int64_t n = 0;
    for (int i = 0; i < shape.nitems; ++i) n += (units[i] + cap - 1) / cap;
    return n * heads;
  };
  auto cap_for = [&](int64_t budget) {
    int lo = std::max(1, (umax + kMaxParts - 1) / kMaxParts), hi = umax;  // umax: one part each
    while (lo < hi) {
      const int mid = (lo + hi) / 2;
      if (entries(mid) <= budget) hi = mid;
      else lo = mid + 1;
    }
    return lo;
  };
  auto est_us = [&](int cap) {
    const double parts_bytes = (double)entries(cap) * slice_bytes / ((double)shape.nitems * heads);
    return std::max((double)cap, mean_load) * unit_us + 2.0 * parts_bytes / kPartBytesPerUs;
  };
  const int64_t b1 = (int64_t)p * shape.nitems * heads;
  int cap = cap_for(b1);
  if (b1 < kCUs) {
    const int cap2 = cap_for(kCUs);
    if (est_us(cap2) < est_us(cap)) cap = cap2;
  }
  shape.cap = cap;
  shape.parts = (umax + cap - 1) / cap;
  return shape.parts > 1 ? shape : uniform_split(1);
}

// workgroups per head of a launch of `items` items (per head) under split sp
int64_t split_entries(const pdy::Split& sp, int64_t items) {
  if (sp.cap == 0) return items * sp.parts;
  int64_t n = 0;
  for (int i = 0; i < sp.nitems; ++i) n += sp.nparts(i);
  return n;
}

// The same split with about half the partial slices (for a fixed-size
// workspace); parts = 1 when nothing is left to split.
pdy::Split halve_split(pdy::Split sp) {
  if (sp.cap == 0) return uniform_split(sp.parts / 2);
  sp.cap *= 2;
  sp.parts = (sp.units(0) + sp.cap - 1) / sp.cap;
  return sp.parts > 1 ? sp : uniform_split(1);
}

// A launch: its workgroups' shape and its split.
struct Launch {
  Shape sh;
  pdy::Split split;
};

// What the choice of a launch looks at: rows of queries over rows of keys, sq
// and sk (one chunk each, `shift` apart, for a context-parallel pair, of which
// `launches` run at a time; the same segments otherwise).
struct Job {
  const Sizes &sq, &sk;
  int causal;
  bool chunk;
  int shift;
  int launches = 1;  // chunk pairs at a time
};

enum Which { FWD, DQ, DKDV };

// One key group (query group) per workgroup: the shape of every launch that
// fills the chip.
Shape base_shape(Which k, const Sizes& sq) {
  return {k == DKDV ? pdy::DkdvCfg<128>::NW : fwd_waves(sq), 1};
}

// A launch's work in one shape: items per head, the heaviest item's units of
// inner work, the estimated time of a unit, the bytes of a partial slice.
struct Work {
  pdy::Split shape;  // for a balanced split
  int64_t items, heads, inner;
  double unit_us, slice;
};
Work work_of(Which k, const Job& j, const Shape& sh) {
  Work w;
  const int tile = sh.tile();
  w.shape = uniform_split(1);
  w.shape.causal = j.causal;
  if (k == DKDV) {
    // the heaviest key tile visits every 64-row query step of every head of
    // its group
    const int rows = pdy::DkdvCfg<128>::BQ, g = (int)(j.sq.hq / j.sq.hkv);
    w.items = grid_items(j.sk, tile);
    w.heads = j.sk.hkv;
    w.inner = (int64_t)tiles_of(j.sq, rows) * g;
    w.unit_us = tile_us((double)rows * tile, j.sq, 8.0, 4.5);
    w.slice = 2.0 * j.sk.T * j.sk.hkv * j.sk.d * 4;
    w.shape.kind = 1;
    w.shape.nitems = tiles_of(j.sk, tile);
    w.shape.total = (int)j.sk.T;
    w.shape.rows = rows;
    w.shape.keys = tile;
    w.shape.group = g;
  } else {
    const int keys = k == FWD ? fwd_key_tile(j.sq, sh) : dq_key_tile(j.sq, sh);
    w.items = grid_items(j.sq, tile);
    w.heads = j.sq.hq;
    w.inner = tiles_of(j.sk, keys);
    w.unit_us = k == FWD ? tile_us((double)tile * keys, j.sq, 4.0, 4.5)
                         : tile_us((double)tile * keys, j.sq, 6.0, 5.0);
    w.slice = (double)j.sq.T * j.sq.hq * j.sq.d * 4;
    w.shape.kind = 0;
    w.shape.nitems = tiles_of(j.sq, tile);
    w.shape.total = (int)j.sq.T;
    w.shape.rows = tile;
    w.shape.keys = keys;
  }
  return w;
}

// p parts per item, balanced for causal single segments.
pdy::Split split_of(const Work& w, const Job& j, int p) {
  // (a split launch has fewer than 512 items, so a slice holds far fewer than
  // the 2^31 floats the combine kernels index with 32 bits; kept as a guard)
  if (j.sk.T == 0 || w.slice / 4 >= 2147483648.0) return uniform_split(1);
  if (j.sq.N == 1 && j.causal && !j.chunk)
    return balanced_split(w.shape, p, w.heads, w.unit_us, w.slice);
  return uniform_split(p);
}

// The launch in the base shape: no split for a context-parallel pair.
Launch base_launch(Which k, const Job& j) {
  const Shape sh = base_shape(k, j.sq);
  const Work w = work_of(k, j, sh);
  const int p = split_parts(w.items * w.heads, w.inner, w.unit_us, w.slice);
  return {sh, p <= 1 || j.chunk ? uniform_split(1) : split_of(w, j, p)};
}

// Estimated time of an unsplit launch over one segment or chunk pair, by
// which its number of groups is chosen.  A unit is a workgroup's time on 128
// keys (forward, dQ) or 64 rows (dK/dV), as measured at d = 128 on a chip that
// is about full; with 1, 2 and 4 groups a unit covers 256, 128 and 64 rows (or
// 256 and 128 keys), so groups cost 6-9 % (two) and 20-40 % (four) of the rate
// and pay where they fill idle CUs or even out the causal ramp:
//   8,192 queries x 8,192 earlier keys, 1 head: forward 183 / 105 / 76 us with
//     1 / 2 / 4 groups, dQ 229 / 130 / 84, dK/dV 325 / 185;
//   16,384 x 16,384 of the diagonal, 4 heads: 415 / 273 / 340, 560 / 361 / 404,
//     770 / 490; the same not causal: 465 / 502 / 650, 643 / 680 / 770, 880 / 931;
//   512 tokens x 8 heads of 64 (4-wave base): forward 12.1 / 10.6 / 8.2 us.
double est_unsplit_us(Which k, const Job& j, const Shape& sh) {
  static constexpr double kUnit[3][3] = {{3.4, 1.85, 1.2}, {4.6, 2.45, 1.45}, {3.2, 1.72, 0}};
  constexpr double kWorkgroupUs = 5.0;  // a workgroup's start and end
  const int tile = sh.tile();
  const bool kv = k == DKDV;
  const Sizes &mine = kv ? j.sk : j.sq, &other = kv ? j.sq : j.sk;
  const int64_t heads = kv ? j.sk.hkv : j.sq.hq, g = kv ? j.sq.hq / j.sq.hkv : 1;
  const int step_log2 = kv ? 6 : 7;
  const int64_t round_up = (1 << step_log2) - 1, n = tiles_of(mine, tile);
  int64_t total = 0, most = 0, least = INT64_MAX;
  if (!j.causal) {
    most = least = ((other.T + round_up) >> step_log2) * g;
    total = n * most;
  }
  for (int64_t i = 0; j.causal && i < n; ++i) {
    // rows or keys that the tile visits
    const int64_t seen =
        kv ? other.T - std::min(other.T, std::max<int64_t>(0, i * tile - j.shift))
           : std::max<int64_t>(0, std::min(other.T, (i + 1) * tile + j.shift));
    const int64_t u = ((seen + round_up) >> step_log2) * g;
    total += u;
    most = std::max(most, u);
    least = std::min(least, u);
  }
  const double rounds = (double)(n * heads) / kCUs, whole = std::ceil(rounds);
  // heaviest first over the CUs: the mean load, plus a light item in the last
  // round where it is not full
  const double units = std::max((double)most, (double)total * heads / kCUs + (whole - rounds) * least);
  // (a 4-wave workgroup alone on its CU: half the rows of an 8-wave one)
  const double unit = sh.nw == 4 ? 0.6 * kUnit[k][0] : kUnit[k][sh.groups / 2];
  return whole * kWorkgroupUs + units * unit * (j.sq.d == 64 ? 0.7 : 1.0);
}

// What two groups of half as many parts save in partial results (and the
// combining launch where none are left), as a share of a split launch's time.
double saved_share(const Launch& base, const Work& w, const Job& j) {
  constexpr double kMovedBytesPerUs = 5.0e6;
  const int p = split_parts(w.items * w.heads, w.inner, w.unit_us, w.slice);
  const double longest = base.split.cap ? base.split.cap : (double)((w.inner + p - 1) / p);
  const double mean = (double)(w.items * w.heads) / kCUs * w.inner * (j.causal ? 0.5 : 1.0);
  return (p * w.slice / kMovedBytesPerUs + (p == 2 ? kLaunchUs : 0.0)) /
         (std::max(longest, mean) * w.unit_us);
}

constexpr int64_t kAverageShort = 512;

// launches of this many workgroups fill the chip in any shape
constexpr int64_t kManyItems = 1024;

// The launch for a job; `base`: that of base_launch, which a small workspace gets.
Launch pick(Which k, const Job& j, const Launch& base) {
  const Work w = work_of(k, j, base.sh);
  const int64_t n = w.items * w.heads;
  auto shape = [&](int groups) { return Shape{8, groups}; };
  // d = 64, causal, a little more than one round of 8-wave query-tile workgroups
  // (two fit a CU, but the causal ramp leaves the second half-empty): 4-wave
  // ones, three or four of which fit a CU, even it out.  10,153 tokens x 2/1 heads
  // (320 workgroups) forward 60 -> 54 us, dQ 73 -> 62; 16,384 x 8 (512) 377 -> 347
  // and 457 -> 415; with 1,024 dQ loses (1.42 -> 1.50 ms), with 256 both do, and
  // unsplit dQ from about two rounds on (38,243 x 4, 600 workgroups, 2.6 -> 2.7 ms;
  // with six heads or more from 2.5).
  // Packed batches (150 random ones each): with six heads or more forward 1.10x,
  // dQ 1.06x, 2 of 106 slower (by 4-5 %); with fewer, whose K/V the eight L2s
  // share, the tiles' second copy of K and V costs up to 14 % of a launch in parts
  // or of more than 448 workgroups (8 x 4,096 x 4 heads forward 130 -> 134 us, 5 x
  // 8,192 x 4 dQ 308 -> 322), while smaller unsplit ones gain (37, 1.0-1.31x).
  if (k != DKDV && j.sq.d == 64 && j.causal && !j.chunk && base.sh.nw == 8 && !base.split.cap) {
    const int parts = base.split.parts;
    const int64_t wgs = n * parts;
    const Shape four{4, 1};
    const bool heads = j.sq.hq >= 6;
    const bool evens =
        j.sq.N == 1 ? k == FWD || parts > 1 || wgs <= (heads ? kCUs * 5 / 2 : 2 * kCUs)
                    : heads || (parts == 1 && wgs <= kCUs * 7 / 4);
    if (evens && wgs > kCUs && wgs < (parts > 1 ? 2 : 3) * kCUs) return {four, base.split};
  }
  if (j.sq.N > 1) {
    // Packed batches, dK/dV over 128-key tiles:
    //   * two 4-wave workgroups per CU where segments are short (on average, of
    //     at most 512 tokens) and fill the chip: 122 of 16-512 tokens, 32/8 heads
    //     190 -> 146 us, 420 of 16-119, 24/8 heads 192 -> 121, 70 of 16-107, 16
    //     heads of 64 21.8 -> 18.7; 32 or 64 equal ones of 512 unchanged, of 1,024
    //     0-15 % slower;
    //   * two query groups where 256-key tiles leave CUs idle.  Unsplit launches
    //     (53 random ones 1.20x, none slower): only while the 128-key workgroups
    //     fit one round and have a few steps each: one head, causal, 32 of 1,024
    //     tokens 51.5 -> 37.9 us (d = 64: 38.5 -> 29.8), 64 of 512 33.7 -> 29.3; but
    //     60 of 1,024 56 -> 74 (d = 64: 40 -> 56), 100 of 512 37 -> 41, 30 of 2,048
    //     without a mask 131 -> 142, 10 of up to 154 x 16 18 -> 22.  Two parts:
    //     always, without parts (47 random ones 1.27x): 16 of 2,048 74.8 -> 60.2,
    //     15 of 4,096 247 -> 222.  Four parts, with half as many: where the partial
    //     results' share of the time is at least 0.2 (d = 128: of 263 random ones
    //     124 1.07x, 8 slower, the rest would be 0.996x) or 0.3 (d = 64, whose
    //     products lose more: of 276, 86 1.04x, 11 slower), so mostly short segments
    //     with many rows: 11 of 16-103 tokens x 32/8 heads 50.9 -> 45.5, 42 of 30-828
    //     x 9/3 175 -> 158; 3 of 16,384 x 1 of 64 297 -> 315.  Not where the four
    //     parts fit two rounds and the two-group workgroups fill both as well (8 of
    //     3,961 x 1 0.86x).
    if (k != DKDV) return base;
    const Shape four{4, 1};
    if (j.sk.maxlen <= kShortSeg && j.sk.T <= kAverageShort * j.sk.N &&
        grid_items(j.sk, four.tile()) * w.heads >= 2 * kCUs)
      return {four, uniform_split(1)};
    if (n >= kCUs) return base;
    const Work w2 = work_of(k, j, shape(2));
    const int64_t n2 = w2.items * w2.heads;
    const int p = base.split.parts;
    if (p == 1 ? n2 > kCUs || w.inner < 4
               : p > 2 && (saved_share(base, w, j) < (j.sq.d == 64 ? 0.3 : 0.2) ||
                           (n <= kCUs / 2 && n2 >= kCUs * 7 / 8)))
      return base;
    return {shape(2), split_of(w2, j, std::max(1, p / 2))};
  }
  if (base.split.parts > 1) {
    // Two groups of half as many parts: as many workgroups and half the partial
    // results, but slower products, so where what is saved (partial results moved,
    // and the combining launch where none are left) is at least this share of the
    // kernel's time.  The shares are those from which on 1,200 random single
    // sequences, timed both ways, gain on the mean.  d = 128, all combining
    // included: 2,500 tokens x 6/2 heads backward 82 -> 73 us, 6,144 x 1 forward
    // 32.7 -> 28.7 and backward 77 -> 69, 8,192 x 4 92 -> 88 and 281 -> 266; below
    // the line 16,128 x 4 forward 283 -> 294, 16,314 x 2/1 dK/dV 247 -> 297.  d =
    // 64, whose one-group forward and dQ share a CU by two: 13,433 x 3 forward 101
    // -> 117 us, 11,282 x 4 97 -> 112; of two parts only where the causal ramp's
    // two rounds of two-group workgroups pair up (8,192 x 8, forward 113 -> 102,
    // 8,853 x 8 119 -> 121).  (Not for the 4-wave query-tile
    // kernels: no gain.)
    if (base.sh.nw == 4) return base;
    constexpr double kNever = 1e9;
    // [d = 64, 128][kernel][two parts, four, balanced]
    static constexpr double kShare[2][3][3] = {
        {{0, kNever, 0.12}, {0, kNever, 0.10}, {0.13, 0.25, 0.16}},
        {{0.11, 0.18, 0.17}, {0.05, 0.08, 0.08}, {0.05, 0.11, 0.05}}};
    const int p = split_parts(n, w.inner, w.unit_us, w.slice);
    if (saved_share(base, w, j) < kShare[j.sq.d == 128][k][p == 2 ? 0 : base.split.cap ? 2 : 1])
      return base;
    const Work w2 = work_of(k, j, shape(2));
    if (p == 2 && j.sq.d == 64 && k != DKDV &&
        (!j.causal || 10 * w2.items * w2.heads > 21 * kCUs))
      return base;
    return {shape(2), split_of(w2, j, p / 2)};
  }
  // a 4-wave launch that has a workgroup for every CU is left alone
  if (j.sk.T == 0 || n >= (base.sh.nw == 4 ? kCUs + 1 : kManyItems)) return base;
  // the diagonal crosses the tiles: their work ramps up
  const bool ramp = j.causal && j.shift < j.sk.T / 2;
  if (j.chunk) {
    // A pair whose two-group launch leaves half the chip idle or more is split
    // (by its sizes alone: its workspace query knows no offsets).  A
    // device's pairs of a zig-zag ring of 8 over 32,768 tokens x 4 heads (2,048
    // rows each): forward 0.78 -> 0.62 ms, backward 2.75 -> 1.52.  (Forward and dQ
    // over fewer than 1,280 keys: no parts, 34 pairs of 768-1,279 keys down to
    // 0.76x.)
    const Work w2 = work_of(k, j, shape(2));
    const int least = k == DKDV ? 8 : 10;
    int p = 1;
    while (p < kMaxSplit && w2.items * w2.heads * p * 2 <= kCUs &&
           w2.inner >= (p == 1 ? least : 8 * p))
      p *= 2;
    if (p > 1) return {shape(2), split_of(w2, j, p)};
    // Two pairs at a time fill each other's last rounds, and groups only cost their
    // rate, once two launches without groups fill the chip (d = 64: more than
    // fill, as two of its workgroups share a CU).  Ring of 8, zig-zag, 4 heads,
    // without / with groups: 131,072 tokens (8,192 rows, 128 workgroups) forward
    // 2.23 / 2.40 ms, 327,680 (320) 12.5 / 13.7, 638,976 (624) 47.2 / 51.0 and its
    // last device's backward 152 / 165; 98,304 (96) 1.56 / 1.50.  The pair over
    // the diagonal evens out its own ramp: with groups (contiguous, 131,072, the
    // second device 0.98 / 0.84).
    if (j.launches > 1 && !ramp && (j.sq.d == 64 ? n > kCUs : 2 * n >= kCUs)) return base;
  }
  if (k != DKDV) {
    // Key groups need a few keys each (up to 128 keys 7-15 % slower, from 256 on
    // faster: 140 random sequences).  Launches of more than a round whose items are
    // even: two of the d = 64 one-group workgroups share a CU, groups' do not (24
    // pairs and sequences 0.82-1.00x); nor do they pay for a forward over the
    // diagonal that is much more than a round (2,901 x 32 causal 77 -> 87 us, a
    // 13,542-row pair x 8 360 -> 379; up to 320 workgroups 1.03-1.39x).
    if (j.sk.T < 256) return base;
    if (j.sq.d == 64 && n > kCUs && !ramp) return base;
    if (j.sq.d == 128 && k == FWD && n > kCUs * 5 / 4 && ramp) return base;
  }
  Launch best = base;
  double t = 0.97 * est_unsplit_us(k, j, base.sh);
  // (8-wave dQ takes four groups only on half the chip: 128 to 312 workgroups
  // alone 0.96-0.99x, and 15 ms for 17 beside another pair.  4-wave ones keep
  // them up to a round: against two groups 1,789 tokens x 12 heads of 64 1.12x,
  // 1,104 x 16 1.06x, 2,048 x 16 1.00x, 1,024 x 32 0.94x.)
  const int most = k == DKDV || (k == DQ && base.sh.nw == 8 && 2 * n > kCUs) ? 2 : 4;
  for (int groups = 2; groups <= most; groups *= 2) {
    const double e = est_unsplit_us(k, j, shape(groups));
    if (e < t) {
      t = e;
      best.sh = shape(groups);
    }
  }
  return best;
}

size_t part_o_bytes(const Sizes& s, int p) { return align256((size_t)p * s.T * s.hq * s.d * 4); }
size_t part_lse_bytes(const Sizes& s, int p) { return align256((size_t)p * s.hq * s.T * 4); }
size_t part_kv_bytes(const Sizes& s, int p) { return align256((size_t)p * s.T * s.hkv * s.d * 4); }

// workspace for a split forward's partial O and LSE (none if it is not split)
size_t fwd_split_bytes(const pdy::Split& sp, const Sizes& sq) {
  return sp.parts > 1 ? part_o_bytes(sq, sp.parts) + part_lse_bytes(sq, sp.parts) : 0;
}

// workspace for a split backward's partial dK, dV (key rows) and dQ
size_t bwd_split_bytes(const pdy::Split& kv, const pdy::Split& q, const Sizes& sq,
                       const Sizes& sk) {
  return (kv.parts > 1 ? 2 * part_kv_bytes(sk, kv.parts) : 0) +
         (q.parts > 1 ? part_o_bytes(sq, q.parts) : 0);
}

// A single segment (N = 1: by the contract cu = [0, T], and max_seqlen = T)
// needs no schedule: item i is its level nt - 1 - i.
bool packed(const Sizes& s) { return s.N > 1; }

// Space of a launch's schedule; a single segment's is not used and has the size
// of the base shape's, so that its callers' workspaces do not depend on the shape.
size_t q_plan_bytes(const Sizes& s, const Shape& sh) {
  return plan_bytes(s, (packed(s) ? sh : base_shape(FWD, s)).tile());
}
size_t kv_plan_bytes(const Sizes& s, const Shape& sh) {
  return plan_bytes(s, (packed(s) ? sh : base_shape(DKDV, s)).tile());
}

// Workspace of a forward: schedule and any split-K partials.
size_t fwd_need(const Launch& l, const Sizes& sq) {
  return q_plan_bytes(sq, l.sh) + fwd_split_bytes(l.split, sq);
}

// Workspace of a backward without its split-K partials: both schedules and D
// (sk: sizes of the key side, the query side for self-attention), and with them.
size_t bwd_fixed(const Shape& kv, const Shape& q, const Sizes& sq, const Sizes& sk) {
  return kv_plan_bytes(sk, kv) + q_plan_bytes(sq, q) + dd_bytes(sq);
}
size_t bwd_need(const Launch& kv, const Launch& q, const Sizes& sq, const Sizes& sk) {
  return bwd_fixed(kv.sh, q.sh, sq, sk) + bwd_split_bytes(kv.split, q.split, sq, sk);
}

// What the workspace queries return: enough for the picked launches and for the
// base ones, causal or not.  (A chunk pair's split does not depend on its
// offsets.)
size_t fwd_workspace_bytes(const Sizes& sq, const Sizes& sk, bool chunk) {
  size_t n = 0;
  for (int causal = 0; causal <= 1; ++causal) {
    const Job j{sq, sk, causal, chunk, 0};
    const Launch base = base_launch(FWD, j);
    n = std::max({n, fwd_need(pick(FWD, j, base), sq), fwd_need(base, sq)});
  }
  return n;
}
size_t bwd_workspace_bytes(const Sizes& sq, const Sizes& sk, bool chunk) {
  size_t n = 0;
  for (int causal = 0; causal <= 1; ++causal) {
    const Job j{sq, sk, causal, chunk, 0};
    const Launch kv = base_launch(DKDV, j), q = base_launch(DQ, j);
    n = std::max({n, bwd_need(pick(DKDV, j, kv), pick(DQ, j, q), sq, sk),
                  bwd_need(kv, q, sq, sk)});
  }
  return n;
}

// segment-major work order from this many tiles in the longest segment on
constexpr int kSegMajorTiles = 8;
bool seg_major(const Sizes& s, int tile) { return tiles_of(s, tile) >= kSegMajorTiles; }

// Whether plan_kernel builds a schedule for a launch of `wgs` workgroups, or they
// place their items themselves: batches of few segments, in the segment-major
// order (a pass over the segments in every wave) also only up to kDirectWork
// segments x workgroups.  Forward, 4/4 heads: 16 segments of about 2,000 tokens
// (8,192) 5 us less than with a schedule, 32 (34,000) 5 us more, 48 of d = 64
// (77,000) 153 against 140; 32/8 heads of 64, 64 of about 1,000 (1.1 million) 475
// against 396 us.  The level-major order's ballots stay ahead throughout.
constexpr int64_t kDirectWork = 16384;
bool needs_plan(const Sizes& s, int tile, int64_t wgs) {
  if (s.N == 1) return false;
  if (!seg_major(s, tile)) return s.N > 64 * pdy::kDirectChunks;
  return s.N > pdy::kDirectSegMajor || s.N * wgs > kDirectWork;
}

pdy::Plan make_plan(const int32_t* cu, int32_t* ws, const Sizes& s, int tile, int64_t wgs) {
  const int nt = tiles_of(s, tile);
  pdy::Plan p;
  p.cu = cu;
  p.n = (int32_t)s.N;
  p.direct = !needs_plan(s, tile, wgs);
  p.tile_log2 = __builtin_ctz((unsigned)tile);  // every shape's tile is a power of two
  p.max_nt = nt;
  p.seg_major = seg_major(s, tile);
  if (p.direct) {
    p.order = p.start = p.total = p.cnt = p.before = nullptr;
    return p;
  }
  p.order = ws + s.N;
  p.cnt = ws + 2 * s.N;
  p.start = ws + 2 * s.N + nt;
  p.total = ws + 2 * s.N + 2 * nt;
  p.before = ws + 2 * s.N + 2 * nt + 1;
  return p;
}

template <typename K>
hipError_t set_lds(K kernel, int bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                             hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

template <int D, int NW, int KG>
hipError_t launch_fwd(const pdy::FwdArgs* a, dim3 grid, hipStream_t st) {
  using C = pdy::FwdCfg<D, NW, KG>;
  if (a == nullptr) return set_lds(pdy::fwd_kernel<D, NW, KG>, C::LDS_BYTES);
  hipLaunchKernelGGL((pdy::fwd_kernel<D, NW, KG>), grid, dim3(C::NT), C::LDS_BYTES, st, *a);
  return hipSuccess;
}

template <int D, int NW, int KG>
hipError_t launch_dq(const pdy::BwdArgs* a, dim3 grid, hipStream_t st) {
  using C = pdy::DqCfg<D, NW, KG>;
  if (a == nullptr) return set_lds(pdy::bwd_dq_kernel<D, NW, KG>, C::LDS_BYTES);
  hipLaunchKernelGGL((pdy::bwd_dq_kernel<D, NW, KG>), grid, dim3(C::NT), C::LDS_BYTES, st, *a);
  return hipSuccess;
}

template <int D, int NW, int QG>
hipError_t launch_dkdv(const pdy::BwdArgs* a, dim3 grid, hipStream_t st) {
  using C = pdy::DkdvCfg<D, QG, NW>;
  if (a == nullptr) return set_lds(pdy::bwd_dkdv_kernel<D, QG, NW>, C::LDS_BYTES);
  hipLaunchKernelGGL((pdy::bwd_dkdv_kernel<D, QG, NW>), grid, dim3(C::NT), C::LDS_BYTES, st, *a);
  return hipSuccess;
}

// The kernels by shape (dK/dV has none of four groups); called without arguments
// they set their attributes.
struct Kernels {
  int nw, groups;
  hipError_t (*fwd[2])(const pdy::FwdArgs*, dim3, hipStream_t);  // d = 64, 128
  hipError_t (*dq[2])(const pdy::BwdArgs*, dim3, hipStream_t);
  hipError_t (*dkdv[2])(const pdy::BwdArgs*, dim3, hipStream_t);
};
template <int NW, int G>
constexpr Kernels kernels_of() {
  Kernels k{NW, G, {launch_fwd<64, NW, G>, launch_fwd<128, NW, G>},
            {launch_dq<64, NW, G>, launch_dq<128, NW, G>}, {nullptr, nullptr}};
  if constexpr (G <= 2) {
    k.dkdv[0] = launch_dkdv<64, NW, G>;
    k.dkdv[1] = launch_dkdv<128, NW, G>;
  }
  return k;
}
constexpr Kernels kKernels[] = {kernels_of<4, 1>(), kernels_of<8, 1>(), kernels_of<8, 2>(),
                                kernels_of<8, 4>()};

const Kernels& kernels(const Shape& sh) {
  for (const Kernels& k : kKernels)
    if (k.nw == sh.nw && k.groups == sh.groups) return k;
  return kKernels[1];  // (not reached: every shape the launches use is listed)
}

// One-time per-process kernel attribute setup (LDS above the 64 KiB default).
hipError_t init_kernels() {
  static hipError_t status = [] {
    for (int d = 0; d < 2; ++d) {
      for (const Kernels& k : kKernels) {
        hipError_t e = k.fwd[d](nullptr, dim3(), nullptr);
        if (e == hipSuccess) e = k.dq[d](nullptr, dim3(), nullptr);
        if (e == hipSuccess && k.dkdv[d]) e = k.dkdv[d](nullptr, dim3(), nullptr);
        if (e != hipSuccess) return e;
      }
    }
    return hipSuccess;
  }();
  return status;
}

pdy_status check_scale(float scale, int32_t causal) {
  if (causal != 0 && causal != 1) return fail(PDY_ERR_INVALID_ARG, "causal must be 0 or 1");
  if (!std::isfinite(scale) || !(scale > 0.f))
    return fail(PDY_ERR_INVALID_ARG, "scale must be finite and > 0");
  return PDY_OK;
}

pdy_status check_ptr(const void* p, const char* name) {
  if (p == nullptr) return fail(PDY_ERR_INVALID_ARG, "%s is NULL", name);
  if (!aligned16(p)) return fail(PDY_ERR_INVALID_ARG, "%s is not 16-byte aligned", name);
  return PDY_OK;
}

// The schedule of s's segments in tiles of `tile` (cu == nullptr: one segment
// of s.T tokens), written to ws
pdy::PlanJob plan_job(const int32_t* cu, int32_t* ws, const Sizes& s, int tile) {
  return pdy::PlanJob{cu, (int)s.N, tile, tiles_of(s, tile), (int)s.T, ws};
}

// one or two schedules in one launch
pdy_status launch_plans(const pdy::PlanJob& a, const pdy::PlanJob* b, hipStream_t st) {
  pdy::PlanJobs jobs;
  jobs.job[0] = a;
  jobs.job[1] = b ? *b : a;
  const dim3 grid(b ? 2 : 1);
  hipError_t e = launch_timed(K_PLAN, st, [&] {
    hipLaunchKernelGGL(pdy::plan_kernel, grid, dim3(pdy::kPlanThreads), 0, st, jobs);
  });
  if (e != hipSuccess) return hip_fail(e, "plan_kernel launch");
  return PDY_OK;
}

}  // namespace

extern "C" {

const char* pdy_status_string(int32_t status) {
  switch (status) {
    case PDY_OK: return "ok";
    case PDY_ERR_INVALID_ARG: return "invalid argument";
    case PDY_ERR_UNSUPPORTED: return "unsupported configuration";
    case PDY_ERR_WORKSPACE: return "workspace too small";
    case PDY_ERR_HIP: return "HIP runtime error";
    default: return "unknown status";
  }
}

const char* pdy_last_error(void) { return g_err; }

size_t attn_fwd_workspace_size(int32_t T, int32_t N, int32_t maxlen, int32_t hq, int32_t hkv,
                               int32_t d) {
  Sizes s;
  if (check_sizes(T, N, maxlen, hq, hkv, d, &s) != PDY_OK) return 0;
  return fwd_workspace_bytes(s, s, false);
}

size_t attn_bwd_workspace_size(int32_t T, int32_t N, int32_t maxlen, int32_t hq, int32_t hkv,
                               int32_t d) {
  Sizes s;
  if (check_sizes(T, N, maxlen, hq, hkv, d, &s) != PDY_OK) return 0;
  return bwd_workspace_bytes(s, s, false);
}

}  // extern "C"

namespace {

// One query chunk against one key/value chunk of the same sequence
// (context-parallel step), or off: rows and keys share cu's segments.
struct Chunk {
  int on = 0;
  int tk = 0;          // key/value rows
  int shift = 0;       // query offset - key offset
  int accumulate = 0;  // backward: add to the gradients instead of writing them
  int launches = 1;    // pairs that the caller runs at a time
};

pdy_status fwd_impl(const void* q, const void* k, const void* v, const int32_t* cu,
                    const Sizes& s, const Sizes& sk, int32_t causal, float scale, void* o,
                    float* lse,
                    void* workspace, size_t workspace_bytes, void* stream, const Chunk& c,
                    const char* who) {
  pdy_status st;
  const Job job{s, sk, causal, c.on != 0, c.shift, c.launches};
  const Launch base = base_launch(FWD, job);
  Launch l = pick(FWD, job, base);
  // (a pair whose workspace was sized for other chunks takes fewer parts)
  while (c.on && workspace_bytes < fwd_need(l, s) && l.split.parts > 1)
    l.split = halve_split(l.split);
  if (workspace_bytes < fwd_need(l, s)) l = base;
  const size_t need = fwd_need(l, s);
  if (workspace_bytes < need)
    return fail(PDY_ERR_WORKSPACE, "workspace has %zu bytes, %s needs %zu", workspace_bytes, who,
                need);
  const pdy::Split& split = l.split;
  const int nsplit = split.parts, tile = l.sh.tile();
  hipError_t e = init_kernels();
  if (e != hipSuccess) return hip_fail(e, "kernel attribute setup");
  hipStream_t hs = reinterpret_cast<hipStream_t>(stream);
  int32_t* ws = reinterpret_cast<int32_t*>(workspace);
  const int64_t wgs = split_entries(split, grid_items(s, tile)) * s.hq;
  if (needs_plan(s, tile, wgs) &&
      (st = launch_plans(plan_job(cu, ws, s, tile), nullptr, hs)) != PDY_OK)
    return st;

  pdy::FwdArgs a;
  a.q = static_cast<const uint16_t*>(q);
  a.k = static_cast<const uint16_t*>(k);
  a.v = static_cast<const uint16_t*>(v);
  a.o = static_cast<uint16_t*>(o);
  a.lse = lse;
  a.plan = make_plan(cu, ws, s, tile, wgs);
  a.total_tokens = (int)s.T;
  a.hq = (int)s.hq;
  a.hkv = (int)s.hkv;
  a.causal = causal;
  a.scale_log2 = scale * pdy::kLog2e;
  a.chunked = c.on;
  a.tk = c.tk;
  a.shift = c.shift;
  a.split = split;
  a.part_o = nullptr;
  a.part_lse = nullptr;
  if (nsplit > 1) {
    uint8_t* w = reinterpret_cast<uint8_t*>(workspace) + q_plan_bytes(s, l.sh);
    a.part_o = reinterpret_cast<float*>(w);
    a.part_lse = reinterpret_cast<float*>(w + part_o_bytes(s, nsplit));
  }
  const dim3 grid((unsigned)wgs);
  e = launch_timed(K_FWD, hs, [&] { (void)kernels(l.sh).fwd[s.d == 128](&a, grid, hs); });
  if (e != hipSuccess) return hip_fail(e, "fwd_kernel launch");
  if (nsplit > 1) {
    const size_t threads = (size_t)s.T * s.hq * (s.d / 8);
    const dim3 blocks((unsigned)((threads + 255) / 256));
    e = launch_timed(K_SPLIT_MERGE, hs, [&] {
      uint16_t* out = static_cast<uint16_t*>(o);
      if (s.d == 64)
        hipLaunchKernelGGL(pdy::split_merge_kernel<64>, blocks, dim3(256), 0, hs, a.part_o,
                           a.part_lse, split, out, lse, (int)s.T, (int)s.hq);
      else
        hipLaunchKernelGGL(pdy::split_merge_kernel<128>, blocks, dim3(256), 0, hs, a.part_o,
                           a.part_lse, split, out, lse, (int)s.T, (int)s.hq);
    });
    if (e != hipSuccess) return hip_fail(e, "split_merge_kernel launch");
  }
  return PDY_OK;
}

pdy_status bwd_impl(const void* q, const void* k, const void* v, const void* o, const float* lse,
                    const void* dout, const int32_t* cu, const Sizes& s, const Sizes& sk,
                    int32_t causal, float scale, float* dq, float* dk, float* dv,
                    void* workspace, size_t workspace_bytes, void* stream, const Chunk& c,
                    const char* who, bool fit_splits) {
  pdy_status st;
  const Job job{s, sk, causal, c.on != 0, c.shift, c.launches};
  const Launch base_k = base_launch(DKDV, job), base_q = base_launch(DQ, job);
  Launch lk = pick(DKDV, job, base_k), lq = pick(DQ, job, base_q);
  // fit_splits: a workspace of fixed size, or sized for other chunks, takes
  // fewer split-K parts (the larger partial buffer halved first) when the chosen
  // ones do not fit
  auto fits = [&] {
    while (fit_splits && bwd_need(lk, lq, s, sk) > workspace_bytes &&
           (lk.split.parts > 1 || lq.split.parts > 1)) {
      const size_t bk = lk.split.parts > 1 ? 2 * part_kv_bytes(sk, lk.split.parts) : 0;
      const size_t bq = lq.split.parts > 1 ? part_o_bytes(s, lq.split.parts) : 0;
      if (bq >= bk) lq.split = halve_split(lq.split);
      else lk.split = halve_split(lk.split);
    }
    return bwd_need(lk, lq, s, sk) <= workspace_bytes;
  };
  if (!fits()) {
    lk = base_k;
    lq = base_q;
    if (!fits())
      return fail(PDY_ERR_WORKSPACE, "workspace has %zu bytes, %s needs %zu", workspace_bytes, who,
                  bwd_need(lk, lq, s, sk));
  }
  const pdy::Split &split_kv = lk.split, &split_q = lq.split;
  const int nsplit_kv = split_kv.parts, nsplit_q = split_q.parts;
  const int qtile = lq.sh.tile(), kvtile = lk.sh.tile();
  hipError_t e = init_kernels();
  if (e != hipSuccess) return hip_fail(e, "kernel attribute setup");
  hipStream_t hs = reinterpret_cast<hipStream_t>(stream);
  uint8_t* const wsb = reinterpret_cast<uint8_t*>(workspace);
  int32_t* ws = reinterpret_cast<int32_t*>(wsb);
  int32_t* ws_q = reinterpret_cast<int32_t*>(wsb + kv_plan_bytes(sk, lk.sh));
  float* dd = reinterpret_cast<float*>(wsb + kv_plan_bytes(sk, lk.sh) + q_plan_bytes(s, lq.sh));

  const int64_t wgs_q = split_entries(split_q, grid_items(s, qtile)) * s.hq;
  const int64_t wgs_kv = split_entries(split_kv, grid_items(sk, kvtile)) * sk.hkv;
  {
    // the query-tile schedule and the key-tile one, where they are needed
    // (packed batches: both sides have the same segments)
    const pdy::PlanJob q_job = plan_job(cu, ws_q, s, qtile);
    const pdy::PlanJob kv_job = plan_job(cu, ws, sk, kvtile);
    const bool need_q = needs_plan(s, qtile, wgs_q), need_kv = needs_plan(sk, kvtile, wgs_kv);
    if (need_q || need_kv) {
      st = launch_plans(need_q ? q_job : kv_job, need_q && need_kv ? &kv_job : nullptr, hs);
      if (st != PDY_OK) return st;
    }
  }
  pdy::BwdArgs a;
  a.q = static_cast<const uint16_t*>(q);
  a.k = static_cast<const uint16_t*>(k);
  a.v = static_cast<const uint16_t*>(v);
  a.o = static_cast<const uint16_t*>(o);
  a.dout = static_cast<const uint16_t*>(dout);
  a.lse = lse;
  a.dd = dd;
  a.dq = dq;
  a.dk = dk;
  a.dv = dv;
  a.plan = make_plan(cu, ws, sk, kvtile, wgs_kv);
  a.plan_q = make_plan(cu, ws_q, s, qtile, wgs_q);
  a.total_tokens = (int)s.T;
  a.hq = (int)s.hq;
  a.hkv = (int)s.hkv;
  a.causal = causal;
  a.scale = scale;
  a.scale_log2 = scale * pdy::kLog2e;
  a.chunked = c.on;
  a.tk = c.tk;
  a.shift = c.shift;
  a.accumulate = c.accumulate;
  a.split_kv = split_kv;
  a.split_q = split_q;
  a.part_dk = a.part_dv = a.part_dq = nullptr;
  {
    uint8_t* w = wsb + bwd_fixed(lk.sh, lq.sh, s, sk);
    if (nsplit_kv > 1) {
      a.part_dk = reinterpret_cast<float*>(w);
      a.part_dv = reinterpret_cast<float*>(w + part_kv_bytes(sk, nsplit_kv));
      w += 2 * part_kv_bytes(sk, nsplit_kv);
    }
    if (nsplit_q > 1) a.part_dq = reinterpret_cast<float*>(w);
  }
  // dQ first: it also writes D = rowsum(dO * O), which dK/dV reads
  const dim3 gq((unsigned)wgs_q);
  e = launch_timed(K_DQ, hs, [&] { (void)kernels(lq.sh).dq[s.d == 128](&a, gq, hs); });
  if (e != hipSuccess) return hip_fail(e, "bwd_dq_kernel launch");
  if (sk.T > 0) {
    const dim3 gkv((unsigned)wgs_kv);
    e = launch_timed(K_DKDV, hs, [&] { (void)kernels(lk.sh).dkdv[s.d == 128](&a, gkv, hs); });
    if (e != hipSuccess) return hip_fail(e, "bwd_dkdv_kernel launch");
  }
  // the parts' partial gradients (dQ, dK, dV), summed in one launch
  pdy::SumJobs jobs{};
  jobs.njobs = 0;
  jobs.accumulate = c.accumulate;
  int64_t sum_blocks = 0;
  auto add_job = [&](const float* parts, float* dst, size_t n, int row_elems,
                     const pdy::Split& sp) {
    const int blocks = (int)((n / 4 + 255) / 256);
    jobs.blocks[jobs.njobs] = blocks;
    jobs.job[jobs.njobs++] = pdy::SumJob{parts, dst, (uint32_t)n, row_elems, sp};
    sum_blocks += blocks;
  };
  if (nsplit_q > 1) add_job(a.part_dq, dq, (size_t)s.T * s.hq * s.d, (int)(s.hq * s.d), split_q);
  if (sk.T > 0 && nsplit_kv > 1) {
    const size_t n = (size_t)sk.T * s.hkv * s.d;
    add_job(a.part_dk, dk, n, (int)(s.hkv * s.d), split_kv);
    add_job(a.part_dv, dv, n, (int)(s.hkv * s.d), split_kv);
  }
  if (jobs.njobs > 0) {
    const dim3 blocks((unsigned)sum_blocks);
    e = launch_timed(K_SPLIT_SUM, hs, [&] {
      hipLaunchKernelGGL(pdy::split_sum_kernel, blocks, dim3(256), 0, hs, jobs);
    });
    if (e != hipSuccess) return hip_fail(e, "split_sum_kernel launch");
  }
  return PDY_OK;
}

// Argument checks of attn_bwd and attn_bwd_noalloc (everything but the
// workspace); s is filled in.  T = 0 passes with PDY_OK before the pointers
// are looked at.
pdy_status bwd_checks(const void* q, const void* k, const void* v, const void* o,
                      const float* lse, const void* dout, const int32_t* cu_seqlens,
                      int32_t num_seqs, int32_t total_tokens, int32_t max_seqlen,
                      int32_t num_heads_q, int32_t num_heads_kv, int32_t head_dim,
                      int32_t causal, float scale, float* dq, float* dk, float* dv, Sizes* s) {
  pdy_status st;
  if ((st = check_sizes(total_tokens, num_seqs, max_seqlen, num_heads_q, num_heads_kv, head_dim,
                        s)) != PDY_OK)
    return st;
  if ((st = check_scale(scale, causal)) != PDY_OK) return st;
  if (s->T == 0) return PDY_OK;
  if ((st = check_ptr(q, "q")) || (st = check_ptr(k, "k")) || (st = check_ptr(v, "v")) ||
      (st = check_ptr(o, "o")) || (st = check_ptr(lse, "lse")) ||
      (st = check_ptr(dout, "dout")) || (st = check_ptr(dq, "dq")) ||
      (st = check_ptr(dk, "dk")) || (st = check_ptr(dv, "dv")))
    return st;
  if (cu_seqlens == nullptr) return fail(PDY_ERR_INVALID_ARG, "cu_seqlens is NULL");
  if ((reinterpret_cast<uintptr_t>(cu_seqlens) & 3u) != 0)
    return fail(PDY_ERR_INVALID_ARG, "cu_seqlens is not 4-byte aligned");
  return PDY_OK;
}

// ---------------------------------------------------------------------------
// Static scratch of attn_bwd_noalloc, for callers that cannot allocate.  A
// file-scope device array: every GPU the library runs on holds its own copy
// (kScratchBytes) from the first use until the process ends.  In host code
// `scratch` only names the symbol; its device address on the current device
// comes from hipGetSymbolAddress, looked up once per device and kept.
// Nothing in it has to start at zero: each call writes every scratch entry
// it reads (schedules, D, partial gradients) before reading it.  Calls that
// overlap on one GPU share the array and race.
// ---------------------------------------------------------------------------
constexpr size_t kScratchBytes = (size_t)64 << 20;
static __device__ __align__(256) uint8_t scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of the current device's scratch.
pdy_status scratch_ptr(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  if (dev < 0 || dev >= kMaxDevices)
    return fail(PDY_ERR_UNSUPPORTED, "device %d is beyond the %d the scratch table covers", dev,
                kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
    if (p == nullptr) return fail(PDY_ERR_HIP, "hipGetSymbolAddress(scratch) returned NULL");
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return PDY_OK;
}

// sizes of a chunk: one segment of t tokens
pdy_status chunk_sizes(int32_t tq, int32_t tk, int32_t hq, int32_t hkv, int32_t d, Sizes* sq,
                       Sizes* sk) {
  pdy_status st;
  if (tq < 0 || tk < 0) return fail(PDY_ERR_INVALID_ARG, "chunk lengths must be >= 0");
  if ((st = check_sizes(tq, 1, tq, hq, hkv, d, sq)) != PDY_OK) return st;
  if ((st = check_sizes(tk, 1, tk, hq, hkv, d, sk)) != PDY_OK) return st;
  return PDY_OK;
}

// pdy_launch_shapes for a job; kernels that would not run keep their zeros
void write_shapes(const Job& j, int32_t* out) {
  std::fill(out, out + 9, 0);
  const bool runs[3] = {j.sq.T > 0, j.sq.T > 0, j.sq.T > 0 && j.sk.T > 0};
  for (int k = 0; k < 3; ++k) {
    if (!runs[k]) continue;
    const Launch l = pick((Which)k, j, base_launch((Which)k, j));
    out[3 * k] = l.sh.nw;
    out[3 * k + 1] = l.sh.groups;
    out[3 * k + 2] = l.split.parts;
  }
}

}  // namespace

extern "C" {

pdy_status pdy_launch_shapes(int32_t total_tokens, int32_t num_seqs, int32_t max_seqlen,
                             int32_t num_heads_q, int32_t num_heads_kv, int32_t head_dim,
                             int32_t causal, int32_t* shapes) {
  g_err[0] = 0;
  Sizes s;
  pdy_status st;
  if ((st = check_sizes(total_tokens, num_seqs, max_seqlen, num_heads_q, num_heads_kv, head_dim,
                        &s)) != PDY_OK)
    return st;
  if (causal != 0 && causal != 1) return fail(PDY_ERR_INVALID_ARG, "causal must be 0 or 1");
  if (shapes == nullptr) return fail(PDY_ERR_INVALID_ARG, "shapes is NULL");
  write_shapes({s, s, causal, false, 0}, shapes);
  return PDY_OK;
}

pdy_status pdy_chunk_launch_shapes(int32_t tq, int32_t tk, int32_t q_offset, int32_t k_offset,
                                   int32_t num_heads_q, int32_t num_heads_kv, int32_t head_dim,
                                   int32_t causal, int32_t launches, int32_t* shapes) {
  g_err[0] = 0;
  Sizes sq, sk;
  pdy_status st;
  if ((st = chunk_sizes(tq, tk, num_heads_q, num_heads_kv, head_dim, &sq, &sk)) != PDY_OK)
    return st;
  if (q_offset < 0 || k_offset < 0) return fail(PDY_ERR_INVALID_ARG, "offsets must be >= 0");
  if (launches < 1) return fail(PDY_ERR_INVALID_ARG, "launches must be >= 1 (got %d)", launches);
  if (causal != 0 && causal != 1) return fail(PDY_ERR_INVALID_ARG, "causal must be 0 or 1");
  if (shapes == nullptr) return fail(PDY_ERR_INVALID_ARG, "shapes is NULL");
  write_shapes({sq, sk, causal, true, q_offset - k_offset, launches}, shapes);
  return PDY_OK;
}

pdy_status attn_fwd(const void* q, const void* k, const void* v, const int32_t* cu_seqlens,
                    int32_t num_seqs, int32_t total_tokens, int32_t max_seqlen, int32_t num_heads_q,
                    int32_t num_heads_kv, int32_t head_dim, int32_t causal, float scale, void* o,
                    float* lse, void* workspace, size_t workspace_bytes, void* stream) {
  g_err[0] = 0;
  Sizes s;
  pdy_status st;
  if ((st = check_sizes(total_tokens, num_seqs, max_seqlen, num_heads_q, num_heads_kv, head_dim,
                        &s)) != PDY_OK)
    return st;
  if ((st = check_scale(scale, causal)) != PDY_OK) return st;
  if (s.T == 0) return PDY_OK;
  if ((st = check_ptr(q, "q")) || (st = check_ptr(k, "k")) || (st = check_ptr(v, "v")) ||
      (st = check_ptr(o, "o")) || (st = check_ptr(lse, "lse")) ||
      (st = check_ptr(workspace, "workspace")))
    return st;
  if (cu_seqlens == nullptr) return fail(PDY_ERR_INVALID_ARG, "cu_seqlens is NULL");
  if ((reinterpret_cast<uintptr_t>(cu_seqlens) & 3u) != 0)
    return fail(PDY_ERR_INVALID_ARG, "cu_seqlens is not 4-byte aligned");
  return fwd_impl(q, k, v, cu_seqlens, s, s, causal, scale, o, lse, workspace, workspace_bytes,
                  stream, Chunk{}, "attn_fwd");
}

size_t attn_fwd_chunk_workspace_size(int32_t tq, int32_t tk, int32_t hq, int32_t hkv, int32_t d) {
  Sizes sq, sk;
  if (chunk_sizes(tq, tk, hq, hkv, d, &sq, &sk) != PDY_OK) return 0;
  return fwd_workspace_bytes(sq, sk, true);
}

size_t attn_bwd_chunk_workspace_size(int32_t tq, int32_t tk, int32_t hq, int32_t hkv, int32_t d) {
  Sizes sq, sk;
  if (chunk_sizes(tq, tk, hq, hkv, d, &sq, &sk) != PDY_OK) return 0;
  return bwd_workspace_bytes(sq, sk, true);
}

pdy_status attn_fwd_chunk(const void* q, const void* k, const void* v, int32_t tq, int32_t tk,
                          int32_t q_offset, int32_t k_offset, int32_t num_heads_q,
                          int32_t num_heads_kv, int32_t head_dim, int32_t causal, float scale,
                          void* o, float* lse, void* workspace, size_t workspace_bytes,
                          void* stream) {
  return attn_fwd_chunk_shared(q, k, v, tq, tk, q_offset, k_offset, num_heads_q, num_heads_kv,
                               head_dim, causal, scale, o, lse, workspace, workspace_bytes, stream,
                               1);
}

pdy_status attn_fwd_chunk_shared(const void* q, const void* k, const void* v, int32_t tq,
                                 int32_t tk, int32_t q_offset, int32_t k_offset,
                                 int32_t num_heads_q, int32_t num_heads_kv, int32_t head_dim,
                                 int32_t causal, float scale, void* o, float* lse, void* workspace,
                                 size_t workspace_bytes, void* stream, int32_t launches) {
  g_err[0] = 0;
  Sizes sq, sk;
  pdy_status st;
  if ((st = chunk_sizes(tq, tk, num_heads_q, num_heads_kv, head_dim, &sq, &sk)) != PDY_OK)
    return st;
  if (q_offset < 0 || k_offset < 0) return fail(PDY_ERR_INVALID_ARG, "offsets must be >= 0");
  if (launches < 1) return fail(PDY_ERR_INVALID_ARG, "launches must be >= 1 (got %d)", launches);
  if ((st = check_scale(scale, causal)) != PDY_OK) return st;
  if (tq == 0) return PDY_OK;
  if ((st = check_ptr(q, "q")) || (st = check_ptr(o, "o")) || (st = check_ptr(lse, "lse")) ||
      (st = check_ptr(workspace, "workspace")))
    return st;
  if (tk > 0 && ((st = check_ptr(k, "k")) || (st = check_ptr(v, "v")))) return st;
  Chunk c;
  c.on = 1;
  c.tk = tk;
  c.shift = q_offset - k_offset;
  c.launches = launches;
  return fwd_impl(q, k, v, nullptr, sq, sk, causal, scale, o, lse, workspace, workspace_bytes, stream,
                  c, "attn_fwd_chunk");
}

pdy_status attn_bwd(const void* q, const void* k, const void* v, const void* o, const float* lse,
                    const void* dout, const int32_t* cu_seqlens, int32_t num_seqs,
                    int32_t total_tokens, int32_t max_seqlen, int32_t num_heads_q,
                    int32_t num_heads_kv, int32_t head_dim, int32_t causal, float scale, float* dq,
                    float* dk, float* dv, void* workspace, size_t workspace_bytes, void* stream) {
  g_err[0] = 0;
  Sizes s;
  pdy_status st;
  if ((st = bwd_checks(q, k, v, o, lse, dout, cu_seqlens, num_seqs, total_tokens, max_seqlen,
                       num_heads_q, num_heads_kv, head_dim, causal, scale, dq, dk, dv, &s)) !=
          PDY_OK ||
      s.T == 0)
    return st;
  if ((st = check_ptr(workspace, "workspace")) != PDY_OK) return st;
  return bwd_impl(q, k, v, o, lse, dout, cu_seqlens, s, s, causal, scale, dq, dk, dv, workspace,
                  workspace_bytes, stream, Chunk{}, "attn_bwd", false);
}

pdy_status attn_bwd_noalloc(const void* q, const void* k, const void* v, const void* o,
                            const float* lse, const void* dout, const int32_t* cu_seqlens,
                            int32_t num_seqs, int32_t total_tokens, int32_t max_seqlen,
                            int32_t num_heads_q, int32_t num_heads_kv, int32_t head_dim,
                            int32_t causal, float scale, float* dq, float* dk, float* dv,
                            void* stream) {
  g_err[0] = 0;
  Sizes s;
  pdy_status st;
  if ((st = bwd_checks(q, k, v, o, lse, dout, cu_seqlens, num_seqs, total_tokens, max_seqlen,
                       num_heads_q, num_heads_kv, head_dim, causal, scale, dq, dk, dv, &s)) !=
          PDY_OK ||
      s.T == 0)
    return st;
  // the scratch attn_bwd takes from its workspace: the tile schedules and D,
  // plus split-K partial gradients where those fit (else fewer parts)
  const size_t need = bwd_fixed(base_shape(DKDV, s), base_shape(FWD, s), s, s);
  if (need > kScratchBytes)
    return fail(PDY_ERR_WORKSPACE,
                "attn_bwd_noalloc needs %zu bytes of scratch for these sizes, more than its "
                "static scratch of %zu bytes (call attn_bwd with a workspace instead)",
                need, kScratchBytes);
  void* ws = nullptr;
  if ((st = scratch_ptr(&ws)) != PDY_OK) return st;
  return bwd_impl(q, k, v, o, lse, dout, cu_seqlens, s, s, causal, scale, dq, dk, dv, ws,
                  kScratchBytes, stream, Chunk{}, "attn_bwd_noalloc", /*fit_splits=*/true);
}

pdy_status attn_bwd_chunk(const void* q, const void* k, const void* v, const void* o,
                          const float* lse, const void* dout, int32_t tq, int32_t tk,
                          int32_t q_offset, int32_t k_offset, int32_t num_heads_q,
                          int32_t num_heads_kv, int32_t head_dim, int32_t causal, float scale,
                          float* dq, float* dk, float* dv, int32_t accumulate, void* workspace,
                          size_t workspace_bytes, void* stream) {
  return attn_bwd_chunk_shared(q, k, v, o, lse, dout, tq, tk, q_offset, k_offset, num_heads_q,
                               num_heads_kv, head_dim, causal, scale, dq, dk, dv, accumulate,
                               workspace, workspace_bytes, stream, 1);
}

pdy_status attn_bwd_chunk_shared(const void* q, const void* k, const void* v, const void* o,
                                 const float* lse, const void* dout, int32_t tq, int32_t tk,
                                 int32_t q_offset, int32_t k_offset, int32_t num_heads_q,
                                 int32_t num_heads_kv, int32_t head_dim, int32_t causal,
                                 float scale, float* dq, float* dk, float* dv, int32_t accumulate,
                                 void* workspace, size_t workspace_bytes, void* stream,
                                 int32_t launches) {
  g_err[0] = 0;
  Sizes sq, sk;
  pdy_status st;
  if ((st = chunk_sizes(tq, tk, num_heads_q, num_heads_kv, head_dim, &sq, &sk)) != PDY_OK)
    return st;
  if (q_offset < 0 || k_offset < 0) return fail(PDY_ERR_INVALID_ARG, "offsets must be >= 0");
  if (launches < 1) return fail(PDY_ERR_INVALID_ARG, "launches must be >= 1 (got %d)", launches);
  if ((st = check_scale(scale, causal)) != PDY_OK) return st;
  if (tq == 0 && tk == 0) return PDY_OK;
  if (tq > 0 && ((st = check_ptr(q, "q")) || (st = check_ptr(o, "o")) ||
                 (st = check_ptr(lse, "lse")) || (st = check_ptr(dout, "dout")) ||
                 (st = check_ptr(dq, "dq"))))
    return st;
  if (tk > 0 && ((st = check_ptr(k, "k")) || (st = check_ptr(v, "v")) ||
                 (st = check_ptr(dk, "dk")) || (st = check_ptr(dv, "dv"))))
    return st;
  if (accumulate != 0 && accumulate != 1)
    return fail(PDY_ERR_INVALID_ARG, "accumulate must be 0 or 1 (got %d)", accumulate);
  if ((st = check_ptr(workspace, "workspace")) != PDY_OK) return st;
  if (tq == 0 && accumulate) return PDY_OK;
  if (tq == 0) {
    // no query rows: the key chunk receives no gradient (a fill kernel, not
    // a memset, so that the call can be captured in a graph)
    hipStream_t hs = reinterpret_cast<hipStream_t>(stream);
    const size_t n = (size_t)tk * num_heads_kv * head_dim;
    const unsigned blocks = (unsigned)((n + 1023) / 1024);
    hipLaunchKernelGGL(pdy::zero_kernel, dim3(blocks), dim3(256), 0, hs, dk, n);
    hipLaunchKernelGGL(pdy::zero_kernel, dim3(blocks), dim3(256), 0, hs, dv, n);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "zero_kernel launch");
    return PDY_OK;
  }
  Chunk c;
  c.on = 1;
  c.tk = tk;
  c.shift = q_offset - k_offset;
  c.accumulate = accumulate;
  c.launches = launches;
  return bwd_impl(q, k, v, o, lse, dout, nullptr, sq, sk, causal, scale, dq, dk, dv, workspace,
                  workspace_bytes, stream, c, "attn_bwd_chunk", /*fit_splits=*/true);
}

pdy_status attn_merge(const void* o_a, const float* lse_a, const void* o_b, const float* lse_b,
                      int32_t total_tokens, int32_t num_heads_q, int32_t head_dim, void* o,
                      float* lse, void* stream) {
  g_err[0] = 0;
  pdy_status st;
  if (total_tokens < 0) return fail(PDY_ERR_INVALID_ARG, "total_tokens must be >= 0");
  if (num_heads_q < 1) return fail(PDY_ERR_INVALID_ARG, "num_heads_q must be >= 1");
  if (head_dim != 64 && head_dim != 128)
    return fail(PDY_ERR_UNSUPPORTED, "head_dim %d not supported (64 or 128)", head_dim);
  if (total_tokens == 0) return PDY_OK;
  if ((st = check_ptr(o_a, "o_a")) || (st = check_ptr(lse_a, "lse_a")) ||
      (st = check_ptr(o_b, "o_b")) || (st = check_ptr(lse_b, "lse_b")) ||
      (st = check_ptr(o, "o")) || (st = check_ptr(lse, "lse")))
    return st;
  hipStream_t hs = reinterpret_cast<hipStream_t>(stream);
  const size_t threads = (size_t)total_tokens * num_heads_q * (head_dim / 8);
  const unsigned blocks = (unsigned)((threads + 255) / 256);
  const auto* a = static_cast<const uint16_t*>(o_a);
  const auto* b = static_cast<const uint16_t*>(o_b);
  auto* out = static_cast<uint16_t*>(o);
  if (head_dim == 64)
    hipLaunchKernelGGL(pdy::merge_kernel<64>, dim3(blocks), dim3(256), 0, hs, a, lse_a, b, lse_b,
                       out, lse, (int)total_tokens, (int)num_heads_q);
  else
    hipLaunchKernelGGL(pdy::merge_kernel<128>, dim3(blocks), dim3(256), 0, hs, a, lse_a, b, lse_b,
                       out, lse, (int)total_tokens, (int)num_heads_q);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "merge_kernel launch");
  return PDY_OK;
}

pdy_status attn_validate_cu_seqlens(const int32_t* cu_seqlens, int32_t num_seqs,
                                    int32_t total_tokens, int32_t* max_seqlen_out, void* stream) {
  g_err[0] = 0;
  if (cu_seqlens == nullptr) return fail(PDY_ERR_INVALID_ARG, "cu_seqlens is NULL");
  if (num_seqs < 1) return fail(PDY_ERR_INVALID_ARG, "num_seqs must be >= 1");
  std::vector<int32_t> h((size_t)num_seqs + 1);
  hipStream_t hs = reinterpret_cast<hipStream_t>(stream);
  hipError_t e = hipMemcpyAsync(h.data(), cu_seqlens, h.size() * 4, hipMemcpyDeviceToHost, hs);
  if (e == hipSuccess) e = hipStreamSynchronize(hs);
  if (e != hipSuccess) return hip_fail(e, "copying cu_seqlens to the host");
  if (h[0] != 0) return fail(PDY_ERR_INVALID_ARG, "cu_seqlens[0] = %d, expected 0", h[0]);
  int32_t mx = 0;
  for (int32_t i = 0; i < num_seqs; ++i) {
    if (h[i + 1] < h[i])
      return fail(PDY_ERR_INVALID_ARG, "cu_seqlens decreases at %d (%d -> %d)", i, h[i], h[i + 1]);
    if (h[i + 1] - h[i] > mx) mx = h[i + 1] - h[i];
  }
  if (h[num_seqs] != total_tokens)
    return fail(PDY_ERR_INVALID_ARG, "cu_seqlens[%d] = %d, expected total_tokens = %d", num_seqs,
                h[num_seqs], total_tokens);
  if (max_seqlen_out) *max_seqlen_out = mx;
  return PDY_OK;
}

int32_t pdy_kernel_count(void) { return K_COUNT; }

const char* pdy_kernel_name(int32_t k) {
  return (k >= 0 && k < K_COUNT) ? kKernelNames[k] : "";
}

pdy_status pdy_profile_start(void) {
  g_err[0] = 0;
  for (auto& r : g_prof_recs) {
    g_prof_pool.push_back(r.a);
    g_prof_pool.push_back(r.b);
  }
  g_prof_recs.clear();
  g_prof_on = true;
  return PDY_OK;
}

pdy_status pdy_profile_stop(int32_t* launches, double* total_ms, int32_t n) {
  g_err[0] = 0;
  g_prof_on = false;
  if (n < 0 || (n > 0 && (launches == nullptr || total_ms == nullptr)))
    return fail(PDY_ERR_INVALID_ARG, "pdy_profile_stop: bad output arrays");
  for (int32_t k = 0; k < n; ++k) {
    launches[k] = 0;
    total_ms[k] = 0.0;
  }
  pdy_status st = PDY_OK;
  for (auto& r : g_prof_recs) {
    float ms = 0.f;
    hipError_t e = hipEventSynchronize(r.b);
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, r.a, r.b);
    if (e != hipSuccess && st == PDY_OK) st = hip_fail(e, "pdy_profile_stop: reading events");
    if (r.kid < n) {
      launches[r.kid] += 1;
      total_ms[r.kid] += ms;
    }
    g_prof_pool.push_back(r.a);
    g_prof_pool.push_back(r.b);
  }
  g_prof_recs.clear();
  return st;
}

}  // extern "C"
