// Window rule and block-set construction shared by the host sizing code and
// the device kernels of the library.
//
// Sec. 2.1: with the bottom-right causal distance delta = i_q + (N_k - N_q) - i_k
// (Eq. fwa_distance), KV head h sees
//   near : 0 <= delta < w_near
//   sink : i_k < w_sink and delta >= 0
//   long : lo_h <= delta < hi_h,  lo_h = w_near + b_h,  hi_h = w_near + b_{h+1}
// with L = max(N_k - w_sink - w_near, 0) and b_h = floor(h L / H_k) over the
// global KV-head index (Eq. fwa_long_range_span, Eq. fwa_global_head).
//
// Sec. 2.3: J_h(i) is the set of KV blocks holding at least one legal pair with
// QO block i, I_h(j) its inverse.  Each window is one contiguous key run per
// query and the runs slide by one key per query, so over a QO block every
// window covers one contiguous key range; J_h(i) is the union of at most three
// block ranges and is found in O(1) per block (likewise I_h(j)).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cowa {

struct HeadGeo {
  int32_t n_q, n_k, w_sink, w_near, tile_q, tile_k;
  int64_t lo, hi;  // long-window distance bounds [lo, hi)
};

__host__ __device__ inline int64_t imin64(int64_t a, int64_t b) { return a < b ? a : b; }
__host__ __device__ inline int64_t imax64(int64_t a, int64_t b) { return a > b ? a : b; }

// Long-window bounds of global KV head hg out of ht heads (64-bit products).
__host__ __device__ inline void long_bounds(int64_t n_k, int64_t w_sink, int64_t w_near, int64_t hg,
                                            int64_t ht, int64_t* lo, int64_t* hi) {
  int64_t span = imax64(n_k - w_sink - w_near, 0);
  *lo = w_near + (hg * span) / ht;
  *hi = w_near + ((hg + 1) * span) / ht;
}

// The same from resolved window bounds (sink, near, long-range [lo, hi)).
__host__ __device__ inline HeadGeo make_geo_bounds(int32_t n_q, int32_t n_k, int32_t sink, int32_t near, int64_t lo,
                                                   int64_t hi, int32_t tile_q, int32_t tile_k) {
  HeadGeo g;
  g.n_q = n_q; g.n_k = n_k; g.w_sink = sink; g.w_near = near; g.tile_q = tile_q; g.tile_k = tile_k;
  g.lo = lo; g.hi = hi;
  return g;
}

// Element predicate of Eq. fwa_support (set union of the three windows).
__host__ __device__ inline bool legal_pair(const HeadGeo& g, int64_t q, int64_t k) {
  if (q >= g.n_q || k >= g.n_k) return false;
  int64_t d = q + (int64_t)(g.n_k - g.n_q) - k;
  if (d < 0) return false;
  return d < g.w_near || k < g.w_sink || (d >= g.lo && d < g.hi);
}

// 32-bit form of the element predicate for kernels: window bounds clamped to
// n_k (a distance never reaches n_k, so a larger bound behaves the same).
struct Geo32 {
  int32_t off, w_near, w_sink, lo, hi, n_q, n_k;
};

__host__ __device__ inline Geo32 geo32(const HeadGeo& g) {
  Geo32 r;
  r.off = g.n_k - g.n_q;
  r.w_near = g.w_near < g.n_k ? g.w_near : g.n_k;
  r.w_sink = g.w_sink < g.n_k ? g.w_sink : g.n_k;
  r.lo = (int32_t)imin64(g.lo, g.n_k);
  r.hi = (int32_t)imin64(g.hi, g.n_k);
  r.n_q = g.n_q;
  r.n_k = g.n_k;
  return r;
}

// Same predicate as legal_pair for in-range positions (q < n_q, k < n_k).
__host__ __device__ inline bool legal32(const Geo32& g, int32_t q, int32_t k) {
  const int32_t d = q + g.off - k;
  // bitwise, not short-circuit: a mask evaluated without branches
  return (q < g.n_q) & (k < g.n_k) & (d >= 0) & ((d < g.w_near) | (k < g.w_sink) | ((d >= g.lo) & (d < g.hi)));
}

// Bits a..b (inclusive) of a 32-bit word, for any a, b (none when a > b or the
// range misses 0..31).
__host__ __device__ inline uint32_t bit_range32(int32_t a, int32_t b) {
  const int32_t lo = a < 0 ? 0 : (a > 32 ? 32 : a);
  const int32_t hi = b < 0 ? 0 : (b > 31 ? 32 : b + 1);
  const int32_t w = hi - lo;  // (32-bit arithmetic only: few registers)
  return w <= 0 ? 0u : (w >= 32 ? ~0u : ((1u << (w & 31)) - 1u) << (lo & 31));
}
__host__ __device__ inline int32_t imin32(int32_t a, int32_t b) { return a < b ? a : b; }
__host__ __device__ inline int32_t imax32(int32_t a, int32_t b) { return a > b ? a : b; }

// legal32 over 32 consecutive keys at once: bit j is legal32(g, q, key0 + j).
// For one query the legal keys are the union of three runs (near, long, sink)
// cut to d >= 0 and k < n_k; each run becomes a range of bits, so a partial
// block's element mask costs a few operations per query and chunk instead of
// the window rule per element.
__host__ __device__ inline uint32_t legal_keys32(const Geo32& g, int32_t q, int32_t key0) {
  const int32_t d0 = q + g.off - key0;                // distance of key0
  const int32_t up = imin32(d0, g.n_k - 1 - key0);    // d >= 0, k < n_k
  const uint32_t m = bit_range32(d0 - g.w_near + 1, up) | bit_range32(d0 - g.hi + 1, imin32(up, d0 - g.lo)) |
                     bit_range32(0, imin32(up, g.w_sink - 1 - key0));
  return q < g.n_q ? m : 0u;  // (a select, not a branch)
}
// The same over 32 consecutive queries for one key: bit i is legal32(g, q0 + i, k).
__host__ __device__ inline uint32_t legal_queries32(const Geo32& g, int32_t q0, int32_t k) {
  const int32_t e0 = q0 + g.off - k;                  // distance of query q0
  const int32_t up = g.n_q - 1 - q0;                  // q < n_q
  const uint32_t m = bit_range32(-e0, imin32(up, g.w_near - 1 - e0)) |
                     bit_range32(imax32(-e0, g.lo - e0), imin32(up, g.hi - 1 - e0)) |
                     (k < g.w_sink ? bit_range32(-e0, up) : 0u);
  return k < g.n_k ? m : 0u;
}

// Up to three ascending, merged inclusive ranges in scalars, built with selects
// only (kernels: indexed arrays would go to scratch memory).  Empty ranges
// have a = kNone and b = kNone - 1 and come last.
constexpr int32_t kNone = 0x3fffffff;
struct Runs3 {
  int32_t a0, b0, a1, b1, a2, b2;
};
__host__ __device__ inline void order2(int32_t& a, int32_t& b, int32_t& c, int32_t& d) {  // (a, b) before (c, d)
  const bool sw = c < a;
  const int32_t ta = sw ? c : a, tb = sw ? d : b, tc = sw ? a : c, td = sw ? b : d;
  a = ta; b = tb; c = tc; d = td;
}
__host__ __device__ inline void runs3_merge(Runs3& r) {
  order2(r.a0, r.b0, r.a1, r.b1);
  order2(r.a1, r.b1, r.a2, r.b2);
  order2(r.a0, r.b0, r.a1, r.b1);
  // merge overlapping or touching runs (an empty run starts at kNone and never merges)
  if (r.a1 != kNone && r.a1 <= r.b0 + 1) {
    r.b0 = imax32(r.b0, r.b1);
    r.a1 = r.a2; r.b1 = r.b2;
    r.a2 = kNone; r.b2 = kNone - 1;
  }
  if (r.a1 != kNone && r.a1 <= r.b0 + 1) {
    r.b0 = imax32(r.b0, r.b1);
    r.a1 = kNone; r.b1 = kNone - 1;
  }
  if (r.a2 != kNone && r.a2 <= r.b1 + 1) {
    r.b1 = imax32(r.b1, r.b2);
    r.a2 = kNone; r.b2 = kNone - 1;
  }
}

// The visible keys of the decoding query (distance-0 key c = N_k - 1): the
// union of the sink, long-range and near windows of Sec. 2.1.
__host__ __device__ inline Runs3 key_runs3(int32_t n_k, int32_t sink, int32_t near, int32_t lo, int32_t hi) {
  const int32_t c = n_k - 1;
  Runs3 r;
  // near: delta in [0, near); sink: keys below sink; long: delta in [lo, hi)
  r.a0 = near >= 1 ? imax32(0, c - near + 1) : kNone;
  r.b0 = near >= 1 ? c : kNone - 1;
  r.a1 = sink >= 1 ? 0 : kNone;
  r.b1 = sink >= 1 ? imin32(sink - 1, c) : kNone - 1;
  const bool has_long = hi > lo && c - lo >= 0;
  r.a2 = has_long ? imax32(0, c - hi + 1) : kNone;
  r.b2 = has_long ? c - lo : kNone - 1;
  runs3_merge(r);
  return r;
}

// Blocks of BK keys that hold a legal pair with some query q0 .. q1 (q1 < n_q):
// fwd_block_ranges for any query range, in 32-bit scalars.
template <int BK>
__host__ __device__ inline Runs3 key_block_runs3(const Geo32& g, int32_t q0, int32_t q1) {
  const int32_t c0 = q0 + g.off, c1 = q1 + g.off;  // keys at distance 0
  Runs3 r;
  r.a0 = g.w_near >= 1 ? imax32(0, c0 - g.w_near + 1) / BK : kNone;
  r.b0 = g.w_near >= 1 ? c1 / BK : kNone - 1;
  r.a1 = g.w_sink >= 1 ? 0 : kNone;
  r.b1 = g.w_sink >= 1 ? imin32(g.w_sink - 1, c1) / BK : kNone - 1;
  const bool has_long = g.hi > g.lo && c1 - g.lo >= 0;
  r.a2 = has_long ? imax32(0, c0 - g.hi + 1) / BK : kNone;
  r.b2 = has_long ? (c1 - g.lo) / BK : kNone - 1;
  runs3_merge(r);
  return r;
}

// Blocks of BQ queries that hold a legal pair with some key k0 .. k1 (k1 < n_k):
// bwd_block_ranges for any key range, in 32-bit scalars.
template <int BQ>
__host__ __device__ inline Runs3 query_block_runs3(const Geo32& g, int32_t k0, int32_t k1) {
  const int32_t cmin = g.off, cmax = g.n_k - 1;  // keys at distance 0 of the first / last query
  auto clip = [&](bool any, int32_t a, int32_t b, int32_t& ra, int32_t& rb) {
    a = imax32(a, cmin);
    b = imin32(b, cmax);
    any = any && a <= b;
    ra = any ? (a - cmin) / BQ : kNone;
    rb = any ? (b - cmin) / BQ : kNone - 1;
  };
  Runs3 r;
  clip(g.w_near >= 1, k0, k1 + g.w_near - 1, r.a0, r.b0);
  clip(g.w_sink >= 1 && k0 < g.w_sink, k0, cmax, r.a1, r.b1);
  clip(g.hi > g.lo, k0 + g.lo, k1 + g.hi - 1, r.a2, r.b2);
  runs3_merge(r);
  return r;
}
__host__ __device__ inline int32_t runs3_count(const Runs3& r) {
  return (r.b0 - r.a0 + 1) + (r.b1 - r.a1 + 1) + (r.b2 - r.a2 + 1);
}

// The dK/dV pass has columns of its own, kColKeys keys of one KV head and sequence,
// and walks a column in steps: one block of 64 queries of one QO head each.
constexpr int kColKeys = 128;

// How a column's steps are cut into parts, whose float32 sums are added in order.
// The cut decides how dK and dV are rounded, so it follows from one KV head of
// one sequence and from the number of heads of the whole model (`heads`)
// alone: a sequence gives the same bits in any batch, and a KV head on any rank.
//   longest   steps of a column past the sink, at most: the near and the
//             long-range run, each spanning up to one block more than its length
//   ordinary  most parts of such a column.  Where the sequence's columns of all
//             heads are few, a workgroup per part fills the device: at most
//             what 0.8 of it takes beyond the first parts (d = 64, two workgroups per
//             compute unit: 448), columns with sink keys, which are cut further,
//             counted as three, and as long as one more part shortens the
//             longest column by more than it costs.
//   sink      most parts of a column with sink keys, which every later query
//             sees: 16, and at most 256 MB of sums over all heads.  Its parts are as
//             long as an ordinary column's, or, where those are whole, half of
//             `longest`, but 128 steps if `longest` has them (8192 tokens, 32/8 heads:
//             parts of 128 steps 441 us, of 72 460)
// Measured (us, 1 / 2 / 3 / 4 / 6 ordinary parts), 32/8 heads, d = 128: 500
// tokens 66 / 52 / 40 / 35 / 32; 1000 95 / 64 / 48 / 65 / 65 (past 256 parts a second
// round); 2048 185 / 116 / 127; 4096 230 / 240.  8/2 heads: 16384 925 / 775.  16/4,
// d = 64: 1000 74 / 48 / 38 / 34 / 30; 4096 146 / 98 / 80 / 86 / 82; 8192 237 / 182 / 193.
struct ColumnRule {
  int32_t longest, ordinary, sink;
};
__host__ __device__ inline ColumnRule column_rule(const Geo32& g, int32_t group, int32_t heads, int32_t head_dim) {
  ColumnRule r;
  const bool wide = head_dim == 128;
  const int32_t width = g.hi - g.lo, bq = (g.n_q + 63) / 64;
  const int32_t near = g.w_near > 0 ? imin32(bq, (kColKeys + g.w_near - 2) / 64 + 2) : 0;
  const int32_t lng = width > 0 ? imin32(bq, (kColKeys + width - 2) / 64 + 2) : 0;
  r.longest = imax32(1, group * imin32(bq, near + lng));
  // (32-bit: capped far above where a column has one part)
  constexpr int32_t kMany = 1 << 20;
  const int32_t h = imin32(heads, kMany);
  const int32_t cols = (int32_t)imin64(kMany, imax64(1, (int64_t)((g.n_k + kColKeys - 1) / kColKeys) * h));
  const int32_t load = cols + (g.w_sink > 0 ? 2 * h : 0), slots = wide ? 256 : 448;
  const int32_t fill = imin32(wide ? 6 : 3, 1 + (8 * slots + 3 * load) / (10 * load));
  // in ns: a step, the launch that sums, a part's start and way through memory
  const int32_t step = (wide ? 2000 : 2600) * imin32(r.longest, 1 << 19), sum = 10000;
  const int32_t part = 1000 + (wide ? 57 : 28) * cols;
  int32_t n = 1;
  // (two parts halve the longest column; with a column per slot they only even out the end)
  if (fill > 1 && step > (cols < slots ? 2 : 8) * (sum + 2 * part)) ++n;
  while (n > 1 && n < fill && step > part * n * (n + 1)) ++n;
  r.ordinary = n;
  const int32_t sinks = (int32_t)imin64(kMany, imax64(1, (int64_t)((g.w_sink + kColKeys - 1) / kColKeys) * h));
  r.sink = imax32(1, imin32(16, 2048 * (128 / head_dim) / sinks));
  return r;
}
// Parts of a column of n_steps steps.
__host__ __device__ inline int32_t column_parts(const ColumnRule& r, bool sink, int32_t n_steps) {
  int32_t len = r.longest, per = r.ordinary;
  if (sink && per == 1) {
    if (len >= 256)
      per = 2;
    else
      len = imin32(len, 128);
  }
  const int32_t most = sink ? r.sink : r.ordinary;
  return n_steps >= 1 << 28 ? most : imax32(1, imin32((n_steps * per + len - 1) / len, most));
}

// Blocks of bk keys that hold a key some query of R consecutive ones sees, at most.
__host__ __device__ inline int64_t row_list_blocks(const Geo32& g, int32_t R, int32_t bk) {
  const int64_t runs = ((int64_t)R + g.w_near) / bk + 2 + ((int64_t)R + g.hi - g.lo) / bk + 2 + (g.w_sink + bk - 1) / bk;
  return imin64(runs, ((int64_t)g.n_k + bk - 1) / bk);
}

// Which shape of the forward and of the dQ pass takes a KV head of a sequence.
// A shape has row tiles and key blocks of its own, which fix how O, LSE and dQ
// are rounded, so the choice follows from that head and that sequence alone (V:
// the visible keys of a row; W: the 256-row tiles of the head's group): a
// sequence gives the same bits in any batch, packed or not, and a head on any
// rank.  Where a call's heads and sequences differ, each shape has a launch that
// takes its own.  The measurements are beside the kernels' launches.
struct RowLoad {
  int64_t v, w;
};
__host__ __device__ inline RowLoad row_load(const Geo32& g, int32_t group) {
  return RowLoad{imin64((int64_t)g.w_near + g.w_sink + (g.hi > g.lo ? g.hi - g.lo : 0), g.n_k), (int64_t)group * g.n_q / 256};
}
// longest block lists that fit beside the buffers of the 64-row shapes (128-key
// blocks, d = 128) and of the dQ pass's 64-key blocks at d = 64
constexpr int32_t kFwdList128 = 8188, kDqList128 = 8192, kDqList64 = 32768;
constexpr int kRowShapes = 3;
// d = 128: 32 rows per wave and 64-key blocks (0) or 64 and 128 (1); d = 64: 32
// rows and 64-key (0) or 128-key blocks (1)
__host__ __device__ inline int32_t fwd_shape(const Geo32& g, int32_t group, int32_t head_dim) {
  const RowLoad r = row_load(g, group);
  if (head_dim == 64) return r.v >= 1024 ? 1 : 0;
  return ((r.v >= 8192 && r.w >= 32) || (r.v >= 4096 && r.w >= 512)) && row_list_blocks(g, 256, 128) <= kFwdList128 ? 1 : 0;
}
// d = 128: 32 rows per wave and 64-key blocks (0), 64 rows and 64-key (1) or 128-key
// blocks (2); d = 64: 32 rows and 64-key blocks (0), or 128-key blocks, which halve
// the list, where a row of more than 2M keys needs it (1)
__host__ __device__ inline int32_t dq_shape(const Geo32& g, int32_t group, int32_t head_dim) {
  const RowLoad r = row_load(g, group);
  if (head_dim == 64) return row_list_blocks(g, 256, 64) > kDqList64 ? 1 : 0;
  if (r.v >= 8192) return r.w >= 32 && row_list_blocks(g, 256, 128) <= kDqList128 ? 2 : 0;
  return r.v >= 4096 && r.w >= 256 ? 1 : 0;
}

// Every pair of queries q0 .. q1 and keys k0 .. k1 lies inside the sequence and
// is legal (tile_full for any query and key range, in 32-bit scalars; bounds
// clamped to n_k).
__host__ __device__ inline bool key_block_full(const Geo32& g, int32_t q0, int32_t q1, int32_t k0, int32_t k1) {
  const int32_t c0 = q0 + g.off, c1 = q1 + g.off;
  const bool in = (q1 < g.n_q) & (k1 < g.n_k) & (k1 <= c0);  // inside, and causal for every pair
  // keys past the sink: every distance in [c0 - k1, c1 - max(k0, sink)] in one window
  const int32_t a = c0 - k1, b = c1 - imax32(k0, g.w_sink);
  const bool win = (b < g.w_near) | ((a >= g.lo) & (b < g.hi)) | ((g.lo == g.w_near) & (b < g.hi));
  return in & ((k1 < g.w_sink) | win);
}

// Up to three inclusive ranges, merged (overlapping or adjacent ranges join).
struct Ranges {
  int32_t n;
  int32_t a[3], b[3];
};

__host__ __device__ inline void ranges_add(Ranges& r, int64_t a, int64_t b) {
  if (a <= b) { r.a[r.n] = (int32_t)a; r.b[r.n] = (int32_t)b; ++r.n; }
}

// Sort by start (ascending) and merge.
__host__ __device__ inline void ranges_merge(Ranges& r) {
  for (int x = 0; x < r.n; ++x)
    for (int y = x + 1; y < r.n; ++y)
      if (r.a[y] < r.a[x]) {
        int32_t ta = r.a[x], tb = r.b[x];
        r.a[x] = r.a[y]; r.b[x] = r.b[y]; r.a[y] = ta; r.b[y] = tb;
      }
  int m = 0;
  for (int x = 0; x < r.n; ++x) {
    if (m > 0 && r.a[x] <= r.b[m - 1] + 1) {
      if (r.b[x] > r.b[m - 1]) r.b[m - 1] = r.b[x];
    } else {
      r.a[m] = r.a[x]; r.b[m] = r.b[x]; ++m;
    }
  }
  r.n = m;
}

__host__ __device__ inline int32_t ranges_count(const Ranges& r) {
  int32_t c = 0;
  for (int x = 0; x < r.n; ++x) c += r.b[x] - r.a[x] + 1;
  return c;
}

// KV-block ranges of J_h(i) (ascending, merged).
__host__ __device__ inline Ranges fwd_block_ranges(const HeadGeo& g, int32_t i) {
  int64_t q0 = (int64_t)i * g.tile_q;
  int64_t q1 = imin64(q0 + g.tile_q, g.n_q) - 1;
  int64_t off = (int64_t)g.n_k - g.n_q;
  int64_t c0 = q0 + off, c1 = q1 + off;  // keys at distance 0 of the first / last query
  Ranges r; r.n = 0;
  if (g.w_near >= 1) ranges_add(r, imax64(0, c0 - g.w_near + 1) / g.tile_k, c1 / g.tile_k);
  if (g.w_sink >= 1) ranges_add(r, 0, imin64(g.w_sink - 1, c1) / g.tile_k);
  if (g.hi > g.lo && c1 - g.lo >= 0) ranges_add(r, imax64(0, c0 - g.hi + 1) / g.tile_k, (c1 - g.lo) / g.tile_k);
  ranges_merge(r);
  return r;
}

// QO-block ranges of I_h(j) (ascending, merged).
__host__ __device__ inline Ranges bwd_block_ranges(const HeadGeo& g, int32_t j) {
  int64_t k0 = (int64_t)j * g.tile_k;
  int64_t k1 = imin64(k0 + g.tile_k, g.n_k) - 1;
  int64_t off = (int64_t)g.n_k - g.n_q;
  int64_t cmin = off, cmax = (int64_t)g.n_k - 1;  // range of distance-0 keys over all queries
  Ranges r; r.n = 0;
  auto add_c = [&](int64_t ca, int64_t cb) {
    ca = imax64(ca, cmin); cb = imin64(cb, cmax);
    if (ca <= cb) ranges_add(r, (ca - off) / g.tile_q, (cb - off) / g.tile_q);
  };
  if (g.w_near >= 1) add_c(k0, k1 + g.w_near - 1);
  if (g.w_sink >= 1 && k0 < g.w_sink) add_c(k0, cmax);
  if (g.hi > g.lo) add_c(k0 + g.lo, k1 + g.hi - 1);
  ranges_merge(r);
  return r;
}

// FULL iff the tile lies inside both sequences and every element pair is legal.
__host__ __device__ inline bool tile_full(const HeadGeo& g, int32_t i, int32_t j) {
  int64_t q0 = (int64_t)i * g.tile_q, k0 = (int64_t)j * g.tile_k;
  if (q0 + g.tile_q > g.n_q || k0 + g.tile_k > g.n_k) return false;
  int64_t q1 = q0 + g.tile_q - 1, k1 = k0 + g.tile_k - 1;
  int64_t off = (int64_t)g.n_k - g.n_q;
  int64_t c0 = q0 + off, c1 = q1 + off;
  if (k0 < g.w_sink) {  // sink keys: legal iff causal
    int64_t ks1 = imin64(k1, (int64_t)g.w_sink - 1);
    if (c0 - ks1 < 0) return false;
  }
  int64_t kn0 = imax64(k0, g.w_sink);
  if (kn0 <= k1) {  // other keys: every distance in [a, b] must be in [0, w_near) u [lo, hi)
    int64_t a = c0 - k1, b = c1 - kn0;
    bool ok = (a >= 0 && b < g.w_near) || (a >= g.lo && b < g.hi) ||
              (g.lo == g.w_near && a >= 0 && b < g.hi);
    if (!ok) return false;
  }
  return true;
}

}  // namespace cowa

namespace cowa {

// Key runs of the single decoding query (N_q = 1, distance-0 key c = N_k - 1),
// ascending and merged: the visible set A_h of Sec. 2.3 (decoding execution).
__host__ __device__ inline Ranges decode_key_runs(int64_t n_k, int64_t w_sink, int64_t w_near, int64_t lo,
                                                  int64_t hi) {
  const int64_t c = n_k - 1;
  Ranges r; r.n = 0;
  if (w_near >= 1) ranges_add(r, imax64(0, c - w_near + 1), c);
  if (w_sink >= 1) ranges_add(r, 0, imin64(w_sink - 1, c));
  if (hi > lo && c - lo >= 0) ranges_add(r, imax64(0, c - hi + 1), c - lo);
  ranges_merge(r);
  return r;
}

}  // namespace cowa
