// Where one workgroup's work lives: its sequence, lengths, tensor rows and
// window, for fixed-length and ragged batches alike.
//
// Grids run over (block row) x (unit) x (head group): in a fixed-length batch
// the row is the block within the sequence and unit = b H_k + h_k; in a ragged
// batch the row is the block over the whole batch (sequence b's blocks follow
// those of b - 1) and unit = h_k, the sequence coming from the block-to-
// sequence map of the schedule.
#pragma once

#include "internal.h"
#include "mfma_tiles.h"
#include "window_rule.h"

namespace cowa {

struct SeqCtx {
  int32_t b;         // sequence
  int32_t tile;      // block within the sequence
  int32_t n_q, n_k;  // its lengths
  int64_t q0, qh;    // row (of d elements) of query 0 of QO head 0; + qh per QO head (Q, O, dO, dQ, LSE, D)
  int64_t k0, kh;    // row of key 0 of KV head 0; + kh per KV head (K, V, dK, dV)
  Geo32 g;           // window of (b, h_k), bounds clamped to n_k
};

// Units of the grid: B H_k for fixed lengths, H_k for a ragged batch.
__host__ __device__ inline int grid_units(const cowa_params& p, const SchedView& sv) {
  return sv.ragged ? p.h_k : p.batch * p.h_k;
}

// qside: the row counts QO blocks (forward, dQ pass), else KV blocks (dK/dV pass).
__device__ inline SeqCtx seq_ctx(const cowa_params& p, const SchedView& sv, int row, int unit, bool qside,
                                 int& hk) {
  SeqCtx c;
  const WinDesc* wd;
  if (!sv.ragged) {
    c.b = unit / p.h_k;
    hk = unit % p.h_k;
    c.tile = row;
    c.n_q = p.n_q;
    c.n_k = p.n_k;
    c.q0 = (int64_t)c.b * p.h_q * p.n_q;
    c.qh = p.n_q;
    c.k0 = (int64_t)c.b * p.h_k * p.n_k;
    c.kh = p.n_k;
    wd = sv.win + hk;
  } else {
    hk = unit;
    c.b = (qside ? sv.qt_seq : sv.kt_seq)[row];
    const SeqDesc sd = sv.seq[c.b];
    c.tile = row - (qside ? sd.qt_off : sd.kt_off);
    c.n_q = sd.n_q;
    c.n_k = sd.n_k;
    c.q0 = sd.q_start;
    c.qh = p.n_q;
    c.k0 = sd.k_start;
    c.kh = p.n_k;
    wd = sv.win + (sv.per_seq_win ? c.b * p.h_k : 0) + hk;
  }
  const WinDesc w = *wd;
  c.g.off = c.n_k - c.n_q;
  c.g.w_near = w.near < c.n_k ? w.near : c.n_k;
  c.g.w_sink = w.sink < c.n_k ? w.sink : c.n_k;
  c.g.lo = w.lo < c.n_k ? w.lo : c.n_k;
  c.g.hi = w.hi < c.n_k ? w.hi : c.n_k;
  c.g.n_q = c.n_q;
  c.g.n_k = c.n_k;
  return c;
}

// Row tiles of a kernel that cuts the queries into its own tiles of R rows
// instead of the schedule's: rows (tiles) of the grid, R, and QO heads per
// workgroup.  Fixed lengths: ceil(N_q / R) rows.  A ragged batch keeps the
// schedule's block-to-sequence map: tile_q / R rows per schedule tile, or, when
// R exceeds tile_q, one row per schedule tile of which every (R / tile_q)-th
// of a sequence starts R rows and the others hold nothing.
// The grid is cut into clusters of cq consecutive rows x the head groups of one
// KV head; cluster c runs on XCD c % 8 (workgroups are dealt to the XCDs
// round-robin by id), so that its workgroups, which stream nearly the same K/V
// blocks, share that XCD's L2.  A cluster spans about 2048 queries: 32 or 64
// workgroups, what an XCD's 32 compute units run at once, for groups of four
// heads; fewer rows when there are less than 16 clusters per XCD (rows of
// unequal length must spread over many clusters to load every XCD alike).
// Rows go out last (longest) to first, whole cluster rows at a time; the unit
// (KV head) of an XCD's cluster rotates from one row range to the next.
// Rows and clusters are rounded up; the padding's workgroups end at once.
struct RowTiles {
  int32_t n_rows, R, hpw, cq, blocks;
  int32_t shape;  // take only the heads of this shape (fwd_shape, dq_shape), or all of them (-1)
};
inline RowTiles row_tiles(const cowa_params& p, const SchedView& sv, int hpw, int R, int shape) {
  RowTiles t;
  t.shape = shape;
  t.R = R;
  t.hpw = hpw;
  if (!sv.ragged)
    t.n_rows = (p.n_q + R - 1) / R;
  else
    t.n_rows = R <= p.tile_q ? sv.n_qt * (p.tile_q / R) : sv.n_qt;
  const int units = grid_units(p, sv), groups = p.h_q / p.h_k / hpw;
  t.cq = cluster_rows(t.n_rows, units, 2048 / R);
  const int64_t clusters = ((int64_t)units * ((t.n_rows + t.cq - 1) / t.cq) + 7) / 8 * 8;
  t.blocks = (int32_t)(clusters * t.cq * groups);
  return t;
}
// Workgroup id -> (row, unit, group); false: padding.
__device__ inline bool row_item(const RowTiles& t, int units, int groups, int id, int& row, int& unit, int& group) {
  const int cs = t.cq * groups;  // workgroups per cluster
  const int n = id >> 3, c = (n / cs) * 8 + (id & 7), item = n % cs;
  const int r = c / units;
  unit = (c % units + r) % units;
  group = item % groups;
  row = t.n_rows - 1 - (r * t.cq + item / groups);
  return row >= 0;
}
// Context of row tile `row`; q0: its first query (>= n_q: the tile is empty).
__device__ inline SeqCtx row_ctx(const cowa_params& p, const SchedView& sv, const RowTiles& rt, int row, int unit, int& hk,
                                 int& q0) {
  if (!sv.ragged) {
    q0 = row * rt.R;
    return seq_ctx(p, sv, row, unit, true, hk);
  }
  const bool sub = rt.R <= p.tile_q;
  const int n = sub ? p.tile_q / rt.R : 1, m = sub ? 1 : rt.R / p.tile_q;
  const SeqCtx sc = seq_ctx(p, sv, row / n, unit, true, hk);
  q0 = sc.tile % m != 0 ? sc.n_q : sc.tile * p.tile_q + (row % n) * rt.R;
  return sc;
}

// The block list of the row tile of queries q0 .. q_last (of at most R), into
// LDS: full blocks from the front, partial ones from the back, both by
// descending key.  Every wave computes the same counts; wave 0 writes.  Returns
// the number of full blocks.
template <int BK>
__device__ inline int build_row_list(const Geo32& g, int q0, int q_last, int R, uint32_t* list, int cap, int wave, int lane,
                                     int& n_ent) {
  const Runs3 runs = key_block_runs3<BK>(g, q0, q_last);
  const int n0 = runs.b0 - runs.a0 + 1, n1 = n0 + runs.b1 - runs.a1 + 1;
  n_ent = n1 + runs.b2 - runs.a2 + 1;
  int n_full = 0;
  for (int c0 = 0; c0 < n_ent; c0 += 64) {
    const int t = n_ent - 1 - (c0 + lane);
    const bool in = t >= 0;
    const int j = t < n0 ? runs.a0 + t : t < n1 ? runs.a1 + (t - n0) : runs.a2 + (t - n1);
    const bool is_full = key_block_full(g, q0, q0 + R - 1, j * BK, j * BK + BK - 1);
    const uint64_t full = __ballot(in && is_full);
    const uint64_t part = __ballot(in && !is_full);
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    if (wave == 0 && in)
      list[is_full ? n_full + __popcll(full & below) : cap - 1 - (c0 - n_full + __popcll(part & below))] = (uint32_t)j;
    n_full += __popcll(full);
  }
  return n_full;
}

}  // namespace cowa
