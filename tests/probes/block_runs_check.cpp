// Host check of the kernels' own block lists (key_block_runs3, query_block_runs3,
// key_block_full)
// against the element rule: random windows (clamped as the kernels clamp
// them), every tile of query rows and key blocks; a block is listed iff it
// holds a legal pair, its ranges ascend without touching, and it is called full
// only if every pair of it is inside the sequence and legal, exactly where the
// schedule's rule (tile_full) says so.
// Build: hipcc -x hip --offload-arch=gfx950 -O1 -I include block_runs_check.cpp
#include "../../paper_2609_32704_amd/csrc/window_rule.h"
#include <stdio.h>
#include <random>
#include <vector>
using namespace cowa;

static long checked = 0, bad = 0;

template <int BK>
void check(HeadGeo hg, int R) {
  hg.tile_q = R;
  hg.tile_k = BK;
  const Geo32 g = geo32(hg);
  const int n_kb = (hg.n_k + BK - 1) / BK;
  for (int q0 = 0; q0 < hg.n_q; q0 += R) {
    const int q1 = (q0 + R < hg.n_q ? q0 + R : hg.n_q) - 1;
    const Runs3 r = key_block_runs3<BK>(g, q0, q1);
    std::vector<char> listed(n_kb, 0);
    const int a[3] = {r.a0, r.a1, r.a2}, b[3] = {r.b0, r.b1, r.b2};
    int last = -2;
    for (int x = 0; x < 3; ++x) {
      if (a[x] == kNone) {
        bad += b[x] != kNone - 1;
        continue;
      }
      bad += a[x] <= last + 1 || a[x] > b[x] || b[x] >= n_kb;
      for (int j = a[x]; j <= b[x] && j < n_kb; ++j) listed[j] = 1;
      last = b[x];
    }
    for (int j = 0; j < n_kb; ++j) {
      bool any = false, all = true;
      for (int q = q0; q < q0 + R; ++q)
        for (int k = j * BK; k < j * BK + BK; ++k) {
          const bool ok = legal_pair(hg, q, k);
          any |= ok;
          all &= ok;
        }
      bad += any != (bool)listed[j];
      const bool full = key_block_full(g, q0, q0 + R - 1, j * BK, j * BK + BK - 1);
      bad += full && !all;
      bad += full != tile_full(hg, q0 / R, j);
      ++checked;
    }
  }
}

// the query blocks of a key block, likewise
template <int BQ>
void check_q(const HeadGeo& hg, int BK) {
  const Geo32 g = geo32(hg);
  const int n_qb = (hg.n_q + BQ - 1) / BQ;
  for (int k0 = 0; k0 < hg.n_k; k0 += BK) {
    const int k1 = (k0 + BK < hg.n_k ? k0 + BK : hg.n_k) - 1;
    const Runs3 r = query_block_runs3<BQ>(g, k0, k1);
    const int a[3] = {r.a0, r.a1, r.a2}, b[3] = {r.b0, r.b1, r.b2};
    std::vector<char> listed(n_qb, 0);
    int last = -2, count = 0;
    for (int x = 0; x < 3; ++x) {
      if (a[x] == kNone) {
        bad += b[x] != kNone - 1;
        continue;
      }
      bad += a[x] <= last + 1 || a[x] > b[x] || b[x] >= n_qb;
      for (int i = a[x]; i <= b[x] && i < n_qb; ++i, ++count) listed[i] = 1;
      last = b[x];
    }
    bad += count != runs3_count(r);
    for (int i = 0; i < n_qb; ++i) {
      bool any = false;
      for (int q = i * BQ; q < i * BQ + BQ; ++q)
        for (int k = k0; k <= k1; ++k) any |= legal_pair(hg, q, k);
      bad += any != (bool)listed[i];
      ++checked;
    }
  }
}

int main() {
  std::mt19937 rng(609);
  auto pick = [&](int lo, int hi) { return std::uniform_int_distribution<int>(lo, hi)(rng); };
  for (int t = 0; t < 600; ++t) {
    HeadGeo hg;
    hg.n_k = pick(1, 700);
    hg.n_q = pick(0, 1) ? hg.n_k : pick(1, hg.n_k);
    hg.w_sink = pick(0, 3) == 0 ? 0 : pick(0, 300);
    hg.w_near = pick(0, 3) == 0 ? 0 : pick(0, 400);
    hg.lo = hg.w_near + (pick(0, 2) == 0 ? 0 : pick(0, 400));
    hg.hi = pick(0, 3) == 0 ? hg.lo : hg.lo + pick(0, 500);
    const int big = pick(0, 9);
    if (big == 0) hg.hi = 1 << 30;  // bounds far past the sequence
    if (big == 1) hg.w_near = 1 << 30;
    if (big == 2) hg.w_sink = 1 << 30;
    const int R = 16 << pick(0, 4);
    check<16>(hg, R);
    check<64>(hg, R);
    check<128>(hg, R);
    check_q<64>(hg, 128);
    check_q<16>(hg, 64);
  }
  printf("checked %ld mismatches %ld\n", checked, bad);
  return bad == 0 ? 0 : 1;
}
