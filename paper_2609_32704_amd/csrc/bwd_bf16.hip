// CoWA backward in bfloat16 on the CDNA4 matrix cores (Alg. 2).
//
// Three launches on the caller's stream:
//
//  1. bwd_pre: D = rowsum(O * dO) per query row (fp32).
//  2. bwd_main (dK, dV): one workgroup of four waves per (column of 128 keys,
//     local KV head h_k, sequence b), or per part of a column (BwdSplit).  K and V
//     of the column stay in registers for the whole workgroup (wave w owns keys
//     [32 w, 32 w + 32)).  The workgroup walks every QO head of the group and,
//     for each, the blocks of 64 queries that see the column (its own list,
//     computed from the windows), one per step; Q and dO of the step after next
//     are copied global -> LDS while the current step computes
//       S = Q K^T, dP = dO V^T, P = exp(S - LSE), dS = P (dP - D),
//       dV^T += dO^T P, dK^T += scale Q^T dS.
//     dK and dV of the column are summed over every QO head of the group
//     inside the workgroup and written once, without atomics; keys that no
//     query sees get zeros.  64-key columns (what 64-key schedule tiles got
//     before) need every wave to read all of Q and dO for 16 keys: 2.5 us per
//     step and CU for half the products of a 2.0 us step here.
//  3. the dQ pass (dq_bf16.hip).  Alg. 2 adds dQ contributions of different KV
//     blocks with atomics; at the paper's 128K scale that is ~5e10 fp32 atomic
//     adds, more than the L2 atomic units sustain, so dQ is instead computed in
//     its own pass that recomputes S and dP (4d extra FLOPs per legal pair) and
//     writes each dQ row once.
#include "internal.h"
#include "window_rule.h"
#include "mfma_tiles.h"
#include "work_item.h"

namespace cowa {
namespace {

// Per query row: nd = -D with D = sum_d O[row, d] dO[row, d] (D/8 lanes per
// row), and nl = -LSE log2(e), the row's exponent offset in base 2; the dK/dV
// pass folds nd into the accumulator input of dP = dO V^T (dP - D comes out of
// the products) and adds nl to the scaled scores.
template <int D>
__global__ void __launch_bounds__(256) bwd_pre(const __bf16* __restrict__ o, const __bf16* __restrict__ d_o,
                                               const float* __restrict__ lse, float* __restrict__ nd,
                                               float* __restrict__ nl, int64_t rows) {
  constexpr int CH = D / 8;
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t row = c / CH;
  const int ch = (int)(c % CH);
  float part = 0.f;
  if (row < rows) {
    const uint4 a = *reinterpret_cast<const uint4*>(o + row * D + ch * 8);
    const uint4 g = *reinterpret_cast<const uint4*>(d_o + row * D + ch * 8);
    const uint32_t aw[4] = {a.x, a.y, a.z, a.w}, gw[4] = {g.x, g.y, g.z, g.w};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      part = fmaf(__uint_as_float(aw[t] << 16), __uint_as_float(gw[t] << 16), part);
      part = fmaf(__uint_as_float(aw[t] & 0xffff0000u), __uint_as_float(gw[t] & 0xffff0000u), part);
    }
  }
#pragma unroll
  for (int off = 1; off < CH; off <<= 1) part += __shfl_xor(part, off);
  if (row < rows && ch == 0) {
    nd[row] = -part;
    nl[row] = -lse[row] * kLog2e;
  }
}

template <int D>
struct BwdCfg {
  static constexpr int NW = 4;            // waves per workgroup
  static constexpr int BK = kColKeys;     // keys per column
  static constexpr int BQ = 64;           // query rows per step
  static constexpr int NKW = BK / NW;     // keys per wave
  static constexpr int NTK = NKW / 16;    // key tiles per wave
  static constexpr int MTQ = BQ / 16;     // query tiles per step
  static constexpr int KSD = D / 32;      // k-steps over d
  static constexpr int MD = D / 16;       // d tiles
  static constexpr int KSQ = BQ / 32;     // k-steps over queries
  using QT = SwzTile<D, BQ>;              // Q or dO rows of one step
  static constexpr int ROWV = 2 * BQ * 4; // per-step row values: LSE [BQ], then D [BQ]
  // LDS: a ring of three stages (Q, dO, row values), then the column's entry lists
  static constexpr int NST = 3;
  __device__ static int q_off(int s) { return s * QT::BYTES; }
  __device__ static int do_off(int s) { return (NST + s) * QT::BYTES; }
  __device__ static int rv_off(int s) { return 2 * NST * QT::BYTES + s * ROWV; }
  static constexpr int MAIN_BYTES = 2 * NST * QT::BYTES + NST * ROWV;
  static constexpr int LOADS_PER_STEP = 2 * QT::LOADS / NW + 1;  // direct loads each wave issues per step
  static constexpr int OUT_BYTES = 2 * BK * (D + 8) * 2;        // dK, dV staging at the end
  static constexpr int LDS_MAX = 160 * 1024;
  // LDS with a list of up to n_qb blocks of BQ queries (16 bits each)
  static int lds_bytes(int n_qb) {
    const int main = MAIN_BYTES + 2 * n_qb;
    return main > OUT_BYTES ? main : OUT_BYTES;
  }
  static int max_qblocks() { return (LDS_MAX - MAIN_BYTES) / 2; }
};

// Workgroups of the pass (BwdSplit): the first n_extra (a multiple of 8, so the
// XCD order of the others is unchanged) take parts 1 .. P-1 of the sink columns;
// the others take n_items columns x PO parts (part 0 of a sink column).  With an
// order table the items are its columns, longest first, each with the batch
// entries and parts side by side (past two workgroups per compute unit in
// chunks of 8 per XCD, so that neighbours share its L2); without one, or with more
// columns than kMaxOrdered unless each is walked whole, they are clusters of 32
// consecutive columns of one KV head that share an XCD's L2.
// Measured (us, clusters / longest first): 8192 tokens, 32/8 heads 516 / 469; 4 x
// 2048 288 / 231; 16384 1199 / 1142; 131072 of one KV head 6930 / 6887; 32768
// (2048 columns) 3977 / 4056.
struct SplitArgs {
  float* part;       // BwdWork::part
  int32_t S, P, PO;  // BwdSplit
  int32_t heads;     // KV heads of the whole model (column_rule)
  int32_t n_extra;   // workgroups of parts 1 .. P-1, rounded up to a multiple of 8
  int32_t rows;      // column rows (column_rows)
  int32_t n_items;   // columns of the grid
  int64_t other;     // first partial of the other columns
  int32_t cap;       // list capacity
};

// The column of (unit, row): its context and first key; false: none starts there.
__device__ inline bool column_ctx(const cowa_params& p, const SchedView& sv, int row, int unit, int& hk, SeqCtx& sc, int& k_first) {
  sc = seq_ctx(p, sv, row, unit, false, hk);
  k_first = sv.ragged ? sc.tile * p.tile_k : row * kColKeys;
  return k_first % kColKeys == 0 && k_first < sc.n_k;
}
// Part `part` of the column at k_first_ of (sequence sc.b, local KV head hk), or,
// WALK, all of its parts, in order (BwdSplit::walk).
template <int D, bool WALK>
__device__ __forceinline__ void walk_column(const cowa_params& p, const SchedView& sv, const SplitArgs& sa,
                                            const __bf16* q, const __bf16* k, const __bf16* v, const __bf16* d_o,
                                            const float* nl, const float* nd, __bf16* dk, __bf16* dv,
                                            unsigned char* smem, int part, int row, int unit, int hk, const SeqCtx& sc,
                                            int k_first_) {
  using C = BwdCfg<D>;
  constexpr int NW = C::NW, BK = C::BK;
  const int j = k_first_ / BK;  // column within the sequence
  const int G = p.h_q / p.h_k;
  const Geo32 g = sc.g;
  const int n_q = sc.n_q, n_k = sc.n_k;

  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int lr = lane & 15, lg = lane >> 4;
  const int64_t k_first = k_first_;
  const int64_t kv_row0 = sc.k0 + (int64_t)hk * sc.kh;
  const __bf16* kbase = k + kv_row0 * D;
  const __bf16* vbase = v + kv_row0 * D;

  // The steps: every QO head of the group x every block of 64 queries that sees
  // the column.  Full blocks are taken first, then partial ones, so that each
  // of the two step loops below is straight-line code (the partial loop adds
  // the element mask).  The blocks (up to three merged ranges, computed from the
  // windows) go into two lists in LDS: full ones from the front, partial ones
  // from the back, ascending.
  const int k_last = (int)k_first + BK < n_k ? (int)k_first + BK - 1 : n_k - 1;
  const Runs3 runs = query_block_runs3<C::BQ>(g, (int)k_first, k_last);
  const int r0 = runs.b0 - runs.a0 + 1, r1 = r0 + runs.b1 - runs.a1 + 1, n_ent = r1 + runs.b2 - runs.a2 + 1;
  const int n_steps = G * n_ent;
  const int n_parts = column_parts(column_rule(g, G, sa.heads, D), (int)k_first < g.w_sink, n_steps);
  if (part >= n_parts) return;
  const int cap = sa.cap;
  uint16_t* list = reinterpret_cast<uint16_t*>(smem + C::MAIN_BYTES);
  int n_full = 0;
  for (int c0 = 0; c0 < n_ent; c0 += 64) {  // every wave builds the same counts; wave 0 writes
    const int t = c0 + lane;
    const bool in = t < n_ent;
    const int i = t < r0 ? runs.a0 + t : t < r1 ? runs.a1 + (t - r0) : runs.a2 + (t - r1);
    const bool is_full = key_block_full(g, i * C::BQ, i * C::BQ + C::BQ - 1, (int)k_first, (int)k_first + BK - 1);
    const uint64_t full = __ballot(in && is_full);
    const uint64_t prt = __ballot(in && !is_full);
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    if (wave == 0 && in)
      list[is_full ? n_full + __popcll(full & below) : cap - 1 - (c0 - n_full + __popcll(prt & below))] = (uint16_t)i;
    n_full += __popcll(full);
  }
  const int n_part = n_ent - n_full;
  const int steps_full = G * n_full;
  // this workgroup's steps: part `part` of n_parts contiguous shares, or all of them
  auto part_end = [&](int x) { return (int)((int64_t)n_steps * (x + 1) / n_parts); };
  const int s_begin = part_end(part - 1);
  const int s_end = WALK ? n_steps : part_end(part);
  // cursor (phase: 0 full / 1 partial, QO head, list index) of step s_begin
  int c_ph, c_k, c_hh;
  {
    c_ph = s_begin < steps_full ? 0 : 1;
    const int r = c_ph ? s_begin - steps_full : s_begin;
    const int nl_ = c_ph ? n_part : n_full;
    c_hh = nl_ > 0 ? r / nl_ : 0;
    c_k = nl_ > 0 ? r % nl_ : 0;
  }
  int n1_ph = c_ph, n1_hh = c_hh, n1_k = c_k;  // the next step (staged)
  int n2_ph = c_ph, n2_hh = c_hh, n2_k = c_k;  // the step after (being staged)
  auto advance = [&](int& ph, int& hh, int& kk) {
    if (++kk == (ph == 0 ? n_full : n_part)) {
      kk = 0;
      if (++hh == G) {
        hh = 0;
        ++ph;
        if (ph == 1 && n_part == 0) ph = 2;  // past the end
      }
    }
  };
  // list entry of a cursor; a cursor past the end names the first entry
  auto entry_of = [&](int ph, int kk) -> int {
    const int idx = ph == 0 ? kk : (ph == 1 ? cap - 1 - kk : (n_full > 0 ? 0 : cap - 1));
    return __builtin_amdgcn_readfirstlane((int)list[idx]);
  };

  // Every operand of a step goes global -> LDS directly, through copies the
  // compiler does not track (dma16_buf/dma4): the Q and dO tiles, and the LSE and
  // D values of its 64 rows (waves 0 and 2 copy the LSE, 1 and 3 the D values,
  // the same data twice).  Each wave issues LOADS_PER_STEP copies per step and
  // waits for them two steps later.  Rows past n_q (partial blocks only, where
  // the mask gives them P = 0) hold zeros or an earlier step's rows.  A cursor
  // past the last step stages a copy of the last head's rows, never read.
  const uint32_t smem_base = lds_addr(smem);
  // Each lane copies the same 16-byte column of its row in every 1 KB piece it
  // takes: its byte offsets within a tile are fixed, and the tile position
  // goes into the (scalar) buffer resource, whose size bounds the reads to the
  // sequence (rows past n_q read as zero).
  constexpr int RPL = 1024 / (D * 2);     // rows per 1 KB piece
  constexpr int PPW = C::QT::LOADS / NW;  // pieces per wave and tile
  uint32_t tile_off[PPW];
  {
    const int row0 = wave * RPL + lane / C::QT::CH;
    const int col = (lane % C::QT::CH) ^ swz<C::QT::CH>(row0);
#pragma unroll
    for (int n = 0; n < PPW; ++n) tile_off[n] = (uint32_t)(((n * NW * RPL + row0) * D + col * 8) * 2);
  }
  // A step's copies are issued in pieces (piece n: 1 KB of Q and of dO per
  // wave; and the row values), one piece every other product group early in
  // the step two before it: issued back to back they hold the wave at the
  // vector memory queue for hundreds of cycles.  (Spread over the whole step
  // they would keep more scalar registers live than the kernel has.)
  struct StageSrc {
    int64_t off;       // byte offset of the step's first row in Q and in dO
    uint32_t bytes;    // bytes from there to the end of the sequence
    const float* rv;   // this lane's LSE or D value
  };
  auto stage_src = [&](int ent, int hh) -> StageSrc {
    hh = hh < G ? hh : G - 1;
    const int q0 = ent * C::BQ;
    const int64_t row_base = sc.q0 + (int64_t)(hk * G + hh) * sc.qh;
    const uint32_t bytes = (uint32_t)(n_q - q0) * D * 2;
    const int r = q0 + lane;
    const int rc = r < n_q ? r : n_q - 1;
    return StageSrc{(row_base + q0) * D * 2, bytes, ((wave & 1) ? nd : nl) + row_base + rc};
  };
  auto stage_piece = [&](const StageSrc& src, int n, int slot) {
    const unsigned char* qb = reinterpret_cast<const unsigned char*>(q) + src.off;
    const unsigned char* ob = reinterpret_cast<const unsigned char*>(d_o) + src.off;
    dma16_buf(tile_off[n], buffer_rsrc(qb, src.bytes), smem_base + C::q_off(slot) + (n * NW + wave) * 1024);
    dma16_buf(tile_off[n], buffer_rsrc(ob, src.bytes), smem_base + C::do_off(slot) + (n * NW + wave) * 1024);
  };
  auto stage_rows = [&](const StageSrc& src, int slot) {
    dma4(src.rv, __builtin_amdgcn_readfirstlane(smem_base + C::rv_off(slot) + (wave & 1) * C::BQ * 4));
  };
  auto stage = [&](int ent, int hh, int slot) {
    const StageSrc src = stage_src(ent, hh);
#pragma unroll
    for (int n = 0; n < PPW; ++n) stage_piece(src, n, slot);
    stage_rows(src, slot);
  };

  // rows past the end of the sequence are not copied: give them finite values
  for (int x = tid; x < 2 * C::NST * C::QT::BYTES / 16; x += blockDim.x)
    reinterpret_cast<uint4*>(smem)[x] = uint4{0u, 0u, 0u, 0u};
  __syncthreads();  // the entry lists and the zeroed stages are in LDS
  // prologue: the first two steps in flight
  if (s_end > s_begin) {
    stage(entry_of(n2_ph, n2_k), n2_hh, 0);  // step s_begin
    advance(n2_ph, n2_hh, n2_k);
    n1_ph = n2_ph, n1_hh = n2_hh, n1_k = n2_k;
    stage(entry_of(n2_ph, n2_k), n2_hh, 1);  // step 1
    advance(n2_ph, n2_hh, n2_k);
  }

  // K and V rows of this wave's keys as B fragments: key nt*16 + lr, d = ks*32 + 8*lg + 0..7
  bf16x8 kf[C::NTK][C::KSD], vf[C::NTK][C::KSD];
#pragma unroll
  for (int nt = 0; nt < C::NTK; ++nt) {
    int64_t kp = k_first + wave * C::NKW + nt * 16 + lr;
    if (kp >= n_k) kp = n_k - 1;  // masked: such keys are in partial blocks only
#pragma unroll
    for (int ks = 0; ks < C::KSD; ++ks) {
      kf[nt][ks] = *reinterpret_cast<const bf16x8*>(kbase + kp * D + ks * 32 + 8 * lg);
      vf[nt][ks] = *reinterpret_cast<const bf16x8*>(vbase + kp * D + ks * 32 + 8 * lg);
    }
  }
  f32x4 dka[C::MD][C::NTK], dva[C::MD][C::NTK];  // dK^T / scale, dV^T: rows d, columns keys
#pragma unroll
  for (int md = 0; md < C::MD; ++md)
#pragma unroll
    for (int nt = 0; nt < C::NTK; ++nt) {
      dka[md][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
      dva[md][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  // per-lane LDS offsets of the row-fragment and transposing reads
  int offr[C::KSD], offt[C::MD];
#pragma unroll
  for (int ks = 0; ks < C::KSD; ++ks) offr[ks] = row8_off<D>(lr, lg, ks);
#pragma unroll
  for (int md = 0; md < C::MD; ++md) offt[md] = tr8_off<D>(lr, lg, md);
  const float c = p.softmax_scale * kLog2e;
  const int k0 = (int)k_first + wave * C::NKW + lr;  // key of column nt*16 + lr
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  // One step on ring slot `slot`:
  //   S = Q K^T, dP = dO V^T, P = exp(S - LSE), dS = P (dP - D),
  //   dV^T += dO^T P, dK^T += Q^T dS (the softmax scale is applied to dK at the end).
  // The 64 rows are taken in two halves of 32 (one k-step of the dV/dK
  // products).  The step is a fixed schedule of groups of four MFMAs, each
  // with the LDS reads of the next group and, where there is one, a chunk of a
  // softmax, so that the matrix cores always have independent work while the
  // vector units run the exponentials:
  //   S/dP(half 0) | S/dP(half 1) + softmax(half 0) | dV/dK(half 0) + softmax(half 1) | dV/dK(half 1)
  // Scheduling fences between groups keep that order.
  f32x4 sacc[C::MTQ][C::NTK], pacc[C::MTQ][C::NTK];  // rows q = mt*16 + 4*lg + r, column key = nt*16 + lr
  bf16x8 pb[C::KSQ][C::NTK], sb[C::KSQ][C::NTK];     // P and dS as B operands, k-slots = queries of a half
  constexpr int NG = 2 * C::KSD;  // S/dP groups per half: (k-step, query tile)
  static_assert(C::MTQ == 4 && C::MD == NG && (8 * C::NTK) % NG == 0, "group schedule layout");
  // S/dP group gi of half hf: k-step gi / 2, query tile 2 hf + gi % 2
  auto sdp_load = [&](const unsigned char* qs, const unsigned char* dos, int hf, int gi, bf16x8& fa, bf16x8& fb) {
    const int ks = gi >> 1, mt = 2 * hf + (gi & 1);
    fa = ld_row8(qs + offr[ks] + mt * 16 * D * 2);
    fb = ld_row8(dos + offr[ks] + mt * 16 * D * 2);
  };
  // (dP accumulates on top of -D of its rows, so it holds dP - D)
  auto sdp_mfma = [&](int hf, int gi, const bf16x8& fa, const bf16x8& fb, const f32x4 (&nd4)[C::MTQ]) {
    const int ks = gi >> 1, mt = 2 * hf + (gi & 1);
#pragma unroll
    for (int nt = 0; nt < C::NTK; ++nt) {
      sacc[mt][nt] = mfma16(fa, kf[nt][ks], ks == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sacc[mt][nt]);
      pacc[mt][nt] = mfma16(fb, vf[nt][ks], ks == 0 ? nd4[mt] : pacc[mt][nt]);
    }
  };
  // dV/dK group md of half hf: d tile md, queries of the half as k-slots
  auto dvdk_load = [&](const unsigned char* qs, const unsigned char* dos, int hf, int md, bf16x8& fa, bf16x8& fb) {
    fa = ld_tr8(dos + offt[md] + hf * 32 * D * 2, D * 2);
    fb = ld_tr8(qs + offt[md] + hf * 32 * D * 2, D * 2);
  };
  auto dvdk_mfma = [&](int hf, int md, const bf16x8& fa, const bf16x8& fb) {
#pragma unroll
    for (int nt = 0; nt < C::NTK; ++nt) {
      dva[md][nt] = mfma16(fa, pb[hf][nt], dva[md][nt]);
      dka[md][nt] = mfma16(fb, sb[hf][nt], dka[md][nt]);
    }
  };
  // Softmax chunk ci of half hf: elements e = ci * EPC .. ci * EPC + EPC - 1 of
  // the lane's 8 NTK, where element e is row r = e % 4 of the lane's four in
  // query tile 2 hf + e / (4 NTK), key tile (e / 4) % NTK.  P and dS are rounded
  // to bf16 into the B-operand layout: k-slot 4 i + r is query row
  // (2 hf + i) * 16 + 4 lg + r.  In a partial block the masked pairs get P = 0
  // through a -inf exponent, selected after the exponent has read the MFMA result.
  constexpr int EPC = 8 * C::NTK / NG;
  // (the row values are nl = -LSE log2(e), so x = S c + nl = (S - LSE) log2(e);
  // pacc already holds dP - D)
  // In a partial block the window rule comes as a bit mask over the half's 32
  // query rows per key (once per half and key tile, shifted to the lane's rows
  // 4 lg + 16 i + r); an illegal pair's exponent becomes -inf by a bit select.
  uint32_t qmask[C::NTK];
  auto soft_chunk = [&](int hf, int ci, const float4 (&l4)[2], bool masked, int q0) {
    if (masked && ci == 0)
#pragma unroll
      for (int nt = 0; nt < C::NTK; ++nt) qmask[nt] = legal_queries32(g, q0 + 32 * hf, k0 + nt * 16) >> (4 * lg);
#pragma unroll
    for (int jj = 0; jj < EPC; ++jj) {
      const int e = ci * EPC + jj, r = e & 3, nt = (e >> 2) % C::NTK, i = e / (4 * C::NTK), mt = 2 * hf + i;
      const float lv = r == 0 ? l4[i].x : r == 1 ? l4[i].y : r == 2 ? l4[i].z : l4[i].w;
      float x = fmaf(sacc[mt][nt][r], c, lv);
      // (a row of a full block has a finite LSE; a masked pair may have LSE = -inf)
      if (masked) {
        const uint32_t m = (uint32_t)((int32_t)(qmask[nt] << (31 - (16 * i + r))) >> 31);
        x = __uint_as_float((__float_as_uint(x) & m) | (0xff800000u & ~m));
      }
      const float pv = __builtin_amdgcn_exp2f(x);
      pb[hf][nt][4 * i + r] = (__bf16)pv;
      sb[hf][nt][4 * i + r] = (__bf16)(pv * pacc[mt][nt][r]);
    }
  };
  // nl of query tile 2 hf + i (the lane's rows 4 lg .. 4 lg + 3)
  auto load_rowv = [&](const float* rowv, int hf, int i, float4 (&l4)[2]) {
    l4[i] = *reinterpret_cast<const float4*>(rowv + (2 * hf + i) * 16 + 4 * lg);
  };

  int slot = 0;  // ring slot of the step being computed (t mod 3)
  auto step = [&](bool masked) {
    const int slot2 = slot == 0 ? 2 : slot - 1;  // (t + 2) mod 3
    const unsigned char* qs = smem + C::q_off(slot);
    const unsigned char* dos = smem + C::do_off(slot);
    const float* rowv = reinterpret_cast<const float*>(smem + C::rv_off(slot));
    const int q0 = entry_of(c_ph, c_k) * C::BQ;
    const StageSrc src2 = stage_src(entry_of(n2_ph, n2_k), n2_hh);

    // groups 0 .. 4 NG - 1: S/dP(half 0), S/dP(half 1), dV/dK(half 0), dV/dK(half 1);
    // operand fragments are read PD groups ahead of their MFMAs
    constexpr int NGT = 4 * NG, PD = 1;
    static_assert(2 * PPW <= NGT, "copy pieces per step");
    auto load_group = [&](int gg, bf16x8& fa, bf16x8& fb) {
      if (gg < NG)
        sdp_load(qs, dos, 0, gg, fa, fb);
      else if (gg < 2 * NG)
        sdp_load(qs, dos, 1, gg - NG, fa, fb);
      else if (gg < 3 * NG)
        dvdk_load(qs, dos, 0, gg - 2 * NG, fa, fb);
      else
        dvdk_load(qs, dos, 1, gg - 3 * NG, fa, fb);
    };
    bf16x8 fa[PD + 1], fb[PD + 1];
    float4 l4[2];  // nl of the half in the softmax
    f32x4 nd4[C::MTQ];  // -D of the step's rows, the accumulator input of dP
#pragma unroll
    for (int mt = 0; mt < C::MTQ; ++mt) nd4[mt] = *reinterpret_cast<const f32x4*>(rowv + C::BQ + mt * 16 + 4 * lg);
#pragma unroll
    for (int gg = 0; gg < PD; ++gg) load_group(gg, fa[gg], fb[gg]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int gg = 0; gg < NGT; ++gg) {
      if (gg + PD < NGT) load_group(gg + PD, fa[(gg + PD) % (PD + 1)], fb[(gg + PD) % (PD + 1)]);
      if (gg % 2 == 0 && gg < 2 * PPW) stage_piece(src2, gg / 2, slot2);
      if (gg == 1) stage_rows(src2, slot2);
      // the row values of a half's first and second query tile are needed by
      // its softmax chunks [0, NG/2) and [NG/2, NG); each is loaded once the
      // previous half no longer reads that register
      if (gg == NG - 2) {
        load_rowv(rowv, 0, 0, l4);
        load_rowv(rowv, 0, 1, l4);
      }
      if (gg == NG + NG / 2) load_rowv(rowv, 1, 0, l4);
      if (gg == 2 * NG) load_rowv(rowv, 1, 1, l4);
      bf16x8& a0 = fa[gg % (PD + 1)];
      bf16x8& b0 = fb[gg % (PD + 1)];
      if (gg < NG)
        sdp_mfma(0, gg, a0, b0, nd4);
      else if (gg < 2 * NG)
        sdp_mfma(1, gg - NG, a0, b0, nd4);
      else if (gg < 3 * NG)
        dvdk_mfma(0, gg - 2 * NG, a0, b0);
      else
        dvdk_mfma(1, gg - 3 * NG, a0, b0);
      if (gg >= NG && gg < 2 * NG) soft_chunk(0, gg - NG, l4, masked, q0);
      if (gg >= 2 * NG && gg < 3 * NG) soft_chunk(1, gg - 2 * NG, l4, masked, q0);
      __builtin_amdgcn_sched_barrier(0);
    }

    // Register placement (the library builds this file with MFMA results in
    // VGPRs): the dK/dV accumulators stay in VGPRs and the K/V fragments in
    // AGPRs, which the MFMAs read directly as B operands.  These empty
    // statements emit nothing; they only pin the register class across steps
    // (otherwise the allocator shuffles values between the two files).
#pragma unroll
    for (int md = 0; md < C::MD; ++md)
#pragma unroll
      for (int nt = 0; nt < C::NTK; ++nt) asm volatile("" : "+v"(dka[md][nt]), "+v"(dva[md][nt]));
#pragma unroll
    for (int nt = 0; nt < C::NTK; ++nt)
#pragma unroll
      for (int ks = 0; ks < C::KSD; ++ks) asm volatile("" : "+a"(kf[nt][ks]), "+a"(vf[nt][ks]));
    // the next step's operands have landed (only the step after may still be in
    // flight), for every wave; and this step's slot is no longer read
    __builtin_amdgcn_s_waitcnt(vmcnt_only(C::LOADS_PER_STEP));
    __syncthreads();
    c_ph = n1_ph, c_k = n1_k;
    n1_ph = n2_ph, n1_hh = n2_hh, n1_k = n2_k;
    advance(n2_ph, n2_hh, n2_k);
    slot = slot == 2 ? 0 : slot + 1;
  };
  const float scale = p.softmax_scale;
  int t = s_begin;
  if constexpr (WALK) {
    // part after part: a part's sums start at zero and are added to those of the
    // parts before, as where a workgroup per part and the second kernel do it
    // (the product by the scale is not fused with the sum there either)
    f32x4 dks[C::MD][C::NTK], dvs[C::MD][C::NTK];
    for (; part < n_parts; ++part) {
      const int end = part_end(part);
      for (; t < (end < steps_full ? end : steps_full); ++t) step(false);
      for (; t < end; ++t) step(true);
#pragma unroll
      for (int md = 0; md < C::MD; ++md)
#pragma unroll
        for (int nt = 0; nt < C::NTK; ++nt) {
          f32x4 a = scale * dka[md][nt];
          asm volatile("" : "+v"(a));
          dks[md][nt] = part == 0 ? a : dks[md][nt] + a;
          dvs[md][nt] = part == 0 ? dva[md][nt] : dvs[md][nt] + dva[md][nt];
          dka[md][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
          dva[md][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
#pragma unroll
    for (int md = 0; md < C::MD; ++md)
#pragma unroll
      for (int nt = 0; nt < C::NTK; ++nt) dka[md][nt] = dks[md][nt], dva[md][nt] = dvs[md][nt];
  } else {
    for (; t < (s_end < steps_full ? s_end : steps_full); ++t) step(false);
    for (; t < s_end; ++t) step(true);
  }

  // the copies staged past the last step must land before their LDS is reused
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (!WALK && n_parts > 1) {
    // float32 partials in register order: element ((md NTK + nt) NW + wave) 64 + lane
    // holds rows d = 16 md + 4 (lane / 16) + 0..3, key wave NKW + 16 nt + lane % 16
    const int64_t col = sa.P > 1 && j < sa.S ? ((int64_t)(sc.b * p.h_k + hk) * sa.S + j) * sa.P + part
                                             : sa.other + ((int64_t)unit * sa.rows + row) * sa.PO + part;
    f32x4* pk = reinterpret_cast<f32x4*>(sa.part + col * 2 * BK * D);
    f32x4* pv = pk + BK * D / 4;
#pragma unroll
    for (int md = 0; md < C::MD; ++md)
#pragma unroll
      for (int nt = 0; nt < C::NTK; ++nt) {
        const int x = ((md * C::NTK + nt) * NW + wave) * 64 + lane;
        pk[x] = scale * dka[md][nt];
        pv[x] = dva[md][nt];
      }
    return;
  }
  const float out_scale = WALK ? 1.f : scale;  // (the sums of a walk hold the scale)
  // write dK and dV of the block: through LDS as [key][d], then 16-byte rows
  __bf16* tk = reinterpret_cast<__bf16*>(smem);                        // [BK][D + 8]
  __bf16* tv = reinterpret_cast<__bf16*>(smem) + BK * (D + 8);         // [BK][D + 8]
#pragma unroll
  for (int md = 0; md < C::MD; ++md)
#pragma unroll
    for (int nt = 0; nt < C::NTK; ++nt)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int key = wave * C::NKW + nt * 16 + lr, d = md * 16 + 4 * lg + rr;
        tk[key * (D + 8) + d] = (__bf16)(out_scale * dka[md][nt][rr]);
        tv[key * (D + 8) + d] = (__bf16)dva[md][nt][rr];
      }
  __syncthreads();
  __bf16* dkb = dk + kv_row0 * D;
  __bf16* dvb = dv + kv_row0 * D;
  for (int x = tid; x < BK * (D / 8); x += blockDim.x) {
    const int key = x / (D / 8), ch = x % (D / 8);
    const int64_t kp = k_first + key;
    if (kp < n_k) {
      *reinterpret_cast<uint4*>(dkb + kp * D + ch * 8) = *reinterpret_cast<const uint4*>(tk + key * (D + 8) + ch * 8);
      *reinterpret_cast<uint4*>(dvb + kp * D + ch * 8) = *reinterpret_cast<const uint4*>(tv + key * (D + 8) + ch * 8);
    }
  }
}

// WALK: BwdSplit::walk, columns with sink keys excepted where they have partials.
template <int D, bool WALK>
__global__ void __launch_bounds__(256, D == 64 && WALK ? 2 : 1) bwd_main(cowa_params p, SchedView sv, SplitArgs sa,
                                                const __bf16* __restrict__ q,
                                                const __bf16* __restrict__ k, const __bf16* __restrict__ v,
                                                const __bf16* __restrict__ d_o, const float* __restrict__ nl,
                                                const float* __restrict__ nd, __bf16* __restrict__ dk,
                                                __bf16* __restrict__ dv) {
  using C = BwdCfg<D>;
  constexpr int BK = C::BK;
  extern __shared__ __align__(1024) unsigned char smem[];

  int part = 0, row, unit;
  const bool extra = (int)blockIdx.x < sa.n_extra;
  if (extra) {
    const int e = blockIdx.x;
    part = 1 + e % (sa.P - 1);
    const int rest = e / (sa.P - 1);
    const int tile = rest % sa.S, us = rest / sa.S;  // us = sequence * h_k + KV head
    if (us >= p.batch * p.h_k) return;               // padding
    if (!sv.ragged) {
      row = tile;
      unit = us;
    } else {
      const SeqDesc sd = sv.seq[us / p.h_k];
      if (tile * BK >= sd.n_k) return;  // a sequence with fewer columns
      row = sd.kt_off + tile * (BK / p.tile_k);
      unit = us % p.h_k;
    }
  } else if (sv.order != nullptr) {
    const int total = sa.n_items * sa.PO, id = blockIdx.x - sa.n_extra, copies = sv.ragged ? 1 : p.batch;
    const int e = total > 512 ? xcd_remap(id, total) : id;
    part = e % sa.PO;
    const int item = e / sa.PO;
    const int c = (int)sv.order[item / copies];
    row = c % sa.rows;
    unit = c / sa.rows + (item % copies) * p.h_k;
  } else {
    const int e = blockIdx.x - sa.n_extra;
    part = e / sa.n_items;
    const WorkItem wi = cluster_item(e % sa.n_items, sa.rows, grid_units(p, sv),
                                     cluster_rows(sa.rows, grid_units(p, sv), 32));
    row = wi.row;
    unit = wi.unit;
  }
  int hk, k_first_;
  SeqCtx sc;
  if (row >= sa.rows || !column_ctx(p, sv, row, unit, hk, sc, k_first_)) return;
  const bool sink = sa.P > 1 && k_first_ / BK < sa.S;
  if (!extra && part > 0 && sink) return;  // a sink column's parts are the extra workgroups
  if (WALK && !sink)
    walk_column<D, true>(p, sv, sa, q, k, v, d_o, nl, nd, dk, dv, smem, part, row, unit, hk, sc, k_first_);
  else
    walk_column<D, false>(p, sv, sa, q, k, v, d_o, nl, nd, dk, dv, smem, part, row, unit, hk, sc, k_first_);
}

// Sum of the partials of each split column (in part order) -> bf16 dK, dV; one
// workgroup per (column, 16-row d tile), each thread the register-order elements
// a lane of bwd_main held for that d tile.  Sink columns first, then, where
// others have parts, every other one (of which those of one part end at once).
template <int D>
__global__ void __launch_bounds__(256) bwd_split_sum(cowa_params p, SchedView sv, SplitArgs sa, int n_sink,
                                                     __bf16* __restrict__ dk, __bf16* __restrict__ dv) {
  using C = BwdCfg<D>;
  constexpr int NW = C::NW, BK = C::BK;
  int row, unit, j;
  int64_t first;  // first partial of the column
  if ((int)blockIdx.x < n_sink) {
    const int c = blockIdx.x, us = c / sa.S;  // (sequence * h_k + KV head) * S + column
    j = c % sa.S;
    first = (int64_t)c * sa.P;
    row = j;
    unit = us;
    if (sv.ragged) {
      const SeqDesc sd = sv.seq[us / p.h_k];
      if (j * BK >= sd.n_k) return;
      row = sd.kt_off + j * (BK / p.tile_k);
      unit = us % p.h_k;
    }
  } else {
    const int c = blockIdx.x - n_sink;
    row = c % sa.rows;
    unit = c / sa.rows;
    first = sa.other + (int64_t)c * sa.PO;
  }
  int hk, k_first;
  SeqCtx sc;
  if (!column_ctx(p, sv, row, unit, hk, sc, k_first)) return;
  j = k_first / BK;
  const int n_k = sc.n_k;
  if ((int)blockIdx.x >= n_sink && sa.P > 1 && j < sa.S) return;
  const int k_last = k_first + BK < n_k ? k_first + BK - 1 : n_k - 1, G = p.h_q / p.h_k;
  const int n_parts = column_parts(column_rule(sc.g, G, sa.heads, D), k_first < sc.g.w_sink,
                                   G * runs3_count(query_block_runs3<C::BQ>(sc.g, k_first, k_last)));
  if (n_parts == 1) return;
  const int64_t row0 = sc.k0 + (int64_t)hk * sc.kh;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const f32x4* src = reinterpret_cast<const f32x4*>(sa.part + first * 2 * BK * D);
  const int md = blockIdx.y;
#pragma unroll
  for (int nt = 0; nt < C::NTK; ++nt) {
    const int x = ((md * C::NTK + nt) * NW + wave) * 64 + lane;
    f32x4 a = src[x], g = src[BK * D / 4 + x];
    for (int pt = 1; pt < n_parts; ++pt) {
      a += src[(int64_t)pt * (2 * BK * D / 4) + x];
      g += src[(int64_t)pt * (2 * BK * D / 4) + BK * D / 4 + x];
    }
    const int64_t kp = (int64_t)k_first + wave * C::NKW + nt * 16 + lr;
    if (kp >= n_k) continue;
    bf16x4 ka, va;
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      ka[rr] = (__bf16)a[rr];
      va[rr] = (__bf16)g[rr];
    }
    const int64_t off = (row0 + kp) * D + md * 16 + 4 * lg;
    *reinterpret_cast<bf16x4*>(dk + off) = ka;
    *reinterpret_cast<bf16x4*>(dv + off) = va;
  }
}

template <int D>
hipError_t launch_main(const cowa_params& p, SchedView sv, const void* q, const void* k, const void* v,
                       const void* d_o, const BwdWork& w, void* dk, void* dv, hipStream_t stream) {
  using C = BwdCfg<D>;
  static_assert(C::OUT_BYTES <= C::LDS_MAX && C::MAIN_BYTES < C::LDS_MAX, "LDS budget");
  const BwdSplit& sp = w.split;
  auto kern = sp.walk ? bwd_main<D, true> : bwd_main<D, false>;
  {
    const hipError_t err = allow_lds(reinterpret_cast<const void*>(kern), C::LDS_MAX);
    if (err != hipSuccess) return err;
  }
  const int copies = sv.ragged ? 1 : p.batch;
  if (!sp.walk && column_count(p) * copies > kMaxOrdered) sv.order = nullptr;  // (many rounds: the L2 matters more)
  SplitArgs sa;
  sa.part = w.part;
  sa.S = sp.S;
  sa.P = sp.P;
  sa.PO = sp.PO;
  sa.heads = p.h_k_total;
  sa.n_extra = sa.P > 1 ? (int32_t)(((int64_t)p.batch * p.h_k * sa.S * (sa.P - 1) + 7) / 8 * 8) : 0;
  sa.rows = column_rows(p, sv.n_kt);
  sa.n_items = sv.order ? (int32_t)column_count(p) * copies : sa.rows * p.h_k * copies;
  sa.other = sa.P > 1 ? sp.n_cols * sa.P : 0;
  // 64-row blocks of the longest sequence
  const int64_t nq = sv.ragged ? (int64_t)sv.max_qt * p.tile_q : p.n_q;
  sa.cap = (int32_t)((nq + C::BQ - 1) / C::BQ);
  if (sa.cap > C::max_qblocks()) return hipErrorInvalidValue;
  const unsigned blocks = (unsigned)sa.n_items * sa.PO + (unsigned)sa.n_extra;
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), C::lds_bytes(sa.cap), stream, p, sv, sa,
                     static_cast<const __bf16*>(q), static_cast<const __bf16*>(k), static_cast<const __bf16*>(v),
                     static_cast<const __bf16*>(d_o), w.nl, w.nd, static_cast<__bf16*>(dk),
                     static_cast<__bf16*>(dv));
  const int n_sink = sa.P > 1 ? (int)sp.n_cols : 0;
  const unsigned sums = (unsigned)n_sink + (sa.PO > 1 ? (unsigned)sp.n_all : 0u);
  if (sums > 0)
    hipLaunchKernelGGL((bwd_split_sum<D>), dim3(sums, C::MD), dim3(256), 0, stream, p, sv, sa, n_sink,
                       static_cast<__bf16*>(dk), static_cast<__bf16*>(dv));
  return hipGetLastError();
}

}  // namespace

// Query blocks of the schedule (up to 128 rows each) that a column's list can hold.
int bwd_main_max_qblocks(int d) { return (d == 128 ? BwdCfg<128>::max_qblocks() : BwdCfg<64>::max_qblocks()) / 2; }

bool bwd_bf16_supported(int d, int tq, int tk) {
  return (d == 64 || d == 128) && (tq == 64 || tq == 128) && (tk == 64 || tk == 128);
}

hipError_t launch_bwd_prepare(const cowa_params& p, const void* o, const void* d_o, const float* lse,
                              const BwdWork& w, hipStream_t stream) {
  const int64_t rows = q_rows(p);
  const int64_t chunks = rows * (p.head_dim / 8);
  const unsigned blocks = (unsigned)((chunks + 255) / 256);
  if (p.head_dim == 128)
    hipLaunchKernelGGL(bwd_pre<128>, dim3(blocks), dim3(256), 0, stream, static_cast<const __bf16*>(o),
                       static_cast<const __bf16*>(d_o), lse, w.nd, w.nl, rows);
  else
    hipLaunchKernelGGL(bwd_pre<64>, dim3(blocks), dim3(256), 0, stream, static_cast<const __bf16*>(o),
                       static_cast<const __bf16*>(d_o), lse, w.nd, w.nl, rows);
  return hipGetLastError();
}

hipError_t launch_bwd_main(const cowa_params& p, const SchedView& sv, const void* q, const void* k, const void* v,
                           const void* d_o, void* dk, void* dv, const BwdWork& w, hipStream_t stream) {
  return p.head_dim == 128 ? launch_main<128>(p, sv, q, k, v, d_o, w, dk, dv, stream)
                           : launch_main<64>(p, sv, q, k, v, d_o, w, dk, dv, stream);
}

}  // namespace cowa
