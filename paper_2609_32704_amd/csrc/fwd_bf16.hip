// CoWA forward in bfloat16 on the CDNA4 matrix cores (Alg. 1).
//
// Work decomposition.  One workgroup of four waves per (row tile, group of hpw
// QO heads that share one KV head, sequence b): every QO head of a GQA group sees
// the same keys, so the heads of a workgroup share each K/V block staged in
// LDS.  Each 64-lane wave owns 32 or 64 query rows of one head (see launch_d),
// so a row tile holds R = 4 x 32 (or 64) / hpw rows: the row tiles and the key
// blocks are the kernel's own, whatever tiles the schedule has, and it computes
// the tile's block list itself from the windows (three merged ranges) instead of
// reading the schedule's.  Every group size gets four waves: with one or two
// waves for groups that 256 / tile_q does not divide, multi-head attention left
// half or three quarters of the SIMDs idle.  Workgroups are grouped per XCD so
// that rows sharing K/V blocks run together on one L2 (row_item).
//
// Per KV block j of J_{h_k}(i), full blocks first, then partial ones:
//   * K_j and V_j are copied global -> LDS with direct 16-byte buffer loads,
//     double buffered and issued a block (K) or half a block (V) ahead.  Rows
//     are stored unpadded with their 16-byte chunks XOR swizzled by row, so the
//     row reads of K and the transposing reads of V hit distinct banks.
//   * S^T = K_j Q^T on v_mfma_f32_32x32x16_bf16 (fp32 accumulate); Q^T stays in
//     registers for the whole row.  The accumulator layout of S^T is the
//     B-operand layout of P^T for O^T += V^T P^T, so P never leaves registers;
//     the V^T fragments come from the row-major V_j through the transposing
//     LDS read (ds_read_b64_tr_b16).
//   * only blocks flagged partial apply the element mask of Eq. fwa_support,
//     as a 32-bit mask of legal keys per query and chunk;
//   * softmax in base 2 with a per-row exponent offset that moves only at
//     block ends and rarely (see below), the scale * log2(e) folded into one
//     fused multiply-add per score, and the row sum l accumulated from the
//     rounded bf16 P^T that enters O, on the matrix cores (one 16x16x32
//     product per 16 keys with a 0/1 selector as A), which keeps the vector
//     ALUs, the busier unit, for the exponentials;
//   * the 32-key chunks of a row form a software pipeline: S^T of chunk n and
//     O^T of chunk n - 2 on the matrix cores while the vector ALUs exponentiate
//     chunk n - 1.
// Finally O = O / l and LSE = (m + log2 l) ln 2 (natural log); O leaves through
// LDS as whole rows.
//
// Two launches per call (TRACK false, then true).  The first tracks no running
// maximum: its offset moves on the row sums, and rows it cannot finish (an
// overflow, or a column without a starting offset whose sum stays tiny) leave
// LSE = NaN.  The second runs the tracked algorithm described below, but only
// in workgroups holding such a row; the others end at once.
#include "internal.h"
#include "window_rule.h"
#include "mfma_tiles.h"
#include "work_item.h"

namespace cowa {
namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// S^T = K Q^T accumulates in VGPRs (mfma32_v), O^T in AGPRs (mfma32).  An O^T product lies
// between the last k-step of a chunk and its softmax; chunk steps without those and
// block ends have these wait states before the results are read.  The
// accumulators pass through the statement, so no reader is moved above it
__device__ inline void mfma_settle(f32x16& a, f32x16& b) {
  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" : "+v"(a), "+v"(b));
}
__device__ inline void mfma_settle(f32x16 (&r)[2]) { mfma_settle(r[0], r[1]); }
__device__ inline void mfma_settle(f32x16 (&r)[1]) { asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" : "+v"(r[0])); }

// max(a, b, c) in one instruction (fmaxf would first quiet each operand that
// the compiler cannot prove canonical: the products above are opaque to it)
__device__ inline float max3(float a, float b, float c) {
  float d;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}

// waves per SIMD that the registers are cut for
constexpr int fwd_occupancy(int nqt) { return nqt == 1 ? 2 : 1; }

// NQT: 32-query tiles per wave (columns of S^T); BK: keys per block
template <int D, int NQT_, int BK>
struct FwdCfg {
  static constexpr int NW = 4;            // waves per workgroup
  static constexpr int NQT = NQT_;
  static constexpr int NQW = 32 * NQT;    // query rows per wave
  static constexpr int KS = D / 16;       // k-steps over d of S^T = K Q^T
  static constexpr int MD = D / 32;       // 32-row d tiles of O^T
  static constexpr int NCH = BK / 32;     // 32-key chunks per block (2 or 4)
  static constexpr int NG = KS + 2 * MD;  // product groups per chunk (NQT products each)
  using T = SwzTile<D, BK>;
  static constexpr int MAIN_BYTES = 4 * T::BYTES;  // K and V of two blocks; then the row's entry list
  static constexpr int LDS_MAX = 160 * 1024;
  static constexpr int OUT_PITCH = 2 * D + 16;             // staged output rows (bytes)
  static constexpr int OUT_BYTES = NW * NQW * OUT_PITCH;   // reuses the K/V buffers and list at the end
  static int lds_bytes(int n_kb) {                         // n_kb: list capacity; + a vote word
    return MAIN_BYTES + 4 * n_kb + 16 > OUT_BYTES ? MAIN_BYTES + 4 * n_kb + 16 : OUT_BYTES;
  }
  static constexpr int max_kblocks() { return (LDS_MAX - MAIN_BYTES - 16) / 4; }
  static_assert(KS == 2 * MD, "S and O groups alternate one to one");
  static_assert(NCH == 2 || NCH == 4, "64- or 128-key blocks");
};

// A workgroup's row tile: its rows (rt.R from query q0 on of each of hpw QO heads,
// group `group` of KV head hk) in sequence sc.
struct RowItem {
  SeqCtx sc;
  int hk, group, q0;
};
__device__ inline bool row_work(const cowa_params& p, const SchedView& sv, const RowTiles& rt, RowItem& it) {
  int row, unit;
  if (!row_item(rt, grid_units(p, sv), p.h_q / p.h_k / rt.hpw, blockIdx.x, row, unit, it.group)) return false;
  it.sc = row_ctx(p, sv, rt, row, unit, it.hk, it.q0);
  return it.q0 < it.sc.n_q;
}

// rt: the launch's rows; R = rows per (workgroup, head)
template <int D, int NQT, int BK, bool TRACK>
__device__ __forceinline__ void fwd_rows(const cowa_params& p, const RowTiles& rt, const RowItem& it, int cap,
                                         unsigned char* smem, const __bf16* __restrict__ q,
                                         const __bf16* __restrict__ k, const __bf16* __restrict__ v,
                                         __bf16* __restrict__ o, float* __restrict__ lse) {
  using C = FwdCfg<D, NQT, BK>;
  using T = typename C::T;
  constexpr int KS = C::KS, MD = C::MD, NCH = C::NCH, NG = C::NG;

  const int hpw = rt.hpw, wph = C::NW / hpw;  // heads per workgroup, waves per head
  const int G = p.h_q / p.h_k;
  const SeqCtx& sc = it.sc;
  const int hk = it.hk, q0 = it.q0;
  const int n_q = sc.n_q, n_k = sc.n_k;
  const int h0 = (hk * (G / hpw) + it.group) * hpw;  // first QO head of this workgroup (all in KV group hk)

  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int l32 = lane & 31, hh = lane >> 5;  // MFMA column and half
  const int hq = h0 + wave / wph;
  const int q_first = q0 + (wave % wph) * C::NQW;
  const Geo32 g = sc.g;
  const __bf16* kbase = k + (sc.k0 + (int64_t)hk * sc.kh) * D;
  const __bf16* vbase = v + (sc.k0 + (int64_t)hk * sc.kh) * D;
  const uint32_t smem_base = lds_addr(smem);
  const int64_t row_base = sc.q0 + (int64_t)hq * sc.qh;
  if constexpr (TRACK) {
    // only the workgroups with a row that the untracked launch left to this
    // one (LSE = NaN) run; the rest end here, uniformly
    int* flag = reinterpret_cast<int*>(smem + C::MAIN_BYTES + 4 * cap);
    if (tid == 0) *flag = 0;
    __syncthreads();
    const int qr = q_first + lane;
    if (__ballot(lane < C::NQW && qr < n_q && __builtin_isnan(lse[row_base + qr])) != 0 && lane == 0) *flag = 1;
    __syncthreads();
    const bool mine = *flag != 0;
    __syncthreads();
    if (!mine) return;
  }

  // The row tile's block list, in LDS: full blocks from the front, partial
  // ones from the back, both by descending key (at most three merged ranges,
  // computed rather than read: the schedule's tiles need not be this kernel's)
  const int q_last = (q0 + rt.R < n_q ? q0 + rt.R : n_q) - 1;
  uint32_t* list = reinterpret_cast<uint32_t*>(smem + C::MAIN_BYTES);
  int n_ent;
  const int n_full = build_row_list<BK>(g, q0, q_last, rt.R, list, cap, wave, lane, n_ent);
  auto entry_at = [&](int t) -> int {
    const int tt = t < n_ent ? t : n_ent - 1;
    const int idx = tt < n_full ? tt : cap - 1 - (tt - n_full);
    return __builtin_amdgcn_readfirstlane(list[idx]);
  };
  // zero the K/V buffers once when the row reaches the last KV block and that
  // is partial: key rows past the end of the sequence are not copied and must
  // hold finite values
  if (n_k % BK != 0 && (q_last + g.off) / BK == n_k / BK)
    for (int x = tid; x < C::MAIN_BYTES / 16; x += 256) reinterpret_cast<u32x4*>(smem)[x] = u32x4{0u, 0u, 0u, 0u};

  // Global -> LDS copies of K and V blocks: each lane copies the same 16-byte
  // column of its row in every 1 KB piece it takes, so its byte offsets within
  // a block are fixed, and the block position goes into the (scalar) buffer
  // resource, whose size bounds the reads to the sequence.
  constexpr int RPL = 1024 / (D * 2);    // rows per 1 KB piece
  constexpr int PPW = T::LOADS / C::NW;  // pieces per wave
  static_assert(T::LOADS % C::NW == 0 && (C::NW * RPL) % 16 == 0, "piece layout");
  uint32_t dma_off[PPW];
  {
    const int row0 = wave * RPL + lane / T::CH;
    const int col = (lane % T::CH) ^ swz<T::CH>(row0);
#pragma unroll
    for (int n = 0; n < PPW; ++n) dma_off[n] = (uint32_t)(((n * C::NW * RPL + row0) * D + col * 8) * 2);
  }
  auto kbuf_off = [](int t) { return (t & 1) * 2 * T::BYTES; };
  auto vbuf_off = [](int t) { return (t & 1) * 2 * T::BYTES + T::BYTES; };
  // piece n of a block copy, issued on its own
  auto stage_piece = [&](const __bf16* base, int kf, int buf_off, int n) {
    const i32x4 rs = buffer_rsrc(base + (int64_t)kf * D, (uint32_t)(n_k - kf) * D * 2);
    dma16_buf(dma_off[n], rs, smem_base + buf_off + wave * 1024 + n * C::NW * 1024);
  };
  auto stage = [&](const __bf16* base, int t, int buf_off) {
    const int kf = entry_at(t) * BK;
#pragma unroll
    for (int n = 0; n < PPW; ++n) stage_piece(base, kf, buf_off, n);
  };
  __syncthreads();  // the list and the zeroed buffers are in LDS
  // The first block's copies go out before the Q^T loads, so that the row
  // start waits for memory once.  (With 128-key blocks V of block 0 is needed
  // from its third chunk; with 64-key blocks it is copied by the first step.)
  auto stage_first = [&]() {
    if (n_ent > 0) {
      stage(kbase, 0, kbuf_off(0));
      if (NCH == 4) stage(vbase, 0, vbuf_off(0));
    }
  };
  stage_first();

  // Q^T fragments (B operands): query column 32 nq + l32, d = 16 ks + 8 hh + 0..7
  bf16x8 qf[NQT][KS];
#pragma unroll
  for (int nq = 0; nq < NQT; ++nq) {
    const int qp = q_first + nq * 32 + l32;
    const bool ok = qp < n_q;
    const __bf16* qrow = q + (row_base + (ok ? qp : 0)) * D;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 val = *reinterpret_cast<const bf16x8*>(qrow + ks * 16 + 8 * hh);
      qf[nq][ks] = ok ? val : bf16x8{};
    }
  }
  // Move the Q^T fragments into AGPRs here, long before the first product: the
  // assembly products read them from AGPRs, and the compiler could otherwise
  // copy them there just before that read, without the wait states a product
  // needs after a vector write of its operands.  (These statements emit
  // nothing themselves.)
#pragma unroll
  for (int nq = 0; nq < NQT; ++nq)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+a"(qf[nq][ks]));
  // LDS fragment offsets for chunk 0 of a tile (the swizzle depends on row % 16,
  // so chunks 32 rows further and k-steps 16 rows further add plain row bytes)
  //  K (A operand of S^T): row l32, columns 16 ks + 8 hh + 0..7;
  //  V^T (A operand of O^T): transposing reads of rows 4 hh + (lane % 16) / 4
  //  (+ 8 for slots 4..7), columns 32 md + 16 ((lane / 16) % 2) + 4 (lane % 4).
  int offk[KS], offv[MD][2];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) offk[ks] = T::off(l32, 2 * ks + hh);
#pragma unroll
  for (int md = 0; md < MD; ++md)
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
      offv[md][hf] = T::off_col(4 * hh + ((lane & 15) >> 2) + 8 * hf, 32 * md + 16 * ((lane >> 4) & 1) + 4 * (lane & 3));
  auto ld_v = [&](const unsigned char* tile, int md, int row_bytes) -> bf16x8 {
    const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(tile + offv[md][0] + row_bytes));
    const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(tile + offv[md][1] + row_bytes));
    const bf16x4 a = __builtin_bit_cast(bf16x4, lo), c2 = __builtin_bit_cast(bf16x4, hi);
    return bf16x8{a[0], a[1], a[2], a[3], c2[0], c2[1], c2[2], c2[3]};
  };

  // O^T accumulators: element (lane, e) is d = 32 md + 8 (e / 4) + 4 hh + e % 4, query 32 nq + l32
  f32x16 oacc[MD][NQT];
  // S^T of two chunks: element (lane, e) is key 8 (e / 4) + 4 hh + e % 4 of the
  // chunk, query 32 nq + l32.  Slots e = 8 kk .. 8 kk + 7 are exactly the keys
  // that lane holds in k-step kk of O^T += V^T P^T (16 keys each), so P^T needs
  // no data movement.
  f32x16 sacc[2][NQT];
  u32x4 pbw[2][2][NQT];  // P^T of two chunks: bf16 pairs, [chunk % 2][k-step][query tile]

  // The exponent offset m (base 2, per query column) starts kHead above the
  // maximum over the first 32 keys of the row's first block, so P = exp2(s c - m)
  // is at most 2^-kHead there and a later score may pass that maximum by
  // kHead + ~110 before P, l or O could overflow (keys more than ~60 below the
  // maximum underflow, 2^-60 of the largest term).  O and l share the offset,
  // so O / l and LSE = (m + log2 l) ln 2 are unaffected, and O is rescaled
  // only when, at the end of a block, a column's maximum has passed the one
  // that m was set from by more than kLimit: then m moves to kHead above it
  // and O, l and the P^T not yet in O are multiplied by 2^(m_old - m) once
  // (rare after the first blocks of a row, never for scores within kLimit).
  // If P, l or O overflowed anyway, the workgroup runs the row again with m
  // set from the row maximum found by the first pass, as it does when m was
  // unset (no legal key among the first 32) but the row has legal keys.
  constexpr float kHead = 64.f, kLimit = 32.f;
  float m_fix[NQT], m_hi[NQT], mu[NQT];  // m_hi: this lane's maximum raw score per column
#pragma unroll
  for (int nq = 0; nq < NQT; ++nq) m_fix[nq] = -INFINITY;
  const float c = p.softmax_scale * kLog2e;
  // Row sums l = sum of the rounded P^T over the keys, per query column, on the
  // matrix cores: the P^T fragment of a 16-key k-step, read as the B operand of
  // a 16x16x32 product, holds in lane L column L % 16 of k-group L / 16, which
  // is query 32 nq + (L % 32) with the keys of half L / 32 (k-groups 0 and 2:
  // queries 0-15, 1 and 3: queries 16-31).  The selector A has ones where
  // (row & 4) == 0 equals (k-group even), so rows 0-3 and 8-11 sum queries 0-15
  // and rows 4-7 and 12-15 queries 16-31; the result rows 4 (L / 16) .. + 3 of
  // lane L then all hold the sum of lane L's own query column L % 32.
  f32x4 lacc[NQT];
  const bf16x8 lsel = ((lane & 4) == 0) == (((lane >> 4) & 1) == 0)
                          ? bf16x8{(__bf16)1.f, (__bf16)1.f, (__bf16)1.f, (__bf16)1.f,
                                   (__bf16)1.f, (__bf16)1.f, (__bf16)1.f, (__bf16)1.f}
                          : bf16x8{};

  float pv[16 * NQT];  // exponentials in flight between the two halves of an element step
  uint32_t lmask[NQT];  // legal keys of the chunk being masked, per query tile
  // element step e of a chunk's softmax (query tile e / 16, slot e % 16), first half
  auto soft_a = [&](auto ec, auto rpc, bool masked, int key0) __attribute__((always_inline)) {
    constexpr int e = decltype(ec)::value, rp = decltype(rpc)::value;
    constexpr int nq = e / 16, s = e % 16;
    if (masked) {  // key0: this lane's first key of the chunk
      // the window rule as a bit mask over the lane's keys key0 .. key0 + 31,
      // once per chunk and query tile; slot s holds key key0 + cs, which an
      // illegal pair turns into -inf (bit select, no compare)
      constexpr int cs = 8 * (s >> 2) + (s & 3);
      if constexpr (s == 0) lmask[nq] = legal_keys32(g, q_first + nq * 32 + l32, key0);
      const uint32_t m = (uint32_t)((int32_t)(lmask[nq] << (31 - cs)) >> 31);
      sacc[rp][nq][s] = __uint_as_float((__float_as_uint(sacc[rp][nq][s]) & m) | (0xff800000u & ~m));
    }
    pv[e] = __builtin_amdgcn_exp2f(fmaf(sacc[rp][nq][s], c, -mu[nq]));
  };
  // second half (odd e): running maximum (TRACK only), bf16 pair
  auto soft_b = [&](auto ec, auto rpc, auto psc) __attribute__((always_inline)) {
    constexpr int e = decltype(ec)::value, rp = decltype(rpc)::value, ps = decltype(psc)::value;
    constexpr int nq = e / 16, s = e % 16;
    if constexpr (s & 1) {
      if constexpr (TRACK) m_hi[nq] = max3(m_hi[nq], sacc[rp][nq][s - 1], sacc[rp][nq][s]);
      const bf16x2 pk = {(__bf16)pv[e - 1], (__bf16)pv[e]};
      pbw[ps][s / 8][nq][(s & 7) >> 1] = __builtin_bit_cast(uint32_t, pk);
    }
  };
  // the element steps that belong to slot `slot` of NS
  auto soft_slot = [&](auto slotc, auto nsc, auto rpc, auto psc, bool masked, int key0) __attribute__((always_inline)) {
    constexpr int slot = decltype(slotc)::value, NS = decltype(nsc)::value;
    static_for<16 * NQT>([&](auto ec) {
      constexpr int e = decltype(ec)::value;
      constexpr int sa = e * NS / (16 * NQT);
      constexpr int sb = sa + 1 < NS ? sa + 1 : sa;
      if constexpr (sa == slot) soft_a(ec, rpc, masked, key0);
      if constexpr (sb == slot) soft_b(ec, rpc, psc);
    });
  };

  // End of a block: move the offset of columns whose maximum has passed it by
  // more than kLimit.  P^T of the block's second-to-last chunk is computed but
  // not yet in O (it enters in the next block's first chunk step), so it is
  // rescaled with O and l; the last chunk is exponentiated after this point.
  // The test is per lane (a column's two lanes hold disjoint keys, and the one
  // holding the maximum sees it); the new offset is kHead above the column
  // maximum.  `hot` records a P above 2^kHot, the only way P, l or O can
  // approach the float range, so the overflow check at the end of a pass runs
  // only then.
  constexpr float kHot = 64.f;
  bool hot = false;
  auto rebase = [&]() __attribute__((always_inline)) {
    bool need = false;
#pragma unroll
    for (int nq = 0; nq < NQT; ++nq) {
      const float e = m_hi[nq] * c - mu[nq];
      need |= e > kLimit - kHead;
      hot |= e > kHot;
    }
    if (__builtin_expect(__ballot(need) == 0, 1)) return;  // (rare: keep it a branch)
    constexpr int PS = (NCH - 2) & 1;  // pair buffer of the pending chunk
#pragma unroll
    for (int nq = 0; nq < NQT; ++nq) {
      const float mh = fmaxf(m_hi[nq], __shfl_xor(m_hi[nq], 32)) * c + kHead;
      const bool mv = mh > mu[nq] + kLimit;
      // the factor 2^(m_old - m) is applied as its square root twice: a jump of
      // the maximum by more than 126 within one block would make it underflow,
      // although the products (the new maximum's own terms among them) are
      // ordinary numbers; the square root stays normal up to a jump of 252,
      // beyond which P has overflowed and the row runs again anyway
      const float f = mv ? __builtin_amdgcn_exp2f(0.5f * (mu[nq] - mh)) : 1.f;
      mu[nq] = mv ? mh : mu[nq];
      lacc[nq] = lacc[nq] * f * f;
#pragma unroll
      for (int md = 0; md < MD; ++md) {  // one tile at a time, back into its AGPRs
#pragma unroll
        for (int x = 0; x < 16; ++x) oacc[md][nq][x] = oacc[md][nq][x] * f * f;
        asm volatile("" : "+a"(oacc[md][nq]));
      }
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          // (a vector element is copied out first: bit-casting the element
          // expression itself reads element 0)
          const uint32_t u = pbw[PS][kk][nq][w];
          const bf16x2 pk = __builtin_bit_cast(bf16x2, u);
          const bf16x2 sc2 = {(__bf16)((float)pk[0] * f * f), (__bf16)((float)pk[1] * f * f)};
          pbw[PS][kk][nq][w] = __builtin_bit_cast(uint32_t, sc2);
        }
    }
  };

  // The same move without a tracked maximum (TRACK false): the row sum l of a
  // column bounds each of its P from above, so when it passes 2^(kLimit -
  // kHead) at a block end (never before some score has passed the first keys'
  // maximum by 15 or more: at most 2^31 keys of at most 2^-kHead each) the
  // offset moves by log2 l + kHead, which leaves every P so far at most
  // 2^-kHead (l itself becomes 2^-kHead) and overshoots the move the maximum
  // would give by at most log2 of the row length.  Both lanes of a column hold
  // the same sum, so they move alike.  The sum lags by the chunks not yet in
  // it (the pending P^T and the last chunk); a P that overflows in the
  // meantime makes l infinite, and the row is left to the tracked launch.
  auto rebase_sum = [&]() __attribute__((always_inline)) {
    bool need = false;
#pragma unroll
    for (int nq = 0; nq < NQT; ++nq) {
      const float l = lacc[nq][0];
      need |= l > 0x1p-32f;
      hot |= !(l <= 0x1p64f);
    }
    if (__builtin_expect(__ballot(need) == 0, 1)) return;  // (rare: keep it a branch)
    constexpr int PS = (NCH - 2) & 1;  // pair buffer of the pending chunk
#pragma unroll
    for (int nq = 0; nq < NQT; ++nq) {
      const float l = lacc[nq][0];
      const bool mv = l > 0x1p-32f && l < INFINITY;  // (an overflowed sum: the row goes to the tracked launch)
      const float dm = mv ? __log2f(l) + kHead : 0.f;
      const float f = mv ? __builtin_amdgcn_exp2f(-0.5f * dm) : 1.f;  // applied twice, as above
      mu[nq] += dm;
      lacc[nq] = lacc[nq] * f * f;
#pragma unroll
      for (int md = 0; md < MD; ++md) {
#pragma unroll
        for (int x = 0; x < 16; ++x) oacc[md][nq][x] = oacc[md][nq][x] * f * f;
        asm volatile("" : "+a"(oacc[md][nq]));
      }
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const uint32_t u = pbw[PS][kk][nq][w];
          const bf16x2 pk = __builtin_bit_cast(bf16x2, u);
          const bf16x2 sc2 = {(__bf16)((float)pk[0] * f * f), (__bf16)((float)pk[1] * f * f)};
          pbw[PS][kk][nq][w] = __builtin_bit_cast(uint32_t, sc2);
        }
    }
  };

  // Software pipeline over the row's 32-key chunks: chunk n has its S^T
  // computed in chunk step n, is exponentiated in step n + 1 and enters
  // O^T += V^T P^T in step n + 2.  Within a chunk step the matrix cores work on
  // S^T (chunk n) and O^T (chunk n - 2) while the vector ALUs turn S^T of chunk
  // n - 1 into P^T: the streams are independent, so the exponentials hide under
  // the products.  Fragments are read PF groups ahead.
  //
  // LDS: K of block t in K buffer t % 2, V of block t in V buffer t % 2.  The
  // O^T products of block t's steps read V of block t - 1 for the chunks two
  // back; with 128-key blocks, V of block t is needed from its third step on,
  // so it is copied in the middle of block t - 1, once V of block t - 2 is no
  // longer read.
  constexpr int PF = 2, RING = PF + 2;
  int k_prev = 0;  // first key of the previous block
  // One block.  FIRST: the row's first block (nothing before its first chunk).
  // MPREV / MCUR: the chunks exponentiated here from the previous / this block
  // need the element mask.
  auto step = [&](int t, auto firstc, auto mprevc, auto mcurc) __attribute__((always_inline)) {
    constexpr bool FIRST = decltype(firstc)::value, MPREV = decltype(mprevc)::value;
    constexpr bool MCUR = decltype(mcurc)::value;
    const int k_first = entry_at(t) * BK;
    // K of block t + 1 goes into the K buffer of block t - 1, which is free
    // (the last block repeats itself).  The copies go out one 1 KB piece per
    // product group: K from the block start; V after K with 64-key blocks (V of
    // block t, into the free buffer of block t - 2), from the mid-block barrier
    // with 128-key blocks.  A burst of them holds the wave at the vector memory
    // queue: issued at once, 64-key blocks took 102 us at 4096 tokens (32/8
    // heads, d = 128), 149 at 1000 queries of 32000 keys and 139 at 100; spread
    // over the groups 100, 146 and 135.
    const int kf_next = entry_at(t + 1) * BK;
    const unsigned char* Kt = smem + kbuf_off(t);
    const unsigned char* Vt = smem + vbuf_off(t);
    const unsigned char* Vp = smem + vbuf_off(t + 1);  // V of block t - 1
    constexpr int NGS = NCH * NG;
    bf16x8 fa[RING];
    // group GG of the block: chunk step j, S^T k-step or O^T (k-step kk, d tile md)
    auto load = [&](auto gc, bf16x8& dst) __attribute__((always_inline)) {
      constexpr int GG = decltype(gc)::value, j = GG / NG, gi = GG % NG;
      constexpr bool S = gi % 2 == 0;
      constexpr int x = gi / 2;
      constexpr int jo = (j + NCH - 2) % NCH;  // chunk of the O^T products within its block
      constexpr bool OLD = j < 2;              // ... of the previous block
      if constexpr (S) {
        dst = ld_row8(Kt + offk[x] + j * 32 * D * 2);
      } else if constexpr (!(FIRST && OLD)) {
        constexpr int kk = x / MD, md = x % MD;
        dst = ld_v(OLD ? Vp : Vt, md, (jo * 32 + kk * 16) * D * 2);
      }
    };
    static_for<PF>([&](auto ic) { load(ic, fa[decltype(ic)::value]); });
    __builtin_amdgcn_sched_barrier(0);
    static_for<NGS>([&](auto gc) {
      constexpr int GG = decltype(gc)::value, j = GG / NG, gi = GG % NG;
      constexpr bool S = gi % 2 == 0;
      constexpr int x = gi / 2;
      constexpr bool OLD = j < 2;
      if constexpr (NCH == 4 && GG == 2 * NG - PF) {
        // middle of a 128-key block, before the first read of V of block t
        // (fragments run PF groups ahead) and after the last read of V of
        // block t - 1 was issued: V of block t is in (its copies were issued
        // before this block's K copies), and once every wave's reads of V of
        // block t - 1 are done, the copy of block t + 1 may overwrite it
        __builtin_amdgcn_s_waitcnt(vmcnt_only(PPW));
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (GG < PPW) stage_piece(kbase, kf_next, kbuf_off(t + 1), GG);
      if constexpr (NCH == 2 && GG >= PPW && GG < 2 * PPW) stage_piece(vbase, k_first, vbuf_off(t), GG - PPW);
      if constexpr (NCH == 4 && GG >= 2 * NG - PF && GG < 2 * NG - PF + PPW)
        stage_piece(vbase, kf_next, vbuf_off(t + 1), GG - (2 * NG - PF));
      if constexpr (GG + PF < NGS) load(std::integral_constant<int, GG + PF>{}, fa[(GG + PF) % RING]);
      const bf16x8& a = fa[GG % RING];
      static_for<NQT>([&](auto mc) {
        constexpr int m = decltype(mc)::value;
        if constexpr (S) {
          if constexpr (x == 0)
            sacc[j & 1][m] = mfma32_v0(a, qf[m][0]);
          else
            sacc[j & 1][m] = mfma32_v(a, qf[m][x], sacc[j & 1][m]);
        } else if constexpr (!(FIRST && OLD)) {
          constexpr int kk = x / MD, md = x % MD;
          oacc[md][m] = mfma32(a, __builtin_bit_cast(bf16x8, pbw[j & 1][kk][m]), oacc[md][m]);
          if constexpr (md == 0) lacc[m] = mfma16(lsel, __builtin_bit_cast(bf16x8, pbw[j & 1][kk][m]), lacc[m]);
        }
        // the softmax of the chunk before chunk j (chunk j - 1 of this block,
        // or the last chunk of the previous block), spread over the products
        constexpr int slot = gi * NQT + m;
        if constexpr (!(FIRST && j == 0)) {
          using SL = std::integral_constant<int, slot>;
          using NSC = std::integral_constant<int, NQT * NG>;
          using RP = std::integral_constant<int, (j + 1) & 1>;
          if constexpr (j == 0)
            soft_slot(SL{}, NSC{}, RP{}, RP{}, MPREV, k_prev + (NCH - 1) * 32 + 4 * hh);
          else
            soft_slot(SL{}, NSC{}, RP{}, RP{}, MCUR, k_first + (j - 1) * 32 + 4 * hh);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      // a chunk step without O^T products (start of the row): its S^T results
      // are read early in the next step, so settle them here
      if constexpr (FIRST && OLD && gi == NG - 1) {
        mfma_settle(sacc[j & 1]);
        __builtin_amdgcn_sched_barrier(0);
      }
    });
    // the last S^T products may still be in flight: wait states before
    // anything reads them
    mfma_settle(sacc[1]);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (TRACK)
      rebase();
    else
      rebase_sum();
    // register placement: O^T accumulators and Q^T fragments in AGPRs (read
    // directly by the matrix cores), S^T and P^T in VGPRs; these emit nothing
#pragma unroll
    for (int md = 0; md < MD; ++md)
#pragma unroll
      for (int nq = 0; nq < NQT; ++nq) asm volatile("" : "+a"(oacc[md][nq]));
#pragma unroll
    for (int nq = 0; nq < NQT; ++nq)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+a"(qf[nq][ks]));
    k_prev = k_first;
    // the next block's K has landed (with 128-key blocks the next V may still
    // be in flight)
    if constexpr (NCH == 4)
      __builtin_amdgcn_s_waitcnt(vmcnt_only(PPW));
    else
      __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();  // ... for every wave, and the freed buffers are no longer read
  };
  // after the last block: the softmax of its last chunk, then the O^T products
  // of its last two chunks
  auto drain = [&](int t) __attribute__((always_inline)) {
    using R1 = std::integral_constant<int, 1>;
    static_for<16 * NQT>([&](auto ec) { soft_a(ec, R1{}, true, k_prev + (NCH - 1) * 32 + 4 * hh); });
    static_for<16 * NQT>([&](auto ec) { soft_b(ec, R1{}, R1{}); });
    if constexpr (NCH == 4) __builtin_amdgcn_s_waitcnt(0);  // (the repeated V copy of the mid-block)
    const unsigned char* Vt = smem + vbuf_off(t);
    static_for<2 * 2 * MD>([&](auto gc) {
      constexpr int GG = decltype(gc)::value, jj = GG / (2 * MD), kk = (GG / MD) % 2, md = GG % MD;
      constexpr int jo = NCH - 2 + jj;  // chunk within the block
      const bf16x8 a = ld_v(Vt, md, (jo * 32 + kk * 16) * D * 2);
#pragma unroll
      for (int nq = 0; nq < NQT; ++nq)
        oacc[md][nq] = mfma32(a, __builtin_bit_cast(bf16x8, pbw[jo & 1][kk][nq]), oacc[md][nq]);
      if constexpr (md == 0)
#pragma unroll
        for (int nq = 0; nq < NQT; ++nq)
          lacc[nq] = mfma16(lsel, __builtin_bit_cast(bf16x8, pbw[jo & 1][kk][nq]), lacc[nq]);
    });
  };
  using TT = std::true_type;
  using FF = std::false_type;
  auto sweep = [&]() __attribute__((always_inline)) {
    int t = 0;
    if (n_full > 0) {
      step(0, TT{}, FF{}, FF{});
      for (t = 1; t < n_full; ++t) step(t, FF{}, FF{}, FF{});
    }
    if (t < n_ent) {
      if (t == 0) {
        step(0, TT{}, TT{}, TT{});
        t = 1;
      }
      for (; t < n_ent; ++t) step(t, FF{}, TT{}, TT{});
    }
    if (n_ent > 0) drain(n_ent - 1);
  };

  int* vote = reinterpret_cast<int*>(smem + C::MAIN_BYTES + 4 * cap);
  // TRACK false: one pass without a tracked maximum (its offset moves on the
  // row sums); rows it cannot finish get LSE = NaN and are run again by the
  // TRACK launch, with up to two passes as described above
  bool flagged = false;
  for (int pass = 0; pass < (TRACK ? 2 : 1); ++pass) {
#pragma unroll
    for (int nq = 0; nq < NQT; ++nq) {
      m_hi[nq] = -INFINITY;
      lacc[nq] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int md = 0; md < MD; ++md) oacc[md][nq] = f32x16{};
    }
    if (pass > 0) stage_first();
    // K of the first block has landed; with 128-key blocks its V
    // may still be in flight (the first block's mid-block wait covers it)
    if constexpr (NCH == 4)
      __builtin_amdgcn_s_waitcnt(vmcnt_only(PPW));
    else
      __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (pass == 0 && n_ent > 0) {
      // offsets from the first 32 keys of the row's first block (in processing
      // order: a full block when the row has one)
      const int kb = entry_at(0) * BK + 4 * hh;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x8 a = ld_row8(smem + offk[ks]);
#pragma unroll
        for (int nq = 0; nq < NQT; ++nq)
          sacc[0][nq] = ks == 0 ? mfma32_v0(a, qf[nq][0]) : mfma32_v(a, qf[nq][ks], sacc[0][nq]);
        mfma_settle(sacc[0]);  // the next k-step reads these accumulators
      }
#pragma unroll
      for (int nq = 0; nq < NQT; ++nq) {
        float cm = -INFINITY;
        const uint32_t lm = legal_keys32(g, q_first + nq * 32 + l32, kb);
#pragma unroll
        for (int x = 0; x < 16; ++x) {
          const bool ok = (lm >> (8 * (x >> 2) + (x & 3))) & 1u;
          cm = fmaxf(cm, ok ? sacc[0][nq][x] : -INFINITY);
        }
        cm = fmaxf(cm, __shfl_xor(cm, 32));
        m_fix[nq] = cm * c;  // -inf for a column without a legal key there
      }
      // Tiles without a full block start at their last keys, which their first
      // rows do not reach when a tile is taller than a chunk.  Such rows take
      // the 32 keys from their own 32-row tile's first distance-0 key on, which hold
      // each row's distance-0 key (K straight from memory: once per row, early
      // tiles only).
      bool unset = false;
#pragma unroll
      for (int nq = 0; nq < NQT; ++nq) unset |= m_fix[nq] == -INFINITY && q_first + nq * 32 + l32 < n_q;
      if (__builtin_expect(__ballot(unset) != 0, 0)) {
#pragma unroll
        for (int nq = 0; nq < NQT; ++nq) {
          const int kd = q_first + nq * 32 + g.off, kr = kd + l32 < n_k ? kd + l32 : n_k - 1;
          const __bf16* krow = kbase + (int64_t)kr * D + 8 * hh;
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) {
            const bf16x8 a = *reinterpret_cast<const bf16x8*>(krow + ks * 16);
            sacc[0][nq] = ks == 0 ? mfma32_v0(a, qf[nq][0]) : mfma32_v(a, qf[nq][ks], sacc[0][nq]);
            mfma_settle(sacc[0]);
            __builtin_amdgcn_sched_barrier(0);  // (one fragment at a time: no registers to spare here)
          }
          float cm = -INFINITY;
          const uint32_t lm = legal_keys32(g, q_first + nq * 32 + l32, kd + 4 * hh);
#pragma unroll
          for (int x = 0; x < 16; ++x) {
            const bool ok = (lm >> (8 * (x >> 2) + (x & 3))) & 1u;
            cm = fmaxf(cm, ok ? sacc[0][nq][x] : -INFINITY);
          }
          cm = fmaxf(cm, __shfl_xor(cm, 32));
          m_fix[nq] = m_fix[nq] == -INFINITY ? cm * c : m_fix[nq];
        }
      }
    }
#pragma unroll
    for (int nq = 0; nq < NQT; ++nq) mu[nq] = m_fix[nq] == -INFINITY ? 0.f : m_fix[nq] + kHead;
    sweep();
    bool far = false;
    if constexpr (TRACK) {
      // was a column's offset unset although it met legal keys later, or did
      // P, l or O overflow (possible only after a P above 2^kHot)?
#pragma unroll
      for (int nq = 0; nq < NQT; ++nq) {
        hot |= m_hi[nq] * c - mu[nq] > kHot;  // (the last chunk came after the last block end)
        const float mh = fmaxf(m_hi[nq], __shfl_xor(m_hi[nq], 32)) * c;  // the column maximum, exponent units
        far |= mh != -INFINITY && m_fix[nq] == -INFINITY;
        m_fix[nq] = mh;  // the offset of a second pass: then P <= 2^-kHead everywhere
      }
    } else {
      // a column without an offset at the start (m = 0) keeps its sum only if
      // that sum is comfortably normal (otherwise it met no legal key, or its
      // P underflowed); an overflow shows in the sum.  A move of the offset
      // leaves 2^-kHead, below the line: such a row runs again from its exact
      // maximum.
#pragma unroll
      for (int nq = 0; nq < NQT; ++nq) {
        const float l = lacc[nq][0];
        hot |= !(l <= 0x1p64f);
        far |= m_fix[nq] == -INFINITY && q_first + nq * 32 + l32 < n_q && !(l >= 0x1p-60f);
      }
    }
    if (__ballot(hot) != 0) {
#pragma unroll
      for (int nq = 0; nq < NQT; ++nq) {
        far |= !__builtin_isfinite(lacc[nq][0]);
#pragma unroll
        for (int md = 0; md < MD; ++md) {
#pragma unroll
          for (int x = 0; x < 16; ++x) far |= !__builtin_isfinite(oacc[md][nq][x]);
          asm volatile("" : "+a"(oacc[md][nq]));
        }
      }
    }
    hot = false;
    // workgroup vote through a word past the block lists
    if (tid == 0) *vote = 0;
    __syncthreads();
    if (far) *vote = 1;
    __syncthreads();
    const bool again = *vote != 0;
    __syncthreads();
    if (!TRACK) flagged = again;
    if (!again) break;
  }

  // O = O / l; LSE = (m + log2 l) ln 2 with the offset m of the last pass (base 2).
  // O goes out through LDS (free here: every wave is past the vote's barriers,
  // its reads are done and its copies have landed): each wave stages its
  // rows and stores whole rows, 16 bytes per lane, instead of 16-byte pieces of
  // 32 rows per store in the accumulator layout.
  constexpr int OP = C::OUT_PITCH;
  unsigned char* ot = smem + wave * C::NQW * OP;
#pragma unroll
  for (int nq = 0; nq < NQT; ++nq) {
    const float lt = lacc[nq][0];
    const int qp = q_first + nq * 32 + l32;
    const float inv = lt > 0.f ? 1.f / lt : 0.f;
#pragma unroll
    for (int md = 0; md < MD; ++md)
#pragma unroll
      for (int j4 = 0; j4 < 4; ++j4) {
        bf16x4 ov;
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) ov[rr] = (__bf16)(oacc[md][nq][4 * j4 + rr] * inv);
        *reinterpret_cast<bf16x4*>(ot + (nq * 32 + l32) * OP + (md * 32 + 8 * j4 + 4 * hh) * 2) = ov;
      }
    if (hh == 0 && qp < n_q) lse[row_base + qp] = flagged ? __builtin_nanf("") : lt > 0.f ? (mu[nq] + __log2f(lt)) * kLn2 : -INFINITY;
  }
  constexpr int CPR = D / 8;  // 16-byte chunks per row
#pragma unroll
  for (int x = 0; x < C::NQW * CPR / 64; ++x) {
    const int idx = x * 64 + lane, row = idx / CPR, ch = idx % CPR;
    if (q_first + row < n_q)
      *reinterpret_cast<u32x4*>(o + (row_base + q_first + row) * D + ch * 8) =
          *reinterpret_cast<const u32x4*>(ot + row * OP + ch * 16);
  }
}

template <int D, int NQT, int BK, bool TRACK>
__global__ void __launch_bounds__(256, fwd_occupancy(NQT))
    fwd_bf16_kernel(cowa_params p, SchedView sv, RowTiles rt, int cap, const __bf16* __restrict__ q,
                    const __bf16* __restrict__ k, const __bf16* __restrict__ v, __bf16* __restrict__ o,
                    float* __restrict__ lse) {
  extern __shared__ __align__(1024) unsigned char smem[];
  RowItem it;
  if (!row_work(p, sv, rt, it)) return;
  if (rt.shape >= 0 && fwd_shape(it.sc.g, p.h_q / p.h_k, D) != rt.shape) return;  // (another launch's)
  fwd_rows<D, NQT, BK, TRACK>(p, rt, it, cap, smem, q, k, v, o, lse);
}

// Both shapes of d = 64, for calls whose sequences and heads differ: they have the
// same row tiles, so each workgroup takes its head's (10 ragged sequences of up to
// 6000 tokens, 16/4 heads: a launch per shape made the
// training pass 422 us instead of 410, this kernel 389 instead of 391).
__global__ void __launch_bounds__(256, fwd_occupancy(1))
    fwd_bf16_d64(cowa_params p, SchedView sv, RowTiles rt, int cap, const __bf16* __restrict__ q,
                 const __bf16* __restrict__ k, const __bf16* __restrict__ v, __bf16* __restrict__ o,
                 float* __restrict__ lse) {
  extern __shared__ __align__(1024) unsigned char smem[];
  RowItem it;
  if (!row_work(p, sv, rt, it)) return;
  if (fwd_shape(it.sc.g, p.h_q / p.h_k, 64) == 1)
    fwd_rows<64, 1, 128, false>(p, rt, it, cap, smem, q, k, v, o, lse);
  else
    fwd_rows<64, 1, 64, false>(p, rt, it, cap, smem, q, k, v, o, lse);
}

// C: the shape (the larger one's LDS of a kernel that has two); list: capacity
template <class C, class Kernel>
hipError_t launch_one(Kernel kern, const cowa_params& p, const SchedView& sv, int64_t list, int shape, const void* q,
                      const void* k, const void* v, void* o, float* lse, hipStream_t stream) {
  const hipError_t err = allow_lds(reinterpret_cast<const void*>(kern), C::LDS_MAX);
  if (err != hipSuccess) return err;
  // as many heads of the group per workgroup as it has, up to one per wave: the
  // fewest query rows per head, and so the fewest masked or unneeded pairs
  const int G = p.h_q / p.h_k, hpw = G % 4 == 0 ? 4 : G % 2 == 0 ? 2 : 1;
  const RowTiles rt = row_tiles(p, sv, hpw, C::NQW * C::NW / hpw, shape);
  const int cap = (int)list;  // (of 256 rows, at least as many as a tile has)
  if (list > C::max_kblocks()) return hipErrorInvalidValue;
  hipLaunchKernelGGL(kern, dim3((unsigned)rt.blocks), dim3(256), C::lds_bytes(cap), stream, p, sv, rt, cap,
                     static_cast<const __bf16*>(q), static_cast<const __bf16*>(k), static_cast<const __bf16*>(v),
                     static_cast<__bf16*>(o), lse);
  return hipGetLastError();
}
template <int D, int NQT, int BK, bool TRACK>
hipError_t launch_shape(const cowa_params& p, const SchedView& sv, int64_t list, int shape, const void* q,
                        const void* k, const void* v, void* o, float* lse, hipStream_t stream) {
  return launch_one<FwdCfg<D, NQT, BK>>(fwd_bf16_kernel<D, NQT, BK, TRACK>, p, sv, list, shape, q, k, v, o, lse, stream);
}

// The shapes of the untracked launch (fwd_shape).  32 rows per wave leave room for two
// waves per SIMD (at d = 128 with 64-key blocks), which hide each other's row
// starts, copies and exponentials, and make twice as many workgroups; 64 rows
// per wave read each K/V fragment from LDS once for two products, which wins
// only where rows are long and many.  V: the visible keys of a row, W: the
// 256-row tiles of the head's group.  Measured at d = 128 (us, 32 rows and 64-key
// blocks / 64 rows and 128-key blocks):
//   1000 tokens, 32/8 heads (V 250, W 15)                23 /   37
//   4096, 32/8 (V 1500, W 64)                            95 /  107
//   2 x 4096, 8/8 heads (V 1000, W 16)                   55 /   68  (121 before: two waves)
//   16384, 32/8, near 4096 (V 5700, W 256)             1111 / 1111
//   8192 dense (V up to 8192, W 128)                    537 /  517
//   32768, 32/8 (V 5900, W 512)                        2039 / 2088
//   2 x 32768, 32/8 (V 5900, W 512)                    4005 / 3857
//   131072, one KV head (V 20000, W 2048)              3091 / 2855
// At d = 64 the exponentials weigh twice as much per product and 32 rows always
// win (65536 tokens, 16/4 heads: 3172 / 3490); 128-key blocks from V = 1024 on
// (3237 against 3472 us there; 27 against 25 at 2048 tokens, V 900).
// (Past 1M keys in a row the list of 128-key blocks does not fit beside its buffers.)
template <int D>
hipError_t launch_d(const cowa_params& p, const SchedView& sv, const RowPlan& plan, const void* q, const void* k,
                    const void* v, void* o, float* lse, hipStream_t stream) {
  const bool one = plan.one_shape();
  hipError_t err = hipSuccess;
  if constexpr (D == 128) {
    static_assert(FwdCfg<128, 2, 128>::max_kblocks() == kFwdList128, "fwd_shape");
    if (plan.used(1)) err = launch_shape<128, 2, 128, false>(p, sv, plan.list128[1], one ? -1 : 1, q, k, v, o, lse, stream);
    if (err == hipSuccess && plan.used(0))
      err = launch_shape<128, 1, 64, false>(p, sv, plan.list64[0], one ? -1 : 0, q, k, v, o, lse, stream);
    if (err == hipSuccess) err = launch_shape<128, 2, 64, true>(p, sv, plan.most64(), -1, q, k, v, o, lse, stream);
  } else {
    if (!one)
      err = launch_one<FwdCfg<64, 1, 128>>(fwd_bf16_d64, p, sv, imax64(plan.list128[1], plan.list64[0]), -1, q, k, v, o,
                                           lse, stream);
    else if (plan.used(1))
      err = launch_shape<64, 1, 128, false>(p, sv, plan.list128[1], -1, q, k, v, o, lse, stream);
    else
      err = launch_shape<64, 1, 64, false>(p, sv, plan.list64[0], -1, q, k, v, o, lse, stream);
    if (err == hipSuccess) err = launch_shape<64, 1, 128, true>(p, sv, plan.most128(), -1, q, k, v, o, lse, stream);
  }
  return err;
}

}  // namespace

// Limits per schedule tile, as the entry point documents them.
int fwd_bf16_max_kblocks(int d, int tk) {
  if (d == 128) return tk == 128 ? FwdCfg<128, 2, 128>::max_kblocks() : FwdCfg<128, 2, 64>::max_kblocks();
  return tk == 128 ? FwdCfg<64, 1, 128>::max_kblocks() : FwdCfg<64, 1, 64>::max_kblocks();
}

bool fwd_bf16_supported(int d, int tq, int tk) {
  return (d == 64 || d == 128) && (tq == 64 || tq == 128) && (tk == 64 || tk == 128);
}

hipError_t launch_fwd_bf16(const cowa_params& p, const SchedView& sv, const RowPlan& plan, const void* q,
                           const void* k, const void* v, void* o, float* lse, hipStream_t stream) {
  return p.head_dim == 128 ? launch_d<128>(p, sv, plan, q, k, v, o, lse, stream)
                           : launch_d<64>(p, sv, plan, q, k, v, o, lse, stream);
}

}  // namespace cowa
