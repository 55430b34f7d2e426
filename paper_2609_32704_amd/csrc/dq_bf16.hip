// CoWA backward, dQ pass, in bfloat16 on the CDNA4 matrix cores (Alg. 2, the
// dQ = scale dS K term).
//
// One workgroup of four waves per (row tile, hpw QO heads of one KV group,
// sequence b): each wave owns 32 or 64 query rows of one head, so a row tile
// holds 4 x 32 (or 64) / hpw rows.  Every QO head of a group sees the same keys, so
// the heads share each K/V block staged in LDS; the row tiles and key blocks
// are the kernel's own and it computes the tile's block list itself.  Per KV
// block, full blocks
// first:
//   S^T = K Q^T and dP^T = V dO^T on v_mfma_f32_32x32x16_bf16, with Q^T and dO^T
//     in registers for the whole row;
//   P^T = exp2(S^T c - LSE log2 e) (LSE from the forward: P is exact, no
//     running maximum) and dS^T = P^T (dP^T - D) on the vector ALUs;
//   dQ^T += K^T dS^T, K^T from the transposing LDS read of the row-major K
//     block.  The S^T accumulator layout is the B-operand layout of dS^T, so dS
//     never leaves registers.
// The 32-key chunks of a row form a software pipeline: chunk step n computes S^T
// and dP^T of chunk n beside the exponentials of chunk n - 1, then dQ^T of
// chunk n - 1.  Alg. 2 adds the dQ terms of different KV blocks with atomics;
// here each row's dQ is complete in registers and written once.  The pass
// recomputes S and dP (the dK/dV pass computed them too).
//
// Shapes.  32 rows per wave and 64-key blocks: 250 registers and 64 KB of LDS
// let two workgroups share a compute unit, and the two waves of a SIMD hide
// each other's row starts, copies, barriers and exponentials.  64 rows per wave
// read each fragment from LDS once for two products, which wins where rows are
// long and many.  Measured at d = 128 (us; 32 rows / 64 rows, 64-key blocks / 64
// rows, 128-key blocks / the pass before, which had 64 rows, 128-key blocks and
// dQ^T two steps behind S^T, and two or one waves for groups that do not divide):
//   1000 tokens, 32/8 heads         22 /    31 /     - /    40
//   8192, 32/8 heads               273 /   277 /     - /   317
//   2 x 4096, 8/8 heads             63 /    80 /     - /   170
//   16384, near 4096 (V 5700)     1386 /  1358 /     - /  1435
//   2 x 32768 (V 5900)            5183 /  5069 /  5144 /  5293
//   131072 (V 20000)             30187 / 29110 / 28655 / 29522
// At d = 64: 8192 tokens, 16/4 heads 93 / 106 / - / 125; 65536 3913 / 4099 / - / 4358.
#include "internal.h"
#include "window_rule.h"
#include "mfma_tiles.h"
#include "work_item.h"

namespace cowa {
namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// S^T and dP^T accumulate in VGPRs (mfma32_v), dQ^T in AGPRs (mfma32), whose products lie
// between the last k-step and the exponentials; block ends have wait states.
__device__ inline void settle(f32x16 (&s)[1], f32x16 (&d)[1]) {
  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" : "+v"(s[0]), "+v"(d[0]));
}
__device__ inline void settle(f32x16 (&s)[2], f32x16 (&d)[2]) {
  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" : "+v"(s[0]), "+v"(s[1]), "+v"(d[0]), "+v"(d[1]));
}

// waves per SIMD that the registers are cut for
constexpr int dq_occupancy(int nqt) { return nqt == 1 ? 2 : 1; }

// NQT: 32-query tiles per wave (columns of S^T); BK: keys per block
template <int D, int NQT_, int BK>
struct Dq32Cfg {
  static constexpr int NW = 4;            // waves per workgroup
  static constexpr int NQT = NQT_;
  static constexpr int NQW = 32 * NQT;    // query rows per wave
  static constexpr int KS = D / 16;       // k-steps over d of S^T and dP^T
  static constexpr int MD = D / 32;       // 32-row d tiles of dQ^T
  static constexpr int NCH = BK / 32;     // 32-key chunks per block
  static constexpr int NG = 3 * KS;       // groups per chunk step: S^T, dP^T and dQ^T per slot x < KS
  using T = SwzTile<D, BK>;
  static constexpr int MAIN_BYTES = 4 * T::BYTES;  // K and V of two blocks; then the row's entry list
  static constexpr int LDS_MAX = 160 * 1024;
  static constexpr int OUT_PITCH = 2 * D + 16;  // staged dQ rows (bytes), in the K/V buffers and list at the end
  static constexpr int OUT_BYTES = NW * NQW * OUT_PITCH;
  static int lds_bytes(int n_kb) {
    return MAIN_BYTES + 4 * n_kb > OUT_BYTES ? MAIN_BYTES + 4 * n_kb : OUT_BYTES;
  }
  static constexpr int max_kblocks() { return (LDS_MAX - MAIN_BYTES) / 4; }
  static_assert(KS == 2 * MD, "one dQ^T product group per k-step slot");
  static_assert(NCH >= 2, "the K buffer of block t - 1 is free within block t");
};

template <int D, int NQT, int BK>
__global__ void __launch_bounds__(256, dq_occupancy(NQT))
    bwd_dq32(cowa_params p, SchedView sv, RowTiles rt, int cap, const __bf16* __restrict__ q,
             const __bf16* __restrict__ k, const __bf16* __restrict__ v, const __bf16* __restrict__ d_o,
             const float* __restrict__ nl, const float* __restrict__ nd, __bf16* __restrict__ dq) {
  using C = Dq32Cfg<D, NQT, BK>;
  using T = typename C::T;
  constexpr int KS = C::KS, MD = C::MD, NCH = C::NCH, NG = C::NG;
  extern __shared__ __align__(1024) unsigned char smem[];

  const int hpw = rt.hpw, wph = C::NW / hpw;  // heads per workgroup, waves per head
  const int G = p.h_q / p.h_k;
  int row, unit, group, hk, q0;
  if (!row_item(rt, grid_units(p, sv), G / hpw, blockIdx.x, row, unit, group)) return;
  const SeqCtx sc = row_ctx(p, sv, rt, row, unit, hk, q0);
  const int n_q = sc.n_q, n_k = sc.n_k;
  if (q0 >= n_q) return;
  if (rt.shape >= 0 && dq_shape(sc.g, G, D) != rt.shape) return;  // (another launch's)
  const int h0 = (hk * (G / hpw) + group) * hpw;  // first QO head (all in KV group hk)

  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int l32 = lane & 31, hh = lane >> 5;  // MFMA column and half
  const int hq = h0 + wave / wph;
  const int q_first = q0 + (wave % wph) * C::NQW;
  const Geo32 g = sc.g;
  const __bf16* kbase = k + (sc.k0 + (int64_t)hk * sc.kh) * D;
  const __bf16* vbase = v + (sc.k0 + (int64_t)hk * sc.kh) * D;
  const uint32_t smem_base = lds_addr(smem);

  // The row tile's block list, in LDS: full blocks from the front, partial
  // ones from the back, both by descending key (at most three merged ranges)
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
  // column of its row in every 1 KB piece it takes (fixed byte offsets within a
  // block); the block position goes into the buffer resource, whose size
  // bounds the reads to the sequence.
  constexpr int RPL = 1024 / (D * 2);  // rows per 1 KB piece
  constexpr int PPW = T::LOADS / 4;    // pieces per wave
  static_assert(T::LOADS % 4 == 0 && (4 * RPL) % 16 == 0, "piece layout");
  uint32_t dma_off[PPW];
  {
    const int row0 = wave * RPL + lane / T::CH;
    const int col = (lane % T::CH) ^ swz<T::CH>(row0);
#pragma unroll
    for (int n = 0; n < PPW; ++n) dma_off[n] = (uint32_t)(((n * 4 * RPL + row0) * D + col * 8) * 2);
  }
  auto kbuf_off = [](int t) { return (t & 1) * 2 * T::BYTES; };
  auto vbuf_off = [](int t) { return (t & 1) * 2 * T::BYTES + T::BYTES; };
  auto stage_piece = [&](const __bf16* base, int kf, int buf_off, int n) {
    const i32x4 rs = buffer_rsrc(base + (int64_t)kf * D, (uint32_t)(n_k - kf) * D * 2);
    dma16_buf(dma_off[n], rs, smem_base + buf_off + wave * 1024 + n * 4 * 1024);
  };
  auto stage = [&](const __bf16* base, int t, int buf_off) {
    const int kf = entry_at(t) * BK;
#pragma unroll
    for (int n = 0; n < PPW; ++n) stage_piece(base, kf, buf_off, n);
  };
  __syncthreads();  // the list and the zeroed buffers are in LDS
  // (issued before the Q and dO loads: the row start waits for memory once)
  if (n_ent > 0) {
    stage(kbase, 0, kbuf_off(0));
    stage(vbase, 0, vbuf_off(0));
  }

  // Q^T and dO^T fragments (B operands): query column 32 nq + l32, d = 16 ks + 8 hh + 0..7;
  // the row values of that query: the exponent offset -LSE log2 e (-inf for a
  // row past n_q or without keys, so P = 0 there) and -D.
  const int64_t row_base = sc.q0 + (int64_t)hq * sc.qh;
  bf16x8 qf[NQT][KS], gf[NQT][KS];
  float mlse[NQT], dn[NQT];
#pragma unroll
  for (int nq = 0; nq < NQT; ++nq) {
    const int qp = q_first + nq * 32 + l32;
    const bool ok = qp < n_q;
    const int64_t row = row_base + (ok ? qp : 0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 a = *reinterpret_cast<const bf16x8*>(q + row * D + ks * 16 + 8 * hh);
      const bf16x8 b = *reinterpret_cast<const bf16x8*>(d_o + row * D + ks * 16 + 8 * hh);
      qf[nq][ks] = ok ? a : bf16x8{};
      gf[nq][ks] = ok ? b : bf16x8{};
    }
    const float nlv = ok ? nl[row] : -INFINITY;
    mlse[nq] = nlv == INFINITY ? -INFINITY : nlv;
    dn[nq] = ok ? nd[row] : 0.f;
  }
  // dQ^T accumulators: element (lane, e) is d = 32 md + 8 (e / 4) + 4 hh + e % 4, query 32 nq + l32
  f32x16 qacc[MD][NQT];
#pragma unroll
  for (int md = 0; md < MD; ++md)
#pragma unroll
    for (int nq = 0; nq < NQT; ++nq) qacc[md][nq] = f32x16{};
  // Move the fragments and accumulators into AGPRs here, long before the first
  // product: the assembly products read Q^T / dO^T from AGPRs, and the compiler
  // would otherwise copy them there just before that read without the wait
  // states a product needs after a vector write of its operands.  These
  // statements emit nothing themselves.
#pragma unroll
  for (int nq = 0; nq < NQT; ++nq) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+a"(qf[nq][ks]), "+a"(gf[nq][ks]));
#pragma unroll
    for (int md = 0; md < MD; ++md) asm volatile("" : "+a"(qacc[md][nq]));
  }
  // LDS fragment offsets for chunk 0 of a block (the swizzle depends on row % 16,
  // so chunks 32 rows further and k-steps 16 rows further add plain row bytes)
  //  K and V rows (A operands of S^T, dP^T): row l32, columns 16 ks + 8 hh + 0..7;
  //  K^T (A operand of dQ^T): transposing reads of rows 4 hh + (lane % 16) / 4
  //  (+ 8 for slots 4..7), columns 32 md + 16 ((lane / 16) % 2) + 4 (lane % 4).
  // The chunk index of a read is XORed with the row's swizzle, so the offset of
  // k-step ks (chunk 2 ks + hh) is that of k-step 0 with bits 2 ks << 4 flipped,
  // and that of d tile md the one of tile 0 with bits 4 md << 4 flipped: one XOR
  // per read instead of a register per offset.
  const int offk0 = T::off(l32, hh);
  int offt0[2];
#pragma unroll
  for (int hf = 0; hf < 2; ++hf) offt0[hf] = T::off_col(4 * hh + ((lane & 15) >> 2) + 8 * hf, 16 * ((lane >> 4) & 1) + 4 * (lane & 3));
  auto offk = [&](int ks) { return offk0 ^ (ks << 5); };
  auto offt = [&](int md, int hf) { return offt0[hf] ^ (md << 6); };
  auto ld_kt = [&](const unsigned char* tile, int md, int row_bytes) -> bf16x8 {
    const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(tile + offt(md, 0) + row_bytes));
    const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(tile + offt(md, 1) + row_bytes));
    const bf16x4 a = __builtin_bit_cast(bf16x4, lo), c2 = __builtin_bit_cast(bf16x4, hi);
    return bf16x8{a[0], a[1], a[2], a[3], c2[0], c2[1], c2[2], c2[3]};
  };

  // S^T and dP^T of two chunks: element (lane, e) is key 8 (e / 4) + 4 hh + e % 4 of
  // the chunk, query 32 nq + l32.  Slots e = 8 kk .. 8 kk + 7 are exactly the keys
  // that lane holds in k-step kk of dQ^T += K^T dS^T (16 keys each).
  f32x16 sacc[2][NQT], pacc[2][NQT];
  u32x4 dsw[2][NQT];  // dS^T of a chunk: bf16 pairs, [k-step][query tile]
  const float c = p.softmax_scale * kLog2e;

  float pv[16 * NQT];   // exponentials in flight between the two halves of an element step
  uint32_t lmask[NQT];  // legal keys of the chunk being masked, per query tile
  // element step e of a chunk (query tile e / 16, slot e % 16), first half: P
  auto soft_a = [&](auto ec, auto rpc, bool masked, int key0) __attribute__((always_inline)) {
    constexpr int e = decltype(ec)::value, rp = decltype(rpc)::value;
    constexpr int nq = e / 16, s = e % 16;
    if (masked) {  // key0: this lane's first key of the chunk
      // the window rule as a bit mask over the lane's keys key0 .. key0 + 31,
      // once per chunk and query tile (slot s holds key key0 + cs)
      constexpr int cs = 8 * (s >> 2) + (s & 3);
      if constexpr (s == 0) lmask[nq] = legal_keys32(g, q_first + nq * 32 + l32, key0);
      const uint32_t m = (uint32_t)((int32_t)(lmask[nq] << (31 - cs)) >> 31);
      sacc[rp][nq][s] = __uint_as_float((__float_as_uint(sacc[rp][nq][s]) & m) | (0xff800000u & ~m));
    }
    pv[e] = __builtin_amdgcn_exp2f(fmaf(sacc[rp][nq][s], c, mlse[nq]));
  };
  // second half (odd e): dS = P (dP - D) of the pair, rounded to bf16
  auto soft_b = [&](auto ec, auto rpc) __attribute__((always_inline)) {
    constexpr int e = decltype(ec)::value, rp = decltype(rpc)::value;
    constexpr int nq = e / 16, s = e % 16;
    if constexpr (s & 1) {
      const float d0 = pv[e - 1] * (pacc[rp][nq][s - 1] + dn[nq]);
      const float d1 = pv[e] * (pacc[rp][nq][s] + dn[nq]);
      const bf16x2 pk = {(__bf16)d0, (__bf16)d1};
      dsw[s / 8][nq][(s & 7) >> 1] = __builtin_bit_cast(uint32_t, pk);
    }
  };
  // the element steps that belong to slot `slot` of NS
  auto soft_slot = [&](auto slotc, auto nsc, auto rpc, bool masked, int key0) __attribute__((always_inline)) {
    constexpr int slot = decltype(slotc)::value, NS = decltype(nsc)::value;
    static_for<16 * NQT>([&](auto ec) {
      constexpr int e = decltype(ec)::value;
      constexpr int sa = e * NS / (16 * NQT);
      constexpr int sb = sa + 1 < NS ? sa + 1 : sa;
      if constexpr (sa == slot) soft_a(ec, rpc, masked, key0);
      if constexpr (sb == slot) soft_b(ec, rpc);
    });
  };

  // LDS: K of block t in K buffer t % 2, V of block t in V buffer t % 2.  The
  // dQ^T products of block t's first chunk step read K of block t - 1, so K of
  // block t + 1 is copied from the end of that step on, once every wave has read
  // K of block t - 1 for the last time; V of block t + 1 is copied from the
  // start of block t.  Both copies go out one 1 KB piece per product group (a
  // burst would hold the wave at the vector memory queue) and land by the end
  // of block t.
  constexpr int PF = 2, RING = PF + 1;
  constexpr int NSG = 2 * KS;  // groups that the exponentials spread over
  int k_prev = 0;  // first key of the previous block
  // One block.  FIRST: the row's first block (nothing before its first chunk).
  // MPREV / MCUR: the chunks turned into dS here from the previous / this block
  // need the element mask.
  auto step = [&](int t, auto firstc, auto mprevc, auto mcurc) __attribute__((always_inline)) {
    constexpr bool FIRST = decltype(firstc)::value, MPREV = decltype(mprevc)::value;
    constexpr bool MCUR = decltype(mcurc)::value;
    const int k_first = entry_at(t) * BK;
    const int kf_next = entry_at(t + 1) * BK;  // (the last block repeats itself)
    const unsigned char* Kt = smem + kbuf_off(t);
    const unsigned char* Vt = smem + vbuf_off(t);
    const unsigned char* Kp = smem + kbuf_off(t + 1);  // K of block t - 1
    constexpr int NGS = NCH * NG;
    constexpr int MID = NG - PF;  // group of the mid-block barrier
    static_assert(MID + PPW <= NGS && PPW <= NGS, "copy pieces per block");
    bf16x8 fa[RING];
    // group GG of the block: chunk step j, slot x, product 0 S^T / 1 dP^T / 2 dQ^T
    constexpr auto gkind = [](int gi) { return gi < 2 * KS ? gi % 2 : 2; };
    constexpr auto gslot = [](int gi) { return gi < 2 * KS ? gi / 2 : gi - 2 * KS; };
    auto load = [&](auto gc, bf16x8& dst) __attribute__((always_inline)) {
      constexpr int GG = decltype(gc)::value, j = GG / NG, gi = GG % NG;
      constexpr int x = gslot(gi), kind = gkind(gi);
      constexpr int jo = (j + NCH - 1) % NCH;  // chunk of the dQ^T products within its block
      constexpr bool OLD = j < 1;             // ... of the previous block
      if constexpr (kind == 0) {
        dst = ld_row8(Kt + offk(x) + j * 32 * D * 2);
      } else if constexpr (kind == 1) {
        dst = ld_row8(Vt + offk(x) + j * 32 * D * 2);
      } else if constexpr (!(FIRST && j == 0)) {
        constexpr int kk = x / MD, md = x % MD;
        dst = ld_kt(OLD ? Kp : Kt, md, (jo * 32 + kk * 16) * D * 2);
      }
    };
    static_for<PF>([&](auto ic) { load(ic, fa[decltype(ic)::value]); });
    __builtin_amdgcn_sched_barrier(0);
    static_for<NGS>([&](auto gc) {
      constexpr int GG = decltype(gc)::value, j = GG / NG, gi = GG % NG;
      constexpr int x = gslot(gi), kind = gkind(gi);
      constexpr bool OLD = j < 1;
      if constexpr (GG == MID) {
        // every read of K of block t - 1 has been issued (fragments run PF
        // groups ahead): once all waves are past them, K of block t + 1 may
        // overwrite that buffer
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (GG < PPW) stage_piece(vbase, kf_next, vbuf_off(t + 1), GG);
      if constexpr (GG >= MID && GG < MID + PPW) stage_piece(kbase, kf_next, kbuf_off(t + 1), GG - MID);
      if constexpr (GG + PF < NGS) load(std::integral_constant<int, GG + PF>{}, fa[(GG + PF) % RING]);
      const bf16x8& a = fa[GG % RING];
      static_for<NQT>([&](auto mc) {
        constexpr int m = decltype(mc)::value;
        if constexpr (kind == 0) {
          if constexpr (x == 0)
            sacc[j & 1][m] = mfma32_v0(a, qf[m][0]);
          else
            sacc[j & 1][m] = mfma32_v(a, qf[m][x], sacc[j & 1][m]);
        } else if constexpr (kind == 1) {
          if constexpr (x == 0)
            pacc[j & 1][m] = mfma32_v0(a, gf[m][0]);
          else
            pacc[j & 1][m] = mfma32_v(a, gf[m][x], pacc[j & 1][m]);
        } else if constexpr (!(FIRST && j == 0)) {
          constexpr int kk = x / MD, md = x % MD;
          qacc[md][m] = mfma32(a, __builtin_bit_cast(bf16x8, dsw[kk][m]), qacc[md][m]);
        }
        // dS^T of the chunk before chunk j (chunk j - 1 of this block, or the
        // last chunk of the previous block), beside the S^T and dP^T products
        if constexpr (!(FIRST && j == 0) && gi < NSG) {
          using SL = std::integral_constant<int, gi * NQT + m>;
          using NSC = std::integral_constant<int, NQT * NSG>;
          using RP = std::integral_constant<int, (j + 1) & 1>;
          if constexpr (j == 0)
            soft_slot(SL{}, NSC{}, RP{}, MPREV, k_prev + (NCH - 1) * 32 + 4 * hh);
          else
            soft_slot(SL{}, NSC{}, RP{}, MCUR, k_first + (j - 1) * 32 + 4 * hh);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      // a chunk step without dQ^T products (start of the row): its S^T and dP^T
      // results are read early in the next step, so settle them here
      if constexpr (FIRST && OLD && gi == NG - 1) {
        settle(sacc[j & 1], pacc[j & 1]);
        __builtin_amdgcn_sched_barrier(0);
      }
    });
    // the last S^T / dP^T products may still be in flight: wait states before
    // anything reads them
    settle(sacc[1], pacc[1]);
    __builtin_amdgcn_sched_barrier(0);
    // register placement: dQ^T accumulators and Q^T / dO^T fragments in AGPRs
    // (read directly by the matrix cores), S^T, dP^T and dS^T in VGPRs; these
    // statements emit nothing
#pragma unroll
    for (int md = 0; md < MD; ++md)
#pragma unroll
      for (int nq = 0; nq < NQT; ++nq) asm volatile("" : "+a"(qacc[md][nq]));
#pragma unroll
    for (int nq = 0; nq < NQT; ++nq)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+a"(qf[nq][ks]), "+a"(gf[nq][ks]));
    k_prev = k_first;
    __builtin_amdgcn_s_waitcnt(0);  // K and V of block t + 1 have landed
    __syncthreads();                // ... for every wave
  };
  // after the last block: dS^T of its last chunk, then the dQ^T products of its
  // last chunk
  auto drain = [&](int t) __attribute__((always_inline)) {
    using R1 = std::integral_constant<int, 1>;
    static_for<16 * NQT>([&](auto ec) { soft_a(ec, R1{}, true, k_prev + (NCH - 1) * 32 + 4 * hh); });
    static_for<16 * NQT>([&](auto ec) { soft_b(ec, R1{}); });
    const unsigned char* Kt = smem + kbuf_off(t);
    static_for<2 * MD>([&](auto gc) {
      constexpr int kk = decltype(gc)::value / MD, md = decltype(gc)::value % MD;
      const bf16x8 a = ld_kt(Kt, md, ((NCH - 1) * 32 + kk * 16) * D * 2);
#pragma unroll
      for (int nq = 0; nq < NQT; ++nq) qacc[md][nq] = mfma32(a, __builtin_bit_cast(bf16x8, dsw[kk][nq]), qacc[md][nq]);
    });
  };
  using TT = std::true_type;
  using FF = std::false_type;

  __builtin_amdgcn_s_waitcnt(0);  // K and V of the first block
  __syncthreads();
  {
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
  }

  // dQ = scale dQ^T, written once per row through LDS: once every wave's last
  // reads are done, each wave stages its rows and stores whole rows, 16
  // bytes per lane, instead of 16-byte pieces of 32 rows per store in the
  // accumulator layout
  const float scale = p.softmax_scale;
  constexpr int OP = C::OUT_PITCH;
  unsigned char* ot = smem + wave * C::NQW * OP;
  __syncthreads();
#pragma unroll
  for (int nq = 0; nq < NQT; ++nq)
#pragma unroll
    for (int md = 0; md < MD; ++md)
#pragma unroll
      for (int j4 = 0; j4 < 4; ++j4) {
        bf16x4 ov;
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) ov[rr] = (__bf16)(scale * qacc[md][nq][4 * j4 + rr]);
        *reinterpret_cast<bf16x4*>(ot + (nq * 32 + l32) * OP + (md * 32 + 8 * j4 + 4 * hh) * 2) = ov;
      }
  constexpr int CPR = D / 8;  // 16-byte chunks per row
#pragma unroll
  for (int x = 0; x < C::NQW * CPR / 64; ++x) {
    const int idx = x * 64 + lane, row = idx / CPR, ch = idx % CPR;
    if (q_first + row < n_q)
      *reinterpret_cast<u32x4*>(dq + (row_base + q_first + row) * D + ch * 8) =
          *reinterpret_cast<const u32x4*>(ot + row * OP + ch * 16);
  }
}

template <int D, int NQT, int BK>
hipError_t launch(const cowa_params& p, const SchedView& sv, int64_t list, int shape, const void* q, const void* k,
                  const void* v, const void* d_o, const float* nl, const float* nd, void* dq, hipStream_t stream) {
  using C = Dq32Cfg<D, NQT, BK>;
  auto kern = bwd_dq32<D, NQT, BK>;
  const hipError_t err = allow_lds(reinterpret_cast<const void*>(kern), C::LDS_MAX);
  if (err != hipSuccess) return err;
  // as many heads of the group per workgroup as it has, up to one per wave
  const int G = p.h_q / p.h_k, hpw = G % 4 == 0 ? 4 : G % 2 == 0 ? 2 : 1;
  const RowTiles rt = row_tiles(p, sv, hpw, C::NQW * C::NW / hpw, shape);
  const int cap = (int)list;  // (of 256 rows, at least as many as a tile has)
  if (list > C::max_kblocks()) return hipErrorInvalidValue;
  hipLaunchKernelGGL(kern, dim3((unsigned)rt.blocks), dim3(256), C::lds_bytes(cap), stream, p, sv, rt, cap,
                     static_cast<const __bf16*>(q), static_cast<const __bf16*>(k), static_cast<const __bf16*>(v),
                     static_cast<const __bf16*>(d_o), nl, nd, static_cast<__bf16*>(dq));
  return hipGetLastError();
}

}  // namespace

// LDS of the dQ pass: two K/V blocks, then one row's block list.  Limits per
// schedule tile, as the entry point documents them.
int bwd_dq_max_kblocks(int d, int tk) { return (160 * 1024 - 4 * tk * d * 2) / 4; }

hipError_t launch_bwd_dq(const cowa_params& p, const SchedView& sv, const RowPlan& plan, const void* q,
                         const void* k, const void* v, const void* d_o, void* dq, const BwdWork& w,
                         hipStream_t stream) {
  // the shapes of the call's heads (dq_shape; measurements at the top of this file)
  static_assert(Dq32Cfg<128, 2, 128>::max_kblocks() == kDqList128 && Dq32Cfg<64, 1, 64>::max_kblocks() == kDqList64,
                "dq_shape");
  hipError_t err = hipSuccess;
  for (int s = kRowShapes - 1; s >= 0 && err == hipSuccess; --s) {
    if (!plan.used(s)) continue;
    const int only = plan.one_shape() ? -1 : s;
    const int64_t l64 = plan.list64[s], l128 = plan.list128[s];
    if (p.head_dim == 128)
      err = s == 2   ? launch<128, 2, 128>(p, sv, l128, only, q, k, v, d_o, w.nl, w.nd, dq, stream)
            : s == 1 ? launch<128, 2, 64>(p, sv, l64, only, q, k, v, d_o, w.nl, w.nd, dq, stream)
                     : launch<128, 1, 64>(p, sv, l64, only, q, k, v, d_o, w.nl, w.nd, dq, stream);
    else
      err = s == 1 ? launch<64, 1, 128>(p, sv, l128, only, q, k, v, d_o, w.nl, w.nd, dq, stream)
                   : launch<64, 1, 64>(p, sv, l64, only, q, k, v, d_o, w.nl, w.nd, dq, stream);
  }
  return err;
}

}  // namespace cowa
