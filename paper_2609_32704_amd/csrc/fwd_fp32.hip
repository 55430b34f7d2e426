// CoWA forward in float32 (Alg. 1) on the fp32 matrix cores.
//
// One workgroup of NW waves per (tile of 16 NQ query rows, QO head, sequence).
// The tile's visible keys are cut into chunks of 16 keys and the waves take
// the chunks in turn, each with its own online softmax (running maximum m,
// running sum l, O rescaled when m moves); at the end the NW partial states are
// merged through LDS.  Splitting the keys rather than the rows over the waves
// gives a 512-token call thousands of waves instead of a few hundred and
// shortens every summation chain (the error against float64 falls with it).
//
// Products are v_mfma_f32_16x16x4_f32 (float32 inputs, float32 accumulation):
//   S^T = K Q^T   A = K (16 keys), B = Q^T (16 queries).  The k-slot order is
//                 free as long as A and B agree: slot lane / 16 of product t of
//                 group g is d = 16 g + 4 (lane / 16) + t, so each lane loads 16
//                 consecutive bytes of its row.
//   O^T += V^T P^T   S^T leaves key 4 (lane / 16) + r of query lane % 16 in
//                 element r, which is the B operand of product r as it stands;
//                 A is V[key][d] with d = 4 (lane % 16) + t for output tile t,
//                 again 16 consecutive bytes per lane.
// K and V go straight from global memory (L2) to registers: no LDS and no
// barrier in the loop; the next chunk's K is in flight during a chunk.
//
// What bounds it: at 512 tokens the chain launch -> window -> Q, K -> few
// chunks -> merge; at thousands of tokens the fp32 matrix rate (the vector-ALU
// kernel before it was bound by its LDS reads and serial reductions).
#include "internal.h"
#include "window_rule.h"
#include "work_item.h"

namespace cowa {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ inline f32x4 mfma4(float a, float b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Shape of a sequence's forward: 16 rows and eight waves (0) up to 256 workgroups
// (one per compute unit), so that every SIMD has work; else four waves (1); at
// d = 128 many tiles take 32 rows per workgroup (2), which halves the K and V reads
// per product (at d = 64 it only costs occupancy).  Waves and rows fix the order of
// the sums, so the tiles of one sequence and the heads of the whole model count,
// not the batch or the heads of this device.  Measured: 512 tokens, 4 heads, d = 64:
// 8.8 us with eight waves, 9.2 with four; 4096 tokens, d = 64, 16 heads: 136 us at 16
// rows, 145 at 32; d = 128, 32 heads: 879 us at 16 rows, 821 at 32 (88 TFLOP/s).  The
// vector-ALU kernel before took 180 us, 3.9 ms and 4.7 ms.
__host__ __device__ inline int fp32_shape(int32_t n_q, int32_t heads, int32_t head_dim) {
  const int64_t wgs = ((int64_t)n_q + 15) / 16 * heads;
  return wgs <= 256 ? 0 : head_dim == 128 && wgs > 4096 ? 2 : 1;
}

// pick: the heads of the whole model if other launches take other sequences, else 0
template <int D, int NQ, int NW>
__global__ void __launch_bounds__(64 * NW, 2)
    fwd_fp32_kernel(cowa_params p, SchedView sv, int pick, const float* __restrict__ q, const float* __restrict__ k,
                    const float* __restrict__ v, float* __restrict__ o, float* __restrict__ lse) {
  constexpr int R = 16 * NQ;     // query rows of the workgroup
  constexpr int CK = 16;         // keys per chunk
  constexpr int GD = D / 16;     // groups of four products over d in S^T; 16-byte loads per row and lane
  constexpr int VD = D / 64;     // 16-byte loads per V row and lane
  constexpr int OP = D + 4;      // LDS row pitch of a partial O (floats)
  __shared__ float so[NW][R][OP];
  __shared__ float sm[NW][R], sl[NW][R];

  const int h = blockIdx.y;
  const int subs = p.tile_q / R;
  const int hk_h = (int)(((int64_t)h * p.h_k) / p.h_q);
  // latest (longest) rows first
  const int rt = (int)gridDim.x - 1 - (int)blockIdx.x;
  int hk;
  const SeqCtx sc = seq_ctx(p, sv, rt / subs, sv.ragged ? hk_h : (int)blockIdx.z * p.h_k + hk_h, true, hk);
  const int i = sc.tile * subs + rt % subs;  // R-row tile within the sequence
  const int n_q = sc.n_q, n_k = sc.n_k;
  const int q0 = i * R;
  if (q0 >= n_q) return;
  if (pick > 0 && fp32_shape(n_q, pick, D) != (NQ == 2 ? 2 : NW == 4 ? 1 : 0)) return;
  const Geo32 g = sc.g;

  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int lr = lane & 15, lg = lane >> 4;
  const int64_t row_base = sc.q0 + (int64_t)h * sc.qh;
  const float* kb = k + (sc.k0 + (int64_t)hk * sc.kh) * D;
  const float* vb = v + (sc.k0 + (int64_t)hk * sc.kh) * D;

  // the tile's chunks: up to three merged ranges of CK-key blocks
  const Runs3 rg = key_block_runs3<CK>(g, q0, (q0 + R < n_q ? q0 + R : n_q) - 1);
  const int n0 = rg.b0 - rg.a0 + 1, n1 = n0 + rg.b1 - rg.a1 + 1, n2 = n1 + rg.b2 - rg.a2 + 1;
  auto chunk_key = [&](int t) -> int {  // first key of chunk t
    return CK * (t < n0 ? rg.a0 + t : t < n1 ? rg.a1 + (t - n0) : rg.a2 + (t - n1));
  };

  f32x4 qf[NQ][GD];
#pragma unroll
  for (int n = 0; n < NQ; ++n) {
    const int qp = q0 + 16 * n + lr;
    const float* qrow = q + (row_base + (qp < n_q ? qp : n_q - 1)) * D;
#pragma unroll
    for (int x = 0; x < GD; ++x) qf[n][x] = *reinterpret_cast<const f32x4*>(qrow + 16 * x + 4 * lg);
  }
  f32x4 acc[NQ][VD][4];  // O^T: d = 64 x + 4 (4 lg + r) + t in element r, query 16 n + lr
  float m[NQ], l[NQ];
#pragma unroll
  for (int n = 0; n < NQ; ++n) {
    m[n] = -INFINITY;
    l[n] = 0.f;
#pragma unroll
    for (int x = 0; x < VD; ++x)
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[n][x][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const float c = p.softmax_scale * 1.4426950408889634f;  // log2(e)

  f32x4 kf[GD];
  auto load_k = [&](int key0) {
    const int kp = key0 + lr;
    const float* krow = kb + (int64_t)(kp < n_k ? kp : n_k - 1) * D + 4 * lg;
#pragma unroll
    for (int x = 0; x < GD; ++x) kf[x] = *reinterpret_cast<const f32x4*>(krow + 16 * x);
  };
  if (wave < n2) load_k(chunk_key(wave));
  for (int t = wave; t < n2; t += NW) {
    const int key0 = chunk_key(t);
    f32x4 vf[4][VD];  // V of key 4 lg + r, d = 64 x + 4 lr + 0..3
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int kp = key0 + 4 * lg + r;
      const float* vrow = vb + (int64_t)(kp < n_k ? kp : n_k - 1) * D + 4 * lr;
#pragma unroll
      for (int x = 0; x < VD; ++x) vf[r][x] = *reinterpret_cast<const f32x4*>(vrow + 64 * x);
    }
    // keys past the end have weight 0, and V 0 as well: an infinity of the last key
    // would otherwise count as 0 x inf
    if (key0 + CK > n_k) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int x = 0; x < VD; ++x)
          if (key0 + 4 * lg + r >= n_k) vf[r][x] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // S^T in two chains per query tile (even and odd groups): shorter sums, and
    // independent products to issue
    f32x4 s[NQ];
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
      f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int x = 0; x < GD; x += 2)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s0 = mfma4(kf[x][e], qf[n][x][e], s0);
          s1 = mfma4(kf[x + 1][e], qf[n][x + 1][e], s1);
        }
      s[n] = s0 + s1;
    }
    if (t + NW < n2) load_k(chunk_key(t + NW));
    const bool full = key_block_full(g, q0, q0 + R - 1, key0, key0 + CK - 1);
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
      // mask (positions past the sequence included), maximum of the query
      const int qp = q0 + 16 * n + lr;
      float mx = -INFINITY;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (!full) s[n][r] = legal32(g, qp, key0 + 4 * lg + r) ? s[n][r] : -INFINITY;
        mx = fmaxf(mx, s[n][r]);
      }
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float m_new = fmaxf(m[n], mx * c);
      const float m_use = m_new == -INFINITY ? 0.f : m_new;
      if (__ballot(m_new > m[n]) != 0) {
        const float alpha = __builtin_amdgcn_exp2f(m[n] - m_use);
        l[n] *= alpha;
#pragma unroll
        for (int x = 0; x < VD; ++x)
#pragma unroll
          for (int tt = 0; tt < 4; ++tt) acc[n][x][tt] *= alpha;
        m[n] = m_new;
      }
      float ps = 0.f;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float pv = __builtin_amdgcn_exp2f(fmaf(s[n][r], c, -m_use));
        s[n][r] = pv;
        ps += pv;
      }
      l[n] += ps;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int x = 0; x < VD; ++x)
#pragma unroll
        for (int tt = 0; tt < 4; ++tt)
#pragma unroll
          for (int n = 0; n < NQ; ++n) acc[n][x][tt] = mfma4(vf[r][x][tt], s[n][r], acc[n][x][tt]);
  }

  // merge the waves' states
#pragma unroll
  for (int n = 0; n < NQ; ++n) {
    float lt = l[n] + __shfl_xor(l[n], 16);
    lt += __shfl_xor(lt, 32);
    if (lg == 0) {
      sm[wave][16 * n + lr] = m[n];
      sl[wave][16 * n + lr] = lt;
    }
#pragma unroll
    for (int x = 0; x < VD; ++x)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        *reinterpret_cast<f32x4*>(&so[wave][16 * n + lr][64 * x + 16 * lg + 4 * r]) =
            f32x4{acc[n][x][0][r], acc[n][x][1][r], acc[n][x][2][r], acc[n][x][3][r]};
  }
  __syncthreads();
  for (int x = tid; x < R * D / 4; x += 64 * NW) {
    const int row = x / (D / 4), d4 = x % (D / 4);
    if (q0 + row >= n_q) break;  // rows ascend with x
    float mm = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) mm = fmaxf(mm, sm[w][row]);
    const float mu = mm == -INFINITY ? 0.f : mm;
    f32x4 ov = {0.f, 0.f, 0.f, 0.f};
    float lt = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float f = __builtin_amdgcn_exp2f(sm[w][row] - mu);
      const f32x4 a = *reinterpret_cast<const f32x4*>(&so[w][row][4 * d4]);
      lt = fmaf(sl[w][row], f, lt);
#pragma unroll
      for (int e = 0; e < 4; ++e) ov[e] = fmaf(a[e], f, ov[e]);
    }
    const float inv = lt > 0.f ? 1.f / lt : 0.f;
    *reinterpret_cast<f32x4*>(o + (row_base + q0 + row) * D + 4 * d4) = ov * inv;
    if (d4 == 0) lse[row_base + q0 + row] = lt > 0.f ? (mm + log2f(lt)) * 0.6931471805599453f : -INFINITY;
  }
}

template <int D, int NQ, int NW>
hipError_t launch(const cowa_params& p, const SchedView& sv, int pick, const float* q, const float* k, const float* v,
                  float* o, float* lse, hipStream_t stream) {
  const dim3 grid((unsigned)sv.n_qt * (p.tile_q / (16 * NQ)), p.h_q, sv.ragged ? 1 : p.batch);
  hipLaunchKernelGGL((fwd_fp32_kernel<D, NQ, NW>), grid, dim3(64 * NW), 0, stream, p, sv, pick, q, k, v, o, lse);
  return hipGetLastError();
}

// A launch takes the sequences of its shape, or (pick 0) all of them.
template <int D>
hipError_t launch_d(const cowa_params& p, const SchedView& sv, const float* q, const float* k, const float* v, float* o,
                    float* lse, hipStream_t stream) {
  const int heads = p.h_q / p.h_k * p.h_k_total;
  const int64_t tiles = (int64_t)sv.n_qt * (p.tile_q / 16);
  bool used[3] = {false, false, false};
  if (tiles > (1 << 23))  // (32 rows keep the grid within the launch limit)
    used[2] = true;
  else if (sv.ragged)
    for (int b = 0; b < p.batch; ++b) {
      const int n_q = p.cu_seqlens_q[b + 1] - p.cu_seqlens_q[b];
      if (n_q > 0) used[fp32_shape(n_q, heads, D)] = true;
    }
  else
    used[fp32_shape(p.n_q, heads, D)] = true;
  const int pick = used[0] + used[1] + used[2] > 1 ? heads : 0;
  hipError_t err = hipSuccess;
  if (used[2]) err = launch<D, 2, 4>(p, sv, pick, q, k, v, o, lse, stream);
  if (err == hipSuccess && used[1]) err = launch<D, 1, 4>(p, sv, pick, q, k, v, o, lse, stream);
  if (err == hipSuccess && used[0]) err = launch<D, 1, 8>(p, sv, pick, q, k, v, o, lse, stream);
  return err;
}

}  // namespace

hipError_t launch_fwd_fp32(const cowa_params& p, const SchedView& sv, const float* q, const float* k,
                           const float* v, float* o, float* lse, hipStream_t stream) {
  return p.head_dim == 64 ? launch_d<64>(p, sv, q, k, v, o, lse, stream)
                          : launch_d<128>(p, sv, q, k, v, o, lse, stream);
}

}  // namespace cowa
