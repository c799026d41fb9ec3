// Edge phase of one MGN message-passing step in fp32 (Sec. 2.1: every edge
// latent is updated by the edge MLP from itself and its two end nodes, then
// each node sums the new messages of its in-edges), with one wave per
// receiver-aligned tile of at most 32 edges.  The products run as split fp16
// products on weights that stream through LDS (split32_common.hpp).
#include "edge_walk.hpp"
#include "split32_common.hpp"

namespace mgn {
namespace dev {

template <int LD>
struct __attribute__((aligned(16))) EdgeFwdLds {
  static constexpr int SL = LD + 4;  // staged row stride: eight lanes' 16-byte writes hit distinct banks
  static constexpr int SR = LD == 128 ? 16 : 8;  // rows staged at a time (two blocks share the LDS)
  u32x4 w[2][X3<LD>::CH];
  __attribute__((aligned(16))) float vec[4][LD];  // b1, b2, gamma, beta
  __attribute__((aligned(16))) float stage[X3_NW][SR * SL];
};

// Forward: e' = e + m (when write_e), agg = receiver sums of m, with
// m = LN(W2 relu(b1 + P_s + P_r + W1e e) + b2) (the node products P = [W1s
// h, W1r h] of the block come from the node kernels).  Two blocks per CU, so
// one block's loads, LayerNorm and barriers lie under the other's MFMAs; that
// leaves 256 registers, hence e is read again for the residual.  Measured per
// launch: 434,558 edges at width 128 0.354 -> 0.189 ms (fp32 MFMA version ->
// this; 0.125 ms without its memory traffic, which alone takes 0.095 ms at the
// copy rate), the eight-patch batch (0.68M edges) at width 160 0.92 -> 0.44 ms.  Rows past a
// tile's end, and tiles past the block's range, read a valid row that is
// never stored or summed.
template <int LD>
__global__ void __launch_bounds__(X3_NT) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_edge_fwd_x3(EdgeTiles tl, const float* e_in, float* e_out, int write_e, const float* __restrict__ Pn, MlpW w,
              float eps, float* __restrict__ agg, float* __restrict__ slots) {
  typedef X3<LD> Z;
  typedef EdgeFwdLds<LD> Lds;
  __shared__ Lds S;
  const int tid = threadIdx.x, lane = tid & 63, row = lane & 31, hh = lane >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int f0 = 8 * hh;  // the lane's first feature
  const u32x4 *W1 = (const u32x4*)w.S1, *W2 = (const u32x4*)w.S2;
  const BlockRange br = block_range(walk_units(tl));
  // the nodes are dealt to all blocks, those without a run among them
  if (tl.run) zero_share<LD>(tl, (int64_t)blockIdx.x * X3_NW + wv, (int64_t)gridDim.x * X3_NW, lane, agg);
  if (br.tb >= br.tend) return;
  gemm_x3_start<LD>(W1, S.w, tid);
  for (int f = tid; f < LD; f += X3_NT) {
    S.vec[0][f] = w.b1[f];
    S.vec[1][f] = w.b2[f];
    S.vec[2][f] = w.gamma[f];
    S.vec[3][f] = w.beta[f];
  }
  const int lastE = (int)(tl.n_edges - 1);
  auto erow = [&](int4 d) { return min(max(d.z + min(row, tile_rows(d) - 1), 0), lastE); };
  EdgeSteps es;
  int4 d = es.first(tl, br.tb + wv, br.stride, br.tend);
  int snd = tl.senders[erow(d)], rcv = tl.receivers[erow(d)];
  __syncthreads();
  float2 carry[2] = {{0.f, 0.f}, {0.f, 0.f}};  // the open segment's sum
  const int n_steps = walk_steps(tl);
  for (int64_t t = br.tb; t < br.tend; t += br.stride)
  for (int st = 0; st < n_steps; ++st) {
    const int4 dn = es.next(tl);
    // formed per step: kept across steps, what depends on them spills
    const int lane = (tid & 63) + opaque_zero(), row = lane & 31, hh = lane >> 5, f0 = 8 * hh;
    const int n = tile_rows(d);
    const TileRow<LD> tr(d, lastE, row, hh);
    const bool chunk = d.y < 0;
    // ---- z1 = W1e e + ((b1 + P_s) + P_r), a1 = relu(z1); the gathered node
    // products are requested while the product runs
    f32x16 acc[Z::NOB];
    float x[Z::KL];
    load_row_x3<LD>(x, tr.at(e_in));
    // P_s and P_r of the features that K step ks has freed x's registers of,
    // summed one step later
    f32x4 p[Z::KL / 4], ps[2], pr[2];
    auto add_p = [&](int ks) {
#pragma unroll
      for (int k = 0; k < 2; ++k)
        p[2 * ks + k] = (*reinterpret_cast<const f32x4*>(S.vec[0] + f0 + 16 * ks + 4 * k) + ps[k]) + pr[k];
    };
    gemm_x3<LD>(acc, x, W1, W2, S.w, 0, tid, [&](int ks) {
      if (ks > 0) add_p(ks - 1);
      const float* q = Pn + f0 + 16 * ks;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        ps[k] = *reinterpret_cast<const f32x4*>(q + (size_t)snd * (2 * LD) + 4 * k);
        pr[k] = *reinterpret_cast<const f32x4*>(q + (size_t)rcv * (2 * LD) + LD + 4 * k);
      }
    });
    add_p(Z::KS - 1);
#pragma unroll
    for (int c = 0; c < Z::KL / 4; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) x[4 * c + r] = relu32(acc[c >> 2][4 * (c & 3) + r] + p[c][r]);
    // ---- z2 = b2 + W2 a1
    gemm_x3<LD>(acc, x, W2, W1, S.w, Z::NC & 1, tid);
#pragma unroll
    for (int c = 0; c < Z::KL / 4; ++c) {
      const f32x4 b2 = *reinterpret_cast<const f32x4*>(S.vec[1] + f0 + Z::pf(c));
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[c >> 2][4 * (c & 3) + r] += b2[r];
    }
    // the next tile's ids, in flight during the LayerNorm
    const int snd_n = tl.senders[erow(dn)], rcv_n = tl.receivers[erow(dn)];
    ln_x3<LD>(acc, hh, eps);
#pragma unroll
    for (int c = 0; c < Z::KL / 4; ++c) {
      const f32x4 ga = *reinterpret_cast<const f32x4*>(S.vec[2] + f0 + Z::pf(c));
      const f32x4 be = *reinterpret_cast<const f32x4*>(S.vec[3] + f0 + Z::pf(c));
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[c >> 2][4 * (c & 3) + r] = ga[r] * acc[c >> 2][4 * (c & 3) + r] + be[r];  // m
    }
    // ---- receiver sums, SR rows at a time, and e_out = e + m: read and
    // written as whole rows here, where the messages lie row by row
    const uint32_t ends = segment_ends(row, n, rcv, d.y);
    float2 tot[2] = {{0.f, 0.f}, {0.f, 0.f}};
    float* stage = S.stage[wv];
#pragma unroll
    for (int r0 = 0; r0 < 32; r0 += Lds::SR) {
      if (row / Lds::SR == r0 / Lds::SR)
#pragma unroll
        for (int c = 0; c < Z::KL / 4; ++c)
          *reinterpret_cast<f32x4*>(stage + (row - r0) * Lds::SL + f0 + Z::pf(c)) =
              f32x4{acc[c >> 2][4 * (c & 3)], acc[c >> 2][4 * (c & 3) + 1], acc[c >> 2][4 * (c & 3) + 2],
                    acc[c >> 2][4 * (c & 3) + 3]};
      wave_lds_sync();
      seg_sums<LD, Lds::SL, Lds::SR>(stage, lane, ends, r0, rcv, chunk, slots + (size_t)(-1 - d.y) * LD, agg, carry,
                                     tot, [&](const float2 (&v)[Lds::SR], int p, bool on) {
        if (!write_e) return;
        float2 e[Lds::SR];
        const uint32_t o = 2 * (on ? p : lane);
#pragma unroll
        for (int u = 0; u < Lds::SR; ++u)
          e[u] = *reinterpret_cast<const float2*>(e_in + tr.base + (size_t)max(min(r0 + u, n - 1), 0) * LD + o);
#pragma unroll
        for (int u = 0; u < Lds::SR; ++u)
          if (r0 + u < n && on)
            *reinterpret_cast<float2*>(e_out + tr.base + (size_t)(r0 + u) * LD + o) =
                float2{e[u].x + v[u].x, e[u].y + v[u].y};
      });
      wave_lds_sync();
    }
    if (n < 32 || (ends >> 31)) carry[0] = carry[1] = float2{0.f, 0.f};  // rows past the end
    if (!tl.run && !chunk && d.y > d.x) zero_empty<LD>(d.x, d.y, tl.rowptr, lane, agg);
    d = dn;
    snd = snd_n;
    rcv = rcv_n;
  }
}

// ================================================================= reverse
// Edge reverse with dW2 in the same pass: per tile, from the block's input
// edge latents e, the node products P (the first layer is recomputed as in
// the forward) and the incoming gradients (ebar_in, aggbar at the receiver),
// it writes zbar = dL/dz1 (for the sender sums and dW1e), the receiver sums R
// of zbar and ebar_out = ebar_in + W1e^T zbar, and accumulates dW2 = sum dz2^T
// a1 (DwAcc), db2, dgamma, dbeta (column sums) and db1 (the sum of the
// receiver sums).  dW1e = sum zbar^T e is a pass of its own over the two
// streams (k_wgrad_x3).  One block per CU.  At width 128 it has eight waves,
// two per SIMD: in 256 registers a wave holds the pieces of a1 and dz2, one
// product and an eighth of dW2 (ebar_in is read twice instead of being kept).
// At width 160 that does not fit, and the block has four waves of 512.
//   Measured per launch: 434,558 edges at width 128 1.11 -> 0.56 ms (fp32 MFMA
// version, dW1e included, -> this; its dW1e pass takes 0.11 ms), the eight-patch
// batch (0.68M edges) at width 160 2.20 -> 1.36 ms.  At width 128, with its loads and
// stores taken away, it still took 0.49 ms: the phases that the eight waves enter
// together bound it.  By counter the waves issue 19% of their time and wait 55%, the
// MFMA pipe is busy 17%; it moves 1.8 GB where its streams are 0.9 (98 registers
// are spilled), at 3.5 TB/s.
// Partials per block: db1 at LD^2, dW2, db2, dgamma, dbeta.
template <int LD>
struct EdgeBwd {
  static constexpr int NW = LD == 128 ? 8 : 4;
  static constexpr int NT = 64 * NW;
  static constexpr int SL = LD + 4;
  static constexpr int SR = LD == 128 ? 8 : 16;  // rows staged for the receiver sums at a time
};
template <int LD>
struct __attribute__((aligned(16))) EdgeBwdLds {
  typedef EdgeBwd<LD> K;
  u32x4 w[2][X3<LD>::CH];
  __attribute__((aligned(16))) float vec[3][LD];  // b1, b2, gamma
  __attribute__((aligned(16))) float stage[K::NW][K::SR * K::SL];
  DwLds<LD, K::NW> dw;
};

template <int LD>
__global__ void __launch_bounds__(EdgeBwd<LD>::NT)
    __attribute__((amdgpu_waves_per_eu(EdgeBwd<LD>::NW / 4, EdgeBwd<LD>::NW / 4)))
k_edge_bwd_x3(EdgeTiles tl, const float* __restrict__ e_in, const float* ebar_in, int have_ebar, float* ebar_out,
              const float* __restrict__ Pn, const float* __restrict__ aggbar, MlpW w, float eps, float* zbar,
              float* __restrict__ R, float* __restrict__ slots, Partials part) {
  typedef X3<LD> Z;
  typedef EdgeBwd<LD> K;
  constexpr int NW = K::NW, NT = K::NT;
  __shared__ EdgeBwdLds<LD> S;
  const int tid = threadIdx.x, lane = tid & 63, row = lane & 31, hh = lane >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int f0 = 8 * hh;  // the lane's first feature
  const u32x4 *W1 = (const u32x4*)w.S1, *W2 = (const u32x4*)w.S2, *W2t = (const u32x4*)w.S2t, *W1t = (const u32x4*)w.S1t;
  const BlockRange br = block_range<NW>(walk_units(tl));
  gemm_x3_start<LD, NT>(W1, S.w, tid);
  for (int f = tid; f < LD; f += NT) {
    S.vec[0][f] = w.b1[f];
    S.vec[1][f] = w.b2[f];
    S.vec[2][f] = w.gamma[f];
  }
  const int lastE = (int)(tl.n_edges - 1);
  auto erow = [&](int4 d) { return min(max(d.z + min(row, tile_rows(d) - 1), 0), lastE); };
  DwAcc<LD, NW> dw2;
  dw2.clear();
  ColSumX3<LD> db2, dga, dbe;
  float2 db1[2] = {{0.f, 0.f}, {0.f, 0.f}};
  EdgeSteps es;
  int4 d = es.first(tl, br.tb + wv, br.stride, br.tend);
  int snd = tl.senders[erow(d)], rcv = tl.receivers[erow(d)];
  if (tl.run) zero_share<LD>(tl, (int64_t)blockIdx.x * NW + wv, (int64_t)gridDim.x * NW, lane, R);
  __syncthreads();
  float2 carry[2] = {{0.f, 0.f}, {0.f, 0.f}};  // the open segment's sum
  const int n_steps = walk_steps(tl);
  for (int64_t t = br.tb; t < br.tend; t += br.stride)
  for (int st = 0; st < n_steps; ++st) {
    const int4 dn = es.next(tl);
    // formed per step: kept across steps, what depends on them spills
    const int lane = (tid & 63) + opaque_zero(), row = lane & 31, hh = lane >> 5, f0 = 8 * hh;
    const int n = tile_rows(d);
    const TileRow<LD> tr(d, lastE, row, hh);
    const bool chunk = d.y < 0, live = row < n;
    // ---- z1 and a1 as in the forward; the mask z1 > 0
    f32x16 acc[Z::NOB];
    float x[Z::KL];
    load_row_x3<LD>(x, tr.at(e_in));
    float a1[Z::KL];
    uint32_t mask[(Z::KL + 31) / 32] = {};
    {
      f32x4 p[Z::KL / 4], ps[2], pr[2];
      auto add_p = [&](int ks) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
          p[2 * ks + k] = (*reinterpret_cast<const f32x4*>(S.vec[0] + f0 + 16 * ks + 4 * k) + ps[k]) + pr[k];
      };
      gemm_x3<LD, NT>(acc, x, W1, W2, S.w, 0, tid, [&](int ks) {
        if (ks > 0) add_p(ks - 1);
        const float* q = Pn + f0 + 16 * ks;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          ps[k] = *reinterpret_cast<const f32x4*>(q + (size_t)snd * (2 * LD) + 4 * k);
          pr[k] = *reinterpret_cast<const f32x4*>(q + (size_t)rcv * (2 * LD) + LD + 4 * k);
        }
      });
      add_p(Z::KS - 1);
#pragma unroll
      for (int v = 0; v < Z::KL; ++v) {
        const float z = acc[v >> 4][v & 15] + p[v >> 2][v & 3];
        a1[v] = relu32(z);
        if (z > 0.f) mask[v >> 5] |= 1u << (v & 31);
      }
      // pinned: the compiler would keep every z1 instead, to compare it later
#pragma unroll
      for (int k = 0; k < (Z::KL + 31) / 32; ++k) asm volatile("" : "+v"(mask[k]));
    }
    // ---- z2 = b2 + W2 a1 and its LayerNorm
    RowPieces<LD> A1;
    float g[Z::KL];
    gemm_keep<LD, NT>(acc, a1, A1, W2, W2t, S.w, Z::NC & 1, tid, [](int) {});
#pragma unroll
    for (int v = 0; v < Z::KL; ++v) acc[v >> 4][v & 15] += S.vec[1][Z::feat(hh, v)];
    const float rstd = ln_x3<LD>(acc, hh, eps);
    // ---- mbar = ebar_in + aggbar[receiver]; dbeta, dgamma; the LayerNorm
    // reverse (padded features: gamma = 0 and xhat is left out, dz2 zero)
#pragma unroll
    for (int c = 0; c < Z::KL / 4; ++c) {
      f32x4 u = *reinterpret_cast<const f32x4*>(aggbar + (size_t)rcv * LD + f0 + Z::pf(c));
      const f32x4 e = *reinterpret_cast<const f32x4*>(tr.at(ebar_in) + Z::pf(c));
#pragma unroll
      for (int r = 0; r < 4; ++r) g[4 * c + r] = (have_ebar ? e[r] : 0.f) + u[r];
      if ((c & 3) == 3) __builtin_amdgcn_sched_barrier(0);  // sixteen values' loads at a time
    }
#pragma unroll
    for (int v = 0; v < Z::KL; ++v) g[v] = live ? g[v] : 0.f;
    dbe.add([&](int v) { return g[v]; }, lane & 15);
    dga.add([&](int v) { return g[v] * acc[v >> 4][v & 15]; }, lane & 15);
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int v = 0; v < Z::KL; ++v) {
      g[v] *= S.vec[2][Z::feat(hh, v)];
      s1 += g[v];
      s2 += g[v] * acc[v >> 4][v & 15];
    }
    const float m1 = sum_hh(s1) * (1.0f / Z::DR), m2 = sum_hh(s2) * (1.0f / Z::DR);
#pragma unroll
    for (int v = 0; v < Z::KL; ++v)
      g[v] = live && (Z::DR == LD || Z::feat(hh, v) < Z::DR) ? rstd * (g[v] - m1 - acc[v >> 4][v & 15] * m2) : 0.f;  // dz2
    db2.add([&](int v) { return g[v]; }, lane & 15);
    // ---- dW2 += dz2^T a1
    RowPieces<LD> G;
    split_row<LD>(G, g, live);
    dw2.add(G, A1, live, S.dw, tid);
    // the next tile's ids
    const int snd_n = tl.senders[erow(dn)], rcv_n = tl.receivers[erow(dn)];
    // ---- zbar = W2^T dz2 where z1 > 0
    gemm_pieces<LD, NT>(acc, [&](int ks) { return G.p[ks]; }, G.e, W2t, W1t, S.w, 0, tid, [](int) {});
#pragma unroll
    for (int v = 0; v < Z::KL; ++v) g[v] = (mask[v >> 5] >> (v & 31)) & 1u ? acc[v >> 4][v & 15] : 0.f;
    // ---- zbar's rows and their receiver sums
    const uint32_t ends = segment_ends(row, n, rcv, d.y);
    float* stage = S.stage[wv];
#pragma unroll
    for (int r0 = 0; r0 < 32; r0 += K::SR) {
      if (row / K::SR == r0 / K::SR)
#pragma unroll
        for (int c = 0; c < Z::KL / 4; ++c)
          *reinterpret_cast<f32x4*>(stage + (row - r0) * K::SL + f0 + Z::pf(c)) =
              f32x4{g[4 * c], g[4 * c + 1], g[4 * c + 2], g[4 * c + 3]};
      wave_lds_sync();
      seg_sums<LD, K::SL, K::SR>(stage, lane, ends, r0, rcv, chunk, slots + (size_t)(-1 - d.y) * LD, R, carry, db1,
                                 [&](const float2 (&v)[K::SR], int p, bool on) {
#pragma unroll
        for (int u = 0; u < K::SR; ++u)
          if (r0 + u < n && on) *reinterpret_cast<float2*>(zbar + tr.base + (size_t)(r0 + u) * LD + 2 * p) = v[u];
      });
      wave_lds_sync();
    }
    if (n < 32 || (ends >> 31)) carry[0] = carry[1] = float2{0.f, 0.f};  // rows past the end
    if (!tl.run && !chunk && d.y > d.x) zero_empty<LD>(d.x, d.y, tl.rowptr, lane, R);
    // ---- ebar_out = ebar_in + W1e^T zbar
    gemm_x3<LD, NT>(acc, g, W1t, W1, S.w, Z::NC & 1, tid);
    {
      const float* q = tr.at(ebar_in);
      float* o = tr.at(ebar_out);
#pragma unroll
      for (int c = 0; c < Z::KL / 4; ++c) {
        f32x4 u = have_ebar ? *reinterpret_cast<const f32x4*>(q + Z::pf(c)) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < 4; ++r) u[r] += acc[c >> 2][4 * (c & 3) + r];
        if (live) *reinterpret_cast<f32x4*>(o + Z::pf(c)) = u;
      }
    }
    d = dn;
    snd = snd_n;
    rcv = rcv_n;
  }
  // ---- block partials: dW2 from the owning waves, the vectors summed over
  // the waves in wave order
  float* base = part.buf + (size_t)blockIdx.x * part.stride + (size_t)LD * LD;
  dw2.store(base + LD, tid);
  __syncthreads();
  float* red = &S.stage[0][0];  // [4][NW][LD]: db1, db2, dgamma, dbeta
  *reinterpret_cast<float2*>(red + wv * LD + 2 * lane) = db1[0];
  if (LD / 2 > 64 && lane + 64 < LD / 2) *reinterpret_cast<float2*>(red + wv * LD + 2 * (lane + 64)) = db1[1];
  db2.put(red + (NW + wv) * LD, lane);
  dga.put(red + (2 * NW + wv) * LD, lane);
  dbe.put(red + (3 * NW + wv) * LD, lane);
  __syncthreads();
  for (int idx = tid; idx < 4 * LD; idx += NT) {
    const int k = idx / LD, f = idx % LD;
    float v = 0.f;
#pragma unroll
    for (int u = 0; u < NW; ++u) v += red[(k * NW + u) * LD + f];
    base[k == 0 ? f : LD + LD * LD + (k - 1) * LD + f] = v;
  }
}

// ======================================================= weight gradient
// Up to three weight gradients dW[o][n] = sum over rows of G[row][o] X[row][n]
// of row-major fp32 [M][LD] streams (DwAcc) in one launch, 128 rows per round,
// the next round's rows in flight while one is added.  Each job has its own
// blocks and partials (blocks [b0, b0 + nb) of the grid), shared out by rows, one
// block per CU in all: three launches that each spread 32,768 rows over all
// CUs left three times the partials, and per MP step of the 32^3 mesh the
// weight gradients and their reductions took 0.24 + 0.044 ms against 0.22 +
// 0.022 ms.  A long job is bound by reading its streams.
template <int LD>
__global__ void __launch_bounds__(X3_NT) __attribute__((amdgpu_waves_per_eu(1, 1)))
k_wgrad_x3(WgradJobs jobs) {
  typedef X3<LD> Z;
  __shared__ DwLds<LD, X3_NW> S;
  const int tid = threadIdx.x, lane = tid & 63, row = lane & 31, f0 = 8 * (lane >> 5);
  const int wv = tid >> 6, b = blockIdx.x;
  int k = 0;
  while (k + 1 < jobs.n && b >= jobs.j[k + 1].b0) ++k;
  const WgradJob job = jobs.j[k];
  const int64_t M = job.M, blk = b - job.b0;
  DwAcc<LD, X3_NW> dw;
  dw.clear();
  const int64_t nr = (M + 32 * X3_NW - 1) / (32 * X3_NW);
  float g[Z::KL], x[Z::KL];
  auto at = [&](int64_t r) { return r * (32 * X3_NW) + 32 * wv + row; };
  auto load = [&](int64_t r) {
    const int64_t u = min(at(r), M - 1);
    load_row_x3<LD>(g, job.G + (size_t)u * LD + f0);
    load_row_x3<LD>(x, job.X + (size_t)u * LD + f0);
  };
  int64_t r = blk;
  if (r < nr) load(r);
  for (; r < nr; r += job.nb) {
    const bool live = at(r) < M;
    dw.add_rows(g, x, live, S, tid, [&] {
      if (r + job.nb < nr) load(r + job.nb);
    });
  }
  dw.store(job.part + (size_t)blk * job.stride, tid);
}

}  // namespace dev

using namespace dev;

// two blocks per CU
static constexpr int kSplitBlocks = 512;

hipError_t launch_edge_fwd_x3(int lat, const EdgeTiles& tl, const void* e_in, void* e_out, int write_e, const void* Pn,
                              const MlpW& w, float eps, float* agg, float* slots, hipStream_t s) {
  if (tl.n_tiles <= 0) return hipSuccess;
  if (tl.n_edges <= 0 || !w.S1 || !w.S2) return hipErrorInvalidValue;
  const EdgeTiles t = plan_runs(tl, X3_NW * kSplitBlocks);
  const int g = unit_blocks(walk_n(t), X3_NW, kSplitBlocks);
#define F(LD)                                                                                                     \
  hipLaunchKernelGGL(k_edge_fwd_x3<LD>, dim3(g), dim3(X3_NT), 0, s, t, (const float*)e_in, (float*)e_out, write_e, \
                     (const float*)Pn, w, eps, agg, slots)
  MGN_BY_WIDTH(lat, F);
#undef F
  return hipGetLastError();
}

// one block per CU
static constexpr int kSplitPartBlocks = 256;

hipError_t launch_edge_bwd_x3(int lat, const EdgeTiles& tl, const void* e, const float* ebar_in, int have_ebar,
                              float* ebar_out, const void* Pn, const float* aggbar, const MlpW& w, float eps,
                              void* zbar, float* R, float* slots, const Partials& part, int* nblocks, hipStream_t s) {
  *nblocks = 0;
  if (tl.n_tiles <= 0) return hipSuccess;
  if (tl.n_edges <= 0 || part.stride < 2LL * lat * lat + 4 * lat || !w.S1 || !w.S2 || !w.S1t || !w.S2t)
    return hipErrorInvalidValue;
  const int nw = lat == 128 ? EdgeBwd<128>::NW : EdgeBwd<160>::NW;
  const int most = std::min(kSplitPartBlocks, part.max_blocks);
  const EdgeTiles t = plan_runs(tl, nw * most);
  const int g = unit_blocks(walk_n(t), nw, most);
  *nblocks = g;
#define F(LD)                                                                                                  \
  hipLaunchKernelGGL(k_edge_bwd_x3<LD>, dim3(g), dim3(EdgeBwd<LD>::NT), 0, s, t, (const float*)e, ebar_in, have_ebar,    \
                     ebar_out, (const float*)Pn, aggbar, w, eps, (float*)zbar, R, slots, part)
  MGN_BY_WIDTH(lat, F);
#undef F
  return hipGetLastError();
}

hipError_t launch_wgrad_x3(int lat, WgradJobs& jobs, const Partials& part, hipStream_t s) {
  int64_t rounds = 0;
  for (int k = 0; k < jobs.n; ++k) rounds += (jobs.j[k].M + 32 * X3_NW - 1) / (32 * X3_NW);
  if (jobs.n <= 0 || rounds <= 0) return hipSuccess;
  const int most = std::min(kSplitPartBlocks, part.max_blocks);
  int b0 = 0;
  for (int k = 0; k < jobs.n; ++k) {
    WgradJob& j = jobs.j[k];
    if (j.M <= 0 || j.stride < (int64_t)lat * lat) return hipErrorInvalidValue;
    const int64_t nr = (j.M + 32 * X3_NW - 1) / (32 * X3_NW);
    // its share of the blocks, rounded down: one block more than CUs would run
    // after all the others
    j.nb = (int)std::max<int64_t>(1, rounds <= most ? nr : nr * most / rounds);
    j.b0 = b0;
    b0 += j.nb;
  }
#define F(LD) hipLaunchKernelGGL(k_wgrad_x3<LD>, dim3(b0), dim3(X3_NT), 0, s, jobs)
  MGN_BY_WIDTH(lat, F);
#undef F
  return hipGetLastError();
}

}  // namespace mgn
