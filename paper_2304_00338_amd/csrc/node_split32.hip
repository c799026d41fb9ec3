// Node phase of one MGN message-passing step in fp32 (Sec. 2.1: every node
// latent is updated by the node MLP from itself and the sum of its incoming
// edge messages, with LayerNorm and a residual), the sender sums of the edge
// reverse and the node encoder's forward, on the split fp16 products of split32_common.hpp: one wave per
// 32-node unit, four waves per block, two blocks per CU.
//   Bound by the latency of a unit's chain of products where there are fewer
// units than waves (32,768 nodes are one unit per SIMD); reading every weight
// line once at the start, to have it in the L2, did not shorten it.  Measured
// per launch at 32,768 nodes, width 128: forward with node products 75 -> 38
// us, reverse 104 -> 57 us; at 17,800 nodes forward 58 -> 30 us (fp32 MFMA
// version, 16-node units -> this).
//
// The first layer acts on the concatenation [h, agg]; it is evaluated as
// (W1h h + W1a agg) + b1 with the two column blocks of W1 (the same linear
// map, in this summation order in the forward and the reverse's recompute).
#include "launch.hpp"
#include "split32_common.hpp"

namespace mgn {
namespace dev {

template <int LD, int NV>
struct __attribute__((aligned(16))) NodeLds {
  u32x4 w[2][X3<LD>::CH];
  __attribute__((aligned(16))) float vec[NV][LD];
};

// x += a vector of LDS, by the lane's values.
template <int LD, class F>
__device__ __forceinline__ void with_vec(const float* vec, int hh, F&& f) {
#pragma unroll
  for (int c = 0; c < X3<LD>::KL / 4; ++c) {
    const f32x4 b = *reinterpret_cast<const f32x4*>(vec + 8 * hh + X3<LD>::pf(c));
#pragma unroll
    for (int r = 0; r < 4; ++r) f(4 * c + r, b[r]);
  }
}

// The node products [W1s y, W1r y] of the next edge MLP into P_out.  par:
// parity of the LDS buffers, kept current; next: the product that follows.
template <int LD>
__device__ __forceinline__ void emit_x3(const float* y, const u32x4* Ws, const u32x4* Wr, const u32x4* next,
                                        u32x4 (*buf)[X3<LD>::CH], int& par, int tid, bool live, float* p) {
  typedef X3<LD> Z;
  f32x16 acc[Z::NOB];
  RowPieces<LD> r;
  gemm_keep<LD, X3_NT>(acc, y, r, Ws, Wr, buf, par, tid, [](int) {});
  par += Z::NC;
  if (live) store_row_x3<LD>(p, [&](int v) { return acc[v >> 4][v & 15]; });
  gemm_pieces<LD, X3_NT>(acc, [&](int ks) { return r.p[ks]; }, r.e, Wr, next, buf, par, tid, [](int) {});
  par += Z::NC;
  if (live) store_row_x3<LD>(p + LD, [&](int v) { return acc[v >> 4][v & 15]; });
}

// z1 = (W1h h + W1a agg) + b1.  Both products add into one accumulator, which
// takes one scale 2^T for the two: the smaller of what each row and its
// matrix would take (the other row is scaled down by the difference).  agg is
// read twice, for its largest value and then into the registers that h leaves.
template <int LD>
__device__ __forceinline__ void node_z1_x3(f32x16 (&acc)[X3<LD>::NOB], float* x, const float* h, const float* agg,
                                           const u32x4* Wh, const u32x4* Wa, const u32x4* next, const float* b1,
                                           u32x4 (*buf)[X3<LD>::CH], int& par, int tid) {
  typedef X3<LD> Z;
  const int wh = weight_exp<LD>(Wh), wa = weight_exp<LD>(Wa);
  load_row_x3<LD>(x, agg);
  const int ea = row_exp<LD>(x);
  load_row_x3<LD>(x, h);
  const int T = min(row_exp<LD>(x) + wh, ea + wa);
  gemm_raw<LD, X3_NT, false>(acc, [&](int ks) { return split8(x + 8 * ks, T - wh); }, Wh, Wa, buf, par, tid,
                             [&](int ks) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const f32x4 u = *reinterpret_cast<const f32x4*>(agg + 16 * ks + 4 * j);
#pragma unroll
      for (int r = 0; r < 4; ++r) x[8 * ks + 4 * j + r] = u[r];
    }
  });
  par += Z::NC;
  gemm_raw<LD, X3_NT, true>(acc, [&](int ks) { return split8(x + 8 * ks, T - wa); }, Wa, next, buf, par, tid,
                            [](int) {});
  par += Z::NC;
  scale_acc<LD>(acc, -T);
  with_vec<LD>(b1, (tid >> 5) & 1, [&](int v, float b) { acc[v >> 4][v & 15] += b; });
}

// Forward: h_out = h + LN(W2 relu(z1) + b2); with EMIT, also the next block's
// node products P_out = [W1s h_out, W1r h_out] ([N][2 LD]) from the next edge
// MLP nx.  Rows past N read row N - 1 and store nothing.
template <int LD, bool EMIT>
__global__ void __launch_bounds__(X3_NT) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_node_fwd_x3(int64_t N, const float* h_in, const float* __restrict__ agg, MlpW w, MlpW nx, float eps, float* h_out,
              float* __restrict__ P_out) {
  typedef X3<LD> Z;
  __shared__ NodeLds<LD, 4> S;
  const int tid = threadIdx.x, row = tid & 31, hh = (tid >> 5) & 1, wv = tid >> 6;
  const u32x4 *Wh = (const u32x4*)w.S1, *Wa = (const u32x4*)w.S1a, *W2 = (const u32x4*)w.S2;
  const BlockRange br = block_range((N + 31) >> 5);
  if (br.tb >= br.tend) return;
  gemm_x3_start<LD>(Wh, S.w, tid);
  for (int f = tid; f < LD; f += X3_NT) {
    S.vec[0][f] = w.b1[f];
    S.vec[1][f] = w.b2[f];
    S.vec[2][f] = w.gamma[f];
    S.vec[3][f] = w.beta[f];
  }
  int par = 0;
  __syncthreads();
  for (int64_t t = br.tb; t < br.tend; t += br.stride) {
    const int64_t u = (t + wv) * 32 + row;
    const bool live = t + wv < br.tend && u < N;
    const size_t o = (size_t)min(u, N - 1) * LD + 8 * hh;
    f32x16 acc[Z::NOB];
    float x[Z::KL];
    node_z1_x3<LD>(acc, x, h_in + o, agg + o, Wh, Wa, W2, S.vec[0], S.w, par, tid);
#pragma unroll
    for (int v = 0; v < Z::KL; ++v) x[v] = relu32(acc[v >> 4][v & 15]);
    // h again, for the residual, in the registers that a1 leaves
    gemm_x3<LD>(acc, x, W2, EMIT ? (const u32x4*)nx.S1s : Wh, S.w, par, tid, [&](int ks) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const f32x4 q = *reinterpret_cast<const f32x4*>(h_in + o + 16 * ks + 4 * j);
#pragma unroll
        for (int r = 0; r < 4; ++r) x[8 * ks + 4 * j + r] = q[r];
      }
    });
    par += Z::NC;
    with_vec<LD>(S.vec[1], hh, [&](int v, float b) { acc[v >> 4][v & 15] += b; });
    ln_x3<LD>(acc, hh, eps);
    with_vec<LD>(S.vec[2], hh, [&](int v, float g) { acc[v >> 4][v & 15] *= g; });
    with_vec<LD>(S.vec[3], hh, [&](int v, float b) { x[v] += acc[v >> 4][v & 15] + b; });
    if (live) store_row_x3<LD>(h_out + o, [&](int v) { return x[v]; });
    if (EMIT)
      emit_x3<LD>(x, (const u32x4*)nx.S1s, (const u32x4*)nx.S1r, Wh, S.w, par, tid, live,
                  P_out + (size_t)min(u, N - 1) * (2 * LD) + 8 * hh);
  }
}

// Reverse of the node phase for the rows of hbar_in = dL/dh_out: the forward
// recomputed (z1 bitwise as in the forward), the LayerNorm reverse (padded
// features of dz2 zeroed), da1 = W2^T dz2, dz1 = da1 where z1 > 0, hbar_part =
// hbar_in + W1h^T dz1 and aggbar = W1a^T dz1.  The rows of a1, dz2 and dz1 go
// to the streams (fp32 [N][LD] each) for the weight-gradient passes (dW1 = sum
// dz1^T [h, agg], dW2 = sum dz2^T a1); db1, db2, dgamma and dbeta are column
// sums, written per block as [4][LD] partials (db1, db2, dgamma, dbeta).
template <int LD>
__global__ void __launch_bounds__(X3_NT) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_node_bwd_x3(int64_t N, const float* __restrict__ h_in, const float* __restrict__ agg,
              const float* __restrict__ hbar_in, MlpW w, float eps, float* __restrict__ hbar_part,
              float* __restrict__ aggbar, float* __restrict__ a1s, float* __restrict__ dz2s, float* __restrict__ dz1s,
              Partials part) {
  typedef X3<LD> Z;
  __shared__ NodeLds<LD, 3> S;
  __shared__ float red[4][X3_NW][LD];
  const int tid = threadIdx.x, lane = tid & 63, row = tid & 31, hh = (tid >> 5) & 1, wv = tid >> 6, i = lane & 15;
  const u32x4 *Wh = (const u32x4*)w.S1, *Wa = (const u32x4*)w.S1a, *W2 = (const u32x4*)w.S2;
  const u32x4 *Wht = (const u32x4*)w.S1t, *Wat = (const u32x4*)w.S1at, *W2t = (const u32x4*)w.S2t;
  const BlockRange br = block_range((N + 31) >> 5);
  gemm_x3_start<LD>(Wh, S.w, tid);
  for (int f = tid; f < LD; f += X3_NT) {
    S.vec[0][f] = w.b1[f];
    S.vec[1][f] = w.b2[f];
    S.vec[2][f] = w.gamma[f];
  }
  ColSumX3<LD> cs[4];  // db1, db2, dgamma, dbeta
  __syncthreads();
  for (int64_t t = br.tb; t < br.tend; t += br.stride) {
    const int64_t u = (t + wv) * 32 + row;
    const bool live = t + wv < br.tend && u < N;
    const size_t o = (size_t)min(u, N - 1) * LD + 8 * hh;
    int par = 0;  // six products: even
    // ---- the forward: z1, its ReLU mask, a1, z2 and its LayerNorm
    f32x16 acc[Z::NOB];
    float x[Z::KL];
    node_z1_x3<LD>(acc, x, h_in + o, agg + o, Wh, Wa, W2, S.vec[0], S.w, par, tid);
    uint32_t mask[(Z::KL + 31) / 32] = {};
#pragma unroll
    for (int v = 0; v < Z::KL; ++v) {
      const float z = acc[v >> 4][v & 15];
      x[v] = relu32(z);
      if (z > 0.f) mask[v >> 5] |= 1u << (v & 31);
    }
    // pinned: the compiler would keep every z1 instead, to compare it later
#pragma unroll
    for (int k = 0; k < (Z::KL + 31) / 32; ++k) asm volatile("" : "+v"(mask[k]));
    if (live) store_row_x3<LD>(a1s + o, [&](int v) { return x[v]; });
    // the incoming gradient arrives in the registers that a1 leaves
    gemm_x3<LD>(acc, x, W2, W2t, S.w, par, tid, [&](int ks) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const f32x4 q = *reinterpret_cast<const f32x4*>(hbar_in + o + 16 * ks + 4 * j);
#pragma unroll
        for (int r = 0; r < 4; ++r) x[8 * ks + 4 * j + r] = q[r];
      }
    });
    par += Z::NC;
    with_vec<LD>(S.vec[1], hh, [&](int v, float b) { acc[v >> 4][v & 15] += b; });
    const float rstd = ln_x3<LD>(acc, hh, eps);
    // ---- dbeta, dgamma (live rows); the LayerNorm reverse
#pragma unroll
    for (int v = 0; v < Z::KL; ++v) x[v] = live ? x[v] : 0.f;
    cs[3].add([&](int v) { return x[v]; }, i);
    cs[2].add([&](int v) { return x[v] * acc[v >> 4][v & 15]; }, i);
    float s1 = 0.f, s2 = 0.f;
    with_vec<LD>(S.vec[2], hh, [&](int v, float g) {
      x[v] *= g;  // dxh
      s1 += x[v];
      s2 += x[v] * acc[v >> 4][v & 15];
    });
    const float m1 = sum_hh(s1) * (1.0f / Z::DR), m2 = sum_hh(s2) * (1.0f / Z::DR);
#pragma unroll
    for (int v = 0; v < Z::KL; ++v)
      x[v] = live && (Z::DR == LD || Z::feat(hh, v) < Z::DR) ? rstd * (x[v] - m1 - acc[v >> 4][v & 15] * m2) : 0.f;
    cs[1].add([&](int v) { return x[v]; }, i);
    if (live) store_row_x3<LD>(dz2s + o, [&](int v) { return x[v]; });
    // ---- da1 = W2^T dz2, dz1 = da1 where z1 > 0
    gemm_x3<LD>(acc, x, W2t, Wht, S.w, par, tid);
    par += Z::NC;
#pragma unroll
    for (int v = 0; v < Z::KL; ++v) x[v] = (mask[v >> 5] >> (v & 31)) & 1u ? acc[v >> 4][v & 15] : 0.f;
    cs[0].add([&](int v) { return x[v]; }, i);
    if (live) store_row_x3<LD>(dz1s + o, [&](int v) { return x[v]; });
    // ---- hbar_part = hbar_in + W1h^T dz1, aggbar = W1a^T dz1
    RowPieces<LD> r;
    gemm_keep<LD, X3_NT>(acc, x, r, Wht, Wat, S.w, par, tid, [&](int ks) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const f32x4 q = *reinterpret_cast<const f32x4*>(hbar_in + o + 16 * ks + 4 * j);
#pragma unroll
        for (int k = 0; k < 4; ++k) x[8 * ks + 4 * j + k] = q[k];
      }
    });
    par += Z::NC;
    if (live) store_row_x3<LD>(hbar_part + o, [&](int v) { return x[v] + acc[v >> 4][v & 15]; });
    gemm_pieces<LD, X3_NT>(acc, [&](int ks) { return r.p[ks]; }, r.e, Wat, Wh, S.w, par, tid, [](int) {});
    if (live) store_row_x3<LD>(aggbar + o, [&](int v) { return acc[v >> 4][v & 15]; });
  }
  // ---- block partials [4][LD]: the waves' column sums added in wave order
#pragma unroll
  for (int k = 0; k < 4; ++k) cs[k].put(red[k][wv], lane);
  __syncthreads();
  float* base = part.buf + (size_t)blockIdx.x * part.stride;
  for (int idx = tid; idx < 4 * LD; idx += X3_NT) {
    const int k = idx / LD, c = idx % LD;
    float v = 0.f;
#pragma unroll
    for (int q = 0; q < X3_NW; ++q) v += red[k][q][c];
    base[idx] = v;
  }
}

// Node encoder (Sec. 2.1: the node features are encoded to the latent width by
// an MLP with LayerNorm): h0 = LN(W2 relu(W1 x + b1) + b2), x the 8 node
// inputs, the first layer (K = 8) as one fp32 fma chain per feature from LDS;
// with EMIT the node products of the first MP block from the first edge MLP
// nx, as the node phase does.
constexpr int NEK = 8;  // node inputs

template <int LD>
struct __attribute__((aligned(16))) NodeEncX3Lds {
  NodeLds<LD, 4> N;
  float4 w1[LD][2];  // W1 [LD][8]
};

template <int LD, bool EMIT>
__global__ void __launch_bounds__(X3_NT) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_node_enc_x3(int64_t N, const float* __restrict__ x_in, MlpW w, MlpW nx, float eps, float* __restrict__ h_out,
              float* __restrict__ P_out) {
  typedef X3<LD> Z;
  __shared__ NodeEncX3Lds<LD> S;
  const int tid = threadIdx.x, row = tid & 31, hh = (tid >> 5) & 1, wv = tid >> 6;
  const u32x4* W2 = (const u32x4*)w.S2;
  const BlockRange br = block_range((N + 31) >> 5);
  if (br.tb >= br.tend) return;
  gemm_x3_start<LD>(W2, S.N.w, tid);
  for (int f = tid; f < LD * NEK; f += X3_NT) reinterpret_cast<float*>(S.w1)[f] = w.W1f[f];
  for (int f = tid; f < LD; f += X3_NT) {
    S.N.vec[0][f] = w.b1[f];
    S.N.vec[1][f] = w.b2[f];
    S.N.vec[2][f] = w.gamma[f];
    S.N.vec[3][f] = w.beta[f];
  }
  int par = 0;
  __syncthreads();
  for (int64_t t = br.tb; t < br.tend; t += br.stride) {
    const int64_t u = (t + wv) * 32 + row;
    const bool live = t + wv < br.tend && u < N;
    const int64_t v0 = min(u, N - 1);
    const float4 xa = *reinterpret_cast<const float4*>(x_in + v0 * NEK);
    const float4 xb = *reinterpret_cast<const float4*>(x_in + v0 * NEK + 4);
    f32x16 acc[Z::NOB];
    float x[Z::KL];
    const NodeEncX3Lds<LD>& L = fresh(S);
    with_vec<LD>(L.N.vec[0], hh, [&](int v, float z) {
      const float4 wa = L.w1[Z::feat(hh, v)][0], wb = L.w1[Z::feat(hh, v)][1];
      z = __builtin_fmaf(wa.x, xa.x, z);
      z = __builtin_fmaf(wa.y, xa.y, z);
      z = __builtin_fmaf(wa.z, xa.z, z);
      z = __builtin_fmaf(wa.w, xa.w, z);
      z = __builtin_fmaf(wb.x, xb.x, z);
      z = __builtin_fmaf(wb.y, xb.y, z);
      z = __builtin_fmaf(wb.z, xb.z, z);
      z = __builtin_fmaf(wb.w, xb.w, z);
      x[v] = relu32(z);
    });
    gemm_x3<LD>(acc, x, W2, EMIT ? (const u32x4*)nx.S1s : W2, S.N.w, par, tid);
    par += Z::NC;
    with_vec<LD>(S.N.vec[1], hh, [&](int v, float b) { acc[v >> 4][v & 15] += b; });
    ln_x3<LD>(acc, hh, eps);
    with_vec<LD>(S.N.vec[2], hh, [&](int v, float g) { acc[v >> 4][v & 15] *= g; });
    with_vec<LD>(S.N.vec[3], hh, [&](int v, float b) { x[v] = acc[v >> 4][v & 15] + b; });
    if (live) store_row_x3<LD>(h_out + v0 * LD + 8 * hh, [&](int v) { return x[v]; });
    if (EMIT)
      emit_x3<LD>(x, (const u32x4*)nx.S1s, (const u32x4*)nx.S1r, W2, S.N.w, par, tid, live,
                  P_out + v0 * (2 * LD) + 8 * hh);
  }
}

// Sender-side sums and the node gradient through the edge MLP's sender and
// receiver blocks: S_v = sum of zbar over the reverses of v's in-edges (the
// out-edges of v), added in edge order from 0.0; hbar_out = hbar_part + W1s^T S +
// W1r^T R.  The rows of S go to S_out (fp32 [N][LD]) for the weight gradients dW1s =
// sum S h^T, dW1r = sum R h^T.
//   Bound by the gather of E rows.  A wave reads whole rows (its unit's reversed
// edge ids are one contiguous piece of rev), RB in flight, and hands each node's
// sum to the node's two lanes through LDS, SN nodes at a time; with a quarter of
// a row per lane, as before, every 16-byte access of a wave spanned 64 cache
// lines.  Measured per launch (fp32 MFMA version -> this): 434,558 edges and 32,768
// nodes at width 128 90 -> 75 us (reading the rows takes 47 at the copy rate; more
// rows in flight made no difference), the eight-patch batch at width 160 203 -> 187
// us, 11,260 edges 21.0 -> 20.8 us (ids and bounds requested per pass: 22.5).
template <int LD>
struct __attribute__((aligned(16))) SrcSumLds {
  static constexpr int SN = LD == 128 ? 16 : 8;  // (two blocks share the LDS)
  static constexpr int SL = LD + 4;
  u32x4 w[2][X3<LD>::CH];
  __attribute__((aligned(16))) float stage[X3_NW][SN * SL];
};

template <int LD>
__global__ void __launch_bounds__(X3_NT) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_node_srcsum_x3(int64_t N, const int32_t* __restrict__ rowptr, const int32_t* __restrict__ receivers,
                 const int32_t* __restrict__ rev, const float* __restrict__ zbar, const float* R,
                 const float* hbar_part, MlpW w, float* hbar_out, float* S_out) {
  typedef X3<LD> Z;
  typedef SrcSumLds<LD> Lds;
  constexpr int RB = LD == 128 ? 32 : 16;  // rows in flight
  constexpr int NP = LD / 2;               // feature pairs of a row
  __shared__ Lds S;
  const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const u32x4 *Ws = (const u32x4*)w.S1st, *Wr = (const u32x4*)w.S1rt;
  const BlockRange br = block_range((N + 31) >> 5);
  if (br.tb >= br.tend) return;
  gemm_x3_start<LD>(Ws, S.w, tid);
  const int ws = weight_exp<LD>(Ws), wr = weight_exp<LD>(Wr);
  __syncthreads();
  for (int64_t t = br.tb; t < br.tend; t += br.stride) {
    const int lane = (tid & 63) + opaque_zero(), row = lane & 31, hh = lane >> 5;
    const int64_t v0 = min((t + wv) * 32, N);  // the unit's first node (N: no unit)
    const bool live = t + wv < br.tend && v0 + row < N;
    const size_t o = (size_t)min(v0 + row, N - 1) * LD + 8 * hh;
    float* st = S.stage[wv];
    float x[Z::KL];
    // the first edges of every SN nodes; no edges past the range
    const int rp = t + wv < br.tend ? rowptr[min(v0 + min(lane, 32 / Lds::SN) * Lds::SN, N)] : 0;
    const int ulast = __builtin_amdgcn_readlane(rp, 32 / Lds::SN) - 1;
    // reversed edge ids and receivers of the next 64 rows, requested a batch ahead
    int id = 0, rc = 0;
    auto ids = [&](int b) {
      if (b <= ulast) {
        id = rev[min(b + lane, ulast)];
        rc = receivers[min(b + lane, ulast)];
      }
    };
    ids(__builtin_amdgcn_readlane(rp, 0));
    load_row_x3<LD>(x, R + o);
    const int er = row_exp<LD>(x);
#pragma unroll 1
    for (int p = 0; p < 32 / Lds::SN; ++p) {
      const int lo = __builtin_amdgcn_readlane(rp, p), hi = __builtin_amdgcn_readlane(rp, p + 1), last = hi - 1;
      const int va = (int)v0 + p * Lds::SN;
#pragma unroll
      for (int u = 0; u < Lds::SN; ++u) {  // nodes without edges
        *reinterpret_cast<float2*>(st + u * Lds::SL + 2 * lane) = float2{0.f, 0.f};
        if (NP > 64 && lane < NP - 64) *reinterpret_cast<float2*>(st + u * Lds::SL + 2 * (lane + 64)) = float2{0.f, 0.f};
      }
      float2 c0 = {0.f, 0.f}, c1 = {0.f, 0.f};
      for (int b = lo; b < hi; b += RB) {
        float2 z0[RB], z1[RB];
#pragma unroll
        for (int u = 0; u < RB; ++u) {
          const float* q = zbar + (size_t)__builtin_amdgcn_readlane(id, u) * LD;
          z0[u] = *reinterpret_cast<const float2*>(q + 2 * lane);
          if (NP > 64) z1[u] = *reinterpret_cast<const float2*>(q + 2 * (lane < NP - 64 ? lane + 64 : lane));
        }
        // row u ends its node's segment
        const int nx = __shfl(rc, min(lane + 1, 63));
        const uint64_t ends = __ballot(b + lane == last || (b + lane < last && nx != rc));
        const int node = rc - va;
        ids(min(b + RB, hi));
#pragma unroll
        for (int u = 0; u < RB; ++u) {
          c0.x += z0[u].x;
          c0.y += z0[u].y;
          if (NP > 64) {
            c1.x += z1[u].x;
            c1.y += z1[u].y;
          }
          if ((ends >> u) & 1u) {
            float* q = st + __builtin_amdgcn_readlane(node, u) * Lds::SL;
            *reinterpret_cast<float2*>(q + 2 * lane) = c0;
            if (NP > 64 && lane < NP - 64) *reinterpret_cast<float2*>(q + 2 * (lane + 64)) = c1;
            c0 = c1 = float2{0.f, 0.f};
          }
        }
      }
      wave_lds_sync();
      if (row / Lds::SN == p) load_row_x3<LD>(x, st + (row % Lds::SN) * Lds::SL + 8 * hh);
      wave_lds_sync();
    }
    if (live) store_row_x3<LD>(S_out + o, [&](int v) { return x[v]; });
    // both products add into one accumulator at one scale (see node_z1_x3)
    f32x16 acc[Z::NOB];
    const int T = min(row_exp<LD>(x) + ws, er + wr);
    gemm_raw<LD, X3_NT, false>(acc, [&](int ks) { return split8(x + 8 * ks, T - ws); }, Ws, Wr, S.w, 0, tid,
                               [&](int ks) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const f32x4 u = *reinterpret_cast<const f32x4*>(R + o + 16 * ks + 4 * j);
#pragma unroll
        for (int r = 0; r < 4; ++r) x[8 * ks + 4 * j + r] = u[r];
      }
    });
    gemm_raw<LD, X3_NT, true>(acc, [&](int ks) { return split8(x + 8 * ks, T - wr); }, Wr, Ws, S.w, Z::NC & 1, tid,
                              [&](int ks) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const f32x4 u = *reinterpret_cast<const f32x4*>(hbar_part + o + 16 * ks + 4 * j);
#pragma unroll
        for (int r = 0; r < 4; ++r) x[8 * ks + 4 * j + r] = u[r];
      }
    });
    scale_acc<LD>(acc, -T);
    if (live) store_row_x3<LD>(hbar_out + o, [&](int v) { return x[v] + acc[v >> 4][v & 15]; });
  }
}

}  // namespace dev

using namespace dev;

// two blocks per CU
static constexpr int kNodeSplitBlocks = 512;
static int node_blocks(int64_t N, int most) {
  return unit_blocks((N + 31) / 32, X3_NW, std::min(kNodeSplitBlocks, most));
}

hipError_t launch_node_fwd_x3(int lat, int64_t N, const float* h_in, const float* agg, const MlpW& w, const MlpW* nx,
                              float eps, float* h_out, float* P_out, hipStream_t s) {
  if (N <= 0) return hipSuccess;
  if ((lat != 128 && lat != 160) || !w.S1 || !w.S1a || !w.S2 || (nx && (!nx->S1s || !nx->S1r || !P_out)))
    return hipErrorInvalidValue;
  const int g = node_blocks(N, kNodeSplitBlocks);
  const MlpW nn = nx ? *nx : w;
#define F(L)                                                                                                          \
  if (nx)                                                                                                             \
    hipLaunchKernelGGL((k_node_fwd_x3<L, true>), dim3(g), dim3(X3_NT), 0, s, N, h_in, agg, w, nn, eps, h_out, P_out); \
  else                                                                                                                \
    hipLaunchKernelGGL((k_node_fwd_x3<L, false>), dim3(g), dim3(X3_NT), 0, s, N, h_in, agg, w, nn, eps, h_out, P_out)
  MGN_BY_WIDTH(lat, F);
#undef F
  return hipGetLastError();
}

hipError_t launch_node_bwd_x3(int lat, int64_t N, const float* h, const float* agg, const float* hbar_in,
                              const MlpW& w, float eps, float* hbar_part, float* aggbar, float* streams,
                              const Partials& part, int* nblocks, hipStream_t s) {
  *nblocks = 0;
  if (N <= 0) return hipSuccess;
  if ((lat != 128 && lat != 160) || !w.S1 || !w.S1a || !w.S2 || !w.S1t || !w.S1at || !w.S2t || part.stride < 4LL * lat)
    return hipErrorInvalidValue;
  const int g = node_blocks(N, part.max_blocks);
  *nblocks = g;
  float* a1s = streams;
  float* dz2s = streams + (size_t)N * lat;
  float* dz1s = streams + (size_t)2 * N * lat;
#define F(L)                                                                                                      \
  hipLaunchKernelGGL(k_node_bwd_x3<L>, dim3(g), dim3(X3_NT), 0, s, N, h, agg, hbar_in, w, eps, hbar_part, aggbar, \
                     a1s, dz2s, dz1s, part)
  MGN_BY_WIDTH(lat, F);
#undef F
  return hipGetLastError();
}

hipError_t launch_node_srcsum_x3(int lat, int64_t N, const int32_t* rowptr, const int32_t* receivers,
                                 const int32_t* rev, const float* zbar, const float* R, const float* hbar_part,
                                 const MlpW& w, float* hbar_out, float* S_out, hipStream_t s) {
  if (N <= 0) return hipSuccess;
  if ((lat != 128 && lat != 160) || !w.S1st || !w.S1rt) return hipErrorInvalidValue;
  const int g = node_blocks(N, kNodeSplitBlocks);
#define F(L)                                                                                                       \
  hipLaunchKernelGGL(k_node_srcsum_x3<L>, dim3(g), dim3(X3_NT), 0, s, N, rowptr, receivers, rev, zbar, R, hbar_part, \
                     w, hbar_out, S_out)
  MGN_BY_WIDTH(lat, F);
#undef F
  return hipGetLastError();
}

hipError_t launch_node_enc_x3(int lat, int64_t N, const float* x, const MlpW& w, const MlpW* nx, float eps,
                              float* h_out, float* P_out, hipStream_t s) {
  if (N <= 0) return hipSuccess;
  if ((lat != 128 && lat != 160) || !w.S2 || (nx && (!nx->S1s || !nx->S1r || !P_out))) return hipErrorInvalidValue;
  const int g = node_blocks(N, kNodeSplitBlocks);
  const MlpW nn = nx ? *nx : w;
#define F(L)                                                                                                       \
  if (nx)                                                                                                          \
    hipLaunchKernelGGL((k_node_enc_x3<L, true>), dim3(g), dim3(X3_NT), 0, s, N, x, w, nn, eps, h_out, P_out);      \
  else                                                                                                             \
    hipLaunchKernelGGL((k_node_enc_x3<L, false>), dim3(g), dim3(X3_NT), 0, s, N, x, w, nn, eps, h_out, P_out)
  MGN_BY_WIDTH(lat, F);
#undef F
  return hipGetLastError();
}

}  // namespace mgn
