// Edge phase of one MGN message-passing step in fp32 (Sec. 2.1: every edge
// latent is updated by the edge MLP from itself and its two end nodes, then
// each node sums the new messages of its in-edges), with one wave per
// receiver-aligned tile of at most 32 edges.  The products run as split fp16
// products on weights that stream through LDS (split32_common.hpp).
#include "launch.hpp"
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

// The tile's rows that end a segment (bit per row).  Rows of a tile are
// sorted by receiver; rcv: the lane's row's receiver.
__device__ __forceinline__ uint32_t segment_ends(int row, int n, int rcv, bool chunk) {
  const int nx = __shfl(rcv, min(row + 1, 31));
  const bool e = row < n && (row == n - 1 || (!chunk && nx != rcv));
  return (uint32_t)__ballot(e);
}

// Forward: e' = e + m (when write_e), agg = receiver sums of m, with
// m = LN(W2 relu(b1 + P_s + P_r + W1e e) + b2) (the node products P = [W1s
// h, W1r h] of the block come from the node kernels).  Two blocks per CU, so
// one block's loads, LayerNorm and barriers lie under the other's MFMAs; that
// leaves 256 registers, hence e is read again for the residual.  Rows past a
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
  const int f0 = Z::KL * hh;
  const u32x4 *W1 = (const u32x4*)w.S1, *W2 = (const u32x4*)w.S2;
  const BlockRange br = block_range(tl.n_tiles);
  if (br.tb >= br.tend) return;
  gemm_x3_start<LD>(W1, S.w, tid);
  for (int f = tid; f < LD; f += X3_NT) {
    S.vec[0][f] = w.b1[f];
    S.vec[1][f] = w.b2[f];
    S.vec[2][f] = w.gamma[f];
    S.vec[3][f] = w.beta[f];
  }
  const int lastE = (int)(tl.n_edges - 1);
  // tile t's descriptor, {0, 0, 0, 0} (no rows) past the range
  auto desc = [&](int64_t t) -> int4 {
    const bool ok = t < br.tend;
    const int4 v = tile_desc(tl.tiles, ok ? t : br.tend - 1);
    return ok ? v : make_int4(0, 0, 0, 0);
  };
  auto erow = [&](int4 d) { return min(max(d.z + min(row, tile_rows(d) - 1), 0), lastE); };
  int4 d = desc(br.tb + wv);
  int snd = tl.senders[erow(d)], rcv = tl.receivers[erow(d)];
  __syncthreads();
  for (int64_t t = br.tb; t < br.tend; t += br.stride) {
    const int4 dn = desc(t + br.stride + wv);
    const int n = tile_rows(d);
    const size_t grow = (size_t)erow(d);
    const bool chunk = d.y < 0;
    // ---- z1 = W1e e + ((b1 + P_s) + P_r), a1 = relu(z1); the gathered node
    // products are requested while the product runs
    f32x16 acc[Z::NOB];
    float x[Z::KL];
    load_row_x3<LD>(x, e_in + grow * LD + f0);
    // P_s and P_r of the features that chunk c has freed x's registers of,
    // summed one chunk later
    constexpr int Q = Z::KL / 4 / Z::NC;
    f32x4 p[Z::KL / 4], ps[Q], pr[Q];
    auto add_p = [&](int c) {
#pragma unroll
      for (int k = 0; k < Q; ++k)
        p[c * Q + k] = (*reinterpret_cast<const f32x4*>(S.vec[0] + f0 + 4 * (c * Q + k)) + ps[k]) + pr[k];
    };
    gemm_x3<LD, 0>(acc, x, W1, W2, S.w, tid, [&](int c) {
      if (c > 0) add_p(c - 1);
      const float* q = Pn + f0 + 4 * c * Q;
#pragma unroll
      for (int k = 0; k < Q; ++k) {
        ps[k] = *reinterpret_cast<const f32x4*>(q + (size_t)snd * (2 * LD) + 4 * k);
        pr[k] = *reinterpret_cast<const f32x4*>(q + (size_t)rcv * (2 * LD) + LD + 4 * k);
      }
    });
    add_p(Z::NC - 1);
#pragma unroll
    for (int c = 0; c < Z::KL / 4; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) x[4 * c + r] = relu(acc[c >> 2][4 * (c & 3) + r] + p[c][r]);
    // ---- z2 = b2 + W2 a1
    gemm_x3<LD, Z::NC & 1>(acc, x, W2, W1, S.w, tid);
#pragma unroll
    for (int c = 0; c < Z::KL / 4; ++c) {
      const f32x4 b2 = *reinterpret_cast<const f32x4*>(S.vec[1] + f0 + 4 * c);
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[c >> 2][4 * (c & 3) + r] += b2[r];
    }
    // the next tile's ids and the residual's e, in flight during the LayerNorm
    const int snd_n = tl.senders[erow(dn)], rcv_n = tl.receivers[erow(dn)];
    if (write_e) load_row_x3<LD>(x, e_in + grow * LD + f0);
    ln_x3<LD>(acc, f0, eps);
#pragma unroll
    for (int c = 0; c < Z::KL / 4; ++c) {
      const f32x4 ga = *reinterpret_cast<const f32x4*>(S.vec[2] + f0 + 4 * c);
      const f32x4 be = *reinterpret_cast<const f32x4*>(S.vec[3] + f0 + 4 * c);
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[c >> 2][4 * (c & 3) + r] = ga[r] * acc[c >> 2][4 * (c & 3) + r] + be[r];  // m
    }
    // ---- e_out = e + m
    if (write_e && row < n) {
      float* op = e_out + grow * LD + f0;
#pragma unroll
      for (int c = 0; c < Z::KL / 4; ++c) {
        f32x4 o;
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = x[4 * c + r] + acc[c >> 2][4 * (c & 3) + r];
        *reinterpret_cast<f32x4*>(op + 4 * c) = o;
      }
    }
    // ---- receiver sums, SR rows at a time
    const uint32_t ends = segment_ends(row, n, rcv, chunk);
    float2 carry[2] = {{0.f, 0.f}, {0.f, 0.f}};
    float* stage = S.stage[wv];
#pragma unroll
    for (int r0 = 0; r0 < 32; r0 += Lds::SR) {
      if (row / Lds::SR == r0 / Lds::SR)
#pragma unroll
        for (int c = 0; c < Z::KL / 4; ++c)
          *reinterpret_cast<f32x4*>(stage + (row - r0) * Lds::SL + f0 + 4 * c) =
              f32x4{acc[c >> 2][4 * (c & 3)], acc[c >> 2][4 * (c & 3) + 1], acc[c >> 2][4 * (c & 3) + 2],
                    acc[c >> 2][4 * (c & 3) + 3]};
      wave_lds_sync();
      seg_sums<LD, Lds::SL, Lds::SR>(stage, lane, ends, r0, rcv, chunk, slots + (size_t)(-1 - d.y) * LD, agg, carry);
      wave_lds_sync();
    }
    if (!chunk && d.y > d.x) zero_empty<LD>(d, tl.rowptr, lane, agg);
    d = dn;
    snd = snd_n;
    rcv = rcv_n;
  }
}

}  // namespace dev

using namespace dev;

// two blocks per CU
static constexpr int kSplitBlocks = 512;

hipError_t launch_edge_fwd_x3(int lat, const EdgeTiles& t, const void* e_in, void* e_out, int write_e, const void* Pn,
                              const MlpW& w, float eps, float* agg, float* slots, hipStream_t s) {
  if (t.n_tiles <= 0) return hipSuccess;
  if (t.n_edges <= 0 || !w.S1 || !w.S2) return hipErrorInvalidValue;
  int g = (int)std::min<int64_t>((t.n_tiles + X3_NW - 1) / X3_NW, kSplitBlocks);
  if (g >= 8) g &= ~7;
#define F(LD)                                                                                                     \
  hipLaunchKernelGGL(k_edge_fwd_x3<LD>, dim3(g), dim3(X3_NT), 0, s, t, (const float*)e_in, (float*)e_out, write_e, \
                     (const float*)Pn, w, eps, agg, slots)
  MGN_BY_WIDTH(lat, F);
#undef F
  return hipGetLastError();
}

}  // namespace mgn
