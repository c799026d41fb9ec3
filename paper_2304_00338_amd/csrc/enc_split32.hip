// Edge encoder in fp32 (Sec. 2.1: the edge features are encoded to the latent
// width by an MLP with LayerNorm), e = LN(W2 relu(W1 f + b1) + b2), on the split
// fp16 products of split32_common.hpp: one wave per 32-edge unit, two blocks per
// CU.  The first layer (K = 4) is one fma chain per feature from b1, k = 0..3, as in
// the reverse (enc_rows32.hip), which so sees the same ReLU mask.
#include "launch.hpp"
#include "split32_common.hpp"

namespace mgn {
namespace dev {

constexpr int EK = 4;  // edge input features

template <int LD>
struct __attribute__((aligned(16))) EdgeEncLds {
  u32x4 w[2][X3<LD>::CH];
  __attribute__((aligned(16))) float4 w1[LD];  // W1 by output feature
  __attribute__((aligned(16))) float vec[4][LD];  // b1, b2, gamma, beta
};

// Rows past E read row E - 1 and store nothing.  Measured per launch (fp32 MFMA
// version -> this): 434,558 edges at width 128 173 -> 85 us (writing e alone takes 47
// at the copy rate), patches of 96k to 119k edges 55 -> 27 us, 0.68M
// edges at width 160 0.39 -> 0.17 ms.
template <int LD>
__global__ void __launch_bounds__(X3_NT) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_edge_enc_x3(int64_t E, const float* __restrict__ f_in, MlpW w, float eps, float* __restrict__ e_out) {
  typedef X3<LD> Z;
  __shared__ EdgeEncLds<LD> S;
  const int tid = threadIdx.x, wv = tid >> 6;
  const u32x4* W2 = (const u32x4*)w.S2;
  const BlockRange br = block_range((E + 31) >> 5);
  if (br.tb >= br.tend) return;
  gemm_x3_start<LD>(W2, S.w, tid);
  for (int f = tid; f < LD; f += X3_NT) {
    S.w1[f] = float4{w.W1f[f * EK], w.W1f[f * EK + 1], w.W1f[f * EK + 2], w.W1f[f * EK + 3]};
    S.vec[0][f] = w.b1[f];
    S.vec[1][f] = w.b2[f];
    S.vec[2][f] = w.gamma[f];
    S.vec[3][f] = w.beta[f];
  }
  auto load = [&](int64_t t) {
    return *reinterpret_cast<const float4*>(f_in + min((t + wv) * 32 + (tid & 31), E - 1) * EK);
  };
  float4 fx = load(br.tb);
  int par = 0;
  __syncthreads();
  for (int64_t t = br.tb; t < br.tend; t += br.stride) {
    const int lane = (tid & 63) + opaque_zero(), row = lane & 31, hh = lane >> 5;
    const int64_t u = (t + wv) * 32 + row;
    const EdgeEncLds<LD>& L = fresh(S);
    f32x16 acc[Z::NOB];
    float x[Z::KL];
#pragma unroll
    for (int v = 0; v < Z::KL; ++v) {
      const float4 wr = L.w1[Z::feat(hh, v)];
      float z = L.vec[0][Z::feat(hh, v)];
      z = __builtin_fmaf(wr.x, fx.x, z);
      z = __builtin_fmaf(wr.y, fx.y, z);
      z = __builtin_fmaf(wr.z, fx.z, z);
      z = __builtin_fmaf(wr.w, fx.w, z);
      x[v] = relu32(z);
    }
    fx = load(t + br.stride);
    gemm_x3<LD>(acc, x, W2, W2, S.w, par, tid);
    par += Z::NC;
#pragma unroll
    for (int v = 0; v < Z::KL; ++v) acc[v >> 4][v & 15] += L.vec[1][Z::feat(hh, v)];
    ln_x3<LD>(acc, hh, eps);
    if (t + wv < br.tend && u < E)
      store_row_x3<LD>(e_out + (size_t)u * LD + 8 * hh, [&](int v) {
        return L.vec[2][Z::feat(hh, v)] * acc[v >> 4][v & 15] + L.vec[3][Z::feat(hh, v)];
      });
  }
}

}  // namespace dev

using namespace dev;

hipError_t launch_edge_enc_x3(int lat, int64_t E, const float* f, const MlpW& w, float eps, void* e_out,
                              hipStream_t s) {
  if (E <= 0) return hipSuccess;
  if (!w.S2) return hipErrorInvalidValue;
  const int g = unit_blocks((E + 31) / 32, X3_NW, 512);  // two blocks per CU
#define F(LD) hipLaunchKernelGGL(k_edge_enc_x3<LD>, dim3(g), dim3(X3_NT), 0, s, E, f, w, eps, (float*)e_out)
  MGN_BY_WIDTH(lat, F);
#undef F
  return hipGetLastError();
}

}  // namespace mgn
