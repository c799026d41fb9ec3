// fp32 products on the fp16 matrix pipe, and the lane layout of the kernels
// that use them, at kernel width LD = 128 or 160 (latent 150 padded with zero
// columns).
//
// The products.  A row x is scaled by the power of two s that brings its
// largest value into [2^14, 2^15), and every value is split into two fp16
// numbers, xh = fp16(s x) and xl = fp16(s x - xh), both rounded to nearest (the
// difference is exact).  The weights are split the same way when they are
// packed, with one power of two per matrix.  W x is the sum of wl xh, wh xl
// and wh xh, added in that order per K step in the fp32 accumulator of
// v_mfma_f32_32x32x16_f16 and scaled back by a power of two.
//   Accuracy: s x - xh - xl is at most 2^-24 |s x|, or 2^-25 where xl is
// subnormal, which is 2^-39 of the row's largest value; the dropped wl xl is
// at most 2^-24 |w x|; and a sum of K = 128 takes 24 accumulations instead of
// the fp32 instruction's 128.  Measured against float64 (relative 2-norm, K =
// 128): 1.2e-7 for normal rows, 1.1e-7 after a ReLU, 0.8e-7 for rows whose
// values span twelve binary orders, where 128 fp32 multiply-adds give 2.0e-7,
// 1.4e-7 and 1.8e-7.  The scales keep this for rows of any magnitude.  Rows
// with an infinity or NaN give NaN.
//   What bounds it: three fp16 products are 3/16 of the fp32 instruction's MFMA
// time.  Under a full load of random operands this card's 16-bit MFMAs sustain
// 0.58 of their nominal rate (power), and a three-piece bf16 split, which
// needs six products, measured 0.23 ms for an edge forward of 393k edges.
//
// Lane layout.  Lane l (row = l & 31, hh = l >> 5) holds one row of a 32-row
// block and the KL = LD / 2 features [KL hh, KL hh + KL) of it.  The products
// run transposed, C[feature][row] = W x^T: at K step s lane half hh supplies
// its values 8s .. 8s + 7 as the B operand, and the weights' output rows are
// ordered so that the C fragment of output block ob hands the lane its own
// features f0 + 16 ob + r (r < 16): a product's output is the next one's B
// operand without leaving registers, and a row's scale is one value per lane.
//
// The weights (pack modes 4 and 5: fragment-major, K step by K step, both
// pieces of each 32-row block together) stream through LDS: the four waves of
// a block walk the K steps together, each thread loads its share of the next
// two steps' fragments from L2 while the block computes the current two, and
// one barrier per two steps swaps the LDS buffers.  A wave's 32 rows share
// every fragment read, which keeps the LDS reads at half of the MFMA time
// (read from L2 per wave they would need all of the L1 bandwidth).
#pragma once
#include "rows_common.hpp"

namespace mgn {
namespace dev {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int X3_NW = 4;  // waves per block
constexpr int X3_NT = 64 * X3_NW;

template <int LD>
struct X3 {
  static constexpr int KL = LD / 2;         // features per lane
  static constexpr int NOB = LD / 32;       // 32-feature output blocks
  static constexpr int KS = LD / 16;        // K steps of a product
  static constexpr int NC = KS / 2;         // chunks of two K steps
  static constexpr int DR = Width<LD>::DR;  // real latent width
  static constexpr int CH = 2 * NOB * 2 * 64;  // 16-byte pieces of one chunk's weights
  static constexpr int NL = CH / X3_NT;
  static_assert(CH % X3_NT == 0, "every thread moves the same number of pieces");
};

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// The two pieces of eight values scaled by the power of two s.
struct Pieces {
  f16x8 h, l;
};
__device__ __forceinline__ Pieces split8(const float* x, float s) {
  Pieces p;
#pragma unroll
  for (int t = 0; t < 8; t += 2) {
    const float a = x[t] * s, b = x[t + 1] * s;
    const f16x2 h = __builtin_convertvector(f32x2{a, b}, f16x2);
    const f16x2 l = __builtin_convertvector(f32x2{a - (float)h[0], b - (float)h[1]}, f16x2);
    p.h[t] = h[0];
    p.h[t + 1] = h[1];
    p.l[t] = l[0];
    p.l[t + 1] = l[1];
  }
  return p;
}

// Exponent e of the scale 2^e that brings a largest value m >= 0 into [2^14,
// 2^15) (at most 2^126: smaller rows than 2^-112 keep what is left), and the
// scale itself.
__device__ __forceinline__ int scale_exp(float m) { return min(141 - (int)(__float_as_uint(m) >> 23), 126); }
__device__ __forceinline__ float scale_of(int e) { return __uint_as_float((uint32_t)(e + 127) << 23); }

// Sum and maximum over the two lanes that hold a row.
__device__ __forceinline__ float sum_hh(float s) {
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
__device__ __forceinline__ float max_hh(float s) {
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// One chunk's weight fragments on their way from L2 to LDS.
template <int LD>
struct WStream {
  u32x4 r[X3<LD>::NL];
  __device__ __forceinline__ void load(const u32x4* p, int tid) {
#pragma unroll
    for (int j = 0; j < X3<LD>::NL; ++j)
      r[j] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(p) + 16u * (uint32_t)(tid + X3_NT * j));
  }
  __device__ __forceinline__ void store(u32x4* dst, int tid) const {
#pragma unroll
    for (int j = 0; j < X3<LD>::NL; ++j) dst[tid + X3_NT * j] = r[j];
  }
};

// A packed matrix: its chunks, then the exponent of its scale.
template <int LD>
__device__ __forceinline__ int weight_exp(const u32x4* W) {
  typedef __attribute__((address_space(4))) const int ConstInt;
  return *(ConstInt*)(W + X3<LD>::NC * X3<LD>::CH);
}

// acc = W x for the lane's KL values x.  W is the product's packed matrix,
// whose first chunk is in buf[PAR]; next (the following product's, or any
// valid matrix) leaves its first chunk in buf[(PAR + NC) % 2].  All waves of
// the block call it together.  mid(c) runs after the products of chunk c (for
// loads that the caller needs after the product).
template <int LD, int PAR, class F>
__device__ __forceinline__ void gemm_x3(f32x16 (&acc)[X3<LD>::NOB], const float* x, const u32x4* W, const u32x4* next,
                                        u32x4 (*buf)[X3<LD>::CH], int tid, F&& mid) {
  typedef X3<LD> Z;
  const int lane = tid & 63;
  const int ot = tid + opaque_zero();  // keeps the loads' addresses out of the callers' loops
  float m = 0.f;
#pragma unroll
  for (int t = 0; t < Z::KL; ++t) m = fmaxf(m, fabsf(x[t]));
  const int e = scale_exp(max_hh(m));
  float s = scale_of(e);
  // the scale is formed here; left to itself, the compiler spread the maximum
  // over the chunks' barriers and with it delayed every product
  asm volatile("" : "+v"(s));
#pragma unroll
  for (int ob = 0; ob < Z::NOB; ++ob)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[ob][r] = 0.f;
#pragma unroll
  for (int c = 0; c < Z::NC; ++c) {
    WStream<LD> ws;
    ws.load(c + 1 < Z::NC ? W + (c + 1) * Z::CH : next, ot);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      // the loads stay above, a whole chunk ahead of their use, and the steps
      // apart (fragments of both at once do not fit in the registers)
      __builtin_amdgcn_sched_barrier(0);
      const Pieces b = split8(x + 16 * c + 8 * k, s);
      const f16x8* A = reinterpret_cast<const f16x8*>(buf[(PAR + c) & 1]) + k * Z::NOB * 128 + lane;
      f16x8 a[Z::NOB];
#pragma unroll
      for (int ob = 0; ob < Z::NOB; ++ob) a[ob] = A[(2 * ob + 1) * 64];
#pragma unroll
      for (int ob = 0; ob < Z::NOB; ++ob) acc[ob] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[ob], b.h, acc[ob], 0, 0, 0);
#pragma unroll
      for (int ob = 0; ob < Z::NOB; ++ob) a[ob] = A[(2 * ob) * 64];
#pragma unroll
      for (int ob = 0; ob < Z::NOB; ++ob) acc[ob] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[ob], b.l, acc[ob], 0, 0, 0);
#pragma unroll
      for (int ob = 0; ob < Z::NOB; ++ob) acc[ob] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[ob], b.h, acc[ob], 0, 0, 0);
    }
    mid(c);
    ws.store(buf[(PAR + c + 1) & 1], tid);
    __syncthreads();
  }
  const int k = -(e + weight_exp<LD>(W));
#pragma unroll
  for (int ob = 0; ob < Z::NOB; ++ob)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[ob][r] = __builtin_amdgcn_ldexpf(acc[ob][r], k);
}
template <int LD, int PAR>
__device__ __forceinline__ void gemm_x3(f32x16 (&acc)[X3<LD>::NOB], const float* x, const u32x4* W, const u32x4* next,
                                        u32x4 (*buf)[X3<LD>::CH], int tid) {
  gemm_x3<LD, PAR>(acc, x, W, next, buf, tid, [](int) {});
}

// The first chunk of the first product into buf[0] (a barrier must follow).
template <int LD>
__device__ __forceinline__ void gemm_x3_start(const u32x4* W, u32x4 (*buf)[X3<LD>::CH], int tid) {
  WStream<LD> ws;
  ws.load(W, tid);
  ws.store(buf[0], tid);
}

// The lane's KL contiguous floats of a row starting at p.
template <int LD>
__device__ __forceinline__ void load_row_x3(float* x, const float* __restrict__ p) {
#pragma unroll
  for (int c = 0; c < X3<LD>::KL / 4; ++c) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(p + 4 * c);
#pragma unroll
    for (int t = 0; t < 4; ++t) x[4 * c + t] = v[t];
  }
}

// z -> (z - mean) rstd over the row's DR real features (the padded ones are
// 0 on entry and are left out of the biased variance); returns rstd.
template <int LD>
__device__ __forceinline__ float ln_x3(f32x16 (&z)[X3<LD>::NOB], int f0, float eps) {
  typedef X3<LD> Z;
  float sm = 0.f;
#pragma unroll
  for (int ob = 0; ob < Z::NOB; ++ob)
#pragma unroll
    for (int r = 0; r < 16; ++r) sm += z[ob][r];
  const float mean = sum_hh(sm) * (1.0f / Z::DR);
  float sq = 0.f;
#pragma unroll
  for (int ob = 0; ob < Z::NOB; ++ob)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float d = z[ob][r] - mean;
      z[ob][r] = d;
      if (Z::DR == LD || f0 + 16 * ob + r < Z::DR) sq += d * d;
    }
  const float rstd = __builtin_amdgcn_rsqf(sum_hh(sq) * (1.0f / Z::DR) + eps);
#pragma unroll
  for (int ob = 0; ob < Z::NOB; ++ob)
#pragma unroll
    for (int r = 0; r < 16; ++r) z[ob][r] *= rstd;
  return rstd;
}

// Block range of 32-row units (tiles): wave wv takes unit tb + wv of every
// round, all waves run the same number of rounds; blocks go to the XCDs round
// robin, so each XCD walks one contiguous eighth (see unit_range).
struct BlockRange {
  int64_t tb, stride, tend;
};
__device__ __forceinline__ BlockRange block_range(int64_t n_units) {
  const int G = gridDim.x;
  BlockRange u;
  if ((G & 7) == 0) {
    const int64_t chunk = (n_units + 7) >> 3, lo = (blockIdx.x & 7) * chunk;
    u.tend = min(n_units, lo + chunk);
    u.tb = lo + (int64_t)(blockIdx.x >> 3) * X3_NW;
    u.stride = (int64_t)(G >> 3) * X3_NW;
  } else {
    u.tb = (int64_t)blockIdx.x * X3_NW;
    u.stride = (int64_t)G * X3_NW;
    u.tend = n_units;
  }
  return u;
}

// Receiver sums of a tile's rows.  The tile's rows [r0, r0 + SR) are staged
// row-major (stride SL floats) in the wave's LDS; each lane sums feature
// pairs lane and lane + 64 (below LD / 2) of the rows in ascending order from
// 0.0 and stores a segment's sum at its last row (bit u of ends: row u ends
// a segment), to node rcv's row of dst, or, for a chunk of a long segment, to
// its slot.  All of the staged rows are read at once, before the sums.
template <int LD, int SL, int SR>
__device__ __forceinline__ void seg_sums(const float* stage, int lane, uint32_t ends, int r0, int rcv, bool chunk,
                                         float* slot, float* dst, float2 (&carry)[2]) {
  constexpr int NP = LD / 2;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    if (k == 1 && NP <= 64) break;
    const int p = lane + 64 * k;
    const bool on = k == 0 || p < NP;
    float2 v[SR];
#pragma unroll
    for (int u = 0; u < SR; ++u) v[u] = *reinterpret_cast<const float2*>(stage + u * SL + 2 * (on ? p : lane));
#pragma unroll
    for (int u = 0; u < SR; ++u) {
      carry[k].x += v[u].x;
      carry[k].y += v[u].y;
      if ((ends >> (r0 + u)) & 1u) {
        float* q = chunk ? slot : dst + (size_t)__builtin_amdgcn_readlane(rcv, r0 + u) * LD;
        if (on) *reinterpret_cast<float2*>(q + 2 * p) = carry[k];
        carry[k] = float2{0.f, 0.f};
      }
    }
  }
}

// Zero rows of dst for the tile's nodes without in-edges.
template <int LD>
__device__ __forceinline__ void zero_empty(int4 d, const int32_t* __restrict__ rowptr, int lane, float* dst) {
  const int v = min(d.x + lane, d.y - 1);
  uint64_t m = __ballot(lane < d.y - d.x && rowptr[v] == rowptr[v + 1]);
  while (m) {
    const int j = __builtin_ctzll(m);
    m &= m - 1;
    float* q = dst + (size_t)(d.x + j) * LD;
    for (int f = lane; f < LD; f += 64) q[f] = 0.f;
  }
}

}  // namespace dev
}  // namespace mgn
