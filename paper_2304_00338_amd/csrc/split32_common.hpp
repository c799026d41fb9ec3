// fp32 products on the fp16 matrix pipe, and the lane layout of the kernels
// that use them, at kernel width LD = 128 or 160 (latent 150 padded with zero
// columns).
//
// The products.  A row x is scaled by the power of two s that brings its
// largest value into [2^14, 2^15), and every value is split into two fp16
// numbers, xh = fp16(s x) and xl = fp16(s x - xh), both rounded to nearest (the
// difference is exact).  The weights are split the same way when they are
// packed, with one power of two per matrix, wl times 2^12 so that it stays normal longer.
// W x is the sum of (2^12 wl) (2^-12 xh), wh xl and wh xh, added in that order per K
// step in the fp32 accumulator of v_mfma_f32_32x32x16_f16 and scaled back by
// a power of two.
//   Accuracy: two pieces hold 22 to 23 bits of a value.  xh + xl is within 2^-23 |s x| of s x (and within
// 2^-25 where xl is subnormal, which is 2^-39 of the row's largest value); a
// weight is held within 2^-23 of itself and 2^-51 of the matrix's largest;
// the dropped wl xl is at most 2^-22 |w x|; and a sum of K = 128 takes 24
// accumulations instead of the fp32 instruction's 128.  Measured against
// float64 (relative 2-norm, K = 128): 1.2e-7 for normal rows, 1.1e-7 after a
// ReLU, 0.8e-7 for rows whose values span twelve binary orders, where 128 fp32
// multiply-adds give 2.0e-7, 1.4e-7 and 1.8e-7.  The scales keep this for rows and
// matrices of any magnitude, and for weights down to 2^-28 of their matrix's largest (one
// scale per matrix without the 2^12: 3e-6 at 2^-20, 5e-4 at 2^-28).  Within a row it holds down to about
// 2^-16 of the largest value: a smaller one loses a bit per factor of two,
// which shows where the larger ones meet weights as much smaller, or zeros.  (A separate
// power of two per row of W, applied to the result where any row has one, cost more: edge
// forward at 434,558 edges 189 -> 232 us, in spilled registers.)  Rows with an
// infinity or NaN give NaN.
//   What bounds it: three fp16 products are 3/16 of the fp32 instruction's MFMA
// time.  Under a full load of random operands this card's 16-bit MFMAs sustain
// 0.58 of their nominal rate (power), and a three-piece bf16 split, which
// needs six products, measured 0.23 ms for an edge forward of 393k edges.
//
// Lane layout.  Lane l (row = l & 31, hh = l >> 5) holds one row of a 32-row
// block and KL = LD / 2 values of it, value v being feature 16 (v / 8) + 8 hh +
// v % 8: the two lanes of a row read or write 64 contiguous bytes in two
// instructions.  (Every 16-byte access of a wave still spans 32 cache lines,
// and the L1 takes one a cycle: with a contiguous half row per lane it was 64,
// and the address traffic of an edge forward took as long as its arithmetic.)
// The products run transposed, C[feature][row] = W x^T: at K step s lane half
// hh supplies its values 8s .. 8s + 7 as the B operand, and the weights' output
// rows are ordered so that the C fragment of output block ob hands the lane
// its own values 16 ob + r (r < 16): a product's output is the next one's B
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
#include "w160_common.hpp"

namespace mgn {
namespace dev {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int X3_NW = 4;  // waves per block (unless a kernel says otherwise)
constexpr int X3_NT = 64 * X3_NW;

template <int LD>
struct X3 {
  static constexpr int KL = LD / 2;         // features per lane
  static constexpr int NOB = LD / 32;       // 32-feature output blocks
  static constexpr int KS = LD / 16;        // K steps of a product
  static constexpr int NC = KS / 2;         // chunks of two K steps
  static constexpr int DR = Width<LD>::DR;  // real latent width
  static constexpr int CH = 2 * NOB * 2 * 64;  // 16-byte pieces of one chunk's weights
  // feature of value v of lane half hh; pf(c): the part that four values c of
  // any half share (feature of value 4c minus 8 hh)
  static constexpr __host__ __device__ int feat(int hh, int v) { return 16 * (v >> 3) + 8 * hh + (v & 7); }
  static constexpr __host__ __device__ int pf(int c) { return 16 * (c >> 1) + 4 * (c & 1); }
};

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// The two pieces of eight values scaled by 2^e.
struct Pieces {
  f16x8 h, l;
};
__device__ __forceinline__ Pieces split8(const float* x, int e) {
  Pieces p;
#pragma unroll
  for (int t = 0; t < 8; t += 2) {
    const float a = __builtin_amdgcn_ldexpf(x[t], e), b = __builtin_amdgcn_ldexpf(x[t + 1], e);
    const f16x2 h = __builtin_convertvector(f32x2{a, b}, f16x2);
    const f16x2 l = __builtin_convertvector(f32x2{a - (float)h[0], b - (float)h[1]}, f16x2);
    p.h[t] = h[0];
    p.h[t + 1] = h[1];
    p.l[t] = l[0];
    p.l[t + 1] = l[1];
  }
  return p;
}

// Eight fp16 values times s.
__device__ __forceinline__ f16x8 scale_f16(f16x8 v, _Float16 s) {
  return v * f16x8{s, s, s, s, s, s, s, s};
}

// The weights' low pieces are packed times 2^kLowExp and meet xh times 2^-kLowExp:
// a low piece is at most 2^3, so this is the largest factor that fits.
constexpr int kLowExp = 12;

// Exponent e of the scale 2^e that brings a largest value m >= 0 into [2^14,
// 2^15) (at most 2^126: smaller rows than 2^-112 keep what is left); kZeroExp
// for 0, kInfExp for an infinity.
constexpr int kZeroExp = 4096, kInfExp = 141 - 255;
__device__ __forceinline__ int scale_exp(float m) {
  return m == 0.f ? kZeroExp : min(141 - (int)(__float_as_uint(m) >> 23), 126);
}

// Sum and maximum over the two lanes that hold a row.
__device__ __forceinline__ float sum_hh(float s) {
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
__device__ __forceinline__ float max_hh(float s) {
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// One chunk's weight fragments on their way from L2 to LDS: each of the NT
// threads moves the same number of pieces.
template <int LD, int NT>
struct WStream {
  static constexpr int NL = X3<LD>::CH / NT;
  static_assert(X3<LD>::CH % NT == 0, "");
  u32x4 r[NL];
  __device__ __forceinline__ void load(const u32x4* p, int tid) {
#pragma unroll
    for (int j = 0; j < NL; ++j)
      r[j] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(p) + 16u * (uint32_t)(tid + NT * j));
  }
  __device__ __forceinline__ void store(u32x4* dst, int tid) const {
#pragma unroll
    for (int j = 0; j < NL; ++j) dst[tid + NT * j] = r[j];
  }
};

// A packed matrix: its chunks, then the exponent of its scale.
template <int LD>
__device__ __forceinline__ int weight_exp(const u32x4* W) {
  typedef __attribute__((address_space(4))) const int ConstInt;
  return *(ConstInt*)(W + X3<LD>::NC * X3<LD>::CH);
}

// Exponent of the lane's row's scale (scale_exp of its largest value).  The
// result is pinned where it is formed: left to itself, the compiler spread the
// maximum over the following product's barriers and with it delayed every
// MFMA.
template <int LD>
__device__ __forceinline__ int row_exp(const float* x) {
  float m = 0.f;
#pragma unroll
  for (int t = 0; t < X3<LD>::KL; ++t) m = fmaxf(m, fabsf(x[t]));
  int e = scale_exp(max_hh(m));
  asm volatile("" : "+v"(e));
  return e;
}

// A row's pieces and its scale's exponent.
template <int LD>
struct RowPieces {
  Pieces p[X3<LD>::KS];
  int e;
};

// acc (+)= 2^(e + W's exponent) W x, where get(ks) gives the pieces of the
// lane's values 8 ks .. 8 ks + 7 scaled by 2^e; ADD keeps what acc holds.  W is the product's packed matrix, whose first chunk is in
// buf[par & 1]; next (the following product's, or any valid matrix) leaves its
// first chunk in buf[(par + NC) & 1].  All NT threads of the block call it
// together.  mid(ks) runs after the products of K step ks (for loads that
// the caller needs after the product).
template <int LD, int NT, bool ADD, class G, class F>
__device__ __forceinline__ void gemm_raw(f32x16 (&acc)[X3<LD>::NOB], G&& get, const u32x4* W, const u32x4* next,
                                         u32x4 (*buf)[X3<LD>::CH], int par, int tid, F&& mid) {
  typedef X3<LD> Z;
  const int lane = tid & 63;
  const int ot = tid + opaque_zero();  // keeps the loads' addresses out of the callers' loops
  // 2^-kLowExp as two fp16; opaque, or a second product of the same row would keep the scaled pieces
  int low = (15 - kLowExp) << 10 | (15 - kLowExp) << 26;
  asm volatile("" : "+s"(low));
  if (!ADD)
#pragma unroll
  for (int ob = 0; ob < Z::NOB; ++ob)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[ob][r] = 0.f;
#pragma unroll
  for (int c = 0; c < Z::NC; ++c) {
    WStream<LD, NT> ws;
    ws.load(c + 1 < Z::NC ? W + (c + 1) * Z::CH : next, ot);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      // the loads stay above, a whole chunk ahead of their use, and the steps
      // apart (fragments of both at once do not fit in the registers)
      __builtin_amdgcn_sched_barrier(0);
      const Pieces b = get(2 * c + k);
      const f16x8 bs = scale_f16(b.h, __builtin_bit_cast(f16x2, low)[0]);
      const f16x8* A = reinterpret_cast<const f16x8*>(buf[(par + c) & 1]) + k * Z::NOB * 128 + lane;
      f16x8 a[Z::NOB];
#pragma unroll
      for (int ob = 0; ob < Z::NOB; ++ob) a[ob] = A[(2 * ob + 1) * 64];
#pragma unroll
      for (int ob = 0; ob < Z::NOB; ++ob) acc[ob] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[ob], bs, acc[ob], 0, 0, 0);
#pragma unroll
      for (int ob = 0; ob < Z::NOB; ++ob) a[ob] = A[(2 * ob) * 64];
#pragma unroll
      for (int ob = 0; ob < Z::NOB; ++ob) acc[ob] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[ob], b.l, acc[ob], 0, 0, 0);
#pragma unroll
      for (int ob = 0; ob < Z::NOB; ++ob) acc[ob] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[ob], b.h, acc[ob], 0, 0, 0);
      mid(2 * c + k);
    }
    ws.store(buf[(par + c + 1) & 1], tid);
    __syncthreads();
  }
}

// acc *= 2^k
template <int LD>
__device__ __forceinline__ void scale_acc(f32x16 (&acc)[X3<LD>::NOB], int k) {
#pragma unroll
  for (int ob = 0; ob < X3<LD>::NOB; ++ob)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[ob][r] = __builtin_amdgcn_ldexpf(acc[ob][r], k);
}

// acc = W x from the row's pieces.
template <int LD, int NT, class G, class F>
__device__ __forceinline__ void gemm_pieces(f32x16 (&acc)[X3<LD>::NOB], G&& get, int e, const u32x4* W,
                                            const u32x4* next, u32x4 (*buf)[X3<LD>::CH], int par, int tid, F&& mid) {
  gemm_raw<LD, NT, false>(acc, get, W, next, buf, par, tid, mid);
  scale_acc<LD>(acc, -(e + weight_exp<LD>(W)));
}

// acc = W x for the lane's KL values x, which are split as the product goes.
template <int LD, int NT = X3_NT, class F>
__device__ __forceinline__ void gemm_x3(f32x16 (&acc)[X3<LD>::NOB], const float* x, const u32x4* W, const u32x4* next,
                                        u32x4 (*buf)[X3<LD>::CH], int par, int tid, F&& mid) {
  const int e = row_exp<LD>(x);
  gemm_pieces<LD, NT>(acc, [&](int ks) { return split8(x + 8 * ks, e); }, e, W, next, buf, par, tid, mid);
}
template <int LD, int NT = X3_NT>
__device__ __forceinline__ void gemm_x3(f32x16 (&acc)[X3<LD>::NOB], const float* x, const u32x4* W, const u32x4* next,
                                        u32x4 (*buf)[X3<LD>::CH], int par, int tid) {
  gemm_x3<LD, NT>(acc, x, W, next, buf, par, tid, [](int) {});
}
// The same, keeping the pieces in row.
template <int LD, int NT, class F>
__device__ __forceinline__ void gemm_keep(f32x16 (&acc)[X3<LD>::NOB], const float* x, RowPieces<LD>& row, const u32x4* W,
                                          const u32x4* next, u32x4 (*buf)[X3<LD>::CH], int par, int tid, F&& mid) {
  row.e = row_exp<LD>(x);
  gemm_pieces<LD, NT>(acc, [&](int ks) { return row.p[ks] = split8(x + 8 * ks, row.e); }, row.e, W, next, buf, par, tid, mid);
}

// The first chunk of the first product into buf[0] (a barrier must follow).
template <int LD, int NT = X3_NT>
__device__ __forceinline__ void gemm_x3_start(const u32x4* W, u32x4 (*buf)[X3<LD>::CH], int tid) {
  WStream<LD, NT> ws;
  ws.load(W, tid);
  ws.store(buf[0], tid);
}

// Rows of a tile in an [E][LD] stream: the tile's first row as a scalar base
// and the lane's own slice as a 32-bit offset from it.  Rows past the tile's
// end are clamped to its last one (an empty tile reads a valid row).
template <int LD>
struct TileRow {
  int64_t base;
  uint32_t off;
  __device__ __forceinline__ TileRow(int4 d, int64_t last, int row, int hh) {
    base = min((int64_t)d.z, last) * LD;
    off = (uint32_t)(max(min(row, tile_rows(d) - 1), 0) * LD + 8 * hh);
  }
  template <class T>
  __device__ __forceinline__ T* at(T* p) const {
    return p + base + off;
  }
};

// The lane's KL values of a row; p points at feature 8 hh of it.
template <int LD>
__device__ __forceinline__ void load_row_x3(float* x, const float* __restrict__ p) {
#pragma unroll
  for (int c = 0; c < X3<LD>::KL / 4; ++c) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(p + X3<LD>::pf(c));
#pragma unroll
    for (int t = 0; t < 4; ++t) x[4 * c + t] = v[t];
  }
}

// z -> (z - mean) rstd over the row's DR real features (the padded ones are
// 0 on entry and are left out of the biased variance); returns rstd.
template <int LD>
__device__ __forceinline__ float ln_x3(f32x16 (&z)[X3<LD>::NOB], int hh, float eps) {
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
      if (Z::DR == LD || Z::feat(hh, 16 * ob + r) < Z::DR) sq += d * d;
    }
  const float rstd = __builtin_amdgcn_rsqf(sum_hh(sq) * (1.0f / Z::DR) + eps);
#pragma unroll
  for (int ob = 0; ob < Z::NOB; ++ob)
#pragma unroll
    for (int r = 0; r < 16; ++r) z[ob][r] *= rstd;
  return rstd;
}

// Block range of 32-row units (tiles): see block_units.
template <int NW = X3_NW>
__device__ __forceinline__ BlockRange block_range(int64_t n_units) {
  return block_units(n_units, gridDim.x, blockIdx.x, NW);
}

// Receiver sums of a tile's rows.  The tile's rows [r0, r0 + SR) are staged
// row-major (stride SL floats) in the wave's LDS; each lane sums feature
// pairs lane and lane + 64 (below LD / 2) of the rows in ascending order from
// 0.0 and stores a segment's sum at its last row (bit u of ends: row u ends
// a segment), to node rcv's row of dst, or, for a chunk of a long segment, to
// its slot, and adds it to tot.  All of the staged rows are read at once, before
// the sums; rows(v, p, on) sees them first (v[u]: the pair p of row r0 + u).
template <int LD, int SL, int SR, class F>
__device__ __forceinline__ void seg_sums(const float* stage, int lane, uint32_t ends, int r0, int rcv, bool chunk,
                                         float* slot, float* dst, float2 (&carry)[2], float2 (&tot)[2], F&& rows) {
  constexpr int NP = LD / 2;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    if (k == 1 && NP <= 64) break;
    const int p = lane + 64 * k;
    const bool on = k == 0 || p < NP;
    float2 v[SR];
#pragma unroll
    for (int u = 0; u < SR; ++u) v[u] = *reinterpret_cast<const float2*>(stage + u * SL + 2 * (on ? p : lane));
    rows(v, p, on);
#pragma unroll
    for (int u = 0; u < SR; ++u) {
      carry[k].x += v[u].x;
      carry[k].y += v[u].y;
      if ((ends >> (r0 + u)) & 1u) {
        float* q = chunk ? slot : dst + (size_t)__builtin_amdgcn_readlane(rcv, r0 + u) * LD;
        if (on) *reinterpret_cast<float2*>(q + 2 * p) = carry[k];
        tot[k].x += carry[k].x;
        tot[k].y += carry[k].y;
        carry[k] = float2{0.f, 0.f};
      }
    }
  }
}

// Stores the lane's KL values of a row; p points at feature 8 hh of it.
template <int LD, class F>
__device__ __forceinline__ void store_row_x3(float* p, F&& get) {
#pragma unroll
  for (int c = 0; c < X3<LD>::KL / 4; ++c)
    *reinterpret_cast<f32x4*>(p + X3<LD>::pf(c)) = f32x4{get(4 * c), get(4 * c + 1), get(4 * c + 2), get(4 * c + 3)};
}

// Column sums over the 32 rows of a block of the lanes' KL values, added up
// block after block: a permlane16 swap and then DPP butterflies halve the
// values held at every step, which leaves lane i + 16 k of half hh with the
// features KL hh + (KL / 2) k + 2i + {0, 1} (v) and, at width 160, one more for
// even i (t).  put() writes a wave's sums into its row of an LDS array [LD].
template <int LD>
struct ColSumX3 {
  static constexpr int H = X3<LD>::KL / 2;
  float2 v = {0.f, 0.f};
  float t = 0.f;
  // get(k): the lane's value k.  The first two halvings run value by value, so
  // that few are held at a time.
  template <class F>
  __device__ __forceinline__ void add(F&& get, int i) {
    auto pair = [&](int k) {
      const auto w = __builtin_amdgcn_permlane16_swap(__float_as_uint(get(k)), __float_as_uint(get(k + H)), false, false);
      return __uint_as_float(w[0]) + __uint_as_float(w[1]);
    };
    float c[16];
    const bool hi = (i >> 3) & 1;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const float a = pair(k), b = pair(k + 16);
      c[k] = (hi ? b : a) + dpp_mov<0x140>(hi ? a : b);
    }
    bfly_step<8, 0x141>(c, (i >> 2) & 1);
    bfly_step<4, 0x1B>(c, (i >> 1) & 1);
    bfly_step<2, 0xB1>(c, i & 1);
    v.x += c[0];
    v.y += c[1];
    if constexpr (H == 40) {
      f32x4 q[10];
#pragma unroll
      for (int k = 0; k < 8; ++k) q[8 + (k >> 2)][k & 3] = pair(32 + k);
      t += w160::colsum16_tail(q, i);
    }
  }
  __device__ __forceinline__ void put(float* red, int lane) const {
    const int i = lane & 15, hh = lane >> 5, k = H * ((lane >> 4) & 1);
    *reinterpret_cast<float2*>(red + X3<LD>::feat(hh, k + 2 * i)) = v;
    if constexpr (H == 40)
      if ((i & 1) == 0)
        red[X3<LD>::feat(hh, k + 32 + ((((i >> 3) & 1) << 2) | (((i >> 2) & 1) << 1) | ((i >> 1) & 1)))] = t;
  }
};

// Weight gradients dW[o][n] += sum over rows of G[row][o] X[row][n], with the
// rows as K, from the rows' pieces.  A row of G carries its own power of two
// 2^eg and the row of X its 2^ex; the pieces are scaled further, by 2^(c - eg -
// ex) <= 1 in all, so that every product carries 2^c, as the accumulators do.
//   c follows the rows: it is lowered to the smallest eg + ex of the NW x 32
// rows that are added together, and raised where that lies more than kDwRise
// above it (at most kDwSpan above its lowest value, so that no sum overflows).
// What a piece has below 2^-24 is lost, so rows that need much scaling lose low bits:
// with half of it in each operand, a row whose products are 2^-30 of 2^c's largest
// stays within 2^-24 of its own largest value, one of 2^-40 within 2^-19, and from 2^-50
// (add) or 2^-78 (add_rows) on they vanish.  (Adding such rows in further passes at their own c keeps all bits.
// Measured on the eight-patch batch, whose ghost nodes' gradients span 2^48
// within those rows: reverse 1.28 -> 1.41 to 1.56 ms a launch, 0.68M edges; and at width 128 a
// pass that is never taken still costs 3% in spilled registers.)  Rows of zeros, and
// rows with an infinity (which become NaN), do not bound c and are not scaled.
//   Each of the NW waves holds 32 rows (lane layout as above) and owns TU x TV
// of the 16 x 16 tiles of dW.  The rows are staged row-major, SR rows at a time
// (SR / NW of every wave), and read back transposed.  Rows that are not live
// must have zero pieces in G.
constexpr int kDwRise = 12, kDwSpan = 70;
template <int LD, int NW>
struct DwShape {
  static constexpr int SL = LD + 16;                 // staged row stride (fp16)
  static constexpr int SR = NW == 8 ? 64 : 32;       // rows staged at a time
  static constexpr int TU = NW == 8 ? LD / 64 : LD / 32, TV = LD / 32;
  static_assert(TU * TV * NW * 256 == LD * LD, "");
};
template <int LD, int NW>
struct __attribute__((aligned(16))) DwLds {
  _Float16 g[2][DwShape<LD, NW>::SR * DwShape<LD, NW>::SL];
  _Float16 x[2][DwShape<LD, NW>::SR * DwShape<LD, NW>::SL];
  int c[NW];
};

// Smallest value over the 32 rows of a wave.
__device__ __forceinline__ int min_rows(int m) {
  m = min(m, __builtin_amdgcn_mov_dpp(m, 0x140, 0xf, 0xf, false));
  m = min(m, __builtin_amdgcn_mov_dpp(m, 0x141, 0xf, 0xf, false));
  m = min(m, __builtin_amdgcn_mov_dpp(m, 0x1B, 0xf, 0xf, false));
  m = min(m, __builtin_amdgcn_mov_dpp(m, 0xB1, 0xf, 0xf, false));
  const auto w = __builtin_amdgcn_permlane16_swap((uint32_t)m, (uint32_t)m, false, false);
  return min((int)w[0], (int)w[1]);
}

template <int LD, int NW>
struct DwAcc {
  typedef DwShape<LD, NW> Sh;
  static constexpr int TU = Sh::TU, TV = Sh::TV;
  static constexpr int NONE = 1 << 20;
  f32x4 a[TU * TV];
  int c = NONE, cmin = NONE;  // no rows yet
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int t = 0; t < TU * TV; ++t) a[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  static __device__ __forceinline__ f16x8 frag(const _Float16* S, int r0, int col0, int i, int q) {
    const bf16* p = reinterpret_cast<const bf16*>(S) + (r0 + q * 8 + (i >> 2)) * Sh::SL + col0 + 4 * (i & 3);
    return __builtin_bit_cast(f16x8, cat8(lds_tr(p), lds_tr(p + 4 * Sh::SL)));
  }
  // Brings c to the block's rows (er: the row's eg + ex, NONE where it does not
  // bound c) and returns the exponent that the row's product lacks to it.
  __device__ __forceinline__ int fit(int er, DwLds<LD, NW>& S, int tid) {
    const int m = min_rows(er);
    if ((tid & 63) == 0) S.c[tid >> 6] = m;
    __syncthreads();  // also: the products of the previous call are done
    int cn = S.c[0];
#pragma unroll
    for (int k = 1; k < NW; ++k) cn = min(cn, S.c[k]);
    cn = __builtin_amdgcn_readfirstlane(cn);
    if (cn < c || (cn > c + kDwRise && cn != NONE)) {
      cn = min(cn, cmin + kDwSpan);
#pragma unroll
      for (int t = 0; t < TU * TV; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) a[t][r] = __builtin_amdgcn_ldexpf(a[t][r], cn - c);
      c = cn;
      cmin = min(cmin, c);
    }
    return er == NONE ? 0 : c - er;
  }
  static __device__ __forceinline__ int bound(int eg, int ex, bool live) {
    return live && max(eg, ex) < kZeroExp && min(eg, ex) > kInfExp ? eg + ex : NONE;
  }
  // The products of the rows that stage(at) writes to S at offset at of its arrays.
  template <class F>
  __device__ __forceinline__ void products(DwLds<LD, NW>& S, int tid, F&& stage) {
    constexpr int RW = Sh::SR / NW;  // rows of a wave staged at a time
    const int lane = tid & 63, row = lane & 31, hh = lane >> 5, wv = tid >> 6, i = lane & 15, q = lane >> 4;
    const int at = (RW * wv + row % RW) * Sh::SL + 8 * hh;
    const int u0 = 16 * TU * (wv / (LD / 16 / TV)), v0 = 16 * TV * (wv % (LD / 16 / TV));
#pragma unroll 1
    for (int r = 0; r < 32 / RW; ++r) {
      if (r > 0) __syncthreads();  // the previous rows' products are done
      if (row / RW == r) stage(at);
      __syncthreads();
#pragma unroll
      for (int r0 = 0; r0 < Sh::SR; r0 += 32) {
        f16x8 ah[TU], al[TU];
#pragma unroll
        for (int u = 0; u < TU; ++u) {
          ah[u] = frag(S.g[0], r0, u0 + 16 * u, i, q);
          al[u] = frag(S.g[1], r0, u0 + 16 * u, i, q);
        }
#pragma unroll
        for (int v = 0; v < TV; ++v) {
          const f16x8 bh = frag(S.x[0], r0, v0 + 16 * v, i, q);
          const f16x8 bl = frag(S.x[1], r0, v0 + 16 * v, i, q);
#pragma unroll
          for (int u = 0; u < TU; ++u) a[u * TV + v] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al[u], bh, a[u * TV + v], 0, 0, 0);
#pragma unroll
          for (int u = 0; u < TU; ++u) a[u * TV + v] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[u], bl, a[u * TV + v], 0, 0, 0);
#pragma unroll
          for (int u = 0; u < TU; ++u) a[u * TV + v] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[u], bh, a[u * TV + v], 0, 0, 0);
        }
      }
    }
  }
  // From the pieces of a product's rows (X's are used up).
  __device__ __forceinline__ void add(const RowPieces<LD>& G, RowPieces<LD>& X, bool live, DwLds<LD, NW>& S, int tid) {
    // down to 2^-12 all of it in X, so that G's pieces seldom need it
    const int k = fit(bound(G.e, X.e, live), S, tid), kx = k < -12 ? k / 2 : k;
    const bool plain = !__any(k != kx);
    const _Float16 sx = (_Float16)__builtin_amdgcn_ldexpf(1.f, kx);
    float sg = __builtin_amdgcn_ldexpf(1.f, k - kx);
#pragma unroll
    for (int u = 0; u < X3<LD>::KS; ++u) {
      X.p[u].h = scale_f16(X.p[u].h, sx);
      X.p[u].l = scale_f16(X.p[u].l, sx);
    }
    products(S, tid, [&](int at) {
      if (plain) {
#pragma unroll
        for (int u = 0; u < X3<LD>::KS; ++u) {
          *reinterpret_cast<f16x8*>(S.g[0] + at + 16 * u) = G.p[u].h;
          *reinterpret_cast<f16x8*>(S.g[1] + at + 16 * u) = G.p[u].l;
        }
      } else {
        asm volatile("" : "+v"(sg));  // scaled here: all of the scaled pieces do not fit beside the others
#pragma unroll
        for (int u = 0; u < X3<LD>::KS; ++u) {
          *reinterpret_cast<f16x8*>(S.g[0] + at + 16 * u) = scale_f16(G.p[u].h, (_Float16)sg);
          *reinterpret_cast<f16x8*>(S.g[1] + at + 16 * u) = scale_f16(G.p[u].l, (_Float16)sg);
        }
      }
#pragma unroll
      for (int u = 0; u < X3<LD>::KS; ++u) {
        *reinterpret_cast<f16x8*>(S.x[0] + at + 16 * u) = X.p[u].h;
        *reinterpret_cast<f16x8*>(S.x[1] + at + 16 * u) = X.p[u].l;
      }
    });
  }
  // From the rows' values, split once their scales are known, which takes no
  // scaling of pieces and no copy of them (per launch of k_wgrad_x3: 434,558 edges and 2 x
  // 32,768 nodes at width 128 172 -> 162 us, 0.68M edges at width 160 414 -> 330 us); then()
  // runs when they are no longer needed.
  template <class F>
  __device__ __forceinline__ void add_rows(const float* g, const float* x, bool live, DwLds<LD, NW>& S, int tid,
                                           F&& then) {
    const int eg = row_exp<LD>(g), ex = row_exp<LD>(x);
    const int k = fit(bound(eg, ex, live), S, tid), kx = k / 2;
    RowPieces<LD> G, X;
#pragma unroll
    for (int u = 0; u < X3<LD>::KS; ++u) {
      G.p[u] = split8(g + 8 * u, live ? eg + k - kx : -10000);
      X.p[u] = split8(x + 8 * u, ex + kx);
    }
    then();
    products(S, tid, [&](int at) {
#pragma unroll
      for (int u = 0; u < X3<LD>::KS; ++u) {
        *reinterpret_cast<f16x8*>(S.g[0] + at + 16 * u) = G.p[u].h;
        *reinterpret_cast<f16x8*>(S.g[1] + at + 16 * u) = G.p[u].l;
        *reinterpret_cast<f16x8*>(S.x[0] + at + 16 * u) = X.p[u].h;
        *reinterpret_cast<f16x8*>(S.x[1] + at + 16 * u) = X.p[u].l;
      }
    });
  }
  // the block's dW [LD][LD]
  __device__ __forceinline__ void store(float* base, int tid) const {
    const int lane = tid & 63, wv = tid >> 6, i = lane & 15, q = lane >> 4;
    const int u0 = 16 * TU * (wv / (LD / 16 / TV)), v0 = 16 * TV * (wv % (LD / 16 / TV));
#pragma unroll
    for (int u = 0; u < TU; ++u)
#pragma unroll
      for (int v = 0; v < TV; ++v)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          base[(size_t)(u0 + 16 * u + 4 * q + r) * LD + v0 + 16 * v + i] = __builtin_amdgcn_ldexpf(a[u * TV + v][r], -c);
  }
};

// The pieces of a whole row of values (zero when not live).
template <int LD>
__device__ __forceinline__ void split_row(RowPieces<LD>& r, const float* x, bool live) {
  r.e = row_exp<LD>(x);
  const int e = live ? r.e : -10000;
#pragma unroll
  for (int k = 0; k < X3<LD>::KS; ++k) r.p[k] = split8(x + 8 * k, e);
}

}  // namespace dev

}  // namespace mgn
