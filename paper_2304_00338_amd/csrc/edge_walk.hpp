// How the waves of an edge kernel walk the edges: steps of at most 32 rows.
//
// The tile table's tiles hold whole in-segments, which leaves rows of a step
// empty: with 13.3 in-edges per node (Kuhn mesh of a cube) a tile holds 27.8 edges
// on average, with 6 per node 30.  Where a wave has several tiles to do, and no node has
// more in-edges than a tile, it takes runs instead (plan_runs): a run is a
// range of consecutive whole segments of at most 32 K edges, walked in K steps
// of 32 rows; a segment may go on in the next step, and the kernel carries its
// sum there.  A segment's rows are added in the same order either way, so its
// sum has the same bits.  Run c ends at the segment that holds edge (c + 1)
// span, span = 32 K - 31: whole segments around span edges are never more than
// 32 K.
#pragma once
#include "launch.hpp"
#include "rows_common.hpp"

namespace mgn {
namespace dev {

__device__ __forceinline__ int const_int(const int32_t* p, int64_t i) {
  typedef __attribute__((address_space(4))) const int ConstInt;
  return ((ConstInt*)p)[i];
}

__device__ __forceinline__ int64_t walk_units(const EdgeTiles& tl) { return tl.run ? tl.n_runs : tl.n_tiles; }
__device__ __forceinline__ int walk_steps(const EdgeTiles& tl) { return tl.run ? tl.run : 1; }

// The steps of one wave, whose units (tiles or runs) are t, t + stride, ... below
// tend.  A step is {node_begin, y, edge_begin, edge_end}: y = -1 - slot for a
// chunk of a long segment (tiles only); otherwise the last row's segment ends
// with the step if and only if its receiver is below y.  Steps past the range
// are {0, 0, 0, 0} (no rows).  All values are wave-uniform scalars.
struct EdgeSteps {
  int64_t t, stride, tend;
  int s, b0, b1, n0, n1;  // step of the run; the run's and the next run's edges
  __device__ __forceinline__ void bounds(const EdgeTiles& tl, int64_t c, int& lo, int& hi) const {
    const bool ok = c < tend;
    const int64_t a = c * tl.span, e = tl.n_edges;
    lo = ok && c > 0 ? const_int(tl.rowptr, const_int(tl.receivers, a)) : 0;
    hi = !ok ? 0 : a + tl.span < e ? const_int(tl.rowptr, const_int(tl.receivers, a + tl.span)) : (int)e;
  }
  __device__ __forceinline__ int4 tile(const EdgeTiles& tl) const {
    const bool ok = t < tend;
    const int4 v = tile_desc(tl.tiles, ok ? t : max(tend - 1, (int64_t)0));
    return ok ? v : make_int4(0, 0, 0, 0);
  }
  __device__ __forceinline__ int4 step(const EdgeTiles& tl) const {
    const int z = min(b0 + 32 * s, b1), w = min(z + 32, b1);
    return make_int4(0, w < b1 ? const_int(tl.receivers, w) : 0x7fffffff, z, w);
  }
  __device__ __forceinline__ int4 first(const EdgeTiles& tl, int64_t t0, int64_t st, int64_t end) {
    t = t0;
    stride = st;
    tend = end;
    if (!tl.run) return tile(tl);
    s = 0;
    bounds(tl, t, b0, b1);
    bounds(tl, t + stride, n0, n1);
    return step(tl);
  }
  __device__ __forceinline__ int4 next(const EdgeTiles& tl) {
    if (!tl.run) {
      t += stride;
      return tile(tl);
    }
    if (++s == tl.run) {
      s = 0;
      t += stride;
      b0 = n0;
      b1 = n1;
      bounds(tl, t + stride, n0, n1);
    }
    return step(tl);
  }
};

// The step's rows that end a segment (bit per row).  Rows are sorted by
// receiver; rcv: the lane's row's receiver (row = the lane's row, 0 .. 31 in
// lanes 0 .. 31); y as above.
__device__ __forceinline__ uint32_t segment_ends(int row, int n, int rcv, int y) {
  const int nx = __shfl(rcv, min(row + 1, 31));
  const bool e = row < n && (row == n - 1 ? y < 0 || rcv < y : y >= 0 && nx != rcv);
  return (uint32_t)__ballot(e);
}

// Zero rows of dst for a tile's nodes without in-edges ...
template <int LD>
__device__ __forceinline__ void zero_empty(int v0, int v1, const int32_t* __restrict__ rowptr, int lane, float* dst) {
  const int v = min(v0 + lane, v1 - 1);
  uint64_t m = __ballot(lane < v1 - v0 && rowptr[v] == rowptr[v + 1]);
  while (m) {
    const int j = __builtin_ctzll(m);
    m &= m - 1;
    float* q = dst + (size_t)(v0 + j) * LD;
    for (int f = lane; f < LD; f += 64) q[f] = 0.f;
  }
}
// ... and, where the waves walk runs, for wave w's even share of all nodes.
template <int LD>
__device__ __forceinline__ void zero_share(const EdgeTiles& tl, int64_t w, int64_t n_waves, int lane, float* dst) {
  const int64_t v1 = tl.n_nodes * (w + 1) / n_waves;
  for (int64_t v = tl.n_nodes * w / n_waves; v < v1; v += 64)
    zero_empty<LD>((int)v, (int)min(v + 64, v1), tl.rowptr, lane, dst);
}

}  // namespace dev
}  // namespace mgn
