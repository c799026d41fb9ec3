"""The walk that the edge launchers choose (plan_runs, unit_blocks), compiled
from the library's own header on the host: runs hold every edge once and at
most the rows of their steps, and the meshes of test_gpu_edge_runs.py are the
ones where it matters (runs, with and without blocks that get none)."""
import os
import subprocess

import numpy as np
import pytest

from paper_2304_00338_amd import build as B
from paper_2304_00338_amd import mgn
from test_gpu_edge_runs import edgeless_mesh, graphs

SRC = r"""
#include "launch.hpp"
#include <cstdio>
int main(int, char** a) {
  mgn::EdgeTiles t{};
  t.n_tiles = atoll(a[1]);
  t.n_edges = atoll(a[2]);
  t.n_long = atoll(a[3]);
  const int nw = atoi(a[4]), most = atoi(a[5]);
  t = mgn::plan_runs(t, nw * most);
  const int64_t n = mgn::walk_n(t);
  const int g = mgn::unit_blocks(n, nw, most);
  int64_t units = 0, idle = 0;
  for (int b = 0; b < g; ++b) {
    const mgn::BlockRange r = mgn::block_units(n, g, b, nw);
    idle += r.tb >= r.tend;
    for (int64_t u = r.tb; u < r.tend; u += r.stride)
      for (int w = 0; w < nw; ++w) units += u + w < r.tend;
  }
  printf("%d %d %lld %d %lld %lld\n", t.run, t.span, (long long)n, g, (long long)units, (long long)idle);
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, exe = d / "plan.cpp", d / "plan"
    src.write_text(SRC)
    subprocess.run([B.HIPCC, "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", B.CSRC, str(src), "-o", str(exe)], check=True)

    def call(n_tiles, n_edges, n_long, nw, most):
        r = subprocess.run([str(exe), *map(str, (n_tiles, n_edges, n_long, nw, most))], check=True, stdout=subprocess.PIPE)
        return dict(zip(("run", "span", "n", "blocks", "units", "idle"), map(int, r.stdout.split())))
    return call


# waves per block and blocks at most of the fp32 forward, the fp32 reverse at
# widths 128 and 160 (the last also the bf16 reverse), the bf16 forward
KERNELS = {"fwd32": (4, 512), "bwd32": (8, 256), "bwd32w": (4, 256), "fwd16": (8, 256)}


@pytest.mark.parametrize("kernel", sorted(KERNELS))
@pytest.mark.parametrize("shape,idle", [((34, 34, 34), 1), ((35, 33, 34), 2), ((40, 40, 40), 0)])
def test_runs_of_meshes(plan, kernel, shape, idle):
    g = mgn.build_graph(*edgeless_mesh(shape))
    n_tiles = g.schedule()[0].shape[0]
    p = plan(n_tiles, g.n_edges, 0, *KERNELS[kernel])
    assert p["run"] > 0 and p["units"] == p["n"]
    if kernel == "fwd32":
        assert p["idle"] == idle
    # the runs' bounds: the segments that hold edges span apart
    a = g.arrays()
    at = np.arange(p["n"], dtype=np.int64) * p["span"]
    lo = a["rowptr"][a["receivers"][at]].astype(np.int64)
    lo[0] = 0
    size = np.diff(np.append(lo, g.n_edges))
    assert at[-1] < g.n_edges and size.min() >= 0 and size.max() <= 32 * p["run"]
    assert plan(n_tiles, g.n_edges, 1, *KERNELS[kernel])["run"] == 0


def test_compared_walks_differ(plan):
    ga, gb, _ = graphs((44, 44, 44))
    for nw, most in KERNELS.values():
        for g, runs in ((ga, True), (gb, False)):
            tiles, longn = g.schedule()
            assert (plan(tiles.shape[0], g.n_edges, longn.shape[0], nw, most)["run"] > 0) == runs


def test_units_are_dealt_once(plan):
    rng = np.random.default_rng(0)
    for n in [1, 7, 8, 9, 31, 32, 33, 2047, 2048, 2049] + list(rng.integers(1, 60000, 20)):
        for nw, most in KERNELS.values():
            p = plan(n, 24 * n, 1, nw, most)
            assert p["units"] == n and 0 < p["blocks"] <= most
