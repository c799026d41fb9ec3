"""Large graphs without a node of more in-edges than a tile are walked in runs
of whole segments, all others tile by tile.  A node's sums add the same rows in
the same order either way, so the same mesh with a component that holds one
such node beside it must give the same outputs and input gradients bit for
bit; parameter gradients differ only in how their sums are grouped."""
import numpy as np
import pytest

import synth
from gpu_util import rel_l2

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2304_00338_amd import mgn  # noqa: E402

GAP = 200  # nodes without edges in the middle and at the end of the mesh


def edgeless_mesh(shape, gap=1500):
    """The mesh with gap nodes without edges before, in the middle of and after its nodes."""
    M = synth.mesh(shape, 5)
    n = M["pos"].shape[0]
    lone = np.random.default_rng(4).random((3, gap, 3))
    cells = M["cells"] + gap + gap * (M["cells"] >= n // 2)
    pos = np.concatenate([lone[0], M["pos"][:n // 2], lone[1], M["pos"][n // 2:], lone[2]])
    return cells, pos.astype(np.float32)


def graphs(shape):
    """The mesh with the edgeless nodes, and the same with the hub's component
    (tetrahedra around an axis: the hub has 41 in-edges) after it."""
    M = synth.mesh(shape, 5)
    n = M["pos"].shape[0]
    cut = n // 2
    cells = M["cells"] + GAP * (M["cells"] >= cut)
    rng = np.random.default_rng(5)
    lone = lambda k: rng.random((k, 3))
    pos = np.concatenate([M["pos"][:cut], lone(GAP), M["pos"][cut:], lone(GAP)]).astype(np.float32)
    n0, k = pos.shape[0], 40
    ring = np.arange(k)
    fan = n0 + np.stack([0 * ring, 0 * ring + 1, 2 + ring, 2 + (ring + 1) % k], 1)
    pos2 = np.concatenate([pos, lone(k + 2).astype(np.float32)])
    return (mgn.build_graph(cells, pos), mgn.build_graph(np.concatenate([cells, fan.astype(cells.dtype)]), pos2), n0)


@pytest.mark.parametrize("prec,latent", [("fp32", 128), ("fp32", 150), ("bf16", 128)])
def test_runs_equal_tiles(prec, latent):
    m = 2
    ga, gb, n0 = graphs((44, 44, 44))
    assert ga.schedule()[1].shape[0] == 0 and gb.schedule()[1].shape[0] > 0
    params = torch.from_numpy(synth.xavier_params(m, 5, latent, randomize_norm=True)).cuda()
    rng = np.random.default_rng(6)
    x = rng.standard_normal((gb.n_nodes, 8)).astype(np.float32)
    w = rng.standard_normal((gb.n_nodes, 4)).astype(np.float32) / n0
    w[n0:] = 0  # the hub's component does not reach the loss
    res = []  # (tests/test_edge_plan.py: the first graph is walked in runs, some blocks without any)
    for g in (ga, gb):
        dg = mgn.DeviceGraph(g)
        xi = torch.from_numpy(x[:g.n_nodes].copy()).cuda()
        wi = torch.from_numpy(w[:g.n_nodes].copy()).cuda()
        ctx = mgn.Context(m, g.n_nodes, g.n_edges, prec, save=True, latent=latent)
        ctx.ws.fill_(255)  # NaN in every float: what is read is written first
        out = mgn.mgn_forward(ctx, dg, params, xi, dg.efeat, save=True)
        gp, gi = torch.zeros_like(params), torch.empty((g.n_nodes, 8), dtype=torch.float32, device="cuda")
        mgn.mgn_backward(ctx, wi, gp, gi)
        torch.cuda.synchronize()
        res.append((out[:n0].cpu().numpy(), gi[:n0].cpu().numpy(), gp.cpu().numpy()))
        # a forward that saves nothing may walk differently
        ctx = mgn.Context(m, g.n_nodes, g.n_edges, prec, latent=latent)
        ctx.ws.fill_(255)
        np.testing.assert_array_equal(mgn.mgn_forward(ctx, dg, params, xi, dg.efeat)[:n0].cpu().numpy(), res[-1][0])
        del ctx, dg
    (oa, ia, pa), (ob, ib, pb) = res
    assert np.isfinite(oa).all() and np.isfinite(pa).all()
    np.testing.assert_array_equal(oa, ob)
    np.testing.assert_array_equal(ia, ib)
    # the same fp32 terms in another grouping: at most about 500 additions in a
    # row, 500 * 2^-24 = 3e-5 of the sum of their magnitudes
    assert rel_l2(pa, pb) < 1e-4


# 34^3, 35 x 33 x 34: the fp32 forward has blocks without a run (the last one; two);
# 40^3: none; see tests/test_edge_plan.py
@pytest.mark.parametrize("shape", [(34, 34, 34), (35, 33, 34), (40, 40, 40)])
@pytest.mark.parametrize("prec,latent", [("fp32", 128), ("fp32", 150), ("bf16", 128)])
def test_edgeless_nodes_get_zero_sums(shape, prec, latent):
    """Nodes without edges at the start, in the middle and at the end of the
    numbering: what the workspace held before is in no output or gradient."""
    m = 2
    cells, pos = edgeless_mesh(shape)
    g = mgn.build_graph(cells, pos)
    dg = mgn.DeviceGraph(g)
    params = torch.from_numpy(synth.xavier_params(m, 5, latent, randomize_norm=True)).cuda()
    rng = np.random.default_rng(7)
    x = torch.from_numpy(rng.standard_normal((g.n_nodes, 8)).astype(np.float32)).cuda()
    w = torch.from_numpy((rng.standard_normal((g.n_nodes, 4)) / g.n_nodes).astype(np.float32)).cuda()
    res = []
    for save, fill in ((True, 0), (True, 255), (False, 255)):  # 255: NaN in every float
        ctx = mgn.Context(m, g.n_nodes, g.n_edges, prec, save=save, latent=latent)
        ctx.ws.fill_(fill)
        res.append([mgn.mgn_forward(ctx, dg, params, x, dg.efeat, save=save).cpu().numpy()])
        if save:
            gp, gi = torch.zeros_like(params), torch.empty((g.n_nodes, 8), dtype=torch.float32, device="cuda")
            mgn.mgn_backward(ctx, w, gp, gi)
            res[-1] += [gp.cpu().numpy(), gi.cpu().numpy()]
        del ctx
    for r in res[1:]:
        for a, b in zip(res[0], r):
            assert np.isfinite(b).all()
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("kind", ["nan", "overflow"])
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("latent", [128, 150])
def test_component_without_finite_values_stays_apart(prec, latent, kind):
    """A component of NaNs, or whose first edge activations overflow, beside a
    finite one: rows past a tile's end are copies of its last row, and must not reach
    the sums of the wave's next tile."""
    m, unit = 2, 5
    A, B = synth.mesh((7, 6, 6), 5), synth.mesh((16, 16, 16), 5)
    na = A["pos"].shape[0]
    g = mgn.build_graph(np.concatenate([A["cells"], B["cells"] + na]), np.concatenate([A["pos"], B["pos"]]))
    dg = mgn.DeviceGraph(g)
    # (the reverse's 1024 waves take the first component's tiles and then tiles of the second)
    assert 1024 < g.schedule()[0].shape[0] <= 2048
    p, v, o = synth.xavier_params(m, 5, latent, randomize_norm=True), {}, 0
    for name, _, shape in synth.param_shapes(m, latent):
        v[name] = p[o:o + int(np.prod(shape))].reshape(shape)
        o += int(np.prod(shape))
    # node type 1 sets latent feature 0 to about 10, from which the edge MLP's unit overflows
    v["enc_node.W1"][unit] = [0, 8, 0, 0, 0, 0, 0, 0]
    v["enc_node.b1"][unit] = -4
    v["enc_node.W2"][0] = 0
    v["enc_node.W2"][0, unit] = 20
    v["enc_node.gamma"][0], v["enc_node.beta"][0] = 1, 0
    v["block0.edge.W1"][unit] = 0
    v["block0.edge.W1"][unit, latent] = 1e38
    v["block0.edge.b1"][unit] = -3e38
    params = torch.from_numpy(p).cuda()
    rng = np.random.default_rng(8)
    x = rng.standard_normal((g.n_nodes, 8)).astype(np.float32)
    x[:, :4] = [1, 0, 0, 0]
    w = torch.from_numpy((rng.standard_normal((g.n_nodes, 4)) / g.n_nodes).astype(np.float32)).cuda()
    res = []
    for bad in (False, True):
        if bad and kind == "nan":
            x[:na] = np.nan
        elif bad:
            x[:na, :4] = [0, 1, 0, 0]
        ctx = mgn.Context(m, g.n_nodes, g.n_edges, prec, save=True, latent=latent)
        out = mgn.mgn_forward(ctx, dg, params, torch.from_numpy(x).cuda(), dg.efeat, save=True)
        gi = torch.empty((g.n_nodes, 8), dtype=torch.float32, device="cuda")
        mgn.mgn_backward(ctx, w, torch.zeros_like(params), gi)
        res.append((out.cpu().numpy(), gi.cpu().numpy()))
        del ctx
    if prec == "fp32":  # (a bf16 ReLU may take a NaN for negative)
        assert not np.isfinite(res[1][0][:na]).any()
    for a, b in zip(*res):
        assert np.isfinite(a).all()
        np.testing.assert_array_equal(a[na:], b[na:])
