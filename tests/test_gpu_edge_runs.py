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
    res = []
    for g in (ga, gb):
        dg = mgn.DeviceGraph(g)
        xi = torch.from_numpy(x[:g.n_nodes].copy()).cuda()
        wi = torch.from_numpy(w[:g.n_nodes].copy()).cuda()
        ctx = mgn.Context(m, g.n_nodes, g.n_edges, prec, save=True, latent=latent)
        out = mgn.mgn_forward(ctx, dg, params, xi, dg.efeat, save=True)
        gp, gi = torch.zeros_like(params), torch.empty((g.n_nodes, 8), dtype=torch.float32, device="cuda")
        mgn.mgn_backward(ctx, wi, gp, gi)
        torch.cuda.synchronize()
        res.append((out[:n0].cpu().numpy(), gi[:n0].cpu().numpy(), gp.cpu().numpy()))
        del ctx, dg
    (oa, ia, pa), (ob, ib, pb) = res
    assert np.isfinite(oa).all() and np.isfinite(pa).all()
    np.testing.assert_array_equal(oa, ob)
    np.testing.assert_array_equal(ia, ib)
    # the same fp32 terms in another grouping: at most about 500 additions in a
    # row, 500 * 2^-24 = 3e-5 of the sum of their magnitudes
    assert rel_l2(pa, pb) < 1e-4
