"""The fp32 kernels form their products from scaled two-piece operands.  The
scales are powers of two, so a network whose hidden layers are rescaled by
one (W1, b1 by 2^k and W2 by 2^-k: a ReLU passes the factor through) must
give the same output bit for bit, and gradients that differ by exactly that
factor, however far the rows and the weights are from one."""
import numpy as np
import pytest

import oracle as O
import synth
from gpu_util import FP32_TOL, rel_l2

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2304_00338_amd import mgn  # noqa: E402


def factors(m, latent, k):
    """Per-parameter factor of the rescaled network."""
    f = []
    for name, _, shape in synth.param_shapes(m, latent):
        kind = name.rsplit(".", 1)[1]
        f.append(np.full(int(np.prod(shape)), {"W1": 2.0 ** k, "b1": 2.0 ** k, "W2": 2.0 ** -k}.get(kind, 1.0)))
    return np.concatenate(f).astype(np.float32)


def call(shape, m, latent, params):
    M = synth.mesh(shape, 3)
    g = mgn.build_graph(M["cells"], M["pos"])
    dg = mgn.DeviceGraph(g)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()
    p, x, w = dev(params), dev(M["node_in"]), dev(synth.loss_weights(g.n_nodes, 3))
    ctx = mgn.Context(m, g.n_nodes, g.n_edges, "fp32", save=True, latent=latent)
    out = mgn.mgn_forward(ctx, dg, p, x, dg.efeat, save=True)
    gp, gi = torch.zeros_like(p), torch.empty((g.n_nodes, 8), dtype=torch.float32, device="cuda")
    mgn.mgn_backward(ctx, w, gp, gi)
    torch.cuda.synchronize()
    return M, out.cpu().numpy(), gp.cpu().numpy(), gi.cpu().numpy()


# one tile, a tile and a row, several blocks with a ragged last one
@pytest.mark.parametrize("shape", [(3, 3), (4, 3, 3), (11, 10, 9)])
@pytest.mark.parametrize("latent", [128, 150])
def test_power_of_two_rescaling_is_exact(shape, latent):
    m = 2
    params = synth.xavier_params(m, 3, latent, randomize_norm=True)
    M, out, gp, gi = call(shape, m, latent, params)
    go = O.build_graph(M["cells"], M["pos"])
    ref = O.mgn_forward(go, params, M["node_in"], go.efeat, m, latent=latent)
    assert rel_l2(out, ref[0] if isinstance(ref, tuple) else ref) < FP32_TOL
    for k in (-40, 1, 40):
        f = factors(m, latent, k)
        _, o2, gp2, gi2 = call(shape, m, latent, params * f)
        np.testing.assert_array_equal(o2, out)
        np.testing.assert_array_equal(gi2, gi)
        np.testing.assert_array_equal(gp2 * f, gp)
