"""The workloads on which this library's speed is judged.

A case is one call (or one forward and backward pair) of the public entry
points on a jittered Kuhn mesh of the unit square or cube, as a program that
trains or serves a mesh surrogate makes it: single MGN calls, integration
steps with and without the reverse, patch-decomposed steps and patch-training
steps, in both precisions and at both latent widths.

Parameters.  Forward-only cases take Xavier weights with small random biases
and gains.  Where gradients come back, the gradient of a ReLU network jumps
at every ReLU input near zero, and two correct implementations differ there
by whole terms; so those cases sit at a point whose first-layer biases are
+6 or -6 in turn and whose first-layer weights are small: half of the hidden
units are active, half are not, none is near its kink, the gradient is unique
and can be compared at the accuracy of the data types.

``exact`` evaluates the same model in float64 with plain torch on an edge
list written down from the grid (the Kuhn split of a grid has one edge along
every non-zero 0/1 offset), in the concatenated form of the edge MLP.
"""
from __future__ import annotations

import itertools
import math

import numpy as np
import torch
import torch.utils.checkpoint

from paper_2304_00338_amd import mgn

NOISE = (0.02, 0.02, 0.03, 0.05)  # input-noise levels of the 3D training step
TABLEAUS = {
    "euler": ([[]], [1.0]),
    "heun2": ([[], [1.0]], [0.5, 0.5]),
    "midpoint": ([[], [0.5]], [0.0, 1.0]),
    "heun3": ([[], [1 / 3], [0.0, 2 / 3]], [0.25, 0.0, 0.75]),
    "rk4": ([[], [0.5], [0.0, 0.5], [0.0, 0.0, 1.0]], [1 / 6, 1 / 3, 1 / 3, 1 / 6]),
}


def listed():
    def c(name, kind, grid, mp, prec, scheme="euler", latent=128, parts="", n_parts=0, ghost=0, interior=""):
        return {"name": name, "kind": kind, "grid": grid, "mp": mp, "prec": prec, "scheme": scheme, "latent": latent,
                "parts": parts, "n_parts": n_parts, "ghost": ghost, "interior": interior}
    return [
        # one MGN call on a small 2D mesh: a solver that asks for single
        # predictions, where the launches and each kernel's latency count
        c("serve-2d-fp32", "forward", "32x32", 2, "fp32"),
        # the allocation-free call of a serving loop, full depth, ragged size
        c("serve-2d-bf16", "noalloc", "45x43", 15, "bf16"),
        # forward and backward of one Euler step on the same small mesh
        c("train-2d-fp32", "train", "32x32", 2, "fp32"),
        # the 3D mesh of 32^3 nodes at full depth, forward and backward
        c("train-3d-fp32", "train", "32x32x32", 15, "fp32"),
        c("train-3d-bf16", "train", "32x32x32", 15, "bf16"),
        # the node and edge counts of one 15-hop slab patch of a 146^3 mesh
        # (40 grid layers, 10 of them the subdomain that the loss covers)
        c("train-slab-bf16", "train", "146x146x40", 2, "bf16", interior="15:25"),
        # inference on the same slab at full depth
        c("step-slab-bf16", "step", "146x146x40", 15, "bf16"),
        # a higher-order rollout step in full precision, odd sizes
        c("rk4-3d-fp32", "step", "33x29x31", 15, "fp32", scheme="rk4"),
        # the 3D training configuration: latent 150, 3 MP steps, Heun's second
        # order, a batch of 12 x 12 x 10 subdomains with 6-hop ghost zones as
        # one union graph, input noise, masked loss, Adam
        c("batch-150-fp32", "batch", "48x36x40", 3, "fp32", "heun2", 150, "4x3x4", 8, 6),
        c("batch-150-bf16", "batch", "48x36x40", 3, "bf16", "heun2", 150, "4x3x4", 8, 6),
        # patch-decomposed inference of a 150k-node 2D mesh in 3 x 4 patches
        c("patches-2d-fp32", "patches", "388x388", 15, "fp32", parts="3x4", ghost=15),
        # a predict-evaluate-correct rollout step of the same mesh
        c("pec-2d-bf16", "pec", "388x388", 15, "bf16"),
    ]


def draw(rng):
    kind = rng.choice(["forward", "noalloc", "train", "train", "step", "batch", "patches", "pec"])
    prec = rng.choice(["fp32", "bf16"])
    c = {"kind": kind, "prec": prec, "scheme": "euler", "latent": rng.choice([128, 128, 150]), "mp": rng.randint(1, 15),
         "parts": "", "n_parts": 0, "ghost": 0, "interior": ""}
    lo, hi = 300, 100000
    if kind == "noalloc":  # what the call's fixed scratch holds
        hi = 3000
    elif kind == "train":
        c["scheme"] = rng.choice(["euler", "euler", "midpoint", "heun2", "rk4"])
        stages = len(TABLEAUS[c["scheme"]][1])
        hi = 30000 // stages
    elif kind == "step":
        c["scheme"] = rng.choice(sorted(TABLEAUS))
        hi = 100000 // len(TABLEAUS[c["scheme"]][1])
    elif kind == "pec":
        hi = 100000
    if kind == "batch":
        c["scheme"] = rng.choice(["euler", "heun2"])
        c["mp"] = rng.randint(1, 3)
        c["latent"] = 150
        c["ghost"] = c["mp"] * len(TABLEAUS[c["scheme"]][1])
        parts = [rng.randint(2, 4) for _ in range(3)]
        size = [p * rng.randint(7, 12) for p in parts]
        c["n_parts"] = rng.randint(2, 8)
    elif kind == "patches":
        c["ghost"] = c["mp"]
        parts = [rng.randint(2, 4), rng.randint(2, 4)]
        size = [p * rng.randint(20, 90) for p in parts]
    else:
        n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        dim = rng.choice([2, 3])
        shape = [rng.uniform(0.8, 1.25) for _ in range(dim)]
        k = (n / math.prod(shape)) ** (1 / dim)
        size, parts = [max(3, round(s * k)) for s in shape], []
    c["grid"] = "x".join(map(str, size))
    c["parts"] = "x".join(map(str, parts)) if kind in ("batch", "patches") else ""
    return c


# ------------------------------------------------------------------- inputs
def ints(text):
    return tuple(int(v) for v in text.split("x"))


def directions(dim):
    return [np.array(d) for d in itertools.product((0, 1), repeat=dim) if any(d)]


def grid_ids(size):
    """Node ids, x fastest, indexed [x, y(, z)]."""
    return np.arange(math.prod(size), dtype=np.int32).reshape(size[::-1]).transpose()


def corner(ids, off):
    return ids[tuple(slice(o, n - 1 + o) for o, n in zip(off, ids.shape))].reshape(-1)


def cells_of(size):
    """The Kuhn split of the grid's cells: one simplex per order of the axes."""
    ids, dim, out = grid_ids(size), len(size), []
    for order in itertools.permutations(range(dim)):
        off, verts = [0] * dim, []
        verts.append(corner(ids, off))
        for ax in order:
            off[ax] = 1
            verts.append(corner(ids, off))
        out.append(np.stack(verts, 1))
    return np.ascontiguousarray(np.concatenate(out))


def coords(size):
    return np.stack([c.transpose().reshape(-1) for c in np.meshgrid(*[np.arange(n) for n in size], indexing="ij")], 1)


def positions(size, rng):
    step = 1.0 / (np.array(size) - 1)
    jitter = rng.uniform(-0.2, 0.2, (math.prod(size), len(size)))
    return ((coords(size) + jitter) * step).astype(np.float32)


def types_of(size):
    """One-hot node types: interior, first face, last face of the last axis,
    other boundary."""
    at = coords(size)
    edge = ((at == 0) | (at == np.array(size) - 1)).any(1)
    t = np.where(at[:, -1] == 0, 1, np.where(at[:, -1] == size[-1] - 1, 2, np.where(edge, 3, 0)))
    return np.eye(4, dtype=np.float32)[t]


def shapes(mp, D):
    """The parameter buffer: (kind, shape) in order, weights as [out, in]."""
    def mlp(din, dout, norm):
        s = [("w1", (D, din)), ("b1", (D,)), ("w2", (dout, D)), ("b2", (dout,))]
        return s + ([("g", (dout,)), ("z", (dout,))] if norm else [])
    s = mlp(8, D, True) + mlp(4, D, True)
    for _ in range(mp):
        s += mlp(3 * D, D, True) + mlp(2 * D, D, True)
    return s + mlp(D, 4, False)


def parameters(mp, D, smooth, rng):
    out = []
    for kind, shape in shapes(mp, D):
        if kind in ("w1", "w2"):
            lim = math.sqrt(6.0 / sum(shape)) * (0.05 if smooth and kind == "w1" else 1.0)
            v = rng.uniform(-lim, lim, shape)
        elif kind == "b1" and smooth:
            v = np.where(np.arange(shape[0]) % 2 == 0, 6.0, -6.0) + rng.uniform(-0.3, 0.3, shape)
        else:
            v = (1.0 if kind == "g" else 0.0) + rng.uniform(-0.3, 0.3, shape)
        out.append(v.reshape(-1))
    return np.concatenate(out).astype(np.float32)


def host_inputs(case, seed):
    """Everything that is drawn, as host arrays."""
    size = ints(case["grid"])
    rng = np.random.default_rng(seed)
    n = math.prod(size)
    y = rng.standard_normal((n, 4)).astype(np.float32)
    if len(size) == 3:
        y[:, 3] = rng.uniform(0, 1, n)  # a volume fraction
    v = {"size": size, "n": n, "pos": positions(size, rng), "types": types_of(size), "y": y,
         "params": parameters(case["mp"], case["latent"], case["kind"] in ("train", "batch"), rng)}
    if case["kind"] == "train":
        w = rng.standard_normal((n, 4)).astype(np.float32)
        if case["interior"]:  # layers of the last axis that the loss covers
            lo, hi = (int(t) for t in case["interior"].split(":"))
            z = coords(size)[:, -1]
            w *= ((z >= lo) & (z < hi))[:, None]
        v["gout"] = w
    if case["kind"] == "batch":
        v["target"] = y + 0.1 * rng.standard_normal((n, 4)).astype(np.float32)
        v["noise"] = rng.standard_normal((n, 4)).astype(np.float32)
        # moments of a run that is under way
        v["m"] = (1e-4 * rng.standard_normal(v["params"].size)).astype(np.float32)
        v["v"] = rng.uniform(1e-8, 1e-6, v["params"].size).astype(np.float32)
        v["ids"] = np.sort(rng.choice(math.prod(ints(case["parts"])), case["n_parts"], replace=False))
    if case["kind"] == "pec":
        v["khist"] = 0.1 * rng.standard_normal((2, n, 4)).astype(np.float32)
    return v


def prepare(case, seed):
    v = host_inputs(case, seed)
    g = mgn.build_graph(cells_of(v["size"]), v["pos"])
    dev = {k: torch.from_numpy(x).cuda() for k, x in v.items()
           if k in ("types", "y", "params", "gout", "target", "noise", "m", "v", "khist")}
    st = dict(case, **dev)
    kind, latent = case["kind"], case["latent"]
    stages = len(TABLEAUS[case["scheme"]][1])

    def context(n, e, save):
        return mgn.Context(case["mp"], n, e, case["prec"], max_stages=stages, save=save, latent=latent,
                           allocate=kind != "noalloc")
    if kind in ("batch", "patches"):
        part = mgn.partition(v["pos"], ints(case["parts"]))
        if kind == "batch":
            st["patches"] = [mgn.DevicePatch(mgn.patch_union([mgn.extract_patch(g, part, int(p), case["ghost"])
                                                              for p in v["ids"]]))]
            st["adam"], st["k"], st["grad"] = mgn.Adam(), 1000, torch.empty_like(dev["params"])
        else:
            st["patches"] = [mgn.DevicePatch(mgn.extract_patch(g, part, p, case["ghost"]))
                             for p in range(int(part.max()) + 1)]
        st["ctx"] = context(max(p.n_nodes for p in st["patches"]), max(p.n_edges for p in st["patches"]), kind == "batch")
        return st
    st["g"] = mgn.DeviceGraph(g)
    st["ctx"] = context(g.n_nodes, g.n_edges, kind == "train")
    if kind in ("forward", "noalloc"):
        st["x"] = torch.cat([dev["types"], dev["y"]], 1)
        st["out"] = torch.empty_like(dev["y"])
    if kind == "train":
        st["grad"], st["gin"] = torch.zeros_like(dev["params"]), torch.empty_like(dev["y"])
    return st


def run(st):
    kind = st["kind"]
    if kind == "forward":
        return mgn.mgn_forward(st["ctx"], st["g"], st["params"], st["x"], st["g"].efeat)
    if kind == "noalloc":
        return mgn.mgn_forward_noalloc(st["ctx"], st["g"], st["params"], st["x"], st["g"].efeat, st["out"])
    if kind == "pec":
        y = mgn.mgn_pec_step(st["ctx"], st["g"], st["params"], st["types"], st["y"], st["khist"], st["g"].efeat)
        return {"y": y, "khist": st["khist"]}
    if kind == "patches":
        return mgn.mgn_patch_step(st["ctx"], st["patches"], st["params"], st["scheme"], st["types"], st["y"])
    if kind == "batch":
        loss = mgn.mgn_train_step(st["ctx"], st["patches"], st["params"], st["scheme"], st["types"], st["y"], st["target"],
                                  st["noise"], st["grad"], st["m"], st["v"], st["adam"], st["k"])
        st["k"] += 1
        return {"loss": loss, "grad": st["grad"], "params": st["params"]}
    save = kind == "train"
    y = mgn.mgn_integrate_step(st["ctx"], st["g"], st["params"], st["scheme"], st["types"], st["y"], st["g"].efeat,
                               save=save)
    if not save:
        return y
    st["grad"].zero_()
    mgn.mgn_backward(st["ctx"], st["gout"], st["grad"], st["gin"])
    return {"y": y, "grad": st["grad"], "gin": st["gin"]}


# ----------------------------------------------------------- what it comes to
def edge_count(size):
    return 2 * sum(math.prod(n - int(d) for n, d in zip(size, o)) for o in directions(len(size)))


def counts(case):
    """(nodes, edges) that the call computes on; for patches an estimate from
    their sizes (the subdomain grown by the ghost depth, cut at the mesh)."""
    size = ints(case["grid"])
    if case["kind"] not in ("batch", "patches"):
        return math.prod(size), edge_count(size)
    parts, k, total = ints(case["parts"]), case["ghost"], [0, 0]
    for at in itertools.product(*[range(p) for p in parts]):
        grown = [min(n, round((a + 1) * n / p) + k) - max(0, round(a * n / p) - k) for a, n, p in zip(at, size, parts)]
        total[0] += math.prod(grown)
        total[1] += edge_count(grown)
    share = case["n_parts"] / math.prod(parts) if case["kind"] == "batch" else 1.0
    return total[0] * share, total[1] * share


def work(case):
    """Per MP step: the edge and node latents are read and written once (they
    outgrow every cache, and an MP step needs its neighbours' results), the
    reverse reads them again and reads and writes their gradients; products at
    two flops a weight and row, with the edge MLP's sender and receiver columns
    once per node, and twice that in the reverse."""
    n, e = counts(case)
    D, mp = case["latent"], case["mp"]
    stages = len(TABLEAUS[case["scheme"]][1])
    back = case["kind"] in ("train", "batch")
    es = 2 if case["prec"] == "bf16" else 4
    step_bytes = e * (2 * D * es + 8) + n * (2 * D * 4 + 4)
    step_flops = e * 2 * 2 * D * D + n * 2 * D * (2 * D + 2 * D + D)
    if back:
        step_bytes += e * (3 * D * es + 8) + n * 3 * D * 4
        step_flops *= 3
    ends = 3 if back else 1
    weights = 4 * sum(math.prod(s) for _, s in shapes(mp, D))
    return {"bytes": stages * (mp * step_bytes + n * 48) + ends * (weights + 16 * e),
            "flops": stages * (mp * step_flops + ends * n * 2 * D * (8 + D + D + 4)) + ends * e * 2 * D * (4 + D)}


def tolerance(case):
    """About four times what separates the library from ``exact``: in fp32
    outputs and gradients 2e-7 to 6e-7; in bf16 gradients 1.0e-3 to 1.8e-3 at
    their kink-free point, and 4.5e-3 to 1.1e-2 in outputs of Xavier weights at
    full depth, where every layer's rounding of its operands travels on."""
    if case["prec"] == "fp32":
        return {"rel": 4e-6}
    return {"rel": 8e-3 if case["kind"] in ("train", "batch") else 3e-2}


# ------------------------------------------------------------------- float64
def mlp_of(p, x):
    """The MLP on the rows of x: ReLU between its layers, then LayerNorm
    where the MLP ends in one."""
    z = torch.relu(x @ p[0].T + p[1]) @ p[2].T + p[3]
    if len(p) == 4:
        return z
    return torch.nn.functional.layer_norm(z, z.shape[-1:], p[4], p[5], 1e-5)


def in_parts(f, rows):
    """f over slices of rows, to bound the memory of the wide products."""
    cut = 1 << 20
    if rows <= cut:
        return f(slice(0, rows))
    return torch.cat([f(slice(a, min(a + cut, rows))) for a in range(0, rows, cut)])


def exact(case, seed):
    v = host_inputs(case, seed)
    size, n = v["size"], v["n"]
    D, mp = case["latent"], case["mp"]
    d64 = lambda a: torch.from_numpy(np.asarray(a)).cuda().double()  # noqa: E731
    # both directions of every grid edge
    ids, pairs = grid_ids(size), []
    for o in directions(len(size)):
        a = ids[tuple(slice(0, m - int(k)) for m, k in zip(size, o))].reshape(-1)
        b = ids[tuple(slice(int(k), m) for m, k in zip(size, o))].reshape(-1)
        pairs += [np.stack([a, b]), np.stack([b, a])]
    snd, rcv = (torch.from_numpy(t.astype(np.int64)).cuda() for t in np.concatenate(pairs, 1))
    pos = d64(v["pos"])
    if pos.shape[1] == 2:
        pos = torch.cat([pos, torch.zeros_like(pos[:, :1])], 1)
    dx = pos[snd] - pos[rcv]
    length = dx.norm(dim=1, keepdim=True)
    if len(size) == 2:
        f = torch.cat([dx[:, :2], length, torch.zeros_like(length)], 1)
    else:
        f = torch.cat([dx, length], 1)
    f = f.float().double()  # the features are float32 inputs
    back = case["kind"] in ("train", "batch")
    flat = d64(v["params"]).requires_grad_(back)
    views, o = [], 0
    for _, s in shapes(mp, D):
        views.append(flat[o:o + math.prod(s)].view(s))
        o += math.prod(s)
    mlps = [views[6 * i:6 * i + 6] for i in range(2 + 2 * mp)] + [views[-4:]]
    types, y = d64(v["types"]), d64(v["y"])

    def block(e, h, i):
        pe, pn = mlps[2 + 2 * i], mlps[3 + 2 * i]
        m = in_parts(lambda s: mlp_of(pe, torch.cat([e[s], h[snd[s]], h[rcv[s]]], 1)), e.shape[0])
        agg = torch.zeros_like(h).index_add(0, rcv, m)
        return e + m, h + mlp_of(pn, torch.cat([h, agg], 1))

    def model(state):
        h = mlp_of(mlps[0], torch.cat([types, state], 1))
        e = in_parts(lambda s: mlp_of(mlps[1], f[s]), f.shape[0]) if mp else None
        for i in range(mp):
            if back:
                e, h = torch.utils.checkpoint.checkpoint(block, e, h, i, use_reentrant=False)
            else:
                e, h = block(e, h, i)
        return mlp_of(mlps[-1], h)

    def step(state):
        a, b = TABLEAUS[case["scheme"]]
        ks = []
        for row in a:
            ks.append(model(state + sum(c * k for c, k in zip(row, ks) if c)))
        return state + sum(c * k for c, k in zip(b, ks))

    with torch.set_grad_enabled(back):
        if case["kind"] in ("forward", "noalloc"):
            return model(y)
        if case["kind"] == "pec":
            k1, k0 = d64(v["khist"])
            kp = model(y + 1.5 * k1 - 0.5 * k0)
            return {"y": y + 0.5 * (kp + k1), "khist": torch.stack([kp, k1])}
        if case["kind"] in ("step", "patches"):
            return step(y)  # patches with a ghost depth of the receptive field equal the whole mesh
        if case["kind"] == "train":
            y.requires_grad_(True)
            out = step(y)
            grad, gin = torch.autograd.grad((out * d64(v["gout"])).sum(), (flat, y))
            return {"y": out.detach(), "grad": grad, "gin": gin}
        # batch: the loss covers the drawn subdomains; the graph of the whole
        # mesh gives the same gradient as their patches
        pos32 = v["pos"].astype(np.float64)
        lo, hi = pos32.min(0), pos32.max(0)
        parts = np.array(ints(case["parts"]))
        at = np.clip(np.floor(parts * (pos32 - lo) / (hi - lo)), 0, parts - 1).astype(np.int64)
        sub = (at * np.concatenate([[1], np.cumprod(parts)[:-1]])).sum(1)
        mask = torch.from_numpy(np.isin(sub, v["ids"])).cuda()
        noisy = y + torch.tensor(NOISE, dtype=torch.float64, device="cuda").float().double() * d64(v["noise"])
        diff = (step(noisy) - d64(v["target"]))[mask]
        loss = diff.square().sum() / (4 * int(mask.sum()))
        grad, = torch.autograd.grad(loss, flat)
        k, b1, b2 = 1000, 0.9, 0.999
        lr = 1e-3 * 1e-4 ** ((k - 1) / 4e6)
        m = b1 * d64(v["m"]) + (1 - b1) * grad
        s = b2 * d64(v["v"]) + (1 - b2) * grad.square()
        p = flat.detach() - lr * (m / (1 - b1 ** k)) / ((s / (1 - b2 ** k)).sqrt() + 1e-8)
        return {"loss": loss.detach().reshape(1), "grad": grad, "params": p}
