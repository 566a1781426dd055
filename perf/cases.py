"""The work that a user of this framework has it do, as timed cases.

Four kinds, each through the package's public entry points:

* ``flow``: one periodic box of spheres run for some hundred steps with its
  residual checks, then the permeability, the drag and the fields (the sweeps,
  the precision study and the wall study are loops of this);
* ``batch``: many independent cells run together on the device (the batch
  study and the solving of training cells);
* ``conv``: one 3x3x3 layer of the warm-start network, forward or backward;
* ``net``: the network as a whole, a training step or the two-grid warm start
  of a pack.

Inputs are drawn from the seed.  ``exact`` repeats a case in plain torch in 64
bits.
"""
from __future__ import annotations

import math
import os

import numpy as np
import torch

from paper_1508_02960_amd import lbm, warmstart

DEV = "cuda"
WEIGHTS = os.path.join(os.path.dirname(os.path.abspath(warmstart.__file__)), "data",
                       "unet64_dense_bf16.npz")
ELEM = {"fp64": 8, "fp32": 4, "fp16": 2, "bf16": 2}
WIDTHS = (32, 64, 128, 256)


def _flow(name, nz, ny, nx, storage, collision, wall, steps, every=100, block=1, pack=0,
          porosity=0.57, tau=0.8, magic=3 / 16, u0=0.01):
    c = dict(kind="flow", nz=nz, ny=ny, nx=nx, storage=storage, collision=collision, wall=wall,
             steps=steps, every=every, block=block, pack=pack, porosity=porosity, tau=tau,
             magic=magic, u0=u0)
    return dict(c, name=name) if name else c


def _batch(name, cells, edge, steps=500, every=100, collision="trt", storage="fp32"):
    c = dict(kind="batch", cells=cells, edge=edge, steps=steps, every=every, collision=collision,
             storage=storage)
    return dict(c, name=name) if name else c


def _conv(name, what, n, d, h, w, ci, co):
    c = dict(kind="conv", what=what, n=n, d=d, h=h, w=w, ci=ci, co=co)
    return dict(c, name=name) if name else c


def _net(name, what, n, edge):
    c = dict(kind="net", what=what, n=n, edge=edge)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the plain method: the Stokes cell of the parity runs, where a step takes microseconds
        _flow("cell32_fp64_sbb", 32, 32, 32, "fp64", "trt", "sbb", 100, porosity=0.78),
        # one point of the Darcy-Forchheimer sweep between two of its checks
        _flow("cell128_fp32_cli", 128, 128, 128, "fp32", "trt", "cli", 200, porosity=0.75),
        # MRT on a box of odd edges in 16-bit storage, small enough for the caches
        _flow("ragged_bf16_mrt", 90, 75, 101, "bf16", "mrt", "sbb", 100, pack=5, porosity=0.6),
        # the 2 x 2 x 2 block of the precision study in 16-bit storage, beyond the caches
        _flow("block256_fp16_cli", 256, 256, 256, "fp16", "trt", "cli", 100, block=2, tau=0.5005,
              magic=6e-6, u0=0.002),
        # the same block at full size in FP32, the benchmark's workload
        _flow("block512_fp32_cli", 512, 512, 512, "fp32", "trt", "cli", 20, every=20, block=2,
              tau=0.5005, magic=6e-6, u0=0.002),
        # an interpolated wall rule with two far nodes, on a random pack (wall study)
        _flow("pack160_fp32_mr", 160, 160, 160, "fp32", "trt", "mr", 100, pack=12, porosity=0.5),
        # a monitored FP64 run: drag, permeability and fields every few steps
        _flow("watch_fp64_cli", 96, 128, 144, "fp64", "srt", "cli", 4, every=4, pack=8,
              porosity=0.5),
        # the batch study's one-sphere cells, one device-side stretch of 500 steps
        _batch("batch48x64", 48, 64),
        # the largest layer of the network, forward, at the training minibatch
        _conv("conv96to32_fwd", "forward", 4, 64, 64, 64, 96, 32),
        # a decoder layer's backward: weights, bias and data gradients
        _conv("conv192to64_bwd", "backward", 4, 32, 32, 32, 192, 64),
        # the warm start of one 128^3 evaluation pack
        _net("warm128", "warm", 1, 128),
        # a training step at the minibatch of the training runs
        _net("train64x4", "train", 4, 64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["flow", "flow", "flow", "batch", "conv", "conv", "net"])
    if kind == "flow":
        storage = rng.choice(["fp64", "fp32", "fp32", "fp16", "bf16"])
        walls = ["sbb", "cli", "cli"]
        if storage in ("fp32", "fp64"):
            walls += ["libb", "qibb", "iebb", "mr"]
        edge = _log_int(rng, 20, 320)
        nz, ny, nx = (max(17, int(edge * rng.uniform(0.7, 1.3))) for _ in range(3))
        if rng.random() < 0.4:  # boxes of whole tiles, as simple-cubic cells mostly are
            nz, ny, nx = (32 * max(1, round(v / 32)) for v in (nz, ny, nx))
        cells = nz * ny * nx
        steps = max(2, min(_log_int(rng, 2, 200), int(1.5e9 / cells)))
        return _flow(None, nz, ny, nx, storage, rng.choice(["trt", "trt", "srt", "mrt"]),
                     rng.choice(walls), steps, every=rng.choice([10, 50, 100]),
                     block=rng.choice([1, 2]), pack=rng.choice([0, rng.randint(2, 20)]),
                     porosity=round(rng.uniform(0.45, 0.8), 3),
                     tau=round(rng.uniform(0.6, 1.0), 4))
    if kind == "batch":
        edge = rng.randint(16, 64)
        cells = max(2, min(_log_int(rng, 2, 200), 48 * 64 ** 3 // edge ** 3))
        return _batch(None, cells, edge, every=rng.choice([50, 100]),
                      storage=rng.choice(["fp32", "fp32", "fp64"]) if cells * edge ** 3 < 4e6
                      else "fp32")
    if kind == "conv":
        ci, co, most = rng.choice([(8, 32, 64), (32, 64, 48), (64, 128, 32), (128, 256, 16),
                                   (384, 128, 16), (192, 64, 32), (96, 32, 64), (32, 8, 64)])
        n, e = rng.randint(1, 4), _log_int(rng, 6, most)
        d, h, w = (max(4, min(most, int(e * rng.uniform(0.8, 1.25)))) for _ in range(3))
        if rng.random() < 0.6:  # the network's boxes are multiples of 8
            d, h, w = (8 * max(1, round(v / 8)) for v in (d, h, w))
        return _conv(None, rng.choice(["forward", "backward"]), n, d, h, w, ci, co)
    if rng.random() < 0.5:
        return _net(None, "warm", rng.randint(1, 2), 16 * rng.randint(2, 8))
    return _net(None, "train", rng.randint(1, 4), 8 * rng.randint(2, 8))


# ------------------------------------------------------------------ inputs

def _spheres(case, rng):
    """Rows cx, cy, cz, r: a simple-cubic block at a random offset, or a pack
    of random centres with one radius, for about the case's porosity."""
    nz, ny, nx = case["nz"], case["ny"], case["nx"]
    edges = np.array([nx, ny, nz], np.float64)
    vol = float(np.prod(edges))
    if case["pack"]:
        n = case["pack"]
        c = rng.uniform(0.0, 1.0, (n, 3)) * edges
        r = (-math.log(case["porosity"]) * vol * 3 / (4 * math.pi * n)) ** (1 / 3)
    else:
        b = case["block"]
        at = np.stack(np.meshgrid(*[np.arange(b)] * 3, indexing="ij"), -1).reshape(-1, 3)
        c = ((at / b + rng.uniform(0.0, 1.0, 3)) * edges) % edges
        r = ((1 - case["porosity"]) * vol * 3 / (4 * math.pi * b ** 3)) ** (1 / 3)
    r = min(r * rng.uniform(0.98, 1.0), 0.9 * float(edges.min()))
    return np.hstack([c, np.full((len(c), 1), r)])


def _drop(case):
    """Density drop across the box that keeps the velocity at the scale of u0."""
    return 3.0 * case["nx"] * case["u0"] * (case["tau"] - 0.5) / 3.0 / (0.01 * case["nx"] ** 2)


def _start_fields(shape, u0, gen):
    """(4, cells) float64 on the GPU: density deviation and a swirling mean
    flow with 1% random velocity."""
    nz, ny, nx = shape
    f = torch.zeros((4, nz, ny, nx), dtype=torch.float64, device=DEV)
    ax = [torch.arange(n, dtype=torch.float64, device=DEV) * (2 * math.pi / n) for n in shape]
    z, y, x = ax[0][:, None, None], ax[1][None, :, None], ax[2][None, None, :]
    f[1] += u0 * (1 + 0.3 * torch.sin(y) * torch.cos(z))
    f[2] += 0.3 * u0 * torch.sin(z) * torch.cos(x)
    f[3] += 0.3 * u0 * torch.sin(x) * torch.cos(y)
    f[0] += 0.1 * u0 * torch.cos(x) * torch.sin(y)
    for i in range(3):
        f[1 + i] += 0.01 * u0 * (2 * torch.rand(shape, generator=gen, device=DEV,
                                                dtype=torch.float64) - 1)
    return f.reshape(4, -1)


def _cells_of(case, seed):
    """The batch study's one-sphere cells, at a forcing that keeps |u| small."""
    rng = np.random.default_rng([seed, 7])
    e, out = case["edge"], []
    for _ in range(case["cells"]):
        d = rng.uniform(40.0, 60.0) * e / 64
        c = rng.uniform(0.0, 1.0, 3) * e
        tau = rng.uniform(0.55, 1.0)
        out.append(dict(spheres=[[c[0], c[1], c[2], d / 2]], tau=tau, magic=3 / 16,
                        delta_rho=10 ** rng.uniform(-6, -3)))
    return out


def _mask(spheres, shape, step=1.0, first=0.0):
    """Solid nodes (bool, on the GPU) of periodic spheres; node i of an axis
    sits at first + step * i and the box is step * nodes long."""
    solid = torch.zeros(shape, dtype=torch.bool, device=DEV)
    edges = [step * n for n in shape]
    pos = [first + step * torch.arange(n, dtype=torch.float64, device=DEV) for n in shape]
    for cx, cy, cz, r in np.reshape(spheres, (-1, 4)):
        for oz in (-1, 0, 1):
            dz = pos[0] - (float(cz) + oz * edges[0])
            for oy in (-1, 0, 1):
                dy = pos[1] - (float(cy) + oy * edges[1])
                for ox in (-1, 0, 1):
                    dx = pos[2] - (float(cx) + ox * edges[2])
                    sel = [torch.nonzero(v.abs() < r).flatten() for v in (dz, dy, dx)]
                    if min(len(s) for s in sel) == 0:
                        continue
                    a, b, c = (slice(int(s[0]), int(s[-1]) + 1) for s in sel)
                    solid[a, b, c] |= ((dx[c] * dx[c])[None, None, :] + (dy[b] * dy[b])[None, :, None]
                                       + (dz[a] * dz[a])[:, None, None]) < float(r) * float(r)
    return solid


def _pack_of(case, seed, i):
    """One random pack of 8-27 equal spheres (1-4 for the small training
    cells), porosity about U[0.35, 0.6]."""
    rng = np.random.default_rng([seed, i, 11])
    n = int(rng.integers(8, 28)) if case["what"] == "warm" else int(rng.integers(1, 5))
    e = case["edge"]
    phi = rng.uniform(0.35, 0.6)
    r = (-math.log(phi) * e ** 3 * 3 / (4 * math.pi * n)) ** (1 / 3)
    return np.hstack([rng.uniform(0.0, float(e), (n, 3)), np.full((n, 1), min(r, 0.9 * e))])


def _conv_inputs(case, seed):
    """Post-ReLU activations x, the FP32 gradient dy of the output and the
    layer's own activation, all on the GPU."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    n, d, h, w, ci, co = (case[k] for k in ("n", "d", "h", "w", "ci", "co"))

    def normal(c):
        return torch.randn((n, d, h, w, c), generator=gen, device=DEV)

    x = torch.relu(normal(ci)).to(torch.bfloat16)
    if case["what"] == "forward":
        return x, None, None
    return x, 1e-2 * normal(co), torch.relu(normal(co)).to(torch.bfloat16)


def _layer_weights(case, seed):
    std = math.sqrt(2.0 / (27 * case["ci"]))
    rng = np.random.default_rng([seed, 3])
    return (rng.standard_normal((case["co"], 27, case["ci"])) * std).astype(np.float32)


def _training_inputs(case, seed):
    """Fluid masks, smooth random targets on the fluid, and their weights."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    e, n = case["edge"], case["n"]
    fluid = torch.stack([~_mask(_pack_of(case, seed, i), (e, e, e)) for i in range(n)])
    a = torch.arange(e, device=DEV, dtype=torch.float64) * (2 * math.pi / e)
    t = torch.zeros((n, e, e, e, 4), device=DEV, dtype=torch.float64)
    ph = torch.rand((n, 4, 3), generator=gen, device=DEV, dtype=torch.float64) * 2 * math.pi
    for i in range(n):
        for k in range(4):
            t[i, ..., k] = (torch.sin(a + ph[i, k, 0])[:, None, None] * torch.sin(a + ph[i, k, 1])[None, :, None]
                            + torch.cos(a + ph[i, k, 2])[None, None, :] + (k == 0))
    return fluid, (t * fluid[..., None]).to(torch.float32)


# ----------------------------------------------------------------- the cases

def prepare(case, seed):
    if case["kind"] == "flow":
        shape = (case["nz"], case["ny"], case["nx"])
        d = lbm.Domain(shape, tau=case["tau"], magic=case["magic"], delta_rho=_drop(case),
                       collision=case["collision"], wall=case["wall"], storage=case["storage"],
                       spheres=_spheres(case, np.random.default_rng(seed)),
                       check_interval=case["every"], device=DEV)
        f = _start_fields(shape, case["u0"], torch.Generator(device=DEV).manual_seed(seed))
        if case["storage"] in ("fp32", "fp64"):
            d.init_equilibrium_device(f)
        else:
            f = f.cpu().numpy().reshape((4,) + shape)
            d.init_equilibrium(f[0], f[1:])
        return dict(case=case, d=d)
    if case["kind"] == "batch":
        e = case["edge"]
        b = lbm.Batch((e, e, e), _cells_of(case, seed), collision=case["collision"], wall="cli",
                      storage=case["storage"], check_interval=case["every"], device=DEV)
        # the launch shape that the study's autotuner found for these cells
        b.set_shape(4, 1)
        b.set_solid_writes(2)
        return dict(case=case, b=b)
    if case["kind"] == "conv":
        ctx = warmstart._Ctx(DEV)
        layer = warmstart.Conv(ctx, case["ci"], case["co"], np.random.default_rng([seed, 3]))
        x, dy, act = _conv_inputs(case, seed)
        return dict(case=case, layer=layer, x=x, dy=dy, act=act)
    if case["what"] == "warm":
        net = warmstart.UNet.load(WEIGHTS, device=DEV)
        e = case["edge"]
        packs = [_pack_of(case, seed, i) for i in range(case["n"])]
        fluid = np.stack([(~_mask(p, (e, e, e))).cpu().numpy() for p in packs])
        return dict(case=case, net=net, packs=packs, fluid=fluid)
    fluid, target = _training_inputs(case, seed)
    net = warmstart.UNet(WIDTHS, seed=seed, device=DEV)
    return dict(case=case, net=net, fluid=fluid.to(torch.uint8), target=target,
                norm=4.0 * float(fluid.sum()))


def run(state):
    case = state["case"]
    if case["kind"] == "flow":
        d = state["d"]
        d.run_to_residual(0.0, case["steps"])
        K, U = d.permeability()
        return dict(K=K, U=U, drag=d.drag(), fields=d.macroscopic_device())
    if case["kind"] == "batch":
        b = state["b"]
        b.run_to_residual(0.0, case["steps"])
        r = b.results()
        return dict(U=r["U"], K=r["K_D"], steps=r["steps"], fields=b.macroscopic_device())
    if case["kind"] == "conv":
        layer, shape = state["layer"], tuple(case[k] for k in ("n", "d", "h", "w"))
        if case["what"] == "forward":
            return layer.forward_act(state["x"], shape)
        dx = layer.backward(state["x"], state["dy"], shape, act=state["act"])
        return dict(dx=dx, gw=layer.gw, gb=layer.gb)
    net = state["net"]
    if case["what"] == "warm":
        e, n = case["edge"], case["n"]
        fine = torch.empty((n, e, e, e, 4), dtype=torch.float32, device=DEV)
        for i, p in enumerate(state["packs"]):
            warmstart.predict_two_grid_device(net, p, e, out=fine[i])
        return dict(targets=fine,
                    start=warmstart.warm_fields_device(net.ctx, fine, state["fluid"], 1e-5, 0.8))
    x = warmstart.network_input(net.ctx, state["fluid"])
    out = net.forward(x)
    loss, g = net.loss(out, state["target"], state["fluid"].float(), state["norm"], sync=False)
    net.backward(g)
    net.adam_step(1e-4)
    return dict(out=out, loss=loss, gw=[l.gw for l in net.layers()],
                gb=[l.gb for l in net.layers()])


def _conv_flops(n, d, h, w, ci, co):
    return 2.0 * 27 * n * d * h * w * ci * co


def _net_layers(n, e):
    """(n, edge, ci, co) of the network's eight convolutions."""
    w = WIDTHS
    return [(n, e, 8, w[0]), (n, e // 2, w[0], w[1]), (n, e // 4, w[1], w[2]),
            (n, e // 8, w[2], w[3]), (n, e // 4, w[3] + w[2], w[2]),
            (n, e // 2, w[2] + w[1], w[1]), (n, e, w[1] + w[0], w[0]), (n, e, w[0], 8)]


def work(case):
    if case["kind"] == "flow":
        cells = case["nz"] * case["ny"] * case["nx"]
        fluid = case["porosity"] * cells
        # the steps; then the mean velocity, the fields and (small) the drag
        return dict(bytes=(2.0 * case["steps"] + 2) * 19 * ELEM[case["storage"]] * fluid + 32.0 * cells,
                    flops=250.0 * case["steps"] * fluid)
    if case["kind"] == "batch":
        cells = case["cells"] * case["edge"] ** 3
        fluid = 0.74 * cells  # mean over diameters U[40, 60] in 64^3
        return dict(bytes=(2.0 * case["steps"] + 1) * 19 * ELEM[case["storage"]] * fluid + 32.0 * cells,
                    flops=250.0 * case["steps"] * fluid)
    if case["kind"] == "conv":
        m = case["n"] * case["d"] * case["h"] * case["w"]
        ci, co = case["ci"], case["co"]
        f = _conv_flops(case["n"], case["d"], case["h"], case["w"], ci, co)
        if case["what"] == "forward":
            return dict(bytes=2.0 * m * (ci + co) + 54.0 * ci * co, flops=f)
        return dict(bytes=m * (2.0 * ci + 6.0 * co + 4.0 * ci) + 27 * 6.0 * ci * co, flops=2 * f)
    if case["what"] == "warm":
        n, e = case["n"], case["edge"]
        f = sum(_conv_flops(a, b, b, b, c, d) for a, b, c, d in _net_layers(n, e // 2))
        return dict(bytes=n * e ** 3 * (16.0 + 1 + 32), flops=f)
    n, e = case["n"], case["edge"]
    layers = _net_layers(n, e)
    f = 3 * sum(_conv_flops(a, b, b, b, c, d) for a, b, c, d in layers) \
        - _conv_flops(n, e, e, e, 8, WIDTHS[0])
    # activations written once and read by the backward pass; the output,
    # its target and gradient; weights, gradients and both Adam moments
    act = sum(4.0 * a * b ** 3 * d for a, b, c, d in layers)
    return dict(bytes=act + n * e ** 3 * 80.0 + 28.0 * sum(27 * c * d for _, _, c, d in layers),
                flops=f)


# ------------------------------------------------- the same in 64-bit torch

E19 = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1),
       (1, 1, 0), (-1, 1, 0), (1, -1, 0), (-1, -1, 0), (1, 0, 1), (-1, 0, 1), (1, 0, -1),
       (-1, 0, -1), (0, 1, 1), (0, -1, 1), (0, 1, -1), (0, -1, -1)]
W19 = [{0: 1 / 3, 1: 1 / 18, 2: 1 / 36}[sum(map(abs, e))] for e in E19]
OPP = [E19.index((-x, -y, -z)) for x, y, z in E19]


def _shift(t, e, m=1):
    """t at x - m e (periodic, last three axes)."""
    return torch.roll(t, (m * e[2], m * e[1], m * e[0]), dims=(-3, -2, -1))


def _distance(spheres, edges, pos, e):
    """First crossing (fraction of the link) with a sphere image, from nodes
    pos (n, 3) along e; 1/2 where none is found."""
    best = torch.full((len(pos),), 2.0, dtype=torch.float64, device=DEV)
    ev = torch.tensor(e, dtype=torch.float64, device=DEV)
    a = float(sum(v * v for v in e))
    for cx, cy, cz, r in np.reshape(spheres, (-1, 4)):
        for o in np.ndindex(3, 3, 3):
            c = [float(v) + (k - 1) * n for v, k, n in zip((cx, cy, cz), o, edges)]
            near = torch.ones(len(pos), dtype=torch.bool, device=DEV)
            for i in range(3):
                near &= (pos[:, i] - c[i]).abs() <= r + 1.0
            at = torch.nonzero(near).flatten()
            if not len(at):
                continue
            dl = pos[at] - torch.tensor(c, dtype=torch.float64, device=DEV)
            h = dl @ ev
            c0 = (dl * dl).sum(1) - float(r) ** 2
            disc = h * h - a * c0
            sq = torch.sqrt(disc.clamp(min=0))
            t = torch.where(h < 0, c0 / (sq - h), (-h - sq) / a)
            ok = (disc >= 0) & (t >= 0) & (t <= 1)
            best[at] = torch.where(ok, torch.minimum(best[at], t), best[at])
    return torch.where(best <= 1, best, torch.full_like(best, 0.5))


class _Plain:
    """D3Q19 in 64 bits: deviations g[k] of shape (cells, nz, ny, nx), boxes
    periodic each on its own; tau, magic and the density drop per box."""

    def __init__(self, boxes, shape, collision, wall, tau, magic, drop, fields):
        self.shape, self.wall, self.collision = shape, wall, collision
        nz, ny, nx = shape
        n = len(boxes)

        def per_box(v):
            return torch.tensor(v, dtype=torch.float64, device=DEV).reshape(n, 1, 1, 1)

        self.tau, self.drop = per_box(tau), per_box(drop)
        self.wp = 1 / self.tau
        self.wm = 1 / (0.5 + per_box(magic) / (self.tau - 0.5)) if collision == "trt" else self.wp
        self.solid = torch.stack([_mask(s, shape) for s in boxes])
        self.links = []  # per pull direction k: flat nodes, wall distance, far nodes, fallbacks
        flat = self.solid.reshape(-1)
        for k in range(1, 19):
            e, j = E19[k], OPP[k]
            at = torch.nonzero((~self.solid & _shift(self.solid, e)).reshape(-1)).flatten()
            b, r = at // (nz * ny * nx), at % (nz * ny * nx)
            z, y, x = r // (ny * nx), r // nx % ny, r % nx
            q = torch.empty(len(at), dtype=torch.float64, device=DEV)
            pos = torch.stack([x, y, z], 1).double()
            for i in range(n) if wall != "sbb" else []:
                mine = torch.nonzero(b == i).flatten()
                if len(mine):
                    q[mine] = _distance(boxes[i], (nx, ny, nz), pos[mine], E19[j])
            far = []
            for m in (1, 2):
                X = x + m * e[0]
                node = ((b * nz + (z + m * e[2]) % nz) * ny + (y + m * e[1]) % ny) * nx + X % nx
                far.append((node, (X >= nx).double() - (X < 0).double()))
            f2 = ~flat[far[0][0]]
            f3 = f2 & ~flat[far[1][0]]
            self.links.append((k, at, b, q, far, f2, f3))
        f = fields.reshape((4, n) + tuple(shape))
        f = torch.where(self.solid[None], torch.zeros_like(f), f) if f.numel() < 2 ** 28 else f
        usq = f[1] ** 2 + f[2] ** 2 + f[3] ** 2
        self.g = [self._geq(k, f[0], f[1:], usq) for k in range(19)]
        for g in self.g:
            g[self.solid] = 0
        if collision == "mrt":
            self._basis()

    def _geq(self, k, rho, u, usq):
        e = E19[k]
        eu = sum(float(c) * v for c, v in zip(e, u) if c) if k else torch.zeros_like(rho)
        return W19[k] * (rho + 3 * eu + 4.5 * eu * eu - 1.5 * usq)

    def _basis(self):
        """d'Humieres' moments with the rates of eq. (MRT): viscous 1/tau, the
        energy pair by 4.6, the rest Pan's s_zeta."""
        M = np.zeros((19, 19))
        for k, (x, y, z) in enumerate(E19):
            e2 = x * x + y * y + z * z
            M[:, k] = [1, 19 * e2 - 30, (21 * e2 * e2 - 53 * e2 + 24) / 2, x, (5 * e2 - 9) * x, y,
                       (5 * e2 - 9) * y, z, (5 * e2 - 9) * z, 3 * x * x - e2,
                       (3 * e2 - 5) * (3 * x * x - e2), y * y - z * z,
                       (3 * e2 - 5) * (y * y - z * z), x * y, y * z, x * z, (y * y - z * z) * x,
                       (z * z - x * x) * y, (x * x - y * y) * z]
        tau = float(self.tau.flatten()[0])
        s_nu, s_e = 1 / tau, 1 / (0.5 + (tau - 0.5) / 4.6)
        s_z = 8 * (2 - s_nu) / (8 - s_nu)
        S = np.full(19, s_z)
        S[[9, 11, 13, 14, 15]] = s_nu
        S[[1, 2]] = s_e
        S[[0, 3, 5, 7]] = 0
        self.R = np.linalg.inv(M) @ np.diag(S) @ M

    def moments(self, g):
        rho = sum(g[1:], g[0].clone())
        u = []
        for i in range(3):
            v = torch.zeros_like(rho)
            for k in range(1, 19):
                if E19[k][i]:
                    v.add_(g[k], alpha=float(E19[k][i]))
            u.append(v)
        return rho, u

    def wall_values(self):
        """Per link list: (k, nodes, the value the rule gives for direction k)."""
        g = [v.reshape(-1) for v in self.g]
        if self.wall == "iebb":
            rho, u = self.moments(self.g)
            rho, u = rho.reshape(-1), [v.reshape(-1) for v in u]
        out = []
        for k, at, b, q, far, f2, f3 in self.links:
            j = OPP[k]
            jw = W19[k] * self.drop.flatten()[b]
            own_j, own_k = g[j][at], g[k][at]

            def read(kk, m):
                node, cross = far[m - 1]
                return g[kk][node] - cross * jw

            if self.wall == "sbb":
                v = own_j
            else:
                f2j = read(j, 1)
                a = torch.where(f2, (1 - 2 * q) / (1 + 2 * q), torch.zeros_like(q))
                cli = a * f2j - a * own_k + own_j
                libb = torch.where(q < 0.5,
                                   torch.where(f2, (1 - 2 * q) * f2j + 2 * q * own_j, own_j),
                                   (1 - 1 / (2 * q)) * own_k + own_j / (2 * q))
                if self.wall == "cli":
                    v = cli
                elif self.wall == "libb":
                    v = libb
                elif self.wall == "qibb":
                    lo = (q * (1 + 2 * q) * own_j + (1 - 4 * q * q) * f2j
                          - q * (1 - 2 * q) * read(j, 2))
                    hi = ((2 * q - 1) / q * own_k + own_j / (q * (2 * q + 1))
                          + (1 - 2 * q) / (2 * q + 1) * read(k, 1))
                    v = torch.where(q < 0.5, torch.where(f3, lo, libb), torch.where(f2, hi, libb))
                elif self.wall == "mr":
                    d = (1 + q) ** 2
                    k1, k2 = (1 - 2 * q - 2 * q * q) / d, q * q / d
                    mr = (k1 * f2j + k2 * read(j, 2) - k1 * own_k - k2 * read(k, 1) + own_j)
                    v = torch.where(f3, mr, cli)
                else:
                    tau = self.tau.flatten()[b]
                    near = far[0][0]
                    e = E19[j]
                    w = torch.where(q < 0.5, torch.ones_like(q), 1 - 3 / (2 * q))
                    ubf = [torch.where(q < 0.5, t[near], w * t[at]) for t in u]
                    X = (2 * q - 1) / torch.where(q < 0.5, tau - 2, tau + 0.5)
                    eub = sum(float(c) * t for c, t in zip(e, ubf))
                    eu1 = sum(float(c) * t[at] for c, t in zip(e, u))
                    uu = sum(t[at] ** 2 for t in u)
                    fs = W19[j] * (rho[at] + 3 * eub + 4.5 * eu1 * eu1 - 1.5 * uu)
                    v = torch.where((q < 0.5) & ~f2, own_j, (1 - X) * own_j + X * fs)
            out.append((k, at, v))
        return out

    def step(self):
        walls = self.wall_values()
        for k in range(1, 19):
            e = E19[k]
            t = _shift(self.g[k], e)
            if e[0] == 1:
                t[..., 0] += W19[k] * self.drop[..., 0]
            elif e[0] == -1:
                t[..., -1] -= W19[k] * self.drop[..., 0]
            self.g[k] = t
        for k, at, v in walls:
            self.g[k].reshape(-1)[at] = v
        g = self.g
        rho, u = self.moments(g)
        usq = u[0] ** 2 + u[1] ** 2 + u[2] ** 2
        if self.collision == "mrt":
            d = [g[k] - self._geq(k, rho, u, usq) for k in range(19)]
            for k in range(19):
                for i in range(19):
                    if abs(self.R[k, i]) > 1e-14:
                        g[k].add_(d[i], alpha=-float(self.R[k, i]))
        else:
            g[0].sub_(self.wp * (g[0] - W19[0] * (rho - 1.5 * usq)))
            for k in range(1, 19):
                j = OPP[k]
                if j < k:
                    continue
                e = E19[k]
                eu = sum(float(c) * v for c, v in zip(e, u) if c)
                dp = self.wp * (0.5 * (g[k] + g[j]) - W19[k] * (rho + 4.5 * eu * eu - 1.5 * usq))
                dm = self.wm * (0.5 * (g[k] - g[j]) - 3 * W19[k] * eu)
                g[k].sub_(dp).sub_(dm)
                g[j].sub_(dp).add_(dm)
        for v in g:
            v[self.solid] = 0

    def fields(self):
        rho, u = self.moments(self.g)
        return torch.stack([rho] + u).reshape(4, -1)

    def mean_velocity(self):
        _, u = self.moments(self.g)
        return torch.stack([v.sum((1, 2, 3)) for v in u], 1) / float(np.prod(self.shape))

    def drag(self):
        F = np.zeros(3)
        for k, at, v in self.wall_values():
            j = OPP[k]
            tot = float((self.g[j].reshape(-1)[at] + v + 2 * W19[k]).sum())
            F += np.array(E19[j]) * tot
        return F


def _bf(t):
    return t.to(torch.bfloat16).double()


def _taps():
    return [(t, (t // 9 - 1, t // 3 % 3 - 1, t % 3 - 1)) for t in range(27)]


def _at_tap(x, o):
    """x at v + o (periodic) over the axes of a channels-last box."""
    return torch.roll(x, (-o[0], -o[1], -o[2]), dims=(1, 2, 3))


def _conv_plain(x, w, b):
    y = torch.zeros(x.shape[:-1] + (w.shape[0],), dtype=torch.float64, device=DEV)
    for t, o in _taps():
        y += (_at_tap(x, o).reshape(-1, x.shape[-1]) @ w[:, t].T).reshape(y.shape)
    return y + b


def _conv_back_plain(x, w, dy, act, need_dx=True):
    """(dx, gw, gb): the ReLU's gradient, whose BF16 rounding is the operand
    of both convolution gradients."""
    dz = torch.where(act > 0, dy, torch.zeros_like(dy)) if act is not None else dy
    gb = dz.reshape(-1, dz.shape[-1]).sum(0)
    dzb = _bf(dz)
    gw, dx = torch.empty_like(w), torch.zeros_like(x) if need_dx else None
    for t, o in _taps():
        gw[:, t] = dzb.reshape(-1, dzb.shape[-1]).T @ _at_tap(x, o).reshape(-1, x.shape[-1])
        if need_dx:
            r = _at_tap(dzb, (-o[0], -o[1], -o[2]))
            dx += (r.reshape(-1, r.shape[-1]) @ w[:, t]).reshape(dx.shape)
    return dx, gw, gb


def _pool_plain(x):
    n, d, h, w, c = x.shape
    return x.reshape(n, d // 2, 2, h // 2, 2, w // 2, 2, c).mean((2, 4, 6))


def _spread(x):
    return x.repeat_interleave(2, 1).repeat_interleave(2, 2).repeat_interleave(2, 3)


def _gather(x):
    return 8 * _pool_plain(x)


class _PlainNet:
    """The four-level network with activations rounded to BF16 between layers."""

    def __init__(self, weights, biases):
        self.w, self.b = weights, biases

    def forward(self, x):
        self.inp, self.out = [], []

        def layer(i, v):
            self.inp.append(v)
            y = _conv_plain(v, self.w[i], self.b[i])
            self.out.append(_bf(torch.relu(y)) if i < 7 else y)
            return self.out[-1]

        e, cur = [], x
        for lvl in range(4):
            cur = layer(lvl, cur if lvl == 0 else _bf(_pool_plain(cur)))
            e.append(cur)
        for i, lvl in enumerate((2, 1, 0)):
            cur = layer(4 + i, torch.cat([_spread(cur), e[lvl]], -1))
        return layer(7, cur)

    def backward(self, g):
        gw, gb, skip = [None] * 8, [None] * 8, {}

        def layer(i, g, need=True):
            dx, gw[i], gb[i] = _conv_back_plain(self.inp[i], self.w[i], g,
                                                self.out[i] if i < 7 else None, need)
            return dx

        g = layer(7, g)
        for lvl in range(3):
            d = layer(6 - lvl, g)
            up = WIDTHS[lvl + 1]
            skip[lvl] = d[..., up:]
            g = _gather(d[..., :up])
        for lvl in (3, 2, 1, 0):
            if lvl < 3:
                g = g + skip[lvl]
            g = layer(lvl, g, lvl > 0)
            if lvl > 0:
                g = _spread(g) / 8
        return gw, gb


def _fresh_weights(seed):
    rng = np.random.default_rng(seed)
    out = []
    for i, (_, _, ci, co) in enumerate([_net_layers(1, 8)[k] for k in range(8)]):
        w = (rng.standard_normal((co, 27, ci)) * np.sqrt(2.0 / (27 * ci))).astype(np.float32)
        t = torch.from_numpy(w).to(DEV) * (0.1 if i == 7 else 1.0)
        out.append(_bf(t))
    return out


def _prolong_plain(t):
    out = t
    for ax in range(3):
        even = 0.75 * out + 0.25 * torch.roll(out, 1, ax)
        odd = 0.75 * out + 0.25 * torch.roll(out, -1, ax)
        out = torch.stack([even, odd], ax + 1).flatten(ax, ax + 1)
    return out


def exact(case, seed):
    if case["kind"] == "flow":
        shape = (case["nz"], case["ny"], case["nx"])
        f = _start_fields(shape, case["u0"], torch.Generator(device=DEV).manual_seed(seed))
        p = _Plain([_spheres(case, np.random.default_rng(seed))], shape, case["collision"],
                   case["wall"], [case["tau"]], [case["magic"]], [_drop(case)], f)
        del f
        for _ in range(case["steps"]):
            p.step()
        U = float(p.mean_velocity()[0, 0])
        return dict(K=(case["tau"] - 0.5) / 3 * U * case["nx"] / (_drop(case) / 3), U=U,
                    drag=p.drag(), fields=p.fields())
    if case["kind"] == "batch":
        cells, e = _cells_of(case, seed), case["edge"]
        p = _Plain([c["spheres"] for c in cells], (e, e, e), case["collision"], "cli",
                   [c["tau"] for c in cells], [c["magic"] for c in cells],
                   [c["delta_rho"] for c in cells],
                   torch.zeros((4, len(cells) * e ** 3), dtype=torch.float64, device=DEV))
        for _ in range(case["steps"]):
            p.step()
        U = p.mean_velocity().cpu().numpy()
        nu = np.array([(c["tau"] - 0.5) / 3 for c in cells])
        drop = np.array([c["delta_rho"] for c in cells])
        return dict(U=U, K=nu * U[:, 0] * e / (drop / 3), steps=None, fields=p.fields())
    if case["kind"] == "conv":
        x, dy, act = _conv_inputs(case, seed)
        w = _bf(torch.from_numpy(_layer_weights(case, seed)).to(DEV))
        if case["what"] == "forward":
            return torch.relu(_conv_plain(x.double(), w, 0.0))
        dx, gw, gb = _conv_back_plain(x.double(), w, dy.double(), act.double())
        return dict(dx=dx, gw=gw, gb=gb)
    if case["what"] == "warm":
        z = np.load(WEIGHTS)
        bits = [np.ascontiguousarray(z["w%d" % i].astype(np.uint32) << 16).view(np.float32)
                for i in range(8)]
        net = _PlainNet([torch.from_numpy(b).to(DEV).double() for b in bits],
                        [torch.from_numpy(z["b%d" % i]).to(DEV).double() for i in range(8)])
        e, n = case["edge"], case["n"]
        scale = float(z["scale"]) * torch.tensor([4.0, 4.0, 4.0, 2.0], dtype=torch.float64, device=DEV)
        fine, start = [], []
        for i in range(n):
            pack = _pack_of(case, seed, i)
            coarse = ~_mask(pack, (e // 2,) * 3, step=2.0, first=0.5)
            x = torch.zeros((1,) + coarse.shape + (8,), dtype=torch.float64, device=DEV)
            x[0, ..., 0] = coarse
            fine.append(_prolong_plain(net.forward(x)[0, ..., :4]) * scale)
            solid = _mask(pack, (e, e, e))
            wall = torch.zeros_like(solid)
            for k in range(1, 19):
                wall |= _shift(solid, E19[k])
            xc = torch.arange(e, dtype=torch.float64, device=DEV) - (e - 1) / 2
            rho = torch.where(solid, torch.zeros((), dtype=torch.float64, device=DEV), -(1e-5 / e) * xc)
            u = fine[-1][..., :3] * ((1e-5 / (3 * e)) / ((0.8 - 0.5) / 3))
            u = torch.where((solid | wall)[..., None], torch.zeros_like(u), u)
            start.append(torch.cat([rho[None], u.permute(3, 0, 1, 2)]).reshape(4, 1, -1))
        return dict(targets=torch.stack(fine), start=torch.cat(start, 1).reshape(4, -1))
    fluid, target = _training_inputs(case, seed)
    net = _PlainNet(_fresh_weights(seed), [0.0] * 8)
    x = torch.zeros(fluid.shape + (8,), dtype=torch.float64, device=DEV)
    x[..., 0] = fluid
    out = net.forward(x)
    norm = 4.0 * float(fluid.sum())
    diff = (out[..., :4] - target.double()) * fluid[..., None]
    g = torch.zeros_like(out)
    g[..., :4] = 2 * diff / norm
    gw, gb = net.backward(g)
    return dict(out=out, loss=(diff ** 2).sum() / norm, gw=gw, gb=gb)
