"""Performance cases of the block-multiresolution solver: the calls a simulation makes.

Each case is a plain dict.  ``prepare`` builds what a program holds before the call (a
:class:`Solver` with its pool, a forest, block data on the GPU, or a predictor's samples and
weights), ``run`` is one pass through the public entry points, ``work`` the bytes and
operations the pass cannot do without, and ``exact`` the same results from dense per-level
arrays in plain torch FP64, without the library.

Kinds of case
  rk4      a time loop on a fixed grid: load the state, ``steps`` RK4 steps, read back
  step     multiresolution steps: set the grid and the state, ``steps`` steps (refine-all,
           RK4, adapt), read back the grid and the state
  analyse  one multiresolution analysis (flags and detail maxima)
  train    one epoch of the refinement predictor (forward, backward, Adam)
  forward  the predictor's logits for a set of feature rows

Grids: every block at level ``base``, refined up to level ``jmax`` towards a few centres (a
strip around the layers for Navier-Stokes) within ``radius``, halved from level to level, and
graded.  A seed moves the whole pattern (for a multiresolution step by half the domain, which
keeps the families, and not at all in the swirl, whose velocity does not move with it) and
draws the sign and, in its last digits, the amplitude, so the block count, also the one a
step's thresholds leave, depends on the case alone.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1902_00088_amd as M
import workloads as W

# ---------------------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------------------

_KEYS = ("kind", "physics", "dim", "bs", "base", "jmax", "radius", "centres", "precision", "steps", "eps", "beta",
         "sweep", "tuned")


def _grid_case(name, *values):
    return dict(zip(_KEYS, values), name=name)


def listed():
    return [
        # the smallest call: a few 17 x 17 blocks on three levels (the constant-advection set-up
        # the tests step through), four RK4 steps on a fixed grid, FP64; launches and latency
        _grid_case("advect 2D 17, small, FP64", "rk4", "const", 2, 17, 2, 4, 0.1, 1, "fp64", 4, 0.0, 0.005, 2, False),
        # the headline run: three blobs in the steady swirl on 16 blocks, every step refining to
        # 64 and coarsening back, mixed precision, schedule chosen by the autotuner
        _grid_case("swirl 2D cycling, mixed", "step", "swirl", 2, 33, 2, 7, 0.0, 3, "mixed", 50, 1e-4, 0.01, 2, True),
        # the swirl study's adaptive runs (narrow pulse, FP64, one-launch steps where the grid
        # allows): a ragged grid of several hundred blocks
        _grid_case("swirl 2D adaptive, FP64", "step", "swirl", 2, 33, 3, 7, 0.13, 4, "fp64", 8, 1e-5, 1e-4, 3, False),
        # the swirl study's equidistant runs: every block on the finest level, FP64
        _grid_case("swirl 2D equidistant, FP64", "step", "swirl", 2, 33, 6, 6, 0.0, 1, "fp64", 4, 0.0, 1e-3, 3, False),
        # RK4 on the 3D benchmark's kind of grid (about 3,000 blocks of 17^3 on three levels),
        # mixed precision and FP64
        _grid_case("advect 3D, mixed", "rk4", "const", 3, 17, 3, 5, 0.13, 4, "mixed", 4, 0.0, 0.0032, 2, False),
        _grid_case("advect 3D, FP64", "rk4", "const", 3, 17, 3, 5, 0.13, 4, "fp64", 2, 0.0, 0.0032, 2, False),
        # whole multiresolution steps in 3D, mixed precision, topology planned on the device
        _grid_case("advect 3D step, mixed", "step", "const", 3, 17, 3, 5, 0.02, 4, "mixed", 8, 1e-4, 0.0032, 2, False),
        # the Navier-Stokes mixing layer: 64 blocks refining to 256 and back, mixed, autotuned
        _grid_case("mixing layer, mixed", "step", "layer", 2, 33, 3, 8, 0.0, 0, "mixed", 10, 1e-3, 0.0, 2, True),
        # the double shear layer with its filter on an adaptive grid of a few thousand blocks
        _grid_case("shear layer, mixed", "step", "shear", 2, 33, 4, 7, 0.05, 0, "mixed", 6, 1e-4, 0.0, 2, False),
        # Navier-Stokes RK4 in FP64 on a ragged grid
        _grid_case("shear layer RK4, FP64", "rk4", "shear", 2, 33, 4, 6, 0.08, 0, "fp64", 2, 0.0, 0.0, 2, False),
        # one analysis of a 3D grid: details, flags and maxima of every block
        _grid_case("analysis 3D", "analyse", "const", 3, 17, 3, 5, 0.13, 4, "fp64", 1, 1e-4, 0.0032, 2, False),
        # one epoch of the predictor on recorded features of the four-field mixing layer
        {"name": "predictor epoch", "kind": "train", "fields": 4, "samples": 16384, "batch": 1024},
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(("rk4", "rk4", "rk4", "step", "step", "step", "analyse", "analyse", "train", "forward"))
    if kind in ("train", "forward"):
        n = log_int(37, 16384)
        return {"kind": kind, "fields": rng.choice((1, 4)), "samples": n, "batch": rng.choice((128, 500, 1024))}
    physics = rng.choice(("const2", "const3", "const3", "swirl", "layer", "shear"))
    precision = rng.choice(("fp64", "mixed"))
    radius = rng.uniform(0.02, 0.16)
    steps = rng.randint(1, 3)
    tuned = False
    centres = rng.randint(1, 4)
    eps = rng.choice((1e-3, 1e-4, 1e-5))
    sweep = 2
    bs = 33
    if physics == "const2":
        bs = rng.choice((17, 33))
        base = rng.randint(1, 4)
        beta = rng.uniform(0.003, 0.01)
        jmax = base + rng.randint(0, 2)
    elif physics == "swirl":
        base = rng.randint(2, 5)
        beta = rng.uniform(0.0002, 0.01)
        jmax = min(6, base + rng.randint(0, 2))
        sweep = rng.choice((2, 3))
    elif physics == "const3":
        bs = 17
        base = rng.randint(1, 3)
        jmax = min(5, base + rng.randint(0, 2))
        beta = rng.uniform(0.0032, 0.01)
        radius = min(radius, 0.1)
    else:
        base = rng.randint(2, 4)
        jmax = min(6, base + rng.randint(0, 2))
        beta = 0.0
        centres = 0
    jmax = max(jmax, 2)
    if kind == "step" and rng.random() < 0.5:
        jmax = min(jmax + 1, 5 if physics == "const3" else 6)   # head room for the safety zone
    if kind == "step" and physics == "const3":
        radius = min(radius, 0.03)
    dim = 3 if physics == "const3" else 2
    return dict(zip(_KEYS, (kind, physics[:5], dim, bs, base, jmax, round(radius, 4), centres, precision, steps, eps,
                            round(beta, 5), sweep, tuned)))


# ---------------------------------------------------------------------------------------
# grids, configurations and initial data
# ---------------------------------------------------------------------------------------

# relative positions of the centres (a seed shifts them by whole base blocks)
_CENTRES = np.array([[0.52, 0.47, 0.55], [0.31, 0.66, 0.40], [0.71, 0.28, 0.33], [0.58, 0.74, 0.69]])
_LAYERS = {"layer": (0.25, 0.75), "shear": (0.5 - 0.25 / 8.0, 0.5 + 0.25 / 8.0)}


def _near(case, level):
    """Blocks of `level` within the level's radius of a centre (or of a layer): boolean [2^level]*dim, x last."""
    nb, dim = 2 ** level, case["dim"]
    r = case["radius"] * 0.5 ** (level - case["base"])
    if r <= 0.0:
        return np.zeros((nb,) * dim, dtype=bool)

    def gap(c):   # periodic distance of a coordinate to each block's interval
        mid = (np.arange(nb) + 0.5) / nb
        d = np.abs(mid - c)
        return np.maximum(np.minimum(d, 1.0 - d) - 0.5 / nb, 0.0)

    out = np.zeros((nb,) * dim, dtype=bool)
    if case["physics"] in _LAYERS:
        for y in _LAYERS[case["physics"]]:
            out |= (gap(y) < r)[:, None]
        return out
    for c in _CENTRES[:case["centres"]]:
        d2 = 0.0
        for a in range(dim):
            shape = [1] * dim
            shape[dim - 1 - a] = nb
            d2 = d2 + gap(c[a]).reshape(shape) ** 2
        out |= d2 < r * r
    return out


def _leaf_maps(case):
    """Leaf maps of the case's grid, unshifted: {level: boolean [2^level]*dim, x last}."""
    dim, base = case["dim"], case["base"]
    # in a multiresolution step's grid the finest level is left for the safety zone
    top = case["jmax"] if case["kind"] != "step" else max(base, case["jmax"] - 1)
    refined = {}
    for l in range(top - 1, 0, -1):
        m = np.ones((2 ** l,) * dim, dtype=bool) if l < base else _near(case, l)
        if l + 1 in refined:
            f = refined[l + 1]
            for a in range(dim):   # a refined block's neighbours have to exist on its level
                f = f | np.roll(f, 1, a) | np.roll(f, -1, a)
            for a in range(dim):
                f = f.reshape(f.shape[:a] + (f.shape[a] // 2, 2) + f.shape[a + 1:]).any(axis=a + 1)
            m = m | f
        refined[l] = m
    leaves = {}
    for l in range(1, top + 1):
        here = np.ones((2 ** l,) * dim, dtype=bool)
        if l > 1:
            here = refined[l - 1]
            for a in range(dim):
                here = np.repeat(here, 2, axis=a)
        leaf = here & ~refined[l] if l in refined else here
        if leaf.any():
            leaves[l] = leaf
    return leaves


def _shift(case, seed):
    rng = np.random.default_rng([seed, 11])
    off = rng.integers(0, 2 ** case["base"], size=case["dim"])
    if case["kind"] == "step":
        off = (off & 1) << (case["base"] - 1)
        if case["physics"] == "swirl":
            off = 0 * off
    return off, rng


def _forest(case, seed):
    off, _ = _shift(case, seed)
    lv, co = [], []
    for l, m in _leaf_maps(case).items():
        for a in range(case["dim"]):
            step = int(off[a]) << (l - case["base"]) if l >= case["base"] else 0
            m = np.roll(m, step, axis=case["dim"] - 1 - a)
        c = np.argwhere(m)[:, ::-1]
        lv.append(np.full(len(c), l, dtype=np.int8))
        co.append(c.astype(np.int32))
    return np.concatenate(lv), np.ascontiguousarray(np.concatenate(co))


def _morton_order(case, levels, coords):
    """Forest order: Morton key of the coordinates on the finest level, x least significant."""
    key = np.zeros(len(levels), dtype=np.uint64)
    fine = coords.astype(np.uint64) << (case["jmax"] - levels.astype(np.int64)).astype(np.uint64)[:, None]
    for bit in range(case["jmax"]):
        for a in range(case["dim"]):
            key |= ((fine[:, a] >> np.uint64(bit)) & np.uint64(1)) << np.uint64(bit * case["dim"] + a)
    return np.argsort(key, kind="stable")


def _config(case, blocks):
    prec = W.MIXED if case["precision"] == "mixed" else W.FP64
    ns = case["physics"] in _LAYERS
    make = {"const": W.C1 if case["dim"] == 2 else W.C4, "swirl": W.C2, "layer": W.C3, "shear": W.DSL}[case["physics"]]
    cfg = make(jmax=max(2, case["jmax"]), eps=case["eps"])
    room = blocks + 64
    if case["kind"] == "step":
        room = max(64, 3 * blocks * 2 ** case["dim"])
    kw = dict(precision=prec, form=W.FORM_FUSED, max_blocks=room, bs=case["bs"])
    if not ns:
        kw["dt"] = 0.5 / (2 ** cfg.jmax * (case["bs"] - 1))
    return cfg.replace(**kw)


def _fields(case, seed, x):
    """Initial fields at the coordinates x[a] (broadcastable, unit domain): [nf] tensors."""
    off, rng = _shift(case, seed)
    rel = [(x[a] - float(off[a]) / 2 ** case["base"]) % 1.0 for a in range(case["dim"])]
    amp = (1.0 + 1e-6 * float(rng.uniform(-1.0, 1.0))) * (1.0 if rng.random() < 0.5 else -1.0)
    if case["physics"] in ("const", "swirl"):
        val = 0.0
        for c in _CENTRES[:max(1, case["centres"])]:
            prod = amp
            for a in range(case["dim"]):
                g = 0.0
                for m in (-1.0, 0.0, 1.0):
                    g = g + torch.exp(-((rel[a] - float(c[a]) - m) ** 2) / case["beta"])
                prod = prod * g
            val = val + prod
        return [val]
    px, py = rel
    theta = np.random.default_rng(3).uniform(0.0, 2.0 * math.pi, 8).tolist()
    y1, y2 = _LAYERS[case["physics"]]
    zero = torch.zeros_like(px + py)
    s = 0.0
    for k in range(1, 9):
        s = s + torch.sin(2.0 * math.pi * k * px + theta[k - 1]) / 8.0
    if case["physics"] == "layer":
        delta = 0.02
        u = 0.5 * (torch.tanh(2.0 * (py - y1) / delta) - torch.tanh(2.0 * (py - y2) / delta) - 1.0)
        env = torch.exp(-((py - y1) / (4 * delta)) ** 2) + torch.exp(-((py - y2) / (4 * delta)) ** 2)
        return [zero + 1.0, u + zero, 1e-3 * amp * s * env, zero + 1.25 * 1.25 / 1.4]
    step = 0.5 * (torch.tanh(240.0 * (py - y1)) - torch.tanh(240.0 * (py - y2)))
    wave = torch.sin(2.0 * math.pi * W.DSL_L * (px - 0.5)) + 0.05 * s
    return [1.0 + step + zero, 2.0 * step - 1.0 + zero, 0.1 * amp * wave + zero, zero + 2.5]


def _sample(case, seed, levels, coords, device):
    """Fields at every node of the given blocks: float64 [n, nf, bs^dim] on `device`."""
    dim, bs, n = case["dim"], case["bs"], len(levels)
    lv = torch.as_tensor(levels.astype(np.int64), device=device)
    co = torch.as_tensor(coords.astype(np.int64), device=device)
    nl = (2 ** lv) * (bs - 1)
    node = torch.arange(bs, device=device)
    x = []
    for a in range(dim):
        shape = [n] + [1] * dim
        shape[dim - a] = bs
        x.append((((co[:, a:a + 1] * (bs - 1) + node) % nl[:, None]).double() / nl[:, None].double()).reshape(shape))
    f = _fields(case, seed, x)
    full = (n,) + (bs,) * dim
    return torch.stack([v.expand(full).reshape(n, bs ** dim) for v in f], dim=1).contiguous()


# ---------------------------------------------------------------------------------------
# prepare, run, work
# ---------------------------------------------------------------------------------------

def _samples(case, seed):
    """Feature rows of recorded blocks (a mean level per field and smooth bins), labels, class
    weights and initial parameters."""
    rng = np.random.default_rng([seed, 12])
    n, nf = case["samples"], case["fields"]
    mean = np.linspace(1.0, 0.0, nf) if nf > 1 else np.array([0.2])
    slope = rng.normal(size=(n, nf, 1, 2))
    b = (np.arange(64) % 8 - 3.5) / 8.0
    c = (np.arange(64) // 8 - 3.5) / 8.0
    x = mean[None, :, None] + 0.3 * rng.normal(size=(n, nf, 1)) + slope[..., 0] * b + slope[..., 1] * c
    x = (x + 0.02 * rng.normal(size=(n, nf, 64))).astype(np.float32)
    steep = np.abs(slope).sum(axis=(1, 2, 3))
    y = np.where(steep > np.quantile(steep, 0.8), 0, np.where(steep < np.quantile(steep, 0.3), 2, 1)).astype(np.int8)
    return {"x": x.reshape(n, nf * 64), "y": y, "mean": x.mean(axis=(0, 2)), "std": x.std(axis=(0, 2)) + np.float32(1e-6),
            "classw": W.class_weights(y), "params": W.mlp_init_params(64 * nf, seed % 65536)}


def _start(state):
    s = state["solver"]
    s.init_forest(state["levels"], state["coords"])
    s.load_blocks(state["data"])


def prepare(case, seed):
    if case["kind"] in ("train", "forward"):
        st = _samples(case, seed)
        # the predictor lives in a solver's context
        cfg = W.C3(jmax=2, max_blocks=64) if case["fields"] == 4 else W.C2(jmax=2, max_blocks=64)
        st["solver"] = M.Solver(cfg)
        st["solver"].mlp_init(st["params"], st["mean"], st["std"])
        st["case"] = case
        return st
    lv, co = _forest(case, seed)
    order = _morton_order(case, lv, co)
    lv, co = lv[order], co[order]
    cfg = _config(case, len(lv))
    s = M.Solver(cfg)
    st = {"case": case, "solver": s, "levels": lv, "coords": co, "dt": cfg.dt,
          "data": _sample(case, seed, lv, co, s.device)}
    _start(st)
    if case["sweep"] != 2:   # the studies' setting
        s.set_graph(0)
        s.set_sweep(case["sweep"])
    if case["tuned"]:
        s.refine_all()
        s.tune(reps=3)
        _start(st)
        s.step(0.0, cfg.dt, 20)   # the library's own choice between graph replay and launches
        _start(st)
    return st


def run(state):
    case, s = state["case"], state["solver"]
    kind = case["kind"]
    if kind == "rk4":
        s.load_blocks(state["data"])
        for k in range(case["steps"]):
            s.rk4(k * state["dt"], state["dt"])
        return s.read_blocks(on_device=True)
    if kind == "step":
        _start(state)
        s.step(0.0, state["dt"], case["steps"])
        lv, co = s.read_forest()
        return [s.read_blocks(on_device=True), lv, co]
    if kind == "analyse":
        flags, maxd = s.mr_pass()
        return [maxd, flags]
    if kind == "train":
        s.mlp_init(state["params"], state["mean"], state["std"])
        loss = s.mlp_train_epoch(state["x"], state["y"], state["classw"], batch=case["batch"])
        return [s.mlp_params(), loss]
    return s.mlp_forward(state["x"])


def work(case):
    if case["kind"] in ("train", "forward"):
        n, nin = case["samples"], 64 * case["fields"]
        per = 2.0 * (nin * 64 + 64 * 64 + 64 * 3)
        params = 4.0 * (nin * 64 + 64 + 64 * 64 + 64 + 64 * 3 + 3)
        if case["kind"] == "forward":
            return {"bytes": 4.0 * n * (nin + 3) + params, "flops": n * per}
        # backward: the weight gradients and the deltas of the upper layers
        back = per + 2.0 * (64 * 64 + 64 * 3)
        batches = -(-n // case["batch"])
        # Adam reads and writes the parameters and both moments once a batch
        return {"bytes": n * (4.0 * nin + 1.0) + batches * 6.0 * params, "flops": n * (per + back)}
    dim, bs = case["dim"], case["bs"]
    nf = 4 if case["physics"] in _LAYERS else 1
    maps = _leaf_maps(case)
    blocks = sum(int(m.sum()) for m in maps.values())
    nodes = float(bs ** dim * nf)
    # operations of one stage at a node, all fields: differences per axis, products and sums
    stage = 230.0 if nf == 4 else 9.0 * dim + 4.0
    if case["kind"] == "analyse":
        return {"bytes": 8.0 * blocks * nodes, "flops": 14.0 * blocks * nodes}
    if case["kind"] == "rk4":
        # u read and the new u written once a step
        return {"bytes": case["steps"] * 16.0 * blocks * nodes,
                "flops": case["steps"] * 4.0 * blocks * (nodes / nf) * (stage + 4.0 * nf)}
    # a step reads the grid before the refinement and writes the grid after the coarsening
    # (about the same); the refined blocks' values need not leave the chip
    fine = sum(int(m.sum()) * (2 ** dim if l < case["jmax"] else 1) for l, m in maps.items())
    return {"bytes": case["steps"] * 16.0 * blocks * nodes,
            "flops": case["steps"] * (4.0 * fine * (nodes / nf) * (stage + 4.0 * nf) + 28.0 * fine * nodes)}


# ---------------------------------------------------------------------------------------
# exact results: dense arrays per level, torch FP64
# ---------------------------------------------------------------------------------------

class _Dense:
    """The method on dense periodic arrays [nf, N_l]*dim of every level (x last): u[l] holds
    the stored values of the level's leaves, own[l] marks the nodes they hold."""

    def __init__(self, case, seed, device):
        self.case, self.dim, self.bs, self.J = case, case["dim"], case["bs"], max(2, case["jmax"])
        self.dev = device
        self.nf = 4 if case["physics"] in _LAYERS else 1
        off, _ = _shift(case, seed)
        self.leaf = {l: torch.zeros((2 ** l,) * self.dim, dtype=torch.bool, device=device)
                     for l in range(1, self.J + 1)}
        for l, m in _leaf_maps(case).items():
            for a in range(self.dim):
                m = np.roll(m, int(off[a]) << (l - case["base"]) if l >= case["base"] else 0, axis=self.dim - 1 - a)
            self.leaf[l] = torch.as_tensor(m, device=device)
        self.u = {}
        for l in self._levels():
            n = 2 ** l * (self.bs - 1)
            x = []
            for a in range(self.dim):
                shape = [1] * self.dim
                shape[self.dim - 1 - a] = n
                x.append((torch.arange(n, device=device).double() / n).reshape(shape))
            f = _fields(case, seed, x)
            self.u[l] = torch.stack([v.expand((n,) * self.dim) for v in f])
        cfg = _config(case, 1)
        self.dt, self.eps, self.phys, self.ph = cfg.dt, cfg.eps, cfg.phys, case["physics"]

    def _levels(self):
        return [l for l in range(1, self.J + 1) if bool(self.leaf[l].any())]

    def _axes(self, a):
        """Array dimension (fields first, x last) of axis a."""
        return self.dim - a

    def _held(self, l):
        """Nodes held by the level's leaves: boolean [N_l]*dim."""
        m = self.leaf[l]
        for d in range(self.dim):
            m = m.repeat_interleave(self.bs - 1, dim=d)
        for d in range(self.dim):
            m = m | torch.roll(m, 1, d)
        return m

    def _predict(self, v):
        for a in range(self.dim):
            d = self._axes(a)
            odd = (9.0 * (v + torch.roll(v, -1, d)) - (torch.roll(v, 1, d) + torch.roll(v, -2, d))) * 0.0625
            shape = list(v.shape)
            shape[d] *= 2
            v = torch.stack([v, odd], dim=d + 1).reshape(shape)
        return v

    def _even(self, v, first):
        for d in range(first, v.dim()):
            v = v.index_select(d, torch.arange(0, v.shape[d], 2, device=self.dev))
        return v

    def sync(self, y, upto=None):
        """V of every level with leaves (and of level `upto`) from the stored values y."""
        top = max(self._levels())
        S, H = {}, {}
        for l in range(top, 0, -1):
            h = self._held(l)
            s = y[l] if l in y else torch.zeros((self.nf,) + tuple(h.shape), dtype=torch.float64, device=self.dev)
            if l + 1 in S:
                he = self._even(H[l + 1], 0)
                s = torch.where(he, self._even(S[l + 1], 1), s)
                h = h | he
            S[l], H[l] = s, h
        V = {1: S[1]}
        for l in range(2, max(top, upto or 0) + 1):
            p = self._predict(V[l - 1])
            V[l] = torch.where(H[l], S[l], p) if l in S else p
        return V

    def _d(self, v, a, l, field=True):
        d = self._axes(a) if field else self._axes(a) - 1
        r = 2 ** l * (self.bs - 1) / 12.0
        return (8.0 * (torch.roll(v, -1, d) - torch.roll(v, 1, d)) - (torch.roll(v, -2, d) - torch.roll(v, 2, d))) * r

    def rhs(self, v, l, t):
        if self.ph == "const":
            return -sum(self.phys[a] * self._d(v, a, l) for a in range(self.dim))
        if self.ph == "swirl":
            x = torch.arange(v.shape[-1], device=self.dev).double() / v.shape[-1]
            s2, s = torch.sin(math.pi * x) ** 2, torch.sin(2.0 * math.pi * x)
            return -(s2[None, :] * s[:, None] * self._d(v, 0, l) - s2[:, None] * s[None, :] * self._d(v, 1, l))
        gam, mu, pr = self.phys[:3]
        kap = mu * gam / ((gam - 1.0) * pr)
        rho, u, w, p = v
        D = lambda q, a: self._d(q, a, l, field=False)  # noqa: E731
        ux, uy, vx, vy, px, py = D(u, 0), D(u, 1), D(w, 0), D(w, 1), D(p, 0), D(p, 1)
        div = ux + vy
        txx, tyy, txy = mu * (2 * ux - 2 / 3 * div), mu * (2 * vy - 2 / 3 * div), mu * (uy + vx)
        T = p / rho
        divq = D(-kap * D(T, 0), 0) + D(-kap * D(T, 1), 1)
        phi = txx * ux + txy * (uy + vx) + tyy * vy
        return torch.stack([-(D(rho * u, 0) + D(rho * w, 1)),
                            -(u * ux + w * uy) - px / rho + (D(txx, 0) + D(txy, 1)) / rho,
                            -(u * vx + w * vy) - py / rho + (D(txy, 0) + D(tyy, 1)) / rho,
                            -(u * px + w * py) - gam * p * div + (gam - 1.0) * (phi - divq)])

    def rk4(self, t):
        dt, lev = self.dt, self._levels()
        k = []
        for a, tt in ((0.0, t), (dt / 2, t + dt / 2), (dt / 2, t + dt / 2), (dt, t + dt)):
            V = self.sync({l: self.u[l] + a * k[-1][l] for l in lev} if k else self.u)
            k.append({l: self.rhs(V[l], l, tt) for l in lev})
        self.u = {l: self.u[l] + dt / 6.0 * ((k[0][l] + k[3][l]) + 2.0 * (k[1][l] + k[2][l])) for l in lev}
        if len(self.phys) > 3 and self.phys[3] > 0.0 and self.ph == "shear":
            V = self.sync(self.u)
            self.u = {l: self._filter(V[l]) for l in lev}

    def _filter(self, q):
        out = 0.0
        for a in range(2):
            d, p = self._axes(a) - 1, q[3]
            dp = (-torch.roll(p, -1, d) + 2.0 * p - torch.roll(p, 1, d)) * 0.25
            m = ((dp - torch.roll(dp, -1, d)) ** 2 + (dp - torch.roll(dp, 1, d)) ** 2) * 0.5
            s = torch.clamp(1.0 - self.phys[3] / (m / (p * p) + 1e-16), min=0.0)
            half = (s + torch.roll(s, -1, d)) * 0.5
            flux = half * (-(torch.roll(q, -1, d + 1) - q) * 0.25)
            out = out + flux - torch.roll(flux, 1, d + 1)
        return q - out

    def details(self):
        """Per level, the largest |detail| of every block position and field; V of the grid is stored back."""
        V = self.sync(self.u)
        out = {}
        for l in self._levels():
            self.u[l] = V[l]
            m = (V[l] - self._predict(self._even(V[l], 1))).abs()
            for d in range(1, self.dim + 1):   # nodes 0..bs-1 of each block, the last shared with the next
                nb = 2 ** l
                shape = m.shape[:d] + (nb, self.bs - 1) + m.shape[d + 1:]
                b = m.reshape(shape)
                last = torch.roll(b.select(d + 1, 0), -1, d)
                m = torch.maximum(b.amax(dim=d + 1), last)
            out[l] = m
        return out

    def refine_all(self):
        lev = self._levels()
        V = self.sync(self.u, upto=min(self.J, max(lev) + 1))
        new = {}
        leaf = {l: torch.zeros_like(m) for l, m in self.leaf.items()}
        for l in lev:
            if l < self.J:
                m = self.leaf[l]
                for d in range(self.dim):
                    m = m.repeat_interleave(2, dim=d)
                leaf[l + 1] |= m
                new[l + 1] = V[l + 1]
            else:
                leaf[l] |= self.leaf[l]
        if self.J in self.u and self.J in new:   # the finest leaves keep their stored values
            new[self.J] = torch.where(self._held(self.J), self.u[self.J], new[self.J])
        elif self.J in self.u:
            new[self.J] = self.u[self.J]
        self.leaf, self.u = leaf, new

    def _grow(self, m):
        for d in range(m.dim()):
            m = m | torch.roll(m, 1, d) | torch.roll(m, -1, d)
        return m

    def coarsen(self, flag):
        """Merge the largest set of complete, flagged families that keeps the grid graded."""
        alive = {}
        for l in range(2, self.J + 1):
            m = self.leaf[l] & flag[l] if l in flag else torch.zeros_like(self.leaf[l])
            for d in range(self.dim):
                m = m.reshape(m.shape[:d] + (m.shape[d] // 2, 2) + m.shape[d + 1:]).all(dim=d + 1)
            alive[l - 1] = m   # mothers, on their own level
        inner, above = {}, torch.zeros_like(self.leaf[self.J])
        for l in range(self.J, 0, -1):   # block positions that are refined
            inner[l] = above
            up = above | self.leaf[l]
            for d in range(self.dim):
                up = up.reshape(up.shape[:d] + (up.shape[d] // 2, 2) + up.shape[d + 1:]).any(dim=d + 1)
            above = up
        changed = True
        while changed:
            changed = False
            for l in range(2, self.J):   # members on level l beside refined positions that stay refined
                bad = self._grow(inner[l] & ~alive[l])
                for d in range(self.dim):
                    bad = bad.reshape(bad.shape[:d] + (bad.shape[d] // 2, 2) + bad.shape[d + 1:]).any(dim=d + 1)
                die = alive[l - 1] & bad
                if bool(die.any()):
                    alive[l - 1] = alive[l - 1] & ~die
                    changed = True
        if not any(bool(m.any()) for m in alive.values()):
            return False
        u = dict(self.u)
        old = {l: self._held(l) for l in self._levels()}
        for l, m in alive.items():
            if not bool(m.any()):
                continue
            kids = m
            for d in range(self.dim):
                kids = kids.repeat_interleave(2, dim=d)
            self.leaf[l + 1] = self.leaf[l + 1] & ~kids
            self.leaf[l] = self.leaf[l] | m
            even = self._even(self.u[l + 1], 1)
            u[l] = torch.where(old[l], self.u[l], even) if l in self.u else even
        self.u = {l: u[l] for l in self._levels()}
        return True

    def adapt(self):
        for _ in range(self.J + 3):
            big = self.details()
            flag = {l: (m < self.eps).all(dim=0) & (l > 1) for l, m in big.items()}
            if not self.coarsen(flag):
                return

    def forest(self):
        lv, co = [], []
        for l in self._levels():
            c = self.leaf[l].nonzero().flip(1).cpu().numpy().astype(np.int32)
            lv.append(np.full(len(c), l, dtype=np.int8))
            co.append(c)
        lv, co = np.concatenate(lv), np.concatenate(co)
        order = _morton_order(self.case, lv, co)
        return lv[order], co[order]

    def blocks(self):
        """Synchronised block values in forest order: [n, nf, bs^dim]."""
        V = self.sync(self.u)
        lv, co = self.forest()
        out = torch.empty((len(lv), self.nf) + (self.bs,) * self.dim, dtype=torch.float64, device=self.dev)
        node = torch.arange(self.bs, device=self.dev)
        for l in self._levels():
            at = np.flatnonzero(lv == l)
            c = torch.as_tensor(co[at].astype(np.int64), device=self.dev)
            n = 2 ** l * (self.bs - 1)
            flat = 0
            for a in reversed(range(self.dim)):
                shape = [len(at)] + [1] * self.dim
                shape[self.dim - a] = self.bs
                flat = flat * n + ((c[:, a:a + 1] * (self.bs - 1) + node) % n).reshape(shape)
            sel = torch.as_tensor(at, device=self.dev)
            for f in range(self.nf):
                out[sel, f] = V[l][f].reshape(-1)[flat]
        return out.reshape(len(lv), self.nf, -1)


def _exact_mlp(case, seed):
    st = _samples(case, seed)
    nf, nin = case["fields"], 64 * case["fields"]
    p = torch.from_numpy(st["params"]).double()
    mean = torch.from_numpy(np.repeat(st["mean"].astype(np.float32), 64)).double()
    std = torch.from_numpy(np.repeat(st["std"].astype(np.float32), 64)).double()
    x = (torch.from_numpy(st["x"]).double() - mean) / std
    cuts = np.cumsum([nin * 64, 64, 64 * 64, 64, 64 * 3])

    def logits(q, z):
        w1, b1, w2, b2, w3, b3 = torch.tensor_split(q, cuts.tolist())
        gelu = torch.nn.functional.gelu
        h = gelu(z @ w1.reshape(nin, 64) + b1)
        return gelu(h @ w2.reshape(64, 64) + b2) @ w3.reshape(64, 3) + b3

    if case["kind"] == "forward":
        return logits(p, x)
    y, cw = torch.from_numpy(st["y"]).long(), torch.from_numpy(st["classw"]).double()
    m, v, losses = torch.zeros_like(p), torch.zeros_like(p), []
    lr, b1, b2 = float(np.float32(1e-3)), float(np.float32(0.9)), float(np.float32(0.999))
    for step, at in enumerate(range(0, len(y), case["batch"]), 1):
        q = p.clone().requires_grad_(True)
        ys = y[at:at + case["batch"]]
        loss = torch.nn.functional.cross_entropy(logits(q, x[at:at + case["batch"]]), ys, weight=cw)
        loss.backward()
        losses.append(float(loss.detach()))
        m = b1 * m + (1 - b1) * q.grad
        v = b2 * v + (1 - b2) * q.grad ** 2
        p = p - lr * (m / (1 - b1 ** step)) / ((v / (1 - b2 ** step)).sqrt() + 1e-8)
    return [p, float(np.mean(losses))]


def exact(case, seed):
    if case["kind"] in ("train", "forward"):
        return _exact_mlp(case, seed)
    if (2 ** case["jmax"] * (case["bs"] - 1)) ** case["dim"] > 2 ** 28:
        return None
    g = _Dense(case, seed, "cuda" if torch.cuda.is_available() else "cpu")
    if case["kind"] == "rk4":
        for k in range(case["steps"]):
            g.rk4(k * g.dt)
        return g.blocks()
    if case["kind"] == "analyse":
        big = g.details()
        lv, co = g.forest()
        maxd = torch.empty((len(lv), g.nf), dtype=torch.float64, device=g.dev)
        for l, m in big.items():
            at = np.flatnonzero(lv == l)
            c = torch.as_tensor(co[at].astype(np.int64), device=g.dev)
            maxd[torch.as_tensor(at, device=g.dev)] = m[(slice(None),) + tuple(c[:, a] for a in reversed(range(g.dim)))].T
        return [maxd, None]
    for k in range(case["steps"]):
        g.refine_all()
        g.rk4(k * g.dt)
        g.adapt()
    return [g.blocks(), None, None]
