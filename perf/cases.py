"""Cases that time what a user has this library do: advance grids, and move
their fields in and out, through the public entry points of
paper_1004_0480_amd.rd.

A case is a dict of plain values.  Its "op" says which call pattern it is:

  advance   a simulation in progress: step n times, then read every species
            into device tensors (the snapshot a long run takes every n steps)
  job       one whole short run: write the initial state, step, read
  ensemble  many grids of uneven size in one Batch, each for its own number
            of steps: write, add, tick until all are done, read
  fields    a checkpoint restore with its check: write every species, reduce
            its mass and energy, read it back

"tuned" cases use the grid as the repository's benchmark does (a stream of
its own, rd_autotune once per shape, hipGraph replay); the others use a grid
as it is created, on the default plan.
"""
import math

import numpy as np
import torch

from paper_1004_0480_amd import rd
from paper_1004_0480_amd import workloads as W

SERVE_EDGES = (32, 48, 64, 96, 128)
SPECIES = {"diffusion": 1, "brusselator": 2, "front_ch": 3, "pollutant": 4, "turing": 2}
# multiplications and additions per cell and step (an fma counts two)
FLOPS = {"diffusion": 14, "brusselator": 37, "front_ch": 78, "pollutant": 80, "turing": 70}


def _case(name, op, model, nx, ny, nz, storage="f32", steps=1, tuned=False, rounding="nearest", grids=0):
    c = dict(op=op, model=model, nx=nx, ny=ny, nz=nz, storage=storage, steps=steps, tuned=tuned,
             rounding=rounding, grids=grids)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one step of a small ragged grid that is looked at after every step
        _case("tiny_step", "advance", "diffusion", 37, 33, 30),
        # the 64^3 diffusion problem from start to end, 100 steps: launches count
        _case("diffusion64_job", "job", "diffusion", 64, 64, 64, steps=100),
        # a mid-size parameter study on a grid that fits no tile
        _case("brusselator_odd", "advance", "brusselator", 101, 90, 77, steps=200),
        # the four production grids, as the benchmark runs them
        _case("brusselator256", "advance", "brusselator", 256, 256, 256, steps=40, tuned=True),
        _case("front384", "advance", "front_ch", 384, 384, 512, steps=20, tuned=True),
        _case("pollutant512", "advance", "pollutant", 512, 512, 128, steps=20, tuned=True),
        _case("diffusion512", "advance", "diffusion", 512, 512, 512, steps=20, tuned=True),
        # reduced storage: to nearest, and stochastic (which keeps small increments)
        _case("brusselator256_bf16", "advance", "brusselator", 256, 256, 256, "bf16", 40),
        _case("front_bf16_stochastic", "advance", "front_ch", 248, 200, 180, "bf16", 30, rounding="stochastic"),
        # the paper's activator-inhibitor problem, 19-point Laplacian, at its 192^3
        _case("turing192", "advance", "turing", 192, 192, 192, steps=40),
        # served requests: cubes of 32 to 128, diffusion and Brusselator mixed
        _case("ensemble64", "ensemble", "mixed", 128, 128, 128, steps=200, grids=64),
        # restore and check a two-species state
        _case("fields_odd", "fields", "brusselator", 403, 301, 300),
    ]


def _edge(rng, lo, hi):
    """A grid extent, spread over the logarithm; half of them a multiple of 8, as users choose."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(8, n // 8 * 8) if rng.random() < 0.5 else n


def _clamp(ext, cells):
    """The extents scaled down to at most this many cells."""
    k = min(1.0, (cells / float(ext[0] * ext[1] * ext[2])) ** (1.0 / 3.0))
    return [max(8, int(e * k)) for e in ext]


def draw(rng):
    kind = rng.choice(["small", "large", "large", "front", "pollutant", "turing", "ensemble", "fields"])
    if kind == "small":
        model = rng.choice(["diffusion", "brusselator"])
        ext = [_edge(rng, 20, 140) for _ in range(3)]
        steps = int(round(math.exp(rng.uniform(0.0, math.log(200.0)))))
        op = rng.choice(["advance", "job"])
        return _case(None, op, model, *ext, steps=steps)
    if kind == "large":
        model = rng.choice(["diffusion", "brusselator"])
        cap = 1.3e8 if model == "diffusion" else 5e7
        ext = _clamp([_edge(rng, 130, 512) for _ in range(3)], cap)
        return _case(None, "advance", model, *ext, rng.choice(["f32", "bf16"]), rng.randint(5, 40),
                     tuned=rng.random() < 0.5)
    if kind == "front":
        ext = _clamp([_edge(rng, 60, 512) for _ in range(3)], 7e7)
        storage = rng.choice(["f32", "bf16"])
        rounding = rng.choice(["nearest", "stochastic"]) if storage == "bf16" else "nearest"
        return _case(None, "advance", "front_ch", *ext, storage, rng.randint(5, 20), rng.random() < 0.5, rounding)
    if kind == "pollutant":
        ext = _clamp([_edge(rng, 60, 512), _edge(rng, 60, 512), _edge(rng, 20, 160)], 3.3e7)
        return _case(None, "advance", "pollutant", *ext, rng.choice(["f32", "bf16"]), rng.randint(5, 20),
                     rng.random() < 0.5)
    if kind == "turing":
        ext = [_edge(rng, 64, 300) for _ in range(3)]
        return _case(None, "advance", "turing", *ext, steps=rng.randint(5, 40))
    if kind == "ensemble":
        return _case(None, "ensemble", "mixed", 128, 128, 128, rng.choice(["f32", "bf16"]),
                     rng.randint(40, 200), grids=rng.randint(8, 64))
    ext = _clamp([_edge(rng, 40, 512) for _ in range(3)], 5e7)
    return _case(None, "fields", rng.choice(["diffusion", "brusselator"]), *ext, rng.choice(["f32", "bf16"]))


# ------------------------------------------------------------------ problems

class Problem:
    """One initial-value problem: plain numbers and device tensors."""

    def __init__(self, model, shape, seed, storage):
        self.model, self.shape = model, shape
        nz, ny, nx = shape
        gen = torch.Generator(device="cuda")
        gen.manual_seed(int(seed))
        ns = SPECIES[model]
        self.ns, self.h, self.stencil, self.params = ns, 1.0, 7, {}
        self.wind = self.sources = None
        self.bc = [[("mirror", 0.0)] * 6 for _ in range(ns)]

        def noise(lo, hi):
            return torch.rand(shape, generator=gen, device="cuda") * (hi - lo) + lo

        if model == "diffusion":
            self.K, self.dt = [[1.0] * 3], 0.1
            r2 = 0.0
            for d, n in enumerate(shape):
                c = torch.arange(n, device="cuda", dtype=torch.float32) - (n - 1) / 2.0
                r2 = r2 + (c * c).reshape([-1 if k == d else 1 for k in range(3)])
            fields = [torch.exp(-r2 / (2.0 * (6.0 * max(shape) / 64.0) ** 2)) + noise(0.0, 1e-3)]
        elif model == "brusselator":
            a, b = 4.5, 6.75
            self.K, self.dt, self.params = [[1.0] * 3, [8.0] * 3], 0.01, {"a": a, "b": b}
            self.bc = [[("periodic", 0.0)] * 6 for _ in range(ns)]
            fields = [a * (1.0 + noise(-0.01, 0.01)), (b / a) * (1.0 + noise(-0.01, 0.01))]
        elif model == "front_ch":
            # a front that has moved some cells in from the held face z = 0
            self.K, self.dt = [[1.0] * 3, [1.0] * 3, [0.0] * 3], 0.005
            self.params = {"k": 1.0, "M": 0.1, "kappa": 1.0, "eps": 1.0, "gamma": 1.0}
            self.bc[0][4] = ("held", 1.0)
            z = torch.arange(nz, device="cuda", dtype=torch.float32).reshape(-1, 1, 1)
            fields = [torch.exp(-z / 12.0).expand(shape).contiguous(), 0.1 * (1.0 + noise(-0.01, 0.01)),
                      -1.0 + 2.0 * torch.exp(-z / 10.0) + noise(-0.01, 0.01)]
            fields[0][0] = 1.0
        elif model == "pollutant":
            umax = 5.0
            self.K = [[50.0, 50.0, 1.0]] * ns
            self.dt = 0.5 / (2.0 * 101.0 + umax)
            self.params = {"decay": 1e-4, "kab": 1e-3}
            for s in range(ns):
                self.bc[s][0] = ("ghost", 0.0)
            self.wind = umax * np.log1p(np.arange(nz, dtype=np.float64)) / math.log(129.0)
            r = np.random.default_rng(int(seed))
            n = 64
            cells = (r.integers(0, min(16, nz), n) * ny + r.integers(0, ny, n)) * nx + r.integers(0, nx, n)
            self.sources = (cells.astype(np.int64), (np.arange(n) % ns).astype(np.int32), np.full(n, 10.0))
            z = torch.arange(nz, device="cuda", dtype=torch.float32).reshape(-1, 1, 1)
            fields = [torch.exp(-z / 20.0) * noise(0.0, 1.0) for _ in range(ns)]
        else:
            self.h, self.stencil, self.dt = 6.2e-3, 19, 5e-4
            self.K = [[5e-5] * 3, [5e-3] * 3]
            self.params = {"alpha": 0.5, "beta": 0.09, "gamma": 26.0}
            fields = [1.0 + noise(-5e-4, 5e-4) for _ in range(ns)]
        self.fields = [f.to(torch.bfloat16) if storage == "bf16" else f.float() for f in fields]

    def spec(self):
        return W.ModelSpec(self.model, self.ns, self.dt, self.h, [list(k) for k in self.K],
                           [list(b) for b in self.bc], dict(self.params), self.wind, self.sources, self.stencil)


def _members(case, seed):
    """Problem kinds, edges and steps of an ensemble's requests."""
    r = np.random.default_rng(int(seed) + 77)
    # one request list per case (the seed draws the fields): the same work in every pass
    p = np.random.default_rng(1000 * case["grids"] + case["steps"])
    out = []
    for _ in range(case["grids"]):
        edge = int(p.choice([e for e in SERVE_EDGES if e <= case["nx"]]))
        model = "brusselator" if p.random() < 0.5 else "diffusion"
        out.append((model, edge, int(p.integers(max(1, case["steps"] // 10), case["steps"] + 1)),
                    int(r.integers(0, 1 << 31))))
    return out


# ------------------------------------------------------------------- the case

_TUNED = set()      # shapes this process has autotuned (the library keeps the plans)


def prepare(case, seed):
    if case["op"] == "ensemble":
        return _prepare_ensemble(case, seed)
    shape = (case["nz"], case["ny"], case["nx"])
    p = Problem(case["model"], shape, seed, case["storage"])
    stream = torch.cuda.Stream() if case["tuned"] else None
    g = rd.Grid(shape, p.ns, p.h, case["storage"], stream=stream)
    g.set_model(p.spec())
    if case["rounding"] == "stochastic":
        g.set_rounding("stochastic", seed=7)
    for s, f in enumerate(p.fields):
        g.write(s, f)
    if case["tuned"]:
        key = (case["model"], shape, case["storage"])
        if key not in _TUNED:
            g.autotune(10)
            _TUNED.add(key)
        g.set_plan(graph_chunk=20)
    out = [torch.empty(shape, dtype=torch.float32, device="cuda") for _ in range(p.ns)]
    return {"case": case, "grid": g, "fields": p.fields, "out": out, "stream": stream}


def _prepare_ensemble(case, seed):
    stream = torch.cuda.Stream()
    batch = rd.Batch(case["grids"], 1 << 36, case["storage"], stream=stream)
    grids, fields, steps, out = [], [], [], []
    for model, edge, n, sd in _members(case, seed):
        p = Problem(model, (edge,) * 3, sd, case["storage"])
        g = rd.Grid(p.shape, p.ns, p.h, case["storage"], stream=stream)
        g.set_model(p.spec())
        grids.append(g)
        fields.append(p.fields)
        steps.append(n)
    total = sum(f.numel() for fs in fields for f in fs)
    flat = torch.empty(total, dtype=torch.float32, device="cuda")
    at = 0
    for fs in fields:
        out.append([])
        for f in fs:
            out[-1].append(flat[at:at + f.numel()].view(f.shape))
            at += f.numel()
    torch.cuda.synchronize()
    return {"case": case, "batch": batch, "grids": grids, "fields": fields, "steps": steps, "out": out,
            "flat": flat, "stream": stream}


def run(state):
    case = state["case"]
    if case["op"] == "ensemble":
        batch = state["batch"]
        for g, fs, n in zip(state["grids"], state["fields"], state["steps"]):
            for s, f in enumerate(fs):
                g.write(s, f, enqueue_only=True)
            batch.add(g, n)
        left = len(state["grids"])
        while left:
            left -= len(batch.step(25))
        for g, outs in zip(state["grids"], state["out"]):
            for s, o in enumerate(outs):
                g.read_device(s, o)
        return state["flat"]
    g, out = state["grid"], state["out"]
    if case["op"] in ("job", "fields"):
        for s, f in enumerate(state["fields"]):
            g.write(s, f)
    sums = []
    if case["op"] == "fields":
        sums = [g.reduce(s) for s in range(len(out))]
    else:
        g.step(case["steps"])
    for s, o in enumerate(out):
        g.read_device(s, o)
    return {"fields": out, "sums": sums}


def work(case):
    """Each input read once and each output written once: the stored state (read and, where
    stepped, written), the device tensors that come in and go out."""
    es = 2 if case["storage"] == "bf16" else 4
    if case["op"] == "ensemble":
        nbytes = flops = 0.0
        for model, edge, n, _ in _members(case, 0):
            cells = edge ** 3
            nbytes += cells * SPECIES[model] * (2 * es + 4)
            flops += float(cells) * n * FLOPS[model]
        return {"bytes": nbytes, "flops": flops}
    cells = float(case["nx"] * case["ny"] * case["nz"])
    values = cells * SPECIES[case["model"]]
    if case["op"] == "fields":
        return {"bytes": values * (2 * es + 4), "flops": values * 3}
    return {"bytes": values * (2 * es + 4), "flops": cells * case["steps"] * FLOPS[case["model"]]}


# ------------------------------------------------- the same in 64 bits, by torch

def _shift(c, axis, d, rule):
    """The neighbour one cell on along an axis, by the face's rule (axis 0, 1, 2 = z, y, x)."""
    kind, value = rule
    n = c.shape[axis]
    edge = n - 1 if d > 0 else 0
    out = torch.roll(c, -d, axis)
    if kind != "periodic":
        face = out.select(axis, edge)
        if kind == "mirror":
            face.copy_(c.select(axis, edge))
        else:
            face.fill_(value)
    return out


def _laplacian(c, K, h, bc, stencil):
    """bc: the six face rules in the order x-, x+, y-, y+, z-, z+."""
    if stencil == 7:
        lap = torch.zeros_like(c)
        for d in range(3):
            if K[d]:
                axis = 2 - d
                lap += (K[d] / (h * h)) * (_shift(c, axis, -1, bc[2 * d]) + _shift(c, axis, 1, bc[2 * d + 1]) - 2.0 * c)
        return lap
    pairs = [_shift(c, 2 - d, -1, bc[2 * d]) + _shift(c, 2 - d, 1, bc[2 * d + 1]) for d in range(3)]
    edges = (_shift(pairs[1], 2, -1, bc[0]) + _shift(pairs[1], 2, 1, bc[1])
             + _shift(pairs[2], 2, -1, bc[0]) + _shift(pairs[2], 2, 1, bc[1])
             + _shift(pairs[2], 1, -1, bc[2]) + _shift(pairs[2], 1, 1, bc[3]))
    return (K[0] / (6.0 * h * h)) * (2.0 * (pairs[0] + pairs[1] + pairs[2]) + edges - 24.0 * c)


MIRROR6 = [("mirror", 0.0)] * 6


def _step64(p, c, em):
    """One explicit step of every species from the old state."""
    q, dt = p.params, p.dt
    lap = [_laplacian(c[s], p.K[s], p.h, p.bc[s], p.stencil) for s in range(p.ns)]
    if p.model == "brusselator":
        uuv = c[0] * c[0] * c[1]
        lap[0] += q["a"] - (q["b"] + 1.0) * c[0] + uuv
        lap[1] += q["b"] * c[0] - uuv
    elif p.model == "turing":
        lap[0] += c[0] - c[0] ** 3 - c[1]
        lap[1] += q["gamma"] * (c[0] - q["alpha"] * c[1] - q["beta"])
    elif p.model == "front_ch":
        mu = (q["gamma"] * c[2] ** 3 - q["eps"] * c[2]
              - q["kappa"] * _laplacian(c[2], [1.0] * 3, p.h, p.bc[2], 7))
        r = q["k"] * c[0] * c[1]
        lap[0] -= r
        lap[1] -= r
        lap[2] += r + q["M"] * _laplacian(mu, [1.0] * 3, p.h, MIRROR6, 7)
    elif p.model == "pollutant":
        u = torch.from_numpy(p.wind).to(c[0].device).reshape(-1, 1, 1) / p.h
        for s in range(p.ns):
            lap[s] += u * (_shift(c[s], 2, -1, p.bc[s][0]) - c[s]) - q["decay"] * c[s] + em[s]
        lap[0] -= q["kab"] * c[0]
        lap[1] += q["kab"] * c[0]
    new = [c[s] + dt * lap[s] for s in range(p.ns)]
    if p.model == "front_ch":
        new[0][0] = p.bc[0][4][1]
    return new


def _run64(p, steps):
    c = [f.double() for f in p.fields]
    em = None
    if p.sources is not None:
        em = [torch.zeros(p.shape, dtype=torch.float64, device="cuda") for _ in range(p.ns)]
        for cell, sp, rate in zip(*p.sources):
            em[int(sp)].view(-1)[int(cell)] += float(rate)
    for _ in range(steps):
        c = _step64(p, c, em)
    return c


def exact(case, seed):
    if case["op"] == "ensemble":
        parts = []
        for model, edge, n, sd in _members(case, seed):
            parts += [f.reshape(-1) for f in _run64(Problem(model, (edge,) * 3, sd, case["storage"]), n)]
        return torch.cat(parts)
    p = Problem(case["model"], (case["nz"], case["ny"], case["nx"]), seed, case["storage"])
    if case["op"] == "fields":
        fields = [f.double() for f in p.fields]
        return {"fields": fields, "sums": [(float(f.sum()), float((f * f).sum())) for f in fields]}
    return {"fields": _run64(p, case["steps"]), "sums": []}
