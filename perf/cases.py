"""The work that programs have this solver do, as cases that can be timed and checked.

A case is one call (or one short run of calls) through the public entry points
of `paper_2310_00177_amd`: single solves, requests through the server, network
evaluations, the adjoint, and training steps.  The scenes follow this
repository's recipe (solid spheres, two-cell slabs, solid walls, a flat or a
wavy free surface, only fluid that touches air) and are drawn on the GPU.

    listed()            the cases
    draw(rng)           another case of the same ranges
    prepare(case, seed) inputs, network and workspaces
    run(state)          one pass, its outputs
    work(case)          bytes and operations that the pass cannot do without
    exact(case, seed)   the outputs in 64 bits, by plain torch
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2310_00177_amd as nps

FLUID, AIR, SOLID = 0, 1, 2
PRECISION = {"fp64": nps.FP64, "fp32": nps.FP32, "bf16": nps.MIXED_BF16, "fp16": nps.MIXED_FP16}
METHOD = {"npsdo": nps.NPSDO, "fpcg": nps.FPCG}
SERVED = (64, 96, 128, 160)   # grids of the served requests

_grids = lambda nz, ny, nx, levels=6: {"nz": nz, "ny": ny, "nx": nx, "levels": levels}   # noqa: E731


def listed() -> list:
    return [
        # One network evaluation on the smallest grid in use, on the library's own
        # scratch: a program that times or traces P alone, bound by launches.
        {"name": "precond_32_fp32_noalloc", "kind": "precond", "precision": "fp32", "noalloc": True,
         **_grids(32, 32, 32)},
        # P on a small ragged grid with a shallow network, whose width is no
        # multiple of any tile.
        {"name": "precond_40x56x72_fp64", "kind": "precond", "precision": "fp64", "noalloc": False,
         **_grids(40, 56, 72, 4)},
        # P inside another program's Krylov method at the usual grid size, mixed precision.
        {"name": "precond_128_bf16", "kind": "precond", "precision": "bf16", "noalloc": False,
         **_grids(128, 128, 128)},
        # P^T, the gradient of a loss in the network's input (and half of the
        # symmetric preconditioner).
        {"name": "transpose_64_fp32", "kind": "transpose", "precision": "fp32", **_grids(64, 64, 64)},
        # The plain method in double precision on the smallest scene: a solve
        # whose kernels are all shorter than a launch.
        {"name": "solve_32_fp64", "kind": "solve", "precision": "fp64", "method": "npsdo", "n_ortho": 2, "tol": 1e-6,
         "scene": "flat", **_grids(32, 32, 32)},
        # A pressure solve of a small interactive scene.
        {"name": "solve_64_bf16", "kind": "solve", "precision": "bf16", "method": "npsdo", "n_ortho": 2, "tol": 1e-6,
         "scene": "flat", **_grids(64, 64, 64)},
        # The benchmark's solve: one frame of a 128^3 scene, mixed precision.
        {"name": "solve_128_bf16", "kind": "solve", "precision": "bf16", "method": "npsdo", "n_ortho": 2, "tol": 1e-6,
         "scene": "flat", **_grids(128, 128, 128)},
        # A dam-break tank of 256 x 128 x 128 in single precision.
        {"name": "solve_128x128x256_fp32", "kind": "solve", "precision": "fp32", "method": "npsdo", "n_ortho": 2,
         "tol": 1e-5, "scene": "flat", **_grids(128, 128, 256)},
        # The largest single solve: 256^3 with waves, to a tight tolerance.
        {"name": "solve_256_fp16", "kind": "solve", "precision": "fp16", "method": "npsdo", "n_ortho": 2, "tol": 1e-8,
         "scene": "wavy", **_grids(256, 256, 256)},
        # Sixteen requests of mixed grid sizes through the server at once:
        # continuous batching past its capacity.
        {"name": "serve_16", "kind": "serve", "precision": "bf16", "requests": 16, "tol": 1e-6, "levels": 6},
        # A training step at the configured size and batch: loss and gradient.
        {"name": "train_16x128_fp32", "kind": "train", "precision": "fp32", "batch": 16, **_grids(128, 128, 128)},
        # A training step of small scenes with the bf16 contraction.
        {"name": "train_4x64_bf16", "kind": "train", "precision": "bf16", "batch": 4, **_grids(64, 64, 64)},
    ]


def _draw_grid(rng, lo, hi, levels) -> dict:
    """Three multiples of 2^(levels-1) around one size between lo and hi cells a side."""
    unit = 1 << (levels - 1)
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return _grids(*(max(1, round(n * rng.uniform(0.7, 1.4) / unit)) * unit for _ in range(3)), levels)


def draw(rng) -> dict:
    kind = rng.choice(("solve", "solve", "solve", "precond", "precond", "transpose", "train", "train", "serve"))
    if kind == "serve":
        return {"kind": "serve", "precision": rng.choice(("bf16", "fp16")), "requests": rng.randint(3, 24),
                "tol": 1e-6, "levels": 6}
    if kind == "solve":
        precision = rng.choice(("fp64", "fp32", "bf16", "bf16", "fp16"))
        # plain PCG is left out: with this preconditioner, which is not quite symmetric, it may not converge
        method = rng.choice(("npsdo", "npsdo", "npsdo", "fpcg"))
        return {"kind": kind, "precision": precision, "method": method,
                "n_ortho": rng.randint(1, 4) if method == "npsdo" else 1,
                "tol": 1e-5 if precision == "fp32" else rng.choice((1e-6, 1e-6, 1e-8)),
                "scene": rng.choice(("flat", "flat", "wavy")),
                **_draw_grid(rng, 32, 96 if precision == "fp64" else 160, rng.choice((5, 6, 6)))}
    levels = rng.choice((2, 3, 4, 5, 6, 6))
    if kind == "precond":
        precision = rng.choice(("fp64", "fp32", "bf16", "fp16"))
        return {"kind": kind, "precision": precision, "noalloc": precision != "fp64" and rng.random() < 0.5,
                **_draw_grid(rng, 24, 140, levels)}
    if kind == "transpose":
        return {"kind": kind, "precision": rng.choice(("fp64", "fp32")), **_draw_grid(rng, 24, 128, levels)}
    return {"kind": kind, "precision": rng.choice(("fp64", "fp32", "fp32", "bf16")), "batch": rng.randint(1, 8),
            **_draw_grid(rng, 24, 100, levels)}


# ---------------------------------------------------------------------------
# scenes, right-hand sides and weights
# ---------------------------------------------------------------------------
def _shape(case) -> tuple:
    return case["nz"], case["ny"], case["nx"]


def _dilate(m: torch.Tensor) -> torch.Tensor:
    """m and its six face neighbours."""
    out = m.clone()
    for axis in range(3):
        n = m.shape[axis]
        out.narrow(axis, 1, n - 1).logical_or_(m.narrow(axis, 0, n - 1))
        out.narrow(axis, 0, n - 1).logical_or_(m.narrow(axis, 1, n - 1))
    return out


def _scene(shape, kind: str, seed: int) -> torch.Tensor:
    """Labels (uint8, on the GPU) of a seeded scene; solid before air before fluid."""
    dev = "cuda"
    nz, ny, nx = shape
    z = (torch.arange(nz, device=dev, dtype=torch.float32) + 0.5)[:, None, None]
    y = (torch.arange(ny, device=dev, dtype=torch.float32) + 0.5)[None, :, None]
    x = (torch.arange(nx, device=dev, dtype=torch.float32) + 0.5)[None, None, :]
    rng = np.random.default_rng(seed)
    wavy = kind == "wavy"
    n_spheres, size = (60 if wavy else 20), min(shape)
    lo, hi = size / 32.0, (size * 0.15625)
    while True:
        lab = torch.zeros(shape, dtype=torch.uint8, device=dev)
        if wavy:
            amp = nz / 16.0
            fx, fy = (int(v) for v in rng.integers(1, 4, 2))
            px, py = (float(v) for v in rng.uniform(0.0, 2.0 * math.pi, 2))
            h = rng.uniform(nz / 2 + amp, 7 * nz / 8 - amp) + amp * torch.sin(2 * math.pi * fx / nx * x + px) * torch.sin(
                2 * math.pi * fy / ny * y + py)
        else:
            h = torch.full((1, 1, 1), float(rng.integers(nz // 2, (7 * nz) // 8 + 1)) + 0.25, device=dev)
        lab.masked_fill_(z >= h, AIR)
        solid = torch.zeros(shape, dtype=torch.bool, device=dev)
        for _ in range(n_spheres):
            c = [float(v) for v in rng.uniform(0.0, 1.0, 3) * np.array(shape)]
            r = float(rng.uniform(lo, hi))
            solid.logical_or_((z - c[0]) ** 2 + (y - c[1]) ** 2 + (x - c[2]) ** 2 <= r * r)
        for _ in range(3 if size >= 48 else 0):
            axis = int(rng.integers(0, 3))
            at = int(rng.integers(2, shape[axis] - 3))
            sl = [slice(at, at + 2)] * 3
            for other in (a for a in range(3) if a != axis):
                n = shape[other]
                length = int(rng.integers(n // 4, 3 * n // 4 + 1))
                off = int(rng.integers(0, n - length + 1))
                sl[other] = slice(off, off + length)
            solid[tuple(sl)] = True
        for axis in range(3):
            solid.select(axis, 0).fill_(True)
            solid.select(axis, shape[axis] - 1).fill_(True)
        lab.masked_fill_(solid, SOLID)
        # only fluid that air reaches through fluid
        fluid = lab == FLUID
        reached, count = _dilate(lab == AIR) & fluid, -1
        while True:
            for _ in range(32):
                reached = _dilate(reached) & fluid
            now = int(reached.sum())
            if now == count:
                break
            count = now
        if count > 0:
            lab.masked_fill_(fluid & ~reached, SOLID)
            return lab
        n_spheres //= 2


def _normal(labels: torch.Tensor, seed: int, dtype) -> torch.Tensor:
    """N(0, 1) on fluid cells, zero elsewhere."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    v = torch.randn(labels.shape, generator=gen, device="cuda", dtype=torch.float64)
    return (v * (labels == FLUID)).to(dtype)


def _sizes(levels: int) -> list:
    """(kind, level, entries) of the parameter blob, in its order."""
    out = []
    for name, count in (("c1", levels), ("c2", levels - 1)):
        for lvl in range(1, count + 1):
            out += [(name + "W", lvl, 27 * 81), (name + "B", lvl, 27)]
    for lvl in range(1, levels):
        out += [("a1W", lvl, 81), ("a1B", lvl, 1), ("a2W", lvl, 81), ("a2B", lvl, 1)]
    return out


def _dense_weights(levels: int, seed: int) -> np.ndarray:
    """Xavier-uniform weights and N(0, 0.05^2) biases: every tap of every kernel in use, as trained weights have it."""
    rng = np.random.default_rng(seed)
    parts = []
    for name, _, n in _sizes(levels):
        bound = math.sqrt(6.0 / (81 + 729)) if name[0] == "c" else math.sqrt(6.0 / (81 + 27))
        parts.append(rng.uniform(-bound, bound, n) if name.endswith("W") else 0.05 * rng.standard_normal(n))
    return np.concatenate(parts)


def _solver_weights(levels: int) -> np.ndarray:
    """Weights that precondition: centre taps, coarser levels scaled by their
    fluid fraction and weighted by 4^(l-1) (random weights stall the iteration)."""
    parts = []
    for name, lvl, n in _sizes(levels):
        v = np.zeros(n)
        if name == "c1W" and lvl > 1:
            v[(13 * 3 + FLUID) * 27 + 13] = 0.5
        elif name in ("c1B", "c2B"):
            v[13] = 0.5 if name == "c1B" and lvl > 1 else 1.0
        elif name in ("a1B", "a2B"):
            v[0] = 1.0 if name == "a1B" else 4.0
        parts.append(v)
    return np.concatenate(parts)


def _request_shapes(case) -> list:
    rng = np.random.default_rng(case["requests"])
    first = [64, 160, 96, 128]   # every size is there, the rest are drawn
    more = [int(n) for n in rng.choice(SERVED, size=case["requests"])]
    return [(n, n, n) for n in (first + more)[:case["requests"]]]


def _inputs(case, seed: int) -> dict:
    kind = case["kind"]
    dtype = torch.float64 if case["precision"] == "fp64" or kind in ("solve", "serve") else torch.float32
    if kind == "serve":
        shapes = _request_shapes(case)
        labels = [_scene(s, "flat", seed * 64 + i) for i, s in enumerate(shapes)]
        return {"labels": labels, "b": [_normal(lab, seed * 64 + i + 1, dtype) for i, lab in enumerate(labels)],
                "params": _solver_weights(case["levels"])}
    if kind == "train":
        labels = torch.stack([_scene(_shape(case), "flat", seed * 64 + i) for i in range(case["batch"])])
        return {"labels": labels, "b": _normal(labels, seed + 1, dtype), "params": _dense_weights(case["levels"], seed)}
    labels = _scene(_shape(case), case.get("scene", "flat"), seed)
    params = _solver_weights(case["levels"]) if kind == "solve" else _dense_weights(case["levels"], seed)
    return {"labels": labels, "b": _normal(labels, seed + 1, dtype), "params": params}


# ---------------------------------------------------------------------------
# the passes
# ---------------------------------------------------------------------------
def prepare(case, seed: int) -> dict:
    s = _inputs(case, seed)
    kind, levels, precision = case["kind"], case["levels"], PRECISION[case["precision"]]
    s["case"], s["net"], s["precision"] = case, nps.Net(s["params"], levels), precision
    if kind == "serve":
        s["labels"] = [lab.cpu().numpy() for lab in s["labels"]]
        s["b"] = [b.cpu().numpy() for b in s["b"]]
        s["server"] = nps.Server(s["net"], hbm_budget=8 << 30, max_slots=16)
    elif kind == "solve":
        s["ws"] = nps.workspace(_shape(case), levels, precision, case["n_ortho"])
        s["x"] = torch.empty_like(s["b"])
    elif kind == "train":
        s["ws"] = nps.train_workspace(_shape(case), levels, precision)
        s["grad"] = torch.zeros(s["params"].size, dtype=torch.float64, device="cuda")
    elif kind == "transpose":
        s["ws"] = nps.train_workspace(_shape(case), levels, precision)
    elif case["noalloc"]:
        s["d"] = torch.empty_like(s["b"])
    else:
        s["ws"] = nps.workspace(_shape(case), levels, precision, 0)
    return s


def _serve(s) -> list:
    server = s["server"]
    ids = [server.submit(lab, b, tol=s["case"]["tol"], precision=s["precision"])
           for lab, b in zip(s["labels"], s["b"])]
    xs = {}
    while len(xs) < len(ids):
        server.step()
        for rid in ids:
            if rid not in xs:
                done = server.poll(rid)
                if done is not None:
                    xs[rid] = done[0]
    return [xs[rid] for rid in ids]


def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "serve":
        return _serve(s)
    if kind == "solve":
        x, _ = nps.solve(s["net"], s["labels"], s["b"], tol=case["tol"], n_ortho=case["n_ortho"],
                         precision=s["precision"], x=s["x"], ws=s["ws"], method=METHOD[case["method"]])
        # the FP32 mode keeps its iterate in float: a single-precision program takes it as such
        return x.float() if case["precision"] == "fp32" else x
    if kind == "train":
        s["grad"].zero_()
        loss = nps.train_step(s["net"], s["labels"], s["b"], s["grad"], s["ws"], precision=s["precision"])
        # parameters and optimiser of a float run are float
        return {"loss": loss, "grad": s["grad"] if case["precision"] == "fp64" else s["grad"].float()}
    if kind == "transpose":
        return nps.apply_precond_transpose(s["net"], s["labels"], s["b"], ws=s["ws"])
    if case["noalloc"]:
        return nps.apply_precond_noalloc(s["net"], s["labels"], s["b"], precision=s["precision"], d=s["d"])
    return nps.apply_precond(s["net"], s["labels"], s["b"], precision=s["precision"], ws=s["ws"])


# ---------------------------------------------------------------------------
# work that cannot be done without
# ---------------------------------------------------------------------------
def _network_flops(cells: float, evaluations: float = 1.0) -> float:
    """The kernels of a scene once (27 taps x 54 counts and a constant) and their application at every evaluation,
    two blocks a level, the levels together 8/7 of the finest."""
    return (8.0 / 7.0) * cells * 2 * (2 * 27 * 55 + evaluations * 2 * 27)


def _solve_work(cells: float, case) -> dict:
    """Iterations by the grid's size (31 at 32^3, 66 at 128^3 to 1e-6; twice that under waves at 256^3); an
    iteration reads and writes each Krylov vector that it updates once."""
    its = 31.0 * (cells / 32.0 ** 3) ** 0.18 * math.log(case["tol"]) / math.log(1e-6)
    if case.get("scene") == "wavy":
        its *= max(1.0, (cells / 64.0 ** 3) ** 0.17)
    wide = 2 if case["precision"] == "fp64" else 1
    return {"bytes": 17.0 * cells + its * 84.0 * wide * cells,
            "flops": _network_flops(cells, its) + its * 40.0 * cells}


def work(case) -> dict:
    if case["kind"] == "serve":
        shapes = _request_shapes(case)
        each = [_solve_work(float(n) ** 3, case) for n, _, _ in shapes]
        return {k: sum(w[k] for w in each) for k in ("bytes", "flops")}
    cells = float(case["nz"] * case["ny"] * case["nx"])
    if case["kind"] == "solve":
        return _solve_work(cells, case)
    word = 8.0 if case["precision"] == "fp64" else 4.0
    flops = _network_flops(cells)
    if case["kind"] == "train":   # forward, adjoint and the weight gradients
        return {"bytes": case["batch"] * cells * (1 + word), "flops": 3.0 * case["batch"] * flops}
    return {"bytes": cells * (1 + 2 * word), "flops": flops}


# ---------------------------------------------------------------------------
# the same results in 64 bits
# ---------------------------------------------------------------------------
_OFFSETS = [(a, b, c) for a in (-1, 0, 1) for b in (-1, 0, 1) for c in (-1, 0, 1)]


def _windows(v: torch.Tensor, fill: float):
    """v(p + o) for each of the 27 offsets o, `fill` outside the grid."""
    nz, ny, nx = v.shape[-3:]
    p = torch.nn.functional.pad(v, (1, 1, 1, 1, 1, 1), value=fill)
    for a, b, c in _OFFSETS:
        yield p[..., 1 + a:1 + a + nz, 1 + b:1 + b + ny, 1 + c:1 + c + nx]


def _pool(v):
    *lead, nz, ny, nx = v.shape
    return v.reshape(*lead, nz // 2, 2, ny // 2, 2, nx // 2, 2).mean(dim=(-5, -3, -1))


def _upsample(v):
    for axis in range(3):
        n = v.shape[axis]
        j = torch.arange(n, device=v.device)
        below, above = (v.index_select(axis, k.clamp(0, n - 1)) for k in (j - 1, j + 1))
        v = torch.stack([0.75 * v + 0.25 * below, 0.75 * v + 0.25 * above], dim=axis + 1)
        v = v.reshape(*v.shape[:axis], 2 * n, *v.shape[axis + 2:])
    return v


class _Plain:
    """The network on one scene in float64 (differentiable in its parameters and its input)."""

    def __init__(self, params: torch.Tensor, levels: int, labels: torch.Tensor):
        self.levels, self.fluid, self.w, at = levels, labels == FLUID, {}, 0
        for name, lvl, n in _sizes(levels):
            self.w[name, lvl] = params[at:at + n]
            at += n
        self.image = [torch.stack([(labels == c).double() for c in range(3)])]
        for _ in range(levels - 1):
            self.image.append(_pool(self.image[-1]))

    def _image_windows(self, lvl):
        """I_c(p + o) for every channel c and offset o: (3, 27, cells)."""
        image = self.image[lvl - 1]
        return torch.stack([torch.stack([v.reshape(-1) for v in _windows(image[c], 1.0 if c == SOLID else 0.0)])
                            for c in range(3)])

    def cconv(self, block, lvl, r):
        n = r.numel()
        parts = math.gcd(n, 4096)   # many short products rather than one long one
        cut = lambda v: v.reshape(-1, parts, n // parts).transpose(0, 1).contiguous()   # noqa: E731
        kernels = torch.matmul(self.w[block + "W", lvl].reshape(27, 81), cut(self._image_windows(lvl).reshape(81, n)))
        kernels = kernels + self.w[block + "B", lvl][:, None]
        window = cut(torch.stack([v.reshape(-1) for v in _windows(r, 0.0)]))
        return (kernels * window).sum(1).reshape(r.shape)

    def aff(self, block, lvl):
        w = self.w[block + "W", lvl].reshape(3, 27)
        sums = self._image_windows(lvl).sum(-1)
        return self.w[block + "B", lvl][0] + (w * sums).sum() / (27.0 * self.image[lvl - 1][0].numel())

    def apply(self, r):
        r, x1 = r * self.fluid, {}
        for lvl in range(1, self.levels):
            x1[lvl] = self.cconv("c1", lvl, r)
            r = _pool(x1[lvl])
        x = self.cconv("c1", self.levels, r)
        for lvl in range(self.levels - 1, 0, -1):
            x = self.aff("a1", lvl) * x1[lvl] + self.aff("a2", lvl) * self.cconv("c2", lvl, _upsample(x))
        return x * self.fluid


class _Matrix:
    """The mixed-boundary 7-point matrix of a scene in float64."""

    FACES = (4, 10, 12, 14, 16, 22)   # the face neighbours among the 27 offsets

    def __init__(self, labels):
        self.fluid = (labels == FLUID).double()
        wet = list(_windows((labels != SOLID).double(), 0.0))
        self.diagonal = sum(wet[k] for k in self.FACES) * self.fluid

    def times(self, x):
        x = x * self.fluid
        near = list(_windows(x, 0.0))
        return (self.diagonal * x - sum(near[k] for k in self.FACES)) * self.fluid

    def solve(self, b, tol=1e-12, most=6000):
        """Conjugate gradients, preconditioned by the diagonal."""
        inverse = torch.where(self.diagonal > 0, 1.0 / self.diagonal.clamp(min=1.0), torch.zeros_like(b))
        x, r = torch.zeros_like(b), b * self.fluid
        z = inverse * r
        d, rz, stop = z.clone(), (r * z).sum(), tol * float(r.norm())
        for k in range(most):
            ad = self.times(d)
            alpha = rz / (d * ad).sum()
            x, r = x + alpha * d, r - alpha * ad
            if k % 50 == 49 and float(r.norm()) < stop:
                break
            z = inverse * r
            rz, old = (r * z).sum(), rz
            d = z + (rz / old) * d
        return x


def exact(case, seed: int):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind == "serve":
        return [_Matrix(lab).solve(b).cpu().numpy() for lab, b in zip(s["labels"], s["b"])]
    if kind == "solve":
        return _Matrix(s["labels"]).solve(s["b"])
    params = torch.from_numpy(s["params"]).cuda()
    if kind == "precond":
        return _Plain(params, case["levels"], s["labels"]).apply(s["b"].double())
    if kind == "transpose":
        r = torch.zeros(_shape(case), dtype=torch.float64, device="cuda", requires_grad=True)
        y = _Plain(params, case["levels"], s["labels"]).apply(r)
        return torch.autograd.grad(y, r, s["b"].double())[0]
    params.requires_grad_(True)
    total = 0.0
    for lab, b in zip(s["labels"], s["b"].double()):
        y = _Plain(params, case["levels"], lab).apply(b)
        loss = (b - _Matrix(lab).times(y)).norm() / case["batch"]
        loss.backward()
        total += float(loss.detach())
    return {"loss": total, "grad": params.grad}
