"""The work that this framework is timed on: calls of its public entry points
over the range of sizes, orders, geometries, precisions and physics that its
own tests, workloads and benchmark use.

A case is a dict of plain values.  Five kinds:

* ``loop``     an explicit time loop: steps from rest or from a saved state,
               with a source and receivers; seismograms and the final state
* ``apply``    one internal-force apply f = -K u
* ``gradient`` a forward run with checkpoints and its discrete adjoint
* ``infer``    a surrogate network's forward pass over a batch
* ``train``    training steps of that network over minibatches (forward, loss,
               backward, Adam) and its weights after them

Inputs are made here with numpy from the case and the seed alone.  ``exact``
evaluates the same mathematics in FP64 with plain torch.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2606_12850_amd as P

# The listed cases, chosen by use:
#   cube4       the parity cube (4^3 elements, NGLL 5, 10 Hz source at the centre, 200 steps, from rest): the
#               smallest run, bound by launches
#   layered64   the throughput run: 64^3 jittered elements in three layers, NGLL 5, geometry rebuilt on the fly,
#               a production run resumed from a saved state
#   ragged5     a force apply on a jittered box of odd extents with the default (stored) geometry
#   box8        a force apply at NGLL 8 on regular elements: the middle of the order sweep
#   box16       the same at NGLL 16, the largest order
#   mixed12     BF16 contractions at NGLL 12, where they are faster than FP32
#   fd64bit     an FP64 run on a regular cube, as the finite-difference check of a gradient makes many of
#   rod8        the acoustic rod of the equal-accuracy experiment at p = 7
#   batch16     sixteen models on one 16^3 mesh: the surrogate's training data
#   gradient24  sensitivity kernels on a regular cube from 64 receivers
#   infer4096   surrogate inference, the largest batch, 64 -> 3 x 512 -> 16 receivers x 3 x 512 samples
#   train128    its training at the default batch
_LISTED = [
    {"name": "cube4", "kind": "loop", "n": 5, "nx": 4, "ny": 4, "nz": 4, "jitter": 0.0, "geometry": "stored",
     "dtype": "f32", "physics": "elastic", "models": 1, "steps": 200, "resume": False},
    {"name": "layered64", "kind": "loop", "n": 5, "nx": 64, "ny": 64, "nz": 64, "jitter": 0.1,
     "geometry": "trilinear", "dtype": "f32", "physics": "elastic", "models": 1, "steps": 40, "resume": True},
    {"name": "ragged5", "kind": "apply", "n": 5, "nx": 33, "ny": 31, "nz": 37, "jitter": 0.1, "geometry": "stored",
     "dtype": "f32", "mode": "f32", "physics": "elastic"},
    {"name": "box8", "kind": "apply", "n": 8, "nx": 24, "ny": 24, "nz": 24, "jitter": 0.0, "geometry": "stored",
     "dtype": "f32", "mode": "f32", "physics": "elastic"},
    {"name": "box16", "kind": "apply", "n": 16, "nx": 11, "ny": 10, "nz": 10, "jitter": 0.0, "geometry": "stored",
     "dtype": "f32", "mode": "f32", "physics": "elastic"},
    {"name": "mixed12", "kind": "apply", "n": 12, "nx": 13, "ny": 14, "nz": 13, "jitter": 0.0, "geometry": "stored",
     "dtype": "f32", "mode": "bf16", "physics": "elastic"},
    {"name": "fd64bit", "kind": "loop", "n": 5, "nx": 16, "ny": 16, "nz": 16, "jitter": 0.0, "geometry": "stored",
     "dtype": "f64", "physics": "elastic", "models": 1, "steps": 60, "resume": False},
    {"name": "rod8", "kind": "loop", "n": 8, "nx": 270, "ny": 1, "nz": 1, "jitter": 0.0, "geometry": "stored",
     "dtype": "f32", "physics": "acoustic", "models": 1, "steps": 300, "resume": True},
    {"name": "batch16", "kind": "loop", "n": 5, "nx": 16, "ny": 16, "nz": 16, "jitter": 0.0, "geometry": "stored",
     "dtype": "f32", "physics": "elastic", "models": 16, "steps": 80, "resume": False},
    {"name": "gradient24", "kind": "gradient", "n": 5, "nx": 24, "ny": 24, "nz": 24, "jitter": 0.0,
     "geometry": "stored", "steps": 60, "every": 20},
    {"name": "infer4096", "kind": "infer", "batch": 4096, "inputs": 64, "hidden": 512, "layers": 3, "outputs": 24576},
    {"name": "train128", "kind": "train", "batch": 128, "inputs": 64, "hidden": 512, "layers": 3, "outputs": 24576,
     "steps": 40},
]

_MAX_NODES = 4_000_000  # of a drawn mesh (the largest listed one has 17 million)


def listed():
    return [dict(c) for c in _LISTED]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _extents(rng, n, nodes):
    """Element counts of a box of about `nodes` nodes, with aspect ratios up to about 3."""
    side = max(1.0, nodes ** (1.0 / 3.0) / (n - 1))
    dims = [max(1, int(round(side * math.exp(rng.uniform(-0.5, 0.5))))) for _ in range(3)]
    while np.prod([(n - 1) * d + 1 for d in dims]) > _MAX_NODES:
        k = dims.index(max(dims))
        dims[k] = max(1, dims[k] * 4 // 5)
        if max(dims) == 1:
            break
    return dims


def draw(rng):
    kind = rng.choice(["loop", "loop", "loop", "apply", "apply", "apply", "apply", "gradient", "infer", "train"])
    if kind in ("infer", "train"):
        case = {"kind": kind, "batch": _log_int(rng, 1, 4096) if kind == "infer" else _log_int(rng, 16, 256),
                "inputs": rng.choice([27, 64]), "hidden": rng.choice([64, 200, 256, 512]),
                "layers": rng.choice([1, 2, 3]), "outputs": _log_int(rng, 48, 24576)}
        return case if kind == "infer" else dict(case, steps=rng.randint(10, 40))
    geometry = rng.choice(["stored", "trilinear"])
    jitter = rng.choice([0.0, 0.1])
    if kind == "gradient":
        n = rng.choice([4, 5, 6, 8])
        nx, ny, nz = _extents(rng, n, _log_int(rng, 5_000, 900_000))
        return {"kind": kind, "n": n, "nx": nx, "ny": ny, "nz": nz, "jitter": jitter, "geometry": geometry,
                "steps": rng.randint(21, 60), "every": rng.randint(10, 20)}
    physics = rng.choice(["elastic", "elastic", "elastic", "acoustic"])
    dtype = "f64" if physics == "elastic" and rng.random() < 0.15 else "f32"
    n = rng.choice([3, 4, 5, 5, 5, 6, 7, 8, 9, 10] if dtype == "f64" else [3, 4, 5, 5, 5, 5, 6, 7, 8, 8, 9, 10, 11, 12,
                                                                            13, 14, 15, 16, 16])
    nodes = _log_int(rng, 3_000, _MAX_NODES if dtype == "f32" else _MAX_NODES // 4)
    case = {"kind": kind, "n": n, "jitter": jitter, "geometry": geometry, "dtype": dtype, "physics": physics}
    if kind == "loop":
        case["models"] = rng.choice([1, 1, 1, 4]) if dtype == "f32" and physics == "elastic" else 1
        nodes = nodes // case["models"]
        case["steps"] = rng.randint(20, 60)
        case["resume"] = rng.choice([True, False])
    else:
        case["mode"] = "f32"
        if dtype == "f32" and physics == "elastic" and n >= 11 and rng.random() < 0.4:
            case["mode"] = rng.choice(["bf16", "f16"])
    case["nx"], case["ny"], case["nz"] = _extents(rng, n, nodes)
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

@functools.lru_cache(maxsize=None)
def _gll(n):
    """GLL nodes, weights and derivative matrix (FP64)."""
    c = np.zeros(n)
    c[-1] = 1.0
    inner = np.polynomial.legendre.legroots(np.polynomial.legendre.legder(c)) if n > 2 else np.zeros(0)
    d1 = np.polynomial.legendre.legder(c)
    d2 = np.polynomial.legendre.legder(d1)
    for _ in range(3):  # polish the roots
        if n > 2:
            inner = inner - np.polynomial.legendre.legval(inner, d1) / np.polynomial.legendre.legval(inner, d2)
    x = np.concatenate([[-1.0], np.sort(inner), [1.0]])
    w = 2.0 / (n * (n - 1) * np.polynomial.legendre.legval(x, c) ** 2)
    dx = x[:, None] - x[None, :]
    np.fill_diagonal(dx, 1.0)
    bary = 1.0 / dx.prod(axis=1)
    D = bary[None, :] / bary[:, None] / dx
    np.fill_diagonal(D, 0.0)
    np.fill_diagonal(D, -D.sum(axis=1))
    return x, w, D


@functools.lru_cache(maxsize=2)
def _numbering(n, nx, ny, nz):
    """ibool [nspec, n^3] and elem_vert [nspec, 8] of a structured box."""
    N = n - 1
    Gx, Gy = nx * N + 1, ny * N + 1
    a = np.arange(n)
    local = (a[None, None, :] + Gx * (a[None, :, None] + Gy * a[:, None, None])).ravel().astype(np.int32)
    ez, ey, ex = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    base = (ex * N + Gx * (ey * N + Gy * (ez * N))).ravel().astype(np.int32)
    corner = np.array([i + (nx + 1) * (j + (ny + 1) * k) for k in (0, 1) for j in (0, 1) for i in (0, 1)], np.int32)
    vbase = (ex + (nx + 1) * (ey + (ny + 1) * ez)).ravel().astype(np.int32)
    return base[:, None] + local[None, :], vbase[:, None] + corner[None, :]


class _Mesh:
    """What Solver.upload_mesh reads."""

    def __init__(self, case, rng):
        self.n, self.nx, self.ny, self.nz = case["n"], case["nx"], case["ny"], case["nz"]
        self.h = _H * (self.n - 1)
        self.ibool, self.elem_vert = _numbering(self.n, self.nx, self.ny, self.nz)
        self.nspec = self.ibool.shape[0]
        self.shape = tuple((self.n - 1) * m + 1 for m in (self.nz, self.ny, self.nx))  # lattice, x fastest
        self.nglob = int(np.prod(self.shape))
        z, y, x = np.meshgrid(*(np.arange(m + 1) * self.h for m in (self.nz, self.ny, self.nx)), indexing="ij")
        vert = np.stack([x, y, z], axis=-1)
        if case["jitter"]:
            move = rng.uniform(-case["jitter"] * self.h, case["jitter"] * self.h, vert.shape)
            vert[1:-1, 1:-1, 1:-1] += move[1:-1, 1:-1, 1:-1]
        self.vert = vert.reshape(-1, 3)


_H = 15.625     # average node spacing in metres (64 elements of NGLL 5 in 4 km)
_VPVS = 1.73
_RHO = 2500.0


def _waves(rng, shape, count, shortest, dtype=np.float64):
    """A sum of `count` cosines on the node lattice, wavelengths from `shortest` nodes up, of unit order."""
    out = np.zeros(shape, dtype)
    for _ in range(count):
        axes = []
        for m in shape:
            k = 2.0 * math.pi / rng.uniform(shortest, 6.0 * shortest)
            axes.append(np.cos(k * np.arange(m) + rng.uniform(0.0, 2.0 * math.pi)).astype(dtype))
        out += axes[0][:, None, None] * (axes[1][:, None] * axes[2][None, :])[None]
    return out / math.sqrt(count)


def _field(rng, mesh, models, comps, scale):
    """A broad-band wave field [models][nglob][comps], down to about five nodes per wavelength."""
    f = np.stack([_waves(rng, mesh.shape, 3, 5.0, np.float32).ravel() for _ in range(comps)], axis=-1) * scale
    if models > 1:
        f = f[None] * rng.uniform(0.5, 1.0, (models, 1, 1)).astype(np.float32)
    return np.ascontiguousarray(f if comps == 3 else f[..., 0], dtype=np.float32)


def _model(case, mesh, rng, models):
    """(moduli..., rho) per element-local point: three layers with a smooth +-5 % perturbation."""
    n3 = mesh.n ** 3
    pert = 1.0 + 0.05 * np.clip(_waves(rng, mesh.shape, 2, 8.0 * (mesh.n - 1)), -1.0, 1.0).ravel()
    vp = pert[mesh.ibool]
    if case.get("physics") == "acoustic":
        kappa = 1000.0 * (1500.0 * vp) ** 2
        return kappa, np.full_like(kappa, 1000.0)
    layer = np.repeat(np.arange(mesh.nz) * 3 // mesh.nz, mesh.nx * mesh.ny)
    vp *= np.array([6000.0, 4000.0, 2500.0])[layer][:, None]
    mu = vp * vp
    lam = mu * (_RHO * (1.0 - 2.0 / _VPVS ** 2))
    mu *= _RHO / _VPVS ** 2
    rho = np.full((mesh.nspec, n3), _RHO)
    if models > 1:
        s = (1.0 + 0.1 * rng.uniform(-1.0, 1.0, (models, 1, 1)))
        return lam[None] * s, mu[None] * s, np.repeat(rho[None], models, axis=0)
    return lam, mu, rho


def _dt(case, mesh):
    """About 0.4 of the smallest node distance over the largest wave speed."""
    x, _, _ = _gll(mesh.n)
    vmax = 1500.0 * 1.05 if case.get("physics") == "acoustic" else 6000.0 * 1.05
    return 0.4 * 0.5 * (x[1] - x[0]) * mesh.h * (0.8 if case["jitter"] else 1.0) / vmax


class _Run:
    """Host inputs of a time loop."""

    def __init__(self, case, mesh, rng):
        nt, self.dt = case["steps"], _dt(case, mesh)
        mid = (mesh.nx // 2) + mesh.nx * ((mesh.ny // 2) + mesh.ny * (mesh.nz // 2))
        self.src_elem = np.array([mid], np.int32)
        self.src_xi = rng.uniform(-0.9, 0.9, (1, 3))
        self.src_dir = np.array([[0.1, -0.2, 1.0]])
        # a wavelet of a few dozen steps, so that a short run meets all of it
        t = np.arange(nt + 2) * self.dt
        f0 = 1.0 / (20.0 * self.dt)
        a = (math.pi * f0 * (t - 1.2 / f0)) ** 2
        self.stf = (1.0e9 * (1.0 - 2.0 * a) * np.exp(-a))[None, :].astype(np.float32)
        m = 64 if case["kind"] == "gradient" else 8
        ex, ey, ez = (rng.integers(max(0, c // 2 - 3), min(c, c // 2 + 4), m) for c in (mesh.nx, mesh.ny, mesh.nz))
        self.rec_elem = (ex + mesh.nx * (ey + mesh.ny * ez)).astype(np.int32)
        self.rec_xi = rng.uniform(-1.0, 1.0, (m, 3))


def _host(case, seed):
    """Everything of a wave case that lies in host memory before the call."""
    rng = np.random.default_rng([int(seed), 2606])
    mesh = _Mesh(case, rng)
    models = case.get("models", 1)
    model = _model(case, mesh, rng, models)
    comps = 1 if case.get("physics") == "acoustic" else 3
    run = u = v = gseis = None
    if case["kind"] != "apply":
        run = _Run(case, mesh, rng)
    if case["kind"] == "apply" or case.get("resume"):
        u = _field(rng, mesh, models, comps, 1.0e-3)
    if case.get("resume"):
        v = _field(rng, mesh, models, comps, 1.0e-3 * (1500.0 if comps == 1 else 3000.0) / (8.0 * _H))
    if case["kind"] == "gradient":
        gseis = rng.standard_normal((64, 3, case["steps"])).astype(np.float32)
    return mesh, model, run, u, v, gseis


def _solver(case, mesh, model):
    acoustic = case.get("physics") == "acoustic"
    s = P.Solver(case["n"], "cuda:0", storage=P.SEMX_F64 if case.get("dtype") == "f64" else P.SEMX_F32,
                 physics=P.SEMX_ACOUSTIC if acoustic else P.SEMX_ELASTIC)
    s.upload_mesh(mesh)
    if case["geometry"] == "trilinear":
        P.semx_set_geometry(s.ctx, P.SEMX_GEOM_TRILINEAR)
    if acoustic:
        s.upload_model_acoustic(*model)
    else:
        s.upload_model(*model)
    if case.get("mode", "f32") != "f32":
        s.set_mode(P.SEMX_C_BF16 if case["mode"] == "bf16" else P.SEMX_C_F16)
    return s


_MINIBATCHES = 4  # of a training run, taken in turn


def _network(case, seed):
    """Packed parameters, inputs and targets."""
    rng = np.random.default_rng([int(seed), 12850])
    widths = [case["inputs"]] + [case["hidden"]] * case["layers"] + [case["outputs"]]
    parts = []
    for a, b in zip(widths[:-1], widths[1:]):
        parts.append(rng.uniform(-1.0, 1.0, a * b).astype(np.float32) * math.sqrt(6.0 / a))
        parts.append(rng.uniform(-0.1, 0.1, b).astype(np.float32))
    lead = (_MINIBATCHES, case["batch"]) if case["kind"] == "train" else (case["batch"],)
    x = rng.standard_normal(lead + (case["inputs"],), dtype=np.float32)
    t = rng.standard_normal(lead + (case["outputs"],), dtype=np.float32) if case["kind"] == "train" else None
    return widths, np.concatenate(parts), x, t


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.case = case
    if case["kind"] in ("infer", "train"):
        from paper_2606_12850_amd.surrogate import MLP
        widths, theta, x, t = _network(case, seed)
        s.net = MLP(widths, case["batch"])
        s.net.set_params(theta)
        s.x = torch.from_numpy(x).cuda()
        s.t = None if t is None else torch.from_numpy(t).cuda()
        return s
    mesh, model, run, u, v, gseis = _host(case, seed)
    if case["kind"] == "gradient":
        from paper_2606_12850_amd.autograd import SeismogramOperator
        s.op = SeismogramOperator(mesh, run.src_elem, run.src_xi, run.src_dir, run.stf, run.rec_elem, run.rec_xi,
                                  run.dt, case["steps"], checkpoint_every=case["every"],
                                  geometry=P.SEMX_GEOM_TRILINEAR if case["geometry"] == "trilinear" else None)
        s.op.run(*model)
        s.gseis = torch.from_numpy(gseis).cuda()
        s.seis = torch.empty((1, 64, 3, case["steps"]), dtype=torch.float32, device="cuda")
        return s
    s.solver = _solver(case, mesh, model)
    real = torch.float64 if case["dtype"] == "f64" else torch.float32
    if u is not None:
        s.u = torch.from_numpy(u).to("cuda", real)
    if case["kind"] == "apply":
        s.f = s.solver.empty_field()
        return s
    if case["dtype"] == "f64":
        P.semx_set_sources_f64(s.solver.ctx, run.src_elem, run.src_xi, run.src_dir, run.stf)
    else:
        P.semx_set_sources(s.solver.ctx, run.src_elem, run.src_xi, run.src_dir, run.stf)
    P.semx_set_receivers(s.solver.ctx, run.rec_elem, run.rec_xi, case["steps"])
    s.solver.nrec, s.solver.nt_max = len(run.rec_elem), case["steps"]
    P.semx_set_dt(s.solver.ctx, run.dt)
    if v is not None:
        s.v = torch.from_numpy(v).to("cuda", real)
        s.a = torch.zeros_like(s.v)
    s.out = [s.solver.empty_field() for _ in range(2)]
    return s


def run(s):
    case = s.case
    if case["kind"] == "infer":
        return s.net.forward(s.x)
    if case["kind"] == "train":
        for k in range(case["steps"]):
            s.net.train_step(s.x[k % _MINIBATCHES], s.t[k % _MINIBATCHES], 1.0e-4)
        return s.net.params()
    if case["kind"] == "gradient":
        ctx = s.op.solver.ctx
        P.semx_reset(ctx)
        P.semx_step(ctx, case["steps"])
        P.semx_read_seismograms(ctx, s.seis, True)
        lam, mu, rho = s.op.gradient(s.gseis)
        return {"seis": s.seis, "lam": lam, "mu": mu, "rho": rho}
    if case["kind"] == "apply":
        return s.solver.apply_force(s.u, s.f)
    ctx, f64 = s.solver.ctx, case["dtype"] == "f64"
    if case["resume"]:
        (P.semx_set_state_f64 if f64 else P.semx_set_state)(ctx, s.u, s.v, s.a, 0)
    else:
        P.semx_reset(ctx)
    P.semx_step(ctx, case["steps"])
    (P.semx_get_state_f64 if f64 else P.semx_get_state)(ctx, s.out[0], s.out[1])
    return {"seis": s.solver.seismograms(), "u": s.out[0], "v": s.out[1]}


def work(case):
    """Inputs read once, outputs written once, per step of a loop."""
    if case["kind"] in ("infer", "train"):
        widths = [case["inputs"]] + [case["hidden"]] * case["layers"] + [case["outputs"]]
        params = sum(a * b + b for a, b in zip(widths[:-1], widths[1:]))
        macs = sum(a * b for a, b in zip(widths[:-1], widths[1:])) * case["batch"]
        io = 4 * case["batch"] * (case["inputs"] + case["outputs"])
        if case["kind"] == "infer":
            return {"bytes": 2 * params + io, "flops": 2 * macs}
        # per step: the 16-bit weights read twice and written, gradients written and read, Adam's three arrays read
        # and written; the weights copied to the host once
        return {"bytes": case["steps"] * (params * (4 + 2 + 8 + 24) + io) + 4 * params, "flops": 6 * macs * case["steps"]}
    n, spec = case["n"], case["nx"] * case["ny"] * case["nz"]
    n3, nodes = n ** 3, ((n - 1) * case["nx"] + 1) * ((n - 1) * case["ny"] + 1) * ((n - 1) * case["nz"] + 1)
    real = 8 if case.get("dtype") == "f64" else 4
    comps = 1 if case.get("physics") == "acoustic" else 3
    models = case.get("models", 1)
    geo = (9 * n3 if case["geometry"] == "stored" and case["jitter"] else 24 if case["jitter"] else 9) * real * spec
    mat = models * spec * n3 * real * (1 if comps == 1 else 2)
    # contractions in three directions and back, and the pointwise map, stress and flux
    flops = models * spec * n3 * (12 * n * comps + (150 if comps == 3 else 40))
    if case["kind"] == "apply":
        return {"bytes": geo + mat + 2 * comps * real * nodes, "flops": flops}
    step = geo + mat + models * nodes * real * (4 * comps + 1)
    if case["kind"] == "loop":
        return {"bytes": case["steps"] * step, "flops": case["steps"] * flops}
    # gradient: the forward run, its recomputation, and the adjoint steps with three FP64 accumulators
    adj = geo + mat + nodes * real * (3 * 5 + 1) + spec * n3 * (3 * 16 + 8)
    return {"bytes": case["steps"] * (2 * step + adj), "flops": case["steps"] * 4 * flops}


# ---------------------------------------------------------------------------
# the same in FP64, plain torch
# ---------------------------------------------------------------------------

def _lagrange(x, at):
    out = np.ones(len(x))
    for a in range(len(x)):
        for b in range(len(x)):
            if a != b:
                out[a] *= (at - x[b]) / (x[a] - x[b])
    return out


class _Exact:
    """The operator in FP64 on the GPU (or the CPU where there is none)."""

    def __init__(self, case, mesh, model):
        self.dev = "cuda" if torch.cuda.is_available() else "cpu"
        self.n, self.nglob = mesh.n, mesh.nglob
        self.mesh = mesh
        x, w, D = _gll(mesh.n)
        t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device=self.dev)  # noqa: E731
        self.D, self.x = t(D), x
        self.ib = torch.as_tensor(mesh.ibool, device=self.dev).long()
        X = t(mesh.vert)[torch.as_tensor(mesh.elem_vert, device=self.dev).long()].reshape(-1, 2, 2, 2, 3)  # c, b, a
        L = t(np.stack([(1.0 - x) / 2.0, (1.0 + x) / 2.0], axis=1))  # [n][2]
        dL = t(np.repeat([[-0.5, 0.5]], mesh.n, axis=0))

        def mapped(lz, ly, lx):
            y = torch.tensordot(X, lx, dims=([3], [1]))       # e c b 3 i
            y = torch.tensordot(y, ly, dims=([2], [1]))       # e c 3 i j
            y = torch.tensordot(y, lz, dims=([1], [1]))       # e 3 i j k
            return y.permute(0, 4, 3, 2, 1)                    # e k j i 3

        J = torch.stack([mapped(L, L, dL), mapped(L, dL, L), mapped(dL, L, L)], dim=-1)  # e k j i 3(x) 3(xi)
        det = torch.linalg.det(J)
        self.G = torch.linalg.inv(J)                          # [.., xi d][x b]
        ww = t(w)
        self.W = det * (ww[:, None, None] * ww[None, :, None] * ww[None, None, :])
        shape = (mesh.nspec,) + (mesh.n,) * 3
        self.acoustic = case.get("physics") == "acoustic"
        self.par = [t(m).reshape(shape) for m in model]
        dens = 1.0 / self.par[0] if self.acoustic else self.par[2]
        self.minv = 1.0 / self.assemble((dens * self.W).reshape(mesh.nspec, -1, 1))

    def assemble(self, e):
        out = torch.zeros((self.nglob, e.shape[-1]), dtype=torch.float64, device=self.dev)
        return out.index_add_(0, self.ib.reshape(-1), e.reshape(-1, e.shape[-1]))

    def gradient(self, u):
        """d u_c / d x_b at every point: [e, k, j, i, c, b]."""
        n = self.n
        ue = u[self.ib].reshape(-1, n, n, n, u.shape[-1])
        d = torch.stack([torch.tensordot(ue, self.D, dims=([3], [1])).permute(0, 1, 2, 4, 3),
                         torch.tensordot(ue, self.D, dims=([2], [1])).permute(0, 1, 4, 2, 3),
                         torch.tensordot(ue, self.D, dims=([1], [1])).permute(0, 4, 1, 2, 3)], dim=-1)
        return d @ self.G

    def force(self, u):
        g = self.gradient(u)
        if self.acoustic:
            s = g / self.par[1][..., None, None]
        else:
            lam, mu, _ = self.par
            s = mu[..., None, None] * (g + g.transpose(-1, -2))
            tr = lam * (g[..., 0, 0] + g[..., 1, 1] + g[..., 2, 2])
            for c in range(3):
                s[..., c, c] += tr
        del g
        phi = (s * self.W[..., None, None]) @ self.G.transpose(-1, -2)  # e k j i c d
        del s
        f = torch.tensordot(phi[..., 0], self.D, dims=([3], [0])).permute(0, 1, 2, 4, 3).clone()
        f += torch.tensordot(phi[..., 1], self.D, dims=([2], [0])).permute(0, 1, 4, 2, 3)
        f += torch.tensordot(phi[..., 2], self.D, dims=([1], [0])).permute(0, 4, 1, 2, 3)
        return -self.assemble(f.reshape(f.shape[0], -1, f.shape[-1]))

    def weights(self, elem, xi):
        """Nodes and interpolation weights of points: [m, n^3] each."""
        w = np.stack([np.einsum("k,j,i->kji", *(_lagrange(self.x, p[d]) for d in (2, 1, 0))).ravel() for p in xi])
        return (self.ib[torch.as_tensor(np.asarray(elem), device=self.dev).long()],
                torch.as_tensor(w, dtype=torch.float64, device=self.dev))


def _exact_loop(case, op, run, u, v, keep=False):
    comps = 1 if op.acoustic else 3
    sn, sw = op.weights(run.src_elem, run.src_xi)
    rn, rw = op.weights(run.rec_elem, run.rec_xi)
    direction = torch.as_tensor(run.src_dir if comps == 3 else np.ones((1, 1)), dtype=torch.float64, device=op.dev)
    stf = run.stf.astype(np.float64)

    def source(f, m):
        return f.index_add_(0, sn.reshape(-1), (float(stf[0, m]) * sw[:, :, None] * direction[:, None, :]).reshape(-1, comps))

    zero = torch.zeros((op.nglob, comps), dtype=torch.float64, device=op.dev)
    u, v = zero.clone() if u is None else u.clone(), zero.clone() if v is None else v.clone()
    a = zero.clone() if case.get("resume") else op.minv * source(zero.clone(), 0)
    dt, seis, us, acc = run.dt, [], [], []
    for m in range(case["steps"]):
        u = u + dt * v + 0.5 * dt * dt * a
        v = v + 0.5 * dt * a
        seis.append((rw[:, :, None] * u[rn]).sum(dim=1))
        a = op.minv * source(op.force(u), m + 1)
        v = v + 0.5 * dt * a
        if keep:
            us.append(u)
            acc.append(a)
    return torch.stack(seis, dim=-1), u, v, us, acc


def _exact_gradient(case, op, run, gseis):
    """The discrete adjoint of the recursion above for d chi / d seis = gseis."""
    seis, _, _, us, acc = _exact_loop(case, op, run, None, None, keep=True)
    rn, rw = op.weights(run.rec_elem, run.rec_xi)
    g = torch.as_tensor(gseis, dtype=torch.float64, device=op.dev)
    dt2, nt = run.dt ** 2, case["steps"]
    p2, p1 = torch.zeros_like(us[0]), torch.zeros_like(us[0])  # psi^{m+2}, psi^{m+1}
    gl, gm, gr = (torch.zeros_like(op.W) for _ in range(3))
    local = lambda w: w[op.ib].reshape(op.W.shape + (3,))  # noqa: E731
    for m in range(nt, 0, -1):
        rhs = torch.zeros_like(p1)
        if m < nt:
            rhs = dt2 * op.force(p1)
            a, b = op.gradient(p1), op.gradient(us[m - 1])
            gl -= dt2 * op.W * a.diagonal(dim1=-2, dim2=-1).sum(-1) * b.diagonal(dim1=-2, dim2=-1).sum(-1)
            gm -= dt2 * op.W * 0.5 * ((a + a.transpose(-1, -2)) * (b + b.transpose(-1, -2))).sum((-1, -2))
            gr -= dt2 * op.W * (local(p1) * local(acc[m - 1])).sum(-1)
        rhs.index_add_(0, rn.reshape(-1), (rw[:, :, None] * g[:, None, :, m - 1]).reshape(-1, 3))
        p2, p1 = p1, 2.0 * p1 - p2 + op.minv * rhs
    gr -= op.W * (local(p1) * local(us[0])).sum(-1)
    back = lambda t: t.reshape(1, op.W.shape[0], -1)  # noqa: E731
    return {"seis": seis[None], "lam": back(gl), "mu": back(gm), "rho": back(gr)}


def _exact_network(case, seed):
    widths, theta, x, t = _network(case, seed)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    th, x = (torch.as_tensor(a, dtype=torch.float64, device=dev) for a in (theta, x))

    def forward(th, h):
        at = 0
        for k, (a, b) in enumerate(zip(widths[:-1], widths[1:])):
            h = h @ th[at:at + a * b].reshape(b, a).T + th[at + a * b:at + a * b + b]
            at += a * b + b
            if k + 2 < len(widths):
                h = torch.nn.functional.silu(h)
        return h

    if case["kind"] == "infer":
        return forward(th, x)
    m, v = torch.zeros_like(th), torch.zeros_like(th)
    for k in range(case["steps"]):
        th.requires_grad_(True)
        y = forward(th, x[k % _MINIBATCHES])
        target = torch.as_tensor(t[k % _MINIBATCHES], dtype=torch.float64, device=dev)
        g, = torch.autograd.grad(((y - target) ** 2).mean(), th)
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        th = th.detach() - 1.0e-4 * (m / (1.0 - 0.9 ** (k + 1))) / ((v / (1.0 - 0.999 ** (k + 1))).sqrt() + 1.0e-8)
    return th


def exact(case, seed):
    if case["kind"] in ("infer", "train"):
        return _exact_network(case, seed)
    mesh, model, run, u, v, gseis = _host(case, seed)
    models = case.get("models", 1)
    outs = []
    for k in range(models):
        op = _Exact(case, mesh, [m[k] for m in model] if models > 1 else model)
        f = lambda w: None if w is None else torch.as_tensor(  # noqa: E731
            w[k] if models > 1 else w, dtype=torch.float64, device=op.dev).reshape(mesh.nglob, -1)
        one = (lambda w: w) if not op.acoustic else (lambda w: w.reshape(mesh.nglob))
        if case["kind"] == "gradient":
            return _exact_gradient(case, op, run, gseis)
        if case["kind"] == "apply":
            return one(op.force(f(u)))
        seis, uu, vv, _, _ = _exact_loop(case, op, run, f(u), f(v))
        outs.append({"seis": seis, "u": one(uu), "v": one(vv)})
    return outs[0] if models == 1 else {k: torch.stack([o[k] for o in outs]) for k in outs[0]}
