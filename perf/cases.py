"""Performance cases of the wave-propagation library: the work its users have
it do, through the Python entry points.

``listed()`` names them and ``draw(rng)`` gives more of the same ranges:

  step     Case.step: time steps of one analysis
  batch    Batch.step: time steps of several models of uneven meshes together
  apply    Case.apply, FP64 (callers that compose their own solvers)
  apply32  Case.apply_f32, the FP32 operator of the inner solves
  rhs      Case.rhs: the right-hand side of the next step
  forward  Mlp.forward: inference of the guess network
  train    Mlp.train: Adam steps of the guess network
  fit      fit_input: input estimation and misfit of one event

Meshes are boxes of cubic cells split into six quadratic tetrahedra, the
interior vertices moved by up to ``jitter`` of a cell.  A program keeps a
mesh for the many models and directions it analyses on it, so the mesh
handles of the last case are kept between calls of ``prepare``; the
materials, the input motion and the state come from the seed.
"""
from __future__ import annotations

import functools
import itertools
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2404_17754_amd as sw

DEV = torch.device("cuda", 0)

# (Vp, Vs, rho): sediment over bedrock
MATERIALS = np.array([[1600.0, 150.0, 1800.0], [2000.0, 500.0, 2000.0]])
EDGES = ((0, 1), (1, 2), (0, 2), (0, 3), (1, 3), (2, 3))
FACES = (((0, 1, 2), (4, 5, 6)), ((0, 1, 3), (4, 8, 7)), ((1, 2, 3), (5, 9, 8)), ((0, 2, 3), (6, 9, 7)))
WARM_STEPS = 8  # steps marched before the timed ones: the guesses have their past increments
RING = 6        # increments the projected guess spans


def _mesh_case(name, kind, nx, ny, nz, **more):
    c = {"name": name, "kind": kind, "nx": nx, "ny": ny, "nz": nz, "cell": 5.0, "dt": 0.005, "jitter": 0.0,
         "interface": 0.3}
    if kind == "step":
        c |= {"precision": "mixed", "guess": "proj", "rtol": 1e-10, "steps": 1}
    return c | more


def listed():
    return [
        # the smallest analysis (100 x 100 x 50 m, 10 m cells): launches and latency
        _mesh_case("step_small", "step", 10, 10, 5, cell=10.0, dt=0.01, interface=0.4),
        # plain FP64 PCG with the extrapolated guess, as parity runs march it; odd sizes, no lattice in the geometry
        _mesh_case("step_fp64", "step", 31, 27, 19, precision="fp64", guess="poly", jitter=0.2),
        # one candidate model of the smallest batched mesh, marched alone with the defaults
        _mesh_case("step_200m", "step", 40, 40, 20),
        # the large analysis (1000 x 1000 x 200 m, 9.6 M tets, 39 M degrees of freedom)
        _mesh_case("step_large", "step", 200, 200, 40),
        # the FP32 operator and the right-hand side (FP64 operator passes) of that mesh, alone
        _mesh_case("apply32_large", "apply32", 200, 200, 40),
        _mesh_case("rhs_large", "rhs", 200, 200, 40),
        # FP64 operator on an ordinary mesh without lattice structure, odd sizes
        _mesh_case("apply_ragged", "apply", 61, 47, 33, jitter=0.2),
        # six candidate models on the three batched meshes (200, 300 and 400 m), marched together
        {"name": "batch_uneven", "kind": "batch", "n200": 3, "n300": 2, "n400": 1, "interface": 0.3, "rtol": 1e-10},
        # inference over a million degrees of freedom
        {"name": "mlp_forward", "kind": "forward", "rows": 1 << 20},
        # training minibatches of the size the guess network is trained with
        {"name": "mlp_train", "kind": "train", "rows": 400000, "batch": 8192, "steps": 25},
        # the input of one event at 400 receivers, 1000 steps, 50 shifts
        {"name": "fit_event", "kind": "fit", "rec": 400, "stride": 20, "blocks": 50, "shifts": 50},
        # a short record at few receivers: the smallest fit
        {"name": "fit_small", "kind": "fit", "rec": 6, "stride": 10, "blocks": 15, "shifts": 15},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("step", "step", "apply", "apply32", "rhs", "batch", "forward", "train", "fit"))
    if kind == "batch":
        return {"kind": kind, "n200": rng.randint(1, 4), "n300": rng.randint(0, 2), "n400": rng.randint(0, 1),
                "interface": round(rng.uniform(0.2, 0.6), 3), "rtol": 1e-10}
    if kind == "forward":
        return {"kind": kind, "rows": _log(rng, 1000, 1 << 20)}
    if kind == "train":
        return {"kind": kind, "rows": _log(rng, 5000, 400000), "batch": _log(rng, 100, 8192), "steps": rng.randint(10, 25)}
    if kind == "fit":
        blocks = rng.randint(8, 50)
        return {"kind": kind, "rec": _log(rng, 4, 400), "stride": rng.randint(5, 20), "blocks": blocks,
                "shifts": rng.randint(4, blocks)}
    # boxes from a few hundred tets to about 2.4 million (the rest of the
    # range is one mesh, the large analysis', which takes long to build)
    nx = _log(rng, 4, 130)
    ny = max(3, min(130, int(nx * rng.uniform(0.6, 1.4))))
    nz = max(3, min(400000 // (nx * ny), int(nx * rng.uniform(0.3, 0.8)) + 2))
    c = _mesh_case("", kind, nx, ny, nz, jitter=rng.choice((0.0, 0.1, 0.2)), interface=round(rng.uniform(0.2, 0.6), 3),
                   dt=rng.choice((0.005, 0.01)))
    del c["name"]
    if kind == "step":
        c["precision"] = rng.choice(("mixed", "mixed", "fp64", "flex", "fp16"))
        c["guess"] = rng.choice(("proj", "poly"))
    return c


# ------------------------------------------------------------------ meshes

def _kuhn():
    """The six tets of a cell as half-cell offsets (6, 10, 3)."""
    tets = []
    for p in itertools.permutations(range(3)):
        e = 2 * np.eye(3, dtype=np.int64)
        v = [np.zeros(3, np.int64), e[p[0]], e[p[0]] + e[p[1]], np.full(3, 2)]
        if np.linalg.det(np.stack([v[1] - v[0], v[2] - v[0], v[3] - v[0]]).astype(float)) < 0:
            v[1], v[2] = v[2], v[1]
        tets.append(np.stack(v + [(v[a] + v[b]) // 2 for a, b in EDGES]))
    return np.stack(tets)


def _box(nx, ny, nz, cell, jitter):
    """Box mesh: nodes on the half-cell lattice, x fastest, surface at z = 0."""
    NX, NY, NZ = 2 * nx + 1, 2 * ny + 1, 2 * nz + 1
    xyz = np.empty((NZ, NY, NX, 3))
    xyz[..., 0] = np.arange(NX) * (cell / 2)
    xyz[..., 1] = (np.arange(NY) * (cell / 2))[:, None]
    xyz[..., 2] = ((np.arange(NZ) - NZ + 1) * (cell / 2))[:, None, None]
    if jitter > 0:
        r = np.random.default_rng([nx, ny, nz])
        xyz[2:-2:2, 2:-2:2, 2:-2:2] += r.uniform(-jitter * cell, jitter * cell, (nz - 1, ny - 1, nx - 1, 3))
        for dz, dy, dx in itertools.product((0, 1), repeat=3):
            if dz + dy + dx:  # edge nodes back to the middle of their edge
                lo = xyz[0:NZ - dz:2, 0:NY - dy:2, 0:NX - dx:2]
                hi = xyz[2 * dz::2, 2 * dy::2, 2 * dx::2]
                n = [min(a, b) for a, b in zip(lo.shape, hi.shape)][:3]
                xyz[dz::2, dy::2, dx::2] = 0.5 * (lo[:n[0], :n[1], :n[2]] + hi[:n[0], :n[1], :n[2]])
    xyz = xyz.reshape(-1, 3)
    off = _kuhn()
    off = ((off[..., 2] * NY + off[..., 1]) * NX + off[..., 0]).astype(np.int32)
    k, j, i = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    base = (((2 * k) * NY + 2 * j) * NX + 2 * i).astype(np.int32).ravel()
    tet10 = (base[:, None, None] + off[None]).reshape(-1, 10)
    # side (role 1) and base (role 2) faces
    edge = ((i == 0) | (i == nx - 1) | (j == 0) | (j == ny - 1) | (k == 0)).ravel()
    tets = (np.nonzero(edge)[0][:, None] * 6 + np.arange(6)).ravel()
    tri, own, role = [], [], []
    for v, e in FACES:
        f = tet10[tets][:, list(v)]
        px, py, pz = f % NX, f // NX % NY, f // (NX * NY)
        for on, r in ((px == 0, 1), (px == NX - 1, 1), (py == 0, 1), (py == NY - 1, 1), (pz == 0, 2)):
            s = np.nonzero(on.all(1))[0]
            tri.append(np.concatenate([f[s], tet10[tets[s]][:, list(e)]], 1))
            own.append(tets[s])
            role.append(np.full(len(s), r, np.uint8))
    return SimpleNamespace(xyz=xyz, tet10=tet10, tri6=np.concatenate(tri).astype(np.int32),
                           face_tet=np.concatenate(own).astype(np.int32), face_role=np.concatenate(role))


@functools.lru_cache(maxsize=3)
def _mesh(nx, ny, nz, cell, jitter):
    """The host mesh, its centroids and its device handle."""
    m = _box(nx, ny, nz, cell, jitter)
    m.centroid = m.xyz[m.tet10[:, :4]].mean(1).astype(np.float32)
    m.handle = sw.Mesh(_context(), m)
    return m


@functools.lru_cache(maxsize=1)
def _context():
    return sw.Context(0)


def _model(m, c, rng, n_steps):
    """One candidate model: a sediment layer of varying thickness, receivers
    on the surface, a stationary band-limited input motion."""
    nx, ny, nz, cell = c["nx"], c["ny"], c["nz"], c["cell"]
    depth = c["interface"] * nz * cell
    x, y = m.centroid[:, 0], m.centroid[:, 1]
    rough = np.zeros(len(x), np.float32)
    for _ in range(6):
        k = rng.normal(0.0, 2.0 * math.pi / (25.0 * cell), 2).astype(np.float32)
        rough += np.cos(k[0] * x + k[1] * y + np.float32(rng.uniform(0, 2 * math.pi)))
    soft = -m.centroid[:, 2] < depth * (1.0 + 0.05 * rough)
    NX, NY = 2 * nx + 1, 2 * ny + 1
    n = _receivers(c)
    gi, gj = (np.arange(n[0]) * NX // n[0]), (np.arange(n[1]) * NY // n[1])
    rec = (2 * nz * NY + gj[:, None]) * NX + gi[None]
    t = np.arange(n_steps + 1) * c["dt"]
    v = np.zeros((n_steps + 1, 3))
    for f in rng.uniform(0.5, 4.0, 24):  # several motions of unequal size, along x1 above all
        v += np.sin(2 * math.pi * f * t + rng.uniform(0, 2 * math.pi))[:, None] * rng.normal(0, 1, 3) * (0.2, 0.05, 0.05)
    w1, w2 = 2 * math.pi, 10 * math.pi
    return SimpleNamespace(mat=MATERIALS, tet_mat=np.where(soft, 0, 1).astype(np.uint8), rec_node=rec.ravel().astype(np.int32),
                           v_in=v, dt=c["dt"], n_steps=n_steps, ray_alpha=2 * 0.02 * w1 * w2 / (w1 + w2),
                           ray_beta=2 * 0.02 / (w1 + w2))


def _field(m, rng, amp):
    """Smooth random vector field at the nodes (3 * n_nodes values)."""
    size = m.xyz.max(0) - m.xyz.min(0)
    X = torch.from_numpy(m.xyz).to(DEV)
    out = torch.zeros_like(X)
    for _ in range(12):
        k = torch.from_numpy(rng.normal(0, 1.0, 3) * 2 * math.pi / np.minimum(size, 100.0)).to(DEV)
        out += torch.cos(X @ k + float(rng.uniform(0, 2 * math.pi)))[:, None] * torch.from_numpy(rng.normal(0, amp, 3)).to(DEV)
    return out.cpu().numpy().ravel()


def _size(c):
    """(nodes, tets, side and base faces)"""
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    return (2 * nx + 1) * (2 * ny + 1) * (2 * nz + 1), 6 * nx * ny * nz, 2 * (2 * nx * nz + 2 * ny * nz + nx * ny)


def _receivers(c):
    """Receivers per side: every surface node, at most 200 x 200 of them (the
    motion of the free surface is what an analysis yields)."""
    return min(200, 2 * c["nx"] + 1), min(200, 2 * c["ny"] + 1)


def _capacity(c):
    """Steps a case has room for (the march starts anew past them)."""
    nx, ny = _receivers(c)
    return max(200, min(20000, int(4e8 / (24 * nx * ny))))


def _start(c, seed, n_steps):
    rng = np.random.default_rng([seed, 17])
    m = _mesh(c["nx"], c["ny"], c["nz"], c["cell"], c["jitter"])
    return m, _model(m, c, rng, n_steps), rng


def _lanes(c):
    """The models of a batch: 100 m deep boxes of 200, 300 and 400 m."""
    return [_mesh_case("", "lane", n, n, 20, interface=c["interface"]) for n, key in ((40, "n200"), (60, "n300"), (80, "n400")) for _ in range(c[key])]


def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind == "step":
        cap = _capacity(c)
        m, model, rng = _start(c, seed, cap)
        case_ = sw.Case(_context(), m.handle, model, rtol=c["rtol"], precision=c["precision"], guess=c["guess"], proj_dim=RING)
        case_.set_state(v=_field(m, rng, 0.1))
        case_.step(WARM_STEPS)
        return {"kind": kind, "case": case_, "wave": case_.waveform_device(), "at": WARM_STEPS, "cap": cap, "n": c["steps"]}
    if kind == "batch":
        cap, cases = 600, []
        for i, lane in enumerate(_lanes(c)):
            m, model, rng = _start(lane, seed * 64 + i, cap)
            g = sw.Case(_context(), m.handle, model, rtol=c["rtol"], precision="mixed", guess="proj", proj_dim=RING)
            g.set_state(v=_field(m, rng, 0.1))
            cases.append(g)
        b = sw.Batch(_context(), cases)
        b.step(WARM_STEPS)
        return {"kind": kind, "case": b, "wave": [g.waveform_device() for g in cases], "at": WARM_STEPS, "cap": cap, "n": 1}
    if kind in ("apply", "apply32", "rhs"):
        m, model, rng = _start(c, seed, 8)
        g = sw.Case(_context(), m.handle, model, precision="mixed" if kind == "apply32" else "fp64")
        if kind == "rhs":
            g.set_state(*(_field(m, rng, a) for a in (1e-3, 0.1, 5.0)))
            return {"kind": kind, "case": g}
        x = torch.from_numpy(_field(m, rng, 1e-3)).to(DEV)
        x += 1e-4 * torch.randn(x.shape, dtype=x.dtype, device=DEV, generator=torch.Generator(DEV).manual_seed(seed))
        return {"kind": kind, "case": g, "x": x.float() if kind == "apply32" else x}
    if kind == "forward":
        return {"kind": kind, "net": sw.Mlp(_context(), _weights(seed)), "x": _rows(c["rows"], seed)[:, :10].contiguous()}
    if kind == "train":
        return {"kind": kind, "net": sw.Mlp(_context(), seed=seed), "rows": _rows(c["rows"], seed), "steps": c["steps"],
                "batch": c["batch"], "seed": seed}
    green, obs = _records(c, seed)
    return {"kind": "fit", "green": green, "obs": obs, "stride": c["stride"], "shifts": c["shifts"]}


def run(state):
    kind = state["kind"]
    if kind in ("step", "batch"):
        g, n = state["case"], state["n"]
        if state["at"] + n > state["cap"]:
            for one in g.cases if kind == "batch" else [g]:
                one.set_state(step=0)
            state["at"] = 0
        g.step(n)
        at = state["at"]
        state["at"] = at + n
        if kind == "batch":
            return [w[at:at + n] for w in state["wave"]]
        return state["wave"][at:at + n]
    if kind == "apply":
        return state["case"].apply("A", state["x"])
    if kind == "apply32":
        return state["case"].apply_f32("A", state["x"])
    if kind == "rhs":
        return state["case"].rhs()
    if kind == "forward":
        return state["net"].forward(state["x"])
    if kind == "train":
        losses = state["net"].train(state["rows"], steps=state["steps"], batch=state["batch"], lr=2e-3, seed=state["seed"])
        return {"losses": losses, "params": state["net"].params()}
    c, err, used, rank, U = sw.fit_input(_context(), state["green"], state["obs"], state["stride"], state["shifts"],
                                         return_response=True)
    return {"c": c, "err": err, "used": used, "rank": rank, "U": U}


# ------------------------------------------------- inputs without a mesh

def _weights(seed):
    """A network as training leaves it: hidden layers of Glorot size, small biases and output layer."""
    r = np.random.default_rng([seed, 3])
    parts = (r.uniform(-0.28, 0.28, 640), r.normal(0, 0.05, 64), r.uniform(-0.22, 0.22, 4096), r.normal(0, 0.05, 64),
             r.normal(0, 0.02, 64), r.normal(0, 0.01, 1))
    return np.concatenate(parts).astype(np.float32)


def _rows(n, seed):
    """Training rows: differences of orders 0..3 of smooth histories (own and
    neighbour mean), materials, target and weight."""
    g = torch.Generator(DEV).manual_seed(seed)

    def rand(*s):
        return torch.rand(*s, device=DEV, generator=g)

    w, ph, amp = 0.02 + 0.1 * rand(n, 1, 1), 6.2832 * rand(n, 2, 1), 0.2 + rand(n, 2, 1)
    a = amp * torch.cos(ph - w * torch.arange(5, device=DEV))  # a[..., 0] is the coming increment
    a = a / a[..., 1:].abs().amax((1, 2), keepdim=True)
    h = a[..., 1:]
    d = torch.stack([h[..., 0], h[..., 0] - h[..., 1], h[..., 0] - 2 * h[..., 1] + h[..., 2],
                     h[..., 0] - 3 * h[..., 1] + 3 * h[..., 2] - h[..., 3]], -1)
    soft = (rand(n, 1) < 0.4).float()
    target = a[:, 0, 0] - 3 * h[:, 0, 0] + 3 * h[:, 0, 1] - h[:, 0, 2]
    return torch.cat([d.reshape(n, 8), 0.3 * soft + (1 - soft), 0.9 * soft + (1 - soft), target[:, None],
                      (0.1 + rand(n, 1)) ** 2], 1).contiguous()


def _records(c, seed):
    """Green's records of the three directions (decaying random responses) and
    the record of an event whose input is a random combination of shifts."""
    g = torch.Generator(DEV).manual_seed(seed)
    n, pairs = c["stride"] * c["blocks"], 3 * c["rec"]
    t = torch.arange(n, dtype=torch.float64, device=DEV)[:, None]
    green = []
    for j in range(3):
        x = torch.randn(n, pairs, dtype=torch.float64, device=DEV, generator=g) * torch.exp(-t / (0.3 * n))
        x = (x + torch.roll(x, 1, 0) + torch.roll(x, 2, 0)) / 3
        x[:3] = 0
        x *= torch.where(torch.arange(pairs, device=DEV) % 3 == j, 1.0, 0.3)
        green.append(x.reshape(n, c["rec"], 3).contiguous())
    co = torch.randn(3, c["shifts"], dtype=torch.float64, device=DEV, generator=g)
    obs = _response(green, co, c["stride"])
    obs = obs + 0.05 * obs.std() * torch.randn(obs.shape, dtype=torch.float64, device=DEV, generator=g)
    return green, obs.contiguous()


def _response(green, co, stride):
    n = green[0].shape[0]
    U = torch.zeros_like(green[0])
    for j in range(3):
        for k in range(co.shape[1]):
            if k * stride < n:
                U[k * stride:] += co[j, k] * green[j][:n - k * stride]
    return U


# ----------------------------------------------------------------- work

# arithmetic of one element of the step operator (stiffness and mass) and of one network row
TET_FLOPS, ROW_FLOPS = 1150, 2 * (10 * 64 + 64 * 64 + 64)


def _pass(c, real):
    """Bytes and operations of one operator pass: ten node numbers and a
    material byte per tet, vertex coordinates, one vector read and one written."""
    nodes, tets, _ = _size(c)
    return 41 * tets + (6 * real + 24 / 8) * nodes, TET_FLOPS * tets


def _step_work(c, its, inner):
    """A step: its CG iterations (operator pass, three vectors updated and the
    preconditioner read), the right-hand side's and the true residual's FP64
    passes, and the FP64 state read and written."""
    nodes = _size(c)[0]
    b, f = _pass(c, inner)
    b64, f64 = _pass(c, 8)
    return its * (b + 8 * 3 * inner * nodes) + 2 * b64 + 12 * 24 * nodes, its * (f + 60 * nodes) + 2 * f64


# CG iterations of one step to 1e-10 in steady state, by guess
ITERATIONS = {"proj": 120, "poly": 130}


def work(case):
    c, kind = case, case["kind"]
    if kind == "step":
        b, f = _step_work(c, ITERATIONS[c["guess"]], 8 if c["precision"] == "fp64" else 4)
        return {"bytes": c["steps"] * b, "flops": c["steps"] * f}
    if kind == "batch":
        w = [_step_work(lane, ITERATIONS["proj"], 4) for lane in _lanes(c)]
        return {"bytes": sum(x[0] for x in w), "flops": sum(x[1] for x in w)}
    if kind in ("apply", "apply32", "rhs"):
        b, f = _pass(c, 4 if kind == "apply32" else 8)
        return {"bytes": b + (48 * _size(c)[0] if kind == "rhs" else 0), "flops": f}
    if kind == "forward":
        return {"bytes": 44 * c["rows"], "flops": ROW_FLOPS * c["rows"]}
    if kind == "train":
        return {"bytes": 48 * c["batch"] * c["steps"], "flops": 3 * ROW_FLOPS * c["batch"] * c["steps"]}
    n, pairs, cols = c["stride"] * c["blocks"], 3 * c["rec"], 4 * c["blocks"]
    return {"bytes": 5 * 8 * n * pairs, "flops": cols * cols * c["stride"] * pairs + 6 * c["shifts"] * n * pairs}


# ---------------------------------------------------------------- exact

def _p2_mass(nv):
    """Reference mass matrix of the quadratic simplex with nv vertices (unit
    measure): integrals of products of barycentric polynomials in closed form."""
    edges = EDGES if nv == 4 else ((0, 1), (1, 2), (2, 0))
    unit = [tuple(int(i == k) for i in range(nv)) for k in range(nv)]

    def add(p, q):
        return tuple(a + b for a, b in zip(p, q))

    shape = [{add(unit[i], unit[i]): 2.0, unit[i]: -1.0} for i in range(nv)] + [{add(unit[a], unit[b]): 4.0} for a, b in edges]

    def integral(p):
        return math.prod(math.factorial(a) for a in p) * math.factorial(nv - 1) / math.factorial(sum(p) + nv - 1)

    return np.array([[sum(x * y * integral(add(p, q)) for p, x in s.items() for q, y in r.items()) for r in shape] for s in shape])


class _Operator:
    """K, M and C_abs of a model applied element by element in FP64 (four-point
    quadrature of the linear strains, closed-form mass)."""

    def __init__(self, m, model):
        def dev(a, dtype=torch.float64):
            return torch.as_tensor(a, dtype=dtype, device=DEV)

        self.n = len(m.xyz)
        self.tet, self.tri = dev(m.tet10, torch.int64), dev(m.tri6, torch.int64)
        X, mat = dev(m.xyz), dev(model.mat)
        prop = mat[dev(model.tet_mat, torch.int64)]
        self.rho = prop[:, 2]
        self.mu = self.rho * prop[:, 1] ** 2
        self.lam = self.rho * prop[:, 0] ** 2 - 2 * self.mu
        x = X[self.tet[:, :4]]
        J = x[:, 1:] - x[:, :1]
        G = torch.linalg.inv(J).transpose(1, 2)
        self.g = torch.cat([-G.sum(1, keepdim=True), G], 1).contiguous()  # barycentric gradients
        self.vol = torch.linalg.det(J) / 6
        self.mass = dev(_p2_mass(4))
        a, b = (5 - math.sqrt(5)) / 20, (5 + 3 * math.sqrt(5)) / 20
        self.dN = []  # dN_i / dL_k at the four points
        for q in range(4):
            L = [b if k == q else a for k in range(4)]
            d = np.zeros((10, 4))
            for k in range(4):
                d[k, k] = 4 * L[k] - 1
            for e, (i, j) in enumerate(EDGES):
                d[4 + e, i], d[4 + e, j] = 4 * L[j], 4 * L[i]
            self.dN.append(dev(d))
        f = X[self.tri[:, :3]]
        nrm = torch.linalg.cross(f[:, 1] - f[:, 0], f[:, 2] - f[:, 0], dim=1)
        self.area = nrm.norm(dim=1) / 2
        nrm = nrm / nrm.norm(dim=1, keepdim=True)
        fp = prop[dev(m.face_tet, torch.int64)]
        zp, zs = fp[:, 2] * fp[:, 0], fp[:, 2] * fp[:, 1]
        self.Z = zs[:, None, None] * torch.eye(3, dtype=torch.float64, device=DEV) + (zp - zs)[:, None, None] * nrm[:, :, None] * nrm[:, None, :]
        self.fmass = dev(_p2_mass(3))
        self.base = dev(m.face_role, torch.int64) == 2

    def __call__(self, x, sM, sK, sC):
        x = x.view(-1, 3)
        y = torch.zeros_like(x)
        for s in range(0, len(self.tet), 500000):
            e = slice(s, s + 500000)
            U = x[self.tet[e]]
            f = torch.zeros_like(U)
            if sM:
                f += (sM * self.rho[e] * self.vol[e])[:, None, None] * torch.matmul(self.mass, U)
            if sK:
                g, lam, mu = self.g[e], self.lam[e], self.mu[e]
                eye = torch.eye(3, dtype=torch.float64, device=DEV)
                for d in self.dN:
                    H = torch.matmul(torch.matmul(d.T, U).transpose(1, 2), g)
                    S = (lam * H.diagonal(dim1=1, dim2=2).sum(1))[:, None, None] * eye + mu[:, None, None] * (H + H.transpose(1, 2))
                    f += (sK * self.vol[e] / 4)[:, None, None] * torch.matmul(d, torch.matmul(g, S))
            y.index_add_(0, self.tet[e].reshape(-1), f.reshape(-1, 3))
        if sC:
            w = torch.matmul(self.fmass, x[self.tri])
            y.index_add_(0, self.tri.reshape(-1), (sC * self.area[:, None, None] * torch.matmul(w, self.Z)).reshape(-1, 3))
        return y.view(-1)

    def force(self, v):
        """Base traction 2 Z v_in: a third of it on each edge node of a face."""
        y = torch.zeros(self.n, 3, dtype=torch.float64, device=DEV)
        f = 2 * (self.area[:, None] / 3) * torch.matmul(self.Z, v)
        f, t = f[self.base], self.tri[self.base]
        for k in (3, 4, 5):
            y.index_add_(0, t[:, k], f)
        return y.view(-1)

    def diagonal(self, sM, sK, sC):
        """Diagonal of the combination (a scalar preconditioner's)."""
        y = torch.zeros(self.n, 3, dtype=torch.float64, device=DEV)
        f = torch.zeros(len(self.tet), 10, 3, dtype=torch.float64, device=DEV)
        f += (sM * self.rho * self.vol)[:, None, None] * self.mass.diagonal()[:, None]
        for d in self.dN:
            G = torch.matmul(d, self.g)
            f += (sK * self.vol / 4)[:, None, None] * (self.mu[:, None, None] * (G * G).sum(2, keepdim=True) + (self.lam + self.mu)[:, None, None] * G * G)
        y.index_add_(0, self.tet.reshape(-1), f.reshape(-1, 3))
        w = (sC * self.area)[:, None, None] * self.fmass.diagonal()[:, None] * self.Z.diagonal(dim1=1, dim2=2)[:, None, :]
        y.index_add_(0, self.tri.reshape(-1), w.reshape(-1, 3))
        return y.view(-1)


def _scales(model):
    return 4 / model.dt ** 2 + 2 * model.ray_alpha / model.dt, 1 + 2 * model.ray_beta / model.dt, 2 / model.dt


def _exact_rhs(op, model, step, u, v, a):
    return (op.force(torch.as_tensor(model.v_in[step + 1], device=DEV)) + op(a + (4 / model.dt + model.ray_alpha) * v, 1, 0, 0)
            + op(v, 0, 0, 1) - op(u - model.ray_beta * v, 0, 1, 0))


def _exact_march(m, model, v0, n):
    """Receiver velocity of step n of the march from u = a = 0, v = v0, every
    step solved to 1e-13 by Jacobi-preconditioned CG."""
    op, sc = _Operator(m, model), _scales(model)
    inv = 1 / op.diagonal(*sc)
    v = torch.from_numpy(v0).to(DEV)
    u, a, x = torch.zeros_like(v), torch.zeros_like(v), torch.zeros_like(v)
    for k in range(n):
        b = _exact_rhs(op, model, k, u, v, a)
        r = b - op(x, *sc)
        z = inv * r
        p, rz, bb = z.clone(), r @ z, float(b.norm())
        for it in range(3000):
            q = op(p, *sc)
            al = rz / (p @ q)
            x = x + al * p
            r = r - al * q
            if it % 8 == 7 and float(r.norm()) <= 1e-13 * bb:
                break
            z = inv * r
            new = r @ z
            p = z + new / rz * p
            rz = new
        u, v, a = u + x, 2 / model.dt * x - v, 4 / model.dt ** 2 * x - 4 / model.dt * v - a
        x = x.clone()
    return v.view(-1, 3)[torch.as_tensor(model.rec_node, dtype=torch.int64, device=DEV)][None]


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "batch":
        return None
    if kind == "step":
        if _size(c)[1] > 250000 or c["steps"] != 1:
            return None
        m, model, rng = _start(c, seed, _capacity(c))
        return _exact_march(m, model, _field(m, rng, 0.1), WARM_STEPS + 1)
    if kind in ("apply", "apply32"):
        m, model, rng = _start(c, seed, 8)
        x = torch.from_numpy(_field(m, rng, 1e-3)).to(DEV)
        x += 1e-4 * torch.randn(x.shape, dtype=x.dtype, device=DEV, generator=torch.Generator(DEV).manual_seed(seed))
        return _Operator(m, model)(x.float().double() if kind == "apply32" else x, *_scales(model))
    if kind == "rhs":
        m, model, rng = _start(c, seed, 8)
        u, v, a = (torch.from_numpy(_field(m, rng, s)).to(DEV) for s in (1e-3, 0.1, 5.0))
        return _exact_rhs(_Operator(m, model), model, 0, u, v, a)
    if kind == "forward":
        w = torch.from_numpy(_weights(seed)).to(DEV).double()
        W1, b1, W2, b2, w3, b3 = torch.split(w, (640, 64, 4096, 64, 64, 1))
        x = _rows(c["rows"], seed)[:, :10].double()
        h = torch.relu(x @ W1.view(64, 10).T + b1)
        return torch.relu(h @ W2.view(64, 64).T + b2) @ w3 + b3
    if kind == "train":
        return None
    green, obs = _records(c, seed)
    n, L, stride = obs.shape[0], c["shifts"], c["stride"]
    wt = 1 / obs.reshape(n, -1).square().sum(0)
    A = torch.zeros(3 * L, n * obs[0].numel(), dtype=torch.float64, device=DEV)
    for j in range(3):
        for k in range(L):
            A[j * L + k].view(n, -1)[k * stride:] = green[j].reshape(n, -1)[:n - k * stride]
    Aw = (A.view(3 * L, n, -1) * wt).view(3 * L, -1)
    w, V = torch.linalg.eigh(A @ Aw.T)
    keep = w > 1e-6 * w[-1]
    co = (V[:, keep] / w[keep]) @ (V[:, keep].T @ (Aw @ obs.reshape(-1)))
    U = (co @ A).view_as(obs)
    err = ((U - obs).reshape(n, -1).norm(dim=0) / obs.reshape(n, -1).norm(dim=0)).mean()
    return {"c": co.view(3, L), "err": float(err), "used": int(obs[0].numel()), "rank": int(keep.sum()), "U": U}
