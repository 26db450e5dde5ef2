"""The work a user of this framework has it do, as cases that can be timed.

Three public paths are covered: the barotropic loop alone on device arrays
(``barotropic_substep_noalloc``), the split-explicit step followed by reading
the state (``DeviceState.step`` and ``read``: a run advances a stretch of
steps, then writes its output), and an ensemble advanced as one batch.

``listed()`` names the cases, ``draw()`` gives more of the same ranges,
``prepare()`` makes what a program holds before the call (the mesh and its
bathymetry are fixed by the case, the ocean on it by the seed), ``run()`` is
one pass, ``work()`` is what the pass cannot do without and ``exact()`` the
same results in plain 64-bit torch.

The oceans are spun up rather than at rest: eddies of 0.1-0.3 m/s that decay
with depth, the surface height in geostrophic balance with them, a stratified
density with weak fronts.  Viscosity and steps scale with the mesh, so that a
state can be stepped again and again.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2105_13484_amd.ssprkse import Batch, DeviceMesh, DeviceState
from synthetic.cases import GRAVITY, RHO0, Params
from synthetic.mesh import icosahedral, planar_hex

FP64, MIXED, MIXED_BT64 = 0, 1, 2


def _hex(name, nx, ny, layers, **kw):
    return dict({"kind": "steps", "name": name, "mesh": "hex", "nx": nx, "ny": ny, "level": 0, "layers": layers,
                 "scheme": 3, "substeps": 20, "precision": FP64, "vcoord": 0, "reconcile": 1, "vmix": 0, "hdiff": 0,
                 "tracer": 0, "graph": False, "steps": 10}, **kw)


def _sphere(name, level, layers, **kw):
    return _hex(name, 0, 0, layers, mesh="sphere", level=level, substeps=kw.pop("substeps", 30), **kw)


def listed():
    return [
        # the barotropic solver on its own, on a regional mesh: a call of a few hundred microseconds
        _hex("loop 64x64", 64, 64, 1, kind="loop"),
        # the same on the headline mesh
        _hex("loop 512x512", 512, 512, 1, kind="loop"),
        # the smallest channel, second-order scheme, with few layers: launches and latency
        _hex("channel 16x16x4", 16, 16, 4, scheme=2, substeps=10, steps=20),
        # one member of an ensemble, run alone in mixed precision as a replayed graph
        _hex("member 64x64x20 mixed", 64, 64, 20, substeps=15, precision=MIXED, graph=True, steps=30),
        # odd sizes: isopycnal layers, second-order scheme, the printed reconciliation
        _hex("ragged 97x46x33 iso", 97, 46, 33, scheme=2, substeps=7, vcoord=1, reconcile=2, steps=20),
        # the smallest served request: coarse globe with land, temperature carried along, mixed precision
        _sphere("globe5 x37 tracer mixed", 5, 37, precision=MIXED, tracer=1, steps=30),
        # an ordinary served request in full precision
        _sphere("globe6 x60", 6, 60, steps=50),
        # a deep request with every optional term, two register chunks of layers, mixed with a 64-bit loop
        _sphere("globe6 x100 all terms", 6, 100, precision=MIXED_BT64, tracer=1, vmix=1, hdiff=1, steps=20),
        # a regional run with implicit vertical mixing
        _hex("basin 256x256x60 vmix", 256, 256, 60, vmix=1, steps=40),
        # the headline workload
        _hex("basin 512x512x60", 512, 512, 60, steps=40),
        # the global eddy-permitting mesh in mixed precision
        _sphere("globe7 x60 mixed", 7, 60, precision=MIXED, steps=30),
        # an uneven ensemble in one batch, replayed as a graph
        _hex("ensemble of 8 mixed", 0, 0, 0, kind="batch", members=8, precision=MIXED, graph=True, steps=20),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cells(case):
    return case["nx"] * case["ny"] if case["mesh"] == "hex" else 10 * 4 ** case["level"] + 2


def draw(rng):
    kind = rng.choice(["loop", "steps", "steps", "steps", "steps", "batch"])
    precision = rng.choice([FP64, FP64, MIXED, MIXED, MIXED_BT64])
    if kind == "batch":
        c = _hex("", 0, 0, 0, kind="batch", members=rng.randint(3, 8), precision=precision, graph=rng.random() < 0.5,
                 steps=rng.randint(10, 20))
    else:
        layers = 1 if kind == "loop" else rng.choice([_log(rng, 1, 128), _log(rng, 16, 100), 60])
        scheme, substeps = rng.choice([2, 3, 3]), rng.randint(5, 30)
        # without the exact reconciliation only SSPRK2-SE with few substeps stays bounded on these oceans
        common = dict(kind=kind, scheme=scheme, substeps=substeps, precision=precision,
                      reconcile=rng.choice([0, 1, 2]) if scheme == 2 and substeps <= 10 else 1, steps=_log(rng, 8, 30), graph=kind == "steps" and rng.random() < 0.3)
        if kind == "steps":
            common.update(vcoord=int(rng.random() < 0.2), vmix=int(rng.random() < 0.3), hdiff=int(rng.random() < 0.2),
                          tracer=int(rng.random() < 0.25))
        if rng.random() < 0.4:
            c = _sphere("", rng.choice([3, 4, 5, 6, 6, 7]), layers, **common)
        else:
            c = _hex("", _log(rng, 12, 500), 2 * _log(rng, 6, 250), layers, **common)
        # no more layers, and steps of them, than the largest listed case has in all
        c["layers"] = min(c["layers"], max(1, 12_000_000 // _cells(c)))
        c["steps"] = min(c["steps"], max(5, 360_000_000 // (_cells(c) * c["layers"])))
    del c["name"]
    return c


# --- the mesh with its bathymetry: fixed by the case -------------------------


@functools.lru_cache(maxsize=6)
def _ground(kind, nx, ny, level):
    """(mesh, H, ocean mask): periodic hexes of 10 km (5 km from 512 on) over a
    1000 m bottom with hills, or the globe with about 30% land, 500-5000 m deep."""
    rng = np.random.default_rng(7)
    if kind == "hex":
        mesh = planar_hex(nx, ny, 5.0e3 if max(nx, ny) >= 512 else 1.0e4)
        x, y = mesh.xCell[:, 0] / mesh.Lx, mesh.xCell[:, 1] / mesh.Ly
        b = sum(rng.uniform(0.5, 1.0) * np.cos(2 * np.pi * (kx * x + ky * y) + rng.uniform(0, 2 * np.pi))
                for kx, ky in ((1, 0), (0, 1), (2, 1), (1, -3)))
        return mesh, 1000.0 + 100.0 * b / np.abs(b).max(), np.ones(mesh.nCells, np.uint8)
    mesh = icosahedral(level)
    xc = mesh.xCell / mesh.radius
    s = np.zeros(mesh.nCells)
    for _ in range(20):
        p = rng.normal(size=3)
        p /= np.linalg.norm(p)
        s += rng.uniform(0.5, 1.5) * np.exp(-(np.arccos(np.clip(xc @ p, -1, 1)) / rng.uniform(0.16, 0.47)) ** 2)
    q = np.quantile(s, 0.7)
    sea = s < q
    return mesh, np.where(sea, np.clip(500 + 4500 * (q - s) / (q - s.min()), 500, 5000), 0.0), sea.astype(np.uint8)


@functools.lru_cache(maxsize=6)
def _device_mesh(kind, nx, ny, level):
    return DeviceMesh(*_ground(kind, nx, ny, level))


def _key(case):
    return case["mesh"], case["nx"], case["ny"], case["level"]


def _params(case):
    mesh, H, _ = _ground(*_key(case))
    width = float(np.median(mesh.dcEdge))
    # gravity waves: 0.3 of a cell per substep for SSPRK3, less for SSPRK2, which damps nothing on the imaginary axis
    sub = (0.3 if case["scheme"] == 3 else 0.07) * width / math.sqrt(GRAVITY * H.max())
    dt = min(case["substeps"] * sub, 1800.0)
    return Params(n_layers=case["layers"], scheme=case["scheme"], substeps=case["substeps"], precision=case["precision"],
                  vcoord=case["vcoord"], reconcile=case["reconcile"], vmix=case["vmix"], hdiff=case["hdiff"],
                  tracer=case["tracer"], dt=dt, nu_h=0.01 * width ** 3 if case["hdiff"] else 0.02 * width,
                  nu_v=1.0e-4, c_drag=1.0e-3, kappa_h=0.01 * width, kappa_v=1.0e-5)


# --- the ocean on it: fixed by the seed --------------------------------------


def _waves(mesh, rng, x):
    """A smooth random field of unit size at the points x: (kind-dependent) plane waves."""
    out = np.zeros(len(x))
    for _ in range(8):
        if mesh.kind == "planar":
            k = np.array([0, 0])
            while not k.any():
                k = rng.integers(-3, 4, size=2)
            phase = 2 * np.pi * (k[0] * x[:, 0] / mesh.Lx + k[1] * x[:, 1] / mesh.Ly)
        else:
            k = rng.normal(size=3)
            phase = (x / mesh.radius) @ (k * rng.uniform(4, 10) / np.linalg.norm(k))
        out += rng.uniform(0.5, 1.0) * np.cos(phase + rng.uniform(0, 2 * np.pi))
    return out / 2.0


def _eddies(mesh, rng):
    """(velocity normal to the edges, surface height): flow along a stream
    function with the height that balances it, and a basin-wide swell on top (on
    the globe the balanced height is itself some metres)."""
    state = rng.bit_generator.state
    at_v = _waves(mesh, rng, mesh.xVertex)
    rng.bit_generator.state = state
    at_c = _waves(mesh, rng, mesh.xCell)
    v = mesh.verticesOnEdge
    u = -(at_v[v[:, 1]] - at_v[v[:, 0]]) / mesh.dvEdge
    scale = 0.1 / np.sqrt(np.mean(u ** 2))
    zeta = scale * at_c * mesh.fCell / GRAVITY
    return scale * u, zeta + 0.3 * _waves(mesh, rng, mesh.xCell) if mesh.kind == "planar" else zeta


def _ocean(case, seed):
    """h, u, rho, h_ref and temperature on the case's mesh (float64 arrays)."""
    mesh, H, mask = _ground(*_key(case))
    L = case["layers"]
    rng = np.random.default_rng([seed, L])
    u0, zeta = _eddies(mesh, rng)
    u1, _ = _eddies(mesh, rng)
    depth = (np.arange(L) + 0.5) / L
    u = np.stack([u0, u1], 1) @ np.stack([0.3 + np.exp(-3 * depth), 0.4 * np.cos(np.pi * depth)])
    h_ref = np.repeat((H / L)[:, None], L, axis=1)
    safe = np.where(mask > 0, H, 1.0)
    h = h_ref * (1.0 + zeta / safe)[:, None]
    T = np.outer(_waves(mesh, rng, mesh.xCell), 0.2 * np.exp(-4 * depth)) + (20.0 - 14.0 * np.outer(H, depth) / H.max())
    T = np.where(mask[:, None] > 0, T, 0.0)
    rho = np.where(mask[:, None] > 0, RHO0 * (1.0 - 2.0e-4 * (T - 10.0)), 0.0)
    return h, u, rho, h_ref, T


def _members(case):
    """The members of a batch: uneven meshes, depths and substeps."""
    rng = np.random.default_rng(11)
    for _ in range(case["members"]):
        n, L, M = rng.choice([64, 96, 128, 192]), rng.choice([20, 40, 60]), rng.integers(10, 31)
        yield dict(case, kind="steps", nx=int(n), ny=int(n), layers=int(L), substeps=int(M))


def _loop_inputs(case, seed):
    """Barotropic velocity, surface height and frozen forcing for the loop alone."""
    mesh, _, mask = _ground(*_key(case))
    rng = np.random.default_rng([seed, 1])
    u, zeta = _eddies(mesh, rng)
    c = mesh.cellsOnEdge
    wet = (mask[c[:, 0]] & mask[c[:, 1]]).astype(float)
    return u * wet, zeta * mask, rng.normal(0.0, 1.0e-6, mesh.nEdges) * wet


def _state(case, seed, stream):
    h, u, rho, h_ref, T = _ocean(case, seed)
    st = DeviceState(_device_mesh(*_key(case)), _params(case), stream=stream)
    st.init(h, u, rho, h_ref)
    if case["tracer"]:
        st.set_tracer(T)
    return st


@functools.lru_cache(maxsize=1)
def _stream():
    """The program's own stream (graphs need one that is not the default)."""
    return torch.cuda.Stream()


def prepare(case, seed):
    if case["kind"] == "loop":
        st = DeviceState(_device_mesh(*_key(case)), _params(case))
        args = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in _loop_inputs(case, seed)]
        return {"case": case, "state": st, "in": args, "out": [torch.empty_like(args[i]) for i in (0, 1, 2)],
                "dt": _params(case).dt}
    stream = _stream() if case["graph"] else None
    if case["kind"] == "batch":
        members = [_state(m, seed + 100 * i, stream) for i, m in enumerate(_members(case))]
        batch = Batch(stream=stream)
        for st in members:
            batch.add(st)
        batch.compile()
        batch.use_graph(case["graph"])
        return {"case": case, "batch": batch, "members": members}
    st = _state(case, seed, stream)
    st.use_graph(case["graph"])
    return {"case": case, "state": st}


def _output(case, st):
    """What is written down after a stretch of steps.  Mixed-precision runs
    compute their velocities in single precision, and their output is kept in
    single precision, as ocean model history files are."""
    out = st.read()
    if case["tracer"]:
        out["T"] = st.read_tracer()
    return out if case["precision"] == FP64 else {k: torch.from_numpy(v).float() for k, v in out.items()}


def run(state):
    case = state["case"]
    if case["kind"] == "loop":
        state["state"].barotropic_substep_noalloc(case["scheme"], case["substeps"], state["dt"], *state["in"], *state["out"])
        out = dict(zip(("ubar", "zeta", "F"), state["out"]))
        return {k: v.float() for k, v in out.items()} if case["precision"] == MIXED else out
    if case["kind"] == "batch":
        state["batch"].step(case["steps"])
        return {f"member {i}": _output(case, st) for i, st in enumerate(state["members"])}
    state["state"].step(case["steps"])
    return _output(case, state["state"])


def work(case):
    """Bytes and operations of one pass.  Per stage of a step the layered state
    is read and written once (u, h, density, temperature); per stage the
    barotropic state, forcing and transport are; the mesh's operator tables are
    read once per stage.  Operations are those of the formulas."""
    if case["kind"] == "batch":
        parts = [work(m) for m in _members(case)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    C = _cells(case)
    E, L, M, stages = 3 * C, case["layers"], case["substeps"], case["scheme"]
    r = 8 if case["precision"] == FP64 else 4
    b = 4 if case["precision"] == MIXED else 8
    loop_bytes = E * (b * 5 + 10 * (b + 2)) + C * (b * 3 + 6 * (b + 2))
    loop_flops = stages * M * (E * 32 + C * 26)
    if case["kind"] == "loop":
        return {"bytes": loop_bytes, "flops": loop_flops}
    layered = E * L * 2 * r + C * L * 8 * 3 + (C * L * 16 if case["tracer"] else 0)
    operations = E * L * (110 + (60 if case["vmix"] else 0) + (30 if case["hdiff"] else 0)) + C * L * (60 + (80 if case["tracer"] else 0))
    step = {"bytes": stages * (layered + loop_bytes), "flops": stages * (operations + loop_flops)}
    state = 8 * ((E + C + (C if case["tracer"] else 0)) * L + E + C)
    return {"bytes": case["steps"] * step["bytes"] + state, "flops": case["steps"] * step["flops"]}


# --- the same in plain 64-bit torch ------------------------------------------


class _Exact:
    """The split-explicit schemes on one mesh; fields are (layers, entities)."""

    def __init__(self, case):
        self.p = _params(case)
        mesh, H, mask = _ground(*_key(case))
        self.dev = "cuda" if torch.cuda.is_available() else "cpu"
        T = self.tensor
        coe, voe = mesh.cellsOnEdge, mesh.verticesOnEdge
        self.c1, self.c2, self.v1, self.v2 = (T(a) for a in (coe[:, 0], coe[:, 1], voe[:, 0], voe[:, 1]))
        self.H, self.dc, self.dv, self.f = T(H), T(mesh.dcEdge), T(mesh.dvEdge), T(mesh.fEdge)
        self.sea = T(mask.astype(bool))
        self.wet = self.sea[self.c1] & self.sea[self.c2]
        slot = np.arange(6)[None, :] < mesh.nEdgesOnCell[:, None]
        e = np.where(slot, mesh.edgesOnCell, 0)
        sign = np.where(coe[e, 0] == np.arange(mesh.nCells)[:, None], 1.0, -1.0)
        self.eoc = T(e)
        self.cdiv = T(np.where(slot, sign * mesh.dvEdge[e], 0.0) / mesh.areaCell[:, None])
        self.cke = T(np.where(slot, 0.25 * mesh.dvEdge[e] * mesh.dcEdge[e], 0.0) / mesh.areaCell[:, None])
        e = mesh.edgesOnVertex
        sign = np.where(voe[e, 1] == np.arange(mesh.nVertices)[:, None], 1.0, -1.0)
        self.eov, self.ccurl = T(e), T(sign * mesh.dcEdge[e] / mesh.areaTriangle[:, None])
        slot = np.arange(10)[None, :] < mesh.nEdgesOnEdge[:, None]
        self.eoe, self.W = T(np.where(slot, mesh.edgesOnEdge, 0)), T(np.where(slot, mesh.weightsOnEdge, 0.0))

    def tensor(self, a):
        t = torch.from_numpy(np.ascontiguousarray(a)).to(self.dev)
        return t.long() if t.dtype == torch.int32 else t

    def mean(self, x):
        return 0.5 * (x[..., self.c1] + x[..., self.c2])

    def grad(self, x):
        return (x[..., self.c2] - x[..., self.c1]) / self.dc

    def div(self, F):
        F = F * self.wet
        return sum(self.cdiv[:, j] * F[..., self.eoc[:, j]] for j in range(6))

    def curl(self, u):
        return sum(self.ccurl[:, j] * u[..., self.eov[:, j]] for j in range(3))

    def perp(self, q, u):
        return sum(self.W[:, j] * (0.5 * (q + q[..., self.eoe[:, j]])) * u[..., self.eoe[:, j]] for j in range(10))

    def lap(self, u):
        z = self.curl(u)
        return (self.grad(sum(self.cdiv[:, j] * u[..., self.eoc[:, j]] for j in range(6)))
                - (z[..., self.v2] - z[..., self.v1]) / self.dv)

    def ssh(self, h):
        return torch.where(self.sea, h.sum(0) - self.H, 0.0)

    def share(self, total, he):
        return torch.where(self.wet, total / torch.where(self.wet, he.sum(0), 1.0), 0.0)

    def column(self, h, v):
        """Flux divergence per layer, the thickness tendency and w at the interfaces."""
        d = self.div(self.mean(h) * v)
        w = torch.zeros(d.shape[0] + 1, d.shape[1], dtype=d.dtype, device=self.dev)
        if self.p.vcoord == 1:
            return -d * self.sea, w
        th = -self.frac * d.sum(0)
        w[:-1] = torch.flip(torch.cumsum(torch.flip(-d - th, [0]), 0), [0]) * self.sea
        return th * self.sea, w

    def tendency(self, u, ut, zeta, h, rho):
        """Everything of the baroclinic right-hand side but the vertical
        viscosity, and the parts that needs: edge thickness and drag speed."""
        p = self.p
        he = torch.where(self.wet, self.mean(h), 1.0)
        K = sum(self.cke[:, j] * u[:, self.eoc[:, j]] ** 2 for j in range(6))
        out = self.perp(self.f, ut) + self.perp(self.mean_v(self.curl(u)), u) - self.grad(K) + p.gravity * self.grad(zeta)
        we = self.mean(self.column(h, u)[1])[1:-1]
        adv = torch.zeros_like(self.pad(u))
        adv[1:-1] = we * (u[:-1] - u[1:]) / (0.5 * (he[:-1] + he[1:]))
        out -= 0.5 * (adv[:-1] + adv[1:])
        drh = rho[:, self.c2] * h[:, self.c2] - rho[:, self.c1] * h[:, self.c1]
        dh = h[:, self.c2] - h[:, self.c1]
        dp = p.gravity * (torch.cumsum(drh, 0) - 0.5 * drh)
        dz = torch.flip(torch.cumsum(torch.flip(dh, [0]), 0), [0]) - 0.5 * dh - (self.H[self.c2] - self.H[self.c1])
        out -= (dp + p.gravity * self.mean(rho) * dz) / (p.rho0 * self.dc)
        lap = self.lap(u)
        out += -p.nu_h * self.lap(lap * self.wet) if p.hdiff else p.nu_h * lap
        return out, he, torch.sqrt(K[-1, self.c1] + K[-1, self.c2])

    def mean_v(self, z):
        return 0.5 * (z[:, self.v1] + z[:, self.v2])

    def pad(self, u):
        return torch.zeros(u.shape[0] + 1, u.shape[1], dtype=u.dtype, device=self.dev)

    def baroclinic(self, u, ubar, zeta, h, rho):
        p, ut = self.p, u - ubar
        rhs, he, speed = self.tendency(u, ut, zeta, h, rho)
        if not p.vmix:
            tau = self.pad(u)
            tau[1:-1] = p.nu_v * (u[:-1] - u[1:]) / (0.5 * (he[:-1] + he[1:]))
            tau[-1] = p.c_drag * speed * u[-1]
            rhs += (tau[:-1] - tau[1:]) / he
        x = (ut + p.dt * rhs) * self.wet
        G = self.share((he * x).sum(0), he) / p.dt
        x = x - p.dt * G
        if p.vmix:
            A = self.pad(u)
            A[1:-1] = p.nu_v / (0.5 * (he[:-1] + he[1:]))
            A[-1] = p.c_drag * speed
            lo, up = -p.dt * A[:-1] / he, -p.dt * A[1:] / he
            x = self.tridiagonal(lo, 1.0 - lo - up, up, x + ubar) - ubar
        return x * self.wet, G

    @staticmethod
    def tridiagonal(lo, di, up, d):
        c, y = torch.empty_like(d), torch.empty_like(d)
        c[0], y[0] = up[0] / di[0], d[0] / di[0]
        for k in range(1, len(d)):
            pivot = di[k] - lo[k] * c[k - 1]
            c[k], y[k] = up[k] / pivot, (d[k] - lo[k] * y[k - 1]) / pivot
        for k in range(len(d) - 2, -1, -1):
            y[k] -= c[k] * y[k + 1]
        return y

    def loop(self, u, z, G, dt, scheme, M):
        """Substeps of the barotropic system: (ubar, zeta, mean transport)."""
        tau, F = dt / M, torch.zeros_like(u)
        Wf = self.W * (0.5 * (self.f[:, None] + self.f[self.eoe]))

        def euler(u, z):
            flux = u * self.mean(z + self.H) * self.wet
            du = (Wf * u[self.eoe]).sum(1) - self.p.gravity * self.grad(z) + G
            return torch.where(self.wet, u + tau * du, 0.0), torch.where(self.sea, z - tau * self.div(flux), 0.0), flux

        for _ in range(M):
            u1, z1, f1 = euler(u, z)
            u2, z2, f2 = euler(u1, z1)
            if scheme == 2:
                u, z, F = 0.5 * (u + u2), 0.5 * (z + z2), F + (f1 + f2) / (2 * M)
                continue
            u3, z3, f3 = euler(0.75 * u + 0.25 * u2, 0.75 * z + 0.25 * z2)
            u, z, F = u / 3 + 2 * u3 / 3, z / 3 + 2 * z3 / 3, F + (f1 + f2 + 4 * f3) / (6 * M)
        return u, z, F

    def thickness(self, h, v, T):
        """One forward stage of thickness and, with T, of the heat content."""
        p = self.p
        th, w = self.column(h, v)
        if T is None:
            return h + p.dt * th, None
        he = self.mean(h)
        flux = torch.zeros_like(w)
        flux[1:-1] = 0.5 * (T[:-1] + T[1:]) * w[1:-1]
        h1 = torch.where(self.sea, h, 1.0)
        flux[1:-1] -= p.kappa_v * (T[:-1] - T[1:]) / (0.5 * (h1[:-1] + h1[1:]))
        tend = self.div(he * (p.kappa_h * self.grad(T) - self.mean(T) * v)) - flux[:-1] + flux[1:]
        return h + p.dt * th, h * T + p.dt * tend * self.sea

    def density(self, T, rho):
        return rho if T is None else self.p.rho0 * (1.0 - self.p.eos_alpha * (T - self.p.eos_tref))

    def over(self, hT, h):
        return None if hT is None else torch.where(self.sea, hT / torch.where(self.sea, h, 1.0), 0.0)

    def step(self, u, h, T, rho):
        p, third = self.p, self.p.scheme == 3
        zeta, he = self.ssh(h), self.mean(h)
        ubar = self.share((he * u).sum(0), he)
        adjust = lambda wanted, he: self.share(wanted, he) if p.reconcile else torch.zeros_like(ubar)  # noqa: E731
        # first stage, then its barotropic loop and its thickness
        x1, G0 = self.baroclinic(u, ubar, zeta, h, self.density(T, rho))
        b1, _, F1 = self.loop(ubar, zeta, G0, p.dt, p.scheme, p.substeps)
        A1 = (he * u).sum(0) * self.wet
        ua = u + adjust(F1 - A1, he)
        h1, hT = self.thickness(h, ua * self.wet, T)
        T1, u1, z1, he1 = self.over(hT, h1), (x1 + b1) * self.wet, self.ssh(h1), self.mean(h1)
        x2, G1 = self.baroclinic(u1, b1, z1, h1, self.density(T1, rho))
        ut = (u - ubar) * self.wet
        if not third:
            b, _, F = self.loop(ubar, zeta, 0.5 * (G0 + G1), p.dt, 2, p.substeps)
            un = (0.5 * (ut + x2) + b) * self.wet
            P = (he1 * un).sum(0)
            fix = adjust(2 * F - ((F1 if p.reconcile == 1 else A1) + P), he1)
            h2, hT2 = self.thickness(h1, (un + fix) * self.wet, T1)
            hn = 0.5 * (h + h2)
            return un, hn, None if T is None else self.over(0.5 * (h * T + hT2), hn)
        b2, _, F2 = self.loop(b1, z1, G1, p.dt, 3, p.substeps)
        A2 = (he1 * u1).sum(0) * self.wet
        h2, hT2 = self.thickness(h1, (u1 + adjust(F2 - A2, he1)) * self.wet, T1)
        hh, bh, xh = 0.75 * h + 0.25 * h2, 0.75 * ubar + 0.25 * b2, 0.75 * ut + 0.25 * x2
        Th = None if T is None else self.over(0.75 * (h * T) + 0.25 * hT2, hh)
        uh, heh = (xh + bh) * self.wet, self.mean(hh)
        x3, Gh = self.baroclinic(uh, bh, self.ssh(hh), hh, self.density(Th, rho))
        b, _, F = self.loop(ubar, zeta, (G0 + G1 + 4 * Gh) / 6, p.dt, 3, p.substeps)
        un = (ut / 3 + 2 * x3 / 3 + b) * self.wet
        P = (heh * (u + un)).sum(0)
        got = (F1 + F2 if p.reconcile == 1 else A1 + A2) + 2 * P
        h3, hT3 = self.thickness(hh, (0.5 * (u + un) + adjust(1.5 * (F - got / 6), heh)) * self.wet, Th)
        hn = h / 3 + 2 * h3 / 3
        return un, hn, None if T is None else self.over(h * T / 3 + 2 * hT3 / 3, hn)

    def run(self, steps, h, u, rho, h_ref, T):
        h, u, rho, h_ref, T = (self.tensor(a).t().contiguous() for a in (h, u, rho, h_ref, T))
        self.frac = torch.where(self.sea, h_ref / torch.where(self.sea, h_ref.sum(0), 1.0), 0.0)
        u = u * self.wet
        T = T if self.p.tracer else None
        for _ in range(steps):
            u, h, T = self.step(u, h, T, rho)
        he = self.mean(h)
        out = {"h": h.t(), "u": u.t(), "zeta": self.ssh(h), "ubar": self.share((he * u).sum(0), he)}
        if T is not None:
            out["T"] = T.t()
        return {k: v.contiguous() for k, v in out.items()}


def exact(case, seed):
    if case["kind"] == "batch":
        return {f"member {i}": exact(m, seed + 100 * i) for i, m in enumerate(_members(case))}
    x = _Exact(case)
    if case["kind"] == "loop":
        u, z, G = (x.tensor(a) for a in _loop_inputs(case, seed))
        return dict(zip(("ubar", "zeta", "F"), x.loop(u, z, G, x.p.dt, case["scheme"], case["substeps"])))
    return x.run(case["steps"], *_ocean(case, seed))
