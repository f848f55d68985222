"""What the step library is timed on: seeded solves through the package's public entry points.

A case is one lattice (``capi.Lattice``), a batch of lattices (``capi.Batch``) or a set of requests to the solve
server (``serve.Server``).  One pass advances it as a user's program does between two looks at its state, and returns
the state it reached: the populations in the program's own device buffers, fields on the host where the program takes
snapshots, or the fields the server hands out.

The lattices are those of ``workloads.py``, the tests and the benchmark: static and density-ratio bubbles, a droplet
on a wall, gravity-driven slugs, open channels, the nine-lattice sweep and the serving mix.  ``draw`` spreads sizes,
step counts, storage formats and options over the same ranges.
"""
import ctypes
import math
import random

import numpy as np
import torch

from paper_1903_01168_amd import capi, serve
from paper_1903_01168_amd import workloads as W

DEVICE = "cuda" if torch.cuda.is_available() else "cpu"

# ------------------------------------------------------------------- cases --


def _case(name, kind, nx, ny, steps, storage="f32", collision="bgk", **kw):
    c = dict(kind=kind, nx=nx, ny=ny, steps=steps, storage=storage, collision=collision, **kw)
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest solve: the 64 x 64 static bubble, a couple of hundred steps between two looks at it.
        _case("bubble 64x64", "bubble", 64, 64, 200, gamma=1),
        # The contact-angle droplet (no-slip walls, MRT with the Navier-Stokes correction), a ragged width.
        _case("wall droplet 100x100", "droplet", 100, 100, 150, collision="mrt", nsc=True, angle=60),
        # The inlet/outlet verification channel: MRT with the correction, 500 x 50.
        _case("open channel 500x50", "channel", 500, 50, 100, collision="mrt", nsc=True, walls="walls"),
        # A monitored run: short bursts of steps, diagnostics and a single-precision snapshot after each.
        _case("snapshots 300x200", "snapshots", 300, 200, 50, collision="mrt", gamma=5),
        # One lattice of the bubble sweep on its own.
        _case("bubble 512x512", "bubble", 512, 512, 100, gamma=10),
        # The second-neighbour isotropic gradient on the sweep's lattice.
        _case("isotropic 512x512", "bubble", 512, 512, 64, collision="mrt", gamma=10, gradient="isotropic"),
        # The sweep: nine density / viscosity ratios advanced together.
        _case("sweep 9 x 512x512", "sweep", 512, 512, 64),
        # The serving mix: a burst of small and mid-sized solves through the server, 16-bit storage.
        _case("serving burst", "serve", 512, 512, 1500, storage="f16s", requests=12),
        # The gravity-driven slug channel in 16-bit storage.
        _case("slugs 4096x256 f16s", "slug", 4096, 256, 64, storage="f16s", gamma=10),
        # The benchmark's open channel, beyond the cache, in both storages that it is quoted in.
        _case("channel 8192x512", "channel", 8192, 512, 40),
        _case("channel 8192x512 f16s", "channel", 8192, 512, 40, storage="f16s"),
        # A large bubble, well beyond the cache.
        _case("bubble 4096x2048", "bubble", 4096, 2048, 40, collision="mrt", gamma=10),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["bubble", "bubble", "droplet", "channel", "channel", "slug", "slug", "snapshots", "sweep", "serve"])
    storage = rng.choice(["f32", "f32", "f32", "f16s", "bf16s"])
    collision = rng.choice(["bgk", "mrt"])
    kw = {}
    if kind == "sweep":
        n = _log(rng, 96, 700)
        return _case(None, kind, n, n, 2 * rng.randint(8, 40), storage, collision)
    if kind == "serve":
        n = 64 * rng.randint(2, 8)
        return _case(None, kind, n, n, _log(rng, 300, 1500), "f16s", "bgk", requests=rng.randint(4, 12))
    if kind == "snapshots":
        return _case(None, kind, rng.randint(60, 600), rng.randint(60, 400), rng.randint(10, 100), "f32", collision,
                     gamma=rng.choice([1, 5, 10]))
    if kind == "droplet":
        return _case(None, kind, rng.randint(60, 300), rng.randint(60, 300), rng.randint(40, 200), storage, "mrt",
                     nsc=rng.random() < 0.7, angle=rng.choice([45, 60, 90, 120]))
    nodes = _log(rng, 64 * 64, 1 << 23)
    steps = max(1, min(rng.randint(30, 220), (1 << 28) // nodes))
    if collision == "mrt" and rng.random() < 0.3:
        kw["nsc"] = True
    if rng.random() < 0.2:
        kw["gradient"] = "isotropic"
    if kind == "bubble":
        nx = int(math.sqrt(nodes) * rng.uniform(0.8, 1.3))
        return _case(None, kind, nx, max(32, nodes // nx), steps, storage, collision, gamma=rng.choice([1, 5, 10, 100]), **kw)
    ny = max(24, int(math.sqrt(nodes / 16) * rng.uniform(0.8, 1.3)))
    nx = max(128, nodes // ny)
    if kind == "slug":
        return _case(None, kind, nx, ny, steps, storage, collision, gamma=rng.choice([5, 10]), **kw)
    return _case(None, kind, nx, ny, steps, storage, collision, walls=rng.choice(["freeslip", "walls", "slip_top"]), **kw)


# ------------------------------------------------------------------ inputs --


def _flow(rng, nx, ny, amplitude, wall_y):
    """A smooth seeded velocity field: a few modes of the box (of a half box along a walled y)."""
    x = (torch.arange(nx, device=DEVICE, dtype=torch.float64) + 0.5) / nx
    y = (torch.arange(ny, device=DEVICE, dtype=torch.float64) + 0.5) / ny
    u = torch.zeros((2, ny, nx), device=DEVICE, dtype=torch.float64)
    for _ in range(3):
        kx, ky, a, b = rng.randint(1, 3), rng.randint(1, 3), rng.uniform(0, 2 * math.pi), rng.uniform(0, 2 * math.pi)
        sy = torch.sin(math.pi * ky * y) if wall_y else torch.sin(2 * math.pi * ky * y + b)
        cy = torch.sin(math.pi * (ky + 1) * y) if wall_y else torch.cos(2 * math.pi * ky * y + b)
        u[0] += sy[:, None] * torch.cos(2 * math.pi * kx * x + a)[None, :]
        u[1] += cy[:, None] * torch.sin(2 * math.pi * kx * x + a)[None, :]
    return u * (amplitude / 3)


def _disk(rng, nx, ny, rho_in, rho_out):
    r = rng.uniform(0.18, 0.28) * min(nx, ny)
    cx, cy = nx * rng.uniform(0.45, 0.55), ny * rng.uniform(0.45, 0.55)
    x = torch.arange(nx, device=DEVICE, dtype=torch.float64)[None, :] + (0.5 - cx)
    y = torch.arange(ny, device=DEVICE, dtype=torch.float64)[:, None] + (0.5 - cy)
    red = (x * x + y * y < r * r).double()
    return red * rho_in, (1.0 - red) * rho_out


def _lattice_input(case, seed, index=0):
    """Parameters and initial fields (rho_r, rho_b, u, inlet colours) of one lattice of a case."""
    rng = random.Random("%d %d" % (seed, index))
    nx, ny, storage, coll = case["nx"], case["ny"], case["storage"], case["collision"]
    inlet, kind = None, case["kind"]
    if kind == "channel":
        c = dict(gamma=5, u_in=0.01) if not case.get("nsc") else dict(gamma=5, u_in=0.03)
        heavy = rng.uniform(0.4, 0.8)
        p = W.inlet_outlet(nx=2, ny=2, storage=storage, collision=coll, walls="walls", **c)["params"]
        p.update(nx=nx, ny=ny, bc_y=case.get("walls", "freeslip"))
        if case.get("nsc"):                     # the verification set-up: the light fluid six times slower
            p.update(u_in_b=0.005, tau_r=1.0, tau_b=1.0)
        red = (torch.arange(ny, device=DEVICE) < int(heavy * ny)).double()[:, None].expand(ny, nx)
        rr, rb = red * 5.0, 1.0 - red
        inlet = np.where(red[:, 0].cpu().numpy() > 0, 1, -1).astype(np.int8)
        u = _flow(rng, nx, ny, 0.002, True)
    elif kind == "slug":
        p = W.slug_params(nx, ny, gamma=case["gamma"], storage=storage, collision=coll)
        edges = W.slug_edges(nx, np.random.default_rng(rng.randrange(1 << 30)), lo=max(16, min(200, nx // 8)),
                             hi=max(32, min(600, nx // 4)))
        heavy = torch.zeros(nx, device=DEVICE, dtype=torch.float64)
        for b, e in enumerate(edges):
            heavy[e:edges[b + 1] if b + 1 < len(edges) else nx] = float(b % 2 == 0)
        rr, rb = heavy[None, :].expand(ny, nx) * float(case["gamma"]), (1.0 - heavy)[None, :].expand(ny, nx)
        u = _flow(rng, nx, ny, 0.002, True)
    elif kind == "droplet":
        p = W.wall_droplet(case["angle"], n=16, storage=storage, collision=coll)["params"]
        p.update(nx=nx, ny=ny)
        w, h = max(8, int(nx * rng.uniform(0.3, 0.4))), max(6, int(ny * rng.uniform(0.15, 0.25)))
        red = torch.zeros((ny, nx), device=DEVICE, dtype=torch.float64)
        red[:h, (nx - w) // 2:(nx - w) // 2 + w] = 1.0
        rr, rb, u = red, 1.0 - red, _flow(rng, nx, ny, 0.002, True)
    elif kind == "sweep":
        g, m = (1, 10, 100)[index // 3], (1, 10, 100)[index % 3]
        p = W.bubble_params(g, m, n=nx, storage=storage, collision=coll)
        rr, rb = _disk(rng, nx, ny, 1.0, float(g))
        u = _flow(rng, nx, ny, 0.002, False)
    else:
        g = case["gamma"]
        p = W.bubble_params(g, g, n=nx, storage=storage, collision=coll, tau_min=0.8)
        p["ny"] = ny
        rr, rb = _disk(rng, nx, ny, 1.0, float(g))
        u = _flow(rng, nx, ny, 0.05 if kind == "snapshots" else 0.002, False)
    if case.get("gradient"):
        p["gradient"] = case["gradient"]
    if case.get("nsc"):
        p.update(collision="mrt", ns_correction=True)
    return p, rr, rb, u, inlet


def _requests(case, seed):
    """A burst of the serving mix: bubbles and slugs of log-uniform sizes and step counts, no larger than the case."""
    side = case["nx"]
    trace = W.serve_trace(seed=seed, n=case["requests"], nodes_lo=64 * 64, nodes_hi=side * side,
                          steps_lo=max(100, case["steps"] // 6), steps_hi=case["steps"], storage=case["storage"])
    rng = random.Random(seed)
    # the same sizes and step counts for every seed, so that passes cost the same; fluids and geometry by the seed
    sizes = W.serve_trace(seed=7, n=case["requests"], nodes_lo=64 * 64, nodes_hi=side * side,
                          steps_lo=max(100, case["steps"] // 6), steps_hi=case["steps"], storage=case["storage"])
    out = []
    for t, s in zip(trace, sizes):
        p = s["params"]
        nx, ny = p["nx"], p["ny"]
        if s["kind"] == "bubble":
            g = min(t["gamma"], 100)
            p = W.bubble_params(g, g, n=nx, storage=case["storage"])
            init = serve.init_disk(nx / 2, ny / 2, nx * rng.uniform(0.2, 0.3), 1.0, 0.0, 0.0, float(g))
        else:
            g = rng.choice(W.SERVE_SLUG_GAMMAS)
            p = W.slug_params(nx, ny, gamma=g, Re=10, storage=case["storage"])
            edges = W.slug_edges(nx, np.random.default_rng(rng.randrange(1 << 30)))
            init = serve.init_bands(edges, float(g), 1.0)
        out.append((p, init, s["steps"]))
    return out


# ------------------------------------------------------- prepare and run --

_STREAM = []


def _stream():
    """The program's one stream."""
    if not _STREAM:
        _STREAM.append(torch.cuda.Stream())
    return _STREAM[0]


def _host(t):
    return t.contiguous().cpu().numpy()


class _OwnBuffers:
    """A lattice whose two population buffers are the program's own tensors; the state is in the one of the step
    counter's parity."""

    def __init__(self, p, rr, rb, u, inlet):
        size = int(capi.load().lbm_buffer_bytes(ctypes.byref(capi.make_params(p))))
        self.p = p
        self.buf = [torch.zeros(size, dtype=torch.uint8, device="cuda") for _ in range(2)]
        torch.cuda.synchronize()
        self.lat = capi.Lattice(p, stream=_stream().cuda_stream, buffers=[b.data_ptr() for b in self.buf])
        self.lat.init(_host(rr), _host(rb), _host(u[0]), _host(u[1]))
        if inlet is not None:
            self.lat.set_inlet_color(inlet)

    def state(self):
        b = self.buf[self.lat.steps_done & 1]
        if self.p["storage"] == "f32":
            return b.view(torch.float32)
        # 16-bit storage, per 64 columns of a row: an FP32 rest population and eight 16-bit values
        blocks = b.view(2, self.p["ny"], -1, 1280)
        rest = blocks[..., :256].view(torch.float32)
        # a rest population is the value itself or, marked by its last bit, the deviation from the rest state
        ref = torch.tensor([rho * _phi(self.p)[k][0] for k, rho in enumerate((self.p["rho0_r"], self.p["rho0_b"]))],
                           dtype=torch.float32).view(2, 1, 1, 1).to("cuda", non_blocking=True)
        rest = rest + ref * (rest.view(torch.int32) & 1)
        kind = torch.float16 if self.p["storage"] == "f16s" else torch.bfloat16
        return {"rest": rest, "deviation": blocks[0, ..., 256:].view(kind),
                "share": blocks[1, ..., 256:].view(torch.uint16).to(torch.float32)}


def prepare(case, seed):
    kind = case["kind"]
    if kind == "serve":
        return dict(kind=kind, requests=_requests(case, seed),
                    server=serve.Server(hbm_budget=8 << 30, max_slots=48, chunk_steps=100, storage=case["storage"]))
    if kind == "snapshots":
        p, rr, rb, u, _ = _lattice_input(case, seed)
        lat = capi.Lattice(p, stream=_stream().cuda_stream)
        lat.init(_host(rr), _host(rb), _host(u[0]), _host(u[1]))
        return dict(kind=kind, lat=lat, steps=case["steps"])
    own = [_OwnBuffers(*_lattice_input(case, seed, i)) for i in range(9 if kind == "sweep" else 1)]
    batch = capi.Batch([o.lat for o in own], stream=_stream().cuda_stream) if kind == "sweep" else None
    return dict(kind=kind, own=own, batch=batch, steps=case["steps"])


def run(state):
    kind = state["kind"]
    if kind == "serve":
        s = state["server"]
        ids = [s.enqueue(p, init, steps, keep_fields=True) for p, init, steps in state["requests"]]
        out = []
        for rid in ids:
            r = s.wait(rid, fields=True)
            s.release(rid)
            out.append(np.stack([r[k] for k in _FIELDS]).astype(np.float16))
        return out
    if kind == "snapshots":
        out = []
        for _ in range(2):
            state["lat"].step(state["steps"])
            d = state["lat"].diag()
            m = state["lat"].moments()
            out.append(dict({k: d[k] for k in ("mass_r", "mass_b", "area_r", "max_u")},
                            **{k: m[k].astype(np.float32) for k in _FIELDS}))
        return out
    if kind == "sweep":
        state["batch"].step(state["steps"])
    else:
        state["own"][0].lat.step(state["steps"])
    with torch.cuda.stream(_stream()):
        return [o.state() for o in state["own"]]


_FIELDS = ("rho_r", "rho_b", "ux", "uy", "p")


def work(case):
    """The state read once and written once, and the steps' arithmetic (about 400 operations a node and step:
    moments, gradient, collision, perturbation and recolouring of 2 x 9 populations)."""
    if case["kind"] == "serve":
        req = [(p["nx"] * p["ny"], steps) for p, _, steps in _requests(case, 0)]
        return {"bytes": sum(n * (16 + 5 * 8) for n, _ in req), "flops": 400.0 * sum(n * s for n, s in req)}
    n = case["nx"] * case["ny"] * (9 if case["kind"] == "sweep" else 1)
    steps = case["steps"] * (2 if case["kind"] == "snapshots" else 1)
    size = 144 if case["storage"] == "f32" else 80
    return {"bytes": float(n * size + (2 * 5 * 8 * n if case["kind"] == "snapshots" else 0)), "flops": 400.0 * n * steps}


# ------------------------------------------------------- the method in 64 bits --

CX = (0, 1, 0, -1, 0, 1, -1, -1, 1)
CY = (0, 0, 1, 0, -1, 1, 1, -1, -1)
CLS = (0, 1, 1, 1, 1, 2, 2, 2, 2)
OPP = (0, 3, 4, 1, 2, 7, 8, 5, 6)
MIRROR = (0, 1, 4, 3, 2, 8, 7, 6, 5)                     # the same c_x, the opposite c_y
WGT = (4 / 9, 1 / 9, 1 / 36)
BCO = (-4 / 27, 2 / 27, 5 / 108)
HERMITE = (-2.0, -0.5, 1.0)                              # (3 |c|^2 - 4) / 2
ISO = {1: 4 / 21, 2: 4 / 45, 4: 1 / 60, 5: 2 / 315, 8: 1 / 5040}
MRT = np.array([[1] * 9, [-4, -1, -1, -1, -1, 2, 2, 2, 2], [4, -2, -2, -2, -2, 1, 1, 1, 1], [0, 1, 0, -1, 0, 1, -1, -1, 1],
                [0, -2, 0, 2, 0, 1, -1, -1, 1], [0, 0, 1, 0, -1, 1, 1, -1, -1], [0, 0, -2, 0, 2, 1, 1, -1, -1],
                [0, 1, -1, 1, -1, 0, 0, 0, 0], [0, 0, 0, 0, 0, 1, -1, 1, -1]], dtype=np.float64)


def _alphas(p):
    a, r, b = p["alpha_light"], p["rho0_r"], p["rho0_b"]
    return (a, 1 - (1 - a) * r / b) if r <= b else (1 - (1 - a) * b / r, a)


def _phi(p):
    return [(a, (1 - a) / 5, (1 - a) / 20) for a in _alphas(p)]


class _Exact:
    """The colour-gradient step of Sec. 2 in plain FP64 tensors."""

    def __init__(self, p, rr, rb, u, inlet):
        self.p, self.phi = p, _phi(p)
        self.k3 = [0.8 - 1.8 * a for a in _alphas(p)]                  # 3 c_s^2 - 1
        self.cs2 = [3 * (1 - a) / 5 for a in _alphas(p)]
        self.nsc = bool(p["ns_correction"])
        self.xper, self.yper = p["bc_x"] == "periodic", p["bc_y"] == "periodic"
        self.slip = {"periodic": (0, 0), "walls": (0, 0), "freeslip": (1, 1), "slip_top": (0, 1)}[p["bc_y"]]
        self.inlet = None if inlet is None else torch.from_numpy(inlet).to(rr.device) > 0
        self.M, self.Mi = (torch.from_numpy(m).to(rr.device) for m in (MRT, np.linalg.inv(MRT)))
        uu = u[0] ** 2 + u[1] ** 2
        self.f = torch.empty((2, 9) + tuple(rr.shape), device=rr.device, dtype=torch.float64)
        for k, rho in enumerate((rr, rb)):
            for i in range(9):
                cu = CX[i] * u[0] + CY[i] * u[1]
                lin = 3 * cu * (1 + HERMITE[CLS[i]] * self.k3[k]) if self.nsc else 3 * cu
                self.f[k, i] = rho * (self.phi[k][CLS[i]] + WGT[CLS[i]] * (lin + 4.5 * cu * cu - 1.5 * uu))

    def pull(self):
        """Streamed and boundary-completed state: N (colour-blind), rho_r, rho_b."""
        p, g = self.p, torch.empty_like(self.f)
        for i in range(9):
            g[:, i] = torch.roll(self.f[:, i], (CY[i], CX[i]), (1, 2))
            if CY[i] and not self.yper:
                row, slip = (0, self.slip[0]) if CY[i] > 0 else (-1, self.slip[1])
                g[:, i, row] = (torch.roll(self.f[:, MIRROR[i], row], CX[i], 1) if slip and CX[i]
                                else self.f[:, OPP[i], row])
        N, rho = g.sum(0), g.sum(1)
        if not self.xper:
            red = self.inlet
            one = torch.ones(N.shape[1], device=N.device, dtype=torch.float64)
            a = N[:, :, 0].clone()
            vx = torch.where(red, p["u_in_r"] * one, p["u_in_b"] * one)
            rin = (a[0] + a[2] + a[4] + 2 * (a[3] + a[6] + a[7])) / (1 - vx)
            H = torch.where(red, self.k3[0] * one, self.k3[1] * one) * rin * vx / 3 if self.nsc else 0
            N[1, :, 0] = a[3] + 2 / 3 * rin * vx - H
            N[5, :, 0] = a[7] - 0.5 * (a[2] - a[4]) + rin * vx / 6 + 0.5 * H
            N[8, :, 0] = a[6] + 0.5 * (a[2] - a[4]) + rin * vx / 6 + 0.5 * H
            rho[0, :, 0], rho[1, :, 0] = torch.where(red, rin, 0 * rin), torch.where(red, 0 * rin, rin)
            a = N[:, :, -1].clone()
            v = [sum(g[k, i, :, -1] for i in range(9) if CX[i] >= 0) / r for k, r in enumerate((p["rho0_r"], p["rho0_b"]))]
            chi = [(x / (v[0] + v[1])).clamp(0, 1) for x in v]
            rho[0, :, -1], rho[1, :, -1] = chi[0] * p["p_out"] / self.cs2[0], chi[1] * p["p_out"] / self.cs2[1]
            ro = rho[0, :, -1] + rho[1, :, -1]
            vx = (a[0] + a[2] + a[4] + 2 * (a[1] + a[5] + a[8])) / ro - 1
            H = (chi[0] * self.k3[0] + chi[1] * self.k3[1]) * ro * vx / 3 if self.nsc else 0
            N[3, :, -1] = a[1] - 2 / 3 * ro * vx + H
            N[6, :, -1] = a[8] - 0.5 * (a[2] - a[4]) - ro * vx / 6 - 0.5 * H
            N[7, :, -1] = a[5] + 0.5 * (a[2] - a[4]) - ro * vx / 6 - 0.5 * H
        return N, rho

    def fields(self):
        N, rho = self.pull()
        t = rho[0] + rho[1]
        ux, uy = self.velocity(N, t)
        return {"rho_r": rho[0], "rho_b": rho[1], "ux": ux, "uy": uy, "p": rho[0] * self.cs2[0] + rho[1] * self.cs2[1]}

    def velocity(self, N, rho):
        return ((N[1] - N[3] + N[5] - N[7] + N[8] - N[6]) / rho + 0.5 * self.p["gx"],
                (N[2] - N[4] + N[5] - N[7] + N[6] - N[8]) / rho + 0.5 * self.p["gy"])

    def padded(self, a):
        """Two ghost rows and columns: periodic wrap, the nearest column beyond an open face, the weighted mean over
        the fluid neighbours beyond a wall (repeated in the second row)."""
        nx = a.shape[1]
        x = torch.arange(-2, nx + 2, device=a.device)
        e = a[:, x % nx if self.xper else x.clamp(0, nx - 1)]
        if self.yper:
            return torch.cat([e[[-2, -1]] if e.shape[0] > 1 else e[[0, 0]], e, e[[0, 1 % e.shape[0]]]])
        inside = torch.ones_like(x, dtype=torch.float64) if self.xper else ((x >= 0) & (x < nx)).double()

        def ghost(row):
            w, v = 4 * inside, 4 * inside * row
            for s in (1, -1):
                near = torch.roll(inside, s)
                if not self.xper:                        # nothing wraps around beyond an open face
                    near[0 if s > 0 else -1] = 0
                w, v = w + near, v + near * torch.roll(row, s)
            g = v / w.clamp(min=1)
            if self.xper:                                # the outermost columns' neighbours wrap
                return g[2 + (x % nx)]
            g[0], g[-1] = torch.where(w[0] > 0, g[0], g[1]), torch.where(w[-1] > 0, g[-1], g[-2])
            return g

        lo, hi = ghost(e[0]), ghost(e[-1])
        return torch.cat([lo[None], lo[None], e, hi[None], hi[None]])

    def gradient(self, a, iso=False):
        e, (ny, nx) = self.padded(a), a.shape
        gx, gy, reach = torch.zeros_like(a), torch.zeros_like(a), 2 if iso else 1
        for dy in range(-reach, reach + 1):
            for dx in range(-reach, reach + 1):
                r2 = dx * dx + dy * dy
                if r2:
                    w = ISO[r2] if iso else (1 / 3 if r2 == 1 else 1 / 12)
                    v = e[2 + dy:2 + dy + ny, 2 + dx:2 + dx + nx]
                    gx, gy = gx + w * dx * v, gy + w * dy * v
        return gx, gy

    def wetted(self, Fx, Fy):
        """Sec. 2.4: the gradient of the wall rows turned to the contact angle."""
        t = math.radians(180 - self.p["contact_angle"])
        for row, n in ((0, 1.0), (-1, -1.0)):
            fx, fy = Fx[row].clone(), Fy[row].clone()
            m = torch.sqrt(fx * fx + fy * fy)
            there, tie = m * m > 1e-24, fx == 0
            nx = torch.where(tie, 0 * fx, torch.sign(fx) * math.sin(t))
            ny = torch.where(tie, torch.ones_like(fx), math.cos(t) * torch.ones_like(fx)) * n
            Fx[row], Fy[row] = torch.where(there, m * nx, fx), torch.where(there, m * ny, fy)
        return Fx, Fy

    def step(self):
        p, (N, rho) = self.p, self.pull()
        rr, rb = rho[0], rho[1]
        t = rr + rb
        ux, uy = self.velocity(N, t)
        vr, vb = rr / p["rho0_r"], rb / p["rho0_b"]
        psi = (vr - vb) / (vr + vb)
        wr, wb, d = 1 / p["tau_r"], 1 / p["tau_b"], p["delta"]
        chi = 2 * wr * wb / (wr + wb)
        eta, lam = 2 * (wr - chi) / d, 2 * (chi - wb) / d
        mid = torch.where(psi > 0, chi + psi * (eta - eta / (2 * d) * psi), chi + psi * (lam + lam / (2 * d) * psi))
        w = torch.where(psi > d, torch.full_like(psi, wr), torch.where(psi < -d, torch.full_like(psi, wb), mid))
        K = rr * self.k3[0] + rb * self.k3[1]
        uu = ux * ux + uy * uy
        neq, guo = torch.empty_like(N), torch.empty_like(N)
        for i in range(9):
            cu = CX[i] * ux + CY[i] * uy
            lin = 3 * cu * (t + HERMITE[CLS[i]] * K) if self.nsc and i else 3 * cu * t
            neq[i] = N[i] - (rr * self.phi[0][CLS[i]] + rb * self.phi[1][CLS[i]]
                             + WGT[CLS[i]] * (lin + t * (4.5 * cu * cu - 1.5 * uu)))
            guo[i] = WGT[CLS[i]] * t * ((3 * (CX[i] - ux) + 9 * cu * CX[i]) * p["gx"] + (3 * (CY[i] - uy) + 9 * cu * CY[i]) * p["gy"])
        if p["collision"] == "mrt":
            m, mg = (torch.tensordot(self.M, a, 1) for a in (neq, guo))
            s = torch.stack([(w if j >= 7 else p["mrt_lambda"] * w) for j in range(9)])
            q = s * m - (1 - 0.5 * s) * mg
            if self.nsc:
                dqx, dqy = self.gradient(-K * ux)[0], self.gradient(-K * uy)[1]
                q[1] -= 3 * (1 - 0.5 * s[1]) * (dqx + dqy)
                q[7] -= (1 - 0.5 * s[7]) * (dqx - dqy)
            ns = N - torch.tensordot(self.Mi, q, 1)
        else:
            ns = N - w * neq + (1 - 0.5 * w) * guo
        Fx, Fy = self.gradient(psi, p["gradient"] == "isotropic")
        if p["contact_angle"] >= 0:
            Fx, Fy = self.wetted(Fx, Fy)
        F2 = Fx * Fx + Fy * Fy
        on = F2 > 1e-24
        Fm = torch.where(on, torch.sqrt(F2), torch.zeros_like(F2))
        inv = torch.where(on, 1 / torch.sqrt(torch.where(on, F2, torch.ones_like(F2))), torch.zeros_like(F2))
        A = 9 * p["sigma"] / 4 * w if p["sigma"] > 0 else p["A"]
        for i in range(9):
            fc = CX[i] * Fx + CY[i] * Fy
            nss = ns[i] + A * (WGT[CLS[i]] * fc * fc * inv - BCO[CLS[i]] * Fm)
            self.f[0, i] = rr / t * nss
            if i:
                length = math.sqrt(CX[i] ** 2 + CY[i] ** 2)
                self.f[0, i] += p["beta"] * rr * rb / (t * t) * fc * inv / length * (rr * self.phi[0][CLS[i]] + rb * self.phi[1][CLS[i]])
            self.f[1, i] = nss - self.f[0, i]

    def area(self, m):
        a, b = m["rho_r"] / self.p["rho0_r"], m["rho_b"] / self.p["rho0_b"]
        return (a / (a + b)).sum()

    def blocks(self, a):
        """[..., ny, nx] as rows of 64-column blocks, zeros beyond nx."""
        pad = -a.shape[-1] % 64
        a = torch.nn.functional.pad(a, (0, pad))
        return a.reshape(*a.shape[:-1], -1, 64)

    def state(self):
        p, ny = self.p, self.f.shape[2]
        b = self.blocks(self.f)                                            # [2, 9, ny, blocks, 64]
        if p["storage"] == "f32":
            return b.permute(0, 2, 3, 1, 4).reshape(-1)
        scale = 4096 / max(p["rho0_r"], p["rho0_b"])
        ref = torch.tensor([p["rho0_r"] * self.phi[0][CLS[i]] for i in range(1, 9)], device=b.device, dtype=torch.float64)
        n = self.f[:, 1:].sum(0)
        dev, share = (n - ref.view(8, 1, 1)) * scale, 65535 * self.f[0, 1:] / n
        flat = [self.blocks(a).permute(1, 2, 0, 3) for a in (dev, share)]   # [ny, blocks, 8, 64]
        return {"rest": b[:, 0], "deviation": flat[0].reshape(ny, -1, 512), "share": flat[1].reshape(ny, -1, 512)}


def exact(case, seed):
    if case["kind"] == "serve":                          # minutes of plain steps
        return None
    out = []
    for i in range(9 if case["kind"] == "sweep" else 1):
        sim = _Exact(*_lattice_input(case, seed, i))
        for _ in range(2 if case["kind"] == "snapshots" else 1):
            for _ in range(case["steps"]):
                sim.step()
            if case["kind"] == "snapshots":
                m = sim.fields()
                out.append(dict({k: v.cpu().numpy() for k, v in m.items()}, mass_r=float(m["rho_r"].sum()), mass_b=float(m["rho_b"].sum()),
                                area_r=float(sim.area(m)), max_u=float(torch.sqrt(m["ux"] ** 2 + m["uy"] ** 2).max())))
        if case["kind"] != "snapshots":
            out.append(sim.state())
    return out
