"""The work that programs have this library do, as measurable cases.

A case is one program's loop body: it advances a lattice (or a box, or a
stream of requests) through the public entry points and reads a result back.
Kinds:

* ``wave``, ``flow``: a periodic D2Q9 lattice that holds a decaying shear wave
  or a smooth random flow, advanced ``steps`` time steps per pass, then read
  (``read``: moments into a device tensor, moments on the host, or diagnostics
  and device moments, as a monitored run does);
* ``tube``, ``walls``: a shocktube experiment from its initial fields to its
  density profile (periodic, or with full-way bounce-back wall columns);
* ``restart``: populations of a checkpoint in, ``steps`` time steps,
  populations of the next checkpoint out, all on the host;
* ``box``: a periodic D3Q27 box with a shear wave;
* ``serve``: a batch of independent requests through the server.

``exact`` restates the method (Eqs. (1), (6), (7) and (11) of arXiv
2501.16000, and its second-order polynomial equilibrium) in plain torch FP64.
"""
import math

import numpy as np
import torch

from paper_2501_16000_amd import oreg, oreg3, serve

STORAGE_BYTES = {"f64": 8, "f32s": 4, "f16s": 2, "bf16s": 2}
FLOPS_2D, FLOPS_3D = 125, 480  # per node and step (FMA = 2)


def _dev():
    return "cuda" if torch.cuda.is_available() else "cpu"


def listed():
    return [
        # The smallest call: the 32 x 32 wave of the viscosity measurement (Fig. 2),
        # read on the host every 50 steps.
        dict(name="wave-32-f64", kind="wave", nx=32, ny=32, storage="f64", eq="guided", coll="oreg",
             theta=1 / 3, tau=0.53, steps=50, read="host"),
        # The first workload: a 128 x 128 rotated wave, 500 steps, moments kept on the device.
        dict(name="wave-128-f64", kind="wave", nx=128, ny=128, storage="f64", eq="guided",
             coll="oreg", theta=1 / 3, tau=0.8, steps=500, read="device"),
        # The walled shocktube of Sec. IV: one row of 800 nodes, 500 steps, density profile.
        dict(name="walls-800x1-f64", kind="walls", nx=800, ny=1, storage="f64", eq="guided",
             coll="oreg", theta=0.35, tau=0.5 + 1e-5 / 0.35, steps=500),
        # The periodic shocktube workload, a long flat lattice in shifted FP32.
        dict(name="tube-16384x4-f32s", kind="tube", nx=16384, ny=4, storage="f32s", eq="guided",
             coll="oreg", theta=1 / 3, tau=0.55, steps=400),
        # An ordinary monitored run on odd sizes: random flow, diagnostics and moments.
        dict(name="flow-777x523-f32s", kind="flow", nx=777, ny=523, storage="f32s", eq="guided",
             coll="oreg", theta=1 / 3, tau=0.7, steps=100, read="diagnostics"),
        # Restart from a checkpoint and write the next one.
        dict(name="restart-512-f64", kind="restart", nx=512, ny=512, storage="f64", eq="guided",
             coll="oreg", theta=1 / 3, tau=0.6, steps=40),
        # The benchmark lattice in FP64 and in shifted FP32.
        dict(name="wave-4096-f64", kind="wave", nx=4096, ny=4096, storage="f64", eq="guided",
             coll="oreg", theta=1 / 3, tau=0.6, steps=20, read="device"),
        dict(name="wave-4096-f32s", kind="wave", nx=4096, ny=4096, storage="f32s", eq="guided",
             coll="oreg", theta=1 / 3, tau=0.6, steps=60, read="device"),
        # The largest lattice: polynomial equilibrium, random flow, FP16 storage.
        dict(name="flow-8192-poly2-f16s", kind="flow", nx=8192, ny=8192, storage="f16s", eq="poly2",
             coll="oreg", theta=1 / 3, tau=0.7, steps=30, read="device"),
        # The D3Q27 benchmark box in FP64, and a smaller odd one in BF16.
        dict(name="box-256-f64", kind="box", nx=256, ny=256, nz=256, storage="f64", eq="guided",
             coll="oreg", theta=1 / 3, tau=0.6, steps=10),
        dict(name="box-100x84x60-bf16s", kind="box", nx=100, ny=84, nz=60, storage="bf16s",
             eq="guided", coll="oreg", theta=1 / 3, tau=0.6, steps=50),
        # The serving mix (sides 32 to 1024), a batch of 24 requests in shifted FP32.
        dict(name="serve-24-f32s", kind="serve", count=24, n_min=32, n_max=1024, steps_min=200,
             steps_max=800, storage="f32s", eq="guided", theta=1 / 3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    storage = rng.choice(["f64", "f64", "f32s", "f32s", "f16s", "bf16s"])
    eq = rng.choice(["guided", "guided", "guided", "poly2"])
    coll = rng.choice(["oreg", "oreg", "oreg", "bgk"])
    theta = 1 / 3 if eq == "poly2" else rng.choice([1 / 3, 1 / 3, 0.35, 0.4])
    tau = round(rng.uniform(0.55, 1.1), 3)
    kind = rng.choice(["wave", "wave", "wave", "flow", "flow", "tube", "walls", "restart", "box",
                       "box", "box", "serve"])
    case = dict(kind=kind, storage=storage, eq=eq, coll=coll, theta=theta, tau=tau)
    if kind in ("wave", "flow"):
        case["nx"], case["ny"] = _log(rng, 32, 4096), _log(rng, 32, 4096)
        most = int(1.2e9 // (case["nx"] * case["ny"]))
        case["steps"] = _log(rng, 1, min(600, most))
        case["read"] = rng.choice(["device", "device", "host", "diagnostics"])
        if case["nx"] * case["ny"] > 1 << 20 and case["read"] == "host":
            case["read"] = "device"
    elif kind in ("tube", "walls"):
        case["nx"], case["ny"] = _log(rng, 200, 16384), rng.randint(1, 64)
        case["steps"] = _log(rng, 50, 500)
    elif kind == "restart":
        case["nx"], case["ny"] = _log(rng, 32, 700), _log(rng, 32, 700)
        case["steps"] = _log(rng, 1, 100)
    elif kind == "box":
        for a in ("nx", "ny", "nz"):
            case[a] = _log(rng, 16, 256)
        case["steps"] = _log(rng, 1, min(100, int(1.5e8 // (case["nx"] * case["ny"] * case["nz"]))))
    else:
        lo = _log(rng, 32, 128)
        case = dict(kind="serve", count=rng.randint(2, 24), n_min=lo, n_max=_log(rng, lo, 800),
                    steps_min=100, steps_max=_log(rng, 200, 800), storage=storage, eq=eq,
                    theta=theta)
    return case


# ---------------------------------------------------------------- inputs --
def _wave(case, rng, dev):
    """A rotated shear wave (fronts along atan(1/2)) of seeded amplitude and phase."""
    nx, ny = case["nx"], case["ny"]
    u0, ph = rng.uniform(0.02, 0.05), rng.uniform(0.0, 1.0)
    x = torch.arange(nx, dtype=torch.float64, device=dev)[None, :]
    y = torch.arange(ny, dtype=torch.float64, device=dev)[:, None]
    amp = u0 * torch.sin(2 * math.pi * (2 * x / nx + y / ny + ph))
    return torch.ones_like(amp), amp * (-1 / math.sqrt(5)), amp * (2 / math.sqrt(5))


def _flow(case, rng, dev):
    """A smooth divergence-free flow: 8 x 8 Fourier modes of seeded phase, max |u| = 0.03."""
    nx, ny, m = case["nx"], case["ny"], 8
    a = torch.tensor(rng.standard_normal((m, m)), device=dev)
    al, be = (torch.tensor(rng.uniform(0, 2 * math.pi, (m, 1)), device=dev) for _ in range(2))
    k = torch.arange(1, m + 1, dtype=torch.float64, device=dev)[:, None]
    a = a / (k ** 2 + k.T ** 2)
    kx, ky = 2 * math.pi / nx * k, 2 * math.pi / ny * k
    px = kx * torch.arange(nx, dtype=torch.float64, device=dev) + al
    py = ky * torch.arange(ny, dtype=torch.float64, device=dev) + be
    ux = (ky * torch.cos(py)).T @ (a.T.contiguous() @ torch.sin(px))
    uy = -(torch.sin(py).T.contiguous() @ (a.T.contiguous() @ (kx * torch.cos(px))))
    scale = 0.03 / float(torch.sqrt(ux * ux + uy * uy).max())
    return torch.ones_like(ux), (ux * scale).contiguous(), (uy * scale).contiguous()


def _tube(case, rng, dev):
    """A density step at rest."""
    nx, ny = case["nx"], case["ny"]
    left, right = 1.5 * rng.uniform(0.95, 1.0), 0.75 * rng.uniform(1.0, 1.05)
    x = torch.arange(nx, device=dev)[None, :].expand(ny, nx)
    rho = torch.where(x < nx // 2, left, right).to(torch.float64).contiguous()
    return rho, torch.zeros_like(rho), torch.zeros_like(rho)


def _box(case, rng, dev):
    """A shear wave with fronts normal to (1, 1, 1) and seeded amplitude and phase."""
    u0, ph = rng.uniform(0.02, 0.05), rng.uniform(0.0, 1.0)
    x, y, z = (torch.arange(case[a], dtype=torch.float64, device=dev) / case[a]
               for a in ("nx", "ny", "nz"))
    amp = u0 * torch.sin(2 * math.pi * (x[None, None, :] + y[None, :, None] + z[:, None, None] + ph))
    return torch.ones_like(amp), amp / math.sqrt(2), -amp / math.sqrt(2), torch.zeros_like(amp)


def _checkpoint(case, rng):
    """Pre-collision populations a little off equilibrium, on the host."""
    shape = (case["ny"], case["nx"])
    rho = 1.0 + 0.05 * rng.uniform(-1, 1, shape)
    u = [torch.from_numpy(0.03 * rng.uniform(-1, 1, shape)) for _ in range(2)]
    f = _equilibrium(_C2, case["eq"], case["theta"], torch.from_numpy(rho), u).numpy()
    return f * (1.0 + 0.02 * rng.uniform(-1, 1, f.shape))


def _requests(case, rng):
    """Requests of the case's own sizes, relaxation times and step counts, with
    initial fields of seeded amplitude and phase on the host."""
    out, mix = [], _rng(16000)
    for _ in range(case["count"]):
        n = int(round(math.exp(mix.uniform(math.log(case["n_min"]), math.log(case["n_max"])))))
        tau = float(mix.uniform(0.52, 1.2))
        steps = int(mix.integers(case["steps_min"], case["steps_max"] + 1))
        fields = _wave(dict(nx=n, ny=n), rng, _dev())
        out.append((n, tau, steps, [t.cpu().numpy() for t in fields]))
    return out


_FIELDS = {"wave": _wave, "flow": _flow, "tube": _tube, "walls": _tube, "box": _box}


def _rng(seed):
    return np.random.Generator(np.random.PCG64(seed))


def _lattice(case):
    return oreg.Lattice(case["nx"], case["ny"], case["tau"], case["theta"], equilibrium=case["eq"],
                        storage=case["storage"], collision=case["coll"],
                        boundary_x="bounceback" if case["kind"] == "walls" else "periodic")


def prepare(case, seed):
    rng, kind, dev = _rng(seed), case["kind"], _dev()
    if kind == "serve":
        # The server and its clients' requests.
        server = serve.Server(memory_budget=2 << 30, pinned_bytes=256 << 20,
                              equilibrium=case["eq"], storage=case["storage"], theta=case["theta"])
        return dict(case=case, server=server, requests=_requests(case, rng))
    if kind == "restart":
        return dict(case=case, lattice=_lattice(case), f=_checkpoint(case, rng))
    fields = _FIELDS[kind](case, rng, dev)
    if kind in ("tube", "walls"):
        # An experiment starts from its fields each time, so they are what is kept.
        return dict(case=case, lattice=_lattice(case), fields=[t.cpu().numpy() for t in fields])
    if kind == "box":
        lat = oreg3.Lattice3(case["nx"], case["ny"], case["nz"], case["tau"], case["theta"],
                             equilibrium=case["eq"], storage=case["storage"],
                             collision=case["coll"])
        shape = (4, case["nz"], case["ny"], case["nx"])
    else:
        lat = _lattice(case)
        shape = (3, case["ny"], case["nx"])
    lat.init(*fields)
    out = torch.empty(shape, dtype=torch.float64, device=dev)
    return dict(case=case, lattice=lat, out=out)


def _serve(server, requests):
    """Submit as room allows, step, and collect results until all are back."""
    got, waiting = {}, list(range(len(requests)))
    while len(got) < len(requests):
        while waiting:
            n, tau, steps, fields = requests[waiting[0]]
            if not server.submit(waiting[0], *fields, tau, steps):
                break
            waiting.pop(0)
        server.step(4)
        while True:
            res = server.poll()
            if res is None:
                break
            got[res.tag] = server.fetch(res)
    return [got[tag] for tag in range(len(requests))]


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "serve":
        return _serve(state["server"], state["requests"])
    lat = state["lattice"]
    if kind in ("tube", "walls"):
        lat.init(*state["fields"])
        lat.step(case["steps"])
        return lat.density_profile()
    if kind == "restart":
        lat.set_populations(state["f"])
        lat.step(case["steps"])
        return lat.populations()
    lat.step(case["steps"])
    if kind == "box" or case["read"] == "device":
        return lat.moments(state["out"])
    if case["read"] == "host":
        return lat.moments()
    return dict(sums=lat.diagnostics(), moments=lat.moments(state["out"]))


def work(case):
    """The state read and written once per pass and the result written once (for
    experiments the initial fields read once), and the arithmetic of every step."""
    sz = STORAGE_BYTES[case["storage"]]
    if case["kind"] == "serve":
        side2 = ((case["n_max"] ** 2 - case["n_min"] ** 2)
                 / max(2 * math.log(case["n_max"] / case["n_min"]), 1e-9)
                 if case["n_max"] > case["n_min"] else case["n_min"] ** 2)
        nodes = case["count"] * side2
        steps = 0.5 * (case["steps_min"] + case["steps_max"])
        return dict(bytes=nodes * (2 * 9 * sz + 48), flops=nodes * steps * FLOPS_2D)
    nodes = case["nx"] * case["ny"] * case.get("nz", 1)
    if case["kind"] == "box":
        return dict(bytes=nodes * (2 * 27 * sz + 32), flops=nodes * case["steps"] * FLOPS_3D)
    flops = nodes * case["steps"] * FLOPS_2D
    if case["kind"] in ("tube", "walls"):
        return dict(bytes=nodes * 24 + case["nx"] * 8, flops=flops)
    if case["kind"] == "restart":
        return dict(bytes=nodes * 2 * 72, flops=flops)
    return dict(bytes=nodes * (2 * 9 * sz + 24), flops=flops)


# ----------------------------------------------------------------- exact --
_C2 = [(0, 0), (1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1)]
_C3 = [(x, y, z) for z in (-1, 0, 1) for y in (-1, 0, 1) for x in (-1, 0, 1)]


def _equilibrium(C, eq, theta, rho, u):
    """f^eq_i(rho, u), [q, ...]; components of c and u in the order x, y(, z)."""
    if eq == "guided":
        axis = [{0: 1 - theta - v * v, 1: (theta + v + v * v) / 2, -1: (theta - v + v * v) / 2}
                for v in u]
        out = []
        for c in C:
            f = rho
            for a, ca in enumerate(c):
                f = f * axis[a][ca]
            out.append(f)
        return torch.stack(out)
    u2 = sum(v * v for v in u)
    out = []
    for c in C:
        w = math.prod(2 / 3 if ca == 0 else 1 / 6 for ca in c)
        cu = sum(ca * v for ca, v in zip(c, u)) if any(c) else torch.zeros_like(rho)
        out.append(rho * w * (1 + 3 * cu + 4.5 * cu * cu - 1.5 * u2))
    return torch.stack(out)


def _moments(C, f):
    rho = f.sum(0)
    j = [sum(c[a] * f[i] for i, c in enumerate(C) if c[a]) for a in range(len(C[0]))]
    return rho, [v / rho for v in j]


def _collide(C, case, f, tau):
    rho, u = _moments(C, f)
    feq = _equilibrium(C, case["eq"], case["theta"], rho, u)
    if case.get("coll", "oreg") == "bgk":
        return f + (feq - f) / tau
    theta, D = case["theta"], len(C[0])
    fneq = f - feq
    # sum_k (c_k c_k - |c_k|^2 / D) f^neq_k, contracted with C C, C = c - u (Eq. 6)
    pi = [[sum(c[a] * c[b] * fneq[i] for i, c in enumerate(C) if c[a] * c[b]) for b in range(D)]
          for a in range(D)]
    tr = sum(pi[a][a] for a in range(D)) / D
    for a in range(D):
        pi[a][a] = pi[a][a] - tr
    g = torch.empty_like(f)
    for i, c in enumerate(C):
        P = [ca - v for ca, v in zip(c, u)]
        s = sum(pi[a][b] * P[a] * P[b] for a in range(D) for b in range(D))
        g[i] = feq[i] * (1 + (1 - 1 / tau) / (2 * theta * theta) * s / rho)
    return g


def _steps(C, case, f, tau, steps):
    axes = [f.dim() - 2 - a for a in range(len(C[0]))]  # array axis (of one f_i) of x, y(, z)
    walls = case["kind"] == "walls"
    opp = [C.index(tuple(-v for v in c)) for c in C]
    for _ in range(steps):
        g = _collide(C, case, f, tau)
        if walls:  # full-way bounce-back: the wall columns reverse every population
            for col in (0, -1):
                g[..., col] = f[opp][..., col]
        for i, c in enumerate(C):
            f[i] = torch.roll(g[i], shifts=c, dims=axes) if any(c) else g[i]
    return f


def exact(case, seed):
    rng, kind, dev = _rng(seed), case["kind"], _dev()
    if kind == "serve":
        out = []
        for n, tau, steps, fields in _requests(case, rng):
            rho, ux, uy = (torch.from_numpy(a).to(dev) for a in fields)
            f = _equilibrium(_C2, case["eq"], case["theta"], rho, [ux, uy])
            rho, u = _moments(_C2, _steps(_C2, case, f, tau, steps))
            out.append(torch.stack([rho, *u]))
        return out
    if kind == "restart":
        f = torch.from_numpy(_checkpoint(case, rng)).to(dev)
        return _steps(_C2, case, f, case["tau"], case["steps"])
    C = _C3 if kind == "box" else _C2
    rho, *u = _FIELDS[kind](case, rng, dev)
    f = _equilibrium(C, case["eq"], case["theta"], rho, u)
    f = _steps(C, case, f, case["tau"], case["steps"])
    rho, u = _moments(C, f)
    if kind in ("tube", "walls"):
        return rho.mean(0)
    m = torch.stack([rho, *u])
    if kind == "box" or case["read"] != "diagnostics":
        return m
    ke = 0.5 * (rho * (u[0] ** 2 + u[1] ** 2)).sum()
    sums = torch.stack([rho.sum(), (rho * u[0]).sum(), (rho * u[1]).sum(), ke,
                        case["theta"] * rho.sum() + ke, torch.zeros_like(ke)])
    return dict(sums=sums, moments=m)
