"""The work this library is used for, as cases that can be timed and compared.

Each case goes through the public entry points (`Lattice`, `Surrogate`) as the
drivers in `runner.py` and `bench.py` do: a lattice is built and kept, a pass
advances it by a group of steps and reads the particles back (the sampling
loops), starts it warm, writes a start field out, or trains and evaluates the
warm-start network.  `exact` restates the method in plain float64 torch over
dense grids, without this package's code.

Kinds of case:
  flow    nbox boxes (cubic with edges drawn from `edges` when nbox > 1),
          `per_box` particles each; a pass is `steps` time steps, then the
          particles, the last force and torque, and what `read` names
  start   the periodic creeping-flow start of one box, and its fields
  warm    network, start field and the first steps of an ensemble
  train   Adam epochs of the network from fresh parameters
  score   predictions, loss and gradient of the network over n samples
"""
import math
import random

import numpy as np
import torch

from paper_2403_05443_amd import Lattice, LBError, Surrogate, make_box

BYTES = {"fp64": 8, "fp32": 4, "fp16": 2, "bf16": 2}
NET = ((64, 8), (64, 64), (6, 64))  # (outputs, inputs) of the network's layers
ROOT3 = 1.0 / 3.0
OVERLAP = -5  # the status of two particles claiming one node


def flow(name=None, **kw):
    case = {"kind": "flow", "nbox": 1, "nx": 0, "ny": 0, "nz": 0, "edges": 0, "per_box": 1, "a": 4.0, "b": 2.0,
            "c": 2.0, "swim": False, "walls": False, "collision": "trt", "tau": 1.0, "storage": "fp32",
            "lattice": 19, "graph": 0, "steps": 25, "read": "none"}
    case.update(kw)
    return dict(case, name=name) if name else case


def listed():
    return [
        # one sampling interval of the smallest run: a settling spheroid in 32^3, double precision,
        # plain launches; launch latency and the particle kernel's chain
        flow("settle_32_fp64", nx=32, ny=32, nz=32, collision="bgk", storage="fp64", steps=50, read="momentum"),
        # an ordinary small run with uneven edges, a triaxial body and the ghost modes projected out
        flow("ragged_45x38x51_reg_fp32", nx=45, ny=38, nz=51, a=6.5, b=4.0, c=2.5, collision="reg", tau=0.8,
             graph=25, read="momentum"),
        # a spheroid turning in a wall-driven shear cell, with the velocity profile written out
        flow("shear_64x128x64_bgk_fp32", nx=64, ny=128, nz=64, a=9.0, b=3.0, c=3.0, walls=True, collision="bgk",
             tau=0.8, graph=25, read="fields"),
        # the inclined settling spheroid of the drift studies, as its drivers sample it
        flow("inclined_128_fp32", nx=128, ny=128, nz=128, a=6.0, tau=0.8, graph=50, steps=50),
        # the same on the larger velocity set
        flow("inclined_128_d3q27_fp32", nx=128, ny=128, nz=128, a=6.0, tau=0.8, lattice=27, graph=25),
        # the throughput workload: 256 uneven boxes, one loaded spheroid each, half precision
        flow("ensemble_256_fp16", nbox=256, edges=3, storage="fp16", graph=25),
        # squirmer suspensions: dilute in a large box, and 5 % by volume
        flow("squirmers_256_512_fp16", nx=256, ny=256, nz=256, per_box=512, a=5.0, b=2.5, c=2.5, swim=True,
             storage="fp16", graph=25),
        flow("squirmers_128_800_fp32", nx=128, ny=128, nz=128, per_box=800, a=5.0, b=2.5, c=2.5, swim=True,
             graph=25),
        # the start field of a settling study's box, written out
        {"name": "start_96_fp64", "kind": "start", "n": 96, "a": 7.5, "b": 2.5, "storage": "fp64"},
        # a held-out ensemble started warm and run to its first sample
        {"name": "warm_64_fp16", "kind": "warm", "nbox": 64, "edges": 103, "storage": "fp16", "steps": 25},
        # some epochs of the network's training, and what a validation pass asks of it
        {"name": "train_8192", "kind": "train", "n": 8192, "batch": 256, "epochs": 5},
        {"name": "score_2048", "kind": "score", "n": 2048},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["flow"] * 6 + ["start", "warm", "train", "score"])
    if kind == "start":
        return {"kind": "start", "n": rng.randint(32, 96), "a": round(rng.uniform(3.0, 9.0), 3),
                "b": round(rng.uniform(2.0, 3.0), 3), "storage": rng.choice(["fp64", "fp32", "fp16"])}
    if kind == "warm":
        return {"kind": "warm", "nbox": _log_int(rng, 2, 64), "edges": rng.randint(200, 9999),
                "storage": rng.choice(["fp16", "fp32"]), "steps": rng.randint(5, 25)}
    if kind == "train":
        return {"kind": "train", "n": _log_int(rng, 300, 8192), "batch": rng.choice([64, 100, 128, 256, 256, 512]),
                "epochs": rng.randint(1, 5)}
    if kind == "score":
        return {"kind": "score", "n": _log_int(rng, 16, 16384)}
    lattice = rng.choice([19, 19, 19, 27])
    storage = rng.choice(["fp64", "fp32", "fp32", "fp16", "fp16", "bf16"])
    opts = {"lattice": lattice, "storage": storage, "collision": rng.choice(["bgk", "trt", "trt", "reg"]),
            "tau": rng.choice([0.8, 1.0]), "graph": rng.choice([0, 25])}
    shape = rng.choice(["one", "one", "walls", "ensemble", "swim"])
    if shape == "ensemble":
        return flow(nbox=_log_int(rng, 2, 64), edges=rng.randint(200, 9999), **opts)
    if shape == "swim":
        m = rng.randint(2, 7)  # cells of 14 to 24 nodes per edge
        n = int(m * rng.uniform(14.0, 24.0))
        n = min(n, 110)
        return flow(nx=n, ny=n, nz=n, per_box=rng.randint(max(2, m ** 3 // 2), m ** 3), a=5.0, b=2.5, c=2.5, swim=True,
                    **opts)
    n = [_log_int(rng, 24, 110) for _ in range(3)]
    amax = min(12.0, (min(n) - 8) / 2.0)
    b = round(rng.uniform(2.0, min(4.0, amax)), 3)
    a = round(rng.uniform(b, amax), 3)
    return flow(nx=n[0], ny=n[1], nz=n[2], a=a, b=b, c=b, walls=shape == "walls",
                read=rng.choice(["none", "momentum", "fields"]), **opts)


# ------------------------------------------------------------------ inputs --

def _unit(rng, n):
    v = [rng.gauss(0.0, 1.0) for _ in range(n)]
    s = math.sqrt(sum(x * x for x in v))
    return tuple(x / s for x in v)


def _scaled(rng, size):
    return tuple(size * x for x in _unit(rng, 3))


def _boxes(case):
    """Edges of the boxes and of their spheroids, which the case fixes, not the seed."""
    if case["kind"] == "start":
        return [(case["n"],) * 3], [(case["a"], case["b"], case["b"])]
    if case["kind"] == "flow" and case["nbox"] == 1:
        return [(case["nx"], case["ny"], case["nz"])], [(case["a"], case["b"], case["c"])]
    rng = random.Random(case["edges"])
    shapes, axes = [], []
    for _ in range(case["nbox"]):
        n = rng.randint(32, 64)
        while True:  # aspect ratio 1 to 5, eight nodes at least between the images
            r, b = rng.uniform(1.0, 5.0), rng.uniform(2.0, 4.0)
            if n - 2.0 * r * b >= 8.0:
                break
        shapes.append((n, n, n))
        axes.append((r * b, b, b))
    return shapes, axes


def _setup(case, seed):
    """What a run is made of: boxes, particles (box, centre, axes, orientation, force, torque, modes)."""
    rng = random.Random(seed)
    shapes, axes = _boxes(case)
    parts = []
    for i, (s, ax) in enumerate(zip(shapes, axes)):
        if case.get("swim"):
            m = math.ceil(case["per_box"] ** ROOT3 - 1e-9)
            cell = s[0] / m
            slack = max(0.0, min(0.25 * cell, 0.5 * (cell - 2.0 * ax[0] - 2.0)))
            for k in sorted(rng.sample(range(m ** 3), case["per_box"])):
                at = ((k % m + 0.5) * cell, (k // m % m + 0.5) * cell, (k // m // m + 0.5) * cell)
                beta = rng.uniform(-3.0, 3.0)
                parts.append((i, tuple(v + rng.uniform(-slack, slack) for v in at), ax, _unit(rng, 4), (0.0,) * 3,
                              (0.0,) * 3, (1e-3, 1e-3 * beta)))
            continue
        centre = tuple((n - 1) / 2.0 + rng.uniform(-0.5, 0.5) for n in s)
        force, torque = _scaled(rng, rng.uniform(1e-5, 1e-4)), _scaled(rng, rng.uniform(1e-4, 1e-3))
        if case["kind"] == "warm":
            torque = (0.0,) * 3
        if case.get("walls"):  # neutrally buoyant: the shear drives it
            force = torque = (0.0,) * 3
        parts.append((i, centre, ax, _unit(rng, 4), force, torque, (0.0, 0.0)))
    wall = 0.01 if case.get("walls") else 0.0
    return {"shapes": shapes, "parts": parts, "wall": wall, "collision": case.get("collision", "trt"),
            "tau": case.get("tau", 1.0), "lattice": case.get("lattice", 19), "storage": case["storage"],
            "counter": not case.get("walls") and not case.get("swim")}


def _lattice(S):
    w = S["wall"]
    boxes = [make_box(*s, walls=w > 0, wall_lo=(-w, 0, 0), wall_hi=(w, 0, 0), init="couette" if w > 0 else "rest")
             for s in S["shapes"]]
    amax = max(max(p[2]) for p in S["parts"])
    lat = Lattice(boxes, collision=S["collision"], tau=S["tau"], storage=S["storage"], counterforce=S["counter"],
                  velocity_scale=0.01 if w > 0 else 1e-3, max_particles=len(S["parts"]), max_semi_axis=max(8.0, amax),
                  lattice=S["lattice"])
    for box, centre, axes, quat, force, torque, modes in S["parts"]:
        pid = lat.add_ellipsoid(centre, axes, quat, box=box)
        if any(force) or any(torque):
            lat.set_external(pid, force, torque)
        if any(modes):
            lat.set_squirmer(pid, *modes)
    return lat


def _weights(rng):
    """Glorot-uniform weights with small biases, flat: W1, b1, W2, b2, W3, b3."""
    out = []
    for fo, fi in NET:
        lim = math.sqrt(6.0 / (fi + fo))
        out += [rng.uniform(-lim, lim, fo * fi), rng.uniform(-0.1, 0.1, fo)]
    return np.concatenate(out).astype(np.float32)


def _samples(rng, n):
    """Inputs and responses of n loaded spheroids, as the surrogate meets them."""
    X = np.empty((n, 8))
    X[:, 0], X[:, 1] = rng.uniform(0.0, 1.6, n), rng.uniform(0.05, 0.4, n)
    v = rng.normal(size=(n, 6))
    X[:, 2:] = v / np.linalg.norm(v, axis=1, keepdims=True)
    k = 1.0 - 2.0 * X[:, 1:2] * np.exp(-0.5 * X[:, :1])
    Y = k * X[:, 2:] * (1.0 + 0.1 * X[:, :1] * np.array([1.0, -1.0, -1.0, 2.0, -1.0, -1.0]))
    return X.astype(np.float32), Y.astype(np.float32)


def _network(case, seed):
    rng = np.random.default_rng(seed)
    p = _weights(rng)
    return (p,) + (_samples(rng, case["n"]) if "n" in case else ())


# -------------------------------------------------------------------- runs --

def prepare(case, seed):
    state = {"case": case}
    if case["kind"] in ("train", "score"):
        state["p"], state["X"], state["Y"] = _network(case, seed)
        state["net"] = Surrogate(max_samples=case["n"], params=state["p"])
        return state
    state["lat"] = lat = _lattice(_setup(case, seed))
    if case["kind"] == "warm":
        state["net"] = Surrogate(max_samples=case["nbox"], params=_network({}, seed)[0])
        lat.set_graph(case["steps"])
    elif case["kind"] == "flow":
        lat.set_graph(case["graph"])
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "train":
        state["net"].set_params(state["p"])
        loss = state["net"].train(state["X"], state["Y"], case["epochs"], batch=case["batch"], lr=1e-3)
        return {"params": state["net"].params(), "loss": np.float32(loss)}
    if case["kind"] == "score":
        y = state["net"].predict(state["X"])
        loss, g = state["net"].grad(state["X"], state["Y"])
        return {"y": y, "grad": g, "loss": np.float32(loss)}
    lat = state["lat"]
    if case["kind"] == "start":
        lat.stokes_start()
        rho, u = lat.fields(0)
        return {"rho": rho, "u": u}
    if case["kind"] == "warm":
        pred = lat.warm_start(state["net"], tol=0.1)
        lat.step(case["steps"])
        return {"pred": pred, "parts": lat.particles()}
    lat.step(case["steps"])
    try:
        out = {"parts": lat.particles()}
    except LBError as err:  # two swimmers met: the run goes on, as in the suspension studies
        if err.status != OVERLAP:
            raise
        out = {"parts": lat.particles()}
    if lat.np == 1:
        out["F"], out["T"] = lat.force_torque(0)
    if case["read"] == "momentum":
        out["momentum"] = lat.momentum(0)
    elif case["read"] == "fields":
        out["rho"], out["u"] = lat.fields(0)
    return out


def work(case):
    """Populations read and written once per step; every output written once."""
    if case["kind"] in ("train", "score"):
        per = 2.0 * sum(fo * fi for fo, fi in NET)  # a sample's forward products
        n, passes = case["n"], case.get("epochs", 1)
        return {"bytes": 4.0 * (14 * n * passes + 2 * 5126), "flops": per * n * (3 * passes if "epochs" in case else 4)}
    shapes, _ = _boxes(case)
    sites = float(sum(x * y * z for x, y, z in shapes))
    q, s = case.get("lattice", 19), BYTES[case["storage"]]
    if case["kind"] == "start":
        return {"bytes": sites * (2 * q * s + 32), "flops": sites * 400.0}
    steps = case["steps"] + (0.5 if case["kind"] == "warm" else 0)
    out = 32.0 * sites if case.get("read") == "fields" else 0.0
    return {"bytes": 2.0 * q * s * sites * steps + out, "flops": 16.0 * q * sites * steps}


# ------------------------------------------------- the method in 64 bits --

def _velocities(q):
    c = [(0, 0, 0)]
    for k in range(3):
        e = [0, 0, 0]
        e[k] = 1
        c += [tuple(e), tuple(-v for v in e)]
    for v in ((1, 1, 0), (1, -1, 0), (1, 0, 1), (1, 0, -1), (0, 1, 1), (0, 1, -1)) + (
            ((1, 1, 1), (1, 1, -1), (1, -1, 1), (-1, 1, 1)) if q == 27 else ()):
        c += [v, tuple(-x for x in v)]
    by_order = (8 / 27, 2 / 27, 1 / 54, 1 / 216) if q == 27 else (1 / 3, 1 / 18, 1 / 36)
    return c, [by_order[sum(map(abs, v))] for v in c]


def _rot(q):
    w, x, y, z = q.unbind(-1)
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                        2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                        2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], -1).reshape(-1, 3, 3)


def _cross(a, b):
    return torch.linalg.cross(a, b, dim=-1)


class _Box:
    """One box of the method on dense grids [direction, z, y, x], deviations from the rest state."""

    def __init__(self, S, box):
        self.dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
        d = lambda v: torch.tensor(v, dtype=torch.float64, device=self.dev)  # noqa: E731
        nx, ny, nz = S["shapes"][box]
        self.n, self.S, self.tau = (nx, ny, nz), S, S["tau"]
        self.c, self.w = _velocities(S["lattice"])
        self.Q = len(self.c)
        P = [p for p in S["parts"] if p[0] == box]
        self.x, self.ax, self.q, self.fext, self.text, modes = (d([p[k] for p in P]) for k in range(1, 7))
        self.xu, self.nd = self.x.clone(), d([nx, ny, nz])
        self.B1, self.B2 = modes.unbind(-1)
        self.q = self.q / self.q.norm(dim=-1, keepdim=True)
        self.M = 4 / 3 * math.pi * self.ax.prod(-1)
        a2 = self.ax ** 2
        self.Ib = self.M[:, None] / 5 * (a2.sum(-1, keepdim=True) - a2)
        self.U, self.W = torch.zeros_like(self.x), torch.zeros_like(self.x)
        self.dm, self.Pp, self.Lp = torch.zeros_like(self.M), self.U.clone(), self.U.clone()
        self.owner = torch.zeros((nz, ny, nx), dtype=torch.int32, device=self.dev)
        walled = S["wall"] > 0
        if walled:
            self.owner[:, 0] = self.owner[:, -1] = -1
        fluid_sites = nx * ny * nz - (2 * nx * nz if walled else 0)
        self.g = -self.fext.sum(0) / fluid_sites if S["counter"] else torch.zeros_like(self.nd)
        self.f = torch.zeros((self.Q, nz, ny, nx), dtype=torch.float64, device=self.dev)
        if walled:  # Couette profile with its first-order non-equilibrium part
            rate = 2 * S["wall"] / (ny - 2.0)
            u = -S["wall"] + rate * (torch.arange(ny, dtype=torch.float64, device=self.dev) - 0.5)
            for i, (cx, cy, _) in enumerate(self.c):
                row = self.w[i] * (3 * cx * u + 4.5 * (cx * u) ** 2 - 1.5 * u * u - 3 * self.tau * cx * cy * rate)
                self.f[i] = row[None, :, None]
        self.place()
        self.links()

    def image(self, r):
        return torch.where(r >= 0.5 * self.nd, r - self.nd, torch.where(r < -0.5 * self.nd, r + self.nd, r))

    def place(self):
        """The node map at the current pose; returns the map before."""
        r = int(math.ceil(float(self.ax.max()))) + 2
        ar = [torch.arange(min(2 * r + 1, n), device=self.dev) - min(2 * r + 1, n) // 2 for n in self.n]
        off = torch.cartesian_prod(*ar)
        n = self.nd.long()
        new = torch.where(self.owner < 0, self.owner, torch.zeros_like(self.owner))
        for p0 in range(0, len(self.x), 256):
            x = self.x[p0:p0 + 256]
            at = torch.remainder(x.round().long()[:, None] + off, n)
            body = torch.einsum("pij,pki->pkj", _rot(self.q[p0:p0 + 256]), self.image(at - x[:, None]))
            inside = ((body / self.ax[p0:p0 + 256, None]) ** 2).sum(-1) < 1
            k, m = inside.nonzero(as_tuple=True)
            s = at[k, m]
            new.view(-1)[s[:, 0] + n[0] * (s[:, 1] + n[1] * s[:, 2])] = (k + p0 + 1).int()
        old, self.owner = self.owner, new
        self.solid = torch.bincount(new[new > 0].long() - 1, minlength=len(self.x)).double()
        return old

    def links(self):
        site, way, pid = [], [], []
        for b in range(1, self.Q):
            c = self.c[b]
            to = torch.roll(self.owner, (-c[2], -c[1], -c[0]), (0, 1, 2))
            s = ((self.owner == 0) & (to > 0)).view(-1).nonzero()[:, 0]
            site.append(s)
            way.append(torch.full_like(s, b))
            pid.append(to.view(-1)[s].long() - 1)
        self.ls, self.lb, self.lp = torch.cat(site), torch.cat(way), torch.cat(pid)
        cc = torch.tensor(self.c, dtype=torch.float64, device=self.dev)
        self.lc, self.lw = cc[self.lb], torch.tensor(self.w, dtype=torch.float64, device=self.dev)[self.lb]
        nx, ny, _ = self.n
        self.lx = torch.stack([self.ls % nx, self.ls // nx % ny, self.ls // (nx * ny)], -1).double()
        self.lo = torch.tensor([0] + [b + 1 if b % 2 else b - 1 for b in range(1, self.Q)], device=self.dev)[self.lb]

    def collide(self):
        f, c, w, om = self.f, self.c, self.w, 1.0 / self.tau
        d = f.sum(0)
        j = [sum(c[i][k] * f[i] for i in range(self.Q) if c[i][k]) for k in range(3)]
        rho = 1 + d
        u = [v / rho for v in j]
        usq = 1.5 * (u[0] ** 2 + u[1] ** 2 + u[2] ** 2)
        out = torch.empty_like(f)
        dot = lambda i: sum((c[i][k] * u[k] for k in range(3) if c[i][k]), torch.zeros_like(rho))  # noqa: E731
        feq = lambda i, cu: w[i] * (d + rho * (3 * cu + 4.5 * cu * cu - usq))  # noqa: E731
        if self.S["collision"] == "reg":
            tr, X = 0.0, {}
            for a in range(3):
                for b in range(a, 3):
                    pi = sum(c[i][a] * c[i][b] * f[i] for i in range(self.Q) if c[i][a] and c[i][b])
                    ruu = rho * u[a] * u[b]
                    X[a, b] = ruu + (1 - om) * (pi - (d * ROOT3 if a == b else 0) - ruu)
                tr = tr + X[a, a]
            for i in range(self.Q):
                s = sum((c[i][a] * c[i][b] * (1 if a == b else 2) * X[a, b] for a, b in X if c[i][a] and c[i][b]),
                        torch.zeros_like(rho))
                out[i] = w[i] * (d + 3 * rho * dot(i) + 4.5 * (s - tr * ROOT3))
        else:
            omm = 1 / (0.5 + 3.0 / 16.0 / (self.tau - 0.5)) if self.S["collision"] == "trt" else om
            out[0] = f[0] - om * (f[0] - feq(0, torch.zeros_like(rho)))
            for i in range(1, self.Q, 2):
                cu = dot(i)
                e, eo = feq(i, cu), feq(i + 1, -cu)
                a = 0.5 * om * (f[i] + f[i + 1] - e - eo)
                b = 0.5 * omm * (f[i] - f[i + 1] - e + eo)
                out[i], out[i + 1] = f[i] - a - b, f[i + 1] - a + b
        if self.S["counter"]:
            for i in range(1, self.Q):
                out[i] += 3 * w[i] * sum(c[i][k] * self.g[k] for k in range(3))
        return out

    def slip(self, p, r):
        """Tangential surface velocity of the squirmers at the links."""
        e, a, b = _rot(self.q)[:, :, 0][p], self.ax[p, 0], self.ax[p, 1]
        z = (r * e).sum(-1)
        perp = r - z[:, None] * e
        rr = perp.norm(dim=-1)
        zc = torch.minimum(torch.maximum(z, -a), a)
        ecc = torch.sqrt(1 - (b / a) ** 2)
        den = torch.sqrt(a * a - (ecc * zc) ** 2)
        sa, sr = -torch.sqrt(a * a - zc * zc) / den, b / a * zc / den
        zeta = (torch.sqrt(rr ** 2 + (z + a * ecc) ** 2) - torch.sqrt(rr ** 2 + (z - a * ecc) ** 2)) / (2 * a * ecc)
        k = -sa * (self.B1[p] + self.B2[p] * zeta)
        ok = rr > 0
        way = sr[:, None] * perp / torch.where(ok, rr, torch.ones_like(rr))[:, None] + sa[:, None] * e
        return torch.where(ok[:, None], k[:, None] * way, torch.zeros_like(way))

    def step(self):
        n, p, c, c6 = len(self.x), self.lp, self.lc, 6 * self.lw
        post = self.collide()
        fb = post.view(self.Q, -1)[self.lb, self.ls]
        r = self.image(self.lx + 0.5 * c - self.x[p])
        rc = _cross(r, c)
        six = torch.cat([c, rc], -1)  # (c, r x c): the row of a link in the 6 x 6 system
        us = self.slip(p, r) if self.S["parts"][0][6] != (0.0, 0.0) else torch.zeros_like(r)
        kus = c6 * (us * c).sum(-1)
        sums = lambda v: torch.zeros((n,) + v.shape[1:], dtype=torch.float64, device=self.dev).index_add_(0, p, v)  # noqa: E731
        F0 = sums((2 * (fb + self.lw) - kus)[:, None] * six)
        Z = sums(c6[:, None, None] * six[:, :, None] * six[:, None, :])
        R = _rot(self.q)
        I = R @ torch.diag_embed(self.Ib) @ R.mT
        w0, u0, z3 = self.W, self.U, torch.zeros_like(self.W[:, 0])
        Wx = torch.stack([z3, -w0[:, 2], w0[:, 1], w0[:, 2], z3, -w0[:, 0], -w0[:, 1], w0[:, 0], z3], -1).view(-1, 3, 3)
        A = Z.clone()
        A[:, :3, :3] += torch.diag_embed(self.M[:, None].expand(-1, 3))
        A[:, 3:, 3:] += I + Wx @ I - I @ Wx
        pend = torch.cat([self.Pp, self.Lp], -1)
        rhs = F0 + pend
        rhs[:, :3] += self.M[:, None] * u0 + self.fext + self.solid[:, None] * self.g
        rhs[:, 3:] += (I @ w0[:, :, None])[:, :, 0] + self.text
        V = torch.linalg.solve(A, rhs)
        self.FT = F0 + pend - (Z @ V[:, :, None])[:, :, 0]
        self.U, self.W = V[:, :3].contiguous(), V[:, 3:].contiguous()
        wsum = sums(self.lw)
        give = torch.where(wsum > 0, self.dm / wsum, torch.zeros_like(wsum))
        back = fb - c6 * (six * V[p]).sum(-1) - kus + give[p] * self.lw
        for i in range(self.Q):
            cx, cy, cz = self.c[i]
            self.f[i] = torch.roll(post[i], (cz, cy, cx), (0, 1, 2))
            if self.S["wall"] > 0 and cy:
                o = 0 if i == 0 else (i + 1 if i % 2 else i - 1)
                y = 1 if cy > 0 else self.n[1] - 2
                self.f[i][:, y] = post[o][:, y] - 6 * self.w[i] * cx * cy * self.S["wall"]
        self.f.view(self.Q, -1)[self.lo, self.ls] = back
        self.dm, self.Pp, self.Lp = torch.zeros_like(self.dm), torch.zeros_like(u0), torch.zeros_like(u0)
        move = 0.5 * (u0 + self.U)
        self.xu = self.xu + move
        self.x = torch.remainder(self.x + move, self.nd)
        wm = 0.5 * (w0 + self.W)
        h = 0.5 * wm.norm(dim=-1, keepdim=True)
        t = torch.cat([torch.cos(h), 0.5 * wm * torch.sinc(h / math.pi)], -1)
        a, v, b, s = t[:, :1], t[:, 1:], self.q[:, :1], self.q[:, 1:]
        self.q = torch.cat([a * b - (v * s).sum(-1, keepdim=True), a * s + b * v + _cross(v, s)], -1)
        self.remap()

    def remap(self):
        old = self.place()
        if not bool((old != self.owner).any()):
            return
        nx, ny, _ = self.n
        w = torch.tensor(self.w, dtype=torch.float64, device=self.dev)[:, None]
        cc = torch.tensor(self.c, dtype=torch.float64, device=self.dev)
        flat = self.f.view(self.Q, -1)
        for gone in (True, False):  # nodes given back first, then nodes taken
            s = ((old > 0) & (self.owner == 0) if gone else (old == 0) & (self.owner > 0)).view(-1).nonzero()[:, 0]
            p = (old if gone else self.owner).view(-1)[s].long() - 1
            r = self.image(torch.stack([s % nx, s // nx % ny, s // (nx * ny)], -1).double() - self.x[p])
            if gone:
                u = self.U[p] + _cross(self.W[p], r)
                cu = cc @ u.mT
                flat[:, s] = w * (3 * cu + 4.5 * cu * cu - 1.5 * (u * u).sum(-1))
                mom = -u
            else:
                mom = flat[:, s].mT @ cc
                self.dm.index_add_(0, p, flat[:, s].sum(0))
            self.Pp.index_add_(0, p, mom)
            self.Lp.index_add_(0, p, _cross(r, mom))
        self.links()

    def fields(self):
        """(density, velocity, momentum) of the fluid, zero elsewhere as the library reports them."""
        d = self.f.sum(0)
        cc = torch.tensor(self.c, dtype=torch.float64, device=self.dev)
        j = torch.einsum("ik,izyx->zyxk", cc, self.f)
        fluid = (self.owner == 0)
        u = torch.where(fluid[..., None], j / (1 + d)[..., None], torch.zeros_like(j))
        return torch.where(fluid, 1 + d, torch.zeros_like(d)).reshape(-1), u.reshape(-1, 3), j[fluid].sum(0)


def _free_flow(P, mu, d):
    """Velocity and pressure at offsets d (k, 3) of the flow a loaded spheroid drives in unbounded
    fluid: Chwang and Wu's singularities on the focal segment, rigid motion inside."""
    _, _, (a, b, _), quat, F, T, _ = P
    dd = lambda v: torch.tensor(v, dtype=torch.float64, device=d.device)  # noqa: E731
    F, T = dd(F), dd(T)
    p = _rot(dd([quat]) / dd([quat]).norm())[0, :, 0]
    e = math.sqrt(1 - (b / a) ** 2)
    e2, f, lg = e * e, a * e, 2 * math.atanh(e)
    if e < 0.5:
        D = [sum(m(k) * e ** (2 * k + 1) / (4 * k * k - 1) for k in range(1, 40))
             for m in (lambda k: 8.0 * k, lambda k: 8.0 * (k + 1), lambda k: 4.0)]
    else:
        D = [-2 * e + (1 + e2) * lg, 2 * e + (3 * e2 - 1) * lg, 2 * e - (1 - e2) * lg]
    s, t = F / (16 * math.pi * mu * f), T / (8 * math.pi * mu * 4 / 3 * f ** 3)
    sp, tp = (s @ p) * p, (t @ p) * p
    U = sp * D[0] / e2 + (s - sp) * D[1] / (2 * e2)
    W = tp * D[2] / (1 - e2) + (t - tp) * D[0] / (2 - e2)
    m = torch.linalg.cross(t - tp, p)
    z = d @ p
    rho2 = torch.clamp((d * d).sum(-1) - z * z, min=0.0)
    inside = z * z / a ** 2 + rho2 / b ** 2 < 1
    x0 = torch.clamp(z, -f, f)
    delta = torch.sqrt(rho2 + (z - x0) ** 2)
    delta = torch.where(inside, torch.full_like(delta, b), delta)
    nodes, weights = np.polynomial.legendre.leggauss(40)
    out = torch.zeros((len(d), 4), dtype=torch.float64, device=d.device)
    for sgn in (-1.0, 1.0):
        tm = torch.asinh((f - sgn * x0) / delta)
        for xk, wk in zip(nodes, weights):
            th = 0.5 * tm * (xk + 1)
            xi = x0 + sgn * delta * torch.sinh(th)
            wq = (0.5 * wk * tm * delta * torch.cosh(th))[:, None]
            r = d - xi[:, None] * p
            i1 = 1 / r.norm(dim=-1, keepdim=True)
            i3, i5 = i1 ** 3, i1 ** 5
            g = ((f - xi) * (f + xi))[:, None]
            sr, rp, rm = (r @ s)[:, None], (r @ p)[:, None], (r @ m)[:, None]
            k2 = (1 - e2) / (4 * (2 - e2)) * g * g
            st = 3 * e2 / (2 - e2) * g * rp * rm
            v = s * i1 + sr * r * i3 - (1 - e2) / (2 * e2) * g * (3 * sr * r * i5 - s * i3)
            v = v + g * torch.linalg.cross(t.expand_as(r), r) * i3 + st * r * i5
            v = v + k2 * (3 * (m * rp + rm * p) * i5 - 15 * rm * rp * r * i5 * i1 * i1)
            out += wq * torch.cat([v, 2 * mu * (sr * i3 + st * i5)], -1)
    rigid = torch.cat([U + torch.linalg.cross(W.expand_as(d), d), torch.zeros_like(z)[:, None]], -1)
    return torch.where(inside[:, None], rigid, out)


def _start_fields(S):
    """Density and velocity after the start from the periodic creeping flow of one spheroid at rest."""
    B, P = _Box(S, 0), S["parts"][0]
    (nx, ny, nz), mu, dev = B.n, (S["tau"] - 0.5) * ROOT3, B.dev
    ar = [torch.arange(n, dtype=torch.float64, device=dev) for n in B.n]
    zz, yy, xx = torch.meshgrid(ar[2], ar[1], ar[0], indexing="ij")
    pos = torch.stack([xx, yy, zz], -1).reshape(-1, 3)
    d = B.image(pos - B.x[0])
    u = torch.cat([_free_flow(P, mu, v) for v in d.split(1 << 18)])
    (a, b, _), F, T = P[2], B.fext[0], B.text[0]
    Rm = _rot(B.q)[0]
    p = Rm[:, 0]
    e2 = 1 - (b / a) ** 2
    tc = T - (T @ p) * p
    m = torch.linalg.cross(tc, p)
    grid = u.view(nz, ny, nx, 4).permute(3, 0, 1, 2)
    hat = torch.fft.fftn(grid, dim=(1, 2, 3))
    fix = torch.zeros_like(hat)
    V = float(nx * ny * nz)
    for iz in range(-2, 3):
        for iy in range(-2, 3):
            for ix in range(-2, 3):
                if ix == iy == iz == 0:
                    continue
                k = 2 * math.pi * torch.tensor([ix, iy, iz], dtype=torch.float64, device=dev) / B.nd
                k2 = k @ k
                ka = ((Rm.T @ k) * B.ax[0]).norm()
                g = -0.5 * torch.linalg.cross(k, T) + 0.5 * e2 / (2 - e2) * ((k @ m) * p + (k @ p) * m)
                fh = F * torch.sin(ka) / ka - 3j * g * (torch.sin(ka) - ka * torch.cos(ka)) / ka ** 3
                fh = fh * torch.exp(-1j * (k @ B.x[0]))
                kf = (k * fh).sum()
                new = torch.cat([(fh - k * kf / k2) / (mu * k2), (-1j * kf / k2)[None]])
                fix[:, iz, iy, ix] = new - hat[:, iz, iy, ix]
    grid = grid + torch.fft.ifftn(fix, dim=(1, 2, 3)).real
    u = grid.permute(1, 2, 3, 0).reshape(-1, 4)
    fluid = (B.owner == 0).view(-1)
    rho = torch.where(fluid, 1 + 3 * (u[:, 3] - u[fluid, 3].mean()), torch.zeros_like(u[:, 3]))
    v = torch.where(fluid[:, None], u[:, :3], torch.zeros_like(u[:, :3]))
    v = v - fluid[:, None] * (rho[:, None] * v).sum(0) / fluid.sum()
    return {"rho": rho.cpu(), "u": v.cpu()}


def _layers(p):
    out, at = [], 0
    for fo, fi in NET:
        out.append((p[at:at + fo * fi].view(fo, fi), p[at + fo * fi:at + fo * fi + fo]))
        at += fo * fi + fo
    return out


def _forward(p, X):
    (w1, b1), (w2, b2), (w3, b3) = _layers(p)
    return torch.tanh(torch.tanh(X @ w1.T + b1) @ w2.T + b2) @ w3.T + b3


def _loss_grad(p, X, Y):
    p = p.detach().requires_grad_(True)
    loss = ((_forward(p, X) - Y) ** 2).mean()
    return loss.detach(), torch.autograd.grad(loss, p)[0]


def _inputs(S):
    """Network inputs and load scales of the particles, one to a box."""
    X, scale = [], []
    for box, _, ax, q, F, T, _ in S["parts"]:
        R = _rot(torch.tensor([q], dtype=torch.float64))[0]
        req = (ax[0] * ax[1] * ax[2]) ** ROOT3
        Fb, Tb = R.T @ torch.tensor(F, dtype=torch.float64), R.T @ torch.tensor(T, dtype=torch.float64) / req
        s = torch.sqrt(Fb @ Fb + Tb @ Tb)
        n = S["shapes"][box]
        shape = torch.tensor([math.log(ax[0] / math.sqrt(ax[1] * ax[2])), ax[0] / (n[0] * n[1] * n[2]) ** ROOT3],
                             dtype=torch.float64)
        X.append(torch.cat([shape, Fb / s, Tb / s]))
        mu = (S["tau"] - 0.5) * ROOT3
        cu = s / (6 * math.pi * mu * req)
        scale.append(torch.block_diag(cu * R, 0.75 / req * cu * R))
    return torch.stack(X), torch.stack(scale)


def exact(case, seed):
    if case["kind"] in ("train", "score"):
        p, X, Y = (torch.from_numpy(v).double() for v in _network(case, seed))
        if case["kind"] == "score":
            loss, g = _loss_grad(p, X, Y)
            return {"y": _forward(p, X), "grad": g, "loss": loss}
        m, v, t = torch.zeros_like(p), torch.zeros_like(p), 0
        for _ in range(case["epochs"]):
            total = 0.0
            for x, y in zip(X.split(case["batch"]), Y.split(case["batch"])):
                loss, g = _loss_grad(p, x, y)
                total, t = total + loss * len(x), t + 1
                m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
                p = p - 1e-3 * (m / (1 - 0.9 ** t)) / (torch.sqrt(v / (1 - 0.999 ** t)) + 1e-8)
        return {"params": p, "loss": total / len(X)}
    S = _setup(case, seed)
    if case["kind"] == "start":
        return _start_fields(S)
    if case["kind"] == "warm":  # the prediction; the run after it starts from the rounded network's
        X, scale = _inputs(S)
        y = _forward(torch.from_numpy(_network({}, seed)[0]).double(), X)
        return {"pred": (scale @ y[:, :, None])[:, :, 0], "parts": {k: None for k in ("U", "W", "q", "x")}}
    if case["nbox"] * case["steps"] > 700:
        return None
    done = []
    for i in range(case["nbox"]):
        B = _Box(S, i)
        for _ in range(case["steps"]):
            B.step()
        done.append((B.xu, B.q, B.U, B.W, B.FT) + (B.fields() if case["read"] != "none" else ()))
    x, q, U, W, FT = (torch.cat([v[k] for v in done]).cpu() for k in range(5))
    out = {"parts": {"x": x, "q": q, "U": U, "W": W}}
    if len(S["parts"]) == 1:
        out["F"], out["T"] = FT[0, :3], FT[0, 3:]
    if case["read"] == "momentum":
        out["momentum"] = done[0][7].cpu()
    elif case["read"] == "fields":
        out["rho"], out["u"] = done[0][5].cpu(), done[0][6].cpu()
    return out
