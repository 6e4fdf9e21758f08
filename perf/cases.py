"""Workloads of the fiber solver as a user's program runs them, for timing and comparison.

A case is one pass of work through the C ABI's binding: advance a simulation (or a batch
of them) by a number of steps and read the flow and the beads back into host memory that
the program keeps (pinned).  A state keeps its simulation between passes, as a production
run does between two outputs, so a pass goes on from where the last one ended.

Kinds:
  channel     one fiber in a Couette channel (Sec. IV): the 64x32, 1024x256 and 8192x2048
              configurations and sizes between them, even and odd, in every storage format;
  suspension  several fibers in one channel;
  sweep       independent channels of a parameter sweep advanced as one batch;
  shapes      the small channels of the shape diagrams, two batches on two streams;
  particle    periodic boxes with one driven disk each (Sec. III.B), two batches, with the
              drag diagnostics of every disk.
"""
import ctypes
import math

import numpy as np
import torch

import workloads
from paper_2212_14153_amd import _lib, serve

ELEM = {"f64": 8, "f32": 4, "f16dev": 2, "bf16dev": 2}
FLOPS_NODE = 115   # one unforced collision: moments, relaxation, inverse transform


def listed():
    return [
        # the smallest call: one step of the 64x32 parity configuration, state read back
        # (an interactive or coupled program); latency and launches only
        dict(name="tiny_step", kind="channel", nx=64, ny=32, beads=5, radius=2.0, l0=2.0,
             conf=0.0, re=1.0, u=0.01, storage="f64", steps=1, populations=True),
        # an odd-sized small channel, a few hundred steps between outputs
        dict(name="small_odd", kind="channel", nx=777, ny=333, beads=12, radius=0.0, l0=0.0,
             conf=0.4, re=4.0, u=0.0, storage="f32", steps=1000, populations=False),
        # the 1024x256 configuration, 20 beads
        dict(name="medium", kind="channel", nx=1024, ny=256, beads=20, radius=3.0, l0=6.4,
             conf=0.0, re=10.0, u=0.01, storage="f32", steps=1000, populations=False),
        # a mid-sized ragged lattice in the two-byte format
        dict(name="mid_f16", kind="channel", nx=2042, ny=611, beads=16, radius=0.0, l0=0.0,
             conf=0.35, re=5.0, u=0.0, storage="f16dev", steps=1000, populations=False),
        # the 8192x2048 production run with a 40-bead fiber, in three storage formats
        dict(name="large_f32", kind="channel", nx=8192, ny=2048, beads=40, radius=4.0, l0=8.0,
             conf=0.0, re=5.0, u=0.01, storage="f32", steps=1000, populations=False),
        dict(name="large_f64", kind="channel", nx=8192, ny=2048, beads=40, radius=4.0, l0=8.0,
             conf=0.0, re=5.0, u=0.01, storage="f64", steps=500, populations=False),
        dict(name="large_bf16", kind="channel", nx=8192, ny=2048, beads=40, radius=4.0, l0=8.0,
             conf=0.0, re=5.0, u=0.01, storage="bf16dev", steps=1000, populations=False),
        # 25 fibers of 10 beads over the large lattice
        dict(name="suspension", kind="suspension", nx=8192, ny=2048, fibers=25, beads=10,
             radius=4.0, re=5.0, storage="f32", steps=500),
        # a parameter sweep of 64 channels (128x64 to 1024x512) advanced together, and the
        # same in the format the serving runs use
        dict(name="sweep_f32", kind="sweep", sims=64, draw_seed=14153, storage="f32",
             steps=1000),
        dict(name="sweep_f16", kind="sweep", sims=64, draw_seed=14153, storage="f16dev",
             steps=1000),
        # 85 small channels (200 x 92 .. 400) of the shape diagrams, 10 beads each
        dict(name="shapes", kind="shapes", sims=85, draw_seed=7, storage="f32", steps=2000),
        # the driven-particle sweep: 64 periodic 200x200 boxes
        dict(name="particle", kind="particle", sims=64, n=200, storage="f32", steps=2000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    storage = rng.choice(["f32", "f32", "f64", "f16dev", "bf16dev"])
    budget = 1.2e9 if storage != "f64" else 0.6e9      # node updates of a pass
    kind = rng.choice(["channel"] * 5 + ["suspension", "sweep", "shapes", "particle"])
    if kind == "channel":
        ny = _log_int(rng, 64, 2048)
        nx = min(8192, int(ny * rng.uniform(2.0, 4.0)))
        steps = max(1, min(1000, int(budget * 10 ** rng.uniform(-1.5, 0.0) / (nx * ny))))
        beads = rng.randint(5, 40)
        conf = rng.uniform(0.2, 0.6)
        while conf * ny / beads < 4.0:                 # bead radius at least 2 nodes
            beads = rng.randint(5, 40) if beads > 12 else beads - 1
        return dict(kind=kind, nx=nx, ny=ny, beads=beads, radius=0.0, l0=0.0,
                    conf=round(conf, 3), re=round(rng.uniform(1.0, 10.0), 2), u=0.0,
                    storage=storage, steps=steps, populations=False)
    if kind == "suspension":
        ny = _log_int(rng, 512, 2048)
        nx = min(8192, int(ny * rng.uniform(2.0, 4.0)))
        fibers = max(2, int(25 * nx * ny / (8192 * 2048) * rng.uniform(0.6, 1.0)))
        return dict(kind=kind, nx=nx, ny=ny, fibers=fibers, beads=rng.randint(6, 10),
                    radius=round(rng.uniform(3.0, 4.0), 2), re=round(rng.uniform(1.0, 8.0), 2),
                    storage=storage, steps=max(1, min(300, int(budget / (nx * ny)))))
    if kind == "sweep":
        return dict(kind=kind, sims=rng.randint(8, 64), draw_seed=rng.randint(1, 10 ** 6),
                    storage=storage, steps=rng.randint(100, 500))
    if kind == "shapes":
        return dict(kind=kind, sims=rng.randint(16, 85), draw_seed=rng.randint(1, 10 ** 6),
                    storage=storage, steps=rng.randint(200, 2000))
    return dict(kind="particle", sims=rng.randint(8, 64), n=rng.randint(96, 240),
                storage=storage, steps=rng.randint(200, 1500))


# ------------------------------------------------------------------ the simulations ----

def _channel(case, rng):
    nx, ny, n = case["nx"], case["ny"], case["beads"]
    l0 = case["l0"] or case["conf"] * ny / n
    radius = case["radius"] or l0 / 2.0
    lc = n * l0
    u = case["u"] or min(max(case["re"] / (15.0 * (lc / ny) ** 2 * ny), 1e-3), 0.05)
    m = workloads.physical_to_lattice(nx=nx, ny=ny, n_beads=n, radius=radius, l0=l0, u_wall=u,
                                      re_ps=case["re"], kappa=10.0 ** rng.uniform(-1.0, 1.0))
    return workloads.Workload(
        name="channel", nx=nx, ny=ny, u_wall=u, nu_f=m["nu_f"], eta_ratio=50.0, xi=1.0,
        n_beads=n, radius=radius, l0=l0, k_s=m["k_s"], k_b=m["k_b"],
        theta0=rng.uniform(0.3, 1.2), cx=nx * rng.uniform(0.1, 0.9),
        cy=ny * rng.uniform(0.49, 0.51), steps=0, storage=case["storage"])


def _suspension(case, seed):
    return workloads.fiber_suspension(
        n_fibers=case["fibers"], beads=case["beads"], nx=case["nx"], ny=case["ny"],
        radius=case["radius"], re_ps=case["re"], kappa=3.3, u_wall=0.01,
        storage=case["storage"], seed=4447 + seed)


def _sims(case, seed):
    """The independent simulations of a batched case: sizes from the case, starts from the
    seed."""
    rng = np.random.default_rng(seed)
    st, n = case["storage"], case["sims"]
    if case["kind"] == "sweep":
        ws = workloads.sweep_sims(n, seed=case["draw_seed"], storage=st)
        return [w.with_(theta0=rng.uniform(0.4, 1.1), cx=w.nx * rng.uniform(0.2, 0.8))
                for w in ws]
    if case["kind"] == "shapes":
        pick = np.random.default_rng(case["draw_seed"])
        pts = [(10.0 ** pick.uniform(-4.5, 1.5), pick.choice([0.2, 0.3, 0.5, 0.6, 0.7, 0.8,
                                                              0.87]),
                pick.choice([0.5, 1.5, 3.0, 4.5, 6.0])) for _ in range(n)]
        return [workloads.flexible_fiber(float(k), float(c), float(r), storage=st,
                                         theta0=rng.uniform(-0.05, 0.05))
                for k, c, r in pts]
    return [workloads.driven_particle(n=case["n"], radius=case["n"] / 20.0, xi=2.5,
                                      force=float(f), storage=st,
                                      offset=tuple(rng.uniform(-0.5, 0.5, 2)))
            for f in np.geomspace(1e-4, 1e-1, n)]


def _sizes(case):
    if case["kind"] in ("channel", "suspension"):
        return [(case["nx"], case["ny"])]
    return [(w.nx, w.ny) for w in _sims(case, 0)]


# ------------------------------------------------------------------------- a pass ------

def _host(shape):
    return torch.empty(shape, dtype=torch.float64, pin_memory=True).numpy()


def _ptr(a):
    return a.ctypes.data_as(ctypes.POINTER(ctypes.c_double))


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    if case["kind"] in ("channel", "suspension"):
        w = (_channel(case, rng) if case["kind"] == "channel"
             else _suspension(case, seed % 100000))
        sim = _lib.simulation_from_workload(w, storage=case["storage"])
        planes = 9 if case.get("populations") else 4
        return dict(case=case, sim=sim, out=_host((planes, w.ny, w.nx)))
    ws = _sims(case, seed)
    params = [_lib.params_from_mapping(w.params(), storage=case["storage"]) for w in ws]
    budget = sum(_lib.fpd_sim_footprint(p) for p in params) + (1 << 26)
    lanes = 1 if case["kind"] == "sweep" and case["storage"] in ("f32", "f64") else 2
    batches = [_lib.Batch(budget, len(ws), storage=case["storage"]) for _ in range(lanes)]
    placed = [(batches[i % lanes], batches[i % lanes].add(p, w.beads(), 1 << 40))
              for i, (p, w) in enumerate(zip(params, ws))]
    return dict(case=case, batches=batches, placed=placed, ws=ws,
                out=_host((4, sum(w.nx * w.ny for w in ws))))


def run(state):
    case, out = state["case"], state["out"]
    if "sim" in state:
        sim = state["sim"]
        sim.step(case["steps"])
        if case.get("populations"):
            _lib.check(_lib.lib().fpd_read_populations(sim.h, _ptr(out)))
        else:
            _lib.check(_lib.lib().fpd_read_fields(sim.h, *[_ptr(out[i]) for i in range(4)]))
        R, V, _ = sim.beads()
        if case.get("populations"):
            return dict(f=out, R=R, V=V)
        return dict(rho=out[0], u=out[1:3], eta=out[3], R=R, V=V)
    serve.run_batches(state["batches"], case["steps"])
    at, beads = 0, []
    for (b, sid), w in zip(state["placed"], state["ws"]):
        n = w.nx * w.ny
        _lib.check(_lib.lib().fpd_batch_read_fields(
            b.h, sid, *[_ptr(out[i, at:at + n]) for i in range(4)]))
        beads.append(b.beads(sid)[:2])
        at += n
    got = dict(rho=out[0], u=out[1:3], eta=out[3], R=np.concatenate([r for r, _ in beads]),
               V=np.concatenate([v for _, v in beads]))
    if case["kind"] == "particle":
        stats = [b.particle_stats(sid) for b, sid in state["placed"]]
        got["drag"] = np.array([[s["Fvisc_x"] + s["Fpres_x"], s["V0x"]] for s in stats])
    return got


def work(case):
    """The populations read and written once, the outputs written once; the collisions."""
    nodes = sum(nx * ny for nx, ny in _sizes(case))
    planes = 9 if case.get("populations") else 4
    return {"bytes": nodes * (18.0 * ELEM[case["storage"]] + 8.0 * planes),
            "flops": float(FLOPS_NODE) * nodes * case["steps"]}


# ------------------------------------------------------- the method in 64-bit torch -----

_EX = (0, 1, 0, -1, 0, 1, -1, -1, 1)
_EY = (0, 0, 1, 0, -1, 1, 1, -1, -1)
_W = (4 / 9,) + (1 / 9,) * 4 + (1 / 36,) * 4


class _Exact:
    """The time step of Sec. II.C on dense 64-bit arrays (pre-collision populations)."""

    def __init__(self, w, dev):
        self.w, self.dev = w, dev
        self.per = w.boundary == 1
        nx, ny = w.nx, w.ny
        d = dict(dtype=torch.float64, device=dev)
        ux = torch.zeros(ny, 1, **d)
        if w.init_flow == 1:
            ux = (w.u_wall * (2.0 * (torch.arange(ny, **d) + 0.5) / ny - 1.0)).reshape(ny, 1)
        self.f = torch.empty(9, ny, nx, **d)
        for k in range(9):
            eu = _EX[k] * ux
            self.f[k] = _W[k] * (1.0 + 3.0 * eu + 4.5 * eu * eu - 1.5 * ux * ux)
        self.R = torch.tensor(w.beads(), **d)
        self.V = torch.zeros_like(self.R)
        self.rc = w.radius + 20.0 * w.xi
        half = int(math.ceil(self.rc)) + 1
        o = torch.arange(-half, half + 1, device=dev)
        self.ox, self.oy = o.reshape(1, 1, -1), o.reshape(1, -1, 1)
        self.once = min(nx, ny if self.per else nx) > 2 * half + 1

    def phi(self):
        """Per bead and box node: flat node index and phi (0 outside the channel)."""
        w, nx, ny = self.w, self.w.nx, self.w.ny
        c = torch.floor(self.R).long()
        x = c[:, :1, None] + self.ox
        y = c[:, 1:, None] + self.oy
        dx = x.double() + 0.5 - self.R[:, :1, None]
        dy = y.double() + 0.5 - self.R[:, 1:, None]
        r = torch.sqrt(dx * dx + dy * dy)
        ph = 0.5 * (torch.tanh((w.radius - r) / w.xi) + 1.0)
        ok = r < self.rc
        if not self.once:     # a box wider than the lattice: the nearest image only
            ok = ok & (2 * dx < nx) & (2 * dx >= -nx)
            if self.per:
                ok = ok & (2 * dy < ny) & (2 * dy >= -ny)
        yy = y % ny if self.per else y.clamp(0, ny - 1)
        if not self.per:
            ok = ok & (y >= 0) & (y < ny)
        return (yy * nx + x % nx).expand_as(ph), torch.where(ok, ph, torch.zeros_like(ph))

    def forces(self):
        w, R = self.w, self.R
        chains = max(w.n_chains, 1)
        X = R.reshape(chains, -1, 2)
        F = torch.zeros_like(X)
        if X.shape[1] > 1:
            d = X[:, 1:] - X[:, :-1]
            L = torch.sqrt((d * d).sum(-1, keepdim=True))
            t = d / L
            s = w.k_s / w.l0 ** 2 * (L - w.l0) * t
            F[:, :-1] += s
            F[:, 1:] -= s
            if X.shape[1] > 2:
                a, b = t[:, :-1], t[:, 1:]
                dot = (a * b).sum(-1, keepdim=True)
                ga = w.k_b * (b - dot * a) / L[:, :-1]
                gb = w.k_b * (a - dot * b) / L[:, 1:]
                F[:, :-2] -= ga
                F[:, 1:-1] += ga - gb
                F[:, 2:] += gb
        return F.reshape(-1, 2) + torch.tensor(w.f_ext, dtype=torch.float64, device=self.dev)

    def spread(self):
        w = self.w
        idx, ph = self.phi()
        A = ph.sum((1, 2))
        C = self.forces() / A[:, None]
        out = torch.zeros(3, w.ny * w.nx, dtype=torch.float64, device=self.dev)
        flat = idx.reshape(-1)
        out[0].index_add_(0, flat, ph.reshape(-1))
        out[1].index_add_(0, flat, (ph * C[:, :1, None]).reshape(-1))
        out[2].index_add_(0, flat, (ph * C[:, 1:, None]).reshape(-1))
        sphi, fx, fy = out.reshape(3, w.ny, w.nx)
        return idx, ph, A, sphi, fx + w.g_body[0], fy + w.g_body[1]

    def moments(self, f):
        rho = f.sum(0)
        jx = f[1] - f[3] + f[5] - f[6] - f[7] + f[8]
        jy = f[2] - f[4] + f[5] + f[6] - f[7] - f[8]
        return rho, jx, jy

    def step(self):
        w, f = self.w, self.f
        idx, ph, A, sphi, fx, fy = self.spread()
        eta = w.nu_f * (1.0 + (w.eta_ratio - 1.0) * sphi)
        s_nu = 1.0 / (3.0 * eta + 0.5)
        s_q = 8.0 * (2.0 - s_nu) / (8.0 - s_nu)
        rho, jx, jy = self.moments(f)
        ux, uy = (jx + 0.5 * fx) / rho, (jy + 0.5 * fy) / rho
        s1, s2 = f[1] + f[2] + f[3] + f[4], f[5] + f[6] + f[7] + f[8]
        u2, uf = rho * (ux * ux + uy * uy), ux * fx + uy * fy
        e = -4.0 * f[0] - s1 + 2.0 * s2
        e = e - w.s_e * (e - (-2.0 * rho + 3.0 * u2)) + (1 - 0.5 * w.s_e) * 6.0 * uf
        p = 4.0 * f[0] - 2.0 * s1 + s2
        p = p - w.s_eps * (p - (rho - 3.0 * u2)) - (1 - 0.5 * w.s_eps) * 6.0 * uf
        qx = -2.0 * (f[1] - f[3]) + f[5] - f[6] - f[7] + f[8]
        qx = qx - s_q * (qx + rho * ux) - (1 - 0.5 * s_q) * fx
        qy = -2.0 * (f[2] - f[4]) + f[5] + f[6] - f[7] - f[8]
        qy = qy - s_q * (qy + rho * uy) - (1 - 0.5 * s_q) * fy
        hn = 1 - 0.5 * s_nu
        xx = f[1] - f[2] + f[3] - f[4]
        xx = xx - s_nu * (xx - rho * (ux * ux - uy * uy)) + hn * 2.0 * (ux * fx - uy * fy)
        xy = f[5] - f[6] + f[7] - f[8]
        xy = xy - s_nu * (xy - rho * ux * uy) + hn * (ux * fy + uy * fx)
        jx, jy = jx + fx, jy + fy
        g = torch.empty_like(f)
        g[0] = rho / 9 - e / 9 + p / 9
        ax, dg = rho / 9 - e / 36 - p / 18, rho / 9 + e / 18 + p / 36
        g[1] = ax + jx / 6 - qx / 6 + xx / 4
        g[3] = ax - jx / 6 + qx / 6 + xx / 4
        g[2] = ax + jy / 6 - qy / 6 - xx / 4
        g[4] = ax - jy / 6 + qy / 6 - xx / 4
        a, b = jx / 6 + qx / 12, jy / 6 + qy / 12
        g[5] = dg + a + b + xy / 4
        g[6] = dg - a + b - xy / 4
        g[7] = dg - a - b + xy / 4
        g[8] = dg + a - b - xy / 4
        for k in range(9):
            f[k] = torch.roll(g[k], (_EY[k], _EX[k]), (0, 1))
        if not self.per:      # half-way bounce-back at the walls moving at -U and +U
            u6 = w.u_wall / 6.0
            f[2, 0], f[5, 0], f[6, 0] = g[4, 0], g[7, 0] - u6, g[8, 0] + u6
            f[4, -1], f[7, -1], f[8, -1] = g[2, -1], g[5, -1] - u6, g[6, -1] + u6
        # Eq. (5) with the populations of the new step and the force of the old one
        rho, jx, jy = self.moments(f)
        vx = ((jx + 0.5 * fx) / rho).reshape(-1)[idx]
        vy = ((jy + 0.5 * fy) / rho).reshape(-1)[idx]
        self.V = torch.stack([(ph * vx).sum((1, 2)) / A, (ph * vy).sum((1, 2)) / A], 1)
        self.R = self.R + self.V

    def outputs(self, populations):
        got = dict(R=self.R, V=self.V)
        if populations:
            got["f"] = self.f
        else:
            _, _, _, sphi, fx, fy = self.spread()
            rho, jx, jy = self.moments(self.f)
            got.update(rho=rho, u=torch.stack([(jx + 0.5 * fx) / rho, (jy + 0.5 * fy) / rho]),
                       eta=self.w.nu_f * (1.0 + (self.w.eta_ratio - 1.0) * sphi))
        return {k: v.cpu().numpy() for k, v in got.items()}


def exact(case, seed):
    """What run() returns for these inputs, in 64-bit torch; None for the batches, whose
    simulations of different sizes would take too long one after the other."""
    if case["kind"] not in ("channel", "suspension"):
        return None
    if case["nx"] * case["ny"] * case["steps"] > 2e10:
        return None
    rng = np.random.default_rng(seed)
    w = (_channel(case, rng) if case["kind"] == "channel"
         else _suspension(case, seed % 100000))
    x = _Exact(w, torch.device("cuda" if torch.cuda.is_available() else "cpu"))
    for _ in range(case["steps"]):
        x.step()
    return x.outputs(bool(case.get("populations")))
