"""The work that users of this framework have it do, as cases that can be timed.

A case is one pass of a user's program through the public entry points of
paper_2608_26908_amd.gpf: a monitored forward run (so many coupled steps, then
the fields that a program writes out), or one evaluation of a loss gradient
(forward run and reverse sweep).  `listed` holds the workloads of this
repository's configurations at sizes from a few thousand cells to 256^3, `draw`
more of the same ranges.

`exact` is the same step in plain torch, in 64 bits and without the library:
the discrete equations as they are stated in include/gpf.h, its derivatives by
torch's automatic differentiation.
"""
import math

import numpy as np
import torch

from paper_2608_26908_amd.workloads import scaled

PARAMS = {"inverse2d": ["delta", "tau_pf", "D", "gbeta"], "inverse3d": ["D", "D1", "tau_pf"]}


def listed():
    F, R = dict(kind="forward"), dict(periodic_x=False, lattice="", eta=0.0, frame=0, restart=False, totals=False)

    def forward(name, workload, n, precision, steps, **kw):
        nx, ny, nz = (list(n) + [1])[:3]
        return dict(F, name=name, workload=workload, nx=nx, ny=ny, nz=nz, precision=precision, steps=steps,
                    **{**R, **kw})

    def inverse(name, kind, workload, n, precision, steps, every):
        nx, ny, nz = (list(n) + [1])[:3]
        return dict(kind=kind, name=name, workload=workload, nx=nx, ny=ny, nz=nz, precision=precision, steps=steps,
                    every=every)

    return [
        # the smallest calls: a parameter study's tiny 2D dendrite, looked at every few steps
        forward("dendrite2d_tiny", "dendrite2d", [48, 40], "fp32", 10),
        # the 2D dendrite of the configurations (128^2, FP64), with its conserved totals
        forward("dendrite2d", "dendrite2d", [128, 128], "fp64", 200, totals=True),
        # the directionally solidified binary eutectic at its configured size
        forward("eutectic2d", "eutectic2d", [1024, 512], "fp32", 50),
        # the four-phase eutectic in 2D, moving frame on (a front search every 25 steps)
        forward("eutectic4_frame", "eutectic4", [144, 700], "fp32", 50, frame=25),
        # the benchmark's workload at full size: 256^3, D3Q19, FP32
        forward("dendrite3d", "dendrite3d", [256, 256, 256], "fp32", 10),
        # a small 3D dendrite, as in a parameter study
        forward("dendrite3d_small", "dendrite3d", [64, 64, 64], "fp32", 25),
        # an odd box in FP64 whose whole state is taken out for a restart file
        forward("dendrite3d_restart", "dendrite3d", [150, 131, 117], "fp64", 10, restart=True, totals=True),
        # the 27-velocity lattice and the shrinkage force, on an odd box
        forward("dendrite3d_q27_shrink", "dendrite3d", [129, 160, 96], "fp32", 10, lattice="D3Q27", eta=0.2),
        # ternary eutectic with convection, half the configured height
        forward("eutectic3d", "eutectic3d", [192, 192, 192], "fp32", 10),
        # four phases in 3D
        forward("eutectic4_3d", "eutectic4_3d", [96, 96, 128], "fp32", 10),
        # parameter inversion on the 2D dendrite: one loss gradient through torch.autograd
        inverse("inverse2d", "inverse2d", "adjoint2d", [256, 256], "fp32", 100, 25),
        # gradient with respect to the diffusivities over a window of the 3D ternary eutectic
        inverse("inverse3d", "inverse3d", "eutectic3d", [96, 96, 96], "fp32", 30, 10),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["dendrite2d", "eutectic2d", "dendrite3d", "dendrite3d", "eutectic3d", "inverse2d", "inverse3d"])
    precision = rng.choice(["fp32", "fp32", "fp64"])
    if kind == "inverse2d":
        n = [size(40, 256), size(40, 256), 1]
        return dict(kind=kind, workload="adjoint2d", nx=n[0], ny=n[1], nz=n[2], precision=precision,
                    steps=size(20, 100), every=rng.choice([10, 20, 25]))
    if kind == "inverse3d":
        n = [size(24, 96), size(24, 96), size(40, 96)]
        return dict(kind=kind, workload="eutectic3d", nx=n[0], ny=n[1], nz=n[2], precision=precision,
                    steps=size(8, 30), every=rng.choice([4, 8, 10]))
    case = dict(kind="forward", periodic_x=rng.random() < 0.3, lattice="", eta=0.0, frame=0,
                restart=rng.random() < 0.25, totals=precision == "fp64" and rng.random() < 0.5, precision=precision)
    if kind == "dendrite2d":
        case.update(workload="dendrite2d", nx=size(32, 1024), ny=size(32, 1024), nz=1, steps=size(5, 200))
    elif kind == "eutectic2d":
        case.update(workload=rng.choice(["eutectic2d", "eutectic4"]), nx=size(64, 1024), ny=size(64, 700), nz=1,
                    steps=size(10, 100), frame=rng.choice([0, 0, 25]))
    elif kind == "dendrite3d":
        case.update(workload="dendrite3d", nx=size(40, 256), ny=size(40, 256), nz=size(40, 256), steps=size(4, 25),
                    lattice=rng.choice(["", "", "D3Q27"]), eta=rng.choice([0.0, 0.0, 0.2]))
    else:
        case.update(workload=rng.choice(["eutectic3d", "eutectic4_3d"]), nx=size(40, 192), ny=size(40, 192),
                    nz=size(48, 384), steps=size(4, 20))
    # no more than the largest listed case: halve the height, then the steps
    while work(case)["bytes"] > 0.5 * work(listed()[4])["bytes"]:
        if case["nz"] > 96:
            case["nz"] = case["nz"] // 2 + 1
        else:
            case["steps"] = max(1, case["steps"] // 2)
    return case


# ---------------------------------------------------------------------------
# the case as the framework takes it
# ---------------------------------------------------------------------------
def _config(case):
    two = case["nz"] == 1
    n = [case["nx"], case["ny"]] + ([] if two else [case["nz"]])
    kw = {}
    if case.get("periodic_x") and case["workload"].startswith("dendrite"):
        kw["periodic"] = [1, 0] if two else [1, 0, 0]
    if case.get("lattice"):
        kw["lattice"] = case["lattice"]
    if case.get("eta"):
        kw["eta"] = [case["eta"], 0.0, 0.0]
    if case.get("frame"):
        kw.update(frame_every=case["frame"], frame_front=24)
    return scaled(case["workload"], n, **kw)


def _fields(case):
    # what a program writes out; a restart file needs the populations too
    return ["phi", "mu", "u"] + (["f"] if case.get("restart") else [])


def _target(cfg, dtype):
    """The microstructure to be matched: a round (2D) or flat (3D) solid that has grown further than the initial one."""
    n = cfg["n"]
    ax = [torch.arange(v, dtype=torch.float64, device="cuda") for v in reversed(n)]
    grid = list(reversed(torch.meshgrid(*ax, indexing="ij")))
    target = torch.zeros([cfg["N"]] + list(reversed(n)), dtype=torch.float64, device="cuda")
    if cfg["init"] == "seed":
        r = torch.sqrt(sum((g - c) ** 2 for g, c in zip(grid, cfg["init_center"])))
        solid = torch.clamp((cfg["init_radius"] + 6.0 - r) / 4.0 + 0.5, 0.0, 1.0)
        target[0] = solid
    else:
        solid = torch.clamp((cfg["lam_height"] + 6.0 - grid[cfg["pull_axis"]]) / 4.0 + 0.5, 0.0, 1.0)
        which = torch.floor(grid[0] / cfg["lam_width"]) % (cfg["N"] - 1)
        for s in range(cfg["N"] - 1):
            target[s] = torch.where(which == s, solid, torch.zeros_like(solid))
    target[-1] = 1.0 - solid
    return target.to(dtype)


def _start_values(cfg, names):
    solute = cfg["D"][cfg["N"] - 1]
    pair = max(max(row) for row in cfg["delta"])
    at = dict(delta=pair, tau_pf=cfg["tau_pf"], D=solute[0], D1=solute[-1], gbeta=cfg["gbeta"][0])
    return [at[k] for k in names]


def prepare(case, seed):
    from paper_2608_26908_amd.gpf import Sim
    cfg = _config(case)
    sim = Sim(cfg, precision=case["precision"], seed=seed)
    state = dict(sim=sim, kind=case["kind"], steps=case["steps"])
    if case["kind"] == "forward":
        state.update(fields=_fields(case), totals=bool(case.get("totals")))
        return state
    dtype = torch.float64 if case["precision"] == "fp64" else torch.float32
    names = PARAMS[case["kind"]]
    state.update(names=names, every=case["every"], target=_target(cfg, dtype), dtype=dtype)
    if case["kind"] == "inverse2d":
        # an inversion starts every run from the same initial state
        state.update(initial=sim.checkpoint(), values=_start_values(cfg, names))
    else:
        sim.set_target(state["target"])
    return state


def run(state):
    sim = state["sim"]
    if state["kind"] == "forward":
        sim.step(state["steps"])
        out = {k: sim.read_device(k) for k in state["fields"]}
        if state["totals"]:
            out["solute"], out["mass"] = sim.reduce("solute"), sim.reduce("mass")
        return out
    if state["kind"] == "inverse2d":
        from paper_2608_26908_amd.gpf import gpf_run
        params = torch.tensor(state["values"], dtype=state["dtype"], requires_grad=True)
        phi = gpf_run(params, sim, state["initial"], state["names"], state["steps"], state["every"])
        loss = 0.5 * ((phi - state["target"]) ** 2).sum()
        loss.backward()
        return {"phi": phi.detach(), "grad": params.grad}
    # the sensitivity of the next window of a run, which goes on from where it is
    sim.record(state["every"])
    sim.step(state["steps"])
    grad = sim.adjoint(sim.loss_seed(), state["names"])
    return {"phi": sim.read_device("phi"), "grad": torch.tensor(grad, dtype=state["dtype"])}


def work(case):
    cfg = _config(case)
    s = 8 if case["precision"] == "fp64" else 4
    cells = case["nx"] * case["ny"] * case["nz"]
    D, N, nc = cfg["dim"], cfg["N"], cfg["nc"]
    Q = 9 if D == 2 else (27 if case.get("lattice") == "D3Q27" else 19)
    state = (N - 1) + nc + Q  # sum phi = 1; U follows from f
    # per cell and step: collision and streaming, the chemical potentials' face fluxes
    flops = 20.0 * Q + 2 * D * (10 * nc * N) + 30
    if case["kind"] == "forward":
        out = N + nc + D + (Q if case["restart"] else 0)
        return {"bytes": float(s) * cells * (2 * state * case["steps"] + 2 * out), "flops": flops * cells * case["steps"]}
    # a gradient: the run, and per reverse step the states read again and the adjoint state read and written
    return {"bytes": float(s) * cells * case["steps"] * (2 * state + state + 2 * state), "flops": 4 * flops * cells * case["steps"]}


# ---------------------------------------------------------------------------
# the same in plain torch, 64 bits
# ---------------------------------------------------------------------------
def _lattice(Q):
    if Q == 9:
        c = [(0, 0), (1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1)]
        w = [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4
    else:
        c = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1, 0), (-1, -1, 0),
             (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1), (-1, 0, 1), (0, 1, 1), (0, -1, -1),
             (0, 1, -1), (0, -1, 1)]
        w = [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12
        if Q == 27:
            c += [(1, 1, 1), (-1, -1, -1), (1, 1, -1), (-1, -1, 1), (1, -1, 1), (-1, 1, -1), (-1, 1, 1), (1, -1, -1)]
            w = [8 / 27] + [2 / 27] * 6 + [1 / 54] * 12 + [1 / 216] * 8
    return c, w


class _Exact:
    """The coupled step on float64 tensors [component, (z,) y, x]; phi, mu, u and the streamed populations f as
    deviations from w_k rho0."""

    def __init__(self, cfg, seed, precision):
        self.cfg, self.D, self.N, self.nc = cfg, cfg["dim"], cfg["N"], cfg["nc"]
        self.per = [bool(v) for v in cfg["periodic"]]
        self.Q = 9 if self.D == 2 else (27 if cfg.get("lattice") == "D3Q27" else 19)
        self.c, self.w = _lattice(self.Q)
        self.opp = [self.c.index(tuple(-v for v in c)) for c in self.c]
        self.qmin2 = 1e-24 if precision == "fp64" else 1e-12
        self.n = list(cfg["n"][: self.D])
        self.shape = list(reversed(self.n))
        self.step_index, self.offset = 0, 0
        self.p = dict(delta=None, tau_pf=cfg["tau_pf"], D=cfg["D"][self.N - 1][0], D1=cfg["D"][self.N - 1][self.nc - 1],
                      gbeta=cfg["gbeta"][0])
        self.coord = [torch.arange(n, dtype=torch.float64, device="cuda").reshape([-1] + [1] * a)
                      for a, n in enumerate(self.n)]  # broadcasts along tensor dimension -1 - a
        phi, mu = self._initial(seed)
        zero = lambda k: torch.zeros([k] + self.shape, dtype=torch.float64, device="cuda")  # noqa: E731
        self.state = (phi, mu, zero(self.D), zero(self.Q))

    def _initial(self, seed):
        cfg = self.cfg
        if cfg["init"] == "seed":
            s = torch.sqrt(sum((x - c) ** 2 for x, c in zip(self.coord, cfg["init_center"]))) - cfg["init_radius"]
            which = torch.zeros(self.shape, dtype=torch.float64, device="cuda")
        else:
            s = self.coord[cfg["pull_axis"]] - cfg["lam_height"]
            which = torch.floor(self.coord[0] / cfg["lam_width"]) % (self.N - 1)
        half = math.pi ** 2 * cfg["eps"] / 8
        s = (s * cfg["dx"]).expand(self.shape)
        solid = 0.5 - 0.5 * torch.sin(4.0 * s.clamp(-half, half) / (math.pi * cfg["eps"]))
        solid = torch.where(s <= -half, torch.ones_like(s), torch.where(s >= half, torch.zeros_like(s), solid))
        phi = torch.zeros([self.N] + self.shape, dtype=torch.float64, device="cuda")
        for a in range(self.N - 1):
            phi[a] = torch.where(which.expand(self.shape) == a, solid, torch.zeros_like(solid))
        phi[-1] = 1.0 - solid
        # SplitMix64 keyed by the seed, counters 2j and 2j + 1, Box-Muller; j = cell nc + i
        cells = int(np.prod(self.n))
        with np.errstate(over="ignore"):
            def bits(j):
                z = np.uint64(seed) + (j + np.uint64(1)) * np.uint64(0x9E3779B97F4A7C15)
                z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
                z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
                return torch.from_numpy(((z ^ (z >> np.uint64(31))) >> np.uint64(11)).astype(np.float64)).cuda()

            j = np.arange(cells * self.nc, dtype=np.uint64) * np.uint64(2)
            u1, u2 = (bits(j) + 1.0) * 2.0 ** -53, bits(j + np.uint64(1)) * 2.0 ** -53
        z = torch.sqrt(-2.0 * torch.log(u1)) * torch.cos(2.0 * math.pi * u2)
        z = z.reshape(self.shape + [self.nc])
        mu = torch.stack([cfg["mu_inf"][i] + cfg["noise_sigma"] * z[..., i] for i in range(self.nc)])
        return phi, mu

    def nb(self, v, a, s):
        """v at the neighbour s = +-1 along axis a; walls repeat the cell."""
        d = v.dim() - 1 - a
        if self.per[a]:
            return torch.roll(v, -s, dims=d)
        n = v.shape[d]
        if s > 0:
            return torch.cat([v.narrow(d, 1, n - 1), v.narrow(d, n - 1, 1)], dim=d)
        return torch.cat([v.narrow(d, 0, 1), v.narrow(d, 0, n - 1)], dim=d)

    def inner(self, a):
        """1 on the +a faces that exist (none on a wall)."""
        if self.per[a]:
            return 1.0
        return (self.coord[a] < self.n[a] - 1).to(torch.float64)

    def div(self, J, a):
        """Difference of the +a and -a face values; J is 0 on wall faces."""
        return J - torch.roll(J, 1, dims=J.dim() - 1 - a)

    def tdev(self, step):
        c = self.cfg
        if c["G"] == 0:
            return c["T_iso"] - c["T_E"]
        return c["G"] * (self.coord[c["pull_axis"]] - (c["y0"] + c["V"] * step - self.offset))

    def gamma_delta(self, a, b):
        d = self.cfg["delta"][a][b]
        if d != 0 and self.p["delta"] is not None:
            d = self.p["delta"]
        return self.cfg["gamma"][a][b], d

    def dA(self, q, gamma, delta):
        if not torch.is_tensor(delta) and delta == 0:
            return [2 * gamma * v for v in q]
        q2, q4 = sum(v * v for v in q), sum(v ** 4 for v in q)
        big = q2 > self.qmin2
        q2s = torch.where(big, q2, torch.ones_like(q2))
        ac = torch.where(big, 1 - delta * (3 - 4 * q4 / q2s ** 2), torch.ones_like(q2))
        out = []
        for v in q:
            g = torch.where(big, 16 * delta * (v ** 3 - v * q4 / q2s) / q2s ** 2, torch.zeros_like(q2))
            out.append(2 * gamma * ac * (ac * v + q2 * g))
        return out

    def h(self, phi):
        out = []
        for b in range(self.N):
            v = phi[b] ** 2 * (3 - 2 * phi[b])
            o = [phi[g] for g in range(self.N) if g != b]
            for i in range(len(o)):
                for k in range(i + 1, len(o)):
                    v = v + 2 * phi[b] * o[i] * o[k]
            out.append(v)
        return out

    def dh(self, phi, b, a):
        """d h_b / d phi_a"""
        rest = [phi[g] for g in range(self.N) if g not in (a, b)]
        if a != b:
            return 2 * phi[b] * sum(rest) if rest else 0.0
        v = 6 * phi[b] * (1 - phi[b])
        for i in range(len(rest)):
            for k in range(i + 1, len(rest)):
                v = v + 2 * rest[i] * rest[k]
        return v

    def comp(self, b, i, mu, td):
        c = self.cfg
        return c["c0"][b][i] + c.get("mT", [[0.0, 0.0]] * 4)[b][i] * td + sum(c["chi"][i][k] * mu[k] for k in range(self.nc))

    def next_phi(self, phi, mu):
        cfg, N, D = self.cfg, self.N, self.D
        dx, eps = cfg["dx"], cfg["eps"]
        td = self.tdev(self.step_index)
        pairs = [(a, b) for a in range(N) for b in range(a + 1, N)]
        grad = [(self.nb(phi, e, 1) - self.nb(phi, e, -1)) * (0.5 / dx) for e in range(D)]
        div, cell = [0.0] * N, [0.0] * N
        for a in range(D):
            pq = self.nb(phi, a, 1)
            pf = 0.5 * (phi + pq)
            gf = [(pq - phi) / dx if e == a else 0.5 * (grad[e] + self.nb(grad[e], a, 1)) for e in range(D)]
            J = [0.0] * N
            for al, be in pairs:
                q = [pf[al] * g[be] - pf[be] * g[al] for g in gf]
                ga = self.dA(q, *self.gamma_delta(al, be))[a]
                J[al] = J[al] - pf[be] * ga
                J[be] = J[be] + pf[al] * ga
            for b in range(N):
                div[b] = div[b] + self.div(J[b] * self.inner(a), a) / dx
        for al, be in pairs:
            q = [phi[al] * g[be] - phi[be] * g[al] for g in grad]
            dq = self.dA(q, *self.gamma_delta(al, be))
            cell[al] = cell[al] + sum(v * g[be] for v, g in zip(dq, grad))
            cell[be] = cell[be] - sum(v * g[al] for v, g in zip(dq, grad))
        psi = []
        for b in range(N):
            r = cfg["dS"][b] * td
            for i in range(self.nc):
                chimu = sum(cfg["chi"][i][k] * mu[k] for k in range(self.nc))
                r = r - 0.5 * mu[i] * chimu - mu[i] * (cfg["c0"][b][i] + cfg.get("mT", [[0.0, 0.0]] * 4)[b][i] * td)
            psi.append(r)
        rate = cfg["dt"] / (self.p["tau_pf"] * eps)
        vv = []
        for al in range(N):
            dW = sum(16 / math.pi ** 2 * cfg["gamma"][al][be] * phi[be] for be in range(N) if be != al)
            drive = sum(psi[be] * self.dh(phi, be, al) for be in range(N))
            vv.append(phi[al] + rate * (eps * (div[al] - cell[al]) - dW / eps - drive))
        vv = torch.stack(vv)
        # the phases present in the 9/19-point neighbourhood, then the projection onto their simplex
        here = phi.detach() > 0
        line = [here | self.nb(here, a, 1) | self.nb(here, a, -1) for a in range(D)]
        act = line[0]
        for a in range(D):
            for b in range(D):
                if a != b:
                    act = act | self.nb(line[a], b, 1) | self.nb(line[a], b, -1)
        u, _ = torch.sort(torch.where(act, vv, torch.full_like(vv, -1e30)), dim=0, descending=True)
        j = torch.arange(1, N + 1, dtype=torch.float64, device=vv.device).reshape([-1] + [1] * D)
        t = (torch.cumsum(u, dim=0) - 1.0) / j
        last = ((u - t > 0) & (j <= act.sum(0))).sum(0, keepdim=True).clamp(min=1) - 1
        new = torch.where(act, torch.clamp(vv - torch.gather(t, 0, last), min=0.0), torch.zeros_like(vv))
        return torch.where(act.sum(0, keepdim=True) <= 1, phi, new)

    def step(self, state):
        cfg, N, D, nc = self.cfg, self.N, self.D, self.nc
        phi, mu, u, f = state
        dx, dt, chi = cfg["dx"], cfg["dt"], cfg["chi"]
        mT = cfg.get("mT", [[0.0, 0.0]] * 4)
        td = self.tdev(self.step_index)
        dtd = -cfg["G"] * cfg["V"] if cfg["G"] != 0 else 0.0
        new = self.next_phi(phi, mu)
        h0, h1 = self.h(phi), self.h(new)
        diff = [[cfg["D"][b][i] for i in range(nc)] for b in range(N)]
        diff[N - 1][0] = self.p["D"]
        if nc > 1:
            diff[N - 1][1] = self.p["D1"]
        C = [[self.comp(b, i, mu, td) for i in range(nc)] for b in range(N)]
        cs = [sum(h1[b] * C[b][i] for b in range(N)) for i in range(nc)]
        M = [sum(new[b] * diff[b][i] for b in range(N)) for i in range(nc)]
        rhs = []
        for i in range(nc):
            d = 0.0
            for a in range(D):
                Mf = 0.5 * (M[i] + self.nb(M[i], a, 1))
                JD = -sum(Mf * chi[i][k] * (self.nb(mu[k], a, 1) - mu[k]) / dx for k in range(nc))
                uf = 0.5 * (u[a] + self.nb(u[a], a, 1)) * (dx / dt)
                J = (JD + uf * 0.5 * (cs[i] + self.nb(cs[i], a, 1))) * self.inner(a)
                d = d + self.div(J, a) / dx
            r = -dt * d
            for b in range(N):
                r = r - C[b][i] * (h1[b] - h0[b]) - h1[b] * mT[b][i] * dtd
            rhs.append(r)
        sh = sum(h1)
        if nc == 1:
            mun = torch.stack([mu[0] + rhs[0] / (sh * chi[0][0])])
        else:
            det = (chi[0][0] * chi[1][1] - chi[0][1] * chi[1][0]) * sh
            mun = torch.stack([mu[0] + (chi[1][1] * rhs[0] - chi[0][1] * rhs[1]) / det,
                               mu[1] + (chi[0][0] * rhs[1] - chi[1][0] * rhs[0]) / det])
        # collision
        tau, rho0 = cfg["tau_lb"], cfg["rho0"]
        dr = f.sum(0)
        rho = rho0 + dr
        mom = [sum(c[a] * f[k] for k, c in enumerate(self.c) if c[a] != 0) for a in range(D)]
        liq = new[N - 1]
        gb = list(cfg["gbeta"])
        gb[0] = self.p["gbeta"]
        buoy = sum(gb[i] * (self.comp(N - 1, i, mun, td + dtd) - cfg["c_ref"][i]) for i in range(nc))
        FB = [torch.zeros_like(dr) for _ in range(D)]
        FB[cfg["grav_axis"]] = -rho * liq * buoy * cfg["grav_sign"]
        for b in range(N):
            eta = (list(cfg.get("eta", [])) + [0.0] * 4)[b]
            if eta:
                g = [(self.nb(new[b], a, 1) - self.nb(new[b], a, -1)) / (2 * dx) for a in range(D)]
                gg = sum(v * v for v in g)
                big = gg > self.qmin2
                amp = torch.where(big, eta * (new[b] - phi[b]) / torch.sqrt(torch.where(big, gg, torch.ones_like(gg))),
                                  torch.zeros_like(gg))
                FB = [F + amp * v for F, v in zip(FB, g)]
        kappa = 2 * (tau - 0.5) / 3 * cfg["h_drag"] / cfg["W0"]
        sol = (1 - liq) ** 2
        iu = torch.where(liq != 0, 1 / (rho * (1 + 0.5 * kappa * sol)), torch.zeros_like(rho))
        un = [(m + 0.5 * F) * iu for m, F in zip(mom, FB)]
        F = [b - kappa * rho * sol * v for b, v in zip(FB, un)]
        uu, uF = sum(v * v for v in un), sum(v * x for v, x in zip(un, F))
        post = []
        for k, (c, w) in enumerate(zip(self.c, self.w)):
            cu = sum((c[a] * un[a] for a in range(D)), torch.zeros_like(dr))
            cF = sum((c[a] * F[a] for a in range(D)), torch.zeros_like(dr))
            feq = w * (dr + rho * (3 * cu + 4.5 * cu * cu - 1.5 * uu))
            post.append(f[k] - (f[k] - feq) / tau + (1 - 0.5 / tau) * w * (3 * (cF - uF) + 9 * cu * cF))
        # streaming, half-way bounce-back
        fn = []
        for k, c in enumerate(self.c):
            v = torch.roll(post[k], [c[a] for a in range(D)], dims=[D - 1 - a for a in range(D)])
            for a in range(D):
                if c[a] != 0 and not self.per[a]:
                    v = torch.where(self.coord[a] == (0 if c[a] > 0 else self.n[a] - 1), post[self.opp[k]], v)
            fn.append(v)
        return new, mun, torch.stack(un), torch.stack(fn)

    def advance(self, steps):
        for _ in range(steps):
            self.state = self.step(self.state)
            self.step_index += 1
            every = self.cfg.get("frame_every", 0)
            if every and self.step_index % every == 0:
                self.move_frame()
        return self.state

    def move_frame(self):
        a = self.cfg["pull_axis"]
        solid = (self.state[0][self.N - 1] <= 0.5)
        if not bool(solid.any()):
            return
        d = int(self.coord[a].expand(self.shape)[solid].max()) - self.cfg["frame_front"]
        if d > 0:
            at = (torch.arange(self.n[a], device="cuda") + d).clamp(max=self.n[a] - 1)
            self.state = tuple(v.index_select(v.dim() - 1 - a, at) for v in self.state)
            self.offset += d

    def full_f(self, f):
        return f + torch.tensor(self.w, dtype=torch.float64, device="cuda").reshape([-1] + [1] * self.D) * self.cfg["rho0"]


def exact(case, seed):
    cfg = _config(case)
    sim = _Exact(cfg, seed, case["precision"])
    if case["kind"] == "forward":
        with torch.no_grad():
            phi, mu, u, f = sim.advance(case["steps"])
            out = {"phi": phi, "mu": mu, "u": u}
            if case.get("restart"):
                out["f"] = sim.full_f(f)
            if case.get("totals"):
                td, h = sim.tdev(sim.step_index), sim.h(phi)
                out["solute"] = torch.stack([sum((h[b] * sim.comp(b, i, mu, td)).sum() for b in range(sim.N))
                                             for i in range(sim.nc)]).cpu()
                out["mass"] = float(sim.full_f(f).sum())
        return out
    # the run's states, then each step's vector-Jacobian product from the last to the first
    names = PARAMS[case["kind"]]
    values = [torch.tensor(v, dtype=torch.float64, device="cuda") for v in _start_values(cfg, names)]
    states = [sim.state]
    with torch.no_grad():
        for _ in range(case["steps"]):
            sim.advance(1)
            states.append(sim.state)
    phi = sim.state[0]
    dtype = torch.float64 if case["precision"] == "fp64" else torch.float32
    lam = [phi - _target(cfg, dtype).double()] + [torch.zeros_like(v) for v in sim.state[1:]]
    grad = torch.zeros(len(names), dtype=torch.float64, device="cuda")
    for n in range(case["steps"] - 1, -1, -1):
        sim.step_index = n
        at = [v.detach().requires_grad_(True) for v in states[n]]
        ps = [v.detach().clone().requires_grad_(True) for v in values]
        sim.p.update(dict(zip(names, ps)))
        with torch.enable_grad():
            out = sim.step(at)
            got = torch.autograd.grad(out, at + ps, grad_outputs=lam, allow_unused=True)
        got = [torch.zeros_like(x) if g is None else g for x, g in zip(at + ps, got)]
        lam, dp = got[:4], got[4:]
        grad += torch.stack(dp)
    return {"phi": phi, "grad": grad.cpu()}
