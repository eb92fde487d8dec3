"""Performance cases of the rod library: what its users run, through the Python binding.

A case names a family and its sizes. The families are those of `workloads`, the
benchmark and the tests: one small rod stepped in short calls, the helix ramp, a
gradient through recorded steps, a batch of independent rods, the twisted rod, a
ragged cilia carpet with its energies, the rod array with all dipole pairs, with a
dipole cutoff and in a periodic box (Ewald sum), rods without dipoles (bonds,
contact and integration alone), the lattice Boltzmann fluid, and a carpet in it.

`prepare` builds what a program keeps between calls (the simulation or lattice
with its buffers), `run` is one call or a short sequence of calls on it, and
`exact` the same result from the model's equations in plain FP64 torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import workloads

STATE = ("x", "v", "q", "w", "F", "T")


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # a short call on the smallest rod (the cantilever test): latency alone
        dict(name="rod_20", family="rod", n=20, precision="fp64", steps=50, graph=0),
        # quasi-static ramp of the magnetic helix: Hertz-Mindlin contact, bond
        # damping, a rest check after every chunk of steps
        dict(name="helix_104_ramp", family="helix", n_bonds=103, precision="mixed", settings=2,
             steps=200, check=100, graph=100),
        # one training iteration: a recorded run and its gradient
        dict(name="adjoint_256", family="adjoint", n=256, precision="fp64", steps=200, every=100),
        # a parameter sweep: independent short rods stepped together
        dict(name="members_32x200", family="members", members=32, n=200, precision="mixed",
             steps=50, graph=50),
        # the twisted rod: contact, a driven end, graph replays
        dict(name="twisted_4096", family="twisted", n=4096, precision="mixed", steps=50, graph=50),
        # a ragged carpet in FP64, its energies read after every few steps
        dict(name="carpet_12x12_energy", family="carpet", gx=12, gy=12, lo=16, hi=128,
             precision="fp64", steps=5, graph=0),
        # the largest all-pairs system, in the layout that the tuner picks for it
        dict(name="rod_array_262144", family="array", gx=32, gy=16, n=512, precision="mixed",
             steps=1, graph=0, layout=2, target=16384),
        # the same rods with a dipole cutoff
        dict(name="cutoff_262144", family="cutoff", gx=32, gy=16, n=512, cutoff=3.0,
             precision="mixed", steps=20, graph=20),
        # rods in a periodic box: Ewald sum
        dict(name="periodic_32768", family="periodic", gx=32, gy=32, n=32, lz=40.0, rcut=16.0,
             precision="mixed", steps=2, graph=0),
        # a million particles without dipoles: bonds, contact lists, integration
        dict(name="rods_1M", family="free", gx=32, gy=32, n=1024, precision="mixed", steps=10,
             graph=10),
        # the fluid alone, between walls, ragged sides
        dict(name="lbm_walls_150x126x130", family="lbm", nx=150, ny=126, nz=130, walls=1, steps=20),
        # a carpet in the fluid: coupled cycles
        dict(name="immersed_16x16", family="immersed", gx=16, gy=16, lo=16, hi=64, nx=128, ny=128,
             nz=96, walls=0, sub=10, cycles=1, precision="mixed"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    fam = rng.choice(["rod", "helix", "adjoint", "members", "twisted", "carpet", "array", "cutoff",
                      "periodic", "free", "lbm", "immersed"])
    prec = rng.choice(["fp64", "mixed"])
    if fam == "rod":
        steps = _log(rng, 10, 200)
        return dict(family=fam, n=_log(rng, 2, 1000), precision=prec, steps=steps,
                    graph=rng.choice([0, steps]))
    if fam == "helix":
        check = _log(rng, 20, 200)
        return dict(family=fam, n_bonds=_log(rng, 40, 300), precision=prec,
                    settings=rng.randint(1, 3), steps=2 * check, check=check,
                    graph=rng.choice([0, check]))
    if fam == "adjoint":
        every = _log(rng, 20, 100)
        return dict(family=fam, n=_log(rng, 12, 512), precision=prec,
                    steps=every * rng.randint(1, 2) + rng.randint(0, 7), every=every)
    if fam == "members":
        steps = _log(rng, 10, 100)
        return dict(family=fam, members=_log(rng, 2, 64), n=_log(rng, 12, 1000), precision=prec,
                    steps=steps, graph=rng.choice([0, steps]))
    if fam == "twisted":
        steps = _log(rng, 10, 100)
        return dict(family=fam, n=_log(rng, 300, 8000), precision=prec, steps=steps, graph=steps)
    if fam == "carpet":
        return dict(family=fam, gx=rng.randint(2, 16), gy=rng.randint(2, 16), lo=16, hi=128,
                    precision=prec, steps=rng.randint(1, 10), graph=0)
    if fam == "array":
        n = _log(rng, 40, 512)
        return dict(family=fam, gx=rng.randint(4, 16), gy=rng.randint(4, 16), n=n, precision=prec,
                    steps=rng.randint(1, 2), graph=0, layout=rng.choice([-1, 2]), target=4096)
    if fam == "cutoff":
        steps = rng.randint(2, 20)
        return dict(family=fam, gx=rng.randint(4, 32), gy=rng.randint(4, 16), n=_log(rng, 40, 512),
                    cutoff=round(rng.uniform(2.2, 3.6), 2), precision=prec, steps=steps,
                    graph=rng.choice([0, steps]))
    if fam == "periodic":
        n = rng.randint(12, 32)
        rcut = round(rng.uniform(6.0, 12.0), 1)
        return dict(family=fam, gx=rng.randint(6, 24), gy=rng.randint(6, 24), n=n,
                    lz=float(max(n + 4, math.ceil(2 * rcut))), rcut=rcut, precision=prec,
                    steps=rng.randint(1, 3), graph=0)
    if fam == "free":
        steps = rng.randint(2, 10)
        return dict(family=fam, gx=rng.randint(4, 32), gy=rng.randint(4, 32), n=_log(rng, 100, 1500),
                    precision=prec, steps=steps, graph=rng.choice([0, steps]))
    if fam == "lbm":
        return dict(family=fam, nx=_log(rng, 24, 160), ny=_log(rng, 24, 160), nz=_log(rng, 24, 160),
                    walls=rng.randint(0, 2), steps=_log(rng, 5, 40))
    g = rng.randint(4, 12)
    return dict(family=fam, gx=g, gy=g, lo=16, hi=48, nx=8 * g, ny=8 * g + rng.randint(0, 9),
                nz=rng.randint(56, 96), walls=rng.randint(0, 2), sub=rng.choice([5, 10]), cycles=1,
                precision=prec)


# ------------------------------------------------------------------ inputs
def _workload(case, seed):
    """The workload dictionary of a case: geometry as the workload defines it, and
    the noise of positions, velocities and (where they vary) dipoles from `seed`."""
    fam = case["family"]
    if fam == "rod":
        w = workloads.cantilever(n=case["n"], sigma=0.0)
    elif fam == "helix":
        w = workloads.magnetic_helix(n_bonds=case["n_bonds"], length=float(case["n_bonds"]))
    elif fam == "adjoint":
        w = workloads.adjoint_rod(n=case["n"], sigma=0.0)
    elif fam == "members":
        w = workloads.ensemble(members=case["members"], n=case["n"], sigma=0.0)
    elif fam == "twisted":
        w = workloads.twisted_rod(n=case["n"], sigma=0.0)
    elif fam in ("carpet", "immersed"):
        w = workloads.cilia_carpet(grid=(case["gx"], case["gy"]), len_range=(case["lo"], case["hi"]),
                                   sigma=0.0)
        if fam == "immersed":  # into the lattice, off its lower faces
            w["x_ref"] = w["x_ref"] + np.array([4.0, 4.0, 2.0])
            w["dt"] = 1.0 / case["sub"]
    elif fam in ("array", "cutoff", "periodic", "free"):
        w = workloads.rod_array(grid=(case["gx"], case["gy"]), n_per_rod=case["n"], sigma=0.0,
                                half_sweep=2000)
        if fam == "cutoff":
            w["dipole_cutoff"] = case["cutoff"]
        elif fam == "free":
            w["dipole_on"] = False
        elif fam == "periodic":  # the lateral pitch goes on across the boundary
            box = (2.0 * case["gx"], 2.0 * case["gy"], case["lz"])
            rcut = min(case["rcut"], 0.5 * min(box))
            alpha = 3.6 / rcut
            w.update(contact_on=False, box=np.asarray(box), ewald_rcut=rcut, ewald_alpha=alpha,
                     ewald_kmax=int(np.ceil(3.6 * alpha * max(box) / np.pi)))
    rng = np.random.default_rng(seed)
    n, free = w["n"], (w["bc"] == 0)[:, None]
    w["x0"] = w["x_ref"] + rng.normal(0.0, 1e-3, (n, 3)) * free
    w["v0"] = rng.normal(0.0, 1e-3, (n, 3)) * free
    w["w0"] = rng.normal(0.0, 1e-3, (n, 3)) * free
    if fam == "adjoint":
        w["m_body"] = rng.normal(0.0, 0.05, (n, 3))
    return w


_D3Q19 = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1, 0),
          (-1, -1, 0), (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1), (-1, 0, 1),
          (0, 1, 1), (0, -1, -1), (0, 1, -1), (0, -1, 1)]
_TAU, _LID = 0.8, 0.02


def _equilibrium(rho, u):
    uu = (u * u).sum(0)
    out = []
    for k, c in enumerate(_D3Q19):
        wt = 1 / 3 if k == 0 else 1 / 18 if k < 7 else 1 / 36
        cu = sum(c[a] * u[a] for a in range(3))
        out.append(wt * rho * (1 + 3 * cu + 4.5 * cu * cu - 1.5 * uu))
    return torch.stack(out)


def _fluid(case, seed):
    """Populations at equilibrium of a flow of a few smooth waves."""
    rng = np.random.default_rng(seed)
    shape = (case["nz"], case["ny"], case["nx"])
    ax = [torch.arange(s, dtype=torch.float64, device="cuda") * (2 * math.pi / s) for s in shape]
    z, y, x = ax[0][:, None, None], ax[1][None, :, None], ax[2][None, None, :]
    f = torch.zeros((4,) + shape, dtype=torch.float64, device="cuda")
    for comp in range(4):
        for _ in range(3):
            k = rng.integers(0, 3, 3)
            f[comp] += rng.normal(0.0, 0.01) * torch.sin(
                int(k[0]) * x + int(k[1]) * y + int(k[2]) * z + rng.uniform(0, 2 * math.pi))
    return _equilibrium(1.0 + 0.1 * f[3], f[:3])


def _lid(case):
    return (_LID, 0.0) if case["walls"] == 1 else (0.0, 0.0)


def _ramp_fields(case, w):
    return workloads.helix_ramp_fields(w, [0.4 + 0.3 * k for k in range(case["settings"])])


# ------------------------------------------------------------------ the calls
def prepare(case, seed):
    from paper_2603_27279_amd import Lattice, RodSim
    fam = case["family"]
    if fam == "lbm":
        return dict(case=case, lat=Lattice(_fluid(case, seed), tau=_TAU, force=(1e-6, 0.0, 0.0),
                                           walls_z=case["walls"], lid=_lid(case)))
    w = _workload(case, seed)
    s = dict(case=case)
    if fam == "helix":
        s["fields"] = _ramp_fields(case, w)
        w["field"] = s["fields"][:1]
    if fam == "adjoint":
        sim = RodSim(w, precision=case["precision"], tape_every=case["every"],
                     tape_capacity=case["steps"])
        s["start"] = [t.clone() for t in (sim.x, sim.v, sim.q, sim.om)]
        s["target"] = torch.as_tensor(w["target"], device="cuda")
    else:
        sim = RodSim(w, precision=case["precision"], graph_steps=case.get("graph", 0))
    if fam == "array":
        sim.dipole_layout(case["layout"], case["target"])
    if fam == "immersed":
        s["lat"] = Lattice(_fluid(case, seed), tau=_TAU, walls_z=case["walls"], lid=_lid(case))
    s["sim"] = sim
    return s


def run(s):
    case = s["case"]
    fam = case["family"]
    if fam == "lbm":
        s["lat"].step(case["steps"])
        rho, u = s["lat"].moments()
        return dict(f=s["lat"].populations(), rho=rho, u=u)
    sim = s["sim"]
    out = {}
    if fam == "helix":
        r = sim.ramp(s["fields"], max_steps=case["steps"], check_every=case["check"], ke_tol=1e-12,
                     watch=[0, sim.n - 1])
        out.update(r)
    elif fam == "adjoint":  # from the same start every time, as an optimiser does
        for t, t0 in zip((sim.x, sim.v, sim.q, sim.om), s["start"]):
            t.copy_(t0)
        sim.tape_begin()
        sim.step(case["steps"])
        gx = torch.zeros_like(sim.x)
        gx[:, -1] = 2.0 * (sim.x[:, -1] - s["target"])
        out["grad"] = sim.grad(gx=gx)
    elif fam == "immersed":
        sim.lbm_cycles(s["lat"], case["sub"], case["cycles"])
        out["f"] = s["lat"].populations()
    else:
        sim.step(case["steps"])
        if fam == "carpet":
            out["energy"] = sim.energy()
    out.update(zip(STATE, (sim.x, sim.v, sim.q, sim.om, sim.F, sim.T)))
    return out


# ------------------------------------------------------------------ work
def work(case):
    """Bytes and operations that a pass cannot do without. A particle's state (19
    doubles) in and out and about 14 doubles of its constants; once per call
    where the system is small enough to stay on the chip, once per step where it
    is not (4 MB of L2 per XCD: about 10,000 particles). About 700 operations per
    particle and step for the bond and the update, 67 per ordered dipole pair
    (93 with Ewald screening, 12 per reciprocal term)."""
    fam = case["family"]
    if fam == "lbm":
        cells = case["nx"] * case["ny"] * case["nz"]
        return {"bytes": cells * (304.0 * case["steps"] + 64.0), "flops": 300.0 * cells * case["steps"]}
    steps = case["steps"] if fam != "immersed" else case["sub"] * case["cycles"]
    if fam == "helix":
        n = case["n_bonds"] + 1
        steps *= case["settings"]
    elif fam in ("carpet", "immersed"):
        n = workloads.cilia_carpet(grid=(case["gx"], case["gy"]), len_range=(case["lo"], case["hi"]),
                                   period=2)["n"]
    elif fam in ("array", "cutoff", "periodic", "free"):
        n = case["gx"] * case["gy"] * case["n"]
    else:
        n = case["n"] * case.get("members", 1)
    evals = steps + (1 if fam == "carpet" else 0)
    per = 416.0 * n
    b = per * (steps if n > 10000 else 1)
    f = 700.0 * n * evals
    if fam == "adjoint":  # recorded run, recomputation, reverse of twice the operations
        b, evals = 4 * per, 4 * steps
        f = 700.0 * n * evals
    if fam == "cutoff":
        f += 67.0 * n * steps * (4.0 / 3.0 * math.pi * case["cutoff"] ** 3 * 0.25)
    elif fam == "periodic":
        w = _workload(dict(case, n=2), 0)
        rc, box, km = w["ewald_rcut"], w["box"], w["ewald_kmax"]
        f += n * steps * (93.0 * 4.0 / 3.0 * math.pi * rc ** 3 * n / float(np.prod(box)) +
                          24.0 * 2.0 / 3.0 * math.pi * km ** 3)
    elif fam != "free":
        f += 67.0 * evals * n * (n // case.get("members", 1))
    if fam == "immersed":
        cells = case["nx"] * case["ny"] * case["nz"]
        b += case["cycles"] * cells * (304.0 + 48.0)
        f += 300.0 * cells * case["cycles"]
    return {"bytes": b, "flops": f}


# ------------------------------------------------------------------ the model in FP64 torch
def _qmul(a, b):
    return torch.stack((a[0] * b[0] - a[1] * b[1] - a[2] * b[2] - a[3] * b[3],
                        a[0] * b[1] + a[1] * b[0] + a[2] * b[3] - a[3] * b[2],
                        a[0] * b[2] - a[1] * b[3] + a[2] * b[0] + a[3] * b[1],
                        a[0] * b[3] + a[1] * b[2] - a[2] * b[1] + a[3] * b[0]))


def _conj(q):
    return torch.cat((q[:1], -q[1:]))


def _unit(q):
    return q / torch.sqrt((q * q).sum(0))


def _cross(a, b):
    return torch.stack((a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0]))


def _rot(q, v):
    t = 2.0 * _cross(q[1:], v)
    return v + q[0] * t + _cross(q[1:], t)


def _near(x, member, rc):
    """Ordered pairs (i, j), i != j, of one member with |x_i - x_j| < rc."""
    c = torch.floor((x - x.min(1, keepdim=True).values) / rc).to(torch.int64) + 1
    d = [int(c[a].max()) + 2 for a in range(3)]
    key = ((member * d[2] + c[2]) * d[1] + c[1]) * d[0] + c[0]
    skey, order = torch.sort(key)
    n = x.shape[1]
    me = torch.arange(n, device=x.device)
    got = []
    for o in range(27):
        k = key + ((o // 9 - 1) * d[1] + (o // 3 % 3 - 1)) * d[0] + (o % 3 - 1)
        b = torch.searchsorted(skey, k)
        cnt = torch.searchsorted(skey, k, right=True) - b
        i = torch.repeat_interleave(me, cnt)
        at = torch.arange(i.numel(), device=x.device) - torch.repeat_interleave(cnt.cumsum(0) - cnt, cnt)
        j = order[b[i] + at]
        r = x[:, i] - x[:, j]
        ok = ((r * r).sum(0) < rc * rc) & (i != j)
        got.append((i[ok], j[ok]))
    return torch.cat([g[0] for g in got]), torch.cat([g[1] for g in got])


class _Model:
    """The bonded-particle model of one workload; vectors [3, N], quaternions [4, N]."""

    def __init__(self, w):
        t = lambda a: torch.as_tensor(np.ascontiguousarray(np.asarray(a, np.float64).T), device="cuda")
        self.w, self.n, self.dt = w, w["n"], float(w["dt"])
        n, off = self.n, np.asarray(w["rod_offset"])
        rod = np.repeat(np.arange(len(off) - 1), np.diff(off))
        mem = np.asarray(w["rod_member"])[rod]
        k = np.flatnonzero(rod[:-1] == rod[1:])
        self.rod, self.mem = torch.as_tensor(rod, device="cuda"), torch.as_tensor(mem, device="cuda")
        self.k = torch.as_tensor(k, device="cuda")
        self.ranges = [(int(np.searchsorted(mem, m)), int(np.searchsorted(mem, m, "right")))
                       for m in range(w["n_members"])]
        d, rho, E, nu = (np.asarray(w["rod_params"])[rod, c] for c in range(4))
        rref = w["x_ref"][k + 1] - w["x_ref"][k]
        r0 = np.linalg.norm(rref, axis=1)
        A, I = math.pi * d ** 2 / 4, math.pi * d ** 4 / 64
        G = E / (2 * (1 + nu))
        self.Kr, self.Ks = t((E * A)[k] / r0), t((12 * E * I)[k] / r0 ** 3)
        self.Kt, self.Kb = t((2 * G * I)[k] / r0), t((E * I)[k] / r0)
        self.r0, self.ri = t(r0), t(rref / r0[:, None])
        self.mass, self.inertia = t(rho * math.pi * d ** 3 / 6), t(rho * math.pi * d ** 5 / 60)
        self.free = torch.as_tensor(w["bc"] == 0, device="cuda")
        self.driven = torch.as_tensor(w["bc"] == 2, device="cuda")
        self.axis = torch.as_tensor(np.asarray(w["drive_axis"], np.float64), device="cuda")
        self.field, self.mb = torch.as_tensor(w["field"], device="cuda"), t(w["m_body"])
        self.x0, self.v0, self.q0, self.w0 = (t(w[a]) for a in ("x0", "v0", "q0", "w0"))
        self.damp = None
        if w["bond_damping"] is not None:
            self.damp = t(np.asarray(w["bond_damping"])[rod[k]])
        self.measure = self.slide = self.fluid = None
        self.Bdip = None

    # -- forces
    def bonds(self, x, v, q, F, T):
        k = self.k
        if not k.numel():
            return F, T
        q1, q2 = q[:, k], q[:, k + 1]
        q2 = torch.where((q1 * q2).sum(0) < 0, -q2, q2)
        qc = _unit(q1 + q2)
        rho = _rot(_conj(qc), x[:, k + 1] - x[:, k])
        r = torch.sqrt((rho * rho).sum(0))
        rh = rho / r
        c = _cross(self.ri, rh - self.ri)
        s2 = (c * c).sum(0)
        some = s2 > 0
        sig = torch.sqrt(torch.where(some, s2, 1.0))
        cg = (self.ri * rh).sum(0)
        gam = torch.where(some, torch.atan2(sig, cg), 0.0)
        g = torch.where(some, gam / sig, 1.0 / cg)
        u0 = _qmul(_conj(qc), q2)
        m = _unit(torch.stack((1.0 + rh[2], -rh[1], rh[0], torch.zeros_like(r))))
        flip = 1.0 + rh[2] <= 1e-12
        if bool(flip.any()):
            m = torch.where(flip, torch.tensor([0.0, 1.0, 0.0, 0.0], device=x.device,
                                               dtype=x.dtype)[:, None], m)
        u = torch.cat((u0[:1], _rot(_conj(m), u0[1:])))
        tn = torch.sqrt(u[0] ** 2 + u[3] ** 2)
        t2 = torch.stack((u[0] / tn, torch.zeros_like(tn), torch.zeros_like(tn), u[3] / tn))
        psi = 4.0 * torch.atan2(u[3], u[0])
        b = _qmul(_qmul(_conj(t2), _qmul(u, u)), _conj(t2))
        b = torch.where(b[0] < 0, -b, b)
        b2 = (b[1:] * b[1:]).sum(0)
        some_b = b2 > 0
        bn = torch.sqrt(torch.where(some_b, b2, 1.0))
        theta = torch.where(some_b, 2.0 * torch.atan2(bn, b[0]), 0.0)
        bend = torch.where(some_b, theta / bn, 2.0 / b[0]) * b[1:]
        frad, ks = self.Kr * (r - self.r0), self.Ks * g
        tb = self.Kb * bend
        tw = self.Kt * psi
        if self.damp is not None:
            idt = 1.0 / self.dt
            frad = frad + self.damp[0] * (_rot(_conj(qc), v[:, k + 1] - v[:, k]) * rh).sum(0)
            if self.measure is not None:
                pg, pp, pb = self.measure
                ks = torch.where(some, ks + self.damp[1] * (gam - pg) * idt / sig, ks)
                dp = psi - pp
                dp = dp - 2 * math.pi * torch.round(dp / (2 * math.pi))
                tb = tb + self.damp[3] * (bend - pb) * idt
                tw = tw + self.damp[2] * dp * idt
            self.measure = (gam, psi, bend)
        tb = torch.stack((tb[0], tb[1], tb[2] + tw))
        f = _rot(qc, frad * rh + r * ks * _cross(c, rh))
        ts = _rot(qc, 0.5 * r * r * ks * c)
        tb = _rot(qc, _rot(m, tb))
        F = F.index_add(1, k, f).index_add(1, k + 1, -f)
        T = T.index_add(1, k, ts + tb).index_add(1, k + 1, ts - tb)
        self.bond_energy = (0.5 * self.Kr * (r - self.r0) ** 2, 0.5 * self.Ks * r * r * gam ** 2,
                            0.5 * self.Kt * psi ** 2, 0.5 * self.Kb * theta ** 2)
        return F, T

    def dipoles(self, x, m):
        w, C = self.w, float(self.w["mu0_4pi"])
        box = None if w["box"] is None else [float(a) for a in w["box"]]
        if w["dipole_cutoff"]:
            i, j = _near(x, self.mem, float(w["dipole_cutoff"]))
            r, mi, mj = x[:, i] - x[:, j], m[:, i], m[:, j]
            u = 1.0 / torch.sqrt((r * r).sum(0))
            a, b, c = (mi * r).sum(0), (mj * r).sum(0), (mi * mj).sum(0)
            z = torch.zeros_like(x)
            return (z.index_add(1, i, 3 * C * u ** 5 * ((c - 5 * a * b * u * u) * r + b * mi + a * mj)),
                    z.index_add(1, i, C * (3 * u ** 5 * b * r - u ** 3 * mj)))
        Fs, Bs = [], []
        for lo, hi in self.ranges:
            xs, ms = x[:, None, lo:hi], m[:, None, lo:hi]
            step = max(1, min(hi - lo, (1 << 25) // (hi - lo)))
            for t in range(lo, hi, step):
                e = min(t + step, hi)
                mi = m[:, t:e, None]
                r = [x[a, t:e, None] - xs[a] for a in range(3)]
                if box:
                    r = [r[a] - box[a] * torch.round(r[a] / box[a]) for a in range(3)]
                r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2]
                other = torch.arange(t, e, device=x.device)[:, None] != torch.arange(
                    lo, hi, device=x.device)[None, :]
                r2 = torch.where(other, r2, 1.0)
                u = 1.0 / torch.sqrt(r2)
                if box:
                    al = w["ewald_alpha"]
                    ar2 = al * al * r2
                    p = 2 * al / math.sqrt(math.pi) / u * torch.exp(-ar2)
                    ec = torch.erfc(al / u)
                    on = other & (r2 < w["ewald_rcut"] ** 2)
                    b1 = torch.where(on, (ec + p) * u ** 3, 0.0)
                    b3 = torch.where(on, (3 * ec + p * (3 + 2 * ar2)) * u ** 5, 0.0)
                    b5 = torch.where(on, (15 * ec + p * (15 + 10 * ar2 + 4 * ar2 * ar2)) * u ** 7, 0.0)
                else:
                    u = torch.where(other, u, 0.0)
                    b1, b3, b5 = u ** 3, 3 * u ** 5, 15 * u ** 7
                a = sum(mi[c] * r[c] for c in range(3))
                b = sum(ms[c] * r[c] for c in range(3))
                c = sum(mi[d] * ms[d] for d in range(3))
                al_, sa, sb = c * b3 - a * b * b5, b3 * a, b3 * b
                Fs.append(C * torch.stack([(al_ * r[d] + sb * mi[d] + sa * ms[d]).sum(1)
                                           for d in range(3)]))
                Bs.append(C * torch.stack([(sb * r[d] - b1 * ms[d]).sum(1) for d in range(3)]))
        F, B = torch.cat(Fs, 1), torch.cat(Bs, 1)
        if box:
            F2, B2 = self.reciprocal(x, m, box)
            F, B = F + C * F2, B + C * (B2 + 4 * w["ewald_alpha"] ** 3 / (3 * math.sqrt(math.pi)) * m)
        return F, B

    def reciprocal(self, x, m, box):
        K, al = int(self.w["ewald_kmax"]), self.w["ewald_alpha"]
        g = np.stack(np.meshgrid(np.arange(0, K + 1), np.arange(-K, K + 1), np.arange(-K, K + 1),
                                 indexing="ij"), -1).reshape(-1, 3)
        half = (g[:, 0] > 0) | ((g[:, 0] == 0) & ((g[:, 1] > 0) | ((g[:, 1] == 0) & (g[:, 2] > 0))))
        g = g[half & ((g * g).sum(1) <= K * K)]
        kv = torch.as_tensor(2 * math.pi * g / np.asarray(box), device=x.device)
        k2 = (kv * kv).sum(1)
        wt = 8 * math.pi / math.prod(box) * torch.exp(-k2 / (4 * al * al)) / k2
        F, B = torch.zeros_like(x), torch.zeros_like(x)
        for lo, hi in self.ranges:
            xs, ms = x[:, lo:hi], m[:, lo:hi]
            for s in range(0, len(kv), 512):
                k, c = kv[s:s + 512], wt[s:s + 512, None]
                ph, mk = k @ xs, k @ ms
                cs, sn = torch.cos(ph), torch.sin(ph)
                Sr, Si = (mk * cs).sum(1, keepdim=True), (mk * sn).sum(1, keepdim=True)
                F[:, lo:hi] += k.T @ (c * mk * (sn * Sr - cs * Si))
                B[:, lo:hi] -= k.T @ (c * (cs * Sr + sn * Si))
        return F, B

    def contacts(self, x, v, om, F, T):
        w, rc = self.w, float(self.w["r_contact"])
        i, j = _near(x.detach(), self.mem, rc)
        ok = (self.rod[i] != self.rod[j]) | ((i - j).abs() > int(w["exclude_depth"]))
        i, j = i[ok], j[ok]
        d = x[:, i] - x[:, j]
        r = torch.sqrt((d * d).sum(0))
        ov = rc - r
        if w["contact_model"] == "hookean":
            self.contact_energy = torch.zeros_like(x[0]).index_add(0, i, 0.25 * w["k_contact"] * ov ** 2)
            return F.index_add(1, i, w["k_contact"] * ov / r * d), T
        E, nu, mu, gn, gt = (float(a) for a in w["contact_hm"])
        n, a = d / r, torch.sqrt(0.25 * rc * ov)
        kn = 4 / 3 * E / (2 * (1 - nu * nu)) * a
        kt = 8 * E / (4 * (2 - nu) * (1 + nu)) * a
        rel = v[:, i] - v[:, j] - 0.5 * r * _cross(om[:, i] + om[:, j], n)
        vn = (rel * n).sum(0)
        vt = rel - vn * n
        fn = torch.clamp(kn * ov - gn * vn, min=0.0)
        s = torch.zeros_like(d)
        if self.slide is not None:  # the displacements of the previous level, dense by pair
            p, had = self.slide[:, i, j], self.had[i, j]
            st = p - (p * n).sum(0) * n
            lt, lp = torch.sqrt((st * st).sum(0)), torch.sqrt((p * p).sum(0))
            st = torch.where(lt > 0, lp / torch.where(lt > 0, lt, 1.0), 1.0) * st
            s = torch.where(had, st + self.dt * vt, s)
        ft = -kt * s - gt * vt
        size = torch.sqrt((ft * ft).sum(0))
        over = size > mu * fn
        ft = torch.where(over, mu * fn / torch.where(over, size, 1.0) * ft, ft)
        s = torch.where(over, -(ft + gt * vt) / kt, s)
        self.slide = torch.zeros((3, self.n, self.n), dtype=x.dtype, device=x.device)
        self.slide[:, i, j] = s
        self.had = torch.zeros((self.n, self.n), dtype=torch.bool, device=x.device)
        self.had[i, j] = True
        return F.index_add(1, i, fn * n + ft), T.index_add(1, i, _cross(-0.5 * r * n, ft))

    def forces(self, x, v, q, om, level):
        w = self.w
        F, T = self.bonds(x, v, q, torch.zeros_like(x), torch.zeros_like(x))
        m = _rot(q, self.mb)
        self.m = m
        if w["dipole_on"]:
            Fd, self.Bdip = self.dipoles(x, m)
            F, T = F + Fd, T + _cross(m, self.Bdip)
        f = self.field[level % self.field.shape[0]][self.mem].T
        G = f[3:].reshape(3, 3, -1)
        self.Bext = f[:3] + (G * x[None]).sum(1)
        F, T = F + (G * m[:, None]).sum(0), T + _cross(m, self.Bext)
        if w["contact_on"]:
            F, T = self.contacts(x, v, om, F, T)
        F = F - w["damping"] * self.mass * v
        T = T - w["damping"] * self.inertia * om
        if self.fluid is not None:
            self.pull = self.mass * (self.fluid - v)
            F = F + self.pull
        return F, T

    # -- time
    def turn(self, level):
        h = math.pi * level / max(1, int(self.w["drive_period"]))
        return torch.cat((torch.tensor([math.cos(h)], dtype=torch.float64, device="cuda"),
                          math.sin(h) * self.axis))[:, None]

    def begin(self, x, v, q, om, level=0):
        q, z = _unit(q), torch.zeros_like(x)
        v, om = torch.where(self.free, v, z), torch.where(self.free, om, z)
        if bool(self.driven.any()):
            q = torch.where(self.driven, self.turn(level), q)
            rate = 2 * math.pi / (self.w["drive_period"] * self.dt)
            om = torch.where(self.driven, rate * self.axis[:, None], om)
        return (x, v, q, om) + self.forces(x, v, q, om, level)

    def step(self, S, level):
        """From level - 1 to level."""
        x, v, q, om, F, T = S
        dt, fr = self.dt, self.free
        v = torch.where(fr, v + 0.5 * dt / self.mass * F, v)
        om = torch.where(fr, om + 0.5 * dt / self.inertia * T, om)
        x = torch.where(fr, x + dt * v, x)
        p = torch.cat((torch.zeros_like(om[:1]), om))
        q1 = _unit(q + 0.5 * dt * _qmul(p, q))
        qh = _unit(q + 0.25 * dt * _qmul(p, q))
        q2 = _unit(qh + 0.25 * dt * _qmul(p, qh))
        q = torch.where(fr, _unit(2.0 * q2 - q1), q)
        if bool(self.driven.any()):
            q = torch.where(self.driven, self.turn(level), q)
        F, T = self.forces(x, v, q, om, level)
        v = torch.where(fr, v + 0.5 * dt / self.mass * F, v)
        om = torch.where(fr, om + 0.5 * dt / self.inertia * T, om)
        return x, v, q, om, F, T

    def energies(self, S, level):
        x, v, q, om = S[:4]
        self.forces(x, v, q, om, level)
        per = [torch.zeros_like(x[0]).index_add(0, self.k, e) for e in self.bond_energy]
        per += [-(self.m * self.Bext).sum(0), -0.5 * (self.m * self.Bdip).sum(0), self.contact_energy,
                0.5 * self.mass * (v * v).sum(0), 0.5 * self.inertia * (om * om).sum(0)]
        return torch.stack([torch.stack([e[lo:hi].sum() for e in per]) for lo, hi in self.ranges])


def _collide(f, g, walls, lid, force=(0.0, 0.0, 0.0)):
    """One lattice step of populations f with the force field g [3, ...] (or None)."""
    e = f.new_tensor(_D3Q19)
    rho = f.sum(0)
    g = [force[a] + (0.0 if g is None else g[a]) for a in range(3)]
    u = torch.stack([((e[:, a, None, None, None] * f).sum(0) + 0.5 * g[a]) / rho for a in range(3)])
    eq, ug = _equilibrium(rho, u), sum(u[a] * g[a] for a in range(3))
    out, nz = torch.zeros_like(f), f.shape[1]
    index = {c: k for k, c in enumerate(_D3Q19)}
    for k, c in enumerate(_D3Q19):
        wt = 1 / 3 if k == 0 else 1 / 18 if k < 7 else 1 / 36
        cu, cg = sum(c[a] * u[a] for a in range(3)), sum(c[a] * g[a] for a in range(3))
        s = f[k] - (f[k] - eq[k]) / _TAU + (1 - 0.5 / _TAU) * wt * (3 * (cg - ug) + 9 * cu * cg)
        moved = torch.roll(s, (c[2], c[1], c[0]), (0, 1, 2))
        if not walls or c[2] == 0:
            out[k] += moved
            continue
        top = c[2] > 0
        keep = slice(1, nz) if top else slice(0, nz - 1)
        edge = nz - 1 if top else 0
        out[k][keep] += moved[keep]
        if top and walls == 2:
            out[index[(c[0], c[1], -c[2])]][edge] += s[edge]
        else:
            lost = 6 * wt * rho[edge] * (c[0] * lid[0] + c[1] * lid[1]) if top else 0.0
            out[index[tuple(-a for a in c)]][edge] += s[edge] - lost
    return out


def _moments(f, force=(0.0, 0.0, 0.0)):
    e, rho = f.new_tensor(_D3Q19), f.sum(0)
    return rho, torch.stack([((e[:, a, None, None, None] * f).sum(0) + 0.5 * force[a]) / rho
                             for a in range(3)])


def _stencil(x, shape, walls):
    """Nodes [64, N] around each particle and their weights (four-point delta)."""
    base = torch.floor(x).to(torch.int64) - 1
    node, wt = 0, 1.0
    for a, axis in ((2, 0), (1, 1), (0, 2)):
        o = torch.arange(4, device=x.device).repeat_interleave(4 ** a).repeat(4 ** (2 - a))
        p = base[a][None] + o[:, None]
        r = (p - x[a][None]).abs()
        near = (3 - 2 * r + torch.sqrt(torch.clamp(1 + 4 * r - 4 * r * r, min=0.0))) / 8
        far = (5 - 2 * r - torch.sqrt(torch.clamp(-7 + 12 * r - 4 * r * r, min=0.0))) / 8
        phi = torch.where(r <= 1, near, torch.where(r <= 2, far, 0.0))
        if walls and a == 2:
            phi = torch.where((p >= 0) & (p < shape[0]), phi, 0.0)
        node, wt = node * shape[axis] + p % shape[axis], wt * phi
    return node, wt


def exact(case, seed):
    fam = case["family"]
    if fam == "lbm":
        f = _fluid(case, seed)
        for _ in range(case["steps"]):
            f = _collide(f, None, case["walls"], _lid(case), (1e-6, 0.0, 0.0))
        rho, u = _moments(f, (1e-6, 0.0, 0.0))
        return dict(f=f, rho=rho, u=u)
    steps = case["steps"] if fam != "immersed" else case["sub"] * case["cycles"]
    w = _workload(case, seed)
    if fam in ("array", "carpet") and w["n"] ** 2 * (steps + 2) > 2e10:
        return None  # the pair sums would take too long
    if fam == "helix":
        fields = _ramp_fields(case, w)
        w["field"] = fields[:1]
    M = _Model(w)
    out = {}
    if fam == "adjoint":
        leaves = dict(m_body=M.mb, field=M.field, x0=M.x0, v0=M.v0, q0=M.q0, w0=M.w0)
        for t in leaves.values():
            t.requires_grad_(True)
    S = M.begin(M.x0, M.v0, M.q0, M.w0)
    if fam == "helix":
        out = dict(x_watch=np.zeros((case["settings"], 2, 3)), ke=np.zeros((case["settings"], 1)),
                   steps=None)
        level = 0
        for k in range(case["settings"]):
            M.field = torch.as_tensor(fields[k:k + 1], device="cuda")
            for _ in range(case["steps"]):
                level += 1
                S = M.step(S, level)
            out["x_watch"][k] = S[0][:, [0, M.n - 1]].T.cpu().numpy()
            out["ke"][k] = float((0.5 * M.mass * (S[1] ** 2).sum(0) +
                                  0.5 * M.inertia * (S[3] ** 2).sum(0)).sum())
    elif fam == "immersed":
        f = _fluid(case, seed)
        shape, level = f.shape[1:], 0
        for _ in range(case["cycles"]):
            _, u = _moments(f)
            node, wt = _stencil(S[0], shape, case["walls"])
            M.fluid = (u.reshape(3, -1)[:, node] * wt).sum(1)
            g = torch.zeros_like(u).reshape(3, -1)
            for _ in range(case["sub"]):
                level += 1
                S = M.step(S, level)
                node, wt = _stencil(S[0], shape, case["walls"])
                for a in range(3):
                    g[a].index_add_(0, node.reshape(-1), (-M.pull[a] / case["sub"] * wt).reshape(-1))
            f = _collide(f, g.reshape(u.shape), case["walls"], _lid(case))
        out["f"] = f
    else:
        for level in range(1, steps + 1):
            S = M.step(S, level)
        if fam == "adjoint":
            target = torch.as_tensor(w["target"], device="cuda")
            loss = ((S[0][:, -1] - target) ** 2).sum()
            got = torch.autograd.grad(loss, list(leaves.values()))
            out["grad"] = dict(zip(leaves, got))
            S = [t.detach() for t in S]
        if fam == "carpet":
            out["energy"] = M.energies(S, steps)
    out.update(zip(STATE, S))
    return out
