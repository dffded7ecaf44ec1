"""The work that programs have this library do, as cases that can be timed and compared.

A case names an entry point (`what`), a mesh (`shape`, `n` vertices a side), a bending model, a
precision and, for the solvers, their budget:

  forces   shell_eval_forces with the energy, from positions and into forces in the caller's order
  apply    shell_hessian_apply, the operator of the implicit step, inside a caller's own solver
  step     shell_step_implicit from a saved state (positions and velocities), with or without the membrane
  batch    shell_batch_step over meshes of all six models and of log-uniform sizes
  static   shell_solve_static of a simply supported plate under a load

Meshes, material and solver settings are those of the package's synthetic workloads (the clamped plate,
the cylinder patch, the sphere cap, the batch specs, the linear plate) and of their benchmark runs; the
large steps take a fixed PCG budget per Newton iteration, as a caller with a frame time to keep sets it,
since their full solves are chaotic in the last bits.  A state starts near the rest shape, displaced and
moving in a few smooth waves drawn from the seed, and is put back before every pass, so that a pass can
be repeated.  A step returns the new positions and velocities in the caller's order, on the device: in
float64, and from a mixed-precision solver in float32, the precision in which such a caller draws or
learns from them.

`exact` is the same mathematics in float64 torch: operators from the rest mesh, forces as the gradient of
the energy, the same recurrences with the same budgets.
"""

from __future__ import annotations

import math
from collections import OrderedDict

import numpy as np
import torch

from paper_2502_10872_amd import inputs as I
from paper_2502_10872_amd import shell as S

DEV = "cuda"
F64, MIXED = S.SHELL_PREC_FP64, S.SHELL_PREC_MIXED
STATIC_MATERIAL = dict(young=2e11, poisson=0.3, thickness=0.01, density=1.0)


def listed():
    return [
        # the smallest call: one force evaluation of the 32 x 32 clamped plate, where launches count
        dict(name="forces plate 32 EP fp64", what="forces", shape="plate", n=32, model="EP", mixed=False,
             membrane=False),
        # a middle size with a side that no tile divides: edge shell and membrane together, in float64
        dict(name="forces cyl 377 ES memb fp64", what="forces", shape="cylinder", n=377, model="ES", mixed=False,
             membrane=True),
        # the benchmark's million-vertex smoothed shell in its own precision
        dict(name="forces cap 1024 SS mixed", what="forces", shape="cap", n=1024, model="SS", mixed=True,
             membrane=False),
        # the step's operator applied by a caller's own solver, a quarter of a million vertices
        dict(name="apply cap 512 SS", what="apply", shape="cap", n=512, model="SS", mixed=False, membrane=False),
        # the smallest step: the 32 x 32 plate solved to 1e-10 (one Newton iteration is exact for a plate)
        dict(name="step plate 32 EP fp64", what="step", shape="plate", n=32, model="EP", mixed=False, membrane=False,
             dt=1 / 60, newton=1, max_pcg=200, rtol=1e-10, its=34),
        # the 256 x 256 FVM cylinder at its benchmark time step, in float64
        dict(name="step cyl 256 FS fp64", what="step", shape="cylinder", n=256, model="FS", mixed=False,
             membrane=False, dt=1 / 30, newton=2, max_pcg=200, rtol=1e-4, its=400),
        # the headline mesh: a million vertices, in both precisions
        dict(name="step cap 1024 SS mixed", what="step", shape="cap", n=1024, model="SS", mixed=True, membrane=False,
             dt=1 / 30, newton=2, max_pcg=100, rtol=1e-4, its=200),
        dict(name="step cap 1024 SS fp64", what="step", shape="cap", n=1024, model="SS", mixed=False, membrane=False,
             dt=1 / 30, newton=2, max_pcg=100, rtol=1e-4, its=200),
        # with the membrane: a mesh of an interactive program, and a million vertices
        dict(name="step cyl 64 SS memb fp64", what="step", shape="cylinder", n=64, model="SS", mixed=False,
             membrane=True, dt=1 / 30, newton=2, max_pcg=50, rtol=1e-4, its=100),
        dict(name="step cyl 1024 SS memb mixed", what="step", shape="cylinder", n=1024, model="SS", mixed=True,
             membrane=True, dt=1 / 30, newton=1, max_pcg=100, rtol=1e-4, its=100),
        # a tick of the server: meshes of all models stepped together in mixed precision
        dict(name="batch 18 mixed", what="batch", count=18, most=256, pick=1, mixed=True, dt=1 / 60, newton=2,
             max_pcg=100, rtol=1e-4, its=200),
        # the linear plate benchmark: one long solve of a small system
        dict(name="static plate 65 SP fp64", what="static", shape="ring", n=65, model="SP", mixed=False,
             membrane=False, its=3400),
    ]


def draw(rng):
    what = rng.choice(["forces", "forces", "apply", "step", "step", "step", "step", "batch", "static"])

    def side(lo, hi):
        return int(round(lo * (hi / lo) ** rng.random()))

    mixed = rng.random() < 0.5
    if what == "batch":
        return dict(what=what, count=rng.randint(3, 18), most=rng.choice([96, 160, 256]), pick=rng.randint(2, 10 ** 6),
                    mixed=mixed, dt=1 / 60, newton=rng.randint(1, 2), max_pcg=rng.randint(20, 80), rtol=1e-4, its=80)
    if what == "static":
        return dict(what=what, shape="ring", n=side(12, 65), model=rng.choice(["EP", "FP", "SP"]), mixed=False,
                    membrane=False, its=1000)
    model = rng.choice(I.MODELS)
    shape = "plate" if model.endswith("P") else rng.choice(["cylinder", "cap"])
    case = dict(what=what, shape=shape, n=side(16, 1000), model=model, mixed=mixed, membrane=False)
    if what == "apply":
        return dict(case, mixed=False)
    case["membrane"] = model.endswith("S") and rng.random() < 0.4
    if what == "forces":
        return case
    if case["membrane"]:
        case["shape"] = "cylinder"
    its = rng.randint(20, 50) if case["membrane"] else rng.randint(20, 80)
    return dict(case, dt=1 / rng.choice([30, 60]), newton=rng.randint(1, 2), max_pcg=its, rtol=1e-4, its=its)


# ------------------------------------------------------------------------------------ meshes and states


def mesh_of(case):
    n, model = case["n"], case["model"]
    if case["shape"] == "plate":
        return I.plate_mesh(n, 1.0, 0.0 if n == 32 else 0.2, 7, model, "clamp_x0")
    if case["shape"] == "ring":
        return I.plate_mesh(n, 8.0, 0.2, 5, model, "ring")
    if case["shape"] == "cylinder":
        return I.workload_cylinder(n, model)
    return I.workload_sphere_cap(n, model)


def batch_meshes(case):
    g = I.rng(case["pick"])
    out = []
    for k in range(case["count"]):
        n = int(round(16 * (case["most"] / 16) ** g.uniform()))
        spec = dict(n=n, model=I.MODELS[k % 6], radius=float(g.uniform(0.3, 2.0)), seed=int(g.integers(0, 2 ** 31 - 1)))
        out.append(I.mesh_from_spec(spec, spacing=0.01))
    return out


def state_of(mesh, seed):
    """Positions and velocities [nv, 3]: a few smooth waves that vanish on the sides of the grid, some
    percent of strain at most, and up to some decimetres per second."""
    g = np.random.Generator(np.random.PCG64(seed))
    n = mesh.meta["n"]
    s = np.tile(np.linspace(0.0, 1.0, n), n)
    t = np.repeat(np.linspace(0.0, 1.0, n), n)
    side = mesh.spacing * (n - 1)
    bump = 16.0 * s * (1 - s) * t * (1 - t)
    out = []
    for amp in (0.002 * side, 0.2 * min(1.0, side)):
        u = np.zeros((mesh.nv, 3))
        for c in range(3):
            for _ in range(3):
                k, l = g.integers(1, 5, 2)
                a, b = g.uniform(0, 2 * math.pi, 2)
                u[:, c] += g.uniform(0.3, 1.0) * np.sin(2 * math.pi * k * s + a) * np.sin(2 * math.pi * l * t + b)
        out.append(amp * u * bump[:, None])
    return mesh.X + out[0], out[1]


def load_of(mesh, seed):
    """A pressure on the plate (per unit area, downwards, varying), lumped to the vertices."""
    g = np.random.Generator(np.random.PCG64(seed))
    area = np.zeros(mesh.nv)
    X, t = mesh.X, mesh.tris
    a3 = 0.5 * np.linalg.norm(np.cross(X[t[:, 1]] - X[t[:, 0]], X[t[:, 2]] - X[t[:, 0]]), axis=1)
    for c in range(3):
        np.add.at(area, t[:, c], a3 / 3.0)
    F = np.zeros((mesh.nv, 3))
    F[:, 2] = -9.81 * area * (1.0 + 0.3 * np.sin(X[:, 0] * g.uniform(0.5, 3.0)) * np.sin(X[:, 1] * g.uniform(0.5, 3.0)))
    return F


class _Raw:
    def __init__(self, ptr, shape):
        self.__cuda_array_interface__ = dict(shape=shape, typestr="<f8", data=(int(ptr), False), version=2)


class Plan:
    """What a program keeps for a mesh: its stencils, Hessian and simulation, the device views of the
    simulation's state and the order they are in (read off a state holding the vertex numbers)."""

    def __init__(self, mesh, model, material, mixed, membrane, sim):
        flags = S.SHELL_FLAG_MEMBRANE if membrane else 0
        self.mesh = mesh
        self.pb = S.Problem(mesh, material, model=model, precision=MIXED if mixed else F64, sim=sim, flags=flags)
        if sim:
            xp, vp = S.shell_sim_device_state(self.pb.sim)
            self.x = torch.as_tensor(_Raw(xp, (mesh.nv, 3)), device=DEV)
            self.v = torch.as_tensor(_Raw(vp, (mesh.nv, 3)), device=DEV)
            ids = np.repeat(np.arange(mesh.nv, dtype=np.float64)[:, None], 3, 1)
            S.shell_sim_set_state(self.pb.sim, ids, ids, 0)
            perm = self.x[:, 0].round().long()
            self.order = torch.empty_like(perm)
            self.order[perm] = torch.arange(mesh.nv, device=DEV)
            torch.cuda.synchronize()

    def snapshot(self, x, v):
        S.shell_sim_set_state(self.pb.sim, x, v, 0)
        snap = self.x.clone(), self.v.clone()
        torch.cuda.synchronize()
        return snap

    def restore(self, snap):
        self.x.copy_(snap[0])
        self.v.copy_(snap[1])

    def result(self, mixed):
        x, v = self.x[self.order], self.v[self.order]
        return (x.float(), v.float()) if mixed else (x, v)


_plans = OrderedDict()  # a program builds a mesh's plan once and steps many states on it


def plan_of(case):
    key = tuple(sorted((k, v) for k, v in case.items()
                       if k in ("what", "shape", "n", "model", "mixed", "membrane", "count", "most", "pick")))
    if key in _plans:
        _plans.move_to_end(key)
        return _plans[key]
    if case["what"] == "batch":
        plan = [Plan(m, m.model, I.MATERIAL, case["mixed"], False, True) for m in batch_meshes(case)]
        batch = S.shell_batch_create([p.pb.sim for p in plan])
        plan = (plan, batch)
    else:
        material = STATIC_MATERIAL if case["what"] == "static" else I.MATERIAL
        plan = Plan(mesh_of(case), case["model"], material, case["mixed"], case["membrane"],
                    case["what"] in ("step", "static"))
    _plans[key] = plan
    while len(_plans) > 24:
        _, old = _plans.popitem(last=False)
        if isinstance(old, tuple):
            S.shell_destroy_batch(old[1])
            old = old[0]
        for p in old if isinstance(old, list) else [old]:
            p.pb.close()
    return plan


def mass_of(mesh, material):
    """The lumped mass, as a caller's own solver holds it."""
    X, t = mesh.X, mesh.tris
    a3 = 0.5 * np.linalg.norm(np.cross(X[t[:, 1]] - X[t[:, 0]], X[t[:, 2]] - X[t[:, 0]]), axis=1)
    m = np.zeros(mesh.nv)
    for c in range(3):
        np.add.at(m, t[:, c], material["density"] * material["thickness"] * a3 / 3.0)
    return m


def prepare(case, seed):
    plan, what = plan_of(case), case["what"]
    if what == "batch":
        plans, batch = plan
        snaps = [p.snapshot(*state_of(p.mesh, seed * 1000 + k)) for k, p in enumerate(plans)]
        params, _ = S.step_params(case["dt"], gravity=I.GRAVITY, max_newton=case["newton"], max_pcg=case["max_pcg"],
                                  pcg_rtol=case["rtol"])
        return dict(what=what, plans=plans, batch=batch, snaps=snaps, params=params, mixed=case["mixed"])
    mesh = plan.mesh
    if what == "static":
        snap = plan.snapshot(mesh.X, np.zeros_like(mesh.X))
        return dict(what=what, plan=plan, snap=snap, load=load_of(mesh, seed))
    x, v = state_of(mesh, seed)
    if what == "forces":
        xd = torch.as_tensor(x, device=DEV)
        fd = torch.empty(mesh.nv, 3, device=DEV, dtype=torch.float32 if case["mixed"] else torch.float64)
        return dict(what=what, plan=plan, x=xd, f=fd, e=torch.empty(1, device=DEV, dtype=torch.float64))
    if what == "apply":
        m = torch.as_tensor(mass_of(mesh, I.MATERIAL), device=DEV)
        p = torch.as_tensor(v, device=DEV)
        return dict(what=what, plan=plan, m=m, p=p, q=torch.empty_like(p))
    params, _ = S.step_params(case["dt"], gravity=I.GRAVITY, max_newton=case["newton"], max_pcg=case["max_pcg"],
                              pcg_rtol=case["rtol"])
    return dict(what=what, plan=plan, snap=plan.snapshot(x, v), params=params, mixed=case["mixed"])


def run(s):
    what = s["what"]
    if what == "forces":
        S.shell_eval_forces(s["plan"].pb.st, s["x"], s["f"], s["e"])
        return s["f"], s["e"]
    if what == "apply":
        S.shell_hessian_apply(s["plan"].pb.h, s["m"], 1.0 / 900.0, s["p"], s["q"])
        return s["q"]
    if what == "batch":
        for p, snap in zip(s["plans"], s["snaps"]):
            p.restore(snap)
        S.shell_batch_step(s["batch"], s["params"], len(s["plans"]))
        return [p.result(s["mixed"]) for p in s["plans"]]
    s["plan"].restore(s["snap"])
    if what == "static":
        S.shell_solve_static(s["plan"].pb.sim, s["load"], max_newton=1, pcg_rtol=1e-10)
        return s["plan"].result(False)[0]
    S.shell_step_implicit(s["plan"].pb.sim, s["params"])
    return s["plan"].result(s["mixed"])


def work(case):
    """Forces: the stencil records and the vertices once.  Solvers: the matrix once per PCG iteration (a
    value and a 16-bit column id per entry) and the state once."""
    real = 4 if case["mixed"] else 8

    def matrix(nv, model, membrane):
        nnz = (13 if model[0] == "E" else 19) * nv
        bytes_, flops = nnz * (real + 2), 6 * nnz
        return (bytes_ + 7 * nv * (9 * real + 2), flops + 126 * nv) if membrane else (bytes_, flops)

    if case["what"] == "batch":
        g = I.rng(case["pick"])
        b = f = 0
        for k in range(case["count"]):
            n = int(round(16 * (case["most"] / 16) ** g.uniform()))
            g.uniform(), g.integers(0, 2 ** 31 - 1)
            mb, mf = matrix(n * n, I.MODELS[k % 6], False)
            b, f = b + case["its"] * mb + 96 * n * n, f + case["its"] * mf
        return dict(bytes=b, flops=f)
    nv, model = case["n"] ** 2, case["model"]
    if case["what"] == "forces":
        k, r, ns = (4, 1, 3 * nv) if model[0] == "E" else (6, 3, 2 * nv)
        shell = model.endswith("S")
        b = ns * (4 * k + real * r * (k - 1 if case["mixed"] else k) + (8 * r if shell else 0)) + nv * (24 + 3 * real)
        f = ns * (60 if k == 4 else 260)
        if case["membrane"]:
            b, f = b + 2 * nv * 52, f + 2 * nv * 120
        return dict(bytes=b, flops=f)
    mb, mf = matrix(nv, model, case["membrane"])
    if case["what"] == "apply":
        return dict(bytes=mb + 56 * nv, flops=mf)
    return dict(bytes=case["its"] * mb + 96 * nv, flops=case["its"] * mf)


# ------------------------------------------------------------------------------------ in 64 bits


class Exact:
    """Bending (and membrane) energy, forces and step of one mesh in float64 torch."""

    def __init__(self, mesh, model, material, membrane):
        self.dev = DEV if torch.cuda.is_available() else "cpu"
        self.X, self.nv = torch.as_tensor(mesh.X, device=self.dev), mesh.nv
        self.shell = model.endswith("S")
        E, nu, h = material["young"], material["poisson"], material["thickness"]
        self.kb, self.nu = E * h ** 3 / (12 * (1 - nu * nu)), nu
        t = np.asarray(mesh.tris, dtype=np.int64)
        self.free = torch.as_tensor(np.asarray(mesh.pinned) == 0, device=self.dev)
        self.mass = torch.as_tensor(mass_of(mesh, material), device=self.dev)
        idx, miss = self._stencils(t, model)
        self.idx = torch.as_tensor(idx, device=self.dev)
        if model[0] == "E":
            B = self._edge_operator()
            self.D = torch.ones(1, 1, dtype=torch.float64, device=self.dev)
        else:
            B = self._tri_operator(torch.as_tensor(miss, device=self.dev), model[0] == "F")
            tt = 0.5 * (1 - nu)
            self.D = self.kb * torch.tensor([[1, nu, 0], [nu, 1, 0], [0, 0, tt]], dtype=torch.float64, device=self.dev)
        self.B = B
        self.k0 = ((B @ self._local(self.X)) * self._normal(self.X)[:, None]).sum(-1) if self.shell else None
        self.G = B.transpose(1, 2) @ (self.D @ B)
        self.kdiag = torch.zeros(self.nv, dtype=torch.float64, device=self.dev)
        self.kdiag.index_add_(0, self.idx.reshape(-1), torch.diagonal(self.G, dim1=1, dim2=2).reshape(-1))
        # a missing flap's id repeats vertex 1 with a zero column, so no cross terms fall on the diagonal
        self.membrane = membrane
        if membrane:
            self.t = torch.as_tensor(t, device=self.dev)
            x0, x1, x2 = (self.X[self.t[:, c]] for c in range(3))
            a, b = x1 - x0, x2 - x0
            n = torch.linalg.cross(a, b)
            two_a = n.norm(dim=1)
            e1 = a / a.norm(dim=1, keepdim=True)
            e2 = torch.linalg.cross(n / two_a[:, None], e1)
            Dm = torch.stack([torch.stack([(a * e1).sum(1), (b * e1).sum(1)], 1),
                              torch.stack([(a * e2).sum(1), (b * e2).sum(1)], 1)], 1)
            self.Gm, self.A = torch.linalg.inv(Dm), 0.5 * two_a
            c = E * h / (1 - nu * nu)
            self.Dm = c * torch.tensor([[1, nu, 0], [nu, 1, 0], [0, 0, 0.5 * (1 - nu)]], dtype=torch.float64,
                                       device=self.dev)

    def _stencils(self, t, model):
        m = len(t)
        base = self.nv
        frm = np.concatenate([t[:, 0], t[:, 1], t[:, 2]])
        to = np.concatenate([t[:, 1], t[:, 2], t[:, 0]])
        opp = np.concatenate([t[:, 2], t[:, 0], t[:, 1]])
        key = frm * base + to
        order = np.argsort(key, kind="stable")
        ks = key[order]

        def across(a, b):  # the vertex opposite the directed edge a -> b, -1 without a triangle there
            q = a * base + b
            at = np.minimum(np.searchsorted(ks, q), 3 * m - 1)
            return np.where(ks[at] == q, opp[order[at]], -1)

        if model[0] == "E":
            other = across(to, frm)
            keep = (other >= 0) & (frm < to)
            return np.stack([opp[keep], frm[keep], to[keep], other[keep]], 1), None
        flaps = np.stack([across(t[:, (i + 2) % 3], t[:, (i + 1) % 3]) for i in range(3)], 1)
        return np.concatenate([t, np.where(flaps < 0, t[:, :1], flaps)], 1), flaps < 0

    def _local(self, x):
        g = x[self.idx]
        return g - g[:, (1 if self.idx.shape[1] == 4 else 0)][:, None]

    def _normal(self, x):
        d = self._local(x)
        if self.idx.shape[1] == 4:
            ua, ub = torch.linalg.cross(d[:, 2], d[:, 0]), torch.linalg.cross(d[:, 3], d[:, 2])
            n = ua / ua.norm(dim=1, keepdim=True) + ub / ub.norm(dim=1, keepdim=True)
        else:
            n = torch.linalg.cross(d[:, 1], d[:, 2])
        return n / n.norm(dim=1, keepdim=True)

    def _edge_operator(self):
        d, n = self._local(self.X), self._normal(self.X)
        la = torch.linalg.cross(d[:, 2], d[:, 0]).norm(dim=1)
        lb = torch.linalg.cross(d[:, 3], d[:, 2]).norm(dim=1)
        a, e, b = (v - (v * n).sum(1, keepdim=True) * n for v in (d[:, 0], d[:, 2], d[:, 3]))
        ee = (e * e).sum(1)
        sp, sq = (a * e).sum(1) / ee, (b * e).sum(1) / ee
        h1, h4 = (a - sp[:, None] * e).norm(dim=1), (b - sq[:, None] * e).norm(dim=1)
        L = torch.stack([1 / h1, -((1 - sp) / h1 + (1 - sq) / h4), -(sp / h1 + sq / h4), 1 / h4], 1)
        return (L * (2 / (h1 + h4) * torch.sqrt(self.kb * 0.5 * (la + lb)))[:, None])[:, None]

    def _tri_operator(self, miss, fvm):
        d = self._local(self.X)
        ns = len(d)
        u = torch.linalg.cross(d[:, 1], d[:, 2])
        two_a = u.norm(dim=1)
        ez = u / two_a[:, None]
        ex = d[:, 1] / d[:, 1].norm(dim=1, keepdim=True)
        ey = torch.linalg.cross(ez, ex)
        P = torch.stack([(d * ex[:, None]).sum(2), (d * ey[:, None]).sum(2)], 2)
        for i in range(3):
            P[:, i + 3] = torch.where(miss[:, i, None], P[:, (i + 1) % 3] + P[:, (i + 2) % 3] - P[:, i], P[:, i + 3])
        L = torch.zeros(ns, 3, 6, dtype=torch.float64, device=self.dev)
        R = torch.zeros(ns, 3, 3, dtype=torch.float64, device=self.dev)
        for i in range(3):
            a, b, f = (i + 1) % 3, (i + 2) % 3, i + 3
            e, w, g = P[:, b] - P[:, a], P[:, i] - P[:, a], P[:, f] - P[:, a]
            ee = (e * e).sum(1)
            st, sf = (w * e).sum(1) / ee, (g * e).sum(1) / ee
            ht, hf = (w - st[:, None] * e).norm(dim=1), (g - sf[:, None] * e).norm(dim=1)
            c = 2 / (ht + hf)
            L[:, i, i], L[:, i, f] = c / ht, c / hf
            L[:, i, a] = -c * ((1 - st) / ht + (1 - sf) / hf)
            L[:, i, b] = -c * (st / ht + sf / hf)
            m = torch.stack([e[:, 1], -e[:, 0]], 1) / ee.sqrt()[:, None]
            R[:, 0, i], R[:, 1, i], R[:, 2, i] = m[:, 0] ** 2, m[:, 1] ** 2, 2 * m[:, 0] * m[:, 1]
        if fvm:
            B = R @ L
        else:
            C = torch.stack([0.5 * P[..., 0] ** 2, 0.5 * P[..., 1] ** 2, 0.5 * P[..., 0] * P[..., 1]], 2)
            B = torch.linalg.solve(L @ C, L)
        for i in range(3):
            w = torch.where(miss[:, i, None], B[:, :, i + 3], torch.zeros_like(B[:, :, 0]))
            B[:, :, (i + 1) % 3] += w
            B[:, :, (i + 2) % 3] += w
            B[:, :, i] -= w
            B[:, :, i + 3] -= w
        if fvm:  # a free edge keeps the curvatures along and across it only (the first one decides)
            done = torch.zeros(ns, dtype=torch.bool, device=self.dev)
            for i in range(3):
                e = P[:, (i + 2) % 3] - P[:, (i + 1) % 3]
                c, s = (e / e.norm(dim=1, keepdim=True)).unbind(1)
                T = torch.stack([torch.stack([c * c, s * s, c * s], 1), torch.stack([s * s, c * c, -c * s], 1)], 1)
                Q = torch.stack([torch.stack([c * c, s * s, 2 * c * s], 1),
                                 torch.stack([s * s, c * c, -2 * c * s], 1)], 2)
                now = miss[:, i] & ~done
                B = torch.where(now[:, None, None], Q @ (T @ B), B)
                done |= miss[:, i]
        return B * torch.sqrt(0.5 * two_a)[:, None, None]

    def energy(self, x):
        C = self.B @ self._local(x)
        if self.shell:
            C = ((C * self._normal(x)[:, None]).sum(2) - self.k0)[:, :, None]
        e = 0.5 * (C * (self.D @ C)).sum()
        if self.membrane:
            F = self._F(x)
            Cg = F.transpose(1, 2) @ F
            eps = torch.stack([0.5 * (Cg[:, 0, 0] - 1), 0.5 * (Cg[:, 1, 1] - 1), Cg[:, 0, 1]], 1)
            e = e + 0.5 * (self.A * (eps * (eps @ self.Dm)).sum(1)).sum()
        return e

    def _F(self, x):
        x0, x1, x2 = (x[self.t[:, c]] for c in range(3))
        return torch.stack([x1 - x0, x2 - x0], 2) @ self.Gm

    def force(self, x):
        x = x.detach().requires_grad_(True)
        e = self.energy(x)
        (g,) = torch.autograd.grad(e, x)
        return -g, e.detach()

    def K(self, p):
        out = torch.zeros_like(p)
        return out.index_add_(0, self.idx.reshape(-1), (self.G @ p[self.idx]).reshape(-1, 3))

    def K_dense(self):
        k = self.idx.shape[1]
        out = torch.zeros(self.nv * self.nv, dtype=torch.float64, device=self.dev)
        at = self.idx[:, :, None] * self.nv + self.idx[:, None, :]
        return out.index_add_(0, at.reshape(-1), self.G.reshape(-1, k * k).reshape(-1)).reshape(self.nv, self.nv)

    def tangent(self, x):
        """The membrane's element matrices [nt, 9, 9] (row 3 a + coordinate): Gauss-Newton part and the
        positive part of the stress."""
        F = self._F(x)
        g = torch.stack([-self.Gm[:, 0] - self.Gm[:, 1], self.Gm[:, 0], self.Gm[:, 1]], 1)
        Bm = torch.stack([g[:, :, None, 0] * F[:, None, :, 0], g[:, :, None, 1] * F[:, None, :, 1],
                          g[:, :, None, 1] * F[:, None, :, 0] + g[:, :, None, 0] * F[:, None, :, 1]], 3).reshape(-1, 9, 3)
        Cg = F.transpose(1, 2) @ F
        eps = torch.stack([0.5 * (Cg[:, 0, 0] - 1), 0.5 * (Cg[:, 1, 1] - 1), Cg[:, 0, 1]], 1)
        s = eps @ self.Dm
        w, V = torch.linalg.eigh(torch.stack([torch.stack([s[:, 0], s[:, 2]], 1), torch.stack([s[:, 2], s[:, 1]], 1)], 1))
        Sp = V @ (w.clamp(min=0)[:, :, None] * V.transpose(1, 2))
        K = self.A[:, None, None] * (Bm @ self.Dm @ Bm.transpose(1, 2))
        gsg = self.A[:, None, None] * (g @ Sp @ g.transpose(1, 2))
        for c in range(3):
            K[:, c::3, c::3] += gsg
        return K

    def step(self, x, v, case):
        dt = case["dt"]
        dt2, free = dt * dt, self.free[:, None].double()
        grav = torch.tensor(I.GRAVITY, dtype=torch.float64, device=self.dev)
        xt, mass = x.clone(), self.mass[:, None]
        xhat = x + free * (dt * v + dt2 * grav)
        x = xhat.clone()
        f, e = self.force(x)
        E0 = 0.5 * (mass * (x - xhat) ** 2).sum() + dt2 * e
        first = None
        for k in range(case["newton"] + 1):
            g = free * (mass * (x - xhat) - dt2 * f)
            gn = float(g.norm())
            first = gn if first is None else first
            if k == case["newton"] or gn == 0.0 or (k > 0 and gn <= 1e-8 * first):
                break
            diag, Km, cols = self.kdiag, None, slice(None)
            if self.membrane:
                Km = self.tangent(x)
                tr = torch.diagonal(Km, dim1=1, dim2=2).reshape(-1, 3, 3).sum(2) / 3
                diag = diag + torch.zeros_like(diag).index_add_(0, self.t.reshape(-1), tr.reshape(-1))

            def A(p):
                q = mass * p + dt2 * self.K(p)
                if Km is not None:
                    el = (Km @ p[self.t].reshape(-1, 9, 1)).reshape(-1, 3)
                    q = q + dt2 * torch.zeros_like(p).index_add_(0, self.t.reshape(-1), el)
                return free * q

            y = self.pcg(A, -g, self.free[:, None] / (self.mass + dt2 * diag)[:, None], case, Km is not None)
            if Km is None:
                x = x + y
                f, _ = self.force(x)
                continue
            slope, a = float((g * y).sum()), 1.0
            for halved in range(7):
                xn = x + a * y
                f, e = self.force(xn)
                En = 0.5 * (mass * (xn - xhat) ** 2).sum() + dt2 * e
                if En <= E0 + 1e-4 * a * slope or halved == 6:
                    break
                a *= 0.5
            x, E0 = xn, En
        return x, (x - xt) / dt

    def pcg(self, A, b, dinv, case, coupled):
        """Jacobi PCG with the case's budget, a recurrence per coordinate (or one, coupled); a solve that
        runs to a tolerance of 1e-10 is taken to the limit of float64 instead."""
        tight = case["rtol"] <= 1e-9
        rtol, most = (1e-14, 20 * case["max_pcg"]) if tight else (case["rtol"], case["max_pcg"])

        def dot(a, c):
            s = (a * c).sum(0)
            return s.sum().expand(3) if coupled else s

        y, r = torch.zeros_like(b), b.clone()
        z = dinv * r
        p, rz, rr = z.clone(), dot(r, z), dot(r, r)
        tol = rtol * rtol * rr
        on = rr > tol
        for it in range(most):
            if it % 10 == 0 and not bool(on.any()):
                break
            q = A(p)
            pq = dot(p, q)
            al = torch.where(on & (pq != 0), rz / pq, torch.zeros_like(rz))
            y, r = y + al * p, r - al * q
            z = dinv * r
            rzn, rr = dot(r, z), dot(r, r)
            be = torch.where(on & (rz != 0), rzn / rz, torch.zeros_like(rz))
            rz = torch.where(on, rzn, rz)
            p = z + be * p
            on = on & (rr > tol)
        return y


def exact(case, seed):
    what = case["what"]
    if what == "batch":
        if case["count"] * case["its"] > 4000:
            return None
        out = []
        for k, m in enumerate(batch_meshes(case)):
            ex = Exact(m, m.model, I.MATERIAL, False)
            x, v = (torch.as_tensor(a, device=ex.dev) for a in state_of(m, seed * 1000 + k))
            out.append(ex.step(x, v, case))
        return out
    mesh = mesh_of(case)
    ex = Exact(mesh, case["model"], STATIC_MATERIAL if what == "static" else I.MATERIAL, case["membrane"])
    if what == "static":
        F = torch.as_tensor(load_of(mesh, seed), device=ex.dev)
        K = ex.K_dense()
        u = torch.zeros_like(F)
        u[ex.free] = torch.linalg.solve(K[ex.free][:, ex.free], F[ex.free])
        return ex.X + u
    x, v = (torch.as_tensor(a, device=ex.dev) for a in state_of(mesh, seed))
    if what == "forces":
        f, e = ex.force(x)
        return f, e.reshape(1)
    if what == "apply":
        return ex.mass[:, None] * v + ex.K(v) / 900.0
    return ex.step(x, v, case)
