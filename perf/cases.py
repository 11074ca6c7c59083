"""Measured cases of the joint piston-gap solver: what a program built on it has it do, through
its public entry points, from the smallest single-condition solve to the 2048 x 1024 joint one.

Kinds (``case["kind"]``):

* ``step``     one hot-path pass: assemble the conditions, PCG solve, force integration and, for
               nine conditions, the finite-difference Jacobian
* ``picard``   one time point of the equilibrium iteration: a cold general-iteration step and a
               warm-started one (``dynamics.equilibrium``)
* ``adjoint``  the base solve and its four adjoint solves in one joint solve (``solve_with_adjoint``)
* ``vjp``      forward and backward of the differentiable force (``autograd.gap_force``)
* ``batch``    three requests of different grids advancing together in one ``gap_batch``
* ``film``     everything around the solve on a given pressure field: assembly, the assembled base
               system, forces, the pressure / shear split and the rebuilt field, with the clamp

Inputs follow the repository's synthetic workloads (``synth``): gap geometry, eccentricities up
to half the clearance, dimples of 5 to 15 um, finite-difference steps of 1e-3 of each scale.
``exact`` computes the same outputs in 64 bits with plain torch: conductances, sources and
forces from their formulas, systems solved by conjugate gradients to stagnation.
"""

import math

import numpy as np
import torch

DEVICE = "cuda:0"
R, L, C, MU = 10e-3, 40e-3, 20e-6, 0.04
U = 2.0 * math.pi * 2000.0 / 60.0 * R
P_IN, P_OUT, P_CAV = 10e6, 0.1e6, 0.0
RATE = 1e-3
DELTA = [1e-3 * C] * 4 + [1e-3 * RATE] * 4
DT = 1e-4


def _step(name, nt, nz, n_cond=9, texture="dimples", eps=1e-10, precond="assor2", neumann=1, scalars="global"):
    return dict(name=name, kind="step", n_theta=nt, n_axial=nz, n_cond=n_cond, texture=texture, eps=eps,
                precond=precond, neumann=neumann, scalars=scalars)


def listed():
    return [
        # the smallest call: one smooth condition on the 64 x 32 grid, all latency
        _step("step_64x32_one_condition", 64, 32, n_cond=1, texture="smooth"),
        # the smallest request size of the served stream, nine conditions
        _step("step_128x64", 128, 64, texture="smooth"),
        # one time point of a dynamics run on an odd, ragged grid
        dict(name="picard_251x97", kind="picard", n_theta=251, n_axial=97, texture="dimples", eps=1e-10),
        # the paper's smaller mesh at its tolerance, with its Jacobi baseline
        _step("step_400x360_jacobi", 400, 360, eps=1e-6, precond="jacobi"),
        # the joint smooth workload
        _step("step_512x256", 512, 256, texture="smooth"),
        # the paper's larger mesh at its tolerance, a pocket texture given as a sampled field
        _step("step_800x760_pockets", 800, 760, eps=1e-6, texture="pockets"),
        # a Neumann order above the paper's, one recurrence per condition
        _step("step_1024x512_order2", 1024, 512, neumann=2, scalars="per_cond"),
        # the headline joint textured workload
        _step("step_2048x1024", 2048, 1024),
        # the adjoint workload: base and adjoint systems together, the adjoint ones at 1e-7
        dict(name="adjoint_1024x512", kind="adjoint", n_theta=1024, n_axial=512, texture="dimples", eps=1e-10),
        # a differentiable force in a torch program, forward and backward, one condition
        dict(name="vjp_512x256", kind="vjp", n_theta=512, n_axial=256, texture="smooth", eps=1e-10),
        # three served requests of different sizes advancing together
        dict(name="batch_128_256_512", kind="batch", n_theta=512, n_axial=256, texture="dimples", eps=1e-10),
        # the one-off passes around a large solve
        dict(name="film_2048x1024", kind="film", n_theta=2048, n_axial=1024, texture="dimples", eps=1e-10),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# widest ring drawn of each kind, so that no drawn case costs more than the listed 2048 x 1024 step
_DRAW_MAX = {"step": 1600, "picard": 800, "adjoint": 1200, "vjp": 1600, "batch": 640, "film": 2048}


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "picard", "adjoint", "vjp", "batch", "film"])
    nt = _log_int(rng, 48, _DRAW_MAX[kind])
    nz = max(20, int(round(nt * rng.uniform(0.3, 0.95))))
    texture = rng.choice(["smooth", "dimples", "dimples", "pockets"])
    if kind != "step":
        return dict(kind=kind, n_theta=nt, n_axial=nz, texture="dimples" if texture == "pockets" else texture,
                    eps=1e-10)
    case = _step("", nt, nz, n_cond=rng.choice([1, 9, 9, 9]), texture=texture, eps=rng.choice([1e-6, 1e-10, 1e-10]),
                 precond=rng.choice(["assor2", "assor2", "assor2", "jacobi"]),
                 scalars=rng.choice(["global", "global", "per_cond"]))
    if case["precond"] == "assor2":
        case["neumann"] = rng.choice([1, 1, 2])
    del case["name"]
    return case


# ---- inputs ------------------------------------------------------------------------------

def _state(rng):
    return rng.uniform(-0.5 * C, 0.5 * C, 4), rng.uniform(-RATE, RATE, 4)


def _dimples(rng):
    """20 x 8 spherical caps over the middle of the gap, depths U(5, 15) um."""
    th = (np.arange(20) + 0.5) * 2.0 * math.pi / 20
    z = 0.2 * L + (np.arange(8) + 0.5) * 0.6 * L / 8
    TH, Z = np.meshgrid(th, z)
    return TH.ravel(), Z.ravel(), np.full(160, 0.5e-3), rng.uniform(5e-6, 15e-6, 160)


def _pocket_depth(depth, th, z):
    """60 x 10 flat pockets with half-cosine edges."""
    def plateau(x, half):
        t = torch.clamp((x.abs() - 0.7 * half) / (0.3 * half), 0.0, 1.0)
        return 0.5 * (1.0 + torch.cos(math.pi * t))

    pitch = 2.0 * math.pi / 60
    dth = torch.remainder(th, pitch) - 0.5 * pitch
    m = torch.clamp(torch.floor((z - 2e-3) / 1e-3), 0, 9)
    dz = z - (2e-3 + (m + 0.5) * 1e-3)
    return depth * plateau(dth, 0.25 * pitch) * plateau(dz, 0.25e-3)


def _points(nt, nz):
    """Angles of centres and east faces (row vectors), axial positions of centres and faces (columns)."""
    i = torch.arange(nt, dtype=torch.float64, device=DEVICE)
    dth, dz = 2.0 * math.pi / nt, L / nz
    zc = (torch.arange(nz, dtype=torch.float64, device=DEVICE) + 0.5) * dz
    zf = torch.arange(nz + 1, dtype=torch.float64, device=DEVICE) * dz
    return (i + 0.5)[None] * dth, (i + 1.0)[None] * dth, zc[:, None], zf[:, None]


def _texture(case, rng):
    """(dimple list or None, depth function of (theta, z) or None)."""
    if case["texture"] == "dimples":
        return _dimples(rng), None
    if case["texture"] == "pockets":
        depth = float(rng.uniform(10e-6, 20e-6))
        return None, lambda th, z: _pocket_depth(depth, th, z)
    return None, None


def _depth(dimples, field):
    """The texture as a depth function of broadcast (theta, z) tensors."""
    if field is not None:
        return field

    def caps(th, z):
        th, z = torch.broadcast_tensors(th, z)
        out = torch.zeros(th.shape, dtype=torch.float64, device=DEVICE)
        if dimples is None:
            return out
        for tc, zc, a, d in zip(*dimples):
            rows = torch.nonzero((z[:, 0] - zc).abs() < a).flatten()
            if rows.numel() == 0:
                continue
            r0, r1 = int(rows[0]), int(rows[-1]) + 1
            dth = torch.remainder(th[r0:r1] - tc + math.pi, 2.0 * math.pi) - math.pi
            r2 = (R * dth) ** 2 + (z[r0:r1] - zc) ** 2
            rho = (a * a + d * d) / (2.0 * d)
            cap = torch.sqrt(torch.clamp(rho * rho - r2, min=0.0)) - (rho - d)
            out[r0:r1] = torch.maximum(out[r0:r1], torch.where(r2 < a * a, cap, 0.0))
        return out

    return caps


def _solver(case, nt, nz, dimples, field, max_cond):
    from paper_2511_06824_amd.solver import JointGapSolver
    planes = None
    if field is not None:
        tc, te, zc, zf = _points(nt, nz)
        planes = [field(tc, zc).contiguous(), field(te, zc).contiguous(), field(tc, zf).contiguous()]
    return JointGapSolver(R, C, L, MU, U, 0.0, P_IN, P_OUT, nt, nz, dimples=dimples, max_cond=max_cond,
                          device=DEVICE, texture=planes)


def _omega(case):
    return 1.8 if case["texture"] == "smooth" else 1.6


def _batch_grids(case):
    nt, nz = case["n_theta"], case["n_axial"]
    return [(max(16, nt // d), max(12, nz // d)) for d in (4, 2, 1)]


def _load(seed):
    rng = np.random.default_rng(seed + 77)
    F_ext = np.array([rng.uniform(-20.0, 20.0), rng.uniform(-20.0, 20.0), rng.uniform(-0.1, 0.1),
                      rng.uniform(-0.1, 0.1)])
    m, inertia = 0.154, 0.128 * L ** 2 / 12.0
    M = np.zeros((4, 4))
    M[0, 0] = M[0, 2] = M[1, 1] = M[1, 3] = 0.5 * m
    M[2, 1], M[2, 3], M[3, 0], M[3, 2] = inertia / L, -inertia / L, -inertia / L, inertia / L
    return F_ext, M


def _field_input(nt, nz, seed):
    """A pressure field for the passes around the solve: the linear drop with smooth waves, some of it below zero."""
    rng = np.random.default_rng(seed + 5)
    tc, _, zc, _ = _points(nt, nz)
    out = []
    for _ in range(9):
        a, b, f = rng.uniform(0.2, 0.6), rng.uniform(0, 2 * math.pi), int(rng.integers(1, 4))
        base = P_IN + (P_OUT - P_IN) * zc / L
        out.append(base + a * P_IN * torch.sin(f * tc + b) * torch.sin(math.pi * zc / L))
    return torch.stack(out)


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    kind, nt, nz = case["kind"], case["n_theta"], case["n_axial"]
    st = {"case": case}
    if kind == "batch":
        from paper_2511_06824_amd import gapsolve as G
        st["requests"] = []
        for k, (a, b) in enumerate(_batch_grids(case)):
            e, ed = _state(rng)
            dim = _dimples(rng) if (k % 2 == 1 and case["texture"] != "smooth") else None
            s = _solver(case, a, b, dim, None, 9)
            st["requests"].append((s, e, ed, s.options(omega=1.6, eps=case["eps"])))
        st["batch"] = _Batch(G)
        return st
    e, ed = _state(rng)
    dimples, field = _texture(case, rng)
    one = kind == "vjp" or case.get("n_cond") == 1
    s = _solver(case, nt, nz, dimples, field, 1 if one else 9)
    st.update(solver=s, e=e, ed=ed)
    if kind == "step":
        from paper_2511_06824_amd import gapsolve as G
        st["opts"] = s.options(omega=_omega(case), eps=case["eps"], neumann=case["neumann"],
                               precond=G.GAP_PRECOND_JACOBI if case["precond"] == "jacobi" else G.GAP_PRECOND_ASSOR2,
                               scalars=G.GAP_SCALARS_PER_COND if case["scalars"] == "per_cond" else
                               G.GAP_SCALARS_GLOBAL)
    elif kind == "adjoint":
        st["opts"] = s.options(omega=_omega(case), eps=case["eps"], eps_adjoint=1e-7)
    elif kind == "vjp":
        st["opts"] = s.options(omega=_omega(case), eps=case["eps"])
        st["te"] = torch.tensor(e, dtype=torch.float64, requires_grad=True)
        st["ted"] = torch.tensor(ed, dtype=torch.float64, requires_grad=True)
        st["w"] = torch.tensor([1.0, -0.5, 20.0, 30.0], dtype=torch.float64)
    elif kind == "picard":
        st["F_ext"], st["mass"] = _load(seed)
        st["opts"] = s.options(omega=_omega(case), eps=case["eps"])
    elif kind == "film":
        st["p"] = _field_input(nt, nz, seed).contiguous()
    return st


class _Batch:
    """The batch handle a serving program keeps."""

    def __init__(self, G):
        self.G, self.handle = G, G.gap_batch_create()

    def __del__(self):
        try:
            self.G.gap_batch_destroy(self.handle)
        except Exception:
            pass


def run(st):
    kind = st["case"]["kind"]
    if kind == "batch":
        return _run_batch(st)
    s = st["solver"]
    if kind == "step":
        if s.max_cond == 1:
            s.assemble(st["e"], st["ed"], None, 1)
            p, _ = s.solve(st["opts"])
            return {"p": p, "F": s.integrate()}
        F, J, _ = s.step(st["e"], st["ed"], DELTA, st["opts"])
        return {"p": s.pressure(), "F": F, "J": J}
    if kind == "picard":
        from paper_2511_06824_amd import dynamics
        e, ed, _, _ = dynamics.equilibrium(s, st["e"], st["ed"], DT, st["F_ext"], st["mass"], DELTA, tol=0.0,
                                           max_picard=2, opts=st["opts"])
        return {"e": e, "edot": ed, "p": s.p.view(9, s.n_axial, s.n_theta)}
    if kind == "adjoint":
        s.assemble(st["e"], st["ed"], None, 1)
        p, J, _ = s.solve_with_adjoint(st["opts"])
        return {"p": p, "J": J, "F": s.integrate()}
    if kind == "vjp":
        from paper_2511_06824_amd.autograd import gap_force
        st["te"].grad = st["ted"].grad = None
        F = gap_force(st["te"], st["ted"], s, st["opts"])
        (F * st["w"]).sum().backward()
        return {"F": F.detach(), "ge": st["te"].grad, "ged": st["ted"].grad, "p": s.pressure()}
    if kind == "film":
        from paper_2511_06824_amd import gapsolve as G
        s.assemble(st["e"], st["ed"], DELTA, 9)
        kx, kz, S = s.read_system(0)
        kw = dict(cavitation=G.GAP_CAVITATION_CLAMP, p_cav=P_CAV, p=st["p"])
        return {"kx": kx, "kz": kz, "S": S, "F": s.integrate(**kw), "split": s.integrate_split(**kw),
                "full": s.full_pressure(**kw)}
    raise ValueError(kind)


def _run_batch(st):
    from paper_2511_06824_amd import gapsolve as G
    b = st["batch"].handle
    stream = torch.cuda.current_stream().cuda_stream
    live = {}
    for s, e, ed, opts in st["requests"]:
        s.assemble(e, ed, DELTA, 9)
        live[G.gap_batch_add(b, s.handle, opts, s.p.data_ptr(), stream)] = s
    while live:
        G.gap_batch_step(b, 32, True, stream)
        for rid in G.gap_batch_poll(b):
            G.gap_batch_remove(b, rid, stream)
            live.pop(rid)
    out = []
    for s, _, _, _ in st["requests"]:
        F = s.integrate()
        out.append({"p": s.pressure(), "F": F, "J": s.jacobian_fd()})
    return out


# ---- work --------------------------------------------------------------------------------

def _solve_work(nt, nz, n_cond, n_op, eps, precond="assor2", neumann=1):
    """One PCG solve.  Iterations: about 0.195 decades^-1 sqrt(condition number) with ASSOR II of
    order 1.  Operations per condition-DOF and iteration: matrix product 9, updates and sums 16,
    preconditioner 1 (Jacobi) or 13 per order.  Bytes: texture read and pressure written once; where
    r, u and the conductances (16 B a condition-DOF, 16 B an operator-DOF) exceed what 256 CUs hold in
    registers and LDS (168 MB), they are read and r, u written each iteration, the pressure every other one."""
    n = nt * nz
    it = 0.195 * -math.log10(eps) * math.hypot(2.0 / math.pi * nt, nz)
    it *= 1.9 if precond == "jacobi" else {1: 1.0, 2: 0.69}[neumann]
    flops = it * n * n_cond * (25.0 + (1.0 if precond == "jacobi" else 13.0 * neumann))
    once = 24.0 * n + 8.0 * n * n_cond
    if 16.0 * n * (n_cond + n_op) > 168e6:
        once += it * n * (40.0 * n_cond + 16.0 * n_op)
    return once, flops


def work(case):
    kind, nt, nz, eps = case["kind"], case["n_theta"], case["n_axial"], case["eps"]
    n = nt * nz
    if kind == "step":
        nc = case["n_cond"]
        b, f = _solve_work(nt, nz, nc, 5 if nc == 9 else 1, eps, case["precond"], case["neumann"])
        f += 150.0 * n * nc
    elif kind == "picard":
        b, f = _solve_work(nt, nz, 9, 5, eps)
        b, f = 2.0 * b, 1.6 * f
    elif kind == "adjoint":
        b, f = _solve_work(nt, nz, 5, 1, eps)
    elif kind == "vjp":
        b, f = _solve_work(nt, nz, 1, 1, eps)
        b, f = 2.0 * b, 2.0 * f
    elif kind == "batch":
        parts = [_solve_work(a, c, 9, 5, eps) for a, c in _batch_grids(case)]
        b, f = sum(p[0] for p in parts), sum(p[1] for p in parts)
    else:
        # texture in, five operators and nine sources out, the base system copied, the pressure read
        # for the forces and the field, the field out
        b = 8.0 * n * (3 + 2 * 5 + 9 + 6 + 9 + 9)
        f = n * 9.0 * (120.0 + 40.0 + 60.0)
    return {"bytes": b, "flops": f}


# ---- exact values in 64 bits ---------------------------------------------------------------

def _film(e, th, z):
    Rc, t = R + C, z / L
    ex, ey = e[0] + (e[2] - e[0]) * t, e[1] + (e[3] - e[1]) * t
    q = C * (2.0 * R + C) - 2.0 * Rc * (ex * torch.cos(th) + ey * torch.sin(th)) + ex * ex + ey * ey
    return q / (torch.sqrt(R * R + q) + R)


def _film_rate(e, ed, th, z):
    Rc, t = R + C, z / L
    ex, ey = e[0] + (e[2] - e[0]) * t, e[1] + (e[3] - e[1]) * t
    exd, eyd = ed[0] + (ed[2] - ed[0]) * t, ed[1] + (ed[3] - ed[1]) * t
    ax, ay = Rc * torch.cos(th) - ex, Rc * torch.sin(th) - ey
    return -(ax * exd + ay * eyd) / torch.sqrt(ax * ax + ay * ay)


class _Exact:
    """One grid with its texture: systems, solutions and forces from the formulas."""

    def __init__(self, nt, nz, depth):
        self.nt, self.nz = nt, nz
        self.tc, self.te, self.zc, self.zf = _points(nt, nz)
        self.dth, self.dz = 2.0 * math.pi / nt, L / nz
        self.dx = R * self.dth
        self.xc, self.xe, self.xf = depth(self.tc, self.zc), depth(self.te, self.zc), depth(self.tc, self.zf)

    def system(self, e, ed):
        """(kx, kz, S) as the framework stores them: east faces, axial faces (ends doubled), source."""
        he = _film(e, self.te, self.zc) + self.xe
        hf = _film(e, self.tc, self.zf) + self.xf
        kx = he ** 3 / (12.0 * MU) * (self.dz / self.dx)
        ends = torch.ones(self.nz + 1, 1, dtype=torch.float64, device=DEVICE)
        ends[0] = ends[-1] = 2.0
        kz = ends * hf ** 3 / (12.0 * MU) * (self.dx / self.dz)
        S = -0.5 * U * (he - torch.roll(he, 1, -1)) * self.dz - _film_rate(e, ed, self.tc, self.zc) * self.dx * self.dz
        bnd = torch.zeros_like(S)
        bnd[0], bnd[-1] = kz[0] * P_IN, kz[-1] * P_OUT
        return kx, kz, S + bnd

    def apply(self, kx, kz, x):
        fe = kx * (x - torch.roll(x, -1, -1))
        y = fe - torch.roll(fe, 1, -1)
        fn = kz[..., 1:-1, :] * (x[..., :-1, :] - x[..., 1:, :])
        y[..., :-1, :] += fn
        y[..., 1:, :] -= fn
        y[..., 0, :] += kz[..., 0, :] * x[..., 0, :]
        y[..., -1, :] += kz[..., -1, :] * x[..., -1, :]
        return y

    def solve(self, kx, kz, S):
        """Batched CG with the Jacobi preconditioner to 1e-14 of the right-hand side, restarted once on the true residual."""
        D = kx + torch.roll(kx, 1, -1) + kz[..., :-1, :] + kz[..., 1:, :]
        x = torch.zeros_like(S)
        dot = lambda a, b: (a * b).sum((-1, -2), keepdim=True)
        goal = 1e-28 * dot(S, S)
        for _ in range(2):
            r = S - self.apply(kx, kz, x)
            z = r / D
            u, rz = z.clone(), dot(r, z)
            for k in range(12 * (self.nt + self.nz)):
                Au = self.apply(kx, kz, u)
                a = rz / torch.clamp(dot(u, Au), min=1e-300)
                x = x + a * u
                r = r - a * Au
                if k % 40 == 39 and bool((dot(r, r) <= goal).all()):
                    break
                z = r / D
                new = dot(r, z)
                u = z + (new / torch.clamp(rz, min=1e-300)) * u
                rz = new
        return x

    def forces(self, e, p, split=False):
        """(Fx, Fy, Mx, My), or the ten values of the pressure / shear split."""
        h = _film(e, self.tc, self.zc) + self.xc
        dpx = (torch.roll(p, -1, -1) - torch.roll(p, 1, -1)) / (2.0 * self.dx)
        mid = (p[2:] - p[:-2]) / (2.0 * self.dz)
        dpz = torch.cat([(p[1:2] - P_IN) / (1.5 * self.dz), mid, (P_OUT - p[-2:-1]) / (1.5 * self.dz)])
        tt, tz = -0.5 * h * dpx + MU * U / h, -0.5 * h * dpz
        c, s, zr = torch.cos(self.tc), torch.sin(self.tc), self.zc - 0.5 * L
        pr = [-p * c, -p * s, zr * p * s, -zr * p * c]
        sh = [-tt * s, tt * c, -zr * tt * c + tz * R * s, -zr * tt * s - tz * R * c]
        dA = self.dx * self.dz
        if split:
            return torch.stack([v.sum() for v in pr + sh + [tz, R * tt]]) * dA
        return torch.stack([(a + b).sum() for a, b in zip(pr, sh)]) * dA

    def joint(self, e, ed):
        """(p, F, J) of the nine conditions."""
        states = [(e, ed)]
        for k in range(8):
            a, b = np.array(e, float), np.array(ed, float)
            (a if k < 4 else b)[k % 4] += DELTA[k]
            states.append((a, b))
        sys = [self.system(a, b) for a, b in states]
        p = self.solve(*(torch.stack([s[i] for s in sys]) for i in range(3)))
        F = torch.stack([self.forces(a, p[k]) for k, (a, _) in enumerate(states)])
        J = (F[1:] - F[0]).T / torch.tensor(DELTA, dtype=torch.float64, device=DEVICE)
        return p, F, J

    def derivative(self, e, ed, rows):
        """p, F and the derivatives w . dF/d(e, edot) for each weight vector of rows."""
        kx, kz, S = self.system(e, ed)
        te = torch.tensor(np.asarray(e), dtype=torch.float64, device=DEVICE, requires_grad=True)
        td = torch.tensor(np.asarray(ed), dtype=torch.float64, device=DEVICE, requires_grad=True)
        p = self.solve(kx, kz, S)
        pv = p.clone().requires_grad_(True)
        F = self.forces(te, pv)
        rhs = [torch.autograd.grad((F * w).sum(), pv, retain_graph=True)[0] for w in rows]
        lam = self.solve(kx.expand(len(rows), -1, -1), kz.expand(len(rows), -1, -1), torch.stack(rhs))
        out = []
        for w, l in zip(rows, lam):
            kx, kz, S = self.system(te, td)
            g = (self.forces(te, p) * w).sum() + (l * (S - self.apply(kx, kz, p))).sum()
            out.append(torch.cat(torch.autograd.grad(g, (te, td))))
        return p, F.detach(), torch.stack(out)


def exact(case, seed):
    kind, nt, nz = case["kind"], case["n_theta"], case["n_axial"]
    rng = np.random.default_rng(seed)
    if kind != "film" and nt * nz > 700_000:
        return None                               # conjugate gradients would take too long here
    if kind == "batch":
        out = []
        for k, (a, b) in enumerate(_batch_grids(case)):
            e, ed = _state(rng)
            dim = _dimples(rng) if (k % 2 == 1 and case["texture"] != "smooth") else None
            p, F, J = _Exact(a, b, _depth(dim, None)).joint(e, ed)
            out.append({"p": p, "F": F, "J": J})
        return out
    e, ed = _state(rng)
    dimples, field = _texture(case, rng)
    x = _Exact(nt, nz, _depth(dimples, field))
    if kind == "step":
        if case["n_cond"] == 1:
            kx, kz, S = x.system(e, ed)
            p = x.solve(kx, kz, S)
            return {"p": p[None], "F": x.forces(e, p)[None]}
        p, F, J = x.joint(e, ed)
        return {"p": p, "F": F, "J": J}
    if kind == "picard":
        F_ext, M = _load(seed)
        cur, e0, p = np.array(ed), np.array(e), None
        pos = e0 + DT * cur
        for _ in range(2):
            p, F, J = x.joint(pos, cur)
            res = F_ext - M @ (cur - ed) / DT + F[0].cpu().numpy()
            J = J.cpu().numpy()
            step = np.linalg.solve(J[:, 4:] - M / DT + DT * J[:, :4], -res)
            pos, cur = pos + DT * step, cur + step
        return {"e": pos, "edot": cur, "p": p}
    if kind == "adjoint":
        p, F, J = x.derivative(e, ed, list(torch.eye(4, dtype=torch.float64, device=DEVICE)))
        return {"p": p, "J": J, "F": F[None]}
    if kind == "vjp":
        w = torch.tensor([1.0, -0.5, 20.0, 30.0], dtype=torch.float64, device=DEVICE)
        p, F, g = x.derivative(e, ed, [w])
        return {"F": F, "ge": g[0, :4], "ged": g[0, 4:], "p": p[None]}
    kx, kz, S = x.system(e, ed)
    p = torch.clamp(_field_input(nt, nz, seed), min=P_CAV)
    es = [np.array(e, float) for _ in range(9)]
    for k in range(4):
        es[k + 1][k] += DELTA[k]
    full = torch.cat([torch.full((9, 1, nt), P_IN, dtype=torch.float64, device=DEVICE), p,
                      torch.full((9, 1, nt), P_OUT, dtype=torch.float64, device=DEVICE)], 1)
    return {"kx": kx, "kz": kz, "S": S, "F": torch.stack([x.forces(a, q) for a, q in zip(es, p)]),
            "split": torch.stack([x.forces(a, q, split=True) for a, q in zip(es, p)]), "full": full}
