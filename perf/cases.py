"""What users of this framework have it do, as timed cases.

Four ways of using it are covered, each through its public entry points:

* ``run``: a state is restored (``LBM.load_state``), advanced by ``steps`` steps, optionally
  with the strain output, and its diagnostics are taken (``lbm_reduce``);
* ``guarded``: the same through ``checkpoint.run_guarded``, which takes the diagnostics and a
  snapshot after every ``check_every`` steps (a production run with its watchdog);
* ``query``: post-processing of a state: the strain by both formulas, the canonical
  populations and the diagnostics;
* ``gradient``: the strain-squared loss and its gradients with respect to the initial
  velocity and the force field (``autograd.strain_loss``, forward and backward).

The workloads are the ones under ``paper_1704_07559_amd/configs`` (their rates, viscosity laws
and forces), on their own boxes and on generic ones. The initial fields are smooth random
solenoidal flows with a mean flow, u_rms of the workloads' 0.04, made on the GPU from the seed.

``exact`` gives the same results from a plain FP64 implementation of the moment-space
collision and the pull streaming in torch.
"""
from __future__ import annotations

import math

import torch
import torch.utils.checkpoint

from paper_1704_07559_amd import autograd, capi, checkpoint, lbm, workloads

LATTICES = {"D3Q19": 19, "D3Q15": 15, "D2Q9": 9}
DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


def _case(kind, lattice, storage, box, steps, visc="smagorinsky", walls=0, **more):
    nx, ny, nz = box
    return {"kind": kind, "lattice": lattice, "storage": storage, "nx": nx, "ny": ny, "nz": nz, "steps": steps,
            "visc": visc, "walls": walls, "strain": more.pop("strain", "none"), **more}


def listed():
    return [
        # the Taylor-Green box of the parity runs: the smallest state, where launches count
        {"name": "tgv32", **_case("run", "D3Q19", "f32", (32, 32, 32), 20, visc="const", strain="yu")},
        # a small LES box (the size of the storage-error runs): launches and latency still matter
        {"name": "les64", **_case("run", "D3Q19", "f32", (64, 64, 64), 20)},
        # an LES box whose rows are neither a power of two nor a multiple of a cache line
        {"name": "les_ragged", **_case("run", "D3Q19", "f32", (171, 133, 95), 12)},
        # the headline LES
        {"name": "les256", **_case("run", "D3Q19", "f32", (256, 256, 256), 12)},
        # the large LES in 16-bit storage
        {"name": "les384_f16", **_case("run", "D3Q19", "f16", (384, 384, 384), 8)},
        # one rank's share of that LES over eight GPUs, in the other 16-bit type
        {"name": "slab384_bf16", **_case("run", "D3Q19", "bf16", (384, 384, 48), 12)},
        # the power-law channel between walls, viscosity from the Chai strain, with its watchdog
        {"name": "channel_powerlaw", **_case("guarded", "D3Q19", "f32", (128, 128, 512), 16, visc="powerlaw", walls=1,
                                             check_every=8)},
        # the LES on the smaller 3D lattice, a box of a generic size
        {"name": "d3q15_200", **_case("run", "D3Q15", "f32", (200, 200, 200), 12)},
        # the large two-dimensional LES
        {"name": "d2q9_4096", **_case("run", "D2Q9", "f32", (4096, 4096, 1), 16)},
        # an ordinary two-dimensional channel with an odd height, strain of the last step kept
        {"name": "d2q9_channel", **_case("run", "D2Q9", "f32", (600, 201, 1), 40, visc="implicit", walls=1,
                                         strain="chai")},
        # post-processing of the headline state
        {"name": "query256", **_case("query", "D3Q19", "f32", (256, 256, 256), 2)},
        # the gradient of the adjoint workload, a shorter run with the same checkpoint recipe
        {"name": "gradient128", **_case("gradient", "D3Q19", "f32", (128, 128, 128), 20, visc="const", every=10,
                                        record_all=0)},
    ]


def _size(rng, lo, hi):
    n = round(math.exp(rng.uniform(math.log(lo), math.log(hi))))
    r = rng.random()
    if r < 0.35:  # sizes people choose: multiples of 32 or of 10
        m = 32 if r < 0.2 else 10
        n = max(m, round(n / m) * m)
    return min(max(n, lo), hi)


def draw(rng):
    kind = rng.choices(["run", "guarded", "query", "gradient"], [60, 10, 15, 15])[0]
    if kind == "gradient":
        box = tuple(_size(rng, 12, 128) for _ in range(3))
        steps = rng.randrange(2, 25)
        return _case(kind, "D3Q19", "f32", box, steps, visc="const", walls=int(rng.random() < 0.3),
                     every=rng.randrange(1, steps + 1), record_all=int(rng.random() < 0.3))
    lattice = rng.choices(["D3Q19", "D3Q15", "D2Q9"], [65, 15, 20])[0]
    storage = rng.choices(["f32", "f16", "bf16"], [60, 25, 15])[0]
    visc = rng.choices(["smagorinsky", "const", "implicit", "powerlaw"], [50, 20, 15, 15])[0]
    if lattice == "D2Q9":
        box = (_size(rng, 40, 4096), _size(rng, 40, 4096), 1)
    else:
        box = tuple(_size(rng, 16, 384) for _ in range(3))
        while box[0] * box[1] * box[2] > 17_000_000:
            box = tuple(_size(rng, 16, 384) for _ in range(3))
    walls = 1 if visc == "powerlaw" else int(rng.random() < 0.25)
    if kind == "query":
        return _case(kind, lattice, storage, box, 2, visc=visc, walls=walls)
    steps = 2 * rng.randrange(1, 7)
    if kind == "guarded":
        return _case(kind, lattice, storage, box, steps, visc=visc, walls=walls, check_every=2 * rng.randrange(1, 4))
    return _case(kind, lattice, storage, box, steps, visc=visc, walls=walls,
                 strain=rng.choices(["none", "yu", "chai"], [80, 10, 10])[0])


# ---- inputs -------------------------------------------------------------------------------

def _params(case) -> capi.Params:
    """Library parameters: the workload the viscosity law belongs to, on the case's box."""
    cfg = workloads.load({"const": "C4" if case["kind"] == "gradient" else "C0", "smagorinsky": "C1", "implicit": "C1",
                          "powerlaw": "C2"}[case["visc"]])
    cfg = dict(cfg, force=cfg["force"] if isinstance(cfg["force"], list) else None)
    p = workloads.params(cfg, storage=case["storage"], lattice=case["lattice"],
                         grid={k: case[k] for k in ("nx", "ny", "nz")})
    if case["visc"] == "implicit":
        p.visc_kind = capi.LBM_VISC_SMAGORINSKY_IMPLICIT
    if case["lattice"] == "D2Q9" and case["walls"]:
        p.force = (1e-6, 0.0, 0.0)
    p.walls_y = case["walls"]
    return p


def _flow(case, seed) -> torch.Tensor:
    """delta_rho and u (4 x nz x ny x nx floats): twelve random solenoidal plane waves of a few
    periods per axis, u_rms 0.04, a mean flow and a weak density wave; between walls the mean
    flow is a parabola and the waves vanish at the walls."""
    gen = torch.Generator().manual_seed(1704 + seed)
    n = (case["nz"], case["ny"], case["nx"])
    flat = case["lattice"] == "D2Q9"
    axes = [(torch.arange(m, device="cuda", dtype=torch.float32) + 0.5) / m for m in n]
    grid = [a.reshape([-1 if i == k else 1 for i in range(3)]) for k, a in enumerate(axes)]
    out = torch.zeros((4,) + n, device="cuda")
    for _ in range(12):
        k = torch.randint(-4, 5, (3,), generator=gen).double()  # periods along z, y, x
        if flat:
            k[0] = 0
        k[2] += k.abs().sum() == 0
        a = torch.randn(3, generator=gen, dtype=torch.float64)
        if flat:
            a[0] = 0
        kl = k / torch.tensor(n)  # the wave vector in lattice units, to which a has to be normal
        a -= kl * (a @ kl) / (kl @ kl)
        a /= max(float(a.norm()), 1e-3)
        phase = 2 * math.pi * float(torch.rand(1, generator=gen))
        wave = sum(2 * math.pi * float(k[i]) * grid[i] for i in range(3)) + phase
        wave = torch.cos(wave)
        for c in range(3):
            out[1 + c] += float(a[2 - c]) * wave
        del wave
    rms = out[1:].double().square().mean().mul(1.0 if not flat else 1.5).sqrt().float()
    out[1:] *= 0.04 / rms
    profile = 4 * grid[1] * (1 - grid[1]) if case["walls"] else torch.ones_like(grid[1])
    out[1:] *= profile
    for c in range(2 if flat else 3):
        out[1 + c] += 0.01 * (c + 1) * profile
    out[0] = 1e-3 + 5e-4 * torch.cos(2 * math.pi * (grid[2] + grid[1] + grid[0]))
    return out


def prepare(case, seed):
    p = _params(case)
    flow = _flow(case, seed)
    state = {"case": case}
    if case["kind"] == "gradient":
        gen = torch.Generator(device="cuda").manual_seed(7559 + seed)
        n = (3, case["nz"], case["ny"], case["nx"])
        state["u0"] = flow[1:].clone().requires_grad_()
        state["F"] = (torch.rand(n, generator=gen, device="cuda") * 2e-6 - 1e-6).requires_grad_()
        state["problem"] = autograd.StrainLossProblem(p, case["steps"], case["every"], bool(case["record_all"]))
        return state
    sim = lbm.LBM(p, flow)
    if case["kind"] == "query":
        sim.step(case["steps"])
    else:
        state["start"] = sim.save_state()
    if case["strain"] != "none":
        state["S"] = torch.empty((sim.ncomp,) + sim.shape, device="cuda")
    state["sim"] = sim
    return state


# ---- one pass -----------------------------------------------------------------------------

def _result(sim, diagnostics):
    """The state after an even number of steps (it is in the buffer the run started from, in the
    layout of the state buffers), the lagged rate and the diagnostics."""
    p = sim.params
    dtype = {capi.LBM_F32: torch.float32, capi.LBM_F16: torch.float16, capi.LBM_BF16: torch.bfloat16}[p.storage]
    out = {"state": sim.f_a.view(dtype).view(p.nz, p.ny, p.q, p.nx), "diagnostics": diagnostics}
    if sim.s_nu is not None:
        out["s_nu"] = sim.s_nu
    return out


def run(state):
    case = state["case"]
    if case["kind"] == "gradient":
        u0, F = state["u0"], state["F"]
        J = autograd.strain_loss(u0, F, state["problem"])
        gu, gF = torch.autograd.grad(J, (u0, F))
        return {"J": J.detach().float(), "grad_u0": gu, "grad_F": gF}
    sim = state["sim"]
    if case["kind"] == "query":
        return {"yu": sim.strain(capi.LBM_STRAIN_YU), "chai": sim.strain(capi.LBM_STRAIN_CHAI),
                "populations": sim.populations(), "diagnostics": capi.lbm_reduce(sim.ctx)}
    sim.load_state(state["start"])
    if case["kind"] == "guarded":
        d = checkpoint.run_guarded(sim, case["steps"], case["check_every"])
        return _result(sim, [d["mass"], *map(float, d["mom"]), d["ke"], d["ss"], d["umax"], float(d["nonfinite"])])
    if case["strain"] == "none":
        sim.step(case["steps"])
        return _result(sim, capi.lbm_reduce(sim.ctx))
    sim.step(case["steps"], S_out=state["S"],
             strain_kind=capi.LBM_STRAIN_YU if case["strain"] == "yu" else capi.LBM_STRAIN_CHAI)
    return {**_result(sim, capi.lbm_reduce(sim.ctx)), "strain": state["S"]}


# ---- the work a pass cannot do without -------------------------------------------------------

# floating-point operations of one node's step (moments, equilibrium, strain, relaxation,
# back-transform), and of one node's step in reverse
STEP_FLOPS = {"D3Q19": 400, "D3Q15": 300, "D2Q9": 160}
ADJOINT_FLOPS = 600


def work(case):
    """Every input read once, every output written once. A run of several steps reads its
    starting state once and writes its last; a gradient reads u0 and F and writes both
    gradients; the steps between are arithmetic."""
    n = case["nx"] * case["ny"] * case["nz"]
    q, size = LATTICES[case["lattice"]], torch.empty((), dtype=DTYPES[case["storage"]]).element_size()
    ncomp = 3 if case["lattice"] == "D2Q9" else 6
    lagged = 4 if case["visc"] in ("smagorinsky", "powerlaw") else 0
    if case["kind"] == "gradient":
        return {"bytes": n * 4 * 12, "flops": n * case["steps"] * (STEP_FLOPS["D3Q19"] + ADJOINT_FLOPS)}
    if case["kind"] == "query":
        return {"bytes": n * (q * size + lagged + 2 * 4 * ncomp + 4 * q), "flops": n * 2 * STEP_FLOPS[case["lattice"]]}
    strain = 4 * ncomp if case["strain"] != "none" else 0
    return {"bytes": n * (2 * (q * size + lagged) + strain), "flops": n * case["steps"] * STEP_FLOPS[case["lattice"]]}


# ---- the same results in 64 bits ---------------------------------------------------------------

def _velocities(q):
    if q == 9:
        return [(0, 0, 0), (1, 0, 0), (0, 1, 0), (-1, 0, 0), (0, -1, 0), (1, 1, 0), (-1, 1, 0), (-1, -1, 0), (1, -1, 0)]
    c = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1)]
    if q == 15:
        for d in ((1, 1, 1), (1, 1, -1), (1, -1, 1), (-1, 1, 1)):
            c += [d, tuple(-a for a in d)]
        return c
    c += [(x, y, 0) for y in (1, -1) for x in (1, -1)]
    c += [(x, 0, z) for z in (1, -1) for x in (1, -1)]
    return c + [(0, y, z) for z in (1, -1) for y in (1, -1)]


def _moments(q, c):
    """Rows of the transformation matrix as polynomials of the velocities (c: 3 x q)."""
    x, y, z = c
    s = x * x + y * y + z * z
    one = torch.ones_like(s)
    if q == 9:
        return torch.stack([one, 3 * s - 4, (9 * s * s - 21 * s + 8) / 2, x, (3 * s - 5) * x, y, (3 * s - 5) * y,
                            x * x - y * y, x * y])
    if q == 15:
        h = (5 * s - 13) / 2
        return torch.stack([one, s - 2, (15 * s * s - 55 * s + 32) / 2, x, h * x, y, h * y, z, h * z, 3 * x * x - s,
                            y * y - z * z, x * y, y * z, x * z, x * y * z])
    h, k = 5 * s - 9, 3 * s - 5
    return torch.stack([one, 19 * s - 30, (21 * s * s - 53 * s + 24) / 2, x, h * x, y, h * y, z, h * z, 3 * x * x - s,
                        k * (3 * x * x - s), y * y - z * z, k * (y * y - z * z), x * y, y * z, x * z,
                        (y * y - z * z) * x, (z * z - x * x) * y, (x * x - y * y) * z])


def _times(A, x):
    """A @ x for a small A and a long x, a few million columns at a time."""
    if x.shape[1] <= 1 << 23:
        return A @ x
    return torch.cat([A @ part.contiguous() for part in x.split(1 << 23, 1)], 1)


NU_ROWS = {9: (7, 8), 15: (9, 10, 11, 12, 13), 19: (9, 11, 13, 14, 15)}
WEIGHTS = {9: (4 / 9, 1 / 9, 1 / 36), 15: (2 / 9, 1 / 9, 0, 1 / 72), 19: (1 / 3, 1 / 18, 1 / 36)}


class Reference:
    """The model in FP64: canonical populations g (q x nz x ny x nx) and the lagged rate."""

    def __init__(self, p, force):
        self.p, self.q = p, p.q
        dev = force.device
        self.cs = _velocities(self.q)
        self.c = torch.tensor(self.cs, dtype=torch.float64, device=dev).T
        self.w = torch.tensor([WEIGHTS[self.q][sum(map(abs, v))] for v in self.cs], dtype=torch.float64, device=dev)
        self.T = _moments(self.q, self.c)
        self.Ti = torch.linalg.inv(self.T.cpu()).to(dev)
        self.s = torch.tensor(list(p.s)[: self.q], dtype=torch.float64, device=dev)
        self.nu_rows = list(NU_ROWS[self.q])
        self.opp = [self.cs.index(tuple(-a for a in v)) for v in self.cs]
        self.F = force  # 3 x N, or 3 x 1
        ab = [(0, 0), (1, 1), (0, 1)] if self.q == 9 else [(0, 0), (1, 1), (2, 2), (0, 1), (1, 2), (0, 2)]
        self.cc = torch.stack([self.c[a] * self.c[b] for a, b in ab])
        self.off = torch.tensor([1.0 if a == b else 2.0 for a, b in ab], dtype=torch.float64, device=dev)

    def equilibrium(self, drho, j):
        cj = _times(self.c.T, j)
        jj = (j * j).sum(0)
        return self.w[:, None] * (drho + 3 * cj + (4.5 * cj * cj - 1.5 * jj) / self.p.rho0)

    def macro(self, g):
        drho, j = g.sum(0), _times(self.c, g) + 0.5 * self.F
        return drho, j, g - self.equilibrium(drho, j)

    def strain_parts(self, neq):
        """S = P + s_nu A: the second moments of the relaxed non-equilibrium part, the rows
        relaxed with s_nu apart."""
        nu = torch.zeros_like(self.s)
        nu[self.nu_rows] = 1
        k = -1.5 / self.p.rho0 * (self.cc @ self.Ti)
        return _times((k * (self.s * (1 - nu))) @ self.T, neq), _times((k * nu) @ self.T, neq)

    def magnitude(self, S):
        return (2 * (self.off[:, None] * S * S).sum(0)).sqrt()

    def rate(self, P, A, s_nu):
        """The rate of the s_nu rows in this collision."""
        p = self.p
        if p.visc_kind == capi.LBM_VISC_CONST:
            return s_nu
        if p.visc_kind == capi.LBM_VISC_SMAGORINSKY_IMPLICIT:
            s = s_nu.clone()
            for _ in range(60):  # a contraction: the viscosity hardly depends on the rate
                s = 1 / (3 * (p.nu0 + p.c_smag ** 2 * self.magnitude(P + s * A)) + 0.5)
            return s
        gamma = self.magnitude(P + s_nu * A)
        if p.visc_kind == capi.LBM_VISC_SMAGORINSKY:
            nu = p.nu0 + p.c_smag ** 2 * gamma
        else:
            nu = (p.K_pl * gamma.clamp_min(1e-300) ** (p.n_pl - 1)).clamp(p.nu_min, p.nu_max)
        return 1 / (3 * nu + 0.5)

    def collide(self, g, s_nu):
        """(post-collision populations, the rate used, the strain of the incoming state)."""
        drho, j, neq = self.macro(g)
        P, A = self.strain_parts(neq)
        s = self.rate(P, A, s_nu)
        implicit = self.p.visc_kind == capi.LBM_VISC_SMAGORINSKY_IMPLICIT
        S = P + (s if implicit else s_nu) * A
        cj, cF = _times(self.c.T, j), _times(self.c.T, self.F)
        Fi = self.w[:, None] * (3 * cF + (9 * cj * cF - 3 * (j * self.F).sum(0)) / self.p.rho0)
        rates = self.s[:, None].expand(self.q, g.shape[1]).clone()
        rates[self.nu_rows] = s.expand(len(self.nu_rows), -1)
        m = rates * _times(self.T, neq) - (1 - 0.5 * rates) * _times(self.T, Fi)
        return g - _times(self.Ti, m), s, S

    def stream(self, post):
        p = self.p
        f = post.reshape(self.q, p.nz, p.ny, p.nx)
        out = []
        for i, (cx, cy, cz) in enumerate(self.cs):
            t = f[i].roll((cz, cy, cx), (0, 1, 2))
            if p.walls_y and cy:
                row = 0 if cy > 0 else p.ny - 1
                t = t.index_copy(1, torch.tensor([row], device=t.device), f[self.opp[i]][:, row:row + 1])
            out.append(t.reshape(-1))
        return torch.stack(out)

    def start(self, drho, u):
        g = self.equilibrium(drho, self.p.rho0 * u)
        return g, torch.full_like(drho, self.s[self.nu_rows[0]].item())


def _exact_gradient(case, seed):
    state = prepare(case, seed)
    n = case["nx"] * case["ny"] * case["nz"]
    u = state["u0"].detach().double().reshape(3, n).requires_grad_()
    F = state["F"].detach().double().reshape(3, n).requires_grad_()
    ref = Reference(state["problem"].params, F)
    g, s = ref.start(torch.zeros(n, dtype=torch.float64, device=u.device), u)

    def step(g, F):
        ref.F = F
        return ref.stream(ref.collide(g, s)[0])

    for _ in range(case["steps"]):
        g = torch.utils.checkpoint.checkpoint(step, g, F, use_reentrant=False)
    ref.F = F
    P, A = ref.strain_parts(ref.macro(g)[2])
    J = (ref.off[:, None] * (P + s * A) ** 2).sum()
    gu, gF = torch.autograd.grad(J, (u, F))
    shape = (3, case["nz"], case["ny"], case["nx"])
    return {"J": J.detach(), "grad_u0": gu.reshape(shape), "grad_F": gF.reshape(shape)}


def exact(case, seed):
    if case["kind"] == "gradient":
        return _exact_gradient(case, seed)
    p = _params(case)
    shape = (case["nz"], case["ny"], case["nx"])
    n = shape[0] * shape[1] * shape[2]
    force = torch.tensor([p.force[a] for a in range(3)], dtype=torch.float64, device="cuda").reshape(3, 1)
    ref = Reference(p, force)
    flow = _flow(case, seed).reshape(4, n).double()
    if p.q == 9:
        flow[3] = 0
    g, s = ref.start(flow[0], flow[1:])
    del flow
    for _ in range(case["steps"]):
        post, s, S = ref.collide(g, s)
        del g
        g = ref.stream(post)
    _, j, neq = ref.macro(g)
    P, A = ref.strain_parts(neq)
    now = P + (ref.rate(P, A, s) if p.visc_kind == capi.LBM_VISC_SMAGORINSKY_IMPLICIT else s) * A
    del neq, P, A
    jj = (j * j).sum(0)
    diagnostics = [float(v) for v in (g.sum(), j[0].sum(), j[1].sum(), j[2].sum(), jj.sum() / (2 * p.rho0),
                                      (ref.off[:, None] * now * now).sum(), jj.max().sqrt() / p.rho0, 0.0)]
    if case["kind"] == "query":
        now = now.reshape((-1,) + shape)
        return {"yu": now, "chai": now, "populations": g.reshape((p.q,) + shape), "diagnostics": diagnostics}
    out = {"state": post.reshape((p.q,) + shape).permute(1, 2, 0, 3).contiguous(), "diagnostics": diagnostics}
    if p.visc_kind in (capi.LBM_VISC_SMAGORINSKY, capi.LBM_VISC_POWERLAW):
        out["s_nu"] = s
    if case["strain"] != "none":
        out["strain"] = S.reshape((-1,) + shape)
    return out
