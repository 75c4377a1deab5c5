"""Performance cases of the finite-volume TVD-RK3 library.

Each case is a problem as the repository's own benchmark, tests and serving stream pose it
(grid, model, precision, options) and one way in which a program calls the library:

  stages    the three fused stages of one CFL step, out of place, the third with the CFL
            reduction (``rk3_stage``, ``rk3_stage3_cfl``): how a time loop drives the solver
  advance   a run of CFL steps from a stored initial state (``advance``)
  rhs       one right-hand side (``rhs``): an outer time integrator or implicit solver
  batch     several independent requests admitted together and stepped through the step
            graph (``Batch.set``, ``Batch.step_graph``): the serving path
  gradient  the kinetic energy's gradient with respect to the initial state of a fixed-dt
            trajectory (``adjoint.advance_fixed_dt`` and its backward pass)

``exact`` evaluates the same discrete scheme with plain torch operations in 64 bits.
"""
from __future__ import annotations

import math

import torch

from paper_2402_05193_amd import adjoint, solver as S

DEVICE = "cuda"
CFL = 0.5
ALPHA_EPS = 1e-8        # volume fraction of the absent fluid
MODELS = {"euler": S.EULER, "ns": S.NS, "five": S.DIM}
P, Z, M = S.PERIODIC, S.ZERO_GRADIENT, S.SYMMETRY
BOUNDARIES = {"periodic": (P,) * 6, "open": (Z,) * 6, "mixed": (Z, Z, M, M, P, P), "walls": (M, Z, P, P, M, M)}
GRIDS = ((64, 64, 64), (96, 96, 96), (128, 128, 128), (192, 96, 96), (256, 128, 128))   # the serving stream's


def _case(name, call, field, nx, ny, nz, model, dtype="f64", bc="periodic", steps=1, recon=0, scheme=0,
          visc_order=0, thinc=0, limiters=-1):
    c = dict(call=call, field=field, nx=nx, ny=ny, nz=nz, model=model, dtype=dtype, bc=bc, steps=steps, recon=recon,
             scheme=scheme, visc_order=visc_order, thinc=thinc, limiters=limiters)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest calls: a one-dimensional two-phase shock tube (200 cells, as the paper's
        # validation), where launches and the latency of one workgroup's march are all there is
        _case("tube_1d", "advance", "riemann", 200, 1, 1, "five", bc="open", steps=10, limiters=1),
        # a two-dimensional isentropic vortex on an odd grid (convergence studies)
        _case("vortex_2d", "advance", "vortex", 150, 150, 1, "euler", steps=5),
        # a small box: the inviscid Taylor-Green vortex at 32^3 (regression runs, parameter sweeps)
        _case("euler_32", "advance", "tgv", 32, 32, 32, "euler", steps=5),
        # one right-hand side on a ragged grid with mixed boundaries, characteristic variables
        _case("char_ragged", "rhs", "smooth", 101, 75, 53, "euler", bc="mixed", recon=1),
        # the paper's single-phase setup: TENO6-A with sixth-order viscous fluxes
        _case("teno_visc6", "advance", "tgv", 128, 128, 128, "ns", scheme=1, visc_order=6),
        # the benchmark's smaller size in FP32
        _case("ns_128_f32", "stages", "tgv", 128, 128, 128, "ns", dtype="f32"),
        # the benchmark: Navier-Stokes Taylor-Green vortex at 256^3, FP64
        _case("ns_256", "stages", "tgv", 256, 256, 256, "ns"),
        # inviscid, an ordinary size
        _case("euler_160", "stages", "tgv", 160, 160, 160, "euler"),
        # the five-equation shock-bubble interaction, limiters on
        _case("bubble", "stages", "bubble", 256, 128, 128, "five", bc="open", limiters=1),
        # the same with interface capturing in FP32, a smaller box
        _case("bubble_thinc_f32", "stages", "bubble", 192, 96, 96, "five", dtype="f32", bc="open", thinc=1, limiters=1),
        # six requests of the serving stream stepped together
        _case("serving", "batch", "riemann", 6, 0, 0, "mixed", dtype="f32", bc="open", steps=2, limiters=1),
        # gradient of a trajectory: decaying turbulence at 64^3
        _case("gradient_64", "gradient", "turbulence", 64, 64, 64, "euler", steps=5),
    ]


def draw(rng):
    def log(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    kind = rng.choice(["tube", "plane", "small", "rhs", "teno", "ns", "euler", "bubble", "batch", "gradient"])
    dtype = rng.choice(["f64", "f64", "f32"])
    if kind == "tube":
        return _case(None, "advance", "riemann", log(60, 2000), 1, 1, rng.choice(["five", "euler"]), bc="open",
                     steps=rng.randint(4, 12), limiters=1)
    if kind == "plane":
        return _case(None, "advance", "vortex", log(40, 600), log(40, 600), 1, "euler", steps=rng.randint(2, 5))
    if kind == "small":
        return _case(None, "advance", "tgv", log(12, 56), log(12, 56), log(12, 56), rng.choice(["euler", "ns"]),
                     dtype=dtype, steps=rng.randint(2, 5))
    if kind == "rhs":
        return _case(None, "rhs", "smooth", log(20, 160), log(20, 160), log(20, 120), rng.choice(["euler", "ns", "five"]),
                     bc=rng.choice(["periodic", "mixed", "walls", "open"]), recon=rng.choice([0, 1]))
    if kind == "teno":
        return _case(None, "advance", "tgv", log(48, 128), log(48, 128), log(48, 128), "ns", scheme=1,
                     visc_order=rng.choice([4, 6, 6]), recon=rng.choice([0, 0, 1]))
    if kind == "ns":
        return _case(None, "stages", "tgv", log(64, 256), log(64, 256), log(64, 256), "ns", dtype=dtype)
    if kind == "euler":
        return _case(None, "stages", "tgv", log(64, 224), log(64, 224), log(64, 224), "euler", dtype=dtype)
    if kind == "bubble":
        ny = log(48, 128)
        return _case(None, "stages", "bubble", 2 * ny, ny, rng.choice([ny, max(40, ny - 7)]), "five", dtype=dtype,
                     bc="open", thinc=rng.choice([0, 1]), limiters=1)
    if kind == "batch":
        return _case(None, "batch", "riemann", rng.randint(2, 8), 0, 0, "mixed", dtype="f32", bc="open",
                     steps=rng.randint(1, 3), limiters=1)
    n = 2 * log(12, 32)      # the trajectory's kept states are 16-byte aligned on even grids
    return _case(None, "gradient", "turbulence", n, n, rng.choice([n, n - 6]), "euler", steps=rng.randint(2, 5))


# ------------------------------------------------------------------ problems
def _requests(case, seed):
    """The members of a batch: single- and two-phase Riemann problems on the serving grids;
    the largest grids stay few, as the case's pass has a bound."""
    if case["call"] != "batch":
        return [case]
    out = []
    for i in range(case["nx"]):
        nx, ny, nz = GRIDS[(0, 1, 0, 2, 1, 0, 3, 1)[i % 8]]
        out.append(dict(case, nx=nx, ny=ny, nz=nz, model=("five", "euler")[i % 2], call="member"))
    return out


def _config(case):
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    kw = dict(nx=nx, ny=ny, nz=nz, model=MODELS[case["model"]], dtype=S.F64 if case["dtype"] == "f64" else S.F32,
              bc=BOUNDARIES[case["bc"]], positivity=case["limiters"], cfl=CFL, recon=case["recon"],
              scheme=case["scheme"], visc_order=case["visc_order"], thinc=case["thinc"])
    if case["field"] in ("tgv", "turbulence"):
        box = 2.0 * math.pi
        kw.update(dx=box / nx, dy=box / ny, dz=box / nz, weno_eps=1e-6 if case["call"] == "gradient" else 0.0)
    elif case["field"] == "vortex":
        kw.update(dx=10.0 / nx, dy=10.0 / ny, dz=10.0 / nx)
    elif case["field"] == "bubble":
        h = 2.0 * 0.089 / nx
        kw.update(dx=h, dy=0.089 / ny, dz=0.089 / nz, gamma1=1.66)
    elif case["field"] == "smooth":
        kw.update(dx=1.0 / nx, dy=1.0 / ny, dz=1.0 / nz, gamma2=1.66)
    else:
        kw.update(dx=1.0 / nx, dy=1.0 / nx, dz=1.0 / nx, gamma2=1.66 if case["model"] == "five" else 1.4)
    if case["model"] == "ns":
        kw.update(mu=1.0 / 1600.0, prandtl=0.72)
    return S.Config(**kw)


def _field(case, cfg, seed):
    """Primitive state of the case in 64 bits."""
    g = torch.Generator(device=DEVICE).manual_seed(int(seed))
    f8 = dict(dtype=torch.float64, device=DEVICE)
    shape = (cfg.nz, cfg.ny, cfg.nx)
    draws = torch.rand(64, generator=g, **f8).tolist()
    x = ((torch.arange(cfg.nx, **f8) + 0.5) * cfg.dx).view(1, 1, -1)
    y = ((torch.arange(cfg.ny, **f8) + 0.5) * cfg.dy).view(1, -1, 1)
    z = ((torch.arange(cfg.nz, **f8) + 0.5) * cfg.dz).view(-1, 1, 1)
    W = torch.zeros((cfg.ncomp,) + shape, **f8)
    what = case["field"]
    if what == "tgv":               # Ma 0.1 Taylor-Green vortex with velocity noise
        W[0] = 1.0
        W[1] = torch.sin(x) * torch.cos(y) * torch.cos(z)
        W[2] = -torch.cos(x) * torch.sin(y) * torch.cos(z)
        W[4] = 1.0 / (1.4 * 0.01) + (torch.cos(2 * x) + torch.cos(2 * y)) * (torch.cos(2 * z) + 2.0) / 16.0
        W[1:4] += 1e-3 * (2.0 * torch.rand((3,) + shape, generator=g, **f8) - 1.0)
    elif what == "turbulence":      # solenoidal, E(k) ~ k^4 exp(-2 (k/4)^2), u_rms 0.3
        k = [torch.fft.fftfreq(n, d=1.0 / n, **f8) for n in shape]
        K = torch.stack(torch.meshgrid(*k, indexing="ij")[::-1])
        k2 = (K * K).sum(0)
        A = torch.fft.fftn(torch.randn((3,) + shape, generator=g, **f8), dim=(1, 2, 3))
        unit = K / torch.where(k2 > 0, k2, 1.0).sqrt()
        A = (A - unit * (unit * A).sum(0)) * torch.sqrt(k2) * torch.exp(-k2 / 16.0)
        vel = torch.fft.ifftn(A, dim=(1, 2, 3)).real
        vel = vel - vel.mean(dim=(1, 2, 3), keepdim=True)
        W[0], W[4] = 1.0, 1.0 / 1.4
        W[1:4] = vel * (0.3 / math.sqrt(float((vel * vel).sum(0).mean()) / 3.0))
    elif what == "vortex":          # isentropic vortex in a uniform stream
        X, Y = x - (4.0 + 2.0 * draws[0]), y - (4.0 + 2.0 * draws[1])
        strength, r2 = 4.0 + 2.0 * draws[2], X * X + Y * Y
        f = strength / (2.0 * math.pi) * torch.exp(0.5 * (1.0 - r2))
        T = 1.0 - 0.4 * strength ** 2 / (8.0 * 1.4 * math.pi ** 2) * torch.exp(1.0 - r2)
        W[0], W[4] = T ** 2.5, T ** 3.5
        W[1], W[2] = 1.0 - f * Y, draws[3] + f * X
    elif what == "smooth":          # a few Fourier modes around an admissible mean
        mean = [0.6, 0.5, 0.1, -0.1, 0.05, 1.0, 0.5] if cfg.ncomp == 7 else [1.0, 0.2, -0.1, 0.15, 1.0]
        for m, v in enumerate(mean):
            W[m] = v
            for q in range(2):
                r = draws[4 * (2 * m + q):4 * (2 * m + q) + 4]
                W[m] += 0.06 * max(abs(v), 0.3) * torch.sin(2 * math.pi * ((1 + int(3 * r[0])) * x + (1 + int(3 * r[1])) * y
                                                                     + int(3 * r[2]) * z + r[3]))
    elif what == "bubble":          # a planar shock in air ahead of a helium bubble, SI units
        ma, H = 1.15 + 0.2 * draws[0], 0.089
        rho_a, p_a, rho_he = 1.2041, 101325.0, 0.1660
        m2 = ma * ma
        p_s = p_a * (1.0 + 2.8 / 2.4 * (m2 - 1.0))
        rho_s = rho_a * 2.4 * m2 / (0.4 * m2 + 2.0)
        u_s = ma * math.sqrt(1.4 * p_a / rho_a) * (1.0 - rho_a / rho_s)
        cy, cz = H * (0.48 + 0.04 * draws[1]), H * (0.48 + 0.04 * draws[2])
        r = torch.sqrt((x - 0.090) ** 2 + (y - cy) ** 2 + (z - cz) ** 2)
        a = ALPHA_EPS + (1.0 - 2.0 * ALPHA_EPS) * 0.5 * (1.0 - torch.tanh((r - 0.25 * H) / cfg.dx))
        shocked = (x < 0.060) & torch.ones_like(r, dtype=torch.bool)
        W[0], W[6] = a * rho_he, a
        W[1] = (1.0 - a) * torch.where(shocked, rho_s, rho_a)
        W[2] = torch.where(shocked, u_s, 0.0)
        W[5] = torch.where(shocked, p_s, p_a)
    else:                           # planar two-state problem normal to x
        left = (torch.arange(cfg.nx, **f8) + 0.5 < 0.5 * cfg.nx).view(1, 1, -1)
        side = [[0.5 + 4.0 * draws[3 * s], -0.5 + draws[3 * s + 1], 0.5 + 4.0 * draws[3 * s + 2]] for s in (0, 1)]
        pick = [torch.where(left, a, b) for a, b in zip(*side)]
        if cfg.ncomp == 7:
            a = torch.where(left, 1.0 - ALPHA_EPS, ALPHA_EPS).to(torch.float64)
            W[0], W[1], W[2], W[5], W[6] = a * pick[0], (1.0 - a) * pick[0], pick[1], pick[2], a
        else:
            W[0], W[1], W[4] = pick
    return W


def _problem(case, seed):
    """(config, conservative state in the case's precision)."""
    cfg = _config(case)
    return cfg, _to_cons(cfg, _field(case, cfg, seed)).to(cfg.torch_dtype).contiguous()


# ------------------------------------------------------------------ the library's calls
def prepare(case, seed):
    if case["call"] == "batch":
        problems = [_problem(c, seed + 101 * i) for i, c in enumerate(_requests(case, seed))]
        size = [(U.numel() + 63) // 64 * 64 for _, U in problems]        # 256-byte aligned members
        start = torch.zeros(sum(size), dtype=torch.float32, device=DEVICE)
        states, members, at = torch.empty_like(start), [], 0
        for (cfg, U), n in zip(problems, size):
            start[at:at + U.numel()] = U.view(-1)
            members.append((cfg, states[at:at + U.numel()].view(cfg.shape), S.workspace(cfg, DEVICE)))
            at += n
        return dict(call="batch", steps=case["steps"], start=start, states=states, members=members,
                    batch=S.Batch(len(members), DEVICE), stream=torch.cuda.Stream())
    cfg, U0 = _problem(case, seed)
    s = dict(call=case["call"], steps=case["steps"], cfg=cfg, U0=U0, ws=S.workspace(cfg, DEVICE))
    s["dt"] = torch.zeros(1, dtype=torch.float64, device=DEVICE)
    if case["call"] == "advance":
        s["U"] = torch.empty_like(U0)
    else:
        S.compute_dt(cfg, U0, s["dt"], s["ws"])
    if case["call"] == "stages":
        s.update(A=torch.empty_like(U0), B=torch.empty_like(U0), C=torch.empty_like(U0), dt_next=torch.zeros_like(s["dt"]))
    elif case["call"] == "rhs":
        s.update(R=torch.empty_like(U0), step=float(s["dt"]))
    elif case["call"] == "gradient":
        s.update(step=float(s["dt"]))
    return s


def run(state):
    s = state
    if s["call"] == "stages":
        S.rk3_stage(s["cfg"], 1, s["U0"], s["U0"], s["A"], dt_dev=s["dt"])
        S.rk3_stage(s["cfg"], 2, s["U0"], s["A"], s["B"], dt_dev=s["dt"])
        S.rk3_stage3_cfl(s["cfg"], s["U0"], s["B"], s["C"], s["dt"], s["dt_next"], s["ws"])
        return [s["C"], s["dt_next"]]
    if s["call"] == "advance":
        s["U"].copy_(s["U0"])
        S.advance(s["cfg"], s["U"], s["steps"], 0.0, s["ws"])
        return s["U"]
    if s["call"] == "rhs":
        return S.rhs(s["cfg"], s["U0"], s["R"], s["step"])
    if s["call"] == "batch":
        here = torch.cuda.current_stream()
        s["stream"].wait_stream(here)
        with torch.cuda.stream(s["stream"]):
            s["states"].copy_(s["start"])
            s["batch"].set(s["members"], fresh=[True] * len(s["members"]))
            s["batch"].step_graph(s["steps"])
        here.wait_stream(s["stream"])
        return [U for _, U, _ in s["members"]]
    U0 = s["U0"].detach().requires_grad_(True)
    loss = adjoint.kinetic_energy(s["cfg"], adjoint.advance_fixed_dt(s["cfg"], U0, s["steps"], s["step"], every=10))
    (grad,) = torch.autograd.grad(loss, U0)
    return [loss.detach(), grad]


# ------------------------------------------------------------------ what a pass cannot do without
def _flops_per_cell(case):
    """Operations of one right-hand side and stage update per cell, from the scheme's formulas."""
    nc = 7 if case["model"] == "five" else 5
    face = 389 * nc if case["scheme"] else (144 * nc if case["recon"] else 95 * nc)
    if case["recon"]:
        face += 30 + 12 * (nc - 2) + 6 * nc
    total = 3 * face + 3 * 91 + 9 * nc + 5 * nc + 13
    if case["model"] == "five":
        total += 35
    if case["model"] == "ns":
        total += 826 if case["visc_order"] == 6 else 286
    return total


def work(case):
    size = flops = 0.0
    for c in _requests(case, 0):
        cells = c["nx"] * c["ny"] * c["nz"]
        state = cells * (7 if c["model"] == "five" else 5) * (8 if c["dtype"] == "f64" else 4)
        stages = {"rhs": 1, "stages": 3}.get(c["call"], 3 * c["steps"])
        # stage 1 reads and writes one state each, stages 2 and 3 read two and write one
        size += state * (2 if c["call"] == "rhs" else 8 * stages / 3)
        flops += cells * _flops_per_cell(c) * stages
        if c["call"] == "gradient":      # the reverse sweep: about three forwards, from the kept stage states
            size += state * 4 * stages
            flops += 3 * cells * _flops_per_cell(c) * stages
    return {"bytes": int(size), "flops": int(flops)}


# ------------------------------------------------------------------ the scheme in 64 bits
class _Gas:
    """Layout and equation of state of a configuration (stiffened gas; isobaric mixture)."""

    def __init__(self, cfg):
        self.cfg, self.two = cfg, cfg.ncomp == 7
        self.V, self.P = (2, 5) if self.two else (1, 4)
        f32 = cfg.dtype == S.F32
        self.weno_eps = cfg.weno_eps or (1e-30 if f32 else 1e-40)
        self.eps_rho, self.eps_rhoc2, self.eps_alpha = (1e-10, 1e-8, 1e-10) if f32 else (1e-12, 1e-10, 1e-12)
        self.limited = self.two if cfg.positivity < 0 else cfg.positivity == 1

    def rho(self, W):
        return W[0] + W[1] if self.two else W[0]

    def mixture(self, a):
        c = self.cfg
        G1, G2 = 1.0 / (c.gamma1 - 1.0), 1.0 / (c.gamma2 - 1.0)
        return a * G1 + (1.0 - a) * G2, a * (c.gamma1 * c.pinf1 * G1) + (1.0 - a) * (c.gamma2 * c.pinf2 * G2)

    def rho_e(self, W):
        c = self.cfg
        if self.two:
            G, Pi = self.mixture(W[6])
            return G * W[5] + Pi
        return (W[4] + c.gamma1 * c.pinf1) / (c.gamma1 - 1.0)

    def rhoc2(self, W):
        if self.two:
            G, Pi = self.mixture(W[6])
            return ((G + 1.0) * W[5] + Pi) / G
        return self.cfg.gamma1 * (W[4] + self.cfg.pinf1)

    def cons(self, W):
        V, rho = self.V, self.rho(W)
        mom = [rho * W[V + i] for i in range(3)]
        E = self.rho_e(W) + 0.5 * sum(mom[i] * W[V + i] for i in range(3))
        return torch.stack([W[m] for m in range(V)] + mom + [E] + ([W[6]] if self.two else []))

    def prim(self, U):
        V, P, c = self.V, self.P, self.cfg
        rho = self.rho(U)
        vel = [U[V + i] / rho for i in range(3)]
        re = U[P] - 0.5 * sum(U[V + i] * vel[i] for i in range(3))
        if self.two:
            G, Pi = self.mixture(U[6])
            return torch.stack([U[0], U[1]] + vel + [(re - Pi) / G, U[6]])
        return torch.stack([U[0]] + vel + [(c.gamma1 - 1.0) * re - c.gamma1 * c.pinf1])

    def flux(self, W, d):
        U, un, V, P = self.cons(W), W[self.V + d], self.V, self.P
        F = [U[m] * un for m in range(len(U))]
        F[V + d] = F[V + d] + W[P]
        F[P] = F[P] + un * W[P]
        return torch.stack(F)


def _to_cons(cfg, W):
    return _Gas(cfg).cons(W)


def _pad(cfg, U, V):
    """State with three halo cells on every side, boundary conditions by index mapping."""
    for d, n in enumerate((cfg.nx, cfg.ny, cfg.nz)):
        lo, hi = cfg.bc[2 * d], cfg.bc[2 * d + 1]
        index, sign = [], []
        for i in range(-3, n + 3):
            b = lo if i < 0 else hi if i >= n else None
            j = i if b is None else i % n if b == P else min(max(i, 0), n - 1) if b == Z else -i - 1 if i < 0 else 2 * n - 1 - i
            index.append(j)
            sign.append(-1.0 if b == M else 1.0)
        U = U.index_select(3 - d, torch.tensor(index, device=U.device))
        s = torch.tensor(sign, dtype=U.dtype, device=U.device).view([-1 if a == 2 - d else 1 for a in range(3)])
        U = torch.cat([U[:V + d], (U[V + d] * s)[None], U[V + d + 1:]])
    return U


def _betas(a, b, c, d, e):
    k = 13.0 / 12.0
    return (k * (a - 2 * b + c) ** 2 + 0.25 * (a - 4 * b + 3 * c) ** 2, k * (b - 2 * c + d) ** 2 + 0.25 * (b - d) ** 2,
            k * (c - 2 * d + e) ** 2 + 0.25 * (3 * c - 4 * d + e) ** 2)


def _weno5z(v, eps):
    a, b, c, d, e = v[:5]
    b0, b1, b2 = _betas(a, b, c, d, e)
    tau = (b0 - b2).abs()
    w = [g * (1.0 + tau / (x + eps)) for g, x in ((0.1, b0), (0.6, b1), (0.3, b2))]
    q = (2 * a - 7 * b + 11 * c) / 6, (5 * c - b + 2 * d) / 6, (2 * c + 5 * d - e) / 6
    return (w[0] * q[0] + w[1] * q[1] + w[2] * q[2]) / (w[0] + w[1] + w[2])


def _teno_cut(v):
    """Adaptive cut-off of a face from its six cells."""
    e = 0.9 * 0.17 / (1.0 - 0.9 * 0.17) * 1e-6
    D = [v[k + 1] - v[k] for k in range(5)]
    eta = [((2 * D[k] * D[k + 1]).abs() + e) / (D[k] ** 2 + D[k + 1] ** 2 + e) for k in range(4)]
    low = torch.minimum(torch.minimum(eta[0], eta[1]), torch.minimum(eta[2], eta[3]))
    m = 1.0 - torch.clamp(low / 0.17, max=1.0)
    return 10.0 ** -torch.floor(10.5 - 3.5 * (1.0 - (1.0 - m) ** 4 * (1.0 + 4.0 * m)))


def _teno6a(v, eps, cut):
    a, b, c, d, e, f = v
    b0, b1, b2 = _betas(a, b, c, d, e)
    A, B, D, E, F = a - c, b - c, d - c, e - c, f - c
    b3 = (D * (11003 * D - 17246 * E + 4642 * F) + E * (7043 * E - 3882 * F) + 547 * F * F) / 240
    b6 = (A * (271779 * A - 2380800 * B - 3462252 * D + 1458762 * E - 245620 * F)
          + B * (5653317 * B + 17905032 * D - 7727988 * E + 1325006 * F)
          + D * (17195652 * D - 15880404 * E + 2863984 * F) + E * (3824847 * E - 1429976 * F) + 139633 * F * F) / 120960
    tau = (b6 - (b0 + 4 * b1 + b2) / 6).abs()
    es = [x + eps for x in (b0, b1, b2, b3)]
    em = torch.minimum(torch.minimum(es[0], es[1]), torch.minimum(es[2], es[3]))
    g = [(em / (em + tau) * (1.0 + tau / x)) ** 6 for x in es]
    limit = cut * sum(g)
    w = [torch.where(x >= limit, k, 0.0) for x, k in zip(g, (1.0, 9.0, 6.0, 4.0))]
    q = ((2 * a - 7 * b + 11 * c) / 6, (5 * c - b + 2 * d) / 6, (2 * c + 5 * d - e) / 6, (3 * c + 13 * d - 5 * e + f) / 12)
    return sum(x * y for x, y in zip(w, q)) / sum(w)


def _reconstruct(gas, w, d):
    """Both states of every face from the six cells w[0..5] around it."""
    cfg = gas.cfg

    def both(v):
        if cfg.scheme:
            cut = _teno_cut(v)
            return _teno6a(v, gas.weno_eps, cut), _teno6a(v[::-1], gas.weno_eps, cut)
        return _weno5z(v, gas.weno_eps), _weno5z(v[::-1], gas.weno_eps)

    if not cfg.recon:
        pairs = [both([x[m] for x in w]) for m in range(cfg.ncomp)]
        return torch.stack([p[0] for p in pairs]), torch.stack([p[1] for p in pairs])
    V, P = gas.V, gas.P
    mean = 0.5 * (w[2] + w[3])
    rc2 = gas.rhoc2(mean)
    z = torch.sqrt(gas.rho(mean) * rc2)
    minus = both([(x[P] - z * x[V + d]) / (2.0 * rc2) for x in w])
    plus = both([(x[P] + z * x[V + d]) / (2.0 * rc2) for x in w])
    sides = []
    kept = {m: both([x[m] for x in w]) for m in range(V, cfg.ncomp) if m not in (V + d, P)}
    dens = {m: both([x[m] - mean[m] / rc2 * x[P] for x in w]) for m in range(V)}
    for s in (0, 1):
        p = rc2 * (minus[s] + plus[s])
        comp = {P: p, V + d: (plus[s] - minus[s]) * rc2 / z}
        comp.update({m: v[s] for m, v in kept.items()})
        comp.update({m: v[s] + mean[m] / rc2 * p for m, v in dens.items()})
        sides.append(torch.stack([comp[m] for m in range(cfg.ncomp)]))
    return sides


def _thinc(W, wl_cells, grad, d, side):
    """THINC state of an interface cell's face: (mask, volume fraction)."""
    am, a0, ap = wl_cells
    inside = (a0 >= 1e-4) & (a0 <= 1.0 - 1e-4) & ((ap - a0) * (a0 - am) > 0)
    theta = torch.where(ap > am, 1.0, -1.0).to(a0.dtype)
    n2 = grad[0] ** 2 + grad[1] ** 2 + grad[2] ** 2
    beta = torch.where(inside, grad[d].abs() / torch.sqrt(torch.where(n2 > 0, n2, 1.0)) + 0.01, 1.0)
    T = (torch.exp(theta * beta * (2 * a0 - 1)) - torch.cosh(beta)) / torch.sinh(beta)
    if side:
        tb = torch.tanh(beta)
        T = (tb + T) / (1.0 + tb * T)
    return inside, 0.5 * (1.0 + theta * T)


def _hllc(gas, d, L, R):
    """(flux, upwinded normal velocity) between the states L and R."""
    V, P = gas.V, gas.P
    rL, rR, uL, uR = gas.rho(L), gas.rho(R), L[V + d], R[V + d]
    c2L, c2R = gas.rhoc2(L) / rL, gas.rhoc2(R) / rR
    qL, qR = torch.sqrt(rL), torch.sqrt(rR)
    ub = (qL * uL + qR * uR) / (qL + qR)
    cb = torch.sqrt((qL * c2L + qR * c2R) / (qL + qR) + 0.5 * qL * qR / (qL + qR) ** 2 * (uR - uL) ** 2)
    sL, sR = torch.minimum(ub - cb, uL - torch.sqrt(c2L)), torch.maximum(ub + cb, uR + torch.sqrt(c2R))
    mL, mR = rL * (sL - uL), rR * (sR - uR)
    star = (R[P] - L[P] + mL * uL - mR * uR) / (mL - mR)
    F = uh = 0.0
    for W, s, u, clip, weight in ((L, sL, uL, sL.clamp(max=0.0), (1.0 + torch.sign(star)) / 2),
                                  (R, sR, uR, sR.clamp(min=0.0), (1.0 - torch.sign(star)) / 2)):
        U, rho = gas.cons(W), gas.rho(W)
        fac = (s - u) / (s - star)
        Us = list(fac * U)
        Us[V + d] = fac * rho * star
        Us[P] = fac * (U[P] + (star - u) * (rho * star + W[P] / (s - u)))
        F = F + weight * (gas.flux(W, d) + clip * (torch.stack(Us) - U))
        uh = uh + weight * (u + clip * (fac - 1.0))
    return F, uh


def _inadmissible(gas, W):
    bad = gas.rhoc2(W) < gas.eps_rhoc2
    if gas.two:
        return bad | (W[0] < gas.eps_rho) | (W[1] < gas.eps_rho) | (W[6] < gas.eps_alpha) | (W[6] > 1.0 - gas.eps_alpha)
    return bad | (W[0] < gas.eps_rho)


def _viscous(gas, W, d, cut):
    """Dissipative flux (momentum, energy) of every face normal to d."""
    cfg, V = gas.cfg, gas.V
    h, six = (cfg.dx, cfg.dy, cfg.dz), cfg.visc_order == 6
    q = torch.cat([W[V:V + 3], (W[gas.P] / W[0])[None]])
    reach = 3 if six else 2

    def centred(f, e):
        """d f / d x_e at the cells whose e-coordinate is interior (others: unused)."""
        g = lambda k: torch.roll(f, -k, dims=2 - e)
        if six:
            return (45 * (g(1) - g(-1)) - 9 * (g(2) - g(-2)) + (g(3) - g(-3))) / (60 * h[e])
        return (8 * (g(1) - g(-1)) - (g(2) - g(-2))) / (12 * h[e])

    def face(f):
        v = [cut(f, k) for k in range(3 - reach, 3 + reach)]
        if six:
            return (150 * (v[2] + v[3]) - 25 * (v[1] + v[4]) + 3 * (v[0] + v[5])) / 256
        return (9 * (v[1] + v[2]) - (v[0] + v[3])) / 16

    def normal(f):
        v = [cut(f, k) for k in range(3 - reach, 3 + reach)]
        if six:
            return (2250 * (v[3] - v[2]) - 125 * (v[4] - v[1]) + 9 * (v[5] - v[0])) / (1920 * h[d])
        return (27 * (v[2] - v[1]) - (v[3] - v[0])) / (24 * h[d])

    dn = [normal(q[c]) for c in range(4)]
    tang = {e: (face(centred(q[d], e)), face(centred(q[e], e))) for e in range(3) if e != d}
    div = dn[d] + sum(t[1] for t in tang.values())
    tau = [cfg.mu * (2 * dn[d] - 2.0 / 3.0 * div) if e == d else cfg.mu * (tang[e][0] + dn[e]) for e in range(3)]
    kappa = cfg.mu * cfg.gamma1 / ((cfg.gamma1 - 1.0) * cfg.prandtl)
    return tau + [sum(face(q[e]) * tau[e] for e in range(3)) + kappa * dn[3]]


def _rhs(gas, U, dt):
    cfg, V, P = gas.cfg, gas.V, gas.P
    n3, h = (cfg.nx, cfg.ny, cfg.nz), (cfg.dx, cfg.dy, cfg.dz)
    W = gas.prim(_pad(cfg, U, V))
    R = torch.zeros_like(U)
    ndim = sum(n > 1 for n in n3)
    if cfg.thinc:
        a = W[6].clamp(0.0, 1.0)
        psi = a ** 0.1 / (a ** 0.1 + (1.0 - a) ** 0.1)
        grad = [(torch.roll(psi, -1, 2 - e) - torch.roll(psi, 1, 2 - e)) / (2 * h[e]) for e in range(3)]
    for d in range(3):
        def cut(f, k, d=d):
            """Cells f-3+k of every face f of direction d, interior in the other axes."""
            lead = f.dim() - 3
            for e in range(3):
                f = f.narrow(lead + 2 - e, k if e == d else 3, n3[e] + (1 if e == d else 0))
            return f

        w = [cut(W, k) for k in range(6)]
        L, Rt = _reconstruct(gas, w, d)
        if cfg.thinc:
            new = []
            for state, k, side in ((L, 2, 1), (Rt, 3, 0)):
                cells = [w[k + o][6] for o in (-1, 0, 1)]
                inside, af = _thinc(W, cells, [cut(g, k) for g in grad], d, side)
                comp = list(state)
                comp[6] = torch.where(inside, af, state[6])
                comp[0] = torch.where(inside, af * w[k][0] / w[k][6], state[0])
                comp[1] = torch.where(inside, (1.0 - af) * w[k][1] / (1.0 - w[k][6]), state[1])
                new.append(torch.stack(comp))
            L, Rt = new
        if gas.limited:
            L = torch.where(_inadmissible(gas, L), w[2], L)
            Rt = torch.where(_inadmissible(gas, Rt), w[3], Rt)
        F, uh = _hllc(gas, d, L, Rt)
        if gas.limited:
            lam, bad = 2 * ndim * dt / h[d], False
            for cell, sg in ((w[2], -lam), (w[3], lam)):
                Uc = gas.cons(cell)
                new = Uc + sg * (F - gas.flux(cell, d))
                if gas.two:
                    new[6] = Uc[6] + sg * (F[6] - Uc[6] * uh)
                bad = bad | _inadmissible(gas, gas.prim(new))
            F1, uh1 = _hllc(gas, d, w[2], w[3])
            F, uh = torch.where(bad, F1, F), torch.where(bad, uh1, uh)
        if cfg.model == S.NS:
            Fd = _viscous(gas, W, d, cut)
            F = torch.stack([F[0]] + [F[1 + c] - Fd[c] for c in range(4)])
        n, ax = n3[d], 3 - d
        R = R - (F.narrow(ax, 1, n) - F.narrow(ax, 0, n)) / h[d]
        if gas.two:
            source = U[6] * (uh.narrow(ax - 1, 1, n) - uh.narrow(ax - 1, 0, n)) / h[d]
            R = torch.cat([R[:6], (R[6] + source)[None]])
    return R


def _cfl_step(gas, U):
    cfg, W = gas.cfg, gas.prim(U)
    h = (cfg.dx, cfg.dy, cfg.dz)
    c = torch.sqrt(gas.rhoc2(W) / gas.rho(W))
    most = max(float(((W[gas.V + d].abs() + c) / h[d]).max()) for d in range(3))
    if cfg.model == S.NS:
        most = max(most, float((14.0 / 3.0 * cfg.mu / min(h) ** 2 / W[0]).max()))
    return cfg.cfl / most


def _rk3(gas, U, dt):
    U1 = U + dt * _rhs(gas, U, dt)
    U2 = 0.75 * U + 0.25 * U1 + 0.25 * dt * _rhs(gas, U1, dt)
    return U / 3.0 + 2.0 / 3.0 * U2 + 2.0 / 3.0 * dt * _rhs(gas, U2, dt)


def exact(case, seed):
    if case["call"] == "batch":
        return [exact(c, seed + 101 * i) for i, c in enumerate(_requests(case, seed))]
    cfg, U = _problem(case, seed)
    gas, U = _Gas(cfg), U.double()
    dt = _cfl_step(gas, U)
    if case["call"] == "rhs":
        return _rhs(gas, U, dt)
    if case["call"] == "stages":
        C = _rk3(gas, U, dt)
        return [C, torch.tensor([_cfl_step(gas, C)], dtype=torch.float64)]
    if case["call"] == "gradient":
        states = [U]
        for _ in range(case["steps"]):
            states.append(_rk3(gas, states[-1], dt).detach())
        last = states[-1].requires_grad_(True)
        loss = 0.5 * ((last[1:4] ** 2).sum(0) / last[0]).sum() * (cfg.dx * cfg.dy * cfg.dz)
        (grad,) = torch.autograd.grad(loss, last)
        for X in reversed(states[:-1]):     # one step's graph at a time
            X = X.detach().requires_grad_(True)
            (grad,) = torch.autograd.grad(_rk3(gas, X, dt), X, grad)
        return [loss.detach(), grad]
    for _ in range(case["steps"]):
        U = _rk3(gas, U, dt)
        dt = _cfl_step(gas, U)
    return U
