"""Cases that time this library the way a flow solver uses it.

Each case is one piece of a wall-modelled channel computation on the GPU, run
through the public entry points of the package:

  operators    the operator pass: psi refresh, velocity residual, Poisson apply
  solve        one pressure solve to 1e-10
  serve        the batched residual of many small channels (one per request)
  serve_solve  the batched pressure solves of like channels
  curved       the residual on the channel with a cosine lower wall
  projection   the pressure-projection substep (divergence, gradient, tau_D,
               element-wise projection)
  helmholtz    the eddy viscosity and the implicit viscous step (GMRES)
  step         one assembled dual-splitting time step
  refresh      what happens between two steps: nodal wall shear, psi from it,
               the velocity onto the new space, vorticity of the result

Velocities are a mean profile with random long waves and jumps of 0.3 u_tau between
the cells, as a running simulation holds them.  Random draws and references
are torch in FP64; the references use the definitions of the terms
(quadrature sums over cells and faces), not the library.
"""
import math

import numpy as np
import torch

import paper_1705_08813_amd as dg
from paper_1705_08813_amd.inputs import MeshConfig

# (velocity degree, Gauss points) with the pressure one degree below
RULES = {2: 4, 3: 5, 4: 7, 5: 8}


def _case(kind, nx, ny, nz, k, **kw):
    c = dict(kind=kind, nx=nx, ny=ny, nz=nz, k=k, nq=RULES[k], gamma=1.8, nu=1.0 / 180.0, f32=False)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: the 4^3 uniform box, all launch latency
        dict(_case("operators", 4, 4, 4, 3, nq=4, gamma=0.0), name="operators-tiny"),
        # the 64 x 32 x 32 channel, k = 4: the benchmark's operator pass
        dict(_case("operators", 64, 32, 32, 4), name="operators-channel"),
        # the same pass on single-precision vectors
        dict(_case("operators", 64, 32, 32, 4, f32=True), name="operators-channel-f32"),
        # the pressure solve of that channel (4.2 M unknowns), FP32 V-cycle
        dict(_case("solve", 64, 32, 32, 4, mixed=True), name="solve-channel"),
        # the pressure solve of a small channel, where launches bound the time
        dict(_case("solve", 16, 8, 8, 4, mixed=True), name="solve-small"),
        # one velocity round of a server: 24 channels of mixed grids and degrees
        dict(_case("serve", 16, 16, 16, 4, count=24, mixed_shapes=True), name="serve-round"),
        # eight like channels that solve together
        dict(_case("serve_solve", 16, 16, 16, 3, count=8, mixed=True), name="serve-solves"),
        # the curved-wall channel, 48 x 24 x 24, k = 5
        dict(_case("curved", 48, 24, 24, 5, gamma=0.0), name="curved-residual"),
        # the projection substep of the 64 x 32 x 32 channel
        dict(_case("projection", 64, 32, 32, 4, nu=1.0 / 2000.0), name="projection-channel"),
        # the implicit viscous step of the same channel
        dict(_case("helmholtz", 64, 32, 32, 4, nu=1.0 / 2000.0, dt=2e-4, enrich=0), name="helmholtz-channel"),
        # a whole time step on a quarter of it
        dict(_case("step", 32, 16, 32, 4, nu=1.0 / 950.0, dt=2e-4, order=2), name="time-step"),
        # the wall-shear and enrichment refresh between the steps
        dict(_case("refresh", 64, 32, 32, 4, nu=1.0 / 2000.0), name="wall-refresh"),
    ]


def draw(rng):
    def size(lo, hi):
        n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        return min(max(n, lo), hi)

    kind = rng.choice(["operators", "operators", "operators", "solve", "solve", "serve", "serve_solve", "curved",
                       "projection", "helmholtz", "step", "refresh"])
    k = rng.choice([2, 3, 4, 4, 5])
    nu = rng.choice([1.0 / 180.0, 1.0 / 395.0, 1.0 / 590.0, 1.0 / 950.0, 1.0 / 2000.0])
    gamma = rng.choice([0.0, 1.2, 1.8])
    if kind == "operators":
        nx, ny, nz = size(3, 64), size(3, 32), size(3, 32)
        if k == 5:
            nx, ny, nz = min(nx, 48), min(ny, 24), min(nz, 24)
        return _case(kind, nx, ny, nz, k, nu=nu, gamma=gamma, f32=rng.random() < 0.4)
    if kind == "solve":
        k = rng.choice([2, 3, 4, 5])
        # multigrid halves the even directions; odd ones stay small
        nx, ny, nz = rng.choice([4, 6, 8, 12, 16, 24, 32, 48]), rng.choice([4, 8, 12, 16, 24]), rng.choice([4, 5, 8, 12, 16, 24])
        return _case(kind, nx, ny, nz, k, nu=nu, gamma=gamma, mixed=rng.random() < 0.7)
    if kind == "serve":
        g = rng.choice([8, 9, 12, 16])
        return _case(kind, g, 8, size(4, 16), k, nu=nu, count=size(2, 24), mixed_shapes=rng.random() < 0.5)
    if kind == "serve_solve":
        nx, ny, nz = rng.choice([(8, 8, 8), (16, 8, 8), (16, 16, 16)])
        return _case(kind, nx, ny, nz, k, nu=nu, count=size(2, 12), mixed=rng.random() < 0.7)
    if kind == "curved":
        return _case(kind, size(4, 48), size(4, 24), size(3, 24), k, nu=nu, gamma=0.0, f32=rng.random() < 0.4)
    if kind == "projection":
        k = rng.choice([2, 3, 4])
        return _case(kind, size(3, 64), size(3, 16), size(3, 32), k, nu=min(nu, 1.0 / 950.0), gamma=gamma)
    if kind == "helmholtz":
        enrich = rng.choice([0, 0, 1])
        k = rng.choice([3, 4])
        return _case(kind, size(6, 32 if not enrich else 16), size(4, 16), size(6, 32 if not enrich else 16), k,
                     nu=min(nu, 1.0 / 590.0), gamma=1.2, dt=rng.choice([1e-4, 2e-4]), enrich=enrich)
    if kind == "step":
        k = rng.choice([3, 4])
        return _case(kind, rng.choice([8, 12, 16, 24, 32]), rng.choice([4, 8, 12, 16]), rng.choice([8, 9, 12, 16, 32]), k,
                     nu=min(nu, 1.0 / 590.0), gamma=1.2, dt=rng.choice([1e-4, 2e-4]), order=rng.choice([1, 2]))
    return _case(kind, size(3, 64), size(3, 32), size(3, 32), min(k, 4), nu=min(nu, 1.0 / 950.0), gamma=gamma)


# ------------------------------------------------------------- the inputs ---

def _config(c, **kw):
    d = dict(nx=c["nx"], ny=c["ny"], nz=c["nz"], gamma=c["gamma"], k_u=c["k"], k_p=c["k"] - 1, nq_u=c["nq"],
             nq_p=c["k"], nq_wn=8, nu=c["nu"], enrich_degree=c.get("enrich", 0))
    if c["kind"] == "curved":
        d["wall_amp"] = 0.3
    d.update(kw)
    return MeshConfig(**d)


def _legendre(n, x):
    p0, p1 = np.ones_like(x), x
    for j in range(2, n + 1):
        p0, p1 = p1, ((2 * j - 1) * x * p1 - (j - 1) * p0) / j
    return p1, n * (x * p1 - p0) / (x * x - 1)


def _gauss(n):
    """Gauss points and weights on [0, 1]."""
    x, w = np.polynomial.legendre.leggauss(n)
    for _ in range(3):
        p, dp = _legendre(n, x)
        x = x - p / dp
    w = 2.0 / ((1.0 - x * x) * _legendre(n, x)[1] ** 2)
    return 0.5 * (x + 1.0), 0.5 * w


def _lobatto(k):
    """The k + 1 Gauss-Lobatto nodes on [0, 1]."""
    c = np.zeros(k + 1)
    c[k] = 1.0
    d = np.polynomial.legendre.legder(c)
    x = np.sort(np.polynomial.legendre.legroots(d).real) if k > 1 else np.zeros(0)
    d2 = np.polynomial.legendre.legder(d)
    for _ in range(3):
        x = x - np.polynomial.legendre.legval(x, d) / np.polynomial.legendre.legval(x, d2)
    return 0.5 * (np.concatenate([[-1.0], x, [1.0]]) + 1.0)


def _basis(nodes, at):
    """Lagrange values and derivatives: [point][node]."""
    n = len(nodes)
    v, d = np.zeros((len(at), n)), np.zeros((len(at), n))
    for i in range(n):
        o = [j for j in range(n) if j != i]
        den = np.prod([nodes[i] - nodes[j] for j in o])
        v[:, i] = np.prod([at - nodes[j] for j in o], axis=0) / den
        for l in o:
            d[:, i] += np.prod([at - nodes[j] for j in o if j != l], axis=0) if n > 2 else 1.0
        d[:, i] /= den
    return v, d


def _vertices(cfg):
    s = 2.0 * np.arange(cfg.ny + 1) / cfg.ny - 1.0
    return np.tanh(cfg.gamma * s) / math.tanh(cfg.gamma) if cfg.gamma else s


def _coordinates(cfg, degree):
    """x, y, z of the nodes, shaped to broadcast over [ez, ey, ex, m, j, i]."""
    g, y = _lobatto(degree), _vertices(cfg)
    t = lambda a: torch.tensor(a, device="cuda")  # noqa: E731
    x = t((np.arange(cfg.nx)[:, None] + g) * cfg.Lx / cfg.nx).view(1, 1, cfg.nx, 1, 1, -1)
    z = t((np.arange(cfg.nz)[:, None] + g) * cfg.Lz / cfg.nz).view(cfg.nz, 1, 1, -1, 1, 1)
    return x, t(y[:-1, None] + np.diff(y)[:, None] * g).view(1, cfg.ny, 1, 1, -1, 1), z


def _random(seed, *shape):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return torch.rand(*shape, dtype=torch.float64, device="cuda", generator=gen) * 2 - 1


def _waves(cfg, degree, seed, count=4):
    """A sum of long waves at the nodes, of amplitude about one."""
    x, y, z = _coordinates(cfg, degree)
    r = np.random.default_rng(seed)
    f = 0
    for _ in range(count):
        kx, ky, kz = r.integers(1, 4), r.integers(1, 3), r.integers(1, 4)
        f = f + r.uniform(0.3, 0.6) * (torch.sin(2 * math.pi * kx * x / cfg.Lx + r.uniform(0, 6.3)) *
                                       torch.cos(math.pi * ky * y / 2 + r.uniform(0, 6.3)) *
                                       torch.sin(2 * math.pi * kz * z / cfg.Lz + r.uniform(0, 6.3)))
    return f


def _velocity(cfg, seed):
    """Wall units: a law-of-the-wall mean profile, long waves that vanish at the
    walls and small jumps; in the wall cells the enrichment (psi = u+ times a
    coefficient near one) carries the mean."""
    _, y, _ = _coordinates(cfg, cfg.k_u)
    yp = (1 - y.abs()).clamp_min(0) / cfg.nu
    mean = torch.log(1 + cfg.kappa * yp) / cfg.kappa + 7.8 * (1 - torch.exp(-yp / 11) - yp / 11 * torch.exp(-yp / 3))
    mean[:, 0] = 0
    mean[:, -1] = 0
    shape = (cfg.nz, cfg.ny, cfg.nx) + (cfg.k_u + 1,) * 3
    wall = 1 - y * y
    comp = [((mean if c == 0 else 0) + wall * _waves(cfg, cfg.k_u, 7 * seed + c)).expand(shape) for c in range(3)]
    u = torch.stack(comp, dim=3).reshape(-1) + 0.3 * _random(seed, cfg.ncell * 3 * (cfg.k_u + 1) ** 3)
    e = 0.02 * _random(seed + 1, cfg.n_enriched, 3, 1).expand(-1, -1, (cfg.enrich_degree + 1) ** 3).clone()
    if cfg.enrich_degree:
        e += 1e-3 * _random(seed + 2, *e.shape)
    e[:, 0] += 1.0
    return torch.cat([u, e.reshape(-1)])


def _tau(cfg, seed):
    """Wall shear stress at the Gauss points of the wall faces: about one, with
    long waves and small noise."""
    g, _ = _gauss(cfg.nq_u)
    x = ((np.arange(cfg.nx)[:, None] + g) / cfg.nx)[None, None, :, None, :]
    z = ((np.arange(cfg.nz)[:, None] + g) / cfg.nz)[None, :, None, :, None]
    r = np.random.default_rng(seed)
    a = r.uniform(0, 2 * math.pi, (2, 2, 1, 1, 1, 1))
    t = 1 + 0.3 * np.sin(4 * math.pi * x + a[0]) * np.sin(2 * math.pi * z + a[1])
    return (t + 0.05 * r.uniform(-1, 1, t.shape)).reshape(-1)


def _pressure(cfg, seed):
    return (_waves(cfg, cfg.k_p, seed).reshape(-1) + 0.02 * _random(seed + 2, cfg.n_p)).contiguous()


def _source(cfg, seed):
    """Right-hand side of the pressure equation: a smooth source and small
    jumps, tested with the nodal basis."""
    g, w = _gauss(cfg.k_p + 1)
    v, _ = _basis(_lobatto(cfg.k_p), g)
    m = v.T @ (w[:, None] * v)
    f = _waves(cfg, cfg.k_p, seed) + 0.05 * _random(seed, cfg.nz, cfg.ny, cfg.nx, *(cfg.k_p + 1,) * 3)
    t = torch.tensor(m, device="cuda")
    h = torch.tensor(np.diff(_vertices(cfg)), device="cuda").view(1, -1, 1, 1, 1, 1)
    return (_tensor(f, t, t, t) * h * (cfg.Lx / cfg.nx) * (cfg.Lz / cfg.nz)).reshape(-1).contiguous()


def _served(c):
    """The configurations of a server's round."""
    shapes = [(8, 8, 8), (16, 8, 8), (16, 16, 16), (32, 16, 16)]
    out = []
    for i in range(c["count"]):
        if c["mixed_shapes"]:
            (nx, ny, nz), k = shapes[i % 4], 2 + (i // 4 + i) % 4
        else:
            (nx, ny, nz), k = (c["nx"], c["ny"], c["nz"]), c["k"]
        out.append(MeshConfig(nx=nx, ny=ny, nz=nz, gamma=1.8, k_u=k, k_p=k - 1, nq_u=RULES[k], nq_p=k, nq_wn=8,
                              nu=c["nu"], omit_step_tables=1))
    return out


def _kept_solve(c, mesh):
    sp = mesh.solve_params(rtol=1e-10, mixed=c["mixed"])
    return sp, mesh.solve_workspace(sp)


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = dict(kind=kind, c=c)
    if kind == "serve":
        cfgs = _served(c)
        s["mesh"] = [dg.Mesh(f, _tau(f, seed + i)) for i, f in enumerate(cfgs)]
        s["u"] = [_velocity(f, seed + i) for i, f in enumerate(cfgs)]
        s["r"] = [torch.empty_like(u) for u in s["u"]]
        s["ws"] = dg.batch_workspace(len(cfgs))
        return s
    if kind == "serve_solve":
        f = _config(c, omit_step_tables=1)
        s["mesh"] = [dg.Mesh(f, _tau(f, seed + i)) for i in range(c["count"])]
        s["b"] = [_source(f, seed + i) for i in range(c["count"])]
        s["sp"] = s["mesh"][0].solve_params(rtol=1e-10, mixed=c["mixed"])
        s["ws"] = [m.solve_workspace(s["sp"]) for m in s["mesh"]]
        s["bws"] = dg.solve_batch_workspace(s["mesh"], s["sp"])
        return s
    f = _config(c)
    tau = _tau(f, seed)
    s["mesh"] = m = dg.Mesh(f, tau)
    if kind == "solve":
        s["b"] = _source(f, seed)
        s["sp"], s["ws"] = _kept_solve(c, m)
        return s
    s["u"] = u = _velocity(f, seed)
    s["p"] = _pressure(f, seed)
    if kind in ("operators", "curved"):
        s["tau"] = torch.tensor(tau, device="cuda")
        if c["f32"]:
            s["u"], s["p"] = u.float(), s["p"].float()
        s["r"] = torch.empty_like(s["u"])
        s["y"] = torch.empty_like(s["p"])
    elif kind == "projection":
        s["div"], s["grad"], s["x"] = torch.empty_like(s["p"]), torch.empty_like(u), torch.empty_like(u)
        s["taud"] = torch.empty(f.ncell, dtype=torch.float64, device="cuda")
        # a solver's tables of the mesh are built once, before its time loop
        m.projection_step(m.divdiv_tau(u, 0.05), u, torch.zeros_like(u), 0.0, s["x"])
    elif kind == "helmholtz":
        s["x"], s["nut"] = torch.empty_like(u), m.eddy_viscosity(u)
        gp = dg._lib.GmresParams(rtol=1e-10, max_iter=1000, restart=30)
        n = dg._lib.check(dg._lib.lib().dg_helmholtz_workspace_bytes(m.handle, dg.ctypes.byref(gp)))
        s["ws"] = torch.empty(int(n), dtype=torch.uint8, device="cuda")
    elif kind == "step":
        s["sp"] = m.step_params(c["dt"], order=c["order"], f=(1.0, 0.0, 0.0))
        n = dg._lib.check(dg._lib.lib().dg_step_workspace_bytes(m.handle, dg.ctypes.byref(s["sp"])))
        s["ws"] = torch.empty(int(n), dtype=torch.uint8, device="cuda")
        s["um"] = u * (1 - c["dt"]) if c["order"] == 2 else None
        s["un"], s["pn"] = torch.empty_like(u), torch.empty_like(s["p"])
        m.projection_step(m.divdiv_tau(u, 0.05), u, torch.zeros_like(u), 0.0, s["un"])
    else:
        s["nodes"] = torch.empty(2, f.nz, f.nx, dtype=torch.float64, device="cuda")
        s["new"], s["om"] = torch.empty_like(u), torch.empty_like(u)
    return s


def run(state):
    s, kind, m = state, state["kind"], state["mesh"]
    if kind == "operators":
        m.update_wall_shear(s["tau"])
        return [m.apply_velocity_residual(s["u"], s["r"]), m.apply_poisson(s["p"], s["y"])]
    if kind == "curved":
        m.update_wall_shear(s["tau"])
        return m.apply_velocity_residual(s["u"], s["r"])
    if kind == "solve":
        return m.solve_poisson(s["b"], sp=s["sp"], workspace=s["ws"])[0]
    if kind == "serve":
        return dg.apply_velocity_residual_batched(m, s["u"], s["r"], workspace=s["ws"])
    if kind == "serve_solve":
        return dg.solve_poisson_batched(m, s["b"], sp=s["sp"], workspaces=s["ws"], batch_ws=s["bws"])[0]
    if kind == "projection":
        m.apply_velocity_divergence(s["u"], s["div"])
        m.apply_pressure_gradient(s["p"], s["grad"])
        m.divdiv_tau(s["u"], 0.05, s["taud"])
        return [s["div"], s["grad"], s["taud"], m.projection_step(s["taud"], s["u"], s["grad"], 1e-3, s["x"])]
    if kind == "helmholtz":
        m.eddy_viscosity(s["u"], nut=s["nut"])
        s["x"].copy_(s["u"])
        return m.solve_helmholtz(s["nut"], 1.5 / s["c"]["dt"], s["u"], s["x"], rtol=1e-10, max_iter=1000,
                                 workspace=s["ws"])[0]
    if kind == "step":
        s["pn"].copy_(s["p"])
        return list(m.dual_splitting_step(s["sp"], s["u"], s["um"], s["pn"], u_np1=s["un"], workspace=s["ws"])[:2])
    # refresh: every pass starts from the same velocity and writes a new vector
    m.wall_shear_nodes(s["u"], s["nodes"])
    m.update_wall_shear_nodes(s["nodes"])
    m.project_velocity(s["u"], s["new"])
    return [s["nodes"], s["new"], m.vorticity_rhs(s["new"], s["om"])]


# ---------------------------------------------------------------- the work ---

def _vel_flops(cfg):
    """Sum-factorized residual: interpolation of three components, products,
    six face planes, and the transposed sweeps."""
    n, q = cfg.k_u + 1, cfg.nq_u
    vol = 2 * 3 * 2 * (n * n * n * q + n * n * q * q + n * q * q * q) + 2 * 2 * 9 * q ** 4
    face = 6 * 2 * 2 * 8 * (n * n * q + n * q * q)
    return cfg.ncell * (vol + face)


def _poisson_flops(cfg):
    n = cfg.k_p + 1
    return cfg.ncell * 2 * 9 * n ** 4


def work(case):
    """Inputs read and outputs written once.  Solves count the applications
    that their iterations cannot do without (about 20 with multigrid, 10 of
    the implicit viscous step), each with its vector read and written."""
    c, kind = case, case["kind"]
    if kind == "serve":
        fs = _served(c)
        return {"bytes": sum(16.0 * f.n_vel for f in fs), "flops": float(sum(_vel_flops(f) for f in fs))}
    f = _config(c)
    b = 4.0 if c["f32"] else 8.0
    if kind in ("operators", "curved"):
        extra = 2 * b * f.n_p if kind == "operators" else 0.0
        return {"bytes": 2 * b * f.n_vel + extra + 8.0 * f.n_tau,
                "flops": float(_vel_flops(f) + (_poisson_flops(f) if kind == "operators" else 0))}
    if kind in ("solve", "serve_solve"):
        n = c.get("count", 1)
        return {"bytes": n * 20 * 16.0 * f.n_p, "flops": float(n * 20 * _poisson_flops(f))}
    if kind == "projection":
        dofs = 3 * (f.k_u + 1) ** 3
        return {"bytes": 8.0 * (6 * f.n_vel + 2 * f.n_p + 2 * f.ncell), "flops": 4.0 * f.ncell * dofs * dofs}
    if kind == "helmholtz":
        return {"bytes": 10 * 4 * 8.0 * f.n_vel, "flops": 10.0 * _vel_flops(f)}
    if kind == "step":
        return {"bytes": 8.0 * (40 * f.n_vel + 60 * f.n_p), "flops": 12.0 * _vel_flops(f)}
    return {"bytes": 8.0 * (4 * f.n_vel + 2 * f.nx * f.nz), "flops": 2.0 * f.n_vel * 9 * (f.k_u + 1)}


# ---------------------------------------------------- references in 64 bits ---

def _tensor(a, mx, my, mz):
    """Three 1-D matrices along the last three axes (z, y, x) of a."""
    a = a @ mx.T
    a = torch.matmul(my, a)
    return torch.matmul(mz, a.flatten(-2)).unflatten(-1, a.shape[-2:])


class _Reference:
    """The terms of the flat channel by quadrature, one cell layer at a time."""

    def __init__(self, cfg, tau):
        t = lambda a: torch.tensor(np.ascontiguousarray(a), device="cuda")  # noqa: E731
        self.cfg, self.t = cfg, t
        self.y = _vertices(cfg)
        self.hx, self.hz, self.hy = cfg.Lx / cfg.nx, cfg.Lz / cfg.nz, np.diff(self.y)
        self.nodes = _lobatto(cfg.k_u)
        self.tau = t(tau).view(2, cfg.nz, cfg.nx, cfg.nq_u, cfg.nq_u)
        self.pen = cfg.ip_factor_u * (cfg.k_u + 1) ** 2

    def enriched(self, ey):
        c = self.cfg
        return (ey == 0 and c.enrich_lower) or (ey == c.ny - 1 and c.enrich_upper)

    def split(self, u):
        c = self.cfg
        n = c.ncell * 3 * (c.k_u + 1) ** 3
        return (u[:n].view(c.nz, c.ny, c.nx, 3, *(c.k_u + 1,) * 3),
                u[n:].view(c.nz, -1, c.nx, 3) if u.numel() > n else None)

    def points(self, ey, face=None, nq_y=None):
        """1-D points and weights (x, y, z) of the volume or a face of layer ey;
        a face has one point, at its place, along its normal."""
        c = self.cfg
        n = [c.nq_u, nq_y or (c.nq_wn if self.enriched(ey) else c.nq_u), c.nq_u]
        r = [_gauss(q) for q in n]
        if face is not None:
            r[face // 2] = (np.array([float(face % 2)]), np.ones(1))
        return r

    def psi(self, ey, pts):
        """psi and its wall-normal derivative at the points, [nz, nx, 1, qz, qy, qx]."""
        c = self.cfg
        lower = ey == 0
        g, _ = _gauss(c.nq_u)
        ix = [int(np.argmin(abs(g - v))) for v in pts[0][0]]
        iz = [int(np.argmin(abs(g - v))) for v in pts[2][0]]
        root = torch.sqrt(self.tau[0 if lower else 1][:, :, iz][:, :, :, ix])[:, :, None, :, None, :]
        yy = self.y[ey] + self.hy[ey] * pts[1][0]
        d = self.t(yy + 1.0 if lower else 1.0 - yy).view(1, 1, 1, 1, -1, 1)
        yp = d * root / c.nu
        k, e = c.kappa, math.exp(-c.kappa * c.B)
        U = torch.minimum(yp, torch.log(yp.clamp_min(1e-30) / e + 1) / k + 1e-300)
        for _ in range(60):  # y+ = U + e^{-kB} (e^{kU} - 1 - kU - (kU)^2/2 - (kU)^3/6): increasing, convex
            q = k * U
            f = U + e * (torch.exp(q) - 1 - q - q * q / 2 - q ** 3 / 6) - yp
            U = U - f / (1 + e * k * (torch.exp(q) - 1 - q - q * q / 2))
        q = k * U
        dU = 1 / (1 + e * k * (torch.exp(q) - 1 - q - q * q / 2))
        return U, dU * root / c.nu * (1.0 if lower else -1.0)

    def mats(self, ey, pts, nodes=None):
        """Values and physical derivatives of the 1-D bases at the points."""
        h = (self.hx, self.hy[ey], self.hz)
        out = []
        for (g, _), hh in zip(pts, h):
            v, d = _basis(self.nodes if nodes is None else nodes, g)
            out.append((self.t(v), self.t(d / hh)))
        return out

    @staticmethod
    def at(a, mats, d=None):
        return _tensor(a, *(mats[i][1 if i == d else 0] for i in range(3)))

    @staticmethod
    def test(f, mats, d=None):
        return _tensor(f, *(mats[i][1 if i == d else 0].T for i in range(3)))

    def field(self, u, ey, pts):
        """u and grad u [.., c, (d)] at points of layer ey, enrichment included."""
        poly, enr = self.split(u)
        mats = self.mats(ey, pts)
        a = poly[:, ey]
        v = self.at(a, mats)
        g = torch.stack([self.at(a, mats, d) for d in range(3)], dim=3)
        if self.enriched(ey):
            ps, dps = self.psi(ey, pts)
            w = enr[:, 0 if ey == 0 or not self.cfg.enrich_lower else 1].view(*a.shape[:3], 1, 1, 1)
            v = v + ps * w
            g[:, :, :, 1] += dps * w
        return v, g

    def weights(self, ey, pts, face=None):
        w = [self.t(p[1] * (1.0 if face is not None and i == face // 2 else h))
             for i, (p, h) in enumerate(zip(pts, (self.hx, self.hy[ey], self.hz)))]
        return w[2].view(-1, 1, 1) * w[1].view(-1, 1) * w[0]

    def other(self, ey, face):
        """Layer across the face and the shift that brings its cells here."""
        d, s = face // 2, face % 2
        if d != 1:
            return ey, lambda a: torch.roll(a, -1 if s else 1, dims=1 if d == 0 else 0)
        n = ey + (1 if s else -1)
        return (n if 0 <= n < self.cfg.ny else None), lambda a: a

    def layers(self, rows):
        """Assemble per-layer (polynomial, enrichment) rows into one vector."""
        poly = torch.stack([r[0] for r in rows], dim=1).reshape(-1)
        enr = [r[1] for r in rows if r[1] is not None]
        return torch.cat([poly, torch.stack(enr, dim=1).reshape(-1)]) if enr else poly

    def rows(self, ey, pts, val, grad):
        """Tests of a value field [.., c] and a gradient field [.., c, d]."""
        mats = self.mats(ey, pts)
        r = self.test(val, mats) if val is not None else 0
        if grad is not None:
            for d in range(3):
                r = r + self.test(grad[:, :, :, d], mats, d)
        e = None
        if self.enriched(ey):
            ps, dps = self.psi(ey, pts)
            e = (0 if val is None else val * ps) + (0 if grad is None else grad[:, :, :, 1] * dps)
            e = e.sum((-1, -2, -3))
        return r, e

    def residual(self, u):
        c, out = self.cfg, []
        for ey in range(c.ny):
            pts = self.points(ey)
            v, g = self.field(u, ey, pts)
            G = (c.nu * (g + g.transpose(2, 3)) - v[:, :, :, None] * v[:, :, None]) * self.weights(ey, pts)
            acc = list(self.rows(ey, pts, None, G))
            for face in range(6):
                d, n = face // 2, 1.0 if face % 2 else -1.0
                pts = self.points(ey, face)
                vm, gm = self.field(u, ey, pts)
                ny, shift = self.other(ey, face)
                h = (self.hx, self.hy[ey], self.hz)[d]
                pen = self.pen / h
                if ny is None:
                    vp, gp, pen = -vm, gm, pen * c.wall_ip_mult
                else:
                    q = self.points(ny, face ^ 1, len(pts[1][0]) if d != 1 else None)
                    vp, gp = (shift(a) for a in self.field(u, ny, q))
                    if d == 1:
                        pen = self.pen / min(h, self.hy[ny])
                un, up = n * vm[:, :, d:d + 1], n * vp[:, :, d:d + 1]
                lam, j = 2 * torch.maximum(un.abs(), up.abs()), vm - vp
                sym = n * ((gm[:, :, :, d] + gm[:, :, d]) + (gp[:, :, :, d] + gp[:, :, d]))
                fv = 0.5 * (vm * un + vp * up) + 0.5 * lam * j - 0.5 * c.nu * sym + pen * c.nu * j
                F = torch.zeros_like(gm)
                F[:, :, :, d] += -0.5 * c.theta * c.nu * n * j
                F[:, :, d] += -0.5 * c.theta * c.nu * n * j
                w = self.weights(ey, pts, face)
                r, e = self.rows(ey, pts, fv * w, F * w)
                acc[0] = acc[0] + r
                if e is not None:
                    acc[1] = acc[1] + e
            out.append(acc)
        return self.layers(out)

    def pressure_mats(self, ey, pts):
        return self.mats(ey, pts, _lobatto(self.cfg.k_p))

    def gradient(self, p):
        c, out = self.cfg, []
        p = p.view(c.nz, c.ny, c.nx, 1, *(c.k_p + 1,) * 3)
        for ey in range(c.ny):
            pts = self.points(ey)
            pq = self.at(p[:, ey], self.pressure_mats(ey, pts)) * self.weights(ey, pts)
            G = torch.zeros(*pq.shape[:2], 3, 3, *pq.shape[3:], dtype=torch.float64, device="cuda")
            for d in range(3):
                G[:, :, d, d] = -pq[:, :, 0]
            acc = list(self.rows(ey, pts, None, G))
            for face in range(6):
                d, n = face // 2, 1.0 if face % 2 else -1.0
                pts = self.points(ey, face)
                pm = self.at(p[:, ey], self.pressure_mats(ey, pts))
                ny, shift = self.other(ey, face)
                if ny is not None:
                    q = self.points(ny, face ^ 1, len(pts[1][0]) if d != 1 else None)
                    pm = 0.5 * (pm + shift(self.at(p[:, ny], self.pressure_mats(ny, q))))
                V = torch.zeros(*pm.shape[:2], 3, *pm.shape[3:], dtype=torch.float64, device="cuda")
                V[:, :, d] = n * pm[:, :, 0] * self.weights(ey, pts, face)
                r, e = self.rows(ey, pts, V, None)
                acc[0] = acc[0] + r
                if e is not None:
                    acc[1] = acc[1] + e
            out.append(acc)
        return self.layers(out)

    def divergence(self, u):
        c, out = self.cfg, []
        for ey in range(c.ny):
            pts = self.points(ey)
            v, _ = self.field(u, ey, pts)
            v, m = v * self.weights(ey, pts), self.pressure_mats(ey, pts)
            r = -sum(self.test(v[:, :, d], m, d) for d in range(3))
            for face in range(6):
                d, n = face // 2, 1.0 if face % 2 else -1.0
                pts = self.points(ey, face)
                vm = self.field(u, ey, pts)[0][:, :, d]
                ny, shift = self.other(ey, face)
                if ny is not None:
                    q = self.points(ny, face ^ 1, len(pts[1][0]) if d != 1 else None)
                    vm = 0.5 * (vm + shift(self.field(u, ny, q)[0][:, :, d]))
                r = r + self.test(n * vm * self.weights(ey, pts, face), self.pressure_mats(ey, pts))
            out.append(r)
        return torch.stack(out, dim=1).reshape(-1)

    def penalty(self, u, dt_over_cr):
        c, out = self.cfg, []
        for ey in range(c.ny):
            pts = self.points(ey)
            v, _ = self.field(u, ey, pts)
            vol = self.hx * self.hy[ey] * self.hz
            mean = (v.square().sum(2).sqrt() * self.weights(ey, pts)).sum((-1, -2, -3)) / vol
            out.append(mean * vol ** (1.0 / 3.0) * dt_over_cr)
        return torch.stack(out, dim=1).reshape(-1)


def _line(cells, h, periodic, k, pen):
    """1-D mass and interior-penalty stiffness matrices of a line of cells."""
    nodes, n = _lobatto(k), k + 1
    g, w = _gauss(n)
    v, d = _basis(nodes, g)
    ends = [_basis(nodes, np.array([e])) for e in (0.0, 1.0)]
    M, A = np.zeros((cells * n, cells * n)), np.zeros((cells * n, cells * n))
    for e in range(cells):
        i = slice(e * n, e * n + n)
        M[i, i] += h[e] * (v.T @ (w[:, None] * v))
        A[i, i] += d.T @ (w[:, None] * d) / h[e]
    for e in range(cells if periodic else cells - 1):
        f = (e + 1) % cells
        jump, mean = np.zeros(cells * n), np.zeros(cells * n)
        jump[e * n:e * n + n] += ends[1][0][0]
        jump[f * n:f * n + n] -= ends[0][0][0]
        mean[e * n:e * n + n] += 0.5 * ends[1][1][0] / h[e]
        mean[f * n:f * n + n] += 0.5 * ends[0][1][0] / h[f]
        A += pen / min(h[e], h[f]) * np.outer(jump, jump) - np.outer(mean, jump) - np.outer(jump, mean)
    return torch.tensor(M, device="cuda"), torch.tensor(A, device="cuda")


def _lines(cfg):
    pen = cfg.ip_factor_p * (cfg.k_p + 1) ** 2
    return [_line(cfg.nx, [cfg.Lx / cfg.nx] * cfg.nx, True, cfg.k_p, pen),
            _line(cfg.ny, list(np.diff(_vertices(cfg))), False, cfg.k_p, pen),
            _line(cfg.nz, [cfg.Lz / cfg.nz] * cfg.nz, True, cfg.k_p, pen)]


def _grid(cfg, p, back=False):
    """Cell-wise pressure vector to a [z, y, x] array of all nodes, or back."""
    n = cfg.k_p + 1
    if back:
        return p.view(cfg.nz, n, cfg.ny, n, cfg.nx, n).permute(0, 2, 4, 1, 3, 5).reshape(-1)
    return p.view(cfg.nz, cfg.ny, cfg.nx, n, n, n).permute(0, 3, 1, 4, 2, 5).reshape(cfg.nz * n, cfg.ny * n, cfg.nx * n)


def _poisson(cfg, p):
    (mx, ax), (my, ay), (mz, az) = _lines(cfg)
    a = _grid(cfg, p)
    return _grid(cfg, _tensor(a, ax, my, mz) + _tensor(a, mx, ay, mz) + _tensor(a, mx, my, az), back=True)


def _poisson_solve(cfg, b):
    """Zero-mean solution by diagonalising the three 1-D pencils."""
    vs, ls = [], []
    for m, a in _lines(cfg):
        c = torch.linalg.inv(torch.linalg.cholesky(m))
        l, q = torch.linalg.eigh(c @ a @ c.T)
        l[0] = 0.0  # constants
        vs.append(c.T @ q)
        ls.append(l)
    f = _tensor(_grid(cfg, b - b.mean()), *(v.T for v in vs))
    lam = ls[2].view(-1, 1, 1) + ls[1].view(-1, 1) + ls[0]
    lam[0, 0, 0] = math.inf
    x = _grid(cfg, _tensor(f / lam, *vs), back=True)
    return x - x.mean()


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "serve":
        return [_Reference(f, _tau(f, seed + i)).residual(_velocity(f, seed + i)) for i, f in enumerate(_served(c))]
    f = _config(c)
    if kind == "solve":
        return _poisson_solve(f, _source(f, seed))
    if kind == "serve_solve":
        return [_poisson_solve(f, _source(f, seed + i)) for i in range(c["count"])]
    if kind == "operators":
        u, p = _velocity(f, seed), _pressure(f, seed)
        if c["f32"]:
            u, p = u.float().double(), p.float().double()
        return [_Reference(f, _tau(f, seed)).residual(u), _poisson(f, p)]
    if kind == "projection":
        ref, u = _Reference(f, _tau(f, seed)), _velocity(f, seed)
        return [ref.divergence(u), ref.gradient(_pressure(f, seed)), ref.penalty(u, 0.05), None]
    # curved cells, Krylov solves and whole steps have no closed form here
    return None
