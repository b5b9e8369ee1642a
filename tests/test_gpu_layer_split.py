"""Operators that take the cells next to an enriched layer apart from the others
once a mesh is large enough, on both sides of that line, against the CPU oracle
on sampled cells (every layer, both ends of the mesh).

Of each pair of meshes the first has as many cells without enrichment as fit the
chip at once and runs one general launch for them, the second a few more and runs
interior and interface layers (1 to 5 layers apart, or one) in launches of their
own, with remainders in the interior's workgroups.  FP64 to 1e-12 of the largest
sampled entry, as in test_gpu_regular_cells.py."""
import numpy as np
import pytest
import torch

import oracle as O
from oracle import project as OP
from oracle import step as OS
from paper_1705_08813_amd import Mesh
from paper_1705_08813_amd.inputs import MeshConfig, Workload, draw_inputs

pytestmark = pytest.mark.gpu

RULE = {2: 4, 3: 5, 4: 7, 5: 8}


def _cfg(nx, ny, nz, k, **kw):
    return MeshConfig(nx=nx, ny=ny, nz=nz, gamma=1.2, k_u=k, k_p=k - 1, nq_u=RULE[k], nq_p=k, nq_wn=8, nu=1.0 / 700,
                      theta=0.7, **kw)


def _id(c):
    return f"{c.nx}x{c.ny}x{c.nz}k{c.k_u}e{c.enrich_lower}{c.enrich_upper}l{c.enrich_degree}"


def _sample(cfg, per_layer=4):
    """Cells of every layer, the mesh's first and last among them."""
    rng = np.random.default_rng(5)
    cells = {0, cfg.ncell - 1}
    for ey in range(cfg.ny):
        for _ in range(per_layer):
            cells.add(int(rng.integers(0, cfg.nx)) + cfg.nx * (ey + cfg.ny * int(rng.integers(0, cfg.nz))))
    return np.array(sorted(cells), dtype=np.int64)


def _rows(cells, n):
    return (cells[:, None] * n + np.arange(n)[None, :]).ravel()


def _close(got, ref, rows, tol=1e-12):
    err = np.abs(got[rows] - ref[rows]).max() / np.abs(ref[rows]).max()
    print(f"[gpu]   {err:.2e}", flush=True)
    assert err <= tol


@pytest.mark.parametrize("cfg", [
    _cfg(32, 5, 16, 2), _cfg(27, 5, 19, 2), _cfg(307, 7, 1, 3), _cfg(28, 7, 11, 3),
    _cfg(16, 4, 32, 4, enrich_upper=0), _cfg(27, 4, 19, 4, enrich_upper=0), _cfg(27, 4, 19, 4, enrich_lower=0),
    _cfg(20, 6, 16, 5), _cfg(19, 6, 17, 5), _cfg(28, 7, 11, 3, enrich_degree=1)], ids=_id)
def test_divergence(cfg):
    print(f"[gpu] divergence {_id(cfg)}", flush=True)
    inp = draw_inputs(Workload("ls", cfg, 61, 0.5, 1.5))
    cells = _sample(cfg)
    c = Mesh(cfg, inp["tau"]).apply_velocity_divergence(torch.tensor(inp["u"], device="cuda")).cpu().numpy()
    _close(c, O.velocity_divergence(cfg, inp["u"], tau=inp["tau"], cells=cells), _rows(cells, (cfg.k_p + 1) ** 3))


# Degree-1 enrichment: three cells a CU for the FP64 residual, four for FP32 and the viscous operator; both walls
# enriched with one to five layers between the interface layers, and one wall.
L1 = [_cfg(20, 6, 16, 2, enrich_degree=1), _cfg(23, 5, 15, 2, enrich_degree=1), _cfg(32, 4, 16, 3, enrich_degree=1),
      _cfg(31, 7, 9, 3, enrich_degree=1), _cfg(27, 5, 13, 4, enrich_degree=1), _cfg(19, 6, 14, 4, enrich_degree=1),
      _cfg(33, 4, 11, 4, enrich_degree=1, enrich_upper=0), _cfg(33, 4, 11, 4, enrich_degree=1, enrich_lower=0)]


@pytest.mark.parametrize("cfg", L1, ids=_id)
def test_l1_residual(cfg):
    print(f"[gpu] l=1 residual {_id(cfg)}", flush=True)
    inp = draw_inputs(Workload("ls", cfg, 62, 0.5, 1.5))
    cells = _sample(cfg)
    rows = _rows(cells, 3 * (cfg.k_u + 1) ** 3)
    mesh = Mesh(cfg, inp["tau"])
    u = torch.tensor(inp["u"], device="cuda")
    _close(mesh.apply_velocity_residual(u).cpu().numpy(), O.velocity_residual(cfg, inp["u"], inp["tau"], cells=cells), rows)
    _close(mesh.apply_convective(u).cpu().numpy(), O.convective_residual(cfg, inp["u"], inp["tau"], cells=cells), rows)
    # FP32: element by element within 4 m u32 R_abs, as in test_gpu_enrich_l1.py
    u32 = inp["u"].astype(np.float32)
    u_r = u32.astype(np.float64)
    ref = O.velocity_residual(cfg, u_r, inp["tau"], cells=cells)[rows]
    bound = 4 * (3 * (cfg.nq_u + cfg.k_u + 1) + 40) * 2.0 ** -24 * O.velocity_residual(cfg, u_r, inp["tau"], cells=cells,
                                                                                     absmode=True)[rows]
    r = mesh.apply_velocity_residual(torch.tensor(u32, device="cuda")).cpu().numpy()[rows].astype(np.float64)
    assert np.all(np.abs(r - ref) <= bound + 1e-30)


@pytest.mark.parametrize("cfg", L1, ids=_id)
def test_l1_viscous_operator(cfg):
    print(f"[gpu] l=1 viscous {_id(cfg)}", flush=True)
    inp = draw_inputs(Workload("ls", cfg, 63, 0.5, 1.5))
    cells = _sample(cfg)
    mesh = Mesh(cfg, inp["tau"])
    u = torch.tensor(inp["u"], device="cuda")
    out = mesh.apply_viscous_multiscale(mesh.eddy_viscosity(u), u).cpu().numpy()
    _close(out, O.viscous_multiscale(cfg, inp["u"], u_nut=inp["u"], tau=inp["tau"], cells=cells),
           _rows(cells, 3 * (cfg.k_u + 1) ** 3))


@pytest.mark.parametrize("cfg", [L1[0], L1[3]], ids=_id)
def test_l1_helmholtz(cfg):
    """M^{-1} A of the solve (interior cells in one pass, the interface layers by
    the general operator and the inverse mass matrix of those layers), by the
    forward residual of the equation with the oracle's operators, to the bound
    of test_gpu_enrich_l1.py."""
    print(f"[gpu] l=1 helmholtz {_id(cfg)}", flush=True)
    inp = draw_inputs(Workload("ls", cfg, 64, 0.5, 1.5))
    mesh = Mesh(cfg, inp["tau"])
    b = np.random.default_rng(65).uniform(-1, 1, cfg.n_vel)
    gamma = 300.0
    nut = mesh.eddy_viscosity(torch.tensor(inp["u"], device="cuda"))
    x, st = mesh.solve_helmholtz(nut, gamma, torch.tensor(b, device="cuda"), rtol=1e-10,
                                 max_iter=20000)  # (restarted GMRES without preconditioner: thousands here)
    res = OS.helmholtz_residual(cfg, inp["u"], inp["tau"], gamma, b, x.cpu().numpy())
    psi = O.psi_volume(cfg, O.enriched_cells(cfg), tau=inp["tau"])
    scale = gamma * np.abs(OP.mass_apply(cfg, b, psi)).max()
    print(f"[gpu]   its {st.iterations} forward residual {np.abs(res).max() / scale:.1e}", flush=True)
    assert st.rel_resid <= 1e-10
    assert np.abs(res).max() <= 1e-8 * scale
