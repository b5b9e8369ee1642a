"""Linear operators of cells without enrichment, evaluated from 1-D operators,
against the CPU oracle's quadrature sums, FP64.

The meshes are the edges of the split: cell counts that leave a remainder in a
workgroup (9, 5, 3, 2 cells at k = 2..5), one cell along a periodic direction
(its own neighbour), layers that all touch an enriched one (ny = 3, 4), walls
without enrichment on one or both sides, no walls at all.  Tolerance 1e-12 of
the largest entry: both sides sum a few hundred products per entry in FP64
(about 1e3 eps).
"""
import numpy as np
import pytest
import torch

import oracle as O
from oracle.step import vorticity_rhs
from paper_1705_08813_amd import Mesh
from paper_1705_08813_amd.inputs import MeshConfig, Workload, draw_inputs

pytestmark = pytest.mark.gpu

RULE = {2: 4, 3: 5, 4: 7, 5: 8}


def _cfg(nx, ny, nz, k, lower=1, upper=1, per=0):
    return MeshConfig(nx=nx, ny=ny, nz=nz, gamma=0.0 if per else 1.2, k_u=k, k_p=k - 1, nq_u=RULE[k], nq_p=k, nq_wn=8,
                      nu=1.0 / 700, enrich_lower=lower, enrich_upper=upper, fully_periodic=per, theta=0.7)


MESHES = [
    _cfg(5, 5, 3, 2), _cfg(2, 6, 1, 2, upper=0), _cfg(1, 3, 3, 2, per=1),
    _cfg(3, 5, 3, 3), _cfg(1, 4, 2, 3, lower=0), _cfg(3, 2, 3, 3, lower=0, upper=0),
    _cfg(2, 7, 1, 4), _cfg(4, 3, 1, 4), _cfg(2, 3, 2, 4, per=1), _cfg(1, 4, 3, 4, upper=0),
    _cfg(1, 5, 3, 5), _cfg(3, 3, 1, 5, lower=0, upper=0),
]
IDS = [f"{c.nx}x{c.ny}x{c.nz}k{c.k_u}e{c.enrich_lower}{c.enrich_upper}p{c.fully_periodic}" for c in MESHES]


def _setup(cfg):
    print(f"[gpu] {cfg.nx}x{cfg.ny}x{cfg.nz} k={cfg.k_u}", flush=True)
    inp = draw_inputs(Workload("r", cfg, 71, 0.5, 1.5))
    return inp, Mesh(cfg, inp["tau"]), torch.tensor(inp["u"], device="cuda")


def _close(got, ref):
    err = np.abs(got.cpu().numpy() - ref).max() / max(np.abs(ref).max(), 1e-300)
    print(f"[gpu]   {err:.2e}", flush=True)
    assert err <= 1e-12


@pytest.mark.parametrize("cfg", MESHES, ids=IDS)
def test_viscous_operator(cfg):
    inp, mesh, u = _setup(cfg)
    nut = mesh.eddy_viscosity(u) if mesh.n_enriched else None
    ref = O.viscous_multiscale(cfg, inp["u"], u_nut=inp["u"], tau=inp["tau"])
    _close(mesh.apply_viscous_multiscale(nut, u), ref)


@pytest.mark.parametrize("cfg", MESHES, ids=IDS)
def test_viscous_operator_with_inverse_mass(cfg):
    """One Arnoldi step of a solve with gamma so large that x = b to rounding:
    the residual that it reports is M^{-1} A b over gamma b."""
    inp, mesh, u = _setup(cfg)
    nut = mesh.eddy_viscosity(u) if mesh.n_enriched else None
    k = mesh.apply_inverse_mass(mesh.apply_viscous_multiscale(nut, u))
    gamma = 3.0 * float(k.norm() / u.norm())
    _, st = mesh.solve_helmholtz(nut, gamma, u, u.clone(), rtol=0.5, max_iter=1)
    assert st.iterations == 0
    assert abs(st.rel_resid - 1.0 / 3.0) <= 1e-10


@pytest.mark.parametrize("cfg", MESHES, ids=IDS)
def test_gradient_and_divergence(cfg):
    inp, mesh, u = _setup(cfg)
    p = torch.tensor(inp["p"], device="cuda")
    _close(mesh.apply_pressure_gradient(p), O.pressure_gradient(cfg, inp["p"], tau=inp["tau"]))
    _close(mesh.apply_velocity_divergence(u), O.velocity_divergence(cfg, inp["u"], tau=inp["tau"]))


@pytest.mark.parametrize("cfg", MESHES, ids=IDS)
def test_vorticity(cfg):
    inp, mesh, u = _setup(cfg)
    b = mesh.vorticity_rhs(u)
    _close(b, vorticity_rhs(cfg, inp["u"], inp["tau"]))
    # the projection: M^{-1} of that vector (enriched cells by the same solver)
    om, mb = mesh.vorticity(u), mesh.apply_inverse_mass(b)
    assert float((om - mb).abs().max()) <= 1e-12 * float(mb.abs().max())


@pytest.mark.parametrize("cfg", MESHES, ids=IDS)
def test_residual(cfg):
    """Convective terms by the line-fused quadrature, viscous ones from 1-D
    operators, and the enriched neighbour's psi u~ on the interface faces."""
    inp, mesh, u = _setup(cfg)
    _close(mesh.apply_velocity_residual(u), O.velocity_residual(cfg, inp["u"], inp["tau"]))
    _close(mesh.apply_convective(u), O.convective_residual(cfg, inp["u"], inp["tau"]))
