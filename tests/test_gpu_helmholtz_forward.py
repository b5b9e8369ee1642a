"""The Helmholtz solve's operator M^{-1} A entry by entry, on the meshes at the
edges of the regular cells' kernels: M^{-1} A runs inside the solve only, so the
solution's forward residual gamma M x + A x - gamma M b is formed with the
oracle's operators.  A component, line or sign mixed up in the fused kernel gives
the solution of another system and a residual of the size of A x / (gamma M x),
about a third here.  Bounds as in test_gpu_enrich_l1.py: 1e-10 for GMRES's own
residual, 1e-8 of the right-hand side's largest entry for the forward one."""
import numpy as np
import pytest
import torch

import oracle as O
from oracle import project as OP
from oracle import step as OS
from test_gpu_regular_cells import IDS, MESHES, _setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg", MESHES, ids=IDS)
def test_forward_residual(cfg):
    inp, mesh, u = _setup(cfg)
    nut = mesh.eddy_viscosity(u) if mesh.n_enriched else None
    k = mesh.apply_inverse_mass(mesh.apply_viscous_multiscale(nut, u))
    gamma = 3.0 * float(k.norm() / u.norm())
    b = np.random.default_rng(72).uniform(-1, 1, cfg.n_vel)
    x, st = mesh.solve_helmholtz(nut, gamma, torch.tensor(b, device="cuda"), rtol=1e-10, max_iter=20000)
    res = OS.helmholtz_residual(cfg, inp["u"] if mesh.n_enriched else None, inp["tau"], gamma, b, x.cpu().numpy())
    psi = O.psi_volume(cfg, O.enriched_cells(cfg), tau=inp["tau"])
    scale = gamma * np.abs(OP.mass_apply(cfg, b, psi)).max()
    print(f"[gpu]   its {st.iterations} forward residual {np.abs(res).max() / scale:.1e}", flush=True)
    assert st.rel_resid <= 1e-10
    assert np.abs(res).max() <= 1e-8 * scale
