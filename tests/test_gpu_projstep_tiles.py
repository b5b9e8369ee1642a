"""Projection step at the edges of its tiles, against the oracle's dense
per-cell solve: layers that fill a 16-cell tile exactly, leave one cell over or
hold a single one, four-cell tiles of enriched cells with a remainder, and
heights that differ from layer to layer (one table each), for every degree (the
reflection classes differ in size with k).  Tolerances and checks are those of
test_gpu_projstep.py."""
import numpy as np
import pytest
import torch

import oracle as O
from oracle import project as OP
from paper_1705_08813_amd import Mesh
from paper_1705_08813_amd.inputs import MeshConfig, Workload, draw_inputs
from test_gpu_projstep import _check

pytestmark = pytest.mark.gpu

RULE = {2: 4, 3: 5, 4: 7, 5: 8}


def _cfg(nx, ny, nz, k, **kw):
    return MeshConfig(nx=nx, ny=ny, nz=nz, gamma=1.1, k_u=k, k_p=k - 1, nq_u=RULE[k], nq_p=k, nq_wn=8, nu=1.0 / 700,
                      **kw)


@pytest.mark.parametrize("cfg", [_cfg(17, 4, 1, 2), _cfg(4, 3, 4, 3), _cfg(17, 2, 1, 4, enrich_upper=0),
                                 _cfg(1, 5, 1, 4), _cfg(4, 2, 4, 5, enrich_upper=0), _cfg(1, 3, 1, 5)],
                         ids=lambda c: f"{c.nx}x{c.ny}x{c.nz}k{c.k_u}")
def test_projection_step_tiles(cfg):
    print(f"[gpu] projection step {cfg.nx}x{cfg.ny}x{cfg.nz} k={cfg.k_u}", flush=True)
    inp = draw_inputs(Workload("ps", cfg, 31, 0.5, 1.5))
    g = np.random.default_rng(32).uniform(-1, 1, cfg.n_vel)
    tau_d = O.divdiv_tau(cfg, inp["u"], 0.05, tau=inp["tau"])
    psi4 = O.psi_volume4(cfg, O.enriched_cells(cfg), tau=inp["tau"])
    ref = OP.projection_step(cfg, inp["u"], g, 0.4, tau_d, psi4)
    _, conds = OP.inverse_mass(cfg, inp["u"], psi4[..., 0], return_cond=True)
    x = Mesh(cfg, inp["tau"]).projection_step(torch.tensor(tau_d, device="cuda"), torch.tensor(inp["u"], device="cuda"),
                                              torch.tensor(g, device="cuda"), 0.4).cpu().numpy()
    _check(cfg, x, ref, conds, range(cfg.ncell), (inp["u"], g, 0.4, tau_d, psi4))
