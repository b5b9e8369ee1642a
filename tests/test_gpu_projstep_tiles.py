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


def test_step_tables_write_only_what_they_need():
    """The mesh workspace reserves at least one layer's dense n x n pair for the
    step tables; the class tables of one height are smaller, and the rest of the
    reservation is neither formed on the host nor copied: it keeps what the
    workspace held."""
    import ctypes
    from paper_1705_08813_amd import _lib
    cfg = MeshConfig(nx=2, ny=2, nz=2, gamma=0.0, k_u=5, k_p=4, nq_u=8, nq_p=5, fully_periodic=1)
    print("[gpu] projection step tables", flush=True)
    L, prm = _lib.lib(), _lib.params_from(cfg)
    nbytes = _lib.check(L.dg_mesh_workspace_bytes(ctypes.byref(prm)))
    mesh = Mesh.__new__(Mesh)
    mesh.cfg, mesh.params, mesh.device = cfg, prm, torch.device("cuda", 0)
    mesh.workspace = torch.full((nbytes,), 0xA5, dtype=torch.uint8, device="cuda")
    mesh.handle = ctypes.c_void_p()
    _lib.check(L.dg_setup_mesh(ctypes.byref(prm), None, ctypes.c_void_p(mesh.workspace.data_ptr()), nbytes,
                               ctypes.c_void_p(torch.cuda.current_stream().cuda_stream), ctypes.byref(mesh.handle)))
    mesh.n_vel, mesh.n_p, mesh.n_enriched = cfg.n_vel, cfg.n_p, 0
    u = torch.tensor(np.random.default_rng(6).uniform(-1, 1, cfg.n_vel), device="cuda")
    words = mesh.workspace[: nbytes // 8 * 8].view(torch.int64)
    poison = int(np.frombuffer(b"\xa5" * 8, dtype=np.int64)[0])
    before = int((words == poison).sum())
    mesh.projection_step(torch.full((cfg.ncell,), 0.1, dtype=torch.float64, device="cuda"), u, u, 0.4)
    written = before - int((words == poison).sum())
    # K^{-1}; one height: 2 ZN + n with ZN = 64 entries a step, steps of the largest class, 16-row tiles of all; the map
    n1 = cfg.k_u + 1
    sizes = [sum(int(np.prod([n1 // 2 if ((p >> d) & 1) ^ (c == d) else (n1 + 1) // 2 for d in range(3)]))
                 for c in range(3)) for p in range(8)]
    zn = 64 * ((max(sizes) + 3) // 4) * sum((s + 15) // 16 for s in sizes)
    n = 3 * n1 ** 3
    assert sum(sizes) == n
    assert 0 < written <= n1 * n1 + 2 * zn + n + (cfg.ny + 1) // 2
    mesh.close()
