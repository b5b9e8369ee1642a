"""FP32 velocity residual of curved cells, alone and in a batch, at the edges of
the face phases and for every rule whose tables a curved FP32 cell reads (with a
wall-normal rule of its own and without), element by element against the
oracle's absolute-value bound 4 m u32 R_abs of test_gpu_parity.py."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1705_08813_amd import Mesh, apply_velocity_residual_batched
from paper_1705_08813_amd.inputs import MeshConfig, Workload, draw_inputs

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24


@pytest.mark.parametrize("nx,ny,nz,k,nq,nqw,lower,upper", [
    (3, 2, 2, 2, 4, 8, 1, 0), (2, 3, 2, 2, 4, 4, 1, 1), (3, 4, 2, 3, 4, 8, 1, 1), (2, 3, 1, 3, 5, 5, 0, 1),
    (1, 3, 2, 3, 5, 8, 1, 1), (2, 3, 2, 4, 7, 8, 1, 0), (1, 2, 1, 4, 7, 8, 1, 1), (2, 3, 1, 5, 8, 8, 1, 1),
    (2, 2, 2, 5, 8, 8, 0, 0)])
def test_curved_residual_f32(nx, ny, nz, k, nq, nqw, lower, upper):
    cfg = MeshConfig(nx=nx, ny=ny, nz=nz, wall_amp=0.25, gamma=1.1, k_u=k, k_p=k - 1, nq_u=nq, nq_p=k, nq_wn=nqw,
                     nu=1.0 / 500, enrich_lower=lower, enrich_upper=upper, theta=0.6)
    print(f"[gpu] curved residual f32 {nx}x{ny}x{nz} k={k} rule {nq}/{nqw} enriched {lower}{upper}", flush=True)
    inp = draw_inputs(Workload("cf", cfg, 43, 0.5, 1.5))
    u32 = inp["u"].astype(np.float32)
    u_r = u32.astype(np.float64)
    bound = 4 * (3 * (nq + k + 1) + 40) * U32 * O.velocity_residual(cfg, u_r, inp["tau"], absmode=True) + 1e-30
    ref = O.velocity_residual(cfg, u_r, inp["tau"])
    mesh = Mesh(cfg, inp["tau"])
    u = torch.tensor(u32, device="cuda")
    rs = [mesh.apply_velocity_residual(u)] + list(apply_velocity_residual_batched([mesh, mesh], [u, u]))
    for r in rs:
        worst = float((np.abs(r.cpu().numpy().astype(np.float64) - ref) / bound).max())
        print(f"[gpu]   max err/bound {worst:.3f}", flush=True)
        assert worst <= 1.0
