"""Coarse end of the multigrid V-cycle as one workgroup's work: meshes whose
whole hierarchy fits (from the finest level on), hierarchies that enter it
further down, thin meshes that coarsen along some directions only, periodic
ones, a coarsest level that is smoothed or solved from memory, for every
pressure degree and both precisions of the cycle.

The solution has to satisfy the oracle's operator (1.05e-10 of ||b'||, as in
test_gpu_solve.py), and the cycle has to be the one of the separate kernels:
the iteration counts are theirs, to two steps (a rounding difference in the
preconditioner can move the last step of a long solve, a wrong transfer or
smoothing step costs many)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1705_08813_amd import Mesh
from paper_1705_08813_amd.inputs import MeshConfig

pytestmark = pytest.mark.gpu

# nx, ny, nz, k_p, periodic, iterations
CASES = [(16, 8, 8, 3, 0, 10), (4, 2, 2, 3, 0, 8), (8, 8, 8, 2, 0, 16), (4, 4, 4, 2, 0, 13), (3, 6, 2, 2, 0, 20),
         (8, 16, 2, 1, 0, 69), (16, 16, 16, 1, 0, 21), (4, 8, 4, 4, 0, 32), (2, 6, 4, 5, 0, 45), (4, 4, 4, 3, 1, 13),
         (6, 12, 3, 3, 0, 35), (12, 5, 4, 3, 0, 14), (32, 2, 1, 3, 0, 10)]


@pytest.mark.parametrize("mixed", [True, False])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[:3])) + f"k{c[3]}p{c[4]}")
def test_coarse_cycle(case, mixed):
    nx, ny, nz, kp, per, its = case
    ku = max(2, min(5, kp + 1))
    cfg = MeshConfig(nx=nx, ny=ny, nz=nz, gamma=0.0 if per else 1.3, k_u=ku, k_p=kp,
                     nq_u={2: 4, 3: 5, 4: 7, 5: 8}[ku], nq_p=kp + 1, nq_wn=8, nu=1.0 / 700, fully_periodic=per,
                     enrich_lower=1 - per, enrich_upper=1 - per)
    print(f"[gpu] {nx}x{ny}x{nz} k_p={kp} periodic={per} mixed={mixed}", flush=True)
    b = np.random.default_rng(5).uniform(-1, 1, cfg.n_p)
    b -= b.mean()
    mesh = Mesh(cfg)
    x, st = mesh.solve_poisson(torch.tensor(b, device="cuda"), sp=mesh.solve_params(rtol=1e-10, mixed=mixed))
    res = np.linalg.norm(b - O.poisson_apply(cfg, x.cpu().numpy())) / np.linalg.norm(b)
    print(f"[gpu]   its={st.outer_its} res={res:.2e}", flush=True)
    assert res <= 1.05e-10
    assert st.outer_its <= its + 2
