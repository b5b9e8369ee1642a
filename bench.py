#!/usr/bin/env python3
"""Benchmark of the enriched DG hot path on one MI355X.

One step = one pass of the operator hot path over the 64x32x32 channel
(tanh grading 1.8, k=4 velocity with the 7-point rule and 7x8x7 points in
the two enriched wall layers, k=3 pressure), all in FP64:
  1. wall-shear update: psi and grad psi by the FP64 Spalding Newton solve,
  2. enriched velocity residual (LLF convective + SIP viscous),
  3. SIP Poisson operator.
value = (velocity DoFs + pressure DoFs) per step / seconds per step.

Inputs are resident in HBM before the timed region.  Per-operator times
come from HIP events recorded on the stream the library launches on.  The
CPU oracle is timed on a bounded sample of the same workload (rank 0).

Usage: python bench.py [--gpus 1] [--steps K] [--warmup W]
"""
from __future__ import annotations

import argparse
import ctypes
import hashlib
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "DG operator DoFs/s (FP64 vs FP32-mixed) at 1e-10 resid; p50/p99 solve latency"
HBM_PEAK_GBS = 8000.0          # MI355X HBM3E
FP64_VEC_TFLOPS = 78.6         # MI355X FP64 vector peak
FP32_VEC_TFLOPS = 157.3
# Memory of the velocity residual: read u, write r (FP64).
BYTES_PER_DOF_F64 = 16.0


def residual_cell_flop(n, q):
    """Floating-point operations that residual_kernel executes for a cell without
    enrichment (n nodes, q points a direction): the products of its sweeps, line
    by line, and the arithmetic at the points."""
    n2, h = n * n, 2 * ((q + 1) // 2)          # h: points of a line as its two half lines take them
    fma = 18 * n2 * n                          # normal derivatives of the six neighbours
    fma += 3 * n2 * q * n + 3 * q * n * q * n + 3 * q * q * h * n        # u at the points
    fma += 6 * (q * q * h * n + q * n * q * n + n2 * q * n) + 9 * n2 * n2  # six products back, derivative tests
    fma += 36 * n * q * n + 36 * q * h * n + 18 * q * h * n + 18 * n * q * n  # traces of both sides, fluxes back
    # viscous lines (traces, stiffness, lifts), weak derivative, cross terms, mass
    fma += 9 * n2 * (n2 + 7 * n) + 3 * n2 * (n2 + 2 * n) + 3 * n2 * (n2 + 6 * n) + 9 * n2 * n2
    return 2 * fma + 12 * q * q * h + 26 * 6 * q * h


def enriched_cell_flop(n, q, y):
    """The same for vel_kernel on an enriched cell (y wall-normal points): sweeps
    and collocation gradients with their transposes, eight trace fields a side."""
    n2 = n * n
    fma = 2 * 3 * (n2 * q * n + q * n * y * n + q * y * q * n)
    fma += 2 * 3 * (2 * q * y * q * q + q * q * y * y)
    fma += 2 * 18 * n2 * n + 3 * 6 * n2 * n    # layers of both sides, face tests onto the lines
    flop = 80 * q * y * q
    for q1, q2 in ((y, q), (q, q), (q, y)):
        fma += 28 * n * q1 * n + 32 * q1 * q2 * n + 16 * q1 * q2 * n + 14 * n2 * q1
        flop += 100 * 2 * q1 * q2
    return 2 * fma + flop


def velocity_flop(m):
    """Operations of one velocity residual on mesh m as its kernels execute them."""
    n = m.k_u + 1
    return ((m.ncell - m.n_enriched) * residual_cell_flop(n, m.nq_u) +
            m.n_enriched * enriched_cell_flop(n, m.nq_u, m.nq_wn))


def kernel_source_hash():
    h = hashlib.sha256()
    for name in ("kern_velocity.hip", "kern_residual.hip", "ip_line.h", "kern_common.h", "kern_poisson.hip"):
        with open(os.path.join(ROOT, "paper_1705_08813_amd", "csrc", name), "rb") as f:
            h.update(f.read())
    return h.hexdigest()[:16]


def load_traffic(n_launch_units):
    """HBM bytes per velocity-residual launch measured with rocprofv3 PMC
    counters (FETCH_SIZE + WRITE_SIZE, scaled by a plain copy of known size),
    or None if missing or taken on a different kernel source."""
    path = os.path.join(ROOT, "profiles", "traffic_velocity_large.json")
    if not os.path.exists(path):
        return None
    with open(path) as f:
        t = json.load(f)
    if t.get("kernel_src_sha") != kernel_source_hash():
        return None
    return t.get("bytes_per_launch")


def cpu_baseline(wl, inp, min_seconds=10.0, max_groups=64):
    """The oracle as it stands on the host cores, on groups of 4 z-slabs of
    the same mesh (8192 cells per group, both enriched layers included):
    velocity residual + Poisson apply, group after group (cycling through the
    mesh) until at least min_seconds of CPU work have been timed."""
    import numpy as np
    import oracle as O
    m = wl.mesh
    nslab = 4
    per_group = nslab * m.nx * m.ny
    O.lib()
    t_vel = t_poi = 0.0
    dofs = 0
    groups = 0
    ngroups_mesh = m.nz // nslab
    while groups < max_groups and (t_vel + t_poi) < min_seconds:
        g = groups % ngroups_mesh
        cells = np.arange(g * per_group, (g + 1) * per_group, dtype=np.int64)
        t0 = time.perf_counter()
        O.velocity_residual(m, inp["u"], inp["tau"], cells=cells)
        t1 = time.perf_counter()
        O.poisson_apply(m, inp["p"], cells=cells)
        t2 = time.perf_counter()
        t_vel += t1 - t0
        t_poi += t2 - t1
        n_enr_in = nslab * m.nx * 2
        dofs += cells.size * 3 * (m.k_u + 1) ** 3 + 3 * n_enr_in + cells.size * (m.k_p + 1) ** 3
        groups += 1
    return {"value": dofs / (t_vel + t_poi), "unit": "DoFs/s", "cores": O.num_threads(), "kind": "oracle",
            "sample": f"{groups} groups of {per_group} cells (4 z-slabs each, cycling through the {m.ncell}-cell "
                      f"mesh): velocity residual {t_vel:.2f} s + Poisson apply {t_poi:.2f} s, {dofs} DoFs"}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-extras", action="store_true")
    ap.add_argument("--solves", type=int, default=5, help="timed Poisson solves per precision (extras)")
    ap.add_argument("--serving-requests", type=int, default=512,
                    help="requests of the serving stream run after the step timing (0: skip)")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="also run a plain device copy of known size (for PMC byte calibration)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (asked for --gpus {args.gpus}); sharding the path over several "
              "GPUs is not built.", file=sys.stderr, flush=True)
        sys.exit(2)

    import numpy as np
    import torch
    from paper_1705_08813_amd import Mesh, _lib
    from paper_1705_08813_amd.inputs import PRESETS, draw_inputs

    dev = torch.device("cuda", 0)
    torch.cuda.set_device(dev)
    wl = PRESETS["large"]
    m = wl.mesh
    inp = draw_inputs(wl)
    mesh = Mesh(m, inp["tau"], device=dev)
    u = torch.tensor(inp["u"], device=dev)
    p = torch.tensor(inp["p"], device=dev)
    tau = torch.tensor(inp["tau"], device=dev)
    r = torch.empty_like(u)
    y = torch.empty_like(p)
    stream = torch.cuda.current_stream()
    n_vel, n_p = mesh.n_vel, mesh.n_p

    def step():
        mesh.update_wall_shear(tau)
        mesh.apply_velocity_residual(u, r)
        mesh.apply_poisson(p, y)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()

    K = args.steps
    ev = [[torch.cuda.Event(enable_timing=True) for _ in range(4)] for _ in range(K)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for k in range(K):
        e = ev[k]
        e[0].record(stream)
        mesh.update_wall_shear(tau)
        e[1].record(stream)
        mesh.apply_velocity_residual(u, r)
        e[2].record(stream)
        mesh.apply_poisson(p, y)
        e[3].record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    t_psi = sum(e[0].elapsed_time(e[1]) for e in ev) / K * 1e-3
    t_vel = sum(e[1].elapsed_time(e[2]) for e in ev) / K * 1e-3
    t_poi = sum(e[2].elapsed_time(e[3]) for e in ev) / K * 1e-3
    dofs_step = n_vel + n_p
    value = dofs_step * K / wall

    vel_flops = velocity_flop(m)
    ach_tflops = vel_flops / t_vel / 1e12
    traffic = load_traffic(n_vel)
    roofline = {"bound": "alu", "achieved": round(ach_tflops, 3), "peak": FP64_VEC_TFLOPS, "unit": "TFLOP/s",
                "frac": round(ach_tflops / FP64_VEC_TFLOPS, 4), "traffic": traffic,
                "kernel": "velocity residual (residual_kernel and enriched vel_kernel launches), FP64",
                "per_launch_ms": round(t_vel * 1e3, 4), "executed_flop_per_dof": round(vel_flops / n_vel, 1)}
    out = {"metric": METRIC, "value": value, "unit": "DoFs/s", "n_gpus": 1, "steps": K, "warmup": args.warmup,
           "ms_per_step": wall / K * 1e3, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
           "dtype": "f64", "data": "synthetic",
           "config": {"workload": "channel 64x32x32, tanh 1.8, k_u=4 (7^3 Gauss points, 7x8x7 in 4096 enriched "
                                  "wall cells), k_p=3 (4^3), FP64: psi refresh + velocity residual + SIP Poisson",
                      "velocity_dofs": n_vel, "pressure_dofs": n_p, "seed": wl.seed,
                      "solve": "extras: SIP Poisson k_p=3 to 1e-10 (true FP64 residual), FP64 flexible CG "
                               "preconditioned by one geometric-multigrid V-cycle with Jacobi-Chebyshev smoothing "
                               "(degree 5 fine, 3 coarse) run in FP32 for 'mixed' (no inner CG) or FP64"},
           "roofline": roofline}
    extras = {"psi_ms": t_psi * 1e3, "velocity_ms": t_vel * 1e3, "poisson_ms": t_poi * 1e3,
              "velocity_GBps_alg": BYTES_PER_DOF_F64 * n_vel / t_vel / 1e9,
              "poisson_GBps_alg": BYTES_PER_DOF_F64 * n_p / t_poi / 1e9,
              "velocity_hbm_frac_alg": BYTES_PER_DOF_F64 * n_vel / t_vel / 1e9 / HBM_PEAK_GBS,
              "poisson_hbm_frac_alg": BYTES_PER_DOF_F64 * n_p / t_poi / 1e9 / HBM_PEAK_GBS,
              "kernel_src_sha": kernel_source_hash()}

    print(f"bench: {K} steps in {wall:.3f} s", file=sys.stderr, flush=True)
    if not args.no_extras:
        # FP32 operator applications on the same data
        u32, p32 = u.float(), p.float()
        r32, y32 = torch.empty_like(u32), torch.empty_like(p32)
        for _ in range(3):
            mesh.apply_velocity_residual(u32, r32)
            mesh.apply_poisson(p32, y32)
        e0, e1, e2 = (torch.cuda.Event(enable_timing=True) for _ in range(3))
        n32 = max(5, K // 2)
        e0.record(stream)
        for _ in range(n32):
            mesh.apply_velocity_residual(u32, r32)
        e1.record(stream)
        for _ in range(n32):
            mesh.apply_poisson(p32, y32)
        e2.record(stream)
        torch.cuda.synchronize()
        tv32 = e0.elapsed_time(e1) / n32 * 1e-3
        tp32 = e1.elapsed_time(e2) / n32 * 1e-3
        extras.update({"velocity_f32_ms": tv32 * 1e3, "poisson_f32_ms": tp32 * 1e3,
                       "f32_step_dofs_per_s": dofs_step / (tv32 + tp32),
                       "velocity_f32_GBps_alg": 8.0 * n_vel / tv32 / 1e9,
                       "poisson_f32_GBps_alg": 8.0 * n_p / tp32 / 1e9})
    if not args.no_extras:
        print("bench: Poisson solves", file=sys.stderr, flush=True)
        # Poisson solve to 1e-10 (same mesh, k=3): mixed precision vs all-FP64
        bsol = torch.tensor(np.random.default_rng(PRESETS["precision"].seed).uniform(-1, 1, n_p), device=dev)
        xs_by_key = {}
        for mixed in (True, False):
            sp = mesh.solve_params(mixed=mixed)
            ws = mesh.solve_workspace(sp)
            mesh.solve_poisson(bsol, sp=sp, workspace=ws)  # warm-up (eigenvalue estimate is cached)
            times, st = [], None
            for _ in range(args.solves):
                x = torch.zeros_like(bsol)
                torch.cuda.synchronize()
                t_s = time.perf_counter()
                x, st = mesh.solve_poisson(bsol, x=x, sp=sp, workspace=ws)
                times.append(time.perf_counter() - t_s)
            times = np.sort(np.array(times))
            key = "solve_mixed" if mixed else "solve_f64"
            xs_by_key[key] = x.cpu().numpy()
            extras[key] = {"median_s": float(np.median(times)), "p50_s": float(np.percentile(times, 50)),
                           "p99_s": float(np.percentile(times, 99)), "outer_its": st.outer_its,
                           "f64_applies": st.op_applies_f64, "f32_applies": st.op_applies_f32,
                           "rel_resid": st.rel_resid, "solves": args.solves,
                           "dofs_per_s": n_p / float(np.median(times))}
        extras["solve_speedup_mixed_vs_f64"] = extras["solve_f64"]["median_s"] / extras["solve_mixed"]["median_s"]
        # Jacobi-preconditioned FP64 CG to 1e-10 (Chebyshev degree 1 is a multiple of Jacobi, so CG takes the
        # Jacobi-PCG iterations): its iteration count times the oracle's cost per iteration is the CPU
        # oracle's solve time
        spj = mesh.solve_params(mixed=False, multigrid=False, cheb_degree=1, max_outer=40000)
        _, stj = mesh.solve_poisson(bsol, sp=spj, workspace=mesh.solve_workspace(spj))
        extras["solve_jacobi_cg_f64"] = {"outer_its": stj.outer_its, "rel_resid": stj.rel_resid,
                                         "seconds": stj.seconds}
        if not args.no_cpu_baseline:
            import oracle as O
            print("bench: oracle residuals of the solutions", file=sys.stderr, flush=True)
            bnp = bsol.cpu().numpy()
            bp = bnp - bnp.mean()
            for key, xs in xs_by_key.items():
                res = bp - O.poisson_apply(m, xs)
                extras[key]["oracle_rel_resid"] = float(np.linalg.norm(res) / np.linalg.norm(bp))
            t_o = time.perf_counter()
            napp = 2
            for _ in range(napp):
                O.poisson_apply(m, bp)
            t_it = (time.perf_counter() - t_o) / napp
            extras["cpu_oracle_solve_f64"] = {
                "kind": "oracle", "cores": O.num_threads(), "method": "Jacobi-preconditioned FP64 CG to 1e-10",
                "iterations": stj.outer_its, "seconds_per_iteration": t_it,
                "estimated_seconds": stj.outer_its * t_it,
                "sample": f"{napp} oracle Poisson applies on the full {m.ncell}-cell mesh timed; the iteration count "
                          "is that of the same Jacobi-preconditioned CG run on the GPU (identical in exact "
                          "arithmetic), vector updates not counted"}
    if not args.no_extras:
        # van Driest enrichment (eq. psi, Appendix A evaluation) on the same mesh: psi refresh and
        # velocity residual (the residual kernel is the same; only the psi tables differ)
        print("bench: van Driest enrichment", file=sys.stderr, flush=True)
        vmesh = Mesh(m.with_(psi_kind=1), inp["tau"], device=dev)
        for _ in range(3):
            vmesh.update_wall_shear(tau)
            vmesh.apply_velocity_residual(u, r)
        e0, e1, e2 = (torch.cuda.Event(enable_timing=True) for _ in range(3))
        nrep = max(5, K // 2)
        e0.record(stream)
        for _ in range(nrep):
            vmesh.update_wall_shear(tau)
        e1.record(stream)
        for _ in range(nrep):
            vmesh.apply_velocity_residual(u, r)
        e2.record(stream)
        torch.cuda.synchronize()
        extras["vandriest"] = {"psi_refresh_ms": e0.elapsed_time(e1) / nrep,
                               "velocity_ms": e1.elapsed_time(e2) / nrep,
                               "psi_points": vmesh.n_enriched * (m.nq_u * m.nq_wn * m.nq_u + 2 * m.nq_u ** 2
                                                                 + 4 * m.nq_u * m.nq_wn)}
        del vmesh
    if not args.no_extras:
        # wall-shear pipeline (Sec. 3.2) on the same mesh and u: nodal tau_w from u, psi refresh
        # from the nodal field, then the residual with that psi
        print("bench: nodal wall shear pipeline", file=sys.stderr, flush=True)
        tn = mesh.wall_shear_nodes(u)
        for _ in range(3):
            mesh.wall_shear_nodes(u, tn)
            mesh.update_wall_shear_nodes(tn)
        ev3 = [torch.cuda.Event(enable_timing=True) for _ in range(3)]
        nrep = max(10, K)
        ev3[0].record(stream)
        for _ in range(nrep):
            mesh.wall_shear_nodes(u, tn)
        ev3[1].record(stream)
        for _ in range(nrep):
            mesh.update_wall_shear_nodes(tn)
        ev3[2].record(stream)
        torch.cuda.synchronize()
        nwall = 2 * m.nx * m.nz
        # algorithmic bytes: u of the wall cells, their enrichment dofs, dpsi/dy at the wall-face points, tau out
        ws_bytes = 8 * nwall * (3 * (m.k_u + 1) ** 3 + 3 + m.nq_u ** 2 + 1)
        t_ws = ev3[0].elapsed_time(ev3[1]) / nrep
        extras["wall_shear"] = {"wall_nodes": nwall, "wall_shear_nodes_ms": t_ws,
                                "alg_bytes": ws_bytes, "GBps_alg": ws_bytes / (t_ws * 1e-3) / 1e9,
                                "nodal_psi_refresh_ms": ev3[1].elapsed_time(ev3[2]) / nrep}
        mesh.update_wall_shear(tau)   # back to the per-point field of the timed steps
        del tn
    if not args.no_extras:
        # switch-off rule and cell-wise L2 projection onto the refreshed space (Sec. 3.2, eq. l2) on the
        # same mesh, with tau_w scaled by 1600 so that the wall cells reach y+ ~ 70-120 (the range where
        # the enrichment is on) and the paper's switch-off threshold y+ = 30
        import numpy as np
        print("bench: projection onto the refreshed space", file=sys.stderr, flush=True)
        pm = Mesh(m.with_(yplus_off=30.0), 1600.0 * inp["tau"], device=dev)
        tnd = torch.tensor(np.random.default_rng(7).uniform(800.0, 2400.0, (2, m.nz, m.nx)), device=dev)
        un = torch.empty_like(u)
        uw = u.clone()
        for _ in range(3):
            pm.update_wall_shear_nodes(tnd)
            pm.project_velocity(u, un)
            pm.project_velocity(uw, uw)
        ev4 = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
        nrep = max(10, K)
        ev4[0].record(stream)
        for _ in range(nrep):
            pm.update_wall_shear_nodes(tnd)
        ev4[1].record(stream)
        for _ in range(nrep):
            pm.project_velocity(u, un)
        ev4[2].record(stream)
        for _ in range(nrep):
            pm.project_velocity(uw, uw)
        ev4[3].record(stream)
        torch.cuda.synchronize()
        nq3 = m.nq_u * m.nq_wn * m.nq_u
        # in place: psi at the volume points of both tables in, the enriched cells' u in and out
        prj_bytes = 8 * pm.n_enriched * (2 * nq3 + 2 * (3 * (m.k_u + 1) ** 3 + 3))
        t_in = ev4[2].elapsed_time(ev4[3]) / nrep
        extras["projection"] = {"enriched_cells": pm.n_enriched, "active": int(pm.enrichment_active().sum().item()),
                                "refresh_with_switch_off_ms": ev4[0].elapsed_time(ev4[1]) / nrep,
                                "project_ms": ev4[1].elapsed_time(ev4[2]) / nrep, "project_in_place_ms": t_in,
                                "in_place_alg_bytes": prj_bytes, "in_place_GBps_alg": prj_bytes / (t_in * 1e-3) / 1e9}
        # inverse velocity mass matrix on the same (y+ ~ 100) space: 16 B per unknown (r in, x out)
        xm = torch.empty_like(u)
        for _ in range(3):
            pm.apply_inverse_mass(u, xm)
        ev5 = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        ev5[0].record(stream)
        for _ in range(nrep):
            pm.apply_inverse_mass(u, xm)
        ev5[1].record(stream)
        torch.cuda.synchronize()
        t_im = ev5[0].elapsed_time(ev5[1]) / nrep
        im_bytes = 16.0 * pm.n_vel
        extras["inverse_mass"] = {"unknowns": pm.n_vel, "ms": t_im, "alg_bytes": im_bytes,
                                  "GBps_alg": im_bytes / (t_im * 1e-3) / 1e9,
                                  "hbm_frac": im_bytes / (t_im * 1e-3) / 8e12}
        del pm, un, uw, tnd, xm
    if not args.no_extras:
        # pressure gradient and velocity divergence terms (Sec. 4.2) on the same mesh and data
        print("bench: pressure gradient and velocity divergence", file=sys.stderr, flush=True)
        gv = torch.empty_like(u)
        cp = torch.empty_like(p)
        for _ in range(3):
            mesh.apply_pressure_gradient(p, gv)
            mesh.apply_velocity_divergence(u, cp)
        ev6 = [torch.cuda.Event(enable_timing=True) for _ in range(3)]
        nrep = max(10, K)
        ev6[0].record(stream)
        for _ in range(nrep):
            mesh.apply_pressure_gradient(p, gv)
        ev6[1].record(stream)
        for _ in range(nrep):
            mesh.apply_velocity_divergence(u, cp)
        ev6[2].record(stream)
        torch.cuda.synchronize()
        t_g = ev6[0].elapsed_time(ev6[1]) / nrep
        t_c = ev6[1].elapsed_time(ev6[2]) / nrep
        # algorithmic bytes: one input and one output vector each
        b_gc = 8.0 * (n_vel + n_p)
        extras["pressure_gradient"] = {"ms": t_g, "GBps_alg": b_gc / (t_g * 1e-3) / 1e9}
        extras["velocity_divergence"] = {"ms": t_c, "GBps_alg": b_gc / (t_c * 1e-3) / 1e9}
        # div-div penalty: tau_D from the velocity, then D u (16 B per unknown plus tau_D)
        td = mesh.divdiv_tau(u, 0.05)
        for _ in range(3):
            mesh.divdiv_tau(u, 0.05, td)
            mesh.apply_divdiv(td, u, gv)
        ev7 = [torch.cuda.Event(enable_timing=True) for _ in range(3)]
        ev7[0].record(stream)
        for _ in range(nrep):
            mesh.divdiv_tau(u, 0.05, td)
        ev7[1].record(stream)
        for _ in range(nrep):
            mesh.apply_divdiv(td, u, gv)
        ev7[2].record(stream)
        torch.cuda.synchronize()
        t_dd = ev7[1].elapsed_time(ev7[2]) / nrep
        extras["divdiv"] = {"tau_ms": ev7[0].elapsed_time(ev7[1]) / nrep, "apply_ms": t_dd,
                            "apply_GBps_alg": 16.0 * n_vel / (t_dd * 1e-3) / 1e9}
        # element-wise projection step (M + D) x = M u_hat - dt P p, a direct solve per cell (per-layer
        # eigenbasis, bordered in enriched cells): u_hat, P p in, x out (24 B per unknown)
        mesh.apply_pressure_gradient(p, gv)
        xs = torch.empty_like(u)
        for _ in range(2):
            mesh.projection_step(td, u, gv, 1e-3, xs)
        ev8 = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        nps = max(3, nrep // 4)
        ev8[0].record(stream)
        for _ in range(nps):
            mesh.projection_step(td, u, gv, 1e-3, xs)
        ev8[1].record(stream)
        torch.cuda.synchronize()
        t_ps = ev8[0].elapsed_time(ev8[1]) / nps
        extras["projection_step"] = {"ms": t_ps, "GBps_alg": 24.0 * n_vel / (t_ps * 1e-3) / 1e9}
        del gv, cp, td, xs
    if not args.no_extras:
        # multiscale viscous operator (Sec. 4.2, eq. viscous_multiscale) with the eddy viscosity of Sec. 2.2,
        # on the same mesh with tau_w scaled by 1600 (wall cells at y+ ~ 70-120, nu_t up to tens of nu)
        print("bench: multiscale viscous operator", file=sys.stderr, flush=True)
        msm = Mesh(m, 1600.0 * inp["tau"], device=dev)
        nut = msm.eddy_viscosity(u)
        ov = torch.empty_like(u)
        for _ in range(3):
            msm.eddy_viscosity(u, nut=nut)
            msm.apply_viscous_multiscale(nut, u, ov)
        ev9 = [torch.cuda.Event(enable_timing=True) for _ in range(3)]
        nrep = max(10, K)
        ev9[0].record(stream)
        for _ in range(nrep):
            msm.eddy_viscosity(u, nut=nut)
        ev9[1].record(stream)
        for _ in range(nrep):
            msm.apply_viscous_multiscale(nut, u, ov)
        ev9[2].record(stream)
        torch.cuda.synchronize()
        t_ms = ev9[1].elapsed_time(ev9[2]) / nrep
        ms_bytes = 16.0 * n_vel + 8.0 * nut.numel()
        extras["viscous_multiscale"] = {"eddy_viscosity_ms": ev9[0].elapsed_time(ev9[1]) / nrep,
                                        "nu_t_points": int(nut.numel()), "apply_ms": t_ms,
                                        "apply_dofs_per_s": n_vel / (t_ms * 1e-3),
                                        "apply_GBps_alg": ms_bytes / (t_ms * 1e-3) / 1e9}
        # one dual-splitting time step (Sec. 4.1) on the same mesh: convective step, pressure with the
        # high-order Neumann data (mixed solve to 1e-10), projection, Helmholtz GMRES (1e-10); BDF2/EXT2,
        # dt = 1e-3 (Courant number about 0.14 on the thinnest wall cells at |u| ~ 1), unit body force
        print("bench: dual-splitting step", file=sys.stderr, flush=True)
        spst = msm.step_params(1e-3, order=2, f=(1.0, 0.0, 0.0), helmholtz_rtol=1e-10)
        sws = torch.empty(int(_lib.check(_lib.lib().dg_step_workspace_bytes(msm.handle, ctypes.byref(spst)))),
                          dtype=torch.uint8, device=dev)
        u_prev = torch.roll(u, 1)
        pst = torch.zeros(n_p, dtype=torch.float64, device=dev)
        un = torch.empty_like(u)
        msm.dual_splitting_step(spst, u, u_prev, pst, u_np1=un, workspace=sws)   # warm-up (eigenvalue estimates)
        step_t, step_st = [], None
        for _ in range(3):
            pst.zero_()
            torch.cuda.synchronize()
            t_s = time.perf_counter()
            _, _, step_st = msm.dual_splitting_step(spst, u, u_prev, pst, u_np1=un, workspace=sws)
            step_t.append(time.perf_counter() - t_s)
        extras["dual_splitting_step"] = {
            "median_s": float(np.median(step_t)), "poisson_its": step_st.poisson.outer_its,
            "poisson_rel_resid": step_st.poisson.rel_resid, "helmholtz_its": step_st.helmholtz.iterations,
            "helmholtz_s": step_st.helmholtz.seconds,
            "helmholtz_rel_resid": step_st.helmholtz.rel_resid, "dt": 1e-3, "order": 2,
            "velocity_dofs": n_vel, "pressure_dofs": n_p}
        del msm, nut, ov, sws, un, pst, u_prev
    if not args.no_extras:
        # the Helmholtz step with degree-1 enrichment weights (Sec. 3.1 eq. enrichment, l = 1) against l = 0
        # (Sec. 5.1 compares the two on a 16^3 channel at Re_tau 950 with grading 1.2): same mesh, same
        # functions (the eight l = 1 coefficients of a component all equal to its l = 0 coefficient, so u,
        # nu_t and the right-hand side are the same fields), gamma0/dt = 1.5e3, GMRES to 1e-10, restart 30
        print("bench: Helmholtz l = 1 against l = 0", file=sys.stderr, flush=True)
        from paper_1705_08813_amd import DgError
        from paper_1705_08813_amd.inputs import MeshConfig, Workload
        wh = Workload("l0l1", MeshConfig(nx=16, ny=16, nz=16, gamma=1.2, k_u=4, nq_u=7, nq_wn=8, k_p=3, nq_p=4,
                                         nu=1.0 / 950), 5, 0.5, 1.5)
        ih = draw_inputs(wh, want=("u", "tau"))
        npoly = wh.mesh.ncell * 3 * (wh.mesh.k_u + 1) ** 3
        hl = {}
        for deg in (0, 1):
            cfg_h = wh.mesh.with_(enrich_degree=deg)
            mh = Mesh(cfg_h, ih["tau"], device=dev)
            uh = torch.tensor(ih["u"], device=dev)
            bh = torch.roll(uh, 7)
            if deg == 1:
                uh = torch.cat([uh[:npoly], uh[npoly:].view(-1, 3, 1).expand(-1, 3, 8).reshape(-1)])
                bh = torch.cat([bh[:npoly], bh[npoly:].view(-1, 3, 1).expand(-1, 3, 8).reshape(-1)])
            nth = mh.eddy_viscosity(uh)
            torch.cuda.synchronize()
            t_h = time.perf_counter()
            try:
                _, sth = mh.solve_helmholtz(nth, 1.5e3, bh, rtol=1e-10, max_iter=4000, restart=30)
                its_h, res_h = sth.iterations, sth.rel_resid
            except DgError:
                its_h, res_h = None, None
            torch.cuda.synchronize()
            hl[f"l{deg}"] = {"gmres_its": its_h, "rel_resid": res_h, "seconds": time.perf_counter() - t_h,
                             "velocity_dofs": mh.n_vel}
            del mh, uh, bh, nth
        if hl["l0"]["gmres_its"] and hl["l1"]["gmres_its"]:
            hl["its_ratio_l1_over_l0"] = hl["l1"]["gmres_its"] / hl["l0"]["gmres_its"]
        hl["mesh"] = "16x16x16, tanh grading 1.2, k_u = 4, nu = 1/950, tau_w ~ U[0.5, 1.5], random u"
        extras["helmholtz_l1_vs_l0"] = hl
        # Poisson iterations on the two meshes of the paper's cost comparison (Sec. 5.1: about 9 iterations for
        # the wall-modeled 12x8x12 mesh with grading 1.6, 22 for the wall-resolved 24^3 mesh with grading 2.25,
        # k = 4, pressure k - 1): multigrid-preconditioned CG (FP64 and mixed) from zero, random right-hand side
        print("bench: Poisson iterations, wall-modeled against wall-resolved mesh", file=sys.stderr, flush=True)
        pit = {}
        for name, (nx_, ny_, nz_, gam) in (("wall_modeled_12x8x12_g1.6", (12, 8, 12, 1.6)),
                                            ("wall_resolved_24x24x24_g2.25", (24, 24, 24, 2.25))):
            cfg_p = MeshConfig(nx=nx_, ny=ny_, nz=nz_, gamma=gam, k_u=4, nq_u=7, nq_wn=8, k_p=3, nq_p=4,
                               nu=1.0 / 950, enrich_lower=1 if ny_ == 8 else 0, enrich_upper=1 if ny_ == 8 else 0,
                               omit_step_tables=1)
            mp_ = Mesh(cfg_p, np.ones(cfg_p.n_tau), device=dev)
            bp_ = torch.tensor(np.random.default_rng(6).uniform(-1, 1, cfg_p.n_p), device=dev)
            row = {}
            for rt_ in (1e-3, 1e-6, 1e-10):
                for mixed in (False, True):
                    spp = mp_.solve_params(rtol=rt_, mixed=mixed)
                    _, stp = mp_.solve_poisson(bp_, sp=spp, workspace=mp_.solve_workspace(spp))
                    row[f"{'mixed' if mixed else 'f64'}_rtol{rt_:g}"] = stp.outer_its
            pit[name] = row
            del mp_, bp_
        pit["paper_iterations"] = {"wall_modeled_12x8x12_g1.6": 9, "wall_resolved_24x24x24_g2.25": 22}
        extras["poisson_iterations_stretching"] = pit
    if not args.no_extras:
        print("bench: curved configuration", file=sys.stderr, flush=True)
        # curved configuration (48x24x24, cosine lower wall, k=5, per-point geometry tables)
        wc = PRESETS["curved"]
        ic = draw_inputs(wc, want=("u", "tau", "p"))
        cmesh = Mesh(wc.mesh, ic["tau"], device=dev)
        cu = torch.tensor(ic["u"], device=dev)
        cr = torch.empty_like(cu)
        cu32, cr32 = cu.float(), torch.empty(cu.numel(), dtype=torch.float32, device=dev)
        nrep = max(5, K // 5)
        times = {}
        for name, (a, b) in (("f64", (cu, cr)), ("f32", (cu32, cr32))):
            for _ in range(2):
                cmesh.apply_velocity_residual(a, b)
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record(stream)
            for _ in range(nrep):
                cmesh.apply_velocity_residual(a, b)
            e1.record(stream)
            torch.cuda.synchronize()
            times[name] = e0.elapsed_time(e1) / nrep * 1e-3
        cm = wc.mesh
        pts = cm.nq_u ** 3 + 6 * cm.nq_u * max(cm.nq_u, cm.nq_wn)   # volume + face points per cell
        geo_b = 10 * 8 * pts * cm.ncell                               # J^-1 and weight, FP64
        extras["curved"] = {"velocity_dofs": cmesh.n_vel, "velocity_f64_ms": times["f64"] * 1e3,
                            "velocity_f32_ms": times["f32"] * 1e3,
                            "f64_dofs_per_s": cmesh.n_vel / times["f64"], "f32_dofs_per_s": cmesh.n_vel / times["f32"],
                            "alg_bytes_per_dof_f64": (16.0 * cmesh.n_vel + geo_b) / cmesh.n_vel,
                            "f64_GBps_alg": (16.0 * cmesh.n_vel + geo_b) / times["f64"] / 1e9,
                            "f32_GBps_alg": (8.0 * cmesh.n_vel + geo_b) / times["f32"] / 1e9}
        # the pressure-projection terms on the curved cells: P, C, tau_D, the div-div penalty, M^-1
        cp = torch.tensor(ic["p"], device=dev)
        cpo = torch.empty(cmesh.n_p, dtype=torch.float64, device=dev)
        ctd = torch.empty(cmesh.n_cells, dtype=torch.float64, device=dev)
        ops = {"pressure_gradient": lambda: cmesh.apply_pressure_gradient(cp, cr),
               "velocity_divergence": lambda: cmesh.apply_velocity_divergence(cu, cpo),
               "divdiv_tau": lambda: cmesh.divdiv_tau(cu, 0.05, ctd),
               "divdiv": lambda: cmesh.apply_divdiv(ctd, cu, cr),
               "inverse_mass": lambda: cmesh.apply_inverse_mass(cu, cr)}
        op_ms = {}
        for name, f in ops.items():
            f()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record(stream)
            for _ in range(3):
                f()
            e1.record(stream)
            torch.cuda.synchronize()
            op_ms[name] = e0.elapsed_time(e1) / 3
        extras["curved"]["projection_terms_ms"] = op_ms
        del cmesh, cu, cr, cu32, cr32, cp, cpo, ctd
    if not args.no_extras and args.serving_requests > 0:
        # serving: seeded Poisson-arrival stream of channel instances (grid, k, nu mixed), each 10
        # velocity-residual applies + one mixed-precision solve to 1e-10; batched velocity rounds
        from paper_1705_08813_amd.inputs import ServingConfig, serving_requests
        from paper_1705_08813_amd.serving import Server
        del mesh
        torch.cuda.empty_cache()
        scfg = ServingConfig(n_requests=args.serving_requests)
        reqs = serving_requests(scfg)
        print(f"bench: serving {len(reqs)} requests", file=sys.stderr, flush=True)
        first_of_k = {}
        for q in reqs:
            first_of_k.setdefault(q.workload.mesh.k_u, q)
        # load every kernel once before the timed stream
        Server(applies=scfg.applies, device=dev).run(list(first_of_k.values()), time_scale=0.0)
        rep = Server(applies=scfg.applies, device=dev).run(reqs)
        srv = rep.summary()
        srv.update({"stream": f"{scfg.n_requests} requests, exponential gaps mean {scfg.mean_interarrival * 1e3:g} ms, "
                              f"grids {list(scfg.grids)}, k {list(scfg.degrees)}, k_p = k-1, "
                              f"{scfg.applies} velocity applies + 1 mixed solve (1e-10) each",
                    "budget_bytes": 32 << 30, "slots": 64, "solves": "batched per velocity round"})
        # the same stream with one solve call per request, and both with every
        # request arriving at once (throughput under a full queue)
        keys = ("makespan_s", "dofs_per_s", "latency_p50_ms", "latency_p99_ms", "latency_max_ms")
        one = Server(applies=scfg.applies, device=dev, batch_solves=False).run(reqs).summary()
        srv["unbatched_solves"] = {k: one[k] for k in keys}
        for bs in (True, False):
            burst = Server(applies=scfg.applies, device=dev, batch_solves=bs).run(reqs, time_scale=0.0).summary()
            srv["burst_" + ("batched" if bs else "unbatched")] = {k: burst[k] for k in keys}
        extras["serving"] = srv
        print(f"bench: serving done in {rep.makespan:.2f} s", file=sys.stderr, flush=True)
    if args.copy_calibration:
        a = torch.empty(1 << 28, dtype=torch.uint8, device=dev)  # 256 MiB
        b = torch.empty_like(a)
        for _ in range(3):
            b.copy_(a)
        torch.cuda.synchronize()
        extras["copy_calibration_bytes"] = a.numel()
    out["extras"] = extras
    if not args.no_cpu_baseline:
        print("bench: CPU oracle baseline", file=sys.stderr, flush=True)
        out["cpu_baseline"] = cpu_baseline(wl, inp)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
