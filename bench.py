"""Benchmark: time to a true relative residual of 1e-6 per right-hand side on
one MI355X, plus the fine-level stencil-apply bandwidth against the HBM peak.

Workload (one "step" = one full solve, all steps of the hot path):
  320^3 physical intervals + 16 PML cells per face (352^3 total, 44.0M nodes),
  h = 10 m, velocity 2000 m/s x (1 + 0.25 g), g a seeded Gaussian random field
  (correlation length 20 cells, max|g| = 1), clipped to [1500, 3000] m/s,
  omega for 6 points per wavelength at the minimum velocity, one point source
  h^-3 at a seeded node at least 6 cells inside the physical box, FP32 complex,
  outer tolerance 1e-6 (true residual recomputed in FP64), fixed solver
  configuration of the paper's performance table.

Prints one JSON line.  `python bench.py --gpus 1 --steps K --warmup W`.
"""
import argparse
import hashlib
import json
import math
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
N_PHYS, N_PML, H, TOL, SEED = 320, 16, 10.0, 1e-6, 2
COUNTER_FILE = os.path.join(ROOT, "profiles", "stencil_apply_352_fp32_counters.txt")
# the stencil kernels (template code), their tiling and the file that instantiates the FP32 ones
STENCIL_SRCS = [os.path.join(ROOT, "paper_2608_22946_amd", "csrc", f)
                for f in ("stencil_impl.h", "tiles.h", "stencil.hip")]


def workload():
    from workloads import grf_velocity, point_source
    from workloads.configs import omega_for_ppw
    vel = grf_velocity(N_PHYS, N_PHYS, N_PHYS, seed=SEED)
    omega = omega_for_ppw(float(vel.min()), H)
    N = N_PHYS + 2 * N_PML
    rng = np.random.default_rng(SEED)
    src = tuple(int(v) for v in rng.integers(N_PML + 6, N_PML + N_PHYS - 6, 3))
    f = point_source((N, N, N), src, H, dtype=np.complex64)
    return vel, omega, f, src


PRECISION_NOTE = {
    "fp64": "fp64 throughout",
    "fp32": "fp32 (outer x, b and true residual in fp64)",
    "mixed": "fp32 arithmetic; the 2h-4h cycle's vectors and K_2h's preconditioned vectors stored in fp16 "
             "(scaled); outer x, b and true residual in fp64",
}


def stencil_hash():
    h = hashlib.sha256()
    for p in STENCIL_SRCS:
        with open(p, "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def recorded_traffic(nodes):
    """HBM bytes per apply from the committed counter summary, if it was taken
    on the current stencil source; else None."""
    if not os.path.exists(COUNTER_FILE):
        return None
    vals = {}
    for line in open(COUNTER_FILE):
        if "=" in line and not line.lstrip().startswith("#"):
            k, v = line.split("=", 1)
            vals[k.strip()] = v.strip()
    if vals.get("stencil_sha") != stencil_hash():
        return None
    try:
        return float(vals["traffic_bytes_per_apply"])
    except (KeyError, ValueError):
        return None


# ---- the cpu_baseline leg: the only code in this file that runs the FP64 oracle (a checker and a
# ---- baseline, never part of the solve); skipped with --no-cpu-baseline

def cpu_model():
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def _omp_threads(n):
    """Set the OpenMP thread count of this process's later parallel regions (the oracle's)."""
    import ctypes
    try:
        ctypes.CDLL("libgomp.so.1").omp_set_num_threads(int(n))
        return True
    except OSError:
        return False


def crop_parity(vel, omega, table, src, precision, crop=64):
    """The benchmark's physics on a crop^3 box around its source (+ N_PML PML cells):
    the GPU solve (this precision, tol 1e-6) against the FP64 oracle solved to 1e-10,
    relative l2 over every node."""
    import torch
    from oracle.oracle import Hierarchy as OracleHierarchy
    from paper_2608_22946_amd import helm
    from workloads import point_source
    sp = np.array(src) - N_PML
    lo = np.clip(sp - crop // 2, 0, N_PHYS - crop)
    vc = np.ascontiguousarray(vel[lo[2]:lo[2] + crop + 1, lo[1]:lo[1] + crop + 1, lo[0]:lo[0] + crop + 1])
    Nc = crop + 2 * N_PML
    s_loc = tuple(int(v) for v in sp - lo + N_PML)
    fc = point_source((Nc, Nc, Nc), s_loc, H)
    # the crop has its own minimum velocity; the frequency stays the benchmark's
    Hc = helm.Hierarchy(torch.from_numpy(vc), H, omega, N_PML, precision=precision, table=table, device="cuda:0")
    cdt = np.complex128 if precision == "fp64" else np.complex64
    uc, its, rel, rc = Hc.solve(torch.from_numpy(fc.astype(cdt)).cuda(), TOL)
    ug = uc.cpu().numpy().astype(np.complex128)
    Hc.close()
    O = OracleHierarchy(vc, H, omega, N_PML, table)
    t0 = time.perf_counter()
    uo, its_o, rel_o, st = O.solve(fc, 1e-10)
    t_o = time.perf_counter() - t0
    O.close()
    return {"crop": f"{crop}^3 + {N_PML} PML around the benchmark source, the benchmark's omega",
            "rel_l2_error": float(np.linalg.norm(ug - uo) / np.linalg.norm(uo)), "gpu_pc_calls": int(its),
            "oracle_tol": 1e-10, "oracle_pc_calls": int(its_o), "oracle_s": round(t_o, 1)}


def cpu_baseline(vel, omega, table, gpu_pc_calls):
    """The FP64 oracle on the host cores: one preconditioner
    application (Algorithm 1) on the full workload, scaled to seconds per
    right-hand side by the GPU run's preconditioner-call count; beside it one
    FP64 A_h apply at the full size on all threads and on one thread."""
    from oracle.oracle import Hierarchy as OracleHierarchy
    from workloads import random_complex
    t0 = time.perf_counter()
    O = OracleHierarchy(vel, H, omega, N_PML, table)
    t_setup = time.perf_counter() - t0
    N = N_PHYS + 2 * N_PML
    r = random_complex((N, N, N), 7)
    r /= np.linalg.norm(r)
    t0 = time.perf_counter()
    O.precond(r)
    t_pc = time.perf_counter() - t0
    cores = int(os.environ.get("OMP_NUM_THREADS", os.cpu_count() or 1))
    t0 = time.perf_counter()
    O.apply(0, 0, r)
    t_ap = time.perf_counter() - t0
    single = None
    if _omp_threads(1):
        t0 = time.perf_counter()
        O.apply(0, 0, r)
        single = time.perf_counter() - t0
        _omp_threads(cores)
    O.close()
    return {"value": t_pc * gpu_pc_calls, "unit": "s per RHS (extrapolated)", "cores": cores, "kind": "oracle",
            "sample": f"one FP64 preconditioner application (Algorithm 1) on the full 352^3 workload took "
                      f"{t_pc:.2f} s; scaled by the GPU solve's {gpu_pc_calls} preconditioner calls",
            "cpu_model": cpu_model(), "setup_s": round(t_setup, 2),
            "apply_s": {"sample": "one FP64 A_h apply on the full 352^3 grid", "threads": cores,
                        "s": round(t_ap, 3), "single_thread_s": None if single is None else round(single, 3)}}


def c4_crop_parity(vel, omega, table, src, npml, precision, crop, crop_tol):
    """The 800^3 workload's physics on a crop^3 + npml box around its source: the GPU
    solve (this precision, tol 1e-6) against the FP64 oracle solved to crop_tol."""
    import torch
    from oracle.oracle import Hierarchy as OracleHierarchy
    from paper_2608_22946_amd import helm
    from workloads import point_source
    n = vel.shape[0] - 1
    dev = torch.device("cuda", 0)
    sp = np.array(src) - npml
    lo = np.clip(sp - crop // 2, 0, n - crop)
    vc = np.ascontiguousarray(vel[lo[2]:lo[2] + crop + 1, lo[1]:lo[1] + crop + 1, lo[0]:lo[0] + crop + 1])
    Nc = crop + 2 * npml
    s_loc = tuple(int(v) for v in sp - lo + npml)
    fc = point_source((Nc, Nc, Nc), s_loc, H)
    Hc = helm.Hierarchy(torch.from_numpy(vc), H, omega, npml, precision=precision, table=table, device=dev)
    uc, its_c, rel_c, rc_c = Hc.solve(torch.from_numpy(fc.astype(np.complex128 if precision == "fp64"
                                                                     else np.complex64)).to(dev), TOL)
    ug = uc.cpu().numpy().astype(np.complex128)
    Hc.close()
    t0 = time.perf_counter()
    O = OracleHierarchy(vc, H, omega, npml, table)
    uo, its_o, rel_o, st_o = O.solve(fc, crop_tol)
    t_or = time.perf_counter() - t0
    O.close()
    err = float(np.linalg.norm(ug - uo) / np.linalg.norm(uo))
    return {"c4": "crop", "crop": f"{crop}^3 + {npml} PML around the source", "precision": precision,
            "gpu_pc_calls": int(its_c), "gpu_relres": float(rel_c), "oracle_pc_calls": its_o,
            "oracle_relres": rel_o, "oracle_s": round(t_or, 1), "rel_l2_error_vs_oracle": err}


def c3_crop_parity(vel, omega, table, srcs, npml, crop=64):
    """The 64-source workload's physics on a crop^3 + npml box holding four of its
    sources: one batched GPU solve of the four (helm_options.batch = 4, tol 1e-6)
    against four FP64 oracle solves to 1e-10, relative l2 per source."""
    import torch
    from oracle.oracle import Hierarchy as OracleHierarchy
    from paper_2608_22946_amd import helm
    from workloads import point_source
    n = vel.shape[0] - 1
    ps = np.array(srcs) - npml                      # physical (x, y, z) of every source
    lo = np.array([int(ps[:, 0].min()), int(ps[:, 1].min()), 0])
    lo = np.clip(lo - 8, 0, n - crop)
    inside = [q for q in ps if np.all(q - lo >= 8) and np.all(q - lo <= crop - 8)][:4]
    vc = np.ascontiguousarray(vel[lo[2]:lo[2] + crop + 1, lo[1]:lo[1] + crop + 1, lo[0]:lo[0] + crop + 1])
    Nc = crop + 2 * npml
    fs = np.stack([point_source((Nc,) * 3, tuple(int(v) for v in q - lo + npml), H) for q in inside])
    Hc = helm.Hierarchy(torch.from_numpy(vc), H, omega, npml, precision="fp32", table=table, device="cuda:0",
                        batch=len(inside))
    u, its, rel, rc = Hc.solve(torch.from_numpy(fs.astype(np.complex64)).cuda(), TOL)
    ug = u.cpu().numpy().astype(np.complex128)
    Hc.close()
    O = OracleHierarchy(vc, H, omega, npml, table)
    errs, t0 = [], time.perf_counter()
    for k in range(len(inside)):
        uo, its_o, rel_o, st = O.solve(fs[k], 1e-10)
        errs.append(float(np.linalg.norm(ug[k] - uo) / np.linalg.norm(uo)))
        print(json.dumps({"multi_rhs": "oracle crop source", "k": k, "rel_l2_error": errs[-1],
                          "oracle_s": round(time.perf_counter() - t0, 1)}), flush=True)
    t_o = time.perf_counter() - t0
    O.close()
    return {"crop": f"{crop}^3 + {npml} PML holding {len(inside)} of the sources, one GPU batch",
            "rel_l2_error_per_source": errs, "gpu_pc_calls": [int(v) for v in its], "oracle_tol": 1e-10,
            "oracle_s": round(t_o, 1)}


# ---- end of the cpu_baseline leg


def green_err(u, N, npml, h, k, src):
    """Sum of the relative l1 errors of the distance-scaled real and imaginary parts
    against the outgoing Green function exp(ikr)/(4 pi r) (Sec. 5.1), on the nodes of
    the physical box whose indices are multiples of 4 and with r >= 2 pi / k."""
    idx = np.arange(0, N + 1, 4)
    phys = idx[(idx >= npml) & (idx <= N - npml)]
    sx, sy, sz = src
    out = [0.0, 0.0, 0.0, 0.0]
    for iz in phys:   # one plane at a time keeps the host memory small
        y, x = np.meshgrid(phys, phys, indexing="ij")
        r = h * np.sqrt((x - sx) ** 2 + (y - sy) ** 2 + float(iz - sz) ** 2)
        m = r >= 2 * np.pi / k
        if not m.any():
            continue
        rr = r[m]
        uh = u[iz][np.ix_(phys, phys)][m].astype(np.complex128)
        G = np.exp(1j * k * rr) / (4 * np.pi * rr)
        out[0] += np.abs(rr * (G.real - uh.real)).sum()
        out[1] += np.abs(rr * G.real).sum()
        out[2] += np.abs(rr * (G.imag - uh.imag)).sum()
        out[3] += np.abs(rr * G.imag).sum()
    return out[0] / out[1] + out[2] / out[3]


def paper_table():
    """The paper's single-GPU results on its own meshes (512^3 total intervals,
    8 PML cells, 6 points per shortest wavelength, FP32, source at the centre
    node): the homogeneous Green-function test over the outer tolerances of its
    tolerance table, and the lens / wedge / barrier media at tol 1e-4.  One JSON
    line per case, with the paper's A100 numbers beside ours."""
    import torch
    from paper_2608_22946_amd import helm
    from workloads import barrier_velocity, homogeneous, lens_velocity, load_iofd_table, point_source, wedge_velocity
    from workloads.configs import omega_for_ppw

    Ntot, npml = 512, 8
    n = Ntot - 2 * npml
    h = 1.0 / n                      # physical box [0, 1]^3, normalised media coordinates
    src = (Ntot // 2,) * 3
    dev = torch.device("cuda", 0)
    table = load_iofd_table()
    f = torch.from_numpy(point_source((Ntot,) * 3, src, h, dtype=np.complex64)).to(dev)
    paper = {"green": {1e-2: (10, 3.057, 3.3231e-2), 1e-3: (12, 3.606, 1.6226e-2), 1e-4: (19, 5.512, 2.4936e-3),
                       1e-5: (25, 7.239, 2.7382e-3)},
             "lens": (12, 4.545), "wedge": (29, 10.863), "barrier": (32, 11.970)}
    cases = [("green", homogeneous(n, n, n, 1.0), (1e-2, 1e-3, 1e-4, 1e-5, 1e-6)),
             ("lens", lens_velocity(n, n, n), (1e-4,)), ("wedge", wedge_velocity(n, n, n), (1e-4,)),
             ("barrier", barrier_velocity(n, n, n), (1e-4,))]
    for name, vel, tols in cases:
        omega = omega_for_ppw(float(vel.min()), h)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        Hh = helm.Hierarchy(torch.from_numpy(vel), h, omega, npml, precision="fp32", table=table, device=dev)
        torch.cuda.synchronize()
        t_setup = time.perf_counter() - t0
        u = torch.empty_like(f)
        for tol in tols:
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            _, its, rel, rc = Hh.solve(f, tol, out=u.unsqueeze(0))
            torch.cuda.synchronize()
            t_solve = time.perf_counter() - t0
            line = {"case": name, "mesh": f"{Ntot}^3", "n_pml": npml, "tol": tol, "pc_calls": int(its),
                    "relres": float(rel), "converged": rc == 0, "t_setup_s": round(t_setup, 3),
                    "t_solve_s": round(t_solve, 3), "solve_per_pc_s": round(t_solve / max(int(its), 1), 4),
                    "precision": "fp32"}
            if name == "green":
                line["err"] = float(green_err(u.cpu().numpy(), Ntot, npml, h, omega, src))
                if tol in paper["green"]:
                    pc, ts, err = paper["green"][tol]
                    line["paper_a100"] = {"pc_calls": pc, "t_solve_s": ts, "err": err}
            else:
                pc, ts = paper[name]
                line["paper_a100"] = {"pc_calls": pc, "t_solve_s": ts}
            print(json.dumps(line), flush=True)
        Hh.close()
        del Hh


def green_pml(cases=((0, 1.119058), (1, 1.119058), (2, 1.119058), (0, 1.5), (0, 2.0), (0, 3.0))):
    """The 512^3 Green-function case of the paper's table (8 PML cells, c = 1, 6 points per
    wavelength, FP32, tol 1e-4) under the alternative readings of the PML profile
    (helm_options.pml_variant) and for several gamma_max: one JSON line each with Err."""
    import torch
    from paper_2608_22946_amd import helm
    from workloads import homogeneous, load_iofd_table, point_source
    from workloads.configs import omega_for_ppw

    Ntot, npml = 512, 8
    n = Ntot - 2 * npml
    h = 1.0 / n
    src = (Ntot // 2,) * 3
    dev = torch.device("cuda", 0)
    table = load_iofd_table()
    f = torch.from_numpy(point_source((Ntot,) * 3, src, h, dtype=np.complex64)).to(dev)
    vel = homogeneous(n, n, n, 1.0)
    omega = omega_for_ppw(1.0, h)
    for variant, gmax in cases:
        Hh = helm.Hierarchy(torch.from_numpy(vel), h, omega, npml, precision="fp32", table=table, device=dev,
                            pml_variant=variant, gamma_max=gmax)
        u, its, rel, rc = Hh.solve(f, 1e-4)
        err = float(green_err(u.cpu().numpy(), Ntot, npml, h, omega, src))
        Hh.close()
        del Hh, u
        print(json.dumps({"case": "green-pml", "mesh": f"{Ntot}^3", "n_pml": npml, "tol": 1e-4,
                          "pml_variant": variant, "gamma_max": gmax, "pc_calls": int(its), "err": err,
                          "paper_a100_err": 2.4936e-3}), flush=True)


def multi_rhs(configs=((1, 1), (4, 1), (1, 4), (1, 8), (2, 4), (2, 8)), seed=3, with_cpu=False):
    """Many right-hand sides on one hierarchy: 256^3 + 16-cell PML (288^3 total), a seeded
    8-layer model (1500..4000 m/s, sharp interfaces), 64 point sources on an 8 x 8 grid in
    the plane 20 cells below the top of the physical box, FP32, tol 1e-6 per source.
    One JSON line per (lanes, batch): lanes solve groups concurrently on their own streams
    (helm_options.lanes), a batch advances that many sources through one set of launches
    (helm_options.batch); (1, 1) is the plain single right-hand-side solver."""
    import torch
    from paper_2608_22946_amd import helm
    from workloads import layered_velocity, load_iofd_table, point_source
    from workloads.configs import omega_for_ppw

    n, npml = 256, 16
    N = n + 2 * npml
    vel = layered_velocity(n, n, n, seed=seed)
    omega = omega_for_ppw(float(vel.min()), H)
    dev = torch.device("cuda", 0)
    table = load_iofd_table()
    xs = [npml + int(round((i + 0.5) * n / 8)) for i in range(8)]
    srcs = [(x, y, npml + 20) for y in xs for x in xs]
    f = torch.from_numpy(np.stack([point_source((N, N, N), s_, H, dtype=np.complex64) for s_ in srcs])).to(dev)
    base = None
    for cfg in configs:
        lanes, batch = cfg[0], cfg[1]
        prec = cfg[2] if len(cfg) > 2 else "fp32"
        Hh = helm.Hierarchy(torch.from_numpy(vel), H, omega, npml, precision=prec, table=table, device=dev,
                            lanes=lanes, batch=batch)
        u = torch.empty_like(f)
        w = lanes * batch
        Hh.solve(f[:w], TOL, out=u[:w])          # warm-up, one group per lane
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        _, its, rel, rc = Hh.solve(f, TOL, out=u)
        torch.cuda.synchronize()
        dt = time.perf_counter() - t0
        per = dt / len(srcs)
        if base is None:
            base = per
        print(json.dumps({"metric": "time-to-rel.res 1e-6 per source, many sources", "value": round(per, 4),
                          "unit": "s per source", "lanes": lanes, "batch": batch, "precision": prec,
                          "speedup_vs_single_rhs": round(base / per, 3), "sources": len(srcs),
                          "total_s": round(dt, 3), "pc_calls_mean": float(np.mean(its)),
                          "pc_calls_max": int(np.max(its)), "max_relres": float(np.max(rel)),
                          "all_converged": rc == 0, "dtype": "f32",
                          "config": {"workload": "layered-288-fp32: 256^3 + 16-cell PML, 8 seeded layers 1500..4000 "
                                                 "m/s, 64 point sources on an 8x8 grid 20 cells deep, tol 1e-6",
                                     "seed": seed}}), flush=True)
        Hh.close()
        del Hh, u
        torch.cuda.empty_cache()
    if with_cpu:
        print(json.dumps({"multi_rhs": "oracle crop", **c3_crop_parity(vel, omega, table, srcs, npml)}), flush=True)


def c4_source(vel, npml, seed=4):
    """Seeded source node (total-grid x, y, z) outside the inclusion (velocity below
    3000 m/s) and at least 6 cells inside the physical box."""
    rng = np.random.default_rng(seed)
    n = vel.shape[0] - 1
    while True:
        p = rng.integers(6, n - 6, 3)
        if vel[p[2], p[1], p[0]] < 3000.0:
            return tuple(int(v) + npml for v in p)


def c4_bench(precision, apply_reps, crop, crop_tol, with_cpu):
    """Largest single-GPU workload: 768^3 + 16 PML cells (800^3 total, 5.1e8 nodes),
    1500 m/s background with a seeded ellipsoidal 4500 m/s inclusion (semi-axes
    150/120/90 cells) times (1 + 0.1 g), g a GRF of correlation length 20 cells, 6
    points per wavelength at the minimum velocity, one seeded source outside the
    inclusion, tol 1e-6.  One warm-up and one timed solve; the fine A_h apply timed
    at this shape; then, as the cpu_baseline leg (crop > 0, with_cpu), the same physics
    on a crop^3 + 16 PML box around the source, solved on the GPU to 1e-6 and by the
    FP64 oracle to crop_tol, compared node by node."""
    import torch
    from paper_2608_22946_amd import helm
    from workloads import ellipsoid_grf_velocity, load_iofd_table, point_source
    from workloads.configs import omega_for_ppw

    n, npml = 768, 16
    N = n + 2 * npml
    t0 = time.perf_counter()
    vel = ellipsoid_grf_velocity(n, n, n, seed=4)
    omega = omega_for_ppw(float(vel.min()), H)
    src = c4_source(vel, npml)
    t_gen = time.perf_counter() - t0
    print(json.dumps({"c4": "inputs", "gen_s": round(t_gen, 1), "c_min": float(vel.min()),
                      "c_max": float(vel.max()), "source": src}), flush=True)
    table = load_iofd_table()
    dev = torch.device("cuda", 0)
    torch.cuda.set_device(dev)
    stream = torch.cuda.current_stream(dev)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    Hh = helm.Hierarchy(torch.from_numpy(vel), H, omega, npml, precision=precision, table=table, device=dev)
    torch.cuda.synchronize()
    t_setup = time.perf_counter() - t0
    nodes = int(np.prod(Hh.shape(0)))
    cdt = Hh.cdtype
    f = torch.zeros(Hh.shape(0), dtype=cdt, device=dev)
    f[src[2], src[1], src[0]] = H ** -3
    x = torch.randn(Hh.shape(0), dtype=cdt, device=dev)
    y = torch.empty_like(x)
    Hh.apply(0, helm.OP_A, x, out=y)
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    ev0.record(stream)
    for _ in range(apply_reps):
        Hh.apply(0, helm.OP_A, x, out=y)
    ev1.record(stream)
    ev1.synchronize()
    t_apply = ev0.elapsed_time(ev1) / 1e3 / apply_reps
    per_node = 36.0 if precision == "fp64" else 20.0
    del x, y
    print(json.dumps({"c4": "apply", "avg_launch_ms": round(t_apply * 1e3, 3),
                      "GBs": round(per_node * nodes / t_apply / 1e9, 1)}), flush=True)
    u = torch.empty_like(f)
    _, its, rel, rc = Hh.solve(f, TOL, out=u.unsqueeze(0))     # warm-up
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    _, its, rel, rc = Hh.solve(f, TOL, out=u.unsqueeze(0))
    torch.cuda.synchronize()
    t_solve = time.perf_counter() - t0
    out = {"metric": "time-to-rel.res 1e-6 per RHS + stencil-apply HBM GB/s vs peak", "value": round(t_solve, 3),
           "unit": "s per RHS", "n_gpus": 1, "dtype": "f64" if precision == "fp64" else "f32",
           "data": "synthetic", "precision": precision,
           "config": {"workload": "ellipsoid-800: 768^3 + 16-cell PML, 1500 m/s with a seeded 4500 m/s ellipsoid "
                                  "(150/120/90 cells) x (1 + 0.1 GRF), 6 ppw at c_min, 1 seeded source, tol 1e-6",
                      "grid_total": N, "n_pml": npml, "nodes_fine": nodes, "source": list(src)},
           "pc_calls": int(its), "relres": float(rel), "converged": rc == 0,
           "solve_per_pc_ms": round(t_solve / max(int(its), 1) * 1e3, 2), "setup_s": round(t_setup, 3),
           "roofline": {"bound": "hbm", "kernel": f"fine-level A_h apply (27-point IOFD, 800^3, {precision})",
                        "achieved": round(per_node * nodes / t_apply / 1e9, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                        "frac": round(per_node * nodes / t_apply / 1e9 / HBM_PEAK_GBS, 4), "traffic": None,
                        "alg_bytes_per_launch": per_node * nodes, "avg_launch_ms": round(t_apply * 1e3, 4)}}
    print(json.dumps(out), flush=True)
    Hh.close()
    del Hh, f, u
    torch.cuda.empty_cache()
    if crop > 0 and with_cpu:
        print(json.dumps(c4_crop_parity(vel, omega, table, src, npml, precision, crop, crop_tol)), flush=True)


def grad_bench(steps, warmup, apply_reps, with_cpu):
    """Adjoint gradient on the benchmark workload: dJ/dm (m = 1/c^2) for the seeded point
    source and a synthetic adjoint source (seeded complex normal values at every physical
    (x, y) node of the receiver plane 20 cells below the top of the physical box), i.e. one
    forward and one adjoint solve to 1e-6 plus the row-local assembly, per step.  Also
    times the fine-level A_h^T apply (the adjoint's operator).  One JSON line."""
    import torch
    from paper_2608_22946_amd import helm
    from workloads import load_iofd_table

    vel, omega, f_np, src = workload()
    table = load_iofd_table()
    dev = torch.device("cuda", 0)
    torch.cuda.set_device(dev)
    stream = torch.cuda.current_stream(dev)
    Hh = helm.Hierarchy(torch.from_numpy(vel), H, omega, N_PML, precision="fp32", table=table, device=dev)
    N = N_PHYS + 2 * N_PML
    zr = N_PML + 20
    rng = np.random.default_rng(SEED + 100)
    s_np = np.zeros_like(f_np)
    s_np[zr, N_PML:N_PML + N_PHYS + 1, N_PML:N_PML + N_PHYS + 1] = (
        rng.standard_normal((N_PHYS + 1, N_PHYS + 1)) + 1j * rng.standard_normal((N_PHYS + 1, N_PHYS + 1)))
    f = torch.from_numpy(f_np).to(dev)
    s = torch.from_numpy(s_np).to(dev)
    nodes = int(np.prod(Hh.shape(0)))

    x = torch.randn(Hh.shape(0), dtype=torch.complex64, device=dev)
    y = torch.empty_like(x)
    for _ in range(3):
        Hh.apply(0, helm.OP_AT, x, out=y)
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    ev0.record(stream)
    for _ in range(apply_reps):
        Hh.apply(0, helm.OP_AT, x, out=y)
    ev1.record(stream)
    ev1.synchronize()
    t_at = ev0.elapsed_time(ev1) / 1e3 / apply_reps
    del x, y

    # forward solve keeping v (checkpoint), then the gradient from it: adjoint solve + assembly
    its = rel = g = None
    v = torch.empty(f.shape, dtype=torch.complex128, device=dev)
    u = torch.empty_like(f)
    for _ in range(warmup):
        _, _, its_f, rel_f, rc_f = Hh.solve_checkpoint(f, TOL, out=u.unsqueeze(0), v_out=v.unsqueeze(0))
        g, its, rel, rc = Hh.grad(f, s, TOL, v=v)
    t_fwd = t_bwd = 0.0
    for _ in range(steps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        _, _, its_f, rel_f, rc_f = Hh.solve_checkpoint(f, TOL, out=u.unsqueeze(0), v_out=v.unsqueeze(0))
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        g, its, rel, rc = Hh.grad(f, s, TOL, v=v)
        torch.cuda.synchronize()
        t_fwd += t1 - t0
        t_bwd += time.perf_counter() - t1
    t_fwd /= steps
    t_bwd /= steps
    # the same gradient with the forward solve inside helm_grad (no checkpoint), once
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    g2, its2, rel2, rc2 = Hh.grad(f, s, TOL)
    torch.cuda.synchronize()
    t_nockpt = time.perf_counter() - t0
    gd = float(torch.linalg.vector_norm(g - g2) / torch.linalg.vector_norm(g2))
    if rc != 0 or rc_f != 0 or not rel[0, 1] <= TOL or not rel_f <= TOL or not bool(torch.isfinite(g).all()):
        print(json.dumps({"error": "gradient solves did not reach the tolerance", "relres": rel.tolist()}))
        sys.exit(1)
    alg = 20.0 * nodes   # 8 B x + 4 B velocity read, 8 B y written per node
    out = {"metric": "time per misfit gradient dJ/dm given the checkpointed forward field (adjoint solve to "
                     "1e-6 + assembly)",
           "value": round(t_bwd, 4), "unit": "s per gradient", "n_gpus": 1, "steps": steps, "warmup": warmup,
           "higher_is_better": False, "dtype": "f32", "data": "synthetic",
           "config": {"workload": "grf-352-fp32 (as the main line) with a synthetic adjoint source on the "
                                  f"receiver plane z = {zr}", "source": list(src), "tol": TOL},
           "forward_solve_s": round(t_fwd, 4), "forward_plus_gradient_s": round(t_fwd + t_bwd, 4),
           "gradient_without_checkpoint_s": round(t_nockpt, 4),
           "checkpoint_vs_resolve_rel_diff": gd,
           "pc_calls_forward": int(its_f), "pc_calls_adjoint": int(its[0, 1]),
           "relres": [float(rel_f), float(rel[0, 1])],
           "roofline": {"bound": "hbm", "kernel": "fine-level A_h^T apply (rows staged per plane in LDS, 352^3, fp32)",
                        "achieved": round(alg / t_at / 1e9, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                        "frac": round(alg / t_at / 1e9 / HBM_PEAK_GBS, 4), "traffic": None,
                        "alg_bytes_per_launch": alg, "avg_launch_ms": round(t_at * 1e3, 4)}}
    if with_cpu:
        out["cpu_baseline"] = cpu_baseline(vel, omega, table, int(its_f) + int(its[0, 1]))
        out["cpu_baseline"]["unit"] = "s per gradient (extrapolated)"
    print(json.dumps(out), flush=True)


def c5_bench(n_dirs=8):
    """Misfit gradient on the 216^3 workload (192^3 + 12 PML cells): GRF velocity (seed 5),
    the true model times (1 + 0.05 exp(-r^2 / (2 * 15^2))) around the box centre (r in cells),
    16 point sources at physical (24 + 48 i, 24 + 48 j, 15), receivers at every physical (x, y)
    node of the plane z = 20, synthetic data from the true model (FP64 solves to 1e-12),
    J = 1/2 sum |u - d|^2 over receivers and sources, 6 points per wavelength at the smaller
    c_min.  Times the FP32 gradient (forward solves with checkpoint, then adjoint solves and
    assembly; tol 1e-6) and checks the FP64 gradient (tol 1e-12) against central differences of J
    along n_dirs seeded smooth velocity directions (max 0.05 m/s).  JSON lines per direction,
    then a summary."""
    import torch
    from paper_2608_22946_amd import helm
    from workloads import grf_velocity, load_iofd_table, point_source
    from workloads.configs import omega_for_ppw
    from workloads.media import gaussian_random_field

    n, npml = 192, 12
    N = n + 2 * npml
    vel0 = grf_velocity(n, n, n, seed=5)
    ax = np.arange(n + 1, dtype=np.float64) - n / 2
    r2 = ax[:, None, None] ** 2 + ax[None, :, None] ** 2 + ax[None, None, :] ** 2
    vel_true = (vel0 * (1.0 + 0.05 * np.exp(-r2 / (2 * 15.0 ** 2)))).astype(np.float32)
    del r2
    omega = omega_for_ppw(float(min(vel0.min(), vel_true.min())), H)
    srcs = [(npml + 24 + 48 * i, npml + 24 + 48 * j, npml + 15) for j in range(4) for i in range(4)]
    zr = npml + 20
    rec = (slice(None), zr, slice(npml, npml + n + 1), slice(npml, npml + n + 1))
    table = load_iofd_table()
    dev = torch.device("cuda", 0)
    torch.cuda.set_device(dev)
    F64 = torch.from_numpy(np.stack([point_source((N, N, N), sp, H) for sp in srcs])).to(dev)
    F32 = F64.to(torch.complex64)

    def hier(vel, prec):
        return helm.Hierarchy(torch.from_numpy(np.ascontiguousarray(vel)), H, omega, npml, precision=prec,
                              table=table, device=dev)

    Ht = hier(vel_true, "fp64")
    d = Ht.solve(F64, 1e-12)[0][rec].clone()
    Ht.close()

    def misfit(vel):
        Hm = hier(vel, "fp64")
        u, its, rel, rc = Hm.solve(F64, 1e-12)
        Hm.close()
        return 0.5 * float((u[rec] - d).abs().pow(2).sum())

    def gradient(prec, tol):
        Hg = hier(vel0, prec)
        F = F64 if prec == "fp64" else F32
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        u, v, its_f, rel_f, rc = Hg.solve_checkpoint(F, tol)
        s = torch.zeros_like(F)
        s[rec] = u[rec] - d.to(F.dtype)
        gm, its, rel, rc2 = Hg.grad(F, s, tol, v=v)
        gc = Hg.grad_to_velocity(gm)
        torch.cuda.synchronize()
        t = time.perf_counter() - t0
        out = gc.double().cpu().numpy()
        Hg.close()
        return out, t, int(np.sum(its_f)), int(np.sum(its[:, 1]))

    g32, t32, pf32, pa32 = gradient("fp32", 1e-6)
    g32, t32, pf32, pa32 = gradient("fp32", 1e-6)   # the second run reuses the timed tiling
    g64, t64, pf64, pa64 = gradient("fp64", 1e-12)
    J0 = misfit(vel0)
    checks = []
    for k in range(n_dirs):
        # m/s, smooth, max |dc| = 0.05: a phase change of a few 1e-3 rad over the ~30 wavelengths of the
        # box keeps J near its linear range (10 m/s moved phases by ~1 rad).  The data residual is only
        # ~1e-4 of |d| here, so the cubic term of J still biases a central difference by O(dc^2):
        # steps dc and dc / 2 and their Richardson extrapolation (4 D(dc/2) - D(dc)) / 3 remove it.
        dc = 0.05 * gaussian_random_field(n, n, n, 15.0, 500 + k)
        cd, ad = [], []
        for scale in (1.0, 0.5):
            vp = (vel0 + scale * dc).astype(np.float32)
            vm = (vel0 - scale * dc).astype(np.float32)
            jp, jm = misfit(vp), misfit(vm)
            cd.append((jp - jm) / 2.0)
            # the velocities evaluated are FP32-rounded: project onto the perturbation actually taken
            ad.append(float(np.sum(g64 * (vp.astype(np.float64) - vm.astype(np.float64)))) / 2.0)
        # the adjoint values for dc and dc / 2 differ only by the rounding of the perturbed velocities
        rich = (4.0 * cd[1] / ad[1] - cd[0] / ad[0]) / 3.0   # extrapolated ratio central difference / adjoint
        checks.append({"dir": k, "central_difference": cd[0], "adjoint": ad[0],
                       "rel_diff": abs(ad[0] - cd[0]) / abs(cd[0]),
                       "rel_diff_half_step": abs(ad[1] - cd[1]) / abs(cd[1]),
                       "rel_diff_richardson": abs(rich - 1.0)})
        print(json.dumps({"c5": "direction", **checks[-1]}), flush=True)
    out = {"c5": "gradient", "workload": "grf-216-grad: 192^3 + 12 PML, GRF seed 5 x (1 + 0.05 Gaussian blob), "
                                        "16 sources, receivers on z = 20, J = 1/2 sum |u - d|^2",
           "nodes_fine": int(N + 1) ** 3, "misfit": J0,
           "data_residual_rel": float(np.sqrt(2 * J0) / float(d.abs().pow(2).sum().sqrt())),
           "fp32_gradient_s": round(t32, 3), "fp32_pc_calls_forward": pf32, "fp32_pc_calls_adjoint": pa32,
           "fp64_gradient_s": round(t64, 3), "fp64_pc_calls_forward": pf64, "fp64_pc_calls_adjoint": pa64,
           "fp32_vs_fp64_gradient_rel_l2": float(np.linalg.norm(g32 - g64) / np.linalg.norm(g64)),
           "fd_check_max_rel_diff": max(c["rel_diff"] for c in checks),
           "fd_check_max_rel_diff_richardson": max(c["rel_diff_richardson"] for c in checks),
           "fd_directions": len(checks)}
    print(json.dumps(out), flush=True)


def marked_solve(precision):
    """One warm solve of the benchmark workload, then one solve between two fills of a
    12,345-element marker tensor, so that a kernel trace can select that solve's launches."""
    import torch
    from paper_2608_22946_amd import helm
    from workloads import load_iofd_table
    vel, omega, f_np, src = workload()
    dev = torch.device("cuda", 0)
    cdt = torch.complex128 if precision == "fp64" else torch.complex64
    Hh = helm.Hierarchy(torch.from_numpy(vel), H, omega, N_PML, precision=precision, table=load_iofd_table(),
                        device=dev)
    f = torch.from_numpy(f_np).to(dev).to(cdt)
    u = torch.empty_like(f)
    Hh.solve(f, TOL, out=u.unsqueeze(0))
    marker = torch.empty(12345, device=dev)
    marker.fill_(1.0)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    _, its, rel, rc = Hh.solve(f, TOL, out=u.unsqueeze(0))
    torch.cuda.synchronize()
    t = time.perf_counter() - t0
    marker.fill_(2.0)
    torch.cuda.synchronize()
    print(json.dumps({"marked_solve_s": round(t, 4), "pc_calls": int(its), "relres": float(rel), "rc": rc,
                      "precision": precision}), flush=True)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--apply-reps", type=int, default=50)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--precision", choices=["fp32", "fp64", "mixed"], default="fp32",
                    help="working precision of the solver (default fp32; the timing line above is quoted on it; "
                         "mixed: fp32 arithmetic with half-precision storage inside the 2h-4h cycle)")
    ap.add_argument("--profile-apply", action="store_true",
                    help="only run the fine-level apply loop and a plain copy of the same size (for counters)")
    ap.add_argument("--paper-table", action="store_true",
                    help="run the paper's 512^3 Green-function and benchmark-media cases instead (JSON line per case)")
    ap.add_argument("--multi-rhs", action="store_true",
                    help="run the 64-source 288^3 layered workload over (lanes, batch) settings instead")
    ap.add_argument("--multi-rhs-configs", default="",
                    help="with --multi-rhs: comma-separated LANESxBATCH[:PRECISION] settings, e.g. 1x1,1x8,2x8:mixed")
    ap.add_argument("--grad", action="store_true",
                    help="time the adjoint misfit gradient on the benchmark workload instead")
    ap.add_argument("--green-pml", action="store_true",
                    help="run the 512^3 Green-function case under the alternative PML readings instead")
    ap.add_argument("--c5", action="store_true",
                    help="run the 216^3 misfit-gradient workload with its central-difference check instead")
    ap.add_argument("--c4", action="store_true",
                    help="run the 800^3 ellipsoid workload (largest single-GPU case) instead")
    ap.add_argument("--crop", type=int, default=128,
                    help="with --c4: physical cells of the oracle-checked crop around the source (0: none)")
    ap.add_argument("--crop-tol", type=float, default=1e-10, help="with --c4: the oracle's tolerance on the crop")
    ap.add_argument("--marked-solve", action="store_true",
                    help="one warm solve, then one solve between two marker fills (for per-launch kernel traces)")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py runs on exactly one GPU: the solver has no multi-GPU path (sharding is a design only).",
              file=sys.stderr)
        sys.exit(2)
    if args.paper_table:
        paper_table()
        return
    if args.marked_solve:
        marked_solve(args.precision)
        return
    if args.multi_rhs:
        if args.multi_rhs_configs:
            cfgs = []
            for c in args.multi_rhs_configs.split(","):   # LANESxBATCH, or LANESxBATCH:PRECISION
                shape, _, prec = c.partition(":")
                lanes, batch = (int(v) for v in shape.split("x"))
                cfgs.append((lanes, batch) + ((prec,) if prec else ()))
            multi_rhs(tuple(cfgs), with_cpu=not args.no_cpu_baseline)
        else:
            multi_rhs(with_cpu=not args.no_cpu_baseline)
        return
    if args.grad:
        grad_bench(args.steps, args.warmup, args.apply_reps, not args.no_cpu_baseline)
        return
    if args.c5:
        c5_bench()
        return
    if args.green_pml:
        green_pml()
        return
    if args.c4:
        c4_bench(args.precision, args.apply_reps, args.crop, args.crop_tol, not args.no_cpu_baseline)
        return

    import torch
    from paper_2608_22946_amd import helm
    from workloads import load_iofd_table

    t_gen = time.perf_counter()
    vel, omega, f_np, src = workload()
    table = load_iofd_table()
    t_gen = time.perf_counter() - t_gen
    dev = torch.device("cuda", 0)
    torch.cuda.set_device(dev)
    stream = torch.cuda.current_stream(dev)

    torch.cuda.synchronize()
    t0 = time.perf_counter()
    fp64 = args.precision == "fp64"
    cdt = torch.complex128 if fp64 else torch.complex64
    Hh = helm.Hierarchy(torch.from_numpy(vel), H, omega, N_PML, precision=args.precision, table=table, device=dev)
    torch.cuda.synchronize()
    t_setup = time.perf_counter() - t0
    # the first setup of a shape in a process times the stencil tilings; later setups of the
    # shape (here: a rebuild of the same hierarchy) reuse them
    Hh.close()
    del Hh
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    Hh = helm.Hierarchy(torch.from_numpy(vel), H, omega, N_PML, precision=args.precision, table=table, device=dev)
    torch.cuda.synchronize()
    t_setup_cached = time.perf_counter() - t0
    nodes = [int(np.prod(Hh.shape(l))) for l in range(3)]
    f = torch.from_numpy(f_np).to(dev).to(cdt)
    # algorithmic bytes per node of an apply: operand in + result out + FP32 velocity
    per_node = 36.0 if fp64 else 20.0

    # ---- fine-level stencil apply: algorithmic bytes / average kernel time (HIP events) ----
    x = torch.randn(Hh.shape(0), dtype=cdt, device=dev)
    y = torch.empty_like(x)
    for _ in range(3):
        Hh.apply(0, helm.OP_A, x, out=y)
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    ev0.record(stream)
    for _ in range(args.apply_reps):
        Hh.apply(0, helm.OP_A, x, out=y)
    ev1.record(stream)
    ev1.synchronize()
    t_apply = ev0.elapsed_time(ev1) / 1e3 / args.apply_reps
    alg_bytes = per_node * nodes[0]
    achieved = alg_bytes / t_apply / 1e9
    # device copy of one fine vector (read + write) on the same stream: the practical streaming rate
    zc = torch.empty_like(x)
    zc.copy_(x)
    ev0.record(stream)
    for _ in range(20):
        zc.copy_(x)
    ev1.record(stream)
    ev1.synchronize()
    copy_gbs = 2 * x.numel() * x.element_size() / (ev0.elapsed_time(ev1) / 1e3 / 20) / 1e9
    del zc
    if args.profile_apply:
        # the fused two-sweep Jacobi from zero on the fine level (A_h, omega_h 0.8), then a plain copy
        # of known size for counter calibration
        ev0.record(stream)
        for _ in range(args.apply_reps):
            Hh.jacobi(0, helm.OP_A, x, 2, 0.8, out=y)
        ev1.record(stream)
        ev1.synchronize()
        t_jac = ev0.elapsed_time(ev1) / 1e3 / args.apply_reps
        z = torch.empty_like(x)
        for _ in range(args.apply_reps):
            z.copy_(x)
        torch.cuda.synchronize()
        print(json.dumps({"apply_ms": t_apply * 1e3, "apply_GBs": achieved, "jacobi2_ms": t_jac * 1e3,
                          "nodes": nodes[0], "copy_bytes_each_way": x.numel() * x.element_size(),
                          "stencil_sha": stencil_hash()}))
        return
    level_gbs = {}
    for lvl in (1, 2):
        xl = torch.randn(Hh.shape(lvl), dtype=cdt, device=dev)
        yl = torch.empty_like(xl)
        Hh.apply(lvl, helm.OP_B, xl, out=yl)
        ev0.record(stream)
        for _ in range(args.apply_reps):
            Hh.apply(lvl, helm.OP_B, xl, out=yl)
        ev1.record(stream)
        ev1.synchronize()
        tl = ev0.elapsed_time(ev1) / 1e3 / args.apply_reps
        level_gbs[f"level{lvl}_B_apply_GBs_cache_resident"] = round(per_node * nodes[lvl] / tl / 1e9, 1)
    del x, y

    # ---- solves: warmup, then exactly K timed steps ----
    u = torch.empty_like(f)
    its = rel = None
    for _ in range(args.warmup):
        _, its, rel, rc = Hh.solve(f, TOL, out=u.unsqueeze(0))
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        _, its, rel, rc = Hh.solve(f, TOL, out=u.unsqueeze(0))
    torch.cuda.synchronize()
    t_total = time.perf_counter() - t0
    ms_step = t_total / args.steps * 1e3
    if rc != 0 or not rel <= TOL:
        print(json.dumps({"error": "solve did not reach the tolerance", "relres": rel, "iters": its}))
        sys.exit(1)

    traffic = None if fp64 else recorded_traffic(nodes[0])   # the committed counters are of the FP32 apply
    pr = args.precision
    out = {
        "metric": "time-to-rel.res 1e-6 per RHS + stencil-apply HBM GB/s vs peak",
        "value": round(ms_step / 1e3, 4),
        "unit": "s per RHS",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_step, 2),
        "higher_is_better": False,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64" if fp64 else "f32",
        "data": "synthetic",
        "config": {"workload": f"grf-352-{pr}: 320^3 + 16-cell PML, GRF velocity 2000 m/s +-25% (corr. 20 cells), "
                               "6 ppw at c_min, 1 seeded point source, tol 1e-6",
                   "grid_total": N_PHYS + 2 * N_PML, "n_pml": N_PML, "nodes_fine": nodes[0], "nrhs": 1,
                   "source": list(src),
                   "tol": TOL,
                   "precision": PRECISION_NOTE[pr]},
        "roofline": {"bound": "hbm", "kernel": f"fine-level A_h apply (27-point IOFD, 352^3, {pr})",
                     "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(achieved / HBM_PEAK_GBS, 4),
                     "traffic": traffic, "alg_bytes_per_launch": alg_bytes,
                     "avg_launch_ms": round(t_apply * 1e3, 4),
                     "copy_GBs": round(copy_gbs, 1), "frac_of_copy": round(achieved / copy_gbs, 4),
                     "counter_GBs": None if traffic is None else round(traffic / t_apply / 1e9, 1),
                     "counter_frac": None if traffic is None else round(traffic / t_apply / 1e9 / HBM_PEAK_GBS, 4),
                     "counter_frac_of_copy": None if traffic is None else round(traffic / t_apply / 1e9 / copy_gbs, 4)},
        "pc_calls": int(its),
        "relres": float(rel),
        "solve_per_pc_ms": round(ms_step / max(int(its), 1), 2),
        "setup_s": round(t_setup, 3),
        "setup_s_tiling_cached": round(t_setup_cached, 4),
        **level_gbs,
    }
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(vel, omega, table, int(its))
        out["parity_vs_oracle"] = crop_parity(vel, omega, table, src, args.precision)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
