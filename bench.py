"""Throughput of the GSPM time step on one MI355X.

One step is one pass of the whole hot path: volume averages, the elastic
right-hand side and its CG solve, the three GSPM stages (field right-hand
sides, 3 + 2 + 3 scalar CG solves, cross-product updates) and the unit-length
projection.  The workload is the 1M-node cube (100^3 nodes, 5.8M
tetrahedra, three random ellipsoidal inclusions, H = -0.5 Ms [100],
dt = 10 ps, CG tolerance 1e-8); the metric is node-steps/s = unique nodes x
steps / wall time, with the mesh and state already resident in HBM when the
timed region starts.

Paths: FP64, mixed (FP64 refinement around FP32 inner CG), mixed with the
extrapolated and with the learned elastic start, the same with the
preconditioned solves (the elastic CG with the lattice Green's operator, the
GS solves with Jacobi), and the optional physics (rotated crystal, local
magnetostatics).  `value` is the fastest mixed-precision path of the
workload's physics that stays within 1e-6 of the FP64 run on m and u.  Prints
one JSON line, including the roofline of that path's dominant kernel (its
launches timed by start and end events the HIP runtime records at each
kernel's own execution, or whole one-launch solves over their iterations, in
extra untimed steps after the timed region) and
the CPU oracle's throughput on a bounded sample of the same workload.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "GSPM node-steps/s at 1M nodes, mixed vs FP64 at 1e-6 rel err; HBM GB/s"
HBM_PEAK_GBS = 8000.0
WEIGHTS_FILE = os.path.join(ROOT, "paper_2510_09812_amd", "weights", "warm_start.f32")
# App. D's rotated frame: the sample axes along the crystal's <111>, <-110>, <11-2>
R111 = np.array([[1, 1, 1], [-1, 1, 0], [-1, -1, 2]], dtype=np.float64) / np.sqrt([[3.0], [2.0], [6.0]])
# committed rocprofv3 counter summaries (HBM bytes per launch) and the kernel sources each was taken on
TRAFFIC = {
    "elastic": ("profiles/traffic_elastic_cg_cube100.json",
                ["paper_2510_09812_amd/csrc/elem_kernels.hip", "paper_2510_09812_amd/csrc/device_common.h"]),
    "gs": ("profiles/traffic_gs_rows_cg_cube100.json",
           ["paper_2510_09812_amd/csrc/row_kernels.hip", "paper_2510_09812_amd/csrc/device_common.h"]),
    # whole GS solves in one launch: bytes of the launches over their iterations
    "gs_one_launch": ("profiles/traffic_resident_gs_cube100.json",
                      ["paper_2510_09812_amd/csrc/resident_kernel.h", "paper_2510_09812_amd/csrc/resident.h",
                       "paper_2510_09812_amd/csrc/device_common.h"]),
}


def kernel_hash(family: str) -> str:
    h = hashlib.sha256()
    for rel in TRAFFIC[family][1]:
        with open(os.path.join(ROOT, rel), "rb") as f:
            h.update(f.read())
    return h.hexdigest()[:16]


def cg_iteration_bytes(n_nodes: int, n_tets: int, real_bytes: int = 8) -> int:
    """Algorithmic bytes of one elastic CG iteration (one fused launch), the
    method's count: connectivity (4 x int32 per tetrahedron), FP64
    coordinates, and nine passes over 3-vectors in the working precision
    (p read and Ap written by the matvec; x, r, p, Ap read or written by the
    CG updates: seven passes).  336 B per node in FP64 and 228 B with FP32
    vectors at six tetrahedra per node; 326.0 MB (FP64) and 221.2 MB (FP32)
    at the 1M-node cube."""
    return 16 * n_tets + 24 * n_nodes + 9 * 3 * real_bytes * n_nodes


def ms_matvec_bytes(n_nodes: int, n_tets: int, real_bytes: int = 4) -> int:
    """Algorithmic bytes of one K^ms matvec launch (y = K^ms x, one scalar
    component): connectivity, FP64 coordinates, x read and y written once.
    124.2 MB with FP32 vectors at 1M nodes."""
    return 16 * n_tets + 24 * n_nodes + 2 * real_bytes * n_nodes


def gs_iteration_bytes(n_nodes: int, n_tets: int, real_bytes: int = 8) -> int:
    """One scalar GS CG iteration: connectivity, coordinates and nine scalar
    vector passes (192 B per node in FP64, 156 B in FP32)."""
    return 16 * n_tets + 24 * n_nodes + 9 * real_bytes * n_nodes


def refinement_bytes(n_nodes: int, n_tets: int, components: int) -> int:
    """One FP64 refinement of the mixed form on `components` vector
    components: the FP64 residual r = b - A x (connectivity, coordinates, x
    and b read, r written), its conversion to FP32 (r read, r32 written) and
    x += d (x read and written, d read)."""
    c = components
    return 16 * n_tets + 24 * n_nodes + c * n_nodes * (3 * 8 + (8 + 4) + (8 + 8 + 4))


def gs3_iteration_bytes(n_nodes: int, n_mag_tets: int, real_bytes: int = 4, jacobi: bool = True) -> int:
    """Algorithmic bytes of one GS CG iteration on three components (one
    fused launch), the method's count: connectivity of the magnetic
    tetrahedra, FP64 coordinates, nine vector passes per component (as
    gs_iteration_bytes) and, with Jacobi preconditioning, the diagonal once."""
    return 16 * n_mag_tets + 24 * n_nodes + 3 * 9 * real_bytes * n_nodes + (real_bytes * n_nodes if jacobi else 0)


def rows_iteration_bytes(n_nodes: int, n_tets: int, real_bytes: int, per_entry: int, diagonal: bool) -> int:
    """What an iteration inside a one-launch solve streams, its vectors being on
    the chip: per entry of the rows `per_entry` coefficients and a 16-bit
    column, and the diagonal.  A closed mesh of V nodes and T tetrahedra has V + T
    edges, each two entries (81.4 + 3.9 MB for the FP32 GS rows of the 1M-node
    cube)."""
    return 2 * (n_nodes + n_tets) * (per_entry * real_bytes + 2) + (real_bytes * n_nodes if diagonal else 0)


def one_launch(n_nodes: int, mixed: bool, elastic: bool) -> bool:
    """Whether the solves run whole in one launch: by rows per workgroup, one
    workgroup per CU of 256."""
    rows = max(64, -(-n_nodes // 256 // 64) * 64)
    return rows <= (1024 if elastic else 4096 if mixed else 2048)


def pcg_matvec_bytes(n_nodes: int, n_tets: int, real_bytes: int = 4) -> int:
    """One launch of the preconditioned elastic iteration's matvec: connectivity,
    coordinates, z and the old direction read, the new direction and q written."""
    return 16 * n_tets + 24 * n_nodes + 4 * 3 * real_bytes * n_nodes


def precond_grid(lo, hi, n_nodes: int):
    """The auxiliary grid of the elastic preconditioner: round(L_a / l) points
    per axis (at least 2), l = (V_cell / n_unique)^(1/3)."""
    L = np.asarray(hi, float) - np.asarray(lo, float)
    ell = (L.prod() / n_nodes) ** (1.0 / 3.0)
    return [max(2, int(np.floor(La / ell + 0.5))) for La in L]


def precond_bytes(n_nodes: int, grid, real_bytes: int = 4) -> int:
    """One application of the elastic preconditioner, counting each array
    once: restriction (row pointers, 8 entries of node id and weight per node,
    r read, three grid arrays written), forward FFT (three grids read, three
    half spectra written), the symbol multiply (spectra read and written, 9
    values per mode), inverse FFT (spectra read, grids written), prolongation
    (coordinates, grids, r and the diagonal read, z written)."""
    s, n = real_bytes, n_nodes
    G = int(np.prod(grid))
    half = (grid[0] // 2 + 1) * grid[1] * grid[2]
    restrict = 4 * G + 8 * n * (4 + s) + 3 * s * n + 3 * s * G
    fft = 3 * s * G + 6 * s * half
    modes = 6 * s * half + 9 * s * half + 6 * s * half
    prolong = 24 * n + 3 * s * G + 3 * s * n + 3 * s * n + 3 * s * n
    return restrict + 2 * fft + modes + prolong


def step_bytes(n_nodes: int, n_tets: int, mech_iters: float, gs_iters: float, real_bytes: int = 8,
               mech_refinements: float = 0.0, other_refinements: float = 0.0, precond: bool = False,
               grid=(1, 1, 1)) -> float:
    """Algorithmic bytes of one step: each elastic CG iteration and each
    scalar GS CG iteration in the precision its vectors use (real_bytes: 8 on
    the FP64 path, 4 for the inner iterations of the mixed path), each FP64
    refinement of the mixed path (elastic ones on three components, the
    others priced as one scalar component, a lower bound), three element
    right-hand-side passes of about 190 B per node and about 200 B per node
    of node passes (averages, updates, projection).  With precond the elastic
    iterations are the preconditioned ones and the GS ones carry the Jacobi
    diagonals."""
    mech = cg_iteration_bytes(n_nodes, n_tets, real_bytes)
    gs = gs_iteration_bytes(n_nodes, n_tets, real_bytes)
    if precond:
        # preconditioned elastic iteration: its matvec, the x/r update (x, r, p, q: five passes), the
        # preconditioner; Jacobi GS: the diagonal once more per component iteration
        mech = (pcg_matvec_bytes(n_nodes, n_tets, real_bytes) + 5 * 3 * real_bytes * n_nodes
                + precond_bytes(n_nodes, grid, real_bytes))
        gs += real_bytes * n_nodes
    rhs = 3 * (16 * n_tets + 24 * n_nodes * 4)
    nodes = 200 * n_nodes
    ref = mech_refinements * refinement_bytes(n_nodes, n_tets, 3) + other_refinements * refinement_bytes(
        n_nodes, n_tets, 1)
    return mech_iters * mech + gs_iters * gs + rhs + nodes + ref


def traffic_from_profile(family: str, path: str, workload: str = "cube100_ellipsoids"):
    """HBM bytes per launch of a kernel of the family ("elastic", "gs") on the
    path from the committed rocprofv3 counter summary, if it was taken on the
    current kernel sources and on this workload."""
    try:
        with open(os.path.join(ROOT, TRAFFIC[family][0])) as f:
            t = json.load(f)
    except (OSError, ValueError):
        return None
    if t.get("kernel_hash") != kernel_hash(family) or not t.get("workload", "").startswith(workload + " "):
        return None
    return t.get(path, {}).get("bytes_per_launch")


def cpu_baseline(case, single_core_case=None) -> dict:
    """The CPU oracle as it stands, built -O3 -march=native on this host, on
    the same workload: assembly is excluded (the paper times setup
    separately); one untimed step from the initial state warms the elastic
    start (as the GPU paths' warm-up steps do), then one step is timed on all
    the threads OpenMP gives the oracle.  With single_core_case, one more
    warm-started step of that (smaller) workload is timed on one thread (its
    untimed first step runs on all of them)."""
    import oracle
    oracle.select_native()

    threads = oracle.num_threads()

    def one(c, timed_threads):
        orc = oracle.Oracle.from_mesh(c.mesh)
        orc.set_params(c.params, hext=c.hext)
        orc.set_m(c.m0)
        orc.step(c.dt, 1)
        oracle.set_num_threads(timed_threads)
        t0 = time.perf_counter()
        st = orc.step(c.dt, 1)
        dt = time.perf_counter() - t0
        oracle.set_num_threads(threads)
        return orc.n / dt, dt, st

    v, dt, st = one(case, threads)
    out = {"value": v, "unit": "node-steps/s", "cores": threads, "kind": "oracle",
           "sample": f"step 2 of {case.name} after one untimed step from the initial state "
                     f"({st['mech_iters']} elastic CG iterations), {threads} OpenMP threads, oracle built "
                     f"-O3 -march=native, global matrix assembly excluded, {dt:.1f} s"}
    if single_core_case is not None:
        v1, dt1, st1 = one(single_core_case, 1)
        out["single_core"] = {"value": v1, "unit": "node-steps/s", "cores": 1,
                              "sample": f"step 2 of {single_core_case.name} after one untimed step "
                                        f"({st1['mech_iters']} elastic CG iterations), 1 thread, {dt1:.1f} s"}
    return out


def run_sweep(case, args) -> int:
    """The hysteresis protocol of a workload with a field sweep (the 3M-node
    cube: 41 fields, 200 steps of 10 ps each): the library's sweep driver with
    no early stop (a dm_tol no step reaches: every point runs its full length), one field
    point per call so that progress is printed.  Prints one JSON line: wall
    time, node-steps/s over the whole sweep and the mbar loop."""
    from paper_2510_09812_amd import gspm
    if case.field_sweep is None:
        print(json.dumps({"error": f"workload {case.name} has no field sweep"}))
        return 2
    params = dict(case.params)
    params["elastic_precond"] = gspm.GSPM_PRECOND_GREEN
    params["gs_precond"] = gspm.GSPM_PRECOND_JACOBI
    t_up = time.perf_counter()
    sim = gspm.Simulation(case.mesh, params, hext=case.field_sweep[0], precision=gspm.GSPM_MIXED)
    sim.set_m(case.m0)
    if args.gs_corrected:
        sim.set_gs_start(gspm.GSPM_GS_START_CORRECTED)
    path = "mixed+precond" + ("+gscorr" if args.gs_corrected else "")
    n = sim.mesh_info()["n_unique"]
    print(f"[sweep] {case.name}: {n} nodes uploaded in {time.perf_counter() - t_up:.1f} s; "
          f"{len(case.field_sweep)} fields x {case.steps} steps", file=sys.stderr, flush=True)
    loop, steps_total = [], 0
    t0 = time.perf_counter()
    for k, h in enumerate(case.field_sweep):
        r = sim.sweep(case.dt, 1e-300, case.steps, hext=np.asarray(h)[None, :], keep_going=True)
        steps_total += int(r["steps"][0])
        mbar = [float(x) for x in r["mbar"][0]]
        loop.append({"h_over_ms": float(h[0] / case.material["Ms"]), "mbar": mbar})
        print(f"[sweep] field {k}: H = {h[0] / case.material['Ms']:+.2f} Ms, mbar_x {mbar[0]:+.4f}, "
              f"{time.perf_counter() - t0:.1f} s", file=sys.stderr, flush=True)
    wall = time.perf_counter() - t0
    sim.close()
    print(json.dumps({"metric": "hysteresis sweep node-steps/s", "value": n * steps_total / wall,
                      "unit": "node-steps/s", "wall_s": wall, "steps": steps_total, "n_gpus": 1,
                      "config": {"workload": case.name, "nodes": n, "fields": len(case.field_sweep),
                                 "steps_per_field": case.steps, "dt_s": case.dt,
                                 "path": path, "cg_tol": case.params["cg_tol"]},
                      "data": "synthetic", "mbar_loop": loop}))
    return 0


def trajectory(case, gs_corrected: bool, log: str = "trajectory") -> dict:
    """The workload's configured trajectory (the 1M-node cube: 500 steps of
    10 ps from the noisy start) on the mixed path with both preconditioners,
    in windows of 50 steps: node-steps/s over the whole run, and per window
    the time and the elastic and GS iterations per step."""
    import torch

    from paper_2510_09812_amd import gspm
    params = dict(case.params)
    params["elastic_precond"] = gspm.GSPM_PRECOND_GREEN
    params["gs_precond"] = gspm.GSPM_PRECOND_JACOBI
    t_up = time.perf_counter()
    sim = gspm.Simulation(case.mesh, params, hext=case.hext, precision=gspm.GSPM_MIXED)
    sim.set_m(case.m0)
    if gs_corrected:
        sim.set_gs_start(gspm.GSPM_GS_START_CORRECTED)
    n = sim.mesh_info()["n_unique"]
    path = "mixed+precond" + ("+gscorr" if gs_corrected else "")
    print(f"[{log}] {case.name}: {n} nodes uploaded in {time.perf_counter() - t_up:.1f} s; "
          f"{case.steps} steps on {path}", file=sys.stderr, flush=True)
    win = 50
    windows, done = [], 0
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    while done < case.steps:
        k = min(win, case.steps - done)
        t1 = time.perf_counter()
        st = sim.step(case.dt, k)
        torch.cuda.synchronize()
        dt = time.perf_counter() - t1
        done += k
        mbar = [float(x) for x in sim.averages()[0]]
        windows.append({"steps": [done - k, done], "ms_per_step": dt / k * 1e3,
                        "mech_iters_per_step": st["mech_iters"] / k, "gs_iters_per_step": st["gs_iters"] / k,
                        "dm_avg_last": st["dm_avg"], "mbar": mbar})
        print(f"[{log}] {path} steps {done - k}-{done}: {dt / k * 1e3:.2f} ms/step, elastic "
              f"{st['mech_iters'] / k:.1f}, GS {st['gs_iters'] / k:.1f} iterations per step, dm_avg {st['dm_avg']:.2e}",
              file=sys.stderr, flush=True)
    wall = time.perf_counter() - t0
    sim.close()
    return {"path": path, "value": n * done / wall, "unit": "node-steps/s", "wall_s": wall, "steps": done,
            "windows": windows}


def run_trajectory(case, args) -> int:
    """Trajectory mode: one JSON line for the configured trajectory."""
    t = trajectory(case, args.gs_corrected)
    print(json.dumps({"metric": "GSPM node-steps/s over the configured trajectory", "value": t["value"],
                      "unit": "node-steps/s", "wall_s": t["wall_s"], "steps": t["steps"], "n_gpus": 1,
                      "config": {"workload": case.name, "dt_s": case.dt, "path": t["path"],
                                 "cg_tol": case.params["cg_tol"]},
                      "data": "synthetic", "windows": t["windows"]}))
    return 0


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", default="cube100_ellipsoids")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-single-core", action="store_true",
                    help="skip the one-thread oracle sample on the 100k-node cube")
    ap.add_argument("--no-profile", action="store_true", help="skip the per-launch timing steps of the elastic CG iteration")
    ap.add_argument("--profile-steps", type=int, default=2,
                    help="untimed steps after the timed region that time every elastic CG iteration kernel")
    ap.add_argument("--block-nodes", type=int, default=0, help="nodes per owner block (0 = library default)")
    ap.add_argument("--precision", choices=("fp64", "mixed", "both"), default="both",
                    help="paths to run; with both, `value` is the mixed path (with the learned warm start when "
                         "trained weights exist) and the other paths are reported beside it")
    ap.add_argument("--no-learned", action="store_true", help="skip the learned warm start path")
    ap.add_argument("--no-rotated", action="store_true",
                    help="skip the path with the crystal rotated to the <111> frame of App. D")
    ap.add_argument("--only", default="",
                    help="comma-separated path names to run (for profiling one path), e.g. mixed+precond")
    ap.add_argument("--no-precond", action="store_true",
                    help="skip the paths with the Green's-operator preconditioned elastic solve")
    ap.add_argument("--trajectory", action="store_true",
                    help="instead of the step benchmark, run the workload's configured number of steps in windows")
    ap.add_argument("--no-trajectory", action="store_true",
                    help="skip the run of the whole configured trajectory that the default output carries")
    ap.add_argument("--gs-corrected", action="store_true",
                    help="trajectory and sweep modes: start the GS solves from the lumped solution plus the last "
                         "correction")
    ap.add_argument("--sweep", action="store_true",
                    help="instead of the step benchmark, run the workload's hysteresis sweep protocol (every field "
                         "point for its configured number of steps) on the mixed path with both preconditioners")
    ap.add_argument("--deterministic", action="store_true",
                    help="also run the preconditioned paths in the bitwise-reproducible mode")
    ap.add_argument("--no-local-demag", action="store_true",
                    help="skip the paths with the local magnetostatic solve (reported beside the headline)")
    ap.add_argument("--copy-calib-mb", type=int, default=0,
                    help="first fill and sum a buffer of this many MiB (HBM counter calibration)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(json.dumps({"error": "the library runs on one GPU; sharding across GPUs is designed, not implemented",
                          "n_gpus": args.gpus}))
        return 2

    import torch

    import workloads as w
    from paper_2510_09812_amd import gspm

    if not torch.cuda.is_available():
        print(json.dumps({"error": "no GPU visible"}))
        return 1
    torch.cuda.set_device(0)
    if args.copy_calib_mb > 0:
        # HBM counter calibration: a fill writes and a sum reads exactly this many MiB
        src = torch.ones(args.copy_calib_mb * (1 << 20) // 8, dtype=torch.float64, device="cuda")
        total = float(src.sum())
        torch.cuda.synchronize()
        print(f"[bench] calibration fill and sum of {args.copy_calib_mb} MiB done ({total:.0f})", file=sys.stderr,
              flush=True)
        del src
    print(f"[bench] building workload {args.workload}", file=sys.stderr, flush=True)
    case = w.CASES[args.workload]()
    if args.sweep:
        return run_sweep(case, args)
    if args.trajectory:
        return run_trajectory(case, args)

    weights = None
    if not args.no_learned and os.path.exists(WEIGHTS_FILE):
        weights = np.fromfile(WEIGHTS_FILE, dtype=np.float32)
        if weights.size != gspm.GSPM_MPNN_PARAMS:
            weights = None

    def run_path(precision: int, warm: int = 0, local_demag: bool = False, rotated: bool = False,
                 precond: bool = False, deterministic: bool = False, gs_corrected: bool = False) -> dict:
        t_up = time.perf_counter()
        params = dict(case.params)
        if rotated:
            params["crystal_rot"] = R111
        if precond:
            params["elastic_precond"] = gspm.GSPM_PRECOND_GREEN
            params["gs_precond"] = gspm.GSPM_PRECOND_JACOBI
        sim = gspm.Simulation(case.mesh, params, hext=case.hext, device=0, profile=False,
                              block_nodes=args.block_nodes, precision=precision, local_demag=local_demag,
                              deterministic=deterministic)
        sim.set_m(case.m0)
        if warm == gspm.GSPM_WARM_LEARNED:
            sim.mpnn_set_params(weights)
        sim.set_warm_start(warm)
        if gs_corrected:
            sim.set_gs_start(gspm.GSPM_GS_START_CORRECTED)
        info = sim.mesh_info()
        t_up = time.perf_counter() - t_up
        tag = (f"{'mixed' if precision else 'fp64'}" + {0: "", 1: "+learned", 2: "+extrapolated"}[warm]
               + ("+local_demag" if local_demag else "") + ("+rotated111" if rotated else "")
               + ("+precond" if precond else "") + ("+gscorr" if gs_corrected else "")
               + ("+deterministic" if deterministic else ""))
        print(f"[bench] {tag}: uploaded {info['n_unique']} nodes, {info['n_tets']} tets in "
              f"{t_up:.1f} s; warmup {args.warmup}", file=sys.stderr, flush=True)
        if args.warmup:
            sim.step(case.dt, args.warmup)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        st = sim.step(case.dt, args.steps)
        torch.cuda.synchronize()
        wall = time.perf_counter() - t0
        print(f"[bench] {tag}: {args.steps} steps in {wall:.3f} s, mech iters {st['mech_iters']}, "
              f"gs iters {st['gs_iters']}, ms iters {st['ms_iters']}, refinements {st['refinements']}, "
              f"learned starts {st['learned_starts']}, min-residual starts {st['minres_starts']}, "
              f"last coefficients {st['warm_coef']}", file=sys.stderr, flush=True)
        out = dict(info=info, st=st, wall=wall, value=info["n_unique"] * args.steps / wall, m=sim.get_m(),
                   u=sim.get_u(), tag=tag)
        if local_demag:
            out["ud"] = sim.get_ud()
            if precision == gspm.GSPM_MIXED:
                # the K^ms operator the inner solves run: device-resident launches between events
                out["ms_matvec_ms"] = sim.time_operator(gspm.GSPM_OP_MS, reps=50)
                print(f"[bench] {tag}: K^ms matvec {out['ms_matvec_ms'] * 1e3:.1f} us per launch (FP32)",
                      file=sys.stderr, flush=True)
        elif not args.no_profile:
            # kernel durations from extra untimed steps: every elastic CG iteration is
            # launched with a start/stop event pair that the runtime records at
            # the kernel's own execution (hipExtLaunchKernelGGL), not in the timed region
            sim.set_profile(True)
            pst = sim.step(case.dt, args.profile_steps)
            out["prof"] = pst
            print(f"[bench] {tag}: {pst['matvec_launches']} elastic CG launches timed, "
                  f"{pst['matvec_ms'] / max(pst['matvec_launches'], 1) * 1e3:.1f} us each", file=sys.stderr, flush=True)
        sim.close()
        return out

    specs = [("fp64", dict(precision=gspm.GSPM_FP64)), ("mixed", dict(precision=gspm.GSPM_MIXED))]
    if not args.no_learned:
        specs.append(("mixed+extrapolated", dict(precision=gspm.GSPM_MIXED, warm=gspm.GSPM_WARM_EXTRAPOLATE)))
    if weights is not None:
        specs.append(("mixed+learned", dict(precision=gspm.GSPM_MIXED, warm=gspm.GSPM_WARM_LEARNED)))
    if not args.no_precond:
        specs += [("fp64+precond", dict(precision=gspm.GSPM_FP64, precond=True)),
                  ("mixed+precond", dict(precision=gspm.GSPM_MIXED, precond=True)),
                  # GS solves started from the lumped solution plus the last step's correction
                  ("fp64+precond+gscorr", dict(precision=gspm.GSPM_FP64, precond=True, gs_corrected=True)),
                  ("mixed+precond+gscorr", dict(precision=gspm.GSPM_MIXED, precond=True, gs_corrected=True))]
        if not args.no_learned:
            specs.append(("mixed+extrapolated+precond", dict(precision=gspm.GSPM_MIXED,
                                                             warm=gspm.GSPM_WARM_EXTRAPOLATE, precond=True)))
        if weights is not None:
            specs.append(("mixed+learned+precond", dict(precision=gspm.GSPM_MIXED, warm=gspm.GSPM_WARM_LEARNED,
                                                        precond=True)))
        if args.deterministic:
            # the bitwise-reproducible mode (fixed-order sums), reported beside the others
            specs += [("fp64+precond+deterministic", dict(precision=gspm.GSPM_FP64, precond=True, deterministic=True)),
                      ("mixed+precond+deterministic", dict(precision=gspm.GSPM_MIXED, precond=True,
                                                           deterministic=True))]
    if not args.no_rotated:
        specs += [("fp64+rotated111", dict(precision=gspm.GSPM_FP64, rotated=True)),
                  ("mixed+rotated111", dict(precision=gspm.GSPM_MIXED, rotated=True))]
    if not args.no_local_demag:
        specs += [("fp64+local_demag", dict(precision=gspm.GSPM_FP64, local_demag=True)),
                  ("mixed+local_demag", dict(precision=gspm.GSPM_MIXED, local_demag=True))]
    only = set(args.only.split(",")) if args.only else None
    paths = {}
    for name, kw in specs:
        if args.precision != "both" and not name.startswith(args.precision):
            continue
        if only is not None and name not in only:
            continue
        paths[name] = run_path(**kw)
    um = lambda u: u - u.mean(axis=0)

    def within_target(k):
        """mixed path within 1e-6 of the FP64 run on m and the mean-removed u"""
        if "fp64" not in paths:
            return True
        f, p = paths["fp64"], paths[k]
        em = np.linalg.norm(p["m"] - f["m"]) / np.linalg.norm(f["m"])
        eu = np.linalg.norm(um(p["u"]) - um(f["u"])) / np.linalg.norm(um(f["u"]))
        return em <= 1e-6 and eu <= 1e-6

    # `value`: the fastest mixed-precision path of the workload's physics that stays within the
    # metric's 1e-6 of the FP64 run (the optional terms are other physics, reported beside it)
    base = [k for k in paths if k.startswith("mixed") and "+local_demag" not in k and "+rotated111" not in k
            and "+deterministic" not in k]
    good = [k for k in base if within_target(k)]
    head_name = (max(good, key=lambda k: paths[k]["value"]) if good
                 else next((k for k in ("mixed", "fp64") if k in paths), next(iter(paths))))
    head = paths[head_name]
    mixed = head_name.startswith("mixed")
    precond = "+precond" in head_name
    info, st, wall, value = head["info"], head["st"], head["wall"], head["value"]
    n, ne = info["n_unique"], info["n_tets"]
    ne_mag = int(np.count_nonzero(case.mesh.tags))
    rb = 4 if mixed else 8
    tname = "float" if mixed else "double"

    # the roofline of the path's dominant kernel, by summed duration over the profile steps: the
    # elastic iteration launch, or the GS CG iteration launch on three components
    roofline = None
    pst = head.get("prof")
    if pst and (pst["matvec_launches"] > 0 or pst["gs_matvec_launches"] > 0):
        if pst["gs_matvec_ms"] > pst["matvec_ms"]:
            launches, tot_ms = pst["gs_matvec_launches"], pst["gs_matvec_ms"]
            path = ("mixed" if mixed else "fp64") + ("+precond" if precond else "")
            whole = one_launch(n, mixed, elastic=False)
            what = "GS CG iteration on three components"
            if whole:
                mb = rows_iteration_bytes(n, ne_mag, rb, 1, diagonal=True)
                kname = f"k_resident<{tname},3>" + (" (Jacobi)" if precond else "")
                traffic = traffic_from_profile("gs_one_launch", path, case.name)
            else:
                mb = gs3_iteration_bytes(n, ne_mag, rb, jacobi=precond)
                kname = f"k_gs_rows_cg<{tname},3>" + (" (Jacobi)" if precond else "")
                traffic = traffic_from_profile("gs", path, case.name)
        else:
            launches, tot_ms = pst["matvec_launches"], pst["matvec_ms"]
            whole = not precond and one_launch(n, mixed, elastic=True)
            what = "elastic CG iteration"
            if whole:
                mb = rows_iteration_bytes(n, ne, rb, 6, diagonal=False)
                kname = f"k_resident<{tname},3,blocks>"
                traffic = None
            elif precond:
                mb = pcg_matvec_bytes(n, ne, rb)
                kname = f"k_strip<{tname},3,3,ElasticPcgOp>"
                traffic = traffic_from_profile("elastic", ("mixed" if mixed else "fp64") + "+precond", case.name)
            else:
                mb = cg_iteration_bytes(n, ne, rb)
                kname = f"k_strip<{tname},3,3,ElasticCgOp>"
                traffic = traffic_from_profile("elastic", "mixed" if mixed else "fp64", case.name)
        avg_s = tot_ms / launches * 1e-3
        achieved = mb / avg_s / 1e9
        # an iteration by launches is priced with the method's vector passes against HBM; inside a one-launch solve the
        # rows stream from Infinity Cache and the chain of an exchange, not a rate, sets the time
        roofline = {"bound": "latency" if whole else "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                    "frac": achieved / HBM_PEAK_GBS, "traffic": traffic, "kernel": kname, "bytes_per_launch": mb,
                    "avg_launch_us": avg_s * 1e6, "launches": launches,
                    "share_of_timed_kernels": {"elastic_ms": pst["matvec_ms"], "gs3_iteration_ms": pst["gs_matvec_ms"]},
                    "timing": (f"events around every one-launch solve of {args.profile_steps} untimed steps after the timed "
                               f"region, refinements included, over their iterations ({what}); bytes and traffic likewise"
                               if whole else
                               f"kernel start/end events (hipExtLaunchKernelGGL) on every working launch ({what}) of "
                               f"{args.profile_steps} untimed steps after the timed region")}
    mech_per_step = st["mech_iters"] / args.steps
    gs_per_step = st["gs_iters"] / args.steps
    mref = st["mech_refinements"] / args.steps
    b_step = step_bytes(n, ne, mech_per_step, gs_per_step, rb, mref, st["refinements"] / args.steps - mref,
                        precond=precond, grid=precond_grid(case.mesh.lo, case.mesh.hi, n))
    per_path = {}
    for k, p in paths.items():
        row = {"value": p["value"], "ms_per_step": p["wall"] / args.steps * 1e3,
               "mech_iters_per_step": p["st"]["mech_iters"] / args.steps,
               "gs_iters_per_step": p["st"]["gs_iters"] / args.steps,
               "refinements_per_step": p["st"]["refinements"] / args.steps,
               "learned_starts": p["st"]["learned_starts"], "minres_starts": p["st"]["minres_starts"]}
        ld = k.endswith("+local_demag")
        if ld:
            row["ms_iters_per_step"] = p["st"]["ms_iters"] / args.steps
        if "prof" in p and p["prof"]["matvec_launches"] > 0:
            row["elastic_cg_launch_us"] = p["prof"]["matvec_ms"] / p["prof"]["matvec_launches"] * 1e3
        if "prof" in p and p["prof"]["gs_matvec_launches"] > 0:
            row["gs3_iteration_launch_us"] = p["prof"]["gs_matvec_ms"] / p["prof"]["gs_matvec_launches"] * 1e3
        ref = "fp64+local_demag" if ld else ("fp64+rotated111" if k.endswith("+rotated111") else "fp64")
        if "+precond" in k:
            row["ref_note"] = "errors against the unpreconditioned FP64 path"
        if ref in paths and k != ref:
            f = paths[ref]
            row["speedup_vs_" + ref] = p["value"] / f["value"]
            row["rel_err_m_vs_" + ref] = float(np.linalg.norm(p["m"] - f["m"]) / np.linalg.norm(f["m"]))
            row["rel_err_u_vs_" + ref] = float(np.linalg.norm(um(p["u"]) - um(f["u"])) / np.linalg.norm(um(f["u"])))
            if ld:
                row["rel_err_ud_vs_" + ref] = float(np.linalg.norm(p["ud"] - f["ud"]) / np.linalg.norm(f["ud"]))
        per_path[k] = row
    ms_roofline = None
    if "mixed+local_demag" in paths:
        t = paths["mixed+local_demag"]["ms_matvec_ms"] * 1e-3
        mb = ms_matvec_bytes(n, ne, 4)
        ms_roofline = {"bound": "hbm", "achieved": mb / t / 1e9, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                       "frac": mb / t / 1e9 / HBM_PEAK_GBS, "traffic": traffic_from_profile("elastic", "ms_mixed", case.name),
                       "kernel": "k_strip<float,1,1,MsMatvecOp<float,1>>", "bytes_per_launch": mb,
                       "avg_launch_us": t * 1e6,
                       "timing": "50 device-resident launches of y = K^ms x between HIP events on the library's stream"}
    out = {
        "metric": METRIC, "value": value, "unit": "node-steps/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": wall / args.steps * 1e3, "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "f32+f64" if mixed else "f64",
        "data": "synthetic",
        "config": {"workload": case.name, "nodes": n, "tets": ne, "dt_s": case.dt, "cg_tol": case.cg_tol,
                   "path": head_name, "block_nodes": args.block_nodes or 256,
                   "precond": ("elastic: lattice Green's operator on the auxiliary grid; GS: Jacobi" if precond
                               else "none (the paper's unpreconditioned CG)"),
                   "gs_start": ("lumped solution + the stage's correction at the last step" if "+gscorr" in head_name
                                else "lumped solution"),
                   "mech_iters_per_step": mech_per_step, "gs_iters_per_step": gs_per_step},
        "roofline": roofline,
        "step_roofline": {"bytes_per_node_step": b_step / n, "roofline_node_steps_per_s": HBM_PEAK_GBS * 1e9 / b_step * n,
                          "frac": value / (HBM_PEAK_GBS * 1e9 / b_step * n),
                          "inputs": {"mech_iters_per_step": mech_per_step, "gs_iters_per_step": gs_per_step,
                                     "real_bytes": 4 if mixed else 8, "mech_refinements_per_step": mref,
                                     "other_refinements_per_step": st["refinements"] / args.steps - mref,
                                     "preconditioned": precond}},
        "paths": per_path,
        "ms_roofline": ms_roofline,
        # device time per phase of the step on the value path (profile steps after the timed region)
        "phase_ms_per_step": ({k: v / args.profile_steps for k, v in pst["phase_ms"].items()} if pst else None),
        "final_residual": st["final_residual"],
    }
    if not args.no_trajectory and not args.no_precond and case.steps > args.warmup + args.steps:
        # the whole configured trajectory beside the timed window (which lies in its transient)
        out["trajectory"] = {t["path"]: {k: v for k, v in t.items() if k != "path"}
                             for t in (trajectory(case, False, "bench"), trajectory(case, True, "bench"))}
    if not args.no_cpu_baseline:
        print("[bench] CPU oracle baseline", file=sys.stderr, flush=True)
        out["cpu_baseline"] = cpu_baseline(case, None if args.no_single_core else w.cube47_sphere())
    else:
        out["cpu_baseline"] = None
    print(json.dumps(out), flush=True)
    return 0


if __name__ == "__main__":
    sys.exit(main())
