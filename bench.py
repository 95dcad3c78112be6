"""Throughput benchmark of the Stein-MAP-Seq hot path on one MI355X.

One benchmark step = Algorithm 2 end to end (predictive initial particles,
L SVGD iterations and the forward recursion at every time step, then the
backtrack) over a batch of independent synthetic sequences already resident
in HBM.  The default workload is the 7-joint arm (N = 1024 particles, d = 7,
L = 100 iterations, T = 100 steps) with a batch of Monte-Carlo sequences.

Printed as one JSON line: SVGD particle-iterations per second (value), the
whole-job Viterbi edge rate, the roofline of the dominant kernel (the fused
step kernel, timed per launch with HIP events on the launch stream), a
lattice-mode forward-recursion bandwidth figure, the CPU oracle timed on a
bounded sample of the same workload, the kernel / bandwidth / particle-count
ablation grid on the 1-D growth model (``kernel_ablation``), the SE(2) pose
scenario with unknown landmark association (``scenario_b``), the 14-D
manipulator (``scenario_d``), the PF-MAP-Seq forward recursion on
bootstrap-PF particle sets (``pf_map_seq``), and
(``batched``) a ragged mix of all
four model families with uneven N and T (4096 sequences) run as batched
plans: the plain method at the full iteration count (the reference MAP
log-posterior of every sequence), then the plain method and the learned
initialisation (trained first on plain runs of a separate, shorter mix) at
fractions of the iterations, with the iterations each needs to match the
reference.
"""
from __future__ import annotations

import argparse
import itertools
import json
import math
import os
import platform
import re
import subprocess
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_FP32 = 157.3e12   # MI355X FP32 peak (FLOP/s), matrix cores and vector ALU alike
PEAK_BF16 = 2.5e15     # dense, 16-bit matrix cores
PEAK_FP64 = 78.6e12
PEAK_HBM = 8.0e12      # B/s

# Counted flops of the observation-gradient evaluation per particle (FMA = 2),
# per model family; used in F_iter = N^2 (6d+6) + N N_p (4d+6) + N (c_obs + 6d).
C_OBS = {"growth1d": 10, "range2d": 60, "cv4d": 150, "arm7": 1100, "lingauss": 16}


def executed_matrix_flops(n: int, n_prev: int, d: int) -> float:
    """16-bit matrix-core flops of one iteration of the matrix-core step: a
    16x16x32 product is 64 flops per pair of a tile and 32 per pair of a sum; two
    products a tile (d <= 3: one) and three a sum (d <= 4: two) in the score and
    Stein passes, and those of a tile per distance."""
    p, w = (3.5 if d > 4 else 3, 2) if d > 3 else (2, 1)
    return 64.0 * (p * n * n_prev + p * n * n + w * n * n / 2)


def flops_per_iteration(n: int, n_prev: int, d: int, name: str) -> float:
    return n * n * (6 * d + 6) + n * n_prev * (4 * d + 6) + n * (C_OBS[name] + 6 * d)


def parse():
    p = argparse.ArgumentParser()
    p.add_argument("--gpus", type=int, default=1)
    p.add_argument("--steps", type=int, default=2)
    p.add_argument("--warmup", type=int, default=1)
    p.add_argument("--workload", default="arm7")
    p.add_argument("--batch", type=int, default=256)
    p.add_argument("--T", type=int, default=None)
    p.add_argument("--cpu-baseline", type=int, default=1)
    p.add_argument("--lattice-n", type=int, default=4096)
    p.add_argument("--lattice-batch", type=int, default=16)
    p.add_argument("--batched-seqs", type=int, default=4096, help="ragged-mix sequences (0: skip)")
    p.add_argument("--train-steps", type=int, default=4000)
    p.add_argument("--train-seqs", type=int, default=700, help="plain sequences whose steps train the proposal")
    p.add_argument("--train-L", type=float, default=2.0,
                   help="iterations of the plain training runs, as a multiple of each family's L")
    p.add_argument("--ablation-mc", type=int, default=50, help="sequences per kernel-ablation row (0: skip)")
    p.add_argument("--scenario-b-mc", type=int, default=10, help="pose-scenario sequences per row (0: skip)")
    p.add_argument("--scenario-d-mc", type=int, default=20, help="14-D arm sequences per row (0: skip)")
    p.add_argument("--pf-map-seq", type=int, default=1, help="PF-MAP-Seq forward-recursion workload (0: skip)")
    p.add_argument("--latency", type=int, default=1, help="small-batch per-step times (0: skip)")
    p.add_argument("--cpu-table", action="store_true",
                   help="only the CPU oracle table (single thread and all-core, four workloads)")
    p.add_argument("--sweep", action="store_true",
                   help="print the batch / N / workload sweeps as one JSON line instead of the benchmark")
    p.add_argument("--copy-probe-mib", type=int, default=0,
                   help="first copy this many MiB device to device three times (calibrates HBM byte counters)")
    return p.parse_args()


TRAFFIC_PROFILE = os.path.join(ROOT, "profiles", "k_step_mfma_arm7_n1024_d7_b256_traffic.md")


def kernel_source_digest() -> str:
    """SHA-256 over the kernel sources (every file under csrc, by name)."""
    import hashlib
    h = hashlib.sha256()
    src = os.path.join(ROOT, "paper_2312_08684_amd", "csrc")
    for f in sorted(os.listdir(src)):
        if f.endswith((".hpp", ".hip", ".h")):
            h.update(f.encode())
            with open(os.path.join(src, f), "rb") as fh:
                h.update(fh.read())
    return h.hexdigest()


def measured_traffic(name: str, B: int, n: int, dt: str):
    """HBM bytes per steady-state launch from the committed counter summary,
    or None when it was taken on other kernel sources or another workload."""
    if (name, B, n, dt) != ("arm7", 256, 1024, "f32") or not os.path.exists(TRAFFIC_PROFILE):
        return None
    fields = {}
    with open(TRAFFIC_PROFILE) as fh:
        for line in fh:
            if ":" in line and line.startswith("- "):
                k, v = line[2:].split(":", 1)
                fields[k.strip()] = v.strip().strip("`")
    if fields.get("kernel sources sha256") != kernel_source_digest():
        return None
    try:
        return float(fields["HBM bytes per launch"])
    except (KeyError, ValueError):
        return None


def device_info(torch) -> dict:
    """The GPU the line was measured on: torch's device properties and, from
    rocminfo, the first GPU agent's compute units and maximum clock, with the
    FP32 matrix-core peak they imply (256 flops per clock per compute unit)."""
    p = torch.cuda.get_device_properties(0)
    info = {"name": p.name, "arch": getattr(p, "gcnArchName", ""), "compute_units": p.multi_processor_count,
            "hbm_bytes": p.total_memory}
    try:
        txt = subprocess.run(["rocminfo"], capture_output=True, text=True, timeout=60).stdout
    except (OSError, subprocess.SubprocessError):
        return info
    for block in txt.split("\nAgent ")[1:]:
        if not re.search(r"Device Type:\s+GPU", block):
            continue
        cu = re.search(r"Compute Unit:\s+(\d+)", block)
        mhz = re.search(r"Max Clock Freq\. \(MHz\):\s+(\d+)", block)
        if cu and mhz:
            info["rocminfo_compute_units"] = int(cu.group(1))
            info["rocminfo_max_clock_mhz"] = int(mhz.group(1))
            info["fp32_matrix_peak_tflops"] = int(cu.group(1)) * int(mhz.group(1)) * 1e6 * 256 / 1e12
        break
    return info


def cpu_model() -> str:
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return platform.processor() or platform.machine()


def cpu_threads() -> int:
    """Host threads for the all-core oracle: the CPU share the process is
    given (OMP_NUM_THREADS), at most the visible cores."""
    n = os.cpu_count() or 1
    try:
        n = min(n, int(os.environ.get("OMP_NUM_THREADS", n)))
    except ValueError:
        pass
    return max(1, n)


def cpu_baseline(name: str):
    """The FP64 oracle on one time step (t = 2) of one sequence of the
    workload: single thread, then all-core (OpenMP over particles; the same
    bits).  `value` is the all-core rate."""
    import oracle as O
    from paper_2312_08684_amd import scenarios as S
    wl = S.make_workload(name, B=1, seed=0, T=2)
    desc, o, n = wl.model, wl.opts, wl.n
    rng = np.random.default_rng(0)
    sd = np.sqrt(desc.q_var[:desc.d])
    xprev = wl.truth[0, 1][None, :] + sd * rng.normal(size=(n, desc.d))
    x_init = O.predictive_init(desc, 2, xprev, n, 1, 0)
    mask = None if wl.mask is None else wl.mask[0, 1]
    res, secs = {}, {}
    cores = cpu_threads()
    for th in (1, cores):
        O.set_threads(th)
        t0 = time.perf_counter()
        x, _, _ = O.svgd_step(desc, 2, xprev, None, wl.z[0, 1], mask, x_init, o.n_iter, o.step)
        O.viterbi_particle(desc, 2, xprev, np.zeros(n), wl.z[0, 1], mask, x)
        secs[th] = time.perf_counter() - t0
        res[th] = x
    same = bool(np.array_equal(res[1], res[cores]))
    return {"value": n * o.n_iter / secs[cores], "unit": "particle-iters/s", "cores": cores, "kind": "oracle",
            "sample": "one time step (t=2) of one %s sequence: N=%d, d=%d, %d SVGD iterations + forward "
                      "recursion, FP64 oracle; %d threads (OpenMP over particles) %.2f s, one thread %.2f s; "
                      "results bit-identical: %s" % (name, n, desc.d, o.n_iter, cores, secs[cores], secs[1], same),
            "single_thread": {"value": n * o.n_iter / secs[1], "seconds": secs[1]},
            "all_core_seconds": secs[cores], "bit_identical": same,
            "host_cpus": os.cpu_count(), "cpu_model": cpu_model()}


# steps timed per workload in the CPU table (the 7-DOF arm truncated to 5)
CPU_TABLE_STEPS = {"growth1d": 50, "range2d": 20, "cv4d": 10, "arm7": 5}


def cpu_table():
    """Algorithm 2 in the FP64 oracle on the first steps of one sequence of
    each workload, single thread and all-core: ms per step, particle-iters/s."""
    import oracle as O
    from paper_2312_08684_amd import scenarios as S
    rows = []
    cores = cpu_threads()
    for name, k in CPU_TABLE_STEPS.items():
        wl = S.make_workload(name, B=1, seed=0)
        T = min(k, wl.T)
        mask = None if wl.mask is None else wl.mask[0][:T]
        row = {"workload": name, "N": wl.n, "d": wl.model.d, "L": wl.opts.n_iter, "steps": T}
        for th, key in ((1, "single"), (cores, "all_core")):
            O.set_threads(th)
            t0 = time.perf_counter()
            r = O.run_sequence(wl.model, T, wl.n, wl.x0[0], wl.z[0][:T], mask, 1, 0, wl.opts.n_iter, wl.opts.step)
            dt = time.perf_counter() - t0
            row[key] = {"ms_per_step": dt / T * 1e3, "particle_iters_per_s": wl.n * wl.opts.n_iter * T / dt,
                        "J": r["J"]}
        row["bit_identical"] = row["single"]["J"] == row["all_core"]["J"]
        rows.append(row)
        print(json.dumps(row), flush=True)
    return {"cores": cores, "cpu_model": cpu_model(), "host_cpus": os.cpu_count(), "rows": rows}


def lattice_bandwidth(torch, smsq, n: int, batch: int, reps: int = 5):
    """Lattice-mode forward recursion on `batch` independent FP32 n x n lattices
    (larger together than the 256 MB last-level cache): edges/s and GB/s."""
    stream = torch.cuda.current_stream()
    gen = torch.Generator(device="cuda").manual_seed(0)
    AB = torch.randn((batch, n, n), generator=gen, device="cuda")
    A = [AB[b] for b in range(batch)]
    ell = torch.randn(n, device="cuda")
    phi_prev = torch.randn(n, device="cuda")
    ws = smsq.workspace()
    for a in A[:2]:
        smsq.viterbi_step(None, "f32", 2, phi_prev, lattice=a, loglik=ell, want_flags=False, ws=ws)
    torch.cuda.synchronize()
    ev0 = torch.cuda.Event(enable_timing=True)
    ev1 = torch.cuda.Event(enable_timing=True)
    ev0.record(stream)
    for _ in range(reps):
        for a in A:
            smsq.viterbi_step(None, "f32", 2, phi_prev, lattice=a, loglik=ell, want_flags=False, ws=ws)
    ev1.record(stream)
    torch.cuda.synchronize()
    sec = ev0.elapsed_time(ev1) / 1e3 / (reps * batch)
    nbytes = n * n * 4 + 3 * n * 4 + n * 4

    # Library references over the same lattices, for the bandwidth a single
    # launch of this size reaches: torch's row maximum (the same reads, no
    # argmax) and a device copy (the same reads plus as many writes).
    def lib_rate(fn, moved):
        for a in A[:2]:
            fn(a)
        torch.cuda.synchronize()
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        for _ in range(reps):
            for a in A:
                fn(a)
        e1.record(stream)
        torch.cuda.synchronize()
        return moved / (e0.elapsed_time(e1) / 1e3 / (reps * batch)) / 1e9

    dst = torch.empty_like(A[0])
    rowmax = lib_rate(lambda a: torch.amax(a, dim=1), n * n * 4 + n * 4)
    copy = lib_rate(lambda a: dst.copy_(a), 2 * n * n * 4)
    # all lattices in one launch (smsq_viterbi_lattice_batch), and a device
    # copy of the same 1 GiB in one call
    ellb = ell.expand(batch, n).contiguous()
    phib = phi_prev.expand(batch, n).contiguous()
    for _ in range(2):
        smsq.viterbi_lattice_batch("f32", phib, AB, ellb, want_flags=False, ws=ws)
    torch.cuda.synchronize()
    e0, e1 = _events(torch)
    e0.record(stream)
    for _ in range(reps):
        smsq.viterbi_lattice_batch("f32", phib, AB, ellb, want_flags=False, ws=ws)
    e1.record(stream)
    torch.cuda.synchronize()
    secb = e0.elapsed_time(e1) / 1e3 / reps
    dstb = torch.empty_like(AB)
    for _ in range(2):
        dstb.copy_(AB)
    torch.cuda.synchronize()
    e0.record(stream)
    for _ in range(reps):
        dstb.copy_(AB)
    e1.record(stream)
    torch.cuda.synchronize()
    copyb = 2 * AB.numel() * 4 / (e0.elapsed_time(e1) / 1e3 / reps) / 1e9
    del dstb
    return {"n": n, "lattices": batch, "edges_per_s": n * n / sec, "us_per_launch": sec * 1e6,
            "GBps": nbytes / sec / 1e9, "frac_hbm": nbytes / sec / PEAK_HBM,
            "bytes_per_launch": nbytes, "torch_rowmax_GBps": rowmax, "torch_copy_GBps": copy,
            "batched": {"us_per_launch": secb * 1e6, "GBps": batch * nbytes / secb / 1e9,
                        "frac_hbm": batch * nbytes / secb / PEAK_HBM, "edges_per_s": batch * n * n / secb,
                        "torch_copy_GBps_same_bytes": copyb}}


# Kernel / bandwidth / particle-count grid of the kernel ablation (Sec. V-E,
# Table VIII) on Scenario A: (kernel, bandwidth scale, N, weights),
# plus the mixture weights from the previous forward-recursion scores.
ABLATION_GRID = [("rbf", 1.0, 10, 0), ("imq", 1.0, 10, 0), ("matern32", 1.0, 10, 0),
                 ("rbf", 0.5, 10, 0), ("rbf", 3.0, 10, 0), ("rbf", 0.5, 40, 0), ("rbf", 3.0, 40, 0),
                 ("rbf", 1.0, 20, 0), ("rbf", 1.0, 40, 0), ("imq", 1.0, 20, 0), ("imq", 1.0, 40, 0),
                 ("matern32", 1.0, 20, 0), ("matern32", 1.0, 40, 0),
                 ("rbf", 1.0, 10, 1), ("rbf", 1.0, 40, 1)]


def mean_run_rmse(err, per_vector=False):
    """err [runs, T, d]: the RMSE of each run over its steps and coordinates
    (per_vector: the root mean squared Euclidean error of the vectors),
    averaged over the runs."""
    sq = np.sum(err ** 2, -1) if per_vector else np.mean(err ** 2, -1)
    return float(np.mean(np.sqrt(np.mean(sq, 1))))


def kernel_ablation(torch, smsq, mc: int):
    """The ablation grid on the paper's Scenario A model (Sec. V-A constants,
    FP64, T = 100, L = 100, eps = 0.5), mc synthetic Monte-Carlo sequences
    per row in one batched run: RMSE of the MAP trajectory against the
    simulated truth, mean J, and the GPU rate."""
    from paper_2312_08684_amd import scenarios as S
    rows = []
    for kernel, bw, n, weights in ABLATION_GRID:
        wl = S.make_workload("scenario_a", B=mc, seed=3000, n=n)
        o = wl.opts
        model = smsq.Model(wl.model)
        x0 = torch.tensor(wl.x0, dtype=torch.float64, device="cuda")
        z = torch.tensor(wl.z, dtype=torch.float64, device="cuda")
        so = smsq.opts(o.n_iter, o.step, bw, kernel=kernel, weights=weights)
        smsq.run_batch(model, "f64", x0, z, None, n, so, 5)   # warm-up
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        xmap, J = smsq.run_batch(model, "f64", x0, z, None, n, so, 5)
        torch.cuda.synchronize()
        dt = time.perf_counter() - t0
        err = xmap.cpu().numpy()[:, 1:] - wl.truth[:, 1:]
        rows.append({"kernel": kernel, "bw_scale": bw, "N": n,
                     "weights": "exp(phi_prev)" if weights else "uniform", "rmse": mean_run_rmse(err),
                     "mean_J": float(J.mean().item()), "seconds": dt,
                     "particle_iters_per_s": mc * wl.T * n * o.n_iter / dt})
    return {"model": "scenario_a (Sec. V-A 1-D benchmark constants), FP64, T=100, L=100, eps=0.5",
            "sequences_per_row": mc, "rows": rows}


# Stein-MAP-Seq RMSE printed for the Sec. V-B pose scenario (10 runs of 630
# steps; per particle count).  Other simulator: context, not a target.
PAPER_SCENARIO_B_RMSE = {10: 0.1121, 20: 0.0971, 40: 0.0983}


def scenario_b_runs(torch, smsq, mc: int):
    """The Sec. V-B pose scenario (SE(2), one range-bearing measurement per
    step from an unknown landmark, outliers in the simulated data), FP32,
    T = 630, L = 100, eps = 1e-4, mc Monte-Carlo sequences per particle count
    in one batched run: RMSE of the MAP trajectory (all three coordinates,
    and position only) against the simulated truth and against the
    noise-free reference loop, mean J, wall time and rates."""
    from paper_2312_08684_amd import scenarios as S
    rows = []
    for n in (10, 20, 40):
        wl = S.make_workload("scenario_b", B=mc, seed=4000, n=n)
        o = wl.opts
        model = smsq.Model(wl.model)
        x0 = torch.tensor(wl.x0, dtype=torch.float32, device="cuda")
        z = torch.tensor(wl.z, dtype=torch.float32, device="cuda")
        so = smsq.opts_from(o)
        smsq.run_batch(model, "f32", x0, z, None, n, so, 6)   # warm-up
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        xmap, J = smsq.run_batch(model, "f32", x0, z, None, n, so, 6)
        torch.cuda.synchronize()
        dt = time.perf_counter() - t0
        xm = xmap.cpu().numpy().astype(np.float64)[:, 1:]
        err = xm - wl.truth[:, 1:]
        ref = S.se2_reference(wl.model, wl.T)[None, 1:]
        rows.append({"N": n, "rmse_state": mean_run_rmse(err),
                     "rmse_position": mean_run_rmse(err[..., :2], per_vector=True),
                     "rmse_state_vs_reference": mean_run_rmse(xm - ref),
                     "paper_rmse": PAPER_SCENARIO_B_RMSE[n],
                     "mean_J": float(J.mean().item()), "seconds": dt, "ms_per_time_step": dt / wl.T * 1e3,
                     "particle_iters_per_s": mc * wl.T * n * o.n_iter / dt})
    return {"model": "scenario_b (Sec. V-B SE(2) pose, unknown landmark association, outliers), FP32, "
                     "T=630, L=100, eps=1e-4", "sequences_per_row": mc, "rows": rows}


# Stein-MAP-Seq end-effector (m) and joint-angle (rad) RMSE printed for the
# Sec. V-D manipulator (20 runs; per particle count).  Context, not a target.
PAPER_SCENARIO_D_RMSE = {10: (0.4686, 0.1918), 20: (0.4624, 0.1843), 30: (0.3560, 0.1720)}


def scenario_d_runs(torch, smsq, mc: int):
    """The Sec. V-D 14-D manipulator (joint angles and velocities, end-effector
    observations), FP32 on the vector-ALU step kernel, T = 100, L = 100,
    eps = 2e-4, mc Monte-Carlo sequences per particle count in one batched
    run: end-effector and joint-angle RMSE of the MAP trajectory against the
    simulated truth, mean J, wall time and rates."""
    from paper_2312_08684_amd import scenarios as S
    rows = []
    for n in (10, 20, 30):
        wl = S.make_workload("scenario_d", B=mc, seed=5000, n=n)
        o, p = wl.opts, wl.model.params
        model = smsq.Model(wl.model)
        x0 = torch.tensor(wl.x0, dtype=torch.float32, device="cuda")
        z = torch.tensor(wl.z, dtype=torch.float32, device="cuda")
        so = smsq.opts_from(o)
        smsq.run_batch(model, "f32", x0, z, None, n, so, 7)   # warm-up
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        xmap, J = smsq.run_batch(model, "f32", x0, z, None, n, so, 7)
        torch.cuda.synchronize()
        dt = time.perf_counter() - t0
        xm = xmap.cpu().numpy().astype(np.float64)[:, 1:]
        fk = lambda q: S.dh_forward_kinematics(q, p[1:8], p[8:15], p[15:22])
        ee = np.array([[fk(v[:7]) for v in run] for run in xm])
        ee_true = np.array([[fk(v[:7]) for v in run] for run in wl.truth[:, 1:]])
        pe, pq = PAPER_SCENARIO_D_RMSE[n]
        rows.append({"N": n, "rmse_end_effector": mean_run_rmse(ee - ee_true, per_vector=True),
                     "rmse_joint_angles": mean_run_rmse(xm[..., :7] - wl.truth[:, 1:, :7]),
                     "paper_rmse_end_effector": pe, "paper_rmse_joint_angles": pq,
                     "mean_J": float(J.mean().item()), "seconds": dt, "ms_per_time_step": dt / wl.T * 1e3,
                     "particle_iters_per_s": mc * wl.T * n * o.n_iter / dt})
    return {"model": "scenario_d (Sec. V-D 7-DoF arm, joint angles and velocities, d=14), FP32, "
                     "T=100, L=100, eps=2e-4", "sequences_per_row": mc, "rows": rows}


# Per-step computation times the paper prints for the range-only scenario
# (Sec. V-C timing table, ms): PF-MAP-Seq by particle count, and
# Stein-MAP-Seq by particle count.  A laptop CPU; context, not a target.
PAPER_SCENARIO_C_MS = {"pf_map_seq": {1000: 58.94, 2000: 162.01, 4000: 505.32},
                       "stein_map_seq": {20: 10.82, 30: 13.60, 40: 16.44}}


def pf_map_seq(torch, smsq):
    """The PF-MAP-Seq forward recursion as a workload of the particle-mode
    kernel: bootstrap-PF particle sets of the range-only model (T = 200, one
    beacon visible in steps 80..120) at N = 1000, 2000, 4000, FP32.  Per N:
    the kernel's time per launch (HIP events around a captured graph of 50
    back-to-back launches of step 100, median of 5 replays), edges/s and the
    counted vector-ALU rate (N N_p (2d + 4) flops per launch); the whole
    recursion + backtrack wall time per step, run eagerly through the binding
    and replayed from a captured graph (one launch per step: each step writes
    its back-pointers into a row of the [T, N] array).  Beside it,
    Stein-MAP-Seq's own per-step time on one sequence at N = 20, 30, 40
    (L = 100, eps = 0.005)."""
    from paper_2312_08684_amd import scenarios as S
    wl = S.make_workload("range2d", B=1, seed=6000)
    T, d = wl.T, wl.model.d
    model = smsq.Model(wl.model)
    ws = smsq.workspace()
    z = torch.tensor(wl.z[0], dtype=torch.float32, device="cuda")
    zm = torch.tensor(wl.mask[0], dtype=torch.uint8, device="cuda")
    x0 = torch.tensor(wl.x0[0][None, :], dtype=torch.float32, device="cuda")
    rows = []

    for n in (1000, 2000, 4000):
        parts = torch.tensor(S.bootstrap_pf_particles(wl.model, wl.x0[0], wl.z[0], wl.mask[0], n, seed=10),
                             dtype=torch.float32, device="cuda")
        psi_all = torch.empty((T, n), dtype=torch.int32, device="cuda")
        phi_buf = [torch.empty(n, dtype=torch.float32, device="cuda") for _ in range(2)]
        phi0 = torch.zeros(1, dtype=torch.float32, device="cuda")

        def recursion():
            phi = phi0
            for t in range(1, T + 1):
                phi, _, _ = smsq.viterbi_step(model, "f32", t, phi, x_prev=x0 if t == 1 else parts[t - 2],
                                              z_t=z[t - 1], z_mask=zm[t - 1], x=parts[t - 1],
                                              want_flags=False, ws=ws, phi_out=phi_buf[t % 2],
                                              psi_out=psi_all[t - 1])
            return smsq.backtrack("f32", psi_all, phi, ws=ws)

        recursion()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        _, J, _ = recursion()
        torch.cuda.synchronize()
        wall = time.perf_counter() - t0
        J_eager = float(J.item())
        # the T + 1 launches replayed (wall per step = the kernels' time); the
        # replayed J must equal the eager one
        ms_graph, (_, Jg, _) = _graph_ms(torch, recursion, T)
        graph_ok = float(Jg.item()) == J_eager
        # kernel alone: step T / 2 launched back to back from a graph
        tm = T // 2
        ph = torch.zeros(n, dtype=torch.float32, device="cuda")
        psi_k = torch.empty(n, dtype=torch.int32, device="cuda")
        phi_k = torch.empty(n, dtype=torch.float32, device="cuda")
        reps = 50

        def steps():
            for _ in range(reps):
                smsq.viterbi_step(model, "f32", tm, ph, x_prev=parts[tm - 2], z_t=z[tm - 1], z_mask=zm[tm - 1],
                                  x=parts[tm - 1], want_flags=False, ws=ws, phi_out=phi_k, psi_out=psi_k)

        ms_kernel, _ = _graph_ms(torch, steps, reps)
        us = ms_kernel * 1e3
        edges = n * n
        rows.append({"N": n, "kernel_us_per_step": us, "edges_per_s": edges / (us * 1e-6),
                     "counted_tflops": edges * (2 * d + 4) / (us * 1e-6) / 1e12,
                     "frac_fp32_peak": edges * (2 * d + 4) / (us * 1e-6) / PEAK_FP32,
                     "wall_ms_per_step": wall / T * 1e3, "graph_wall_ms_per_step": ms_graph,
                     "graph_replays_match_eager": graph_ok, "J": J_eager,
                     "paper_ms_per_step": PAPER_SCENARIO_C_MS["pf_map_seq"][n]})
    assert smsq.device_status(ws) == smsq.OK
    stein = []
    for n in (20, 30, 40):
        w2 = S.make_workload("range2d", B=1, seed=6000, n=n, n_iter=100, step=0.005)
        m2 = smsq.Model(w2.model)
        x0s = torch.tensor(w2.x0[0], dtype=torch.float32, device="cuda")
        zs = torch.tensor(w2.z[0], dtype=torch.float32, device="cuda")
        ms = torch.tensor(w2.mask[0], dtype=torch.uint8, device="cuda")
        so = smsq.opts_from(w2.opts)
        smsq.run_sequence(m2, "f32", x0s, zs, ms, n, so, 3)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        smsq.run_sequence(m2, "f32", x0s, zs, ms, n, so, 3)
        torch.cuda.synchronize()
        stein.append({"N": n, "ms_per_step": (time.perf_counter() - t0) / w2.T * 1e3,
                      "paper_ms_per_step": PAPER_SCENARIO_C_MS["stein_map_seq"][n]})
    return {"model": "range2d (stand-in for Sec. V-C), FP32, T=200; PF particle sets from a bootstrap PF "
                     "with stratified resampling", "kernel": "k_viterbi_particle_rows", "rows": rows,
            "stein_map_seq_one_sequence": stein}


def _events(torch):
    return torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)


def _graph_ms(torch, run, reps):
    """run() (reps launches) captured once in a hipGraph after a warm-up on a
    side stream, replayed 5 times: the median wall time per launch in ms from
    HIP events around each replay, and run()'s return value."""
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        run()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = run()
    times = []
    for _ in range(5):
        e0, e1 = _events(torch)
        e0.record()
        graph.replay()
        e1.record()
        torch.cuda.synchronize()
        times.append(e0.elapsed_time(e1) / reps)
    del graph
    return sorted(times)[2], out


def sweep(torch, smsq):
    """Sweeps of the measurement plan: the arm7 SVGD step against the batch
    size, the forward recursion against N (lattice mode FP32 / FP64, particle
    mode), and Algorithm 2 end to end per workload at one sequence and at a
    Monte-Carlo batch."""
    from paper_2312_08684_amd import scenarios as S
    out = {}
    # (1) teacher-forced arm7 step t = 2, N = N_p = 1024, L = 100, HIP events
    rows = []
    for B in (1, 8, 32, 128, 256, 1024):
        wl = S.make_workload("arm7", B=B, seed=0, T=2)
        o, d, n = wl.opts, wl.model.d, wl.n
        model = smsq.Model(wl.model)
        rng = np.random.default_rng(0)
        xp = torch.tensor(wl.truth[:, 1][:, None, :] + 0.02 * rng.normal(size=(B, n, d)), dtype=torch.float32,
                          device="cuda")
        x = torch.empty((B, n, d), dtype=torch.float32, device="cuda")
        z = torch.tensor(wl.z[:, 1], dtype=torch.float32, device="cuda")
        php = torch.zeros((B, n), dtype=torch.float32, device="cuda")
        ws = smsq.workspace()
        so = smsq.opts_from(o)
        stream = torch.cuda.current_stream()
        for _ in range(3):
            smsq.batch_step(model, "f32", 2, xp, php, z, None, x, so, seed=1, ws=ws)
        reps = 10 if B <= 256 else 4
        e0, e1 = _events(torch)
        e0.record(stream)
        for _ in range(reps):
            smsq.batch_step(model, "f32", 2, xp, php, z, None, x, so, seed=1, ws=ws)
        e1.record(stream)
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / reps
        fl = B * o.n_iter * flops_per_iteration(n, n, d, "arm7")
        rows.append({"B": B, "ms_per_launch": ms, "tflops": fl / ms / 1e9, "frac": fl / (ms / 1e3) / PEAK_FP32,
                     "particle_iters_per_s": B * n * o.n_iter / (ms / 1e3)})
    out["svgd_step_arm7_vs_batch"] = rows
    # (2) forward recursion against N
    rows = []
    gen = torch.Generator(device="cuda").manual_seed(0)
    for dt, tdt in (("f32", torch.float32), ("f64", torch.float64)):
        for n in (32, 256, 512, 1024, 4096):
            es = 4 if dt == "f32" else 8
            # distinct lattices, up to 1 GiB together (above the 256 MB last-level cache at N = 4096)
            nlat = max(1, min(16, (1 << 30) // (n * n * es)))
            As = [torch.randn((n, n), generator=gen, device="cuda", dtype=tdt) for _ in range(nlat)]
            ell = torch.randn(n, generator=gen, device="cuda", dtype=tdt)
            php = torch.randn(n, generator=gen, device="cuda", dtype=tdt)
            ws = smsq.workspace()
            reps = 48
            phi_k = torch.empty(n, dtype=tdt, device="cuda")
            psi_k = torch.empty(n, dtype=torch.int32, device="cuda")

            def lattices():
                for r in range(reps):
                    smsq.viterbi_step(None, dt, 2, php, lattice=As[r % nlat], loglik=ell, want_flags=False, ws=ws,
                                      phi_out=phi_k, psi_out=psi_k)

            sec = _graph_ms(torch, lattices, reps)[0] / 1e3
            nbytes = n * n * es + 3 * n * es + 4 * n
            del As
            rows.append({"mode": "lattice", "dtype": dt, "N": n, "us_per_launch": sec * 1e6,
                         "edges_per_s": n * n / sec, "GBps": nbytes / sec / 1e9, "frac_hbm": nbytes / sec / PEAK_HBM})
    for (name, n), (dt, tdt) in itertools.product((("range2d", 256), ("cv4d", 512), ("arm7", 1024), ("range2d", 4096)),
                                                 (("f32", torch.float32), ("f64", torch.float64))):
        wl = S.make_workload(name, B=1, seed=0, T=2, n=n)
        model = smsq.Model(wl.model)
        d = wl.model.d
        rng = np.random.default_rng(1)
        xp = torch.tensor(wl.truth[0, 1] + 0.02 * rng.normal(size=(n, d)), dtype=tdt, device="cuda")
        x = torch.tensor(wl.truth[0, 2] + 0.02 * rng.normal(size=(n, d)), dtype=tdt, device="cuda")
        z = torch.tensor(wl.z[0, 1], dtype=tdt, device="cuda")
        mk = torch.tensor(wl.mask[0, 1], dtype=torch.uint8, device="cuda") if wl.mask is not None else None
        php = torch.zeros(n, dtype=tdt, device="cuda")
        ws = smsq.workspace()
        reps = 50
        phi_k = torch.empty(n, dtype=tdt, device="cuda")
        psi_k = torch.empty(n, dtype=torch.int32, device="cuda")

        def particles():
            for _ in range(reps):
                smsq.viterbi_step(model, dt, 2, php, x_prev=xp, z_t=z, z_mask=mk, x=x, want_flags=False, ws=ws,
                                  phi_out=phi_k, psi_out=psi_k)

        sec = _graph_ms(torch, particles, reps)[0] / 1e3
        rows.append({"mode": "particle (one sequence, rows over the chip)", "model": name, "dtype": dt, "N": n,
                     "us_per_launch": sec * 1e6, "edges_per_s": n * n / sec})
    out["viterbi_vs_n"] = rows
    # (3) Algorithm 2 end to end per workload: one sequence and a batch
    rows = []
    for name, batches in (("growth1d", (1, 50, 256)), ("range2d", (1, 20, 256)), ("cv4d", (1, 20, 256)),
                          ("arm7", (1, 20, 256))):
        for B in batches:
            T = 20 if name == "arm7" and B == 256 else None
            wl = S.make_workload(name, B=B, seed=7, T=T)
            o, dt = wl.opts, wl.dtype
            td = smsq.torch_dtype(dt)
            model = smsq.Model(wl.model)
            x0 = torch.tensor(wl.x0, dtype=td, device="cuda")
            z = torch.tensor(wl.z, dtype=td, device="cuda")
            mk = torch.tensor(wl.mask, dtype=torch.uint8, device="cuda") if wl.mask is not None else None
            so = smsq.opts_from(o)
            smsq.run_batch(model, dt, x0, z, mk, wl.n, so, 3)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            smsq.run_batch(model, dt, x0, z, mk, wl.n, so, 3)
            torch.cuda.synchronize()
            sec = time.perf_counter() - t0
            rows.append({"workload": name, "dtype": dt, "B": B, "N": wl.n, "T": wl.T, "L": o.n_iter,
                         "seconds": sec, "sequences_per_s": B / sec,
                         "particle_iters_per_s": B * wl.T * wl.n * o.n_iter / sec,
                         "edges_per_s": B * (wl.n + (wl.T - 1) * wl.n * wl.n) / sec})
    out["run_batch_per_workload"] = rows
    return out


def batched_mix(torch, smsq, count: int, train_steps: int, train_seqs: int, train_L: float = 2.0):
    """Ragged mix (family uniform over the four, N from {32..1024}, T in
    [50, 200]) as one batched plan per run, hipGraph replay, autotuned.  The
    plain method at the full iteration count gives the reference J of every
    sequence; the plain method and the learned initialisation then run at
    1/4, 1/2, 3/4 (and the learned one at all) of the iterations, and each
    sequence's L' is the smallest fraction whose J matches the reference."""
    from paper_2312_08684_amd import learned as LI
    from paper_2312_08684_amd import scenarios as S
    spec = LI.mix(count, seed=11, T_lo=50, T_hi=200)
    mx = LI.Mix(spec)
    pi = sum(n * T * S.PRESETS[f][2] for (f, n, T, _) in spec)   # particle-iterations at full L
    dims = {"growth1d": 1, "range2d": 2, "cv4d": 4, "arm7": 7}
    flops_full = sum(S.PRESETS[f][2] * (flops_per_iteration(n, 1, dims[f], f) +
                                        (T - 1) * flops_per_iteration(n, n, dims[f], f)) for (f, n, T, _) in spec)
    plan, Jfull, t_full, _, _ = LI.run(mx, 1.0, tune=True)
    print("batched: plain at L, %.2f s" % t_full, file=sys.stderr, flush=True)
    info = plan.info()
    del plan
    fracs = (0.25, 0.5, 0.75)
    plain = {1.0: (Jfull, t_full)}
    for f in fracs:
        _, J, t, _, _ = LI.run(mx, f, warm=False)
        plain[f] = (J, t)
        print("batched: plain at %g L, %.2f s" % (f, t), file=sys.stderr, flush=True)
    # the converged reference: the plain method at twice the iterations
    _, J2, t2, _, _ = LI.run(mx, 2.0, warm=False)
    plain[2.0] = (J2, t2)
    # proposal: trained on plain runs of a separate, shorter mix; gated per
    # family on a validation mix
    t0 = time.perf_counter()
    tspec = LI.mix(train_seqs, seed=1, T_lo=20, T_hi=40)
    tplan, _, _, tmodels, tseqs = LI.run(tspec, train_L, warm=False)
    ex = LI.examples(tplan, tspec, tseqs)
    n_examples = len(ex)
    mlp = smsq.InitMLP(seed=5, max_batch=max(4096, count))
    losses = LI.train(mlp, tmodels, ex, steps=train_steps, batch=512, lr=1e-3, log_every=train_steps // 4)
    print("batched: proposal trained, NLL %.3f" % losses[-1], file=sys.stderr, flush=True)
    del tplan, ex
    gain = LI.choose_gate(mlp, LI.mix(64, seed=3, T_lo=50, T_hi=200), 0.5)
    gate = {f: g["use"] for f, g in gain.items()}
    t_train = time.perf_counter() - t0
    learned = {}
    for f in fracs + (1.0,):
        _, J, t, _, _ = LI.run(mx, f, mlp=mlp, gate=gate, warm=False)
        learned[f] = (J, t)
        print("batched: learned at %g L, %.2f s" % (f, t), file=sys.stderr, flush=True)
    Lp = LI.iterations_to_match({f: v[0] for f, v in plain.items() if f <= 1.0}, Jfull, spec)
    Ll = LI.iterations_to_match({f: v[0] for f, v in learned.items()}, Jfull, spec)
    # against the converged reference (plain at 2 L); a sequence that no run
    # of up to L matches counts at 2 (the reference's own budget)
    Lp2 = LI.iterations_to_match({f: v[0] for f, v in plain.items()}, J2, spec)
    Ll2 = LI.iterations_to_match({f: v[0] for f, v in learned.items()}, J2, spec)
    fam = np.array([sp[0] for sp in spec])

    def row(J, t, frac_L):
        per = {}
        for f in LI.FAMILIES:
            idx = np.flatnonzero(fam == f)
            per[f] = {"matched_frac": float(np.mean(LI.matched(J[idx], Jfull[idx], [spec[i] for i in idx]))),
                      "mean_J_gap": float(np.mean(J[idx] - Jfull[idx]))}
        return {"seconds": t, "sequences_per_s": count / t, "particle_iters_per_s": pi * frac_L / t,
                "matched_frac": float(np.mean(LI.matched(J, Jfull, spec))), "mean_J_gap": float(np.mean(J - Jfull)),
                "per_family": per}

    def lprime(Lx, cap=None):
        ok = ~np.isnan(Lx)
        full = np.where(ok, Lx, cap) if cap is not None else Lx
        per = {f: {"mean": float(np.mean(Lx[(fam == f) & ok])) if np.any((fam == f) & ok) else None,
                   "reached": float(np.mean(ok[fam == f])),
                   "mean_all": float(np.mean(full[fam == f])) if cap is not None else None} for f in LI.FAMILIES}
        return {"mean": float(np.mean(Lx[ok])), "reached": float(np.mean(ok)),
                "mean_all": float(np.mean(full)) if cap is not None else None, "per_family": per}

    def vs_ref(J, Jr):
        per = {f: {"matched_frac": float(np.mean(LI.matched(J[fam == f], Jr[fam == f],
                                                             [spec[i] for i in np.flatnonzero(fam == f)]))),
                   "mean_J_gap": float(np.mean(J[fam == f] - Jr[fam == f]))} for f in LI.FAMILIES}
        return {"matched_frac": float(np.mean(LI.matched(J, Jr, spec))), "mean_J_gap": float(np.mean(J - Jr)),
                "per_family": per}

    return {"sequences": count, "families": "growth1d range2d cv4d arm7", "N": "32..1024", "T": "50..200",
            "workgroup_waves": info["waves"], "tuned_ms_per_step": info["tuned_ms"],
            "plain": {str(f): row(J, t, f) for f, (J, t) in sorted(plain.items())},
            "learned": {str(f): row(J, t, f) for f, (J, t) in sorted(learned.items())},
            "iterations_to_match": {"fractions": [0.25, 0.5, 0.75, 1.0], "plain": lprime(Lp), "learned": lprime(Ll)},
            "converged_reference": {
                "what": "plain method at 2 L (every family); L' of a sequence no run up to L matches counts as 2",
                "plain_L_vs_2L": vs_ref(Jfull, J2), "learned_L_vs_2L": vs_ref(learned[1.0][0], J2),
                "reference_seconds": t2,
                "iterations_to_match": {"fractions": [0.25, 0.5, 0.75, 1.0, 2.0], "plain": lprime(Lp2, 2.0),
                                        "learned": lprime(Ll2, 2.0)}},
            "plain_full_roofline": {"counted_flops": flops_full, "tflops": flops_full / t_full / 1e12,
                                    "frac_fp32_peak": flops_full / t_full / PEAK_FP32,
                                    "note": "whole plan wall time (graph replay), one run at the full L"},
            "proposal": {"train_sequences": len(tspec), "train_T": "20..40", "train_examples": n_examples,
                         "train_steps": train_steps, "train_L": train_L, "train_nll": losses,
                         "gate_per_family": gain,
                         "setup_seconds": t_train},
            "match_rule": "J >= J_plain_full - 1e-3 max(|J_plain_full|, T)"}


def latency(torch, smsq):
    """Algorithm 2 per-step time for small batches of the 7-DOF arm (N = 1024,
    L = 100) and the clutter model (N = 512, L = 50): one workgroup per
    sequence against the multi-workgroup steps the drivers choose."""
    from paper_2312_08684_amd import scenarios as S
    rows = []
    for name, B, T in (("arm7", 1, 10), ("arm7", 8, 10), ("arm7", 32, 10), ("cv4d", 1, 20), ("cv4d", 32, 20)):
        wl = S.make_workload(name, B=B, seed=3, T=T)
        model = smsq.Model(wl.model)
        x0 = torch.tensor(wl.x0, dtype=torch.float32, device="cuda")
        z = torch.tensor(wl.z, dtype=torch.float32, device="cuda")
        mk = torch.tensor(wl.mask, dtype=torch.uint8, device="cuda") if wl.mask is not None else None
        row = {"workload": name, "B": B, "N": wl.n, "L": wl.opts.n_iter, "T": T}
        for sk, key in (("mfma", "one_workgroup_ms_per_step"), ("auto", "ms_per_step")):
            o = smsq.opts_from(wl.opts, step_kernel=sk)
            ws = smsq.workspace(model.workspace_size("f32", B, T, wl.n))
            smsq.run_batch(model, "f32", x0, z, mk, wl.n, o, 3, ws=ws)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            smsq.run_batch(model, "f32", x0, z, mk, wl.n, o, 3, ws=ws)
            torch.cuda.synchronize()
            row[key] = (time.perf_counter() - t0) / T * 1e3
            assert smsq.device_status(ws) == smsq.OK
        rows.append(row)
    return rows


def main():
    args = parse()
    if args.cpu_table:
        print(json.dumps(cpu_table()), flush=True)
        return
    if args.gpus != 1:
        print("bench.py runs on one GPU only: this build has no multi-GPU path "
              "(sequences shard across GPUs with no exchange; see the design notes)", file=sys.stderr)
        sys.exit(2)
    import torch
    from paper_2312_08684_amd import scenarios as S
    from paper_2312_08684_amd import smsq

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    smsq.load()
    if args.sweep:
        print(json.dumps(sweep(torch, smsq)), flush=True)
        return
    if args.copy_probe_mib > 0:
        nbytes = args.copy_probe_mib << 20
        src = torch.ones(nbytes // 4, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        print("copy probe: %d bytes read and written, 3 copies" % nbytes, file=sys.stderr, flush=True)
        del src, dst
    name = args.workload
    wl = S.make_workload(name, B=args.batch, seed=0, T=args.T)
    desc, o = wl.model, wl.opts
    B, T, n, d, L = wl.batch, wl.T, wl.n, desc.d, o.n_iter
    dt = wl.dtype
    td = smsq.torch_dtype(dt)
    model = smsq.Model(desc)
    x0 = torch.tensor(wl.x0, dtype=td, device="cuda")
    z = torch.tensor(wl.z, dtype=td, device="cuda")
    mask = torch.tensor(wl.mask, dtype=torch.uint8, device="cuda") if wl.mask is not None else None
    parts = torch.empty((B, T, n, d), dtype=td, device="cuda")
    psi = torch.empty((B, T, n), dtype=torch.int32, device="cuda")
    phis = torch.empty((B, T, n), dtype=td, device="cuda")
    ws = smsq.workspace()
    so = smsq.opts_from(o)
    stream = torch.cuda.current_stream()
    x0v = x0.view(B, 1, d)

    def one_pass(events=None):
        for t in range(1, T + 1):
            xp = x0v if t == 1 else parts[:, t - 2]
            php = None if t == 1 else phis[:, t - 2]
            if events is not None:
                events[t - 1][0].record(stream)
            smsq.batch_step(model, dt, t, xp, php, z[:, t - 1], None if mask is None else mask[:, t - 1],
                            parts[:, t - 1], so, seed=1, phi=phis[:, t - 1], psi=psi[:, t - 1], ws=ws)
            if events is not None:
                events[t - 1][1].record(stream)
        return smsq.backtrack(dt, psi, phis[:, T - 1].contiguous(), parts, x0, ws=ws)

    for _ in range(args.warmup):
        one_pass()
    torch.cuda.synchronize()
    assert smsq.device_status(ws) == smsq.OK, "non-finite values in warm-up"

    events = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(T)]
    step_ms = []
    kernel_ms = []
    for _ in range(args.steps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        one_pass(events)
        torch.cuda.synchronize()
        step_ms.append((time.perf_counter() - t0) * 1e3)
        kernel_ms.append([e0.elapsed_time(e1) for e0, e1 in events])
    ms = float(np.mean(step_ms))
    particle_iters = B * T * n * L
    edges = B * (n * 1 + (T - 1) * n * n)
    flops_total = B * L * (flops_per_iteration(n, 1, d, name) + (T - 1) * flops_per_iteration(n, n, d, name))
    kern = np.array(kernel_ms)                     # [steps, T] ms per launch
    if T >= 2:
        k_avg_ms = float(kern[:, 1:].mean())       # steady-state launches (n_prev = n)
        flops_launch = B * L * flops_per_iteration(n, n, d, name)
        launch_kind = "steady-state launch"
    else:
        k_avg_ms = float(kern[:, 0].mean())        # the only launch: one previous particle
        flops_launch = B * L * flops_per_iteration(n, 1, d, name)
        launch_kind = "first launch (one previous particle)"
    counted = flops_launch / (k_avg_ms / 1e3)
    # FP32 operands run as split 16-bit ones: the matrix-core kernel is priced
    # by what it executes there, the others by the method's counted work
    matrix = dt == "f32" and n > 64 and d <= 7
    executed = B * L * executed_matrix_flops(n, n if T >= 2 else 1, d) if matrix else flops_launch
    achieved = executed / (k_avg_ms / 1e3)
    peak = PEAK_FP64 if dt == "f64" else PEAK_BF16 if matrix else PEAK_FP32
    lat = lattice_bandwidth(torch, smsq, args.lattice_n, args.lattice_batch)
    out = {
        "metric": "SVGD particle-iters/s",
        "value": particle_iters / (ms / 1e3),
        "unit": "particle-iters/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": dt,
        "data": "synthetic",
        "config": {"workload": "%s N=%d d=%d L=%d T=%d eps=%g, batch of %d sequences" % (
            name, n, d, L, T, o.step, B), "batch": B, "N": n, "d": d, "L": L, "T": T},
        "viterbi_edges_per_s": edges / (ms / 1e3),
        "sequences_per_s": B / (ms / 1e3),
        "counted_tflops": flops_total / (ms / 1e3) / 1e12,
        "roofline": {"bound": "mfma", "achieved": achieved / 1e12, "peak": peak / 1e12, "unit": "TFLOP/s",
                     "frac": achieved / peak, "traffic": measured_traffic(name, B, n, dt) if T >= 2 else None,
                     "kernel": ("k_step_mfma (fused SVGD iterations + forward recursion, FP32 operands split over the "
                                "16-bit matrix units)" if matrix else
                                "vector-ALU step (fused SVGD iterations + forward recursion)")
                     + ", " + launch_kind,
                     "kernel_avg_ms": k_avg_ms, "flops_per_launch": executed,
                     "counted_flops_per_launch": flops_launch, "counted_tflops": counted / 1e12},
        "viterbi_lattice": lat,
        "device": device_info(torch),
    }
    if args.ablation_mc > 0:
        out["kernel_ablation"] = kernel_ablation(torch, smsq, args.ablation_mc)
    if args.scenario_b_mc > 0:
        out["scenario_b"] = scenario_b_runs(torch, smsq, args.scenario_b_mc)
    if args.scenario_d_mc > 0:
        out["scenario_d"] = scenario_d_runs(torch, smsq, args.scenario_d_mc)
    if args.pf_map_seq:
        out["pf_map_seq"] = pf_map_seq(torch, smsq)
    if args.latency:
        out["latency"] = latency(torch, smsq)
    if args.batched_seqs > 0:
        out["batched"] = batched_mix(torch, smsq, args.batched_seqs, args.train_steps, args.train_seqs, args.train_L)
    if args.cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(name)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
