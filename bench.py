#!/usr/bin/env python3
"""Benchmark of the N-shaped partition Crank-Nicolson path on one MI355X.

Headline workload (one "step" = one pass of the whole hot path): the Lie-split ADI step of a
4096 x 4096 TDSE grid (dx = dy = 0.1, dt = 0.01, soft-core 2D potential, seeded random psi0):
an x-sweep over 4096 contiguous lines of 4096 unknowns, then a y-sweep over 4096 interleaved
lines, each a full CN step (explicit half-step fused into the N-shaped solve).  Every step is
one captured hipGraph.  value = solved complex unknowns per second (2 x 4096^2 per step).

Also reported (extra): the 2^28-unknown explicit solve with its partition sweep, the plain 1D
workload (N = 65536, one solve + 200 steps), the uneven batch (10^4 systems, 50 steps) and the
differentiated propagation (2^20 x 2000 steps), a 2^24-row propagation with a field (20
steps, one fused pass per step) and one 2^22-row matrix with 16 right-hand sides, each with the
oracle timed beside it.

Usage: python bench.py [--gpus 1] [--steps K] [--warmup W] [--no-extra] [--cpu-seconds S]
                       [--copy-ref] [--only-large] [--only-propagate] [--only-absorbing]
  --cpu-seconds 0 skips the oracle's full 100-step run of the headline grid (about 15 s on 16
  threads; the baseline and parity then use one step); --only-large times only the 2^28 solve,
  --only-propagate only the 2^24-row fused propagation, --only-absorbing only the 2^24-row
  steps with an absorbing potential.
"""
from __future__ import annotations

import argparse
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0  # MI355X HBM3E, published
BYTES_PER_UNKNOWN_STEP = 40  # CN step: read psi (16) + V (8), write psi (16)
BYTES_PER_UNKNOWN_SOLVE_2PASS = 144  # general solve out of core: 64 + 64 + 16
BYTES_PER_UNKNOWN_SOLVE_MIN = 80  # read a, b, c, d, write x


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def parse():
    p = argparse.ArgumentParser()
    p.add_argument("--gpus", type=int, default=1)
    p.add_argument("--steps", type=int, default=100)
    p.add_argument("--warmup", type=int, default=5)
    p.add_argument("--no-extra", action="store_true")
    p.add_argument("--cpu-seconds", type=float, default=10.0)
    p.add_argument("--only-large", action="store_true",
                   help="time only the 2^28 explicit solve (automatic plan), for profiling")
    p.add_argument("--only-propagate", action="store_true",
                   help="time only the 2^24-row fused propagation, for profiling")
    p.add_argument("--only-absorbing", action="store_true",
                   help="time only the 2^24-row steps with an absorbing potential, for profiling")
    p.add_argument("--only-uneven", action="store_true",
                   help="time only the uneven batch (steps and a propagation), for profiling")
    p.add_argument("--only-multi-rhs", action="store_true",
                   help="time only the 2^22 x 16 shared-matrix solve, for profiling")
    p.add_argument("--only-radial", action="store_true",
                   help="time only the partial-wave steps, for profiling")
    p.add_argument("--only-latency", action="store_true",
                   help="only the step times of the latency-bound sequences (plain 1D, 200 steps "
                        "in a graph; the differentiated workload's forward and reverse mode), "
                        "without oracle or finite differences (for profiling)")
    p.add_argument("--copy-ref", action="store_true",
                   help="first run a plain 256 MiB device copy three times (a reference of known "
                        "size for scaling hardware byte counters)")
    return p.parse_args()


def timed_events(torch, fn, reps):
    """Run fn reps times, HIP events around each call on the current stream; ms per call."""
    evs = [torch.cuda.Event(enable_timing=True) for _ in range(reps + 1)]
    torch.cuda.synchronize()
    evs[0].record()
    for i in range(reps):
        fn()
        evs[i + 1].record()
    evs[-1].synchronize()
    return [evs[i].elapsed_time(evs[i + 1]) for i in range(reps)]


def source_fingerprint():
    import glob
    import hashlib

    h = hashlib.sha256()
    for p in sorted(glob.glob(os.path.join(ROOT, "paper_2205_00856_amd", "csrc", "*"))):
        with open(p, "rb") as f:
            h.update(f.read())
    return h.hexdigest()[:16]


def measured_traffic(profile_name):
    """HBM bytes per launch from the committed counter summary, or None when the kernel
    sources have changed since the counters were taken."""
    import re

    path = os.path.join(ROOT, "profiles", profile_name)
    try:
        text = open(path).read()
    except OSError:
        return None
    m = re.search(r"traffic_bytes_per_launch: (\d+) sources: ([0-9a-f]+)", text)
    if not m or m.group(2) != source_fingerprint():
        return None
    return float(m.group(1))


def rel_l2(x, y):
    import numpy as np

    return float(np.linalg.norm(x - y) / np.linalg.norm(y))


def cpu_threads():
    n = os.cpu_count() or 1
    env = os.environ.get("OMP_NUM_THREADS")
    if env and env.isdigit():
        n = min(n, int(env))
    return max(1, min(n, 16))


def main():
    args = parse()
    if args.gpus != 1:
        print(f"bench.py runs on exactly one GPU (the method's single-device path); "
              f"--gpus {args.gpus} is not supported", file=sys.stderr)
        sys.exit(2)
    import numpy as np
    import torch

    import paper_2205_00856_amd as cn
    import workloads

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    dev = torch.device("cuda", 0)
    torch.cuda.set_device(dev)

    if args.copy_ref:
        src = torch.ones(1 << 24, dtype=torch.complex128, device=dev)
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst

    if args.only_large:
        print(json.dumps(large_system(torch, np, cn, dev, sweep=False, oracle_parity=False)),
              flush=True)
        return
    if args.only_propagate:
        print(json.dumps(long_propagate(torch, np, cn, dev, parity=False)), flush=True)
        return
    if args.only_absorbing:
        print(json.dumps(absorbing_large(torch, np, cn, workloads, dev)), flush=True)
        return
    if args.only_uneven:
        print(json.dumps(uneven_timing(torch, np, cn, workloads, dev)), flush=True)
        return
    if args.only_multi_rhs:
        print(json.dumps(multi_rhs(torch, np, cn, dev, oracle=False)), flush=True)
        return
    if args.only_radial:
        print(json.dumps(radial(torch, np, cn, workloads, dev, parity=False)), flush=True)
        return
    if args.only_latency:
        print(json.dumps(latency_legs(torch, np, cn, workloads, dev)), flush=True)
        return

    # ---------------------------------------------------------------- headline: ADI 4096^2
    w = workloads.adi_2d()
    ny, nx = w["psi0"].shape
    psi0 = torch.from_numpy(w["psi0"].ravel()).to(dev)
    V = torch.from_numpy(w["V"].ravel()).to(dev)
    psi = psi0.clone()
    Lx = cn.Layout.contiguous(nx, ny)
    Ly = cn.Layout.interleaved(ny, nx)
    cn.reserve(Lx)
    cn.reserve(Ly)

    def adi_step():
        cn.step(psi, V, w["dx"], w["dt"], v_scale=0.5, out=psi, layout=Lx)
        cn.step(psi, V, w["dy"], w["dt"], v_scale=0.5, out=psi, layout=Ly)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        adi_step()  # plans and workspace exist before capture
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        adi_step()
    # parity against the oracle: one captured step, and the workload's full run of w["steps"]
    # replays from psi0 (the oracle's timed run of the same steps is the cpu_baseline)
    psi.copy_(psi0)
    graph.replay()
    torch.cuda.synchronize()
    one = psi.cpu().numpy().reshape(ny, nx)
    psi.copy_(psi0)
    for _ in range(w["steps"]):
        graph.replay()
    torch.cuda.synchronize()
    full = psi.cpu().numpy().reshape(ny, nx)
    norm_full = float(np.sum(np.abs(full) ** 2) * w["dx"] * w["dy"])
    parity = parity_full = None
    cpu_baseline = None
    nthr = cpu_threads()
    try:
        import oracle

        t0 = time.perf_counter()
        state = oracle.adi_step(w["psi0"], w["V"], w["dx"], w["dy"], w["dt"], nthr)
        t_cpu = time.perf_counter() - t0
        parity = rel_l2(one, state)
        nsteps_cpu = 1
        if args.cpu_seconds > 0:
            # the whole run (100 steps of the 4096^2 grid, about 15 s on 16 threads)
            t0 = time.perf_counter()
            for _ in range(w["steps"] - 1):
                state = oracle.adi_step(state, w["V"], w["dx"], w["dy"], w["dt"], nthr)
            t_cpu += time.perf_counter() - t0
            nsteps_cpu = w["steps"]
            parity_full = rel_l2(full, state)
        cpu_baseline = {
            "value": 2 * nx * ny * nsteps_cpu / max(t_cpu, 1e-9),
            "unit": "complex unknowns/s",
            "cores": nthr,
            "kind": "oracle",
            "sample": f"{nsteps_cpu} full ADI steps of the 4096x4096 grid from psi0 (serial FP64 "
                      f"Thomas per line, lines spread over {nthr} threads), {t_cpu:.1f} s",
        }
    except Exception as ex:  # noqa: BLE001 - the baseline leg must not hide the GPU result
        log("cpu baseline / parity leg failed:", repr(ex))

    psi.copy_(psi0)
    for _ in range(args.warmup):
        graph.replay()
    per_step = timed_events(torch, graph.replay, args.steps)
    total_ms = float(np.sum(per_step))
    ms_step = total_ms / args.steps
    unknowns_per_step = 2 * nx * ny
    value = unknowns_per_step * args.steps / (total_ms * 1e-3)
    norm = float(torch.sum(torch.abs(psi) ** 2).item() * w["dx"] * w["dy"])
    # dominant kernel: the x-sweep (one launch of the fused CN-step tile kernel), timed with
    # events around each of its launches on the stream it runs on, over --steps ADI steps run
    # eagerly behind a backlog of graph replays: the host enqueues the events and launches while
    # the replays run, so no host launch gap falls inside a bracket, and each x-sweep sits
    # between two y-sweeps as in the graph (back to back the x-sweeps alone run into the power
    # limit).  The rocprofv3 kernel trace of the same command gives the same mean within a few
    # per cent.
    launch_src = "events around each eager x-sweep launch, behind a backlog of graph replays"
    stream = torch.cuda.current_stream()
    for _ in range(10):
        graph.replay()  # backlog: the host enqueues the eager launches while these run
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
          for _ in range(args.steps)]
    for e0, e1 in ev:
        e0.record(stream)
        cn.step(psi, V, w["dx"], w["dt"], v_scale=0.5, out=psi, layout=Lx)
        e1.record(stream)
        cn.step(psi, V, w["dy"], w["dt"], v_scale=0.5, out=psi, layout=Ly)
    torch.cuda.synchronize()
    x_ms = [e0.elapsed_time(e1) for e0, e1 in ev]
    launch_ms = float(np.mean(x_ms))
    algo_bytes = BYTES_PER_UNKNOWN_STEP * nx * ny
    achieved = algo_bytes / (launch_ms * 1e-3) / 1e9

    result = {
        "metric": "complex unknowns/s per CN step (ADI line solves)",
        "value": value,
        "unit": "complex unknowns/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "c128",
        "data": "synthetic",
        "config": {
            "workload": "adi_2d: 4096x4096 TDSE grid, Lie-split CN step = x-sweep (4096 "
                        "contiguous lines) + y-sweep (4096 interleaved lines), dx=dy=0.1, "
                        "dt=0.01, V/2 per sweep, one hipGraph per step",
            "unknowns_per_step": unknowns_per_step,
            "plan_x": cn.describe_plan(Lx, True),
            "plan_y": cn.describe_plan(Ly, True),
        },
        "effective_GBps": BYTES_PER_UNKNOWN_STEP * unknowns_per_step / (ms_step * 1e-3) / 1e9,
        "roofline": {
            "bound": "hbm",
            "achieved": achieved,
            "peak": HBM_PEAK_GBS,
            "unit": "GB/s",
            "frac": achieved / HBM_PEAK_GBS,
            "traffic": measured_traffic("adi_4096sq_steps_one_pass.md"),
            "kernel": "k_rowstep<M=8,W=8>: the x-sweep (N-shaped solve and step of 4096 "
                      "lines of 4096 in one pass)",
            "algorithmic_bytes_per_launch": algo_bytes,
            "launch_ms": launch_ms,
            "launch_ms_source": launch_src,
            "launch_ms_median": float(np.median(x_ms)),
        },
        "cpu_baseline": cpu_baseline,
        "parity_rel_l2_first_step": parity,
        "parity_rel_l2_after_steps": parity_full,
        "parity_steps": w["steps"],
        "norm_drift_after_steps": abs(norm_full - 1.0),
        "norm_after": norm,
    }

    ex = {}
    if not args.no_extra:
        ex = extras(torch, np, cn, workloads, dev)

        def get(leg, key):
            v = ex.get(leg, {})
            return v.get(key) if isinstance(v, dict) else None

        # relative L2 against the oracle of each workload's whole run, at its full size
        result["parity_full_size"] = {
            "plain_1d_solve": get("plain_1d", "parity_rel_l2_solve"),
            "plain_1d_psi_200": get("plain_1d", "parity_rel_l2_200"),
            "plain_1d_psi_200_resident": get("plain_1d", "parity_rel_l2_200_resident"),
            "adi_2d_psi_100": parity_full,
            "large_system_2^28_x": get("large_system_2^28", "parity_rel_l2"),
            "uneven_batch_psi_50": get("uneven_batch", "parity_rel_l2_50_steps"),
            "differentiated_psi_2000": get("differentiated", "parity_rel_l2_psi_T"),
            "differentiated_loss": get("differentiated", "parity_rel_loss"),
            "differentiated_fd_64": get("differentiated", "fd_rel_l2_64"),
        }
    emit(result, ex)


def emit(result, legs):
    """The other workloads' results on lines of their own, then the headline as one JSON line, short
    enough for a reader that keeps the end of the output."""
    for name, leg in legs.items():
        print(f"leg {name}: {json.dumps(leg)}", flush=True)
    print(json.dumps({**result, "legs": list(legs)}), flush=True)


def large_system(torch, np, cn, dev, sweep=True, oracle_parity=True):
    """The 2^28-unknown explicit solve on the seeded workload (workloads.large_system: V_j ~
    U(-1, 0) on dx = 0.01, dt = 0.02, then d complex normal; a, b, c assembled on the GPU),
    timed with the automatic plan and over the partition sweep; the oracle's serial Thomas solve
    of the same arrays gives the parity of the automatic plan's x and is the CPU baseline."""
    import workloads

    w = workloads.large_system()
    N = w["n"]
    sha = workloads.digest(w["V"], w["d"])
    V = torch.from_numpy(w["V"]).to(dev)
    a, b, c = cn.assemble(V, w["dx"], w["dt"])
    del V
    d = torch.from_numpy(w["d"]).to(dev)
    x = torch.empty_like(d)
    rows = []
    parts = (0, 64, 128, 256, 512, 1024, 2048, 4096, 8192, 16384) if sweep else (0,)
    x_auto = None
    for T in parts:
        # 64: one row per lane (every block a joint row); 8192 and 16384: chunked partitions
        # (their rows do not fit one workgroup's registers; the second pass reads each chunk
        # twice, 208 B per unknown instead of 144)
        M = 2 if T == 128 else (0 if T in (0, 64, 8192, 16384) else 4)
        L = cn.Layout.contiguous(N, 1, partition=T, rows_per_thread=M)
        cn.solve(a, b, c, d, out=x, layout=L)
        if T == 0:
            x_auto = x.cpu().numpy()
        ts = timed_events(torch, lambda: cn.solve(a, b, c, d, out=x, layout=L), 10)
        med = float(np.median(ts))
        rows.append({"partition": T, "rows_per_thread": M, "ms_median": med,
                     "ms_min": float(np.min(ts)),
                     "GBps_144": BYTES_PER_UNKNOWN_SOLVE_2PASS * N / (med * 1e-3) / 1e9,
                     "plan": cn.describe_plan(L)})
    if sweep:
        levels_sweep, model = nesting_sweep(torch, np, cn, a, b, c, d, x, N)
        tuned = autotune_leg(torch, np, cn, a, b, c, d, x, N, rows[0]["ms_median"])
    # T's Hermitian part is I, so |x - x*| <= |T x - d|: the residual over |x| bounds the
    # relative forward error of the last solve
    r = a * x
    r[1:] += b[1:] * x[:-1]
    r[:-1] += c[:-1] * x[1:]
    r -= d
    rn = float(torch.linalg.vector_norm(r))
    resid = rn / float(torch.linalg.vector_norm(d))
    fwd_bound = rn / float(torch.linalg.vector_norm(x))
    del r, a, b, c, d, x
    torch.cuda.empty_cache()
    auto = rows[0]
    out = {
        "unknowns_per_solve": N,
        "inputs_sha256_16": sha,
        "auto_ms": auto["ms_median"],
        "auto_unknowns_per_s": N / (auto["ms_median"] * 1e-3),
        "auto_frac_of_peak_80B_compulsory": BYTES_PER_UNKNOWN_SOLVE_MIN * N
                                            / (auto["ms_median"] * 1e-3) / 1e9 / HBM_PEAK_GBS,
        "auto_frac_of_peak_144B_two_pass": auto["GBps_144"] / HBM_PEAK_GBS,
        "residual_rel": resid,
        "forward_error_bound_rel": fwd_bound,
        "paper_optimum_single_level_partition": math.sqrt(N),
        "sweep": rows,
    }
    if sweep:
        out["nesting_sweep"] = levels_sweep
        out["paper_model"] = model
        out["autotune"] = tuned
    if oracle_parity:
        ref = {}

        def make(o):
            oa, ob, oc = o.cn_coeffs(w["V"], w["dx"], w["dt"])
            return lambda: ref.setdefault("x", o.thomas(oa, ob, oc, w["d"]))

        out["cpu_baseline"] = oracle_timed(
            "serial FP64 Thomas on the whole 2^28-row system (same arrays, 1 thread)", make, N,
            out["auto_unknowns_per_s"])
        if "x" in ref:
            out["parity_rel_l2"] = rel_l2(x_auto, ref["x"])
    return out


def nesting_sweep(torch, np, cn, a, b, c, d, x, N):
    """The paper's nesting depth on the 2^28 solve (Sec. 5.5.1, Eqs. (7)-(9)): L partition
    levels of T-row tiles (cn_layout.levels = L), then the serial RS stage on the n / T^L joint
    rows left, for several T and L; stage times from the plan log.  The model
    t = alpha L T + beta n / T^L (parallel stages proportional to the block, the serial RS to
    the rows it eliminates) is fitted to the measured times; delta = sqrt(alpha / beta) and the
    optimal ratio per level (beta n / alpha)^(1/(L+1)) = n^(1/(L+1)) / delta^(2/(L+1)) are set
    beside the measured optimum and the paper's n^(1/(L+1))."""
    pts = []
    grid = [(1, 1024), (1, 2048), (1, 4096), (1, 8192), (1, 16384), (2, 128), (2, 256),
            (2, 512), (2, 1024), (3, 128), (3, 256), (3, 512)]
    for Lv, T in grid:
        M = 2 if T == 128 else (0 if T > 4096 else 4)
        L = cn.Layout.contiguous(N, 1, partition=T, rows_per_thread=M, levels=Lv)
        cn.solve(a, b, c, d, out=x, layout=L)
        reps = 3 if N // T ** Lv <= (1 << 16) else 1
        ts = timed_events(torch, lambda: cn.solve(a, b, c, d, out=x, layout=L), reps)
        cn.profile(True)
        cn.solve(a, b, c, d, out=x, layout=L)
        cn.profile(False)
        st = cn.profile_report()
        par = sum(ms for lab, ms in st if "serial-RS" not in lab)
        rs = sum(ms for lab, ms in st if "serial-RS" in lab)
        top = N // T ** Lv + 1
        pts.append({"levels": Lv, "partition": T, "rows_per_thread": M,
                    "ms_median": float(np.median(ts)), "stage_ms_partition_levels": par,
                    "stage_ms_serial_rs": rs, "serial_rs_rows": top,
                    "beta_us_per_rs_row": rs * 1e3 / top, "plan": cn.describe_plan(L)})
    # least squares for t = alpha L T + beta N / T^L
    A = np.array([[p["levels"] * p["partition"], N / p["partition"] ** p["levels"]] for p in pts])
    t = np.array([p["ms_median"] for p in pts])
    (alpha, beta), *_ = np.linalg.lstsq(A, t, rcond=None)
    model = {"form": "t_ms = alpha * L * T + beta * n / T^L (n = 2^28)",
             "alpha_ms": float(alpha), "beta_ms": float(beta),
             "fit_rel_residual": float(np.linalg.norm(A @ [alpha, beta] - t) / np.linalg.norm(t))}
    if alpha > 0 and beta > 0:
        delta = math.sqrt(alpha / beta)
        model["delta"] = delta
        model["optimal_ratio_fitted"] = {str(Lv): (beta * N / alpha) ** (1.0 / (Lv + 1))
                                         for Lv in (1, 2, 3, 4)}
    model["optimal_ratio_paper"] = {str(Lv): N ** (1.0 / (Lv + 1)) for Lv in (1, 2, 3, 4)}
    best = {}
    for p in pts:
        k = str(p["levels"])
        if k not in best or p["ms_median"] < best[k]["ms_median"]:
            best[k] = {"partition": p["partition"], "ms_median": p["ms_median"]}
    model["measured_best_per_L"] = best
    # beta straight from the serial RS stage time per eliminated row (one level: 2^16..2^18
    # joint rows whose slots come from HBM; smaller top systems sit in the L2 and cost less)
    model["beta_us_per_rs_row_L1"] = float(np.median([p["beta_us_per_rs_row"] for p in pts
                                                      if p["levels"] == 1]))
    return pts, model


def autotune_leg(torch, np, cn, a, b, c, d, x, N, heuristic_ms):
    """cn_autotune on the 2^28 solve: the timed candidates and the chosen plan, timed again
    against the automatic (heuristic) plan."""
    L = cn.Layout.contiguous(N, 1)
    rep = cn.autotune(L, d, x, a=a, b=b, c=c)
    ts = timed_events(torch, lambda: cn.solve(a, b, c, d, out=x, layout=L), 10)
    return {"report": rep, "tuned_ms": float(np.median(ts)), "heuristic_ms": heuristic_ms,
            "tuned_plan": cn.describe_plan(L)}


def long_propagate(torch, np, cn, dev, parity=True):
    """A 2^24-row CN sequence with a field: dx = 0.05, dt = 0.01, soft-core V on the grid,
    x E_k with E ~ N(0, 0.05^2), seeded complex-normal psi; cn_propagate of 20 steps, whose
    two-pass plan runs one fused pass per step (48 B per unknown and step: read psi, V, x,
    write psi)."""
    import workloads

    n, steps, dx, dt = 1 << 24, 20, 0.05, 0.01
    g = np.random.default_rng(1005)
    x = workloads.grid_1d(n, dx)
    V = workloads.softcore(x)
    E = g.normal(0.0, 0.05, steps)
    psi0 = workloads.complex_normal(g, n)
    tV, tx, p0 = (torch.from_numpy(np.ascontiguousarray(a)).to(dev) for a in (V, x, psi0))
    L = cn.Layout.contiguous(n, 1)
    psi = p0.clone()
    cn.propagate(psi, tV, dx, dt, steps, E=E, xgrid=tx, layout=L)
    ts = timed_events(torch, lambda: cn.propagate(psi, tV, dx, dt, steps, E=E, xgrid=tx,
                                                  layout=L), 5)
    med = float(np.median(ts)) / steps
    out = {"n": n, "steps": steps, "us_per_step": med * 1e3,
           "unknowns_per_s": n / (med * 1e-3),
           "GBps_48": 48 * n / (med * 1e-3) / 1e9,
           "frac_of_peak_48B": 48 * n / (med * 1e-3) / 1e9 / HBM_PEAK_GBS,
           "plan": cn.describe_plan(L, True)}
    if parity:
        ns = 3
        ps = p0.clone()
        cn.propagate(ps, tV, dx, dt, ns, E=E[:ns], xgrid=tx, layout=L)
        ref = {}
        out["cpu_baseline"] = oracle_timed(
            f"{ns} CN steps of the 2^24-row system with the field (serial FP64 Thomas, 1 thread)",
            lambda o: (lambda: ref.setdefault("x", o.cn_propagate(psi0, V, dx, dt, ns, x,
                                                                  E[:ns]))),
            ns * n, out["unknowns_per_s"])
        if "x" in ref:
            out["parity_rel_l2_3_steps"] = rel_l2(ps.cpu().numpy(), ref["x"])
    return out


def multi_rhs(torch, np, cn, dev, oracle=True):
    """One 2^22-row matrix (the 2^28 solve's distribution) with 16 right-hand sides: the batch
    reads the matrix of system 0 (shared_coefficients), against the same batch with the matrix
    copied for every right-hand side.  Algorithmic bytes of the shared solve: each right-hand
    side's d and x (32 B per unknown) plus the matrix once (48 B per row)."""
    n, k = 1 << 22, 16
    g = torch.Generator(device=dev)
    g.manual_seed(1006)
    V = torch.rand(n, dtype=torch.float64, device=dev, generator=g) - 1.0
    a, b, c = cn.assemble(V, 0.01, 0.02)
    d = torch.empty(k * n, dtype=torch.complex128, device=dev)
    d.real.normal_(generator=g)
    d.imag.normal_(generator=g)
    x = torch.empty_like(d)
    Ls = cn.Layout.contiguous(n, k, shared_coefficients=True)
    cn.solve(a, b, c, d, out=x, layout=Ls)
    ts = timed_events(torch, lambda: cn.solve(a, b, c, d, out=x, layout=Ls), 10)
    med = float(np.median(ts))
    xs = x.clone()
    A, B, C = (t.repeat(k) for t in (a, b, c))
    Lr = cn.Layout.contiguous(n, k)
    cn.solve(A, B, C, d, out=x, layout=Lr)
    tr = timed_events(torch, lambda: cn.solve(A, B, C, d, out=x, layout=Lr), 10)
    medr = float(np.median(tr))
    same = rel_l2(xs.cpu().numpy(), x.cpu().numpy())
    del A, B, C
    algo = (32 * k + 48) * n
    out = {"n": n, "rhs": k, "ms_shared": med, "ms_replicated": medr,
           "unknowns_per_s": k * n / (med * 1e-3),
           "GBps_algorithmic": algo / (med * 1e-3) / 1e9,
           "frac_of_peak": algo / (med * 1e-3) / 1e9 / HBM_PEAK_GBS,
           "shared_vs_replicated_rel_l2": same,
           "plan": cn.describe_plan(Ls)}
    if not oracle:
        return out
    ref = {}
    a0, b0, c0 = (t.cpu().numpy() for t in (a, b, c))
    dd = d.cpu().numpy()
    def both(o):
        def run():
            ref["x0"] = o.thomas(a0, b0, c0, dd[:n])
            ref["xl"] = o.thomas(a0, b0, c0, dd[(k - 1) * n:])
        return run

    out["cpu_baseline"] = oracle_timed(
        "serial FP64 Thomas on right-hand sides 0 and 15 (1 thread)", both, 2 * n,
        out["unknowns_per_s"])
    if "xl" in ref:
        xh = xs.cpu().numpy()
        out["parity_rel_l2_rhs_0"] = rel_l2(xh[:n], ref["x0"])
        out["parity_rel_l2_rhs_last"] = rel_l2(xh[(k - 1) * n:], ref["xl"])
    return out


def oracle_timed(sample, make, units, gpu_units_per_s, threads=1):
    """The oracle timed on a bounded sample of a workload (make(oracle) returns the call)."""
    try:
        import oracle

        fn = make(oracle)
        t0 = time.perf_counter()
        fn()
        t = max(time.perf_counter() - t0, 1e-9)
        return {"value": units / t, "unit": "complex unknowns/s", "cores": threads,
                "kind": "oracle", "sample": f"{sample}, {t:.2f} s",
                "gpu_over_oracle": gpu_units_per_s / (units / t)}
    except Exception as ex:  # noqa: BLE001
        return {"error": repr(ex)}


def extras(torch, np, cn, workloads, dev):
    out = {}
    # ----------------------------------------------------------- 2^28 explicit solve
    try:
        out["large_system_2^28"] = large_system(torch, np, cn, dev, sweep=True)
        torch.cuda.empty_cache()
    except Exception as ex:  # noqa: BLE001
        out["large_system_2^28"] = {"error": repr(ex)}
    # ----------------------------------------------------------- plain 1D
    try:
        w = workloads.plain_1d()
        psi0 = torch.from_numpy(w["psi0"]).to(dev)
        V = torch.from_numpy(w["V"]).to(dev)
        L = cn.Layout.contiguous(w["n"], 1)
        cn.reserve(L)
        # one materialised solve (a, b, c from the operator; d = explicit half-step of psi0)
        a, b, c = cn.assemble(V, w["dx"], w["dt"])
        d = cn.rhs(psi0, V, w["dx"], w["dt"])
        x = torch.empty_like(d)
        ts_solve = timed_events(torch, lambda: cn.solve(a, b, c, d, out=x, layout=L), 20)
        x_solve = x.cpu().numpy()
        # the plan for sequences: the autotuner times 8 chained steps per candidate tile
        heur_plan = cn.describe_plan(L, True)
        tmp = torch.empty_like(psi0)
        tune_rep = cn.autotune(L, psi0, tmp, V=V, dx=w["dx"], dt=w["dt"], sequence=True)
        del tmp
        # 200 chained steps: eager, then captured as one graph
        psi = psi0.clone()
        ts_eager = timed_events(torch, lambda: cn.propagate(psi, V, w["dx"], w["dt"], w["steps"]), 3)
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            cn.propagate(psi, V, w["dx"], w["dt"], 1)
        torch.cuda.current_stream().wait_stream(side)
        gr = torch.cuda.CUDAGraph()
        with torch.cuda.graph(gr):
            cn.propagate(psi, V, w["dx"], w["dt"], w["steps"])
        psi.copy_(psi0)
        gr.replay()
        torch.cuda.synchronize()
        norm = float(torch.sum(torch.abs(psi) ** 2).item() * w["dx"])
        psi200 = psi.cpu().numpy()
        ts_graph = timed_events(torch, gr.replay, 5)
        med = float(np.median(ts_graph))
        # the same 200 steps as one resident launch (cn_propagate_resident)
        pr = psi0.clone()
        cn.propagate_resident(pr, V, w["dx"], w["dt"], w["steps"])
        torch.cuda.synchronize()
        psi200_res = pr.cpu().numpy()
        ts_res = timed_events(torch, lambda: cn.propagate_resident(pr, V, w["dx"], w["dt"],
                                                                    w["steps"]), 5)
        out["plain_1d"] = {"n": w["n"], "steps": w["steps"],
                           "us_per_step_resident": float(np.median(ts_res)) * 1e3 / w["steps"],
                           "solve_us": float(np.median(ts_solve)) * 1e3,
                           "ms_per_200_steps_graph": med,
                           "us_per_step_graph": med * 1e3 / w["steps"],
                           "us_per_step_eager": float(np.median(ts_eager)) * 1e3 / w["steps"],
                           "unknowns_per_s": w["n"] * w["steps"] / (med * 1e-3),
                           "norm_after_200": norm,
                           "plan": cn.describe_plan(L, True),
                           "heuristic_plan": heur_plan,
                           "autotune_sequence": tune_rep}
        ref = {}
        out["plain_1d"]["cpu_baseline"] = oracle_timed(
            "200 CN steps of the 65536-row system (serial FP64 Thomas, 1 thread)",
            lambda o: (lambda: ref.setdefault("x", o.cn_propagate(w["psi0"], w["V"], w["dx"],
                                                                  w["dt"], w["steps"]))),
            w["n"] * w["steps"], out["plain_1d"]["unknowns_per_s"])
        if "x" in ref:
            out["plain_1d"]["parity_rel_l2_200"] = rel_l2(psi200, ref["x"])
            out["plain_1d"]["parity_rel_l2_200_resident"] = rel_l2(psi200_res, ref["x"])
        # the one materialised solve against the oracle's assembly, half-step and Thomas solve
        import oracle

        oa, ob, oc = oracle.cn_coeffs(w["V"], w["dx"], w["dt"])
        od = oracle.cn_rhs(w["psi0"], w["V"], w["dx"], w["dt"])
        out["plain_1d"]["parity_rel_l2_solve"] = rel_l2(x_solve, oracle.thomas(oa, ob, oc, od))
    except Exception as ex:  # noqa: BLE001
        out["plain_1d"] = {"error": repr(ex)}
    # ----------------------------------------------------------- absorbing potential V - iW
    try:
        out["absorbing"] = absorbing(torch, np, cn, workloads, dev)
        torch.cuda.empty_cache()
    except Exception as ex:  # noqa: BLE001
        out["absorbing"] = {"error": repr(ex)}
    # ----------------------------------------------------------- uneven batch
    try:
        wl = workloads.uneven_batch()
        L = cn.Layout.uneven(wl["offsets"])
        psi = torch.from_numpy(wl["psi0"]).to(dev)
        V = torch.from_numpy(wl["V"]).to(dev)
        dxs = torch.from_numpy(wl["dx"]).to(dev)
        rows = int(wl["offsets"][-1])
        cn.reserve(L)
        cn.step(psi, V, 0.0, wl["dt"], dx_per_system=dxs, out=psi, layout=L)
        ts = timed_events(torch, lambda: cn.step(psi, V, 0.0, wl["dt"], dx_per_system=dxs, out=psi,
                                                 layout=L), wl["steps"])
        med = float(np.median(ts))
        # the same 50 steps as one cn_propagate call (two-pass systems fused across steps),
        # against 50 single steps from the same state
        p0 = psi.clone()
        pstep = p0.clone()
        for _ in range(wl["steps"]):
            cn.step(pstep, V, 0.0, wl["dt"], dx_per_system=dxs, out=pstep, layout=L)
        pprop = p0.clone()
        cn.propagate(pprop, V, 0.0, wl["dt"], wl["steps"], dx_per_system=dxs, layout=L)
        prop_vs_steps = rel_l2(pprop.cpu().numpy(), pstep.cpu().numpy())
        del pstep
        tsq = timed_events(torch, lambda: cn.propagate(pprop, V, 0.0, wl["dt"], wl["steps"],
                                                       dx_per_system=dxs, layout=L), 3)
        med_prop = float(np.median(tsq)) / wl["steps"]
        del pprop, p0
        # the autotuner on this batch: its candidates timed, then the chosen plan (which later
        # calls with this automatic layout take) against the automatic one timed above
        La = cn.Layout.uneven(wl["offsets"])
        outbuf = torch.empty_like(psi)
        tune_rep = cn.autotune(La, psi, outbuf, V=V, dt=wl["dt"], dx_per_system=dxs)
        tst = timed_events(torch, lambda: cn.step(psi, V, 0.0, wl["dt"], dx_per_system=dxs,
                                                  out=psi, layout=La), 10)
        tuned = {"report": tune_rep, "tuned_ms_per_step": float(np.median(tst)),
                 "heuristic_ms_per_step": med, "tuned_plan": cn.describe_plan(La, True)[:300]}
        del outbuf
        # the fixed-plan baseline: one persistent launch over all systems (1024-row tiles)
        Lp = cn.Layout.uneven(wl["offsets"], partition=1024, rows_per_thread=4)
        cn.reserve(Lp)
        tsp = timed_events(torch, lambda: cn.step(psi, V, 0.0, wl["dt"], dx_per_system=dxs,
                                                  out=psi, layout=Lp), 10)
        out["uneven_batch"] = {"systems": wl["batch"], "rows": rows, "steps": wl["steps"],
                               "ms_per_step": med, "unknowns_per_s": rows / (med * 1e-3),
                               "GBps_40": BYTES_PER_UNKNOWN_STEP * rows / (med * 1e-3) / 1e9,
                               "plan": cn.describe_plan(L, True)[:400],
                               "ms_per_step_propagate": med_prop,
                               "propagate_vs_single_steps_rel_l2": prop_vs_steps,
                               "persistent_plan_ms_per_step": float(np.median(tsp)),
                               "persistent_plan": cn.describe_plan(Lp, True)[:200],
                               "autotune": tuned}
        # the workload's whole run: 50 steps of cn_propagate from psi0, against the oracle's
        # 50 batched steps (its timed run is the CPU baseline)
        p50 = torch.from_numpy(wl["psi0"]).to(dev)
        cn.propagate(p50, V, 0.0, wl["dt"], wl["steps"], dx_per_system=dxs, layout=L)
        p50 = p50.cpu().numpy()
        nthr = cpu_threads()
        ref = {}

        def run50(o):
            def run():
                st = wl["psi0"]
                for _ in range(wl["steps"]):
                    st = o.cn_step_batched(wl["offsets"], st, wl["V"], wl["dx"], wl["dt"], nthr)
                ref["x"] = st
            return run

        out["uneven_batch"]["cpu_baseline"] = oracle_timed(
            f"the {wl['steps']} CN steps of all 10^4 systems (serial FP64 Thomas per system, "
            f"{nthr} threads)", run50, rows * wl["steps"],
            out["uneven_batch"]["unknowns_per_s"], nthr)
        if "x" in ref:
            offs = wl["offsets"]
            num_s = np.add.reduceat(np.abs(p50 - ref["x"]) ** 2, offs[:-1])
            den_s = np.add.reduceat(np.abs(ref["x"]) ** 2, offs[:-1])
            out["uneven_batch"]["parity_rel_l2_50_steps"] = float(np.sqrt(num_s.sum()
                                                                          / den_s.sum()))
            out["uneven_batch"]["parity_worst_system_50_steps"] = float(np.sqrt(
                (num_s / den_s).max()))
        del p50, ref
    except Exception as ex:  # noqa: BLE001
        out["uneven_batch"] = {"error": repr(ex)}
    # ----------------------------------------------------------- differentiated propagation
    try:
        out["differentiated"] = differentiated(torch, np, workloads, dev)
    except Exception as ex:  # noqa: BLE001
        out["differentiated"] = {"error": repr(ex)}
    # ----------------------------------------------------------- one matrix, 16 right-hand sides
    try:
        out["multi_rhs_2^22x16"] = multi_rhs(torch, np, cn, dev)
        torch.cuda.empty_cache()
    except Exception as ex:  # noqa: BLE001
        out["multi_rhs_2^22x16"] = {"error": repr(ex)}
    # ----------------------------------------------------------- partial waves (radial, Sec. 3)
    try:
        out["radial_2^16x64"] = radial(torch, np, cn, workloads, dev)
        torch.cuda.empty_cache()
    except Exception as ex:  # noqa: BLE001
        out["radial_2^16x64"] = {"error": repr(ex)}
    # ----------------------------------------------------------- 2^24-row fused propagation
    try:
        out["propagate_2^24"] = long_propagate(torch, np, cn, dev)
        torch.cuda.empty_cache()
    except Exception as ex:  # noqa: BLE001
        out["propagate_2^24"] = {"error": repr(ex)}
    return out


def radial(torch, np, cn, workloads, dev, parity=True):
    """Partial waves of an atom in a field (Sec. 3): 64 waves (l = 0..63) on 2^16 radial points
    (dr = 0.1, soft Coulomb V = -1/sqrt(r^2 + 0.5)), dt = 0.02, a seeded field E_k ~ N(0, 0.05^2);
    each step is the CN step in r of every wave (64 systems of 2^16 rows) and the CN step in l
    at every radial point (2^16 interleaved systems of 64 rows).  100 steps captured in one
    graph; the oracle runs the first 3 steps for parity."""
    nr, nl, dr, dt, steps = 1 << 16, 64, 0.1, 0.02, 100
    g = np.random.default_rng(1007)
    r = dr * np.arange(1, nr + 1)
    V = -1.0 / np.sqrt(r * r + 0.5)
    E = g.normal(0.0, 0.05, steps)
    psi0 = workloads.complex_normal(g, nl * nr)
    psi0 /= np.linalg.norm(psi0)
    tV = torch.from_numpy(V).to(dev)
    p0 = torch.from_numpy(psi0).to(dev)
    cn.reserve(cn.Layout.contiguous(nr, nl))
    cn.reserve(cn.Layout(n=nl, batch=nr, elem_stride=nr, batch_stride=1))
    x = p0.clone()
    cn.radial_step(x, tV, dr, dt, E[0], 0, nl, out=x)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    gr = torch.cuda.CUDAGraph()
    with torch.cuda.graph(gr, stream=side):
        for k in range(steps):
            cn.radial_step(x, tV, dr, dt, float(E[k]), 0, nl, out=x)
    x.copy_(p0)
    gr.replay()
    torch.cuda.synchronize()
    norm = float(torch.linalg.vector_norm(x))
    ts = timed_events(torch, gr.replay, 5)
    us = float(np.median(ts)) * 1e3 / steps
    res = {"nr": nr, "nl": nl, "steps": steps, "us_per_step": us,
           "unknowns_per_s": nr * nl / (us * 1e-6), "norm_after_100": norm,
           "plan_r": cn.describe_plan(cn.Layout.contiguous(nr, nl), True),
           "plan_l": cn.describe_plan(cn.Layout(n=nl, batch=nr, elem_stride=nr, batch_stride=1))}
    if not parity:
        return res
    ns = 3
    x3 = p0.clone()
    for k in range(ns):
        cn.radial_step(x3, tV, dr, dt, float(E[k]), 0, nl, out=x3)
    x3 = x3.cpu().numpy()
    ref = {}

    def run3(o):
        def run():
            st = psi0
            for k in range(ns):
                st = o.radial_step(st, V, dr, dt, float(E[k]), 0, nl)
            ref["x"] = st
        return run

    res["cpu_baseline"] = oracle_timed(
        f"the first {ns} partial-wave steps (serial FP64 Thomas per wave and per radial point, "
        f"1 thread)", run3, ns * nr * nl, res["unknowns_per_s"])
    if "x" in ref:
        res["parity_rel_l2_3_steps"] = rel_l2(x3, ref["x"])
    return res


def uneven_timing(torch, np, cn, workloads, dev):
    """The uneven batch alone (automatic plan): 10 single steps, then 10 steps of cn_propagate."""
    wl = workloads.uneven_batch()
    L = cn.Layout.uneven(wl["offsets"])
    psi = torch.from_numpy(wl["psi0"]).to(dev)
    V = torch.from_numpy(wl["V"]).to(dev)
    dxs = torch.from_numpy(wl["dx"]).to(dev)
    rows = int(wl["offsets"][-1])
    cn.reserve(L)
    cn.step(psi, V, 0.0, wl["dt"], dx_per_system=dxs, out=psi, layout=L)
    ts = timed_events(torch, lambda: cn.step(psi, V, 0.0, wl["dt"], dx_per_system=dxs, out=psi,
                                             layout=L), 10)
    tp = timed_events(torch, lambda: cn.propagate(psi, V, 0.0, wl["dt"], 10, dx_per_system=dxs,
                                                  layout=L), 2)
    med, medp = float(np.median(ts)), float(np.median(tp)) / 10
    return {"rows": rows, "ms_per_step": med, "ms_per_step_propagate": medp,
            "GBps_40_step": 40 * rows / (med * 1e-3) / 1e9,
            "GBps_40_propagate": 40 * rows / (medp * 1e-3) / 1e9,
            "plan": cn.describe_plan(L, True)}


def absorbing(torch, np, cn, workloads, dev):
    """Steps with an absorbing potential (non-Hermitian H) through the fused kernels: the plain
    1D workload with a ramp at both walls, 200 steps in a graph and as one resident launch, with
    the oracle's 200 steps for parity; and 2^24 rows, 10 steps per call, beside the materialised
    form."""
    res = {}
    w = workloads.absorbing_1d()
    psi0 = torch.from_numpy(w["psi0"]).to(dev)
    V = torch.from_numpy(w["V"]).to(dev)
    W = torch.from_numpy(w["W"]).to(dev)
    L = cn.Layout.contiguous(w["n"], 1)
    cn.reserve(L)
    psi = psi0.clone()
    cn.propagate(psi, V, w["dx"], w["dt"], 1, W=W, layout=L)
    torch.cuda.synchronize()
    gr = torch.cuda.CUDAGraph()
    with torch.cuda.graph(gr):
        cn.propagate(psi, V, w["dx"], w["dt"], w["steps"], W=W, layout=L)
    psi.copy_(psi0)
    gr.replay()
    torch.cuda.synchronize()
    psi200 = psi.cpu().numpy()
    med = float(np.median(timed_events(torch, gr.replay, 5)))
    # the same 200 steps as one resident launch
    pr = psi0.clone()
    cn.propagate_resident(pr, V, w["dx"], w["dt"], w["steps"], W=W)
    torch.cuda.synchronize()
    psi200_res = pr.cpu().numpy()
    med_res = float(np.median(timed_events(
        torch, lambda: cn.propagate_resident(pr, V, w["dx"], w["dt"], w["steps"], W=W), 5)))
    n0 = float(np.sum(np.abs(w["psi0"]) ** 2))
    res["1d_65536"] = {"steps": w["steps"], "us_per_step_graph": med * 1e3 / w["steps"],
                       "us_per_step_resident": med_res * 1e3 / w["steps"],
                       "unknowns_per_s": w["n"] * w["steps"] / (med * 1e-3),
                       "norm_left_after_200": float(np.sum(np.abs(psi200) ** 2)) / n0}
    ref = {}
    res["1d_65536"]["cpu_baseline"] = oracle_timed(
        "200 absorbing CN steps of the 65536-row system (serial FP64 Thomas, 1 thread)",
        lambda o: (lambda: ref.setdefault("x", o.cn_propagate(w["psi0"], w["V"], w["dx"],
                                                              w["dt"], w["steps"], W=w["W"]))),
        w["n"] * w["steps"], res["1d_65536"]["unknowns_per_s"])
    if "x" in ref:
        res["1d_65536"]["parity_rel_l2_200"] = rel_l2(psi200, ref["x"])
        res["1d_65536"]["parity_rel_l2_200_resident"] = rel_l2(psi200_res, ref["x"])
    del psi, psi0, V, W, pr
    res["2^24"] = absorbing_large(torch, np, cn, workloads, dev)
    return res


def absorbing_large(torch, np, cn, workloads, dev):
    """2^24 rows with an absorbing ramp, 10 steps per timed cn_propagate call: the fused
    kernels (one pass per step, 48 B per unknown and step: read psi, V, W, write psi), beside
    the materialised form of the same steps (T assembled once, then per step the explicit side
    into d and the general two-pass solve: 48 + 144 = 192 B per unknown and step), run here
    through cn_rhs and cn_tridiag_solve."""
    n, steps = 1 << 24, 10
    g = np.random.default_rng(1010)
    Vb = torch.from_numpy(g.uniform(-1.0, 0.0, n)).to(dev)
    Wb = torch.from_numpy(workloads.absorber(n)).to(dev)
    p0 = torch.from_numpy(workloads.complex_normal(g, n)).to(dev)
    Lb = cn.Layout.contiguous(n, 1)
    cn.reserve(Lb)
    pb = p0.clone()
    cn.propagate(pb, Vb, 0.01, 0.02, 1, W=Wb, layout=Lb)
    ts = timed_events(torch, lambda: cn.propagate(pb, Vb, 0.01, 0.02, steps, W=Wb, layout=Lb), 3)
    us = float(np.median(ts)) * 1e3 / steps
    # materialised: the same steps from the same state, compared with the fused result
    a, b, c = cn.assemble(Vb, 0.01, 0.02, W=Wb)
    d = torch.empty_like(p0)
    pm = p0.clone()

    def mat_steps():
        for _ in range(steps):
            cn.rhs(pm, Vb, 0.01, 0.02, W=Wb, out=d)
            cn.solve(a, b, c, d, out=pm, layout=Lb)

    pf = p0.clone()
    cn.propagate(pf, Vb, 0.01, 0.02, steps, W=Wb, layout=Lb)
    mat_steps()
    agree = rel_l2(pf.cpu().numpy(), pm.cpu().numpy())
    tm = timed_events(torch, mat_steps, 3)
    us_m = float(np.median(tm)) * 1e3 / steps
    return {"steps": steps, "us_per_step": us, "unknowns_per_s": n / (us * 1e-6),
            "GBps_48": 48.0 * n / (us * 1e-6) / 1e9,
            "frac_of_8TBps_48B": 48.0 * n / (us * 1e-6) / 8e12,
            "plan": cn.describe_plan(Lb, absorbing=True),
            "materialised_us_per_step": us_m,
            "materialised_frac_of_8TBps_192B": 192.0 * n / (us_m * 1e-6) / 8e12,
            "fused_vs_materialised_rel_l2": agree}


def latency_legs(torch, np, cn, workloads, dev):
    """Step times of the latency-bound sequences alone: the plain 1D workload (200 steps in
    one graph, with the automatic plan and after the sequence autotuner; and as one resident
    launch) and the differentiated workload's 2000-step forward with checkpoints and its
    reverse mode (C ABI directly)."""
    out = {}
    w = workloads.plain_1d()
    psi0 = torch.from_numpy(w["psi0"]).to(dev)
    V = torch.from_numpy(w["V"]).to(dev)
    L = cn.Layout.contiguous(w["n"], 1)
    cn.reserve(L)

    def graph_us():
        psi = psi0.clone()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            cn.propagate(psi, V, w["dx"], w["dt"], 1)
        torch.cuda.current_stream().wait_stream(side)
        gr = torch.cuda.CUDAGraph()
        with torch.cuda.graph(gr):
            cn.propagate(psi, V, w["dx"], w["dt"], w["steps"])
        gr.replay()
        torch.cuda.synchronize()
        return float(np.median(timed_events(torch, gr.replay, 5))) * 1e3 / w["steps"]

    out["plain_1d_heuristic"] = {"plan": cn.describe_plan(L, True), "us_per_step": graph_us()}
    tmp = torch.empty_like(psi0)
    rep = cn.autotune(L, psi0, tmp, V=V, dx=w["dx"], dt=w["dt"], sequence=True)
    out["plain_1d_tuned"] = {"plan": cn.describe_plan(L, True), "us_per_step": graph_us(),
                             "autotune": rep}
    del tmp
    pr = psi0.clone()
    cn.propagate_resident(pr, V, w["dx"], w["dt"], w["steps"])
    out["plain_1d_resident"] = {"us_per_step": float(np.median(timed_events(
        torch, lambda: cn.propagate_resident(pr, V, w["dx"], w["dt"], w["steps"]), 5)))
        * 1e3 / w["steps"]}
    d = workloads.differentiated()
    n, steps, K = d["n"], d["steps"], d["ckpt"]
    Ld = cn.Layout.contiguous(n, 1)
    tV, tx, p0, g0 = (torch.from_numpy(np.ascontiguousarray(a)).to(dev)
                      for a in (d["V"], d["x"], d["psi0"], d["phi"]))
    ckpt = torch.empty(((steps + K - 1) // K) * n, dtype=torch.complex128, device=dev)
    dV = torch.zeros(n, dtype=torch.float64, device=dev)
    dE = torch.zeros(steps, dtype=torch.float64, device=dev)
    psi = p0.clone()
    g = g0.clone()

    def fwd():
        psi.copy_(p0)
        cn.propagate(psi, tV, d["dx"], d["dt"], steps, E=d["E"], xgrid=tx, ckpt=ckpt, K=K,
                     layout=Ld)

    def bwd():
        g.copy_(g0)
        cn.propagate_adjoint(ckpt, g, tV, d["dx"], d["dt"], steps, K, E=d["E"], xgrid=tx, dV=dV,
                             dE=dE, layout=Ld)

    fwd()
    bwd()
    tf = float(np.median(timed_events(torch, fwd, 3)))
    tb = float(np.median(timed_events(torch, bwd, 3)))
    out["differentiated"] = {"plan": cn.describe_plan(Ld, True), "forward_ms": tf,
                             "backward_ms": tb, "forward_us_per_step": tf * 1e3 / steps,
                             "backward_us_per_step": tb * 1e3 / steps}
    return out


def differentiated(torch, np, workloads, dev):
    """N = 2^20, 2000 steps, checkpoint every 50: forward and backward wall time (inclusive
    ratio), gradients of |<phi|psi_T>|^2 w.r.t. V (32 coordinates) and E (32) against central
    finite differences of the forward."""
    from paper_2205_00856_amd import autograd as ag

    w = workloads.differentiated()
    dx, dt, K = w["dx"], w["dt"], w["ckpt"]
    tV = torch.tensor(w["V"], device=dev, requires_grad=True)
    tE = torch.tensor(w["E"], device=dev, requires_grad=True)
    tx = torch.tensor(w["x"], device=dev)
    p0 = torch.tensor(w["psi0"], device=dev)
    phi = torch.tensor(w["phi"], device=dev)

    # the plan for the sequence: the autotuner times 8 chained steps per candidate tile (the
    # reverse mode's recompute and recursion run on the same plan)
    import paper_2205_00856_amd as cn

    Lw = cn.Layout.contiguous(w["n"], 1)
    tmp = torch.empty_like(p0)
    tune_rep = cn.autotune(Lw, p0, tmp, V=tV.detach(), dx=dx, dt=dt, E=float(w["E"][0]),
                           xgrid=tx, sequence=True)
    del tmp

    def fwd(Vt, Et):
        return ag.cn_propagate(p0, Vt, Et, dx, dt, xgrid=tx, K=K)

    def loss_of(out):
        return torch.abs((torch.conj(phi) * out).sum() * dx) ** 2

    with torch.no_grad():
        fwd(tV.detach(), tE.detach())  # warm-up (plans, workspace)
    tf, tb = [], []
    for _ in range(3):
        tV.grad = None
        tE.grad = None
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        out = fwd(tV, tE)
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        L = loss_of(out)
        torch.cuda.synchronize()
        t2 = time.perf_counter()
        L.backward()
        torch.cuda.synchronize()
        t3 = time.perf_counter()
        tf.append(t1 - t0)
        tb.append(t3 - t2)
    gV = tV.grad.detach().cpu().numpy()
    gE = tE.grad.detach().cpu().numpy()
    norm = float(torch.sum(torch.abs(out) ** 2).item() * dx)
    # finite differences on 64 coordinates
    rng = np.random.default_rng(2004)
    dens = np.abs(w["psi0"]) ** 2 + np.abs(w["phi"]) ** 2
    cand = np.nonzero(dens > 1e-6 * dens.max())[0]
    js = rng.choice(cand, 32, replace=False)
    ks = rng.choice(w["steps"], 32, replace=False)
    h = 1e-4
    num, ana = [], []
    with torch.no_grad():
        Vd, Ed = tV.detach(), tE.detach()
        for j in js:
            Vp, Vm = Vd.clone(), Vd.clone()
            Vp[j] += h
            Vm[j] -= h
            num.append(float(loss_of(fwd(Vp, Ed)) - loss_of(fwd(Vm, Ed))) / (2 * h))
            ana.append(float(gV[j]))
        for k in ks:
            Ep, Em = Ed.clone(), Ed.clone()
            Ep[k] += h
            Em[k] -= h
            num.append(float(loss_of(fwd(Vd, Ep)) - loss_of(fwd(Vd, Em))) / (2 * h))
            ana.append(float(gE[k]))
    num = np.asarray(num)
    ana = np.asarray(ana)
    fwd_s = float(np.median(tf))
    bwd_s = float(np.median(tb))
    # the reverse mode without checkpoints: each segment's states rebuilt backwards from the
    # state at its end (psi_T for the last) beside the recursion, for the same gradient at psi_T
    o = out.detach().clone().requires_grad_(True)
    loss_of(o).backward()
    gT = o.grad.detach()
    psiT_dev = o.detach()
    dVr = torch.zeros(w["n"], dtype=torch.float64, device=dev)
    dEr = torch.zeros(w["steps"], dtype=torch.float64, device=dev)

    def bwd_rec():
        gg = gT.clone()
        dVr.zero_()
        cn.propagate_adjoint_reconstruct(psiT_dev, gg, tV.detach(), dx, dt, w["steps"], K,
                                         E=w["E"], xgrid=tx, dV=dVr, dE=dEr, layout=Lw)

    bwd_rec()
    trec = float(np.median(timed_events(torch, bwd_rec, 3))) * 1e-3
    # the forward as one resident launch (cn_propagate_resident, checkpoints from registers)
    with torch.no_grad():
        ag.cn_propagate(p0, tV.detach(), tE.detach(), dx, dt, xgrid=tx, K=K, resident=True)
    tfr = []
    for _ in range(3):
        tV.grad = None
        tE.grad = None
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        out_r = ag.cn_propagate(p0, tV, tE, dx, dt, xgrid=tx, K=K, resident=True)
        torch.cuda.synchronize()
        tfr.append(time.perf_counter() - t0)
    loss_of(out_r).backward()
    resident = {
        "forward_ms": float(np.median(tfr)) * 1e3,
        "forward_us_per_step": float(np.median(tfr)) * 1e6 / w["steps"],
        "adjoint_over_forward": bwd_s / float(np.median(tfr)),
        "rel_l2_psi_T_vs_chained": float(torch.linalg.vector_norm(out_r.detach() - out.detach())
                                         / torch.linalg.vector_norm(out.detach())),
        "rel_l2_dV_vs_chained": float(np.linalg.norm(tV.grad.detach().cpu().numpy() - gV)
                                      / np.linalg.norm(gV)),
    }
    reconstruct = {
        "backward_ms": trec * 1e3,
        "adjoint_over_forward": trec / fwd_s,
        "rel_l2_dV_vs_checkpointed": float(np.linalg.norm(dVr.cpu().numpy() - gV)
                                           / np.linalg.norm(gV)),
        "rel_l2_dE_vs_checkpointed": float(np.linalg.norm(dEr.cpu().numpy() - gE)
                                           / np.linalg.norm(gE)),
        "memory": f"two segment buffers of {K + 1} states, no checkpoints "
                  f"(checkpointed: {(w['steps'] + K - 1) // K} stored states + the buffers)",
    }
    # the oracle beside it: the whole 2000-step propagation (1 thread), against which the
    # GPU's psi_T and loss are compared
    psiT = out.detach().cpu().numpy()
    ref = {}
    cpu = oracle_timed(
        f"all {w['steps']} steps of the 2^20-row propagation with the field term (serial FP64 "
        f"Thomas, 1 thread)",
        lambda o: (lambda: ref.setdefault("x", o.cn_propagate(w["psi0"], w["V"], dx, dt,
                                                              w["steps"], xgrid=w["x"],
                                                              E=w["E"]))),
        w["n"] * w["steps"], w["n"] * w["steps"] / fwd_s)
    par = par_loss = None
    if "x" in ref:
        par = rel_l2(psiT, ref["x"])
        ref_loss = abs(np.sum(np.conj(w["phi"]) * ref["x"]) * dx) ** 2
        par_loss = abs(float(L.item()) - ref_loss) / ref_loss
    return {
        "cpu_baseline": cpu,
        "parity_rel_l2_psi_T": par,
        "parity_rel_loss": par_loss,
        "n": w["n"], "steps": w["steps"], "checkpoint_every": K,
        "forward_ms": fwd_s * 1e3, "backward_ms": bwd_s * 1e3,
        "forward_us_per_step": fwd_s * 1e6 / w["steps"],
        "backward_us_per_step": bwd_s * 1e6 / w["steps"],
        "adjoint_over_forward": bwd_s / fwd_s,
        "loss": float(L.item()), "norm_T": norm,
        "fd_rel_l2_64": float(np.linalg.norm(ana - num) / np.linalg.norm(num)),
        "fd_max_rel_per_coord": float(np.max(np.abs(ana - num) / np.maximum(np.abs(num), 1e-300))),
        "fd_step": h,
        "phi_draw": list(map(float, w["phi_params"])),
        "plan": cn.describe_plan(Lw, True),
        "autotune_sequence": tune_rep,
        "reverse_reconstruction": reconstruct,
        "forward_resident": resident,
    }


if __name__ == "__main__":
    main()
