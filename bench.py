#!/usr/bin/env python3
"""Benchmark of the ensemble flood hot path on one MI355X.

Workload (default): 2000 x 2000 cells (4.0 M, 3 m), 96 members, FP32 state,
urban synthetic DEM, Chicago storm, per-member lognormal Manning scales and
rain multipliers, particle filter every 600 s on 10 depth gauges.

One benchmark step = one assimilation cycle: every member advances 600 s of
simulated time (adaptive Eq. 4 steps, one fused kernel launch per step for
all members) followed by the filter update (gauge gather, weights, N_eff,
systematic resampling and member copy when N_eff < 0.8 N).  Observations
come from a hidden truth member run beforehand plus N(0, 0.05^2) noise.
Every cycle lies inside the one-hour storm: after its sixth window the
ensemble restarts from its initial state (a device snapshot taken at t = 0,
restored on the device inside the timed region), so cycle k covers window
k mod 6.

`value` is member-cell-updates per second (MCU/s) over the timed cycles,
counted from the per-member step counters, filter updates and restarts
included, on the library's captured-graph path.  The JSON line also carries
the roofline of the step kernel (a HIP event pair around every captured batch
of steps in the timed region, so the duration per step launch also holds the
step's small planner kernel and the gaps between kernels; a kernel trace of the
same command gives the step kernel's own duration), the FP64 oracle timed on
the host cores, and in `detail` the other parts of the metric, each outside the
timed region:
  * step kernels alone (MCU over summed kernel time);
  * forward + adjoint over the first 900 s of the same ensemble (Manning-field
    and rain-multiplier gradients of a 10-s gauge misfit, checkpoints every
    1024 steps, so that each member group's tape is one segment) against the
    forward alone over the same window, one handle each, timed twice in turns
    from the dry state and compared by their means;
  * batched against plain (one handle and one launch per member) on this
    workload over its first window, and on the four-catchment batch
    (512^2, 768x1536, 1024^2, 2000^2, 24 members each) over its first 300 s;
  * the running maximum depth tracked through the first window (its cost) and
    the ensemble products of every cell (Sec. 4.4, Figs. 15-16);
  * the same ensemble with land cover (Table 1) over its first window;
  * the same ensemble with two stream outlets (inflow hydrographs) over its
    first window and a filter cycle on depths and streamflow together;
  * the streaming ceiling of one elementwise kernel (2 GiB in, 2 GiB out).

The timed cycles run last among full-size launches of the step kernel, so
that a kernel trace of this command can isolate them (the last `launches`
dispatches of that kernel with the full ensemble's grid).
"""
from __future__ import annotations

import argparse
import hashlib
import json
import multiprocessing as mp
import os
import re
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
BYTES_PER_MCU = 24.0    # h, qx, qy read + written once per member-cell-step (FP32)
KERNEL_NAMES = {1: "k_step", 2: "k_march", 3: "k_marchv"}
KERNEL_TITLES = {1: "k_step (tiled fused step)", 2: "k_march (row-march fused step)",
                 3: "k_marchv (vectorised row-march fused step)"}
KERNEL_SOURCES = ("paper_2302_08341_amd/csrc/flood_kernels.hip", "paper_2302_08341_amd/csrc/flood_device.h",
                  "paper_2302_08341_amd/csrc/flood_internal.h", "paper_2302_08341_amd/csrc/flood_rows.h")


def log(msg):
    print("[bench] " + msg, file=sys.stderr, flush=True)


def _cpu_worker(args):
    """Run one member of the workload with the oracle for n_steps from the dry start."""
    cfg, member, n_steps = args
    import oracle
    import workloads as W
    wl = W.CONFIGS[cfg["config"]](cfg["ny"], cfg["nx"], cfg["members"])
    c = wl.catchments[0]
    m = oracle.Model.from_workload(wl)
    mem = oracle.Member.dry(m, s=c.n_scale[member], mu=c.rain_mult[member])
    t0 = time.perf_counter()
    n = oracle.advance(m, mem, wl.t_end, max_steps=n_steps)
    el = time.perf_counter() - t0
    return n * c.ny * c.nx, el


def cpu_model():
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    import platform
    return platform.processor() or "unknown"


def cpu_baseline(cfg, cores, n_steps):
    ctx = mp.get_context("spawn")
    jobs = [(cfg, i % cfg["members"], n_steps) for i in range(cores)]
    t0 = time.perf_counter()
    # close and join rather than the context manager's terminate: the workers end
    # on their own instead of by a signal (profilers that preload a library into
    # every child can stall on a signalled exit)
    pool = ctx.Pool(cores)
    try:
        res = pool.map(_cpu_worker, jobs)
        pool.close()
    except BaseException:
        pool.terminate()
        raise
    finally:
        pool.join()
    wall = time.perf_counter() - t0
    mcu = sum(r[0] for r in res)
    busy = max(r[1] for r in res)
    return {"value": mcu / busy, "unit": "MCU/s", "cores": cores, "kind": "oracle",
            "cpu_model": cpu_model(), "host_cpus": os.cpu_count(),
            "sample": "FP64 serial oracle, one process per core, each running one member of the same "
                      "workload for its first %d steps from the dry start (%d member-runs, %.1f s per "
                      "process, %.1f s wall incl. start-up)" % (n_steps, cores, busy, wall)}


_COMMENT = re.compile(r"//[^\n]*|/\*.*?\*/", re.S)


def kernel_source_hash():
    """Hash of the step kernel's sources with comments and layout taken out: an
    edit of comments or whitespace leaves the kernel, and so its counters, as they
    were."""
    h = hashlib.sha256()
    for p in KERNEL_SOURCES:
        with open(os.path.join(ROOT, p)) as f:
            code = _COMMENT.sub(" ", f.read())
        h.update(" ".join(code.split()).encode())
        h.update(b"\0")
    return h.hexdigest()[:16]


def measured_traffic(kernel, workload_tag, alg_bytes=None):
    """HBM bytes per launch from the committed counter summary of this kernel and
    workload, if it was taken on the current kernel sources, and (given this
    run's algorithmic bytes per launch) on the same timed launches, i.e. the
    summary's own algorithmic bytes per launch agree within 0.5 %; else None."""
    path = os.path.join(ROOT, "profiles", "%s_%s_traffic.md" % (kernel, workload_tag))
    if not os.path.exists(path):
        return None
    vals = {}
    with open(path) as f:
        for line in f:
            if line.startswith("- ") and ":" in line:
                k, v = line[2:].split(":", 1)
                vals[k.strip()] = v.strip().strip("`")
    if vals.get("kernel_sources_sha256") != kernel_source_hash():
        return None
    try:
        traffic = float(vals["traffic_bytes_per_launch"])
        if alg_bytes is not None:
            own = float(vals["algorithmic_bytes_per_launch"])
            if abs(own - alg_bytes) > 0.005 * alg_bytes:
                return None
        return traffic
    except (KeyError, ValueError):
        return None


def ensemble_args(c, members, n_scale=None, rain_mult=None):
    return dict(dem=c.dem, manning=c.manning, dx=c.dx, edge_kind=c.edge_kind, edge_slope=c.edge_slope,
                n_members=len(members) if n_scale is None else len(n_scale),
                n_scale=c.n_scale[members] if n_scale is None else n_scale,
                rain_mult=c.rain_mult[members] if rain_mult is None else rain_mult)


def truth_depths(FloodEnsemble, wl, times):
    """Gauge depths of a hidden truth member (drawn from the same prior) at the
    given times.  Runs on the tiled kernel so that the step kernel measured below
    sees only ensemble launches."""
    c = wl.catchments[0]
    truth = FloodEnsemble([ensemble_args(c, None, [c.truth_n_scale], [c.truth_rain_mult])], wl.rain,
                          rain_interval=wl.rain_interval, real_bytes=wl.real_bytes, step_kernel=1,
                          tile_rows=4, chunks_per_block=1, march_rows=8, march_members=1)
    out = {}
    for t in sorted(times):
        truth.step(t)
        out[t] = truth.field(0)[c.gauges[:, 0], c.gauges[:, 1]]
    truth.close()
    return out


def elementwise_ceiling(torch):
    """One elementwise kernel reading and writing 2 GiB each: the attainable
    streaming rate, and the known-size kernel for scaling the memory counters."""
    x = torch.ones(1 << 29, dtype=torch.float32, device="cuda")
    ea, eb = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    y = x + 1.0
    torch.cuda.synchronize()
    ea.record()
    for _ in range(5):
        y = x + 1.0
    eb.record()
    torch.cuda.synchronize()
    gbs = 5 * 2 * x.numel() * 4 / (ea.elapsed_time(eb) * 1e-3) / 1e9
    del x, y
    torch.cuda.empty_cache()
    return gbs


def leg_adjoint(FloodEnsemble, wl, obs_adj, window, sample_dt, ckpt, reps=2):
    """Forward + adjoint over [0, window] of the full ensemble against the forward
    alone, one handle each, timed in turns reps times and compared by their means.
    Every run starts from the dry state (set before the clock starts); the
    adjoint's scratch stays on its handle between runs, as in a calibration loop
    that calls the adjoint again and again."""
    c = wl.catchments[0]
    ncell = c.ny * c.nx
    obs = np.stack([obs_adj[t] for t in sorted(obs_adj)])
    dry = (np.zeros((c.ny, c.nx)), np.zeros((c.ny, c.nx + 1)), np.zeros((c.ny + 1, c.nx)))
    fwd = FloodEnsemble.from_workload(wl)
    adj = FloodEnsemble.from_workload(wl)

    def restart(e):
        for i in range(c.n_members):
            e.set_state(i, *dry, 0.0)

    def steps(e):
        return int(e.ledger()["steps"].sum())

    t_fwd, t_adj = [], []
    for r in range(reps):
        if r:
            restart(fwd)
            restart(adj)
        s0 = steps(fwd)
        t0 = time.perf_counter()
        fwd.step(window)
        t_fwd.append(time.perf_counter() - t0)
        steps_fwd = steps(fwd) - s0
        log("adjoint leg: forward alone %.2f s" % t_fwd[-1])
        s0 = steps(adj)
        t0 = time.perf_counter()
        loss, gn, gm = adj.adjoint(0, window, sample_dt, c.gauges, obs, ckpt_every=ckpt)
        t_adj.append(time.perf_counter() - t0)
        steps_adj = steps(adj) - s0
        log("adjoint leg: forward + adjoint %.2f s" % t_adj[-1])
    fwd.close()
    adj.close()
    tf, ta = float(np.mean(t_fwd)), float(np.mean(t_adj))
    return {"workload": "first %.0f s of the same ensemble (%d x %d cells x %d members), loss = squared misfit "
                        "at %d gauges every %.0f s, checkpoints every %d steps" % (
                            window, c.ny, c.nx, c.n_members, c.gauges.shape[0], sample_dt, ckpt),
            "fwd_adj_MCUps": steps_adj * ncell / ta, "fwd_MCUps": steps_fwd * ncell / tf,
            "member_steps": steps_adj, "fwd_s": tf, "fwd_adj_s": ta, "adj_over_fwd": ta / tf,
            "runs_fwd_s": t_fwd, "runs_fwd_adj_s": t_adj,
            "loss": float(loss), "grad_n_norm": float(np.linalg.norm(gn)),
            "grad_mult_mean_abs": float(np.mean(np.abs(gm)))}


def leg_c4(FloodEnsemble, W, window, per_catch):
    """Four uneven catchments in one batched handle against one handle per member."""
    wl = W.config4()
    ens = FloodEnsemble.from_workload(wl)
    t0 = time.perf_counter()
    ens.step(window)
    t_b = time.perf_counter() - t0
    conf = ens.config()
    steps = [ens.ledger(i)["steps"] for i in range(len(wl.catchments))]
    ens.close()
    mcu = sum(int(s.sum()) * c.ny * c.nx for s, c in zip(steps, wl.catchments))
    # plain: a sample of members per catchment, each alone; the full job's plain
    # time is the per-member mean times the member count, catchment by catchment
    plain_time = 0.0
    sampled = []
    for j, c in enumerate(wl.catchments):
        ts = []
        for m in range(per_catch):
            e = FloodEnsemble([ensemble_args(c, [m])], wl.rain, rain_interval=wl.rain_interval,
                              real_bytes=wl.real_bytes)
            t0 = time.perf_counter()
            e.step(window)
            ts.append(time.perf_counter() - t0)
            if int(e.ledger()["steps"][0]) != int(steps[j][m]):
                raise RuntimeError("plain and batched member step counts differ")
            e.close()
        plain_time += c.n_members * float(np.mean(ts))
        sampled.append(float(np.mean(ts)))
    log("four-catchment leg: batched %.2f s, plain (estimated) %.2f s" % (t_b, plain_time))
    return {"workload": "512^2, 768x1536, 1024^2, 2000^2 cells x 24 members each, first %.0f s" % window,
            "batched_MCUps": mcu / t_b, "plain_MCUps": mcu / plain_time, "speedup": plain_time / t_b,
            "batched_s": t_b, "plain_s_estimated": plain_time,
            "plain_sample": "%d members per catchment run alone; mean seconds per member %s" % (
                per_catch, [round(x, 4) for x in sampled]),
            "batched_config": conf}


def leg_products(FloodEnsemble, wl, window):
    """Running maximum depth tracked through the first window, then the ensemble
    products of every cell (probability of reaching 0.2 m, 10/50/90 % maxima)."""
    import torch
    c = wl.catchments[0]
    ncell = c.ny * c.nx
    ens = FloodEnsemble.from_workload(wl, track_peak=True)
    t0 = time.perf_counter()
    ens.step(window)
    t_step = time.perf_counter() - t0
    steps = int(ens.ledger()["steps"].sum())
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    prob, pc = ens.products(0.2, (0.1, 0.5, 0.9))
    t_prod = time.perf_counter() - t0
    ens.close()
    log("products leg: %.2f s stepping with running maxima, %.3f s products" % (t_step, t_prod))
    return {"workload": "first %.0f s of this ensemble with running maxima; products of every cell" % window,
            "tracked_MCUps": steps * ncell / t_step, "products_s": t_prod,
            "products": "P(max depth >= 0.2 m) and 10/50/90 %% maxima, %d cells x %d members" % (ncell, c.n_members),
            "cells_reaching_0.2m_in_any_member": int(np.count_nonzero(prob > 0))}


def leg_land_cover(FloodEnsemble, W, args):
    """The same grid and ensemble with land cover (Table 1): per-member class
    roughness, runoff coefficient, drainage of hardened ground; first window."""
    import torch
    wl = W.config5(args.ny, args.nx, args.members, with_land_cover=True)
    c = wl.catchments[0]
    ncell = c.ny * c.nx
    ens = FloodEnsemble.from_workload(wl)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ens.step(args.window)
    torch.cuda.synchronize()
    t_step = time.perf_counter() - t0
    led = ens.ledger()
    steps = int(led["steps"].sum())
    ens.close()
    log("land cover leg: %.2f s, %d member steps" % (t_step, steps))
    return {"workload": "first %.0f s of this ensemble with land cover (3 classes, %.0f %% hardened ground)"
                        % (args.window, 100.0 * np.mean(c.land_class == W.CLASS_HARD)),
            "MCUps": steps * ncell / t_step,
            "drained_over_rain": float(led["drain"].sum() / led["rain_in"].sum())}


def leg_streams(FloodEnsemble, W, args):
    """The same grid and ensemble with two stream outlets (inflow hydrographs,
    Sec. 4.1) over its first window, then one filter cycle on the depth gauges and
    the two streamflow sections together with 5 % relative error (Sec. 4.4)."""
    import torch
    wl = W.config5(args.ny, args.nx, args.members, with_inflow=True)
    c = wl.catchments[0]
    ncell = c.ny * c.nx
    ens = FloodEnsemble.from_workload(wl)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ens.step(args.window)
    torch.cuda.synchronize()
    t_step = time.perf_counter() - t0
    led = ens.ledger()
    steps = int(led["steps"].sum())
    K = c.gauges.shape[0]
    y = np.concatenate([np.array([ens.field(i)[c.gauges[:, 0], c.gauges[:, 1]] for i in (0,)]),
                        ens.sections()[:1]], axis=1)[0]
    obs = y * np.random.default_rng(wl.seed + 9).normal(1.0, 0.05, size=y.size)
    floor = np.concatenate([np.full(K, 0.01), np.full(len(c.sections), 0.01)])
    t0 = time.perf_counter()
    neff, _, res = ens.assimilate_obs(0, c.gauges, obs, floor, alpha=0.05, neff_frac=0.8, u0=0.5)
    t_pf = time.perf_counter() - t0
    ens.close()
    log("streams leg: %.2f s stepping, filter on %d depths + %d flows %.4f s" % (t_step, K, len(c.sections), t_pf))
    return {"workload": "first %.0f s of this ensemble with two stream outlets (inflow hydrographs on 4 edge "
                        "links) and 2 streamflow sections" % args.window,
            "MCUps": steps * ncell / t_step,
            "inflow_over_rain": float(led["inflow"].sum() / led["rain_in"].sum()),
            "filter_depths_and_flows_s": t_pf, "filter_neff": neff, "filter_resampled": bool(res)}


class ClockSampler:
    """Samples the GPU compute clock from sysfs in a host thread (read-only; the
    memory clock of this part is fixed).  Reports median / min / max MHz."""

    def __init__(self, period=0.05):
        import glob
        import threading
        paths = sorted(glob.glob("/sys/class/drm/card*/device/pp_dpm_sclk"))
        self.path = paths[0] if paths else None
        self.period = period
        self.samples = []
        self._stop = threading.Event()
        self._thread = threading.Thread(target=self._run, daemon=True)

    def _read(self):
        try:
            for line in open(self.path):
                if line.rstrip().endswith("*"):
                    return float(line.split(":")[1].strip().split("Mhz")[0].split("MHz")[0])
        except (OSError, ValueError, IndexError):
            return None
        return None

    def _run(self):
        while not self._stop.is_set():
            v = self._read()
            if v is not None:
                self.samples.append(v)
            self._stop.wait(self.period)

    def start(self):
        if self.path:
            self._thread.start()
        return self

    def stop(self):
        if not self.path:
            return None
        self._stop.set()
        self._thread.join()
        if not self.samples:
            return None
        v = np.array(self.samples)
        return {"median_MHz": float(np.median(v)), "min_MHz": float(v.min()), "max_MHz": float(v.max()),
                "samples": int(v.size)}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=2)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--config", type=int, default=5)
    ap.add_argument("--ny", type=int, default=2000)
    ap.add_argument("--nx", type=int, default=2000)
    ap.add_argument("--members", type=int, default=96)
    ap.add_argument("--window", type=float, default=600.0, help="simulated seconds per assimilation cycle")
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--cpu-steps", type=int, default=60)
    ap.add_argument("--cpu-cores", type=int, default=0)
    ap.add_argument("--no-kernel-timing", action="store_true")
    ap.add_argument("--no-adjoint", action="store_true")
    ap.add_argument("--adj-window", type=float, default=900.0)
    ap.add_argument("--adj-sample", type=float, default=10.0)
    ap.add_argument("--adj-ckpt", type=int, default=1024)
    ap.add_argument("--adj-reps", type=int, default=2, help="forward and forward + adjoint runs, in turns")
    ap.add_argument("--no-plain", action="store_true")
    ap.add_argument("--plain-members", type=int, default=8)
    ap.add_argument("--no-c4", action="store_true")
    ap.add_argument("--no-products", action="store_true")
    ap.add_argument("--no-land-cover", action="store_true")
    ap.add_argument("--no-streams", action="store_true")
    ap.add_argument("--land-cover", action="store_true",
                    help="with --kernel-only: the ensemble with land cover (Table 1)")
    ap.add_argument("--c4-window", type=float, default=300.0)
    ap.add_argument("--c4-plain-members", type=int, default=2)
    ap.add_argument("--mi", type=int, default=0)
    ap.add_argument("--rows", type=int, default=0)
    ap.add_argument("--cpb", type=int, default=0)
    ap.add_argument("--kernel", type=int, default=0, help="0 autotune, 1 tiled, 2 row-march, 3 vectorised")
    ap.add_argument("--march-rows", type=int, default=0)
    ap.add_argument("--march-members", type=int, default=0)
    ap.add_argument("--kernel-only", type=int, default=0,
                    help="after the warm-up, time this many single steps in which every member steps "
                         "and print their average instead of the benchmark line")
    args = ap.parse_args()

    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) > 1:
        print("bench.py measures one GPU (--gpus 1): the ensemble's members would shard across GPUs with no "
              "communication between filter updates, and only the single-GPU path is timed here.",
              file=sys.stderr)
        sys.exit(2)

    cfg = {"config": args.config, "ny": args.ny, "nx": args.nx, "members": args.members}
    cpu = None
    if not args.no_cpu and not args.kernel_only:
        cores = args.cpu_cores or min(16, os.cpu_count() or 1)
        log("oracle baseline on %d cores" % cores)
        cpu = cpu_baseline(cfg, cores, args.cpu_steps)
        log("oracle baseline %.3e MCU/s" % cpu["value"])

    if args.kernel_only:
        # one step per call: batches of captured steps would add launches with no member left to step
        os.environ["FLOOD_GRAPH_STEPS"] = "1"
    import torch
    import workloads as W
    from paper_2302_08341_amd import FloodEnsemble

    torch.cuda.set_device(0)
    if args.land_cover and not args.kernel_only:
        ap.error("--land-cover times the step kernel only (with --kernel-only); the benchmark line "
                 "carries the land-cover leg in detail")
    wl = (W.config5(args.ny, args.nx, args.members, with_land_cover=True) if args.land_cover
          else W.CONFIGS[args.config](args.ny, args.nx, args.members))
    c = wl.catchments[0]
    N = c.n_members
    ncell = c.ny * c.nx
    K = c.gauges.shape[0]
    sigma = np.full(K, wl.obs_sigma)
    n_cycles = args.warmup + args.steps
    # the storm hour holds n_win windows; cycle k covers window k mod n_win and a
    # cycle at window 0 after the first restarts from the initial state
    n_win = max(1, int(round(wl.t_end / args.window)))
    hour_times = [(j + 1) * args.window for j in range(n_win)]
    win_times = [hour_times[k % n_win] for k in range(n_cycles)]
    n_adj = int(round(args.adj_window / args.adj_sample))
    adj_times = [(i + 1) * args.adj_sample for i in range(n_adj)] if not args.no_adjoint else []
    log("workload ready: %d x %d cells x %d members" % (c.ny, c.nx, N))
    # the filter's observations and draws have their own truth run and random stream,
    # so the timed cycles are the same whichever other legs run
    rng = np.random.default_rng(wl.seed + 7)
    truth = truth_depths(FloodEnsemble, wl, hour_times)
    obs_all = [W.obs_noise(rng, truth[win_times[k]], wl.obs_sigma) for k in range(n_cycles)]
    draws = [W.pf_draws(rng, N) for _ in range(n_cycles)]
    rng_adj = np.random.default_rng(wl.seed + 8)
    obs_adj = ({t: W.obs_noise(rng_adj, v, wl.obs_sigma) for t, v in truth_depths(FloodEnsemble, wl, adj_times).items()}
               if adj_times else {})
    log("truth observations done")
    detail = {}

    # forward + adjoint first: the timed cycles below are then the last full-size step launches
    if adj_times and not args.kernel_only:
        detail["fwd_adj"] = leg_adjoint(FloodEnsemble, wl, obs_adj,
                                        args.adj_window, args.adj_sample, args.adj_ckpt, max(1, args.adj_reps))
    if not args.no_c4 and not args.kernel_only:
        detail["batched_vs_plain_c4"] = leg_c4(FloodEnsemble, W, args.c4_window, args.c4_plain_members)
    if not args.no_products and not args.kernel_only:
        detail["ensemble_products"] = leg_products(FloodEnsemble, wl, args.window)
    if not args.no_land_cover and not args.kernel_only and args.config == 5:
        detail["land_cover"] = leg_land_cover(FloodEnsemble, W, args)
    if not args.no_streams and not args.kernel_only and args.config == 5:
        detail["streams"] = leg_streams(FloodEnsemble, W, args)

    ens = FloodEnsemble.from_workload(wl, member_interleave=args.mi, tile_rows=args.rows,
                                      chunks_per_block=args.cpb, step_kernel=args.kernel,
                                      march_rows=args.march_rows, march_members=args.march_members)
    conf = ens.config()
    ens.snapshot()             # the initial state, restored at the start of every later storm hour
    log("ensemble ready, step kernel %d" % conf["step_kernel"])
    resampled = []
    cycle_log = []
    n_plain = 0 if (args.no_plain or args.kernel_only) else min(args.plain_members, N)
    snap = {}

    restarts = []

    def cycle(k):
        if k and k % n_win == 0:
            ens.restore()
            restarts.append(k)
        s0 = int(ens.ledger()["steps"].sum())
        t0 = time.perf_counter()
        ens.step(win_times[k])
        t1 = time.perf_counter()
        s1 = int(ens.ledger()["steps"].sum())
        if k == 0:
            for m in range(n_plain):
                snap[m] = ens.field(m)
        u0, beta = draws[k]
        neff, anc, res = ens.assimilate(0, c.gauges, obs_all[k], sigma, 0.8, u0, beta)
        t2 = time.perf_counter()
        resampled.append(bool(res))
        cycle_log.append({"window_end_s": win_times[k], "step_s": t1 - t0, "filter_s": t2 - t1,
                          "member_steps": s1 - s0, "neff": float(neff)})

    for k in range(args.warmup):
        cycle(k)
    torch.cuda.synchronize()
    log("warm-up done")
    if args.kernel_only:
        # every launch steps every member: single steps of 0.02 s, shorter than Eq. 4 allows here
        t = win_times[args.warmup - 1] if args.warmup else 0.0
        l0 = ens.ledger()
        ens.timing(1)          # an event pair around every step launch
        for i in range(args.kernel_only):
            ens.step(t + 0.02 * (i + 1))
        ens.timing(0)
        l1 = ens.ledger()
        avg_ms, launches = ens.get_timing()
        steps = int((l1["steps"] - l0["steps"]).sum())
        full = steps // args.kernel_only
        gbs = BYTES_PER_MCU * full * ncell / (avg_ms * 1e-3) / 1e9 if launches == args.kernel_only else None
        print(json.dumps({"kernel_only": True, "members_per_launch": full, "real_launches": args.kernel_only,
                          "timed_launches": launches, "avg_launch_ms": avg_ms, "algorithmic_GBps": gbs,
                          "elementwise_copy_GBps": elementwise_ceiling(torch), "config": ens.config()}))
        return

    if not args.no_kernel_timing:
        ens.timing(2)          # an event pair around every captured batch; the graph path stays on
    torch.cuda.synchronize()
    clocks = ClockSampler().start()
    t0 = time.perf_counter()
    for k in range(args.warmup, n_cycles):
        cycle(k)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    clock_stats = clocks.stop()
    if not args.no_kernel_timing:
        ens.timing(0)
    led1 = ens.ledger()
    avg_ms, launches = ens.get_timing()
    conf_end = ens.config()
    log("timed cycles done: %.2f s" % elapsed)

    # per-cycle counts: a restart sets the ledger's step counters back with the state
    member_steps = int(sum(cl["member_steps"] for cl in cycle_log[args.warmup:]))
    mcu = member_steps * ncell
    value = mcu / elapsed
    mass = float(np.max(np.abs(led1["storage"] - (led1["rain_in"] - led1["outflow"] + led1["clamp"]))
                        / np.maximum(led1["rain_in"], 1e-30)))
    ens.close()

    workload_tag = "urban%dx%dx%d" % (c.ny, c.nx, N)
    kname = KERNEL_NAMES.get(conf["step_kernel"], "k_step")
    roof = None
    if launches:
        mcu_per_launch = mcu / launches
        alg_bytes = BYTES_PER_MCU * mcu_per_launch
        achieved = alg_bytes / (avg_ms * 1e-3) / 1e9
        traffic = measured_traffic(kname, workload_tag, alg_bytes)
        roof = {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": traffic,
                "kernel": KERNEL_TITLES.get(conf["step_kernel"], kname),
                "avg_launch_ms": round(avg_ms, 4), "launches": launches,
                "timing": "a HIP event pair around every captured batch of %d step launches in the timed region "
                          "(the graph path that value is measured on); a step launch's time holds the step kernel, "
                          "which plans its own step, and the gaps between launches" % conf_end["graph_steps"],
                "algorithmic_bytes_per_launch": round(alg_bytes),
                "traffic_over_algorithmic": round(traffic / alg_bytes, 3) if traffic else None,
                "kernel_sources_sha256": kernel_source_hash()}
        detail["step_launches_only_MCUps"] = mcu / (launches * avg_ms * 1e-3)

    if n_plain:
        # plain: one handle and one launch per member over the first window
        c0 = cycle_log[0]
        t_plain, s_plain = 0.0, 0
        exact = True
        for m in range(n_plain):
            e = FloodEnsemble([ensemble_args(c, [m])], wl.rain, rain_interval=wl.rain_interval,
                              real_bytes=wl.real_bytes)
            ta = time.perf_counter()
            e.step(win_times[0])
            t_plain += time.perf_counter() - ta
            s_plain += int(e.ledger()["steps"][0])
            exact &= bool(np.array_equal(e.field(0), snap[m]))
            e.close()
        plain_rate = s_plain * ncell / t_plain
        batched_rate = c0["member_steps"] * ncell / c0["step_s"]
        detail["batched_vs_plain"] = {
            "workload": "first %.0f s of this ensemble from the dry start" % args.window,
            "batched_MCUps": batched_rate, "plain_MCUps": plain_rate, "speedup": batched_rate / plain_rate,
            "plain_sample": "%d members each run alone in its own handle" % n_plain,
            "plain_bit_identical": exact}
        log("plain leg done")

    detail["copy_ceiling_GBps"] = elementwise_ceiling(torch)
    # the step's own access pattern without its arithmetic, halo cells or prologue rows
    from paper_2302_08341_amd import flood as _fl
    pat = {}
    for wps in (0, 4):
        pat[wps] = _fl.flood_probe_stream(c.ny, c.nx, N, conf_end["march_rows"], 5, wps)
    detail["pattern_ceiling"] = {
        "GBps": pat[0][0], "ms_per_launch": pat[0][1],
        "GBps_at_4_waves_per_simd": pat[4][0], "ms_per_launch_at_4_waves_per_simd": pat[4][1],
        "what": "flood_probe_stream: the vectorised step's streams (3 state arrays in and out, bed and roughness "
                "in, 16-byte accesses, %d-row strips of 256 cells) with no arithmetic, all %d members every "
                "launch; at its own occupancy (8 waves per SIMD) and capped at the step kernel's (4)"
                % (conf_end["march_rows"], N)}
    detail["gpu_clock_in_timed_region"] = clock_stats
    detail.update({"member_steps": member_steps, "mcu": mcu, "elapsed_s": elapsed, "cycles": cycle_log[args.warmup:],
                   "resampled": resampled[args.warmup:], "restarts_at_cycles": restarts,
                   "mass_balance_rel_since_last_restart": mass,
                   "paper_context": "8x P100: 4.69e10 MCU/s (96 x 4.0 M cells x 14,400 steps in 118 s)"})

    out = {
        "metric": "member-cell-updates/s fwd & fwd+adj; % HBM peak; batched vs plain, 96x4M",
        "value": value,
        "unit": "MCU/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": elapsed / args.steps * 1e3,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32" if wl.real_bytes == 4 else "f64",
        "data": "synthetic",
        "config": {"workload": "urban %dx%d cells x %d members, FP32, PF every %.0f s (%d gauges); one step = "
                               "one %.0f s assimilation cycle" % (c.ny, c.nx, N, args.window, K, args.window),
                   "cells": ncell, "members": N, "window_s": args.window,
                   "storm_s": wl.t_end, "timed_windows_end_s": win_times[args.warmup:],
                   "member_interleave": conf["member_interleave"], "tile_rows": conf["tile_rows"],
                   "chunks_per_block": conf["chunks_per_block"], "step_kernel": conf["step_kernel"],
                   "march_rows": conf["march_rows"], "march_members": conf["march_members"],
                   "march_order": conf["march_order"]},
        "roofline": roof,
        "cpu_baseline": cpu,
        "detail": detail,
    }
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
