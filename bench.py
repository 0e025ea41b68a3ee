"""Benchmark of the octahedron-model hot path on one MI355X.

Workload: 2^17 x 2^17 periodic lattice (1.7e10 sites, 4.3 GB packed), flat
zig-zag start, p = 1, q = 0, seed 1, with the exact width measured at the
paper's sampling times t_{i+1} = (t_i + 10) e^m, m = 0.01 (Sec. III).  One
step is one MCS: a full sweep (every block staged in LDS, 64 in-LDS steps,
aligned store) plus the width whenever a sampling time falls on it.  W
untimed warmup sweeps run first; then exactly K steps are timed.

Prints one JSON line: whole-job site updates/s, the sweep kernel's HBM
roofline fraction (algorithmic 0.5 B per site update over the kernel's mean
launch time, measured with HIP events on the simulation's stream), and the
oracle timed on the host cores on a bounded sample of the same workload.
"""
import argparse
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0  # MI355X HBM3E, published
# HBM bytes per sweep launch at 2^17 x 2^17 from rocprofv3 FETCH_SIZE and
# WRITE_SIZE, each scaled by its reading for a plain 1 GiB copy
# (profiles/sweep_kernel_L131072_hbm_counters.md).  Reported only while the
# sweep sources hash to the value the counters were taken on.
TRAFFIC_MEASURED = {"sources_sha256_16": "1aa4edb808fdc8b1", "L": 1 << 17, "bytes": 8.625e9}
# VALU issue per site update of the growth sweep from rocprofv3 SQ_INSTS_VALU
# and SQ_INSTS_VALU_INT64 (profiles/sweep_kernel_L131072_sq_counters.md): 20.8
# wave instructions per 64 updates plus 2.7 for the second issue cycle of the
# 64-bit multiplies.  Against 256 CUs x 64 lanes x 2.4 GHz of 32-bit lanes
# this gives the ALU ceiling of the sweep; same source key as the traffic.
VALU_MEASURED = {"sources_sha256_16": "1aa4edb808fdc8b1", "lane_ops_per_update": 23.5}
ALU_PEAK_TOPS = 256 * 64 * 2.4e9 / 1e12  # 39.3 T 32-bit lane operations/s
SWEEP_SOURCES = ("sweep_core.h", "sweep.hip", "okpz_internal.h")
METRIC = "site updates/s (+% HBM roofline) at L=2^17; realizations/s batched vs plain; serving p50/p99"


def log(msg):
    """Progress of the legs on stderr (the JSON line stays alone on stdout)."""
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


METRICS_PATH = None  # --metrics-jsonl: one JSON row per finished leg


def metric_row(leg, fields):
    """Append one row (wall-clock time, leg name and the leg's figures) to
    the --metrics-jsonl file, when one was given."""
    if METRICS_PATH is None:
        return
    row = {"time": time.time(), "leg": leg}
    row.update(fields)
    with open(METRICS_PATH, "a") as f:
        f.write(json.dumps(row) + "\n")


def single_core_rate(L, budget_s):
    """Oracle site updates/s of a flat L x L lattice (p = 1, q = 0, seed 1)
    on one host core, the paper's non-parallel reference point (Sec. II)."""
    import oracle

    threads = oracle.num_threads()
    oracle.set_num_threads(1)
    try:
        lat = oracle.flat(L, L)
        H, s, t0 = 0, 0, time.perf_counter()
        while True:
            H = oracle.sweep(lat, 1.0, 0.0, 1, s, H)
            s += 1
            el = time.perf_counter() - t0
            if el >= budget_s or s >= 400:
                break
    finally:
        oracle.set_num_threads(threads)
    return {"L": L, "mcs": s, "seconds": el, "value": L * L * s / el}


def cpu_baseline(okpz, sim, seed, p, q, budget_s=12.0, max_block_rows=192, chunk=16):
    """The oracle, untuned, on the host cores, on a bounded sample of the
    benchmark's own workload: one sweep (the next MCS of the 2^17 run) of a
    band of whole block rows, taken from the GPU's lattice before that sweep
    and advanced with the oracle's window sweep (OpenMP over the band's
    blocks).  The oracle's result is compared bit for bit with the GPU's
    lattice after the sweep.  Then one core on flat 4096^2 and 8192^2
    lattices (the paper's CPU reference is one core; Sec. II sees a jump
    between log2 L = 12 and 13 when the lattice leaves the CPU's cache)."""
    import numpy as np

    import oracle

    L = sim.Lx
    Bx, By, _ = oracle.geometry(L, L)
    s = sim.time()
    sx, sy = oracle.block_shift(seed, s, Bx, By)
    nb = min(max_block_rows, L // By)
    chunk = min(chunk, nb)
    y0 = sy  # block row 0 of sweep s starts at row sy
    pre = [sim.get_rows(y0 + k * By, chunk * By) for k in range(0, nb, chunk)]
    sim.sweep(1)
    threads = oracle.num_threads()
    done, el, checked = 0, 0.0, 0
    for k, rows in enumerate(pre):
        w = oracle.Window(rows, 0, (y0 + k * chunk * By) % L, L, L, 0)
        t0 = time.perf_counter()
        w.sweep(p, q, seed, s)
        el += time.perf_counter() - t0
        vx0, vy0, vx1, vy1 = w.valid
        done += (vx1 - vx0) * (vy1 - vy0)
        post = sim.get_rows(y0 + k * chunk * By, chunk * By)
        if not np.array_equal(post[vy0:vy1, vx0:vx1], rows[vy0:vy1, vx0:vx1]):
            raise AssertionError(f"GPU sweep {s} differs from the oracle in block rows "
                                 f"{k * chunk}..{(k + 1) * chunk - 1}")
        checked += (vx1 - vx0) // Bx * ((vy1 - vy0) // By)
        if el >= budget_s:
            break
    del pre
    single = [single_core_rate(n, budget_s / 4) for n in (4096, 8192)]
    return {"value": done / el, "unit": "site updates/s", "cores": threads, "kind": "oracle",
            "sample": f"sweep {s} (MCS {s + 1}) of the {L}x{L} run, {checked} blocks of "
                      f"{Bx}x{By} ({done} site updates) in whole block rows from the GPU's "
                      f"lattice before the sweep, oracle window sweep with OpenMP over blocks, "
                      f"{el:.1f} s; result equal bit for bit to the GPU's",
            "single_core": {"cores": 1, "value": single[0]["value"],
                            "sample": "flat 4096x4096, p=1 q=0, seed 1",
                            "by_L": single}}


def ensemble_jobs(scale):
    """The finite-size-scaling ensemble: 512 realizations, L = 32 (1 + r mod 32)
    (32 sizes 32 .. 1024, 16 each), p = 1, q = 0, seed 1000 + r, run to
    t = scale * 20 L^1.6 MCS (scale = 1 is the full steady-state run)."""
    jobs = []
    for r in range(512):
        L = 32 * (1 + r % 32)
        jobs.append((L, L, 1.0, 0.0, 1000 + r, max(1, int(math.ceil(scale * 20 * L ** 1.6)))))
    return jobs


def batch_leg(scale, m=0.001, plain_scale=None):
    """Realizations/s of the ensemble: one persistent launch (after the
    autotuner picks the mapping) vs a per-realization loop of okpz_sweep /
    okpz_width launches, same jobs, same sampling times, same GPU.

    plain_scale: time the per-realization loop on one realization per size
    at t = plain_scale x 20 L^1.6 instead of all 512 at `scale`, and
    extrapolate: the loop's time is one launch per MCS and per sample plus a
    fixed cost per realization, so it grows linearly in t and in the number
    of realizations (16 per size)."""
    from paper_1110_6745_amd import okpz

    jobs = ensemble_jobs(scale)
    work = sum(L * L * t for L, _, _, _, _, t in jobs)
    b = okpz.Batch(jobs, m)
    t0 = time.perf_counter()
    # the trial runs the longest job 1/20 of its length, at most 20 000 MCS
    # (six candidates: at most a few percent of a full-length run)
    mapping = b.autotune(max(2, min(20000, int(max(t for *_, t in jobs)) // 20)))
    tune_s = time.perf_counter() - t0
    t0 = time.perf_counter()
    if scale >= 0.05:
        # a long run reports its progress between slices of about 20 s
        dev_ms = b.run(slice_ms=20000.0, progress=lambda d: log(
            f"ensemble: {d} of {len(jobs)} realizations done, {time.perf_counter() - t0:.0f} s"))
    else:
        dev_ms = b.run()
    batched_s = time.perf_counter() - t0
    log(f"ensemble: batched {batched_s:.2f} s + autotune {tune_s:.2f} s (mapping {mapping})")
    # spot check: one job of each size class run alone gives the same samples
    spot = {}
    for r in (0, 31):
        L, _, p, q, seed, t_max = jobs[r]
        sim = okpz.okpz_init(L, L, p, q, seed)
        ref = [(t,) + sim.width(t) for t in okpz.sampling_times(t_max, m)]
        sim.free()
        t, s1, s2 = b.samples(r)
        spot[r] = list(zip(t.tolist(), s1.tolist(), s2.tolist()))
        assert spot[r] == ref, "batched job differs"
    hist_L = 1024
    # steady state: W^2 of L = 1024 saturates near t_x ~ L^z, z ~ 1.6 (Sec. IV);
    # samples from 2 L^1.6 on when the run reaches it, else the growth regime
    t_sat = int(2 * hist_L ** 1.6)
    t_from = t_sat if jobs[31][5] > t_sat else jobs[31][5] // 2
    regime = "steady state (t >= 2 L^1.6)" if t_from == t_sat else "growth regime (t < 2 L^1.6)"
    n_cum, _, kappa = b.w2_cumulants(hist_L, hist_L, t_from)
    hist_hi = float(math.ceil(3.0 * kappa[0]))  # three times the mean W^2
    counts, under, over = b.w2_histogram(hist_L, hist_L, t_from, 0.0, hist_hi, 40)
    b.free()
    if plain_scale is None:
        t0 = time.perf_counter()
        for L, _, p, q, seed, t_max in jobs:
            sim = okpz.okpz_init(L, L, p, q, seed)
            for t in okpz.sampling_times(t_max, m):
                sim.width(t)
            sim.free()
        plain_s = time.perf_counter() - t0
        plain_how = "measured: all 512 realizations, one after another"
        # a stronger loop: 16 host threads, each running whole realizations
        # on its own simulation (own stream), so that the short, latency-bound
        # launch sequences of different realizations overlap on the device
        from concurrent.futures import ThreadPoolExecutor

        def one(job):
            L, _, p, q, seed, t_max = job
            sim = okpz.okpz_init(L, L, p, q, seed)
            out = [(t,) + sim.width(t) for t in okpz.sampling_times(t_max, m)]
            sim.free()
            return out

        t0 = time.perf_counter()
        with ThreadPoolExecutor(16) as ex:
            res = list(ex.map(one, jobs))
        streams_s = time.perf_counter() - t0
        for r, ref in spot.items():
            assert res[r] == ref, "threaded loop differs"
    else:
        sample = ensemble_jobs(plain_scale)[:32]
        t0 = time.perf_counter()
        for L, _, p, q, seed, t_max in sample:
            sim = okpz.okpz_init(L, L, p, q, seed)
            for t in okpz.sampling_times(t_max, m):
                sim.width(t)
            sim.free()
        sample_s = time.perf_counter() - t0
        plain_s = sample_s * 16 * scale / plain_scale
        plain_how = (f"extrapolated: one realization per size at t = {plain_scale:g} x 20 L^1.6 "
                     f"took {sample_s:.2f} s, x 16 per size x {scale / plain_scale:g} in t")
    return {"workload": f"512 realizations, L = 32..1024 step 32 (16 each), p=1 q=0, "
                        f"t = {scale:g} x 20 L^1.6 MCS (scale {scale:g} of the full run), "
                        f"W^2 at t_(i+1)=(t_i+10)e^{m:g}",
            "scale": scale, "site_updates": work, "batched_s": batched_s,
            "batched_device_ms": dev_ms, "autotune_s": tune_s,
            "plain_s": plain_s, "plain": plain_how,
            **({"plain_16_streams_s": streams_s,
                "plain_16_streams": "measured: all 512 realizations, 16 host threads each running "
                                    "whole realizations on its own simulation and stream",
                "speedup_vs_16_streams": streams_s / batched_s} if plain_scale is None else {}),
            "realizations_per_s_batched": 512 / batched_s,
            "realizations_per_s_batched_incl_autotune": 512 / (batched_s + tune_s),
            "realizations_per_s_plain": 512 / plain_s, "speedup": plain_s / batched_s,
            "speedup_incl_autotune": plain_s / (batched_s + tune_s),
            "batched_site_updates_per_s": work / batched_s,
            "mapping": {"threads": mapping[0], "workgroups": mapping[1]},
            "w2_histogram_L1024": {"t_from": t_from, "regime": regime, "lo": 0.0, "hi": hist_hi,
                                   "counts": counts.tolist(), "under": under, "over": over},
            "w2_cumulants_L1024": {"t_from": t_from, "regime": regime, "samples": n_cum,
                                   "kappa": kappa.tolist()}}


def medium_leg(t_max=10000, seeds=8, n_times=64):
    """The medium workload: 4096 x 4096 lattices, p = 1, q = 0 and p = 0.95,
    q = 0.05, 8 seeds each, 10^4 MCS, exact W^2 at 64 log-spaced times (the
    Sec. III recurrence with the m that gives 64 times up to t_max), as one
    persistent batch."""
    from paper_1110_6745_amd import okpz

    m_lo, m_hi = 1e-3, 10.0
    for _ in range(60):  # bisect m for n_times sampling times
        m = math.sqrt(m_lo * m_hi)
        if len(okpz.sampling_times(t_max, m)) > n_times:
            m_lo = m
        else:
            m_hi = m
    m = m_hi
    times = okpz.sampling_times(t_max, m)
    L = 4096
    jobs = [(L, L, p, q, 1 + r, t_max) for p, q in ((1.0, 0.0), (0.95, 0.05)) for r in range(seeds)]
    b = okpz.Batch(jobs, m)
    t0 = time.perf_counter()
    dev_ms = b.run()
    el = time.perf_counter() - t0
    w2 = {}
    for j, (_, _, p, q, _, _) in enumerate(jobs):
        t, s1, s2 = b.samples(j)
        w = [(L * L * int(a2) - int(a1) * int(a1)) / (L * L) ** 2 for a1, a2 in zip(s1, s2)]
        w2.setdefault(f"p={p:g} q={q:g}", []).append(w)
    b.free()
    work = len(jobs) * L * L * t_max
    return {"workload": f"{len(jobs)} realizations of {L}x{L}: (p,q) = (1,0) and (0.95,0.05), "
                        f"{seeds} seeds each, {t_max} MCS, W^2 at {len(times)} times "
                        f"(t_(i+1)=(t_i+10)e^m, m={m:.4f})",
            "seconds": el, "device_ms": dev_ms, "site_updates_per_s": work / el,
            "realizations_per_s": len(jobs) / el, "times": times,
            "mean_w2": {k: [sum(c) / len(c) for c in zip(*v)] for k, v in w2.items()}}


def serve_leg(n_jobs=64, rate=50.0, seed=7):
    """Continuous batching of a served job stream (Poisson arrivals, mean
    1/rate s; L = 2^U{6..13}; p ~ U[0.6, 1]; q = 0 or 1 - p; t_max
    log-uniform in [10^3, 10^4]; job seed = index + 1).  Runs the stream at
    `rate` (above capacity: the achieved rate is the serving capacity) and
    again at half of that measured capacity; reports p50/p99 latency
    (finish - arrival), jobs/s and achieved vs offered site updates/s."""
    import numpy as np

    from paper_1110_6745_amd import okpz

    def one(r):
        stream = okpz.job_stream(n_jobs, r, seed)
        work = sum(L * L * t for _, (L, _, _, _, _, t) in stream)
        sv = okpz.Server(hbm_budget=64 << 30, max_slots=64, quantum_sites=1 << 31, m=0.01)
        t0 = sv.now() + 0.05
        ids = [sv.submit(job, t0 + a) for a, job in stream]
        sv.drain(timeout_s=300.0)
        info = [sv.job(i) for i in ids]
        st = sv.stats()
        sv.free()
        lat = np.array([j["finish"] - j["arrival"] for j in info])
        span = max(j["finish"] for j in info) - t0
        offered_span = stream[-1][0]
        return {"jobs": n_jobs, "rate_jobs_per_s": r, "offered_site_updates_per_s": work / offered_span,
                "achieved_site_updates_per_s": work / span, "jobs_per_s": n_jobs / span,
                "latency_p50_s": float(np.percentile(lat, 50)),
                "latency_p99_s": float(np.percentile(lat, 99)),
                "quanta": st["quanta"], "device_s": st["device_ms"] / 1e3, "wall_s": span}

    out = {"workload": f"{n_jobs} jobs, Poisson arrivals, L=2^U{{6..13}}, p~U[0.6,1], q=0 or 1-p, "
                       f"t_max log-uniform [1e3,1e4], W^2 at t_(i+1)=(t_i+10)e^0.01, seed {seed}",
           "at_rate": one(rate)}
    capacity = out["at_rate"]["achieved_site_updates_per_s"]
    stream = okpz.job_stream(n_jobs, 1.0, seed)
    per_job = sum(L * L * t for _, (L, _, _, _, _, t) in stream) / n_jobs
    out["at_half_capacity"] = one(0.5 * capacity / per_job)
    return out


def sweep_sources_hash():
    import hashlib

    h = hashlib.sha256()
    for f in SWEEP_SOURCES:
        with open(os.path.join(ROOT, "paper_1110_6745_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def copy_calibration(nbytes=1 << 30):
    """A plain device copy of known size, for scaling the HBM byte counters."""
    import torch

    a = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    b = torch.empty_like(a)
    b.copy_(a)
    torch.cuda.synchronize()
    del a, b


def size_scan(okpz, sizes, budget_ms=150.0):
    """Device time per MCS of one lattice per size (flat start, p = 1, q = 0,
    seed 1), from HIP events on the lattice's stream: the per-lattice path
    across sizes, where small lattices cannot fill the device."""
    import torch

    out = []
    for L in sizes:
        sim = okpz.okpz_init(L, L, 1.0, 0.0, 1)
        sim.sweep(2)
        st = torch.cuda.ExternalStream(sim.stream())
        n = max(4, min(4000, int(budget_ms * 1.3e9 / (L * L))))
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(st)
        sim.sweep(n)
        e1.record(st)
        e1.synchronize()
        ms = e0.elapsed_time(e1) / n
        out.append({"L": L, "mcs": n, "ms_per_mcs": ms, "site_updates_per_s": L * L / (ms * 1e-3),
                    "ns_per_site": ms * 1e6 / (L * L)})
        sim.free()
    return out


def delayed_leg(okpz, L, p, q, seed, steps, warmup=2):
    """The paper's own thread-level contract, delayed cell borders (Sec. II),
    on a second L x L lattice: mean sweep time from HIP events on the
    lattice's stream and its HBM roofline fraction (0.5 B per site update)."""
    import torch

    sim = okpz.okpz_init(L, L, p, q, seed)
    sim.set_cell_borders(okpz.OKPZ_CELLS_DELAYED)
    sim.sweep(warmup)
    st = torch.cuda.ExternalStream(sim.stream())
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
          for _ in range(steps)]
    for a, b in ev:
        a.record(st)
        sim.sweep(1)
        b.record(st)
    ev[-1][1].synchronize()
    sim.free()
    ms = sum(a.elapsed_time(b) for a, b in ev) / steps
    gbs = 0.5 * L * L / (ms * 1e-3) / 1e9
    return {"cell_borders": "delayed", "workload": f"{L}x{L}, flat init, p=1 q=0, seed 1, "
                                                   f"MCS {warmup}..{warmup + steps}",
            "sweep_kernel_ms": ms, "sweep_site_updates_per_s": L * L / (ms * 1e-3),
            "roofline": {"bound": "hbm", "achieved": gbs, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                         "frac": gbs / HBM_PEAK_GBS}}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--L", type=int, default=1 << 17)
    ap.add_argument("--threads", type=int, default=1024, help="sweep workgroup size")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--calib", action="store_true", help="run a 1 GiB copy first (counters)")
    ap.add_argument("--batch-scale", type=float, default=0.005,
                    help="ensemble leg: fraction of the full t = 20 L^1.6 (0 skips it)")
    ap.add_argument("--serve-jobs", type=int, default=64, help="serving leg: jobs (0 skips it)")
    ap.add_argument("--cell-borders", choices=("dead", "delayed"), default="dead",
                    help="thread-cell borders of the tiled dynamics")
    ap.add_argument("--size-scan", type=int, default=1,
                    help="1: time one lattice per size 2^8 .. 2^16 (0 skips it)")
    ap.add_argument("--in-place", action="store_true",
                    help="one lattice copy updated in place (fits 2^20 x 2^20 on one GPU)")
    ap.add_argument("--psd-calls", type=int, default=3,
                    help="spectrum of the final surface: timed calls (0 skips it)")
    ap.add_argument("--delayed-steps", type=int, default=20,
                    help="delayed-border leg: timed MCS of a second lattice (0 skips it)")
    ap.add_argument("--plain-scale", type=float, default=None,
                    help="ensemble leg: extrapolate the per-realization loop from one "
                         "realization per size at this fraction of 20 L^1.6")
    ap.add_argument("--medium", action="store_true",
                    help="also run the 4096^2 workload (2 x 8 seeds, 10^4 MCS) as one batch")
    ap.add_argument("--w2-out", default=None,
                    help="write every width sample of the timed steps to this JSON file")
    ap.add_argument("--metrics-jsonl", default=None,
                    help="append one JSON row per finished leg to this file")
    args = ap.parse_args()
    global METRICS_PATH
    METRICS_PATH = args.metrics_jsonl
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (asked for {args.gpus}); independent "
              "realizations shard trivially and one lattice is not split across GPUs here",
              file=sys.stderr)
        sys.exit(2)

    import torch

    from paper_1110_6745_amd import okpz

    torch.cuda.set_device(0)
    if args.calib:
        copy_calibration()
    L = args.L
    p, q, seed = 1.0, 0.0, 1
    N = L * L
    stream = torch.cuda.current_stream()
    if args.in_place:
        nbytes = okpz.okpz_required_bytes_in_place(L, L)
        buf = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        sim = okpz.okpz_init_in_place(L, L, p, q, seed, buf.data_ptr(), nbytes, stream.cuda_stream)
    else:
        nbytes = okpz.okpz_required_bytes(L, L)
        buf = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        sim = okpz.okpz_init_on(L, L, p, q, seed, buf.data_ptr(), nbytes, stream.cuda_stream)
    sim.set_threads(args.threads)
    if args.cell_borders == "delayed":
        sim.set_cell_borders(okpz.OKPZ_CELLS_DELAYED)

    sim.sweep(args.warmup)
    torch.cuda.synchronize()
    t_lo, t_hi = args.warmup, args.warmup + args.steps
    samples = set(t for t in okpz.sampling_times(t_hi, 0.01) if t_lo < t <= t_hi)
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
          for _ in range(args.steps)]
    widths = []

    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(args.steps):
        ev[i][0].record(stream)
        sim.sweep(1)
        ev[i][1].record(stream)
        if (t_lo + i + 1) in samples:
            widths.append((t_lo + i + 1,) + sim.width())
        if args.steps >= 1000 and (i + 1) % 500 == 0:
            log(f"step {t_lo + i + 1} of {t_hi}")
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0

    sweep_ms = sum(a.elapsed_time(b) for a, b in ev) / args.steps
    value = N * args.steps / elapsed
    achieved_gbs = 0.5 * N / (sweep_ms * 1e-3) / 1e9
    w2 = [(t, (N * s2 - s1 * s1) / (N * N)) for t, s1, s2 in widths]
    if args.w2_out:
        late = ev[-min(100, args.steps):]
        with open(args.w2_out, "w") as f:
            json.dump({"L": L, "p": p, "q": q, "seed": seed, "t_lo": t_lo, "t_hi": t_hi,
                       "cell_borders": args.cell_borders, "sweep_ms_mean": sweep_ms,
                       "sweep_ms_last_100": sum(a.elapsed_time(b) for a, b in late) / len(late),
                       "wall_s": elapsed,
                       "samples": [{"t": t, "sum_h": s1, "sum_h2": s2,
                                    "w2": (N * s2 - s1 * s1) / (N * N), "mean_h": s1 / N}
                                   for t, s1, s2 in widths]}, f)
    traffic = None
    src_key = sweep_sources_hash()
    if (L == TRAFFIC_MEASURED["L"] and not args.in_place and args.cell_borders == "dead"
            and src_key == TRAFFIC_MEASURED["sources_sha256_16"]):
        traffic = TRAFFIC_MEASURED["bytes"]
    alu = None
    if (args.cell_borders == "dead" and not args.in_place and args.threads == 1024
            and src_key == VALU_MEASURED["sources_sha256_16"]):
        ops = N / (sweep_ms * 1e-3) * VALU_MEASURED["lane_ops_per_update"] / 1e12
        alu = {"bound": "alu", "achieved": ops, "peak": ALU_PEAK_TOPS, "unit": "T lane-ops/s",
               "frac": ops / ALU_PEAK_TOPS,
               "lane_ops_per_update": VALU_MEASURED["lane_ops_per_update"]}

    out = {
        "metric": METRIC,
        "value": value,
        "unit": "site updates/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": 1e3 * elapsed / args.steps,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "u32",
        "data": "synthetic",
        "config": {"workload": f"octahedron model {L}x{L} periodic, flat init, p=1 q=0, seed 1, "
                               f"MCS {t_lo}..{t_hi}, exact W^2 at t_(i+1)=(t_i+10)e^0.01",
                   "Lx": L, "Ly": L, "p": p, "q": q, "seed": seed,
                   "width_samples": len(widths), "threads_per_workgroup": args.threads,
                   "cell_borders": args.cell_borders,
                   "lattice_copies": 1 if args.in_place else 2},
        "sweep_kernel_ms": sweep_ms,
        "sweep_site_updates_per_s": N / (sweep_ms * 1e-3),
        # the sweep is bound by VALU issue, not HBM (8.5 % of it): with its
        # instruction count measured for these sources, the roofline is the
        # ALU one; the HBM fraction is kept beside it
        "roofline": ({**alu, "traffic": traffic} if alu else
                     {"bound": "hbm", "achieved": achieved_gbs, "peak": HBM_PEAK_GBS,
                      "unit": "GB/s", "frac": achieved_gbs / HBM_PEAK_GBS, "traffic": traffic}),
        "roofline_hbm": {"bound": "hbm", "achieved": achieved_gbs, "peak": HBM_PEAK_GBS,
                         "unit": "GB/s", "frac": achieved_gbs / HBM_PEAK_GBS, "traffic": traffic},
        "w2_last": w2[-1] if w2 else None,
    }
    if args.psd_calls > 0 and L & (L - 1) == 0:
        sim.psd()  # the first call allocates its scratch
        t0 = time.perf_counter()
        for _ in range(args.psd_calls):
            sx, sy = sim.psd()
        psd_ms = 1e3 * (time.perf_counter() - t0) / args.psd_calls
        out["psd"] = {"L": L, "t": t_hi, "ms_per_call": psd_ms, "calls": args.psd_calls,
                      "S_direction_avg_n1_n2": [0.5 * (sx[1] + sy[1]), 0.5 * (sx[2] + sy[2])]}
        log(f"spectrum: {psd_ms:.3f} ms per call")
    log(f"sweep leg: {sweep_ms:.3f} ms per MCS, {value:.4g} site updates/s")
    metric_row("sweep", {"L": L, "steps": args.steps, "ms_per_step": out["ms_per_step"],
                         "sweep_kernel_ms": sweep_ms, "site_updates_per_s": value,
                         "hbm_frac": out["roofline_hbm"]["frac"], "width_samples": len(widths)})
    if not args.no_cpu_baseline and args.cell_borders == "dead":
        out["cpu_baseline"] = cpu_baseline(okpz, sim, seed, p, q)
        log("cpu baseline done")
        metric_row("cpu_baseline", {"site_updates_per_s": out["cpu_baseline"]["value"],
                                    "cores": out["cpu_baseline"]["cores"],
                                    "single_core": out["cpu_baseline"]["single_core"]["value"]})
    sim.free()
    del buf
    torch.cuda.synchronize()
    if args.delayed_steps > 0 and args.cell_borders == "dead" and not args.in_place:
        out["delayed_cells"] = delayed_leg(okpz, L, p, q, seed, args.delayed_steps)
        log(f"delayed-border leg: {out['delayed_cells']['sweep_kernel_ms']:.3f} ms per MCS")
        metric_row("delayed_cells", {k: out["delayed_cells"][k]
                                     for k in ("sweep_kernel_ms", "sweep_site_updates_per_s")})
    if args.size_scan:
        out["size_scan"] = size_scan(okpz, [1 << k for k in range(8, 17)])
        log("size scan done")
        for r in out["size_scan"]:
            metric_row("size_scan", r)
    if args.batch_scale > 0:
        out["batched_vs_plain"] = batch_leg(args.batch_scale, plain_scale=args.plain_scale)
        bp = out["batched_vs_plain"]
        log(f"ensemble leg: speedup {bp['speedup']:.3g}"
            + (f", {bp['speedup_vs_16_streams']:.3g} against 16 streams" if "speedup_vs_16_streams" in bp else ""))
        metric_row("ensemble", {k: bp[k] for k in ("scale", "batched_s", "autotune_s", "plain_s",
                                                   "speedup", "batched_site_updates_per_s")})
    if args.medium:
        out["medium"] = medium_leg()
        log(f"medium leg: {out['medium']['seconds']:.2f} s")
        metric_row("medium", {k: out["medium"][k] for k in ("seconds", "site_updates_per_s")})
    if args.serve_jobs > 0:
        out["serving"] = serve_leg(args.serve_jobs, 50.0)
        log("serving leg done")
        for k in ("at_rate", "at_half_capacity"):
            metric_row("serving_" + k, out["serving"][k])
    if "cpu_baseline" in out:
        one = out["cpu_baseline"]["single_core"]["value"]
        out["paper_context"] = {
            "speedup_vs_one_cpu_core": 240,
            "hardware": "NVIDIA Tesla C2070 (Fermi) against one core of an Intel Core i5 750 "
                        "at 3 GHz running non-parallel code; time per MCS, bare simulation "
                        "time without host-device transfers (abstract, Sec. II, Sec. V)",
            "this_run_vs_one_host_core": out["sweep_site_updates_per_s"] / one,
            "note": "context only: different hardware, RNG and CPU code"}
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
