#!/usr/bin/env python3
"""Throughput of the exact edge-posterior path on one MI355X.

One step = one whole solve (local scores, alpha, forward and backward
sweeps, Gamma, edge sums and invariants) over one synthetic dataset that is
already resident in HBM. Rate = n * 2^n lattice cells per second.

Default headline: n = 30 binary variables, m = 500 samples, d = 3, FP32-scaled
form. Comparison lines time the plain FP64 log-space form and n = 25. The CPU
baseline is the oracle (FP64 log-space, OpenMP) on a bounded sample of the
same dataset.

Prints one JSON line.
"""
import argparse
import hashlib
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "n·2^n DP cells/s at n=25,30 (FP32-scaled vs FP64); served solves/s + p99"
HBM_PEAK_GBS = 8000.0
STORE_BYTES = {"fp32": 5, "fp64": 8}


# Kernels timed alone by the phase timer (one launch each per solve) and the
# timer entry that brackets each.
SINGLE_LAUNCH = {"alpha_tile": "k_alpha_lin", "gamma_tile": "k_gamma_tile_lin"}


def kernel_bytes(phase, n, prec):
    """Algorithmic HBM bytes of one launch, E bytes per stored value: the
    alpha tile kernel writes n 2^(n-1) entries; the Gamma in-tile kernel consumes, for
    every endpoint v and every S not containing v, L(S) and Rp(S+v): 2E per
    (v, S) pair, n 2^(n-1) pairs."""
    E = STORE_BYTES[prec]
    A = n * 2 ** (n - 1)
    if phase == "alpha_tile":
        return E * A
    if phase == "gamma_tile":
        return 2 * E * A
    raise ValueError(phase)


# Variants of a comparison line: environment settings read by the library's
# plan (at each call), so the same entry point times another form.
VARIANTS = {
    "": {},
    # alpha never materialised: the sweeps rebuild it from 9-bit block seeds
    # (the library's choice only where alpha would not fit the device)
    "fused": {"BN_FUSED_ALPHA": "1"},
    # alpha materialised whatever the size (the default up to n = 31)
    "mat": {"BN_FUSED_ALPHA": "0"},
    # no linear tiles: every zeta step in the FP32-scaled form itself (FP32
    # significand adds with exponent alignment), alpha materialised
    "nolin": {"BN_LINEAR_TILES": "0"},
}


def measure(bn, torch, datagen, name, prec, steps, warmup, variant=""):
    env = VARIANTS[variant]
    saved = {k: os.environ.get(k) for k in env}
    os.environ.update(env)
    try:
        return _measure(bn, torch, datagen, name, prec, steps, warmup, variant)
    finally:
        for k, v in saved.items():
            if v is None:
                os.environ.pop(k, None)
            else:
                os.environ[k] = v


def _measure(bn, torch, datagen, name, prec, steps, warmup, variant):
    ds, p = datagen.workload(name)
    n, m, d = ds.n, ds.m, p["d"]
    ws = torch.empty(bn.workspace_bytes(n, d, m, prec), dtype=torch.uint8, device="cuda")
    data = torch.from_numpy(ds.data).cuda()
    post = torch.empty((n, n), dtype=torch.float64, device="cuda")
    diag = torch.zeros(8, dtype=torch.float64, device="cuda")
    timers = [bn.Timer() for _ in range(warmup + steps)]

    def solve(k):
        bn.edge_posteriors_dev(data, ds.arity, d, prec, ws, post, diag, ess=p["ess"],
                               timer=timers[k])

    for k in range(warmup):
        solve(k)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for k in range(steps):
        solve(warmup + k)
    torch.cuda.synchronize()
    sec = time.perf_counter() - t0
    ph = [timers[warmup + k].read() for k in range(steps)]
    phases = {key: sum(x[key] for x in ph) / steps for key in ph[0]}
    dg = diag.cpu().tolist()
    res = dict(workload=name, precision=prec, variant=variant or "default", n=n, m=m, d=d,
               steps=steps, warmup=warmup, workspace_bytes=ws.numel(),
               seconds=sec, ms_per_step=1e3 * sec / steps,
               cells_per_s=n * 2 ** n * steps / sec, phases_ms=phases, log_LV=dg[0],
               max_invariant_residual=dg[1], saturated=int(dg[2]), flushed=int(dg[3]),
               fallback=int(dg[7]), post=post.cpu().numpy())
    # the library's plan holds alpha (5 bytes per entry) unless the fused
    # sweeps run: a smaller workspace means alpha is never materialised
    res["fused"] = prec == "fp32" and res["workspace_bytes"] < 5 * n * 2 ** (n - 1)
    for t in timers:
        t.close()
    del ws, data, post, diag
    torch.cuda.empty_cache()
    return res


def kernel_source_digest():
    """SHA-256 over the kernel sources: a counter record holds only for the
    kernels it was taken on."""
    h = hashlib.sha256()
    for name in ("bn_kernels.hip", "bn_kernels.h", "bn_device.h", "bn_math.h"):
        with open(os.path.join(ROOT, "paper_1408_1664_amd", "csrc", name), "rb") as f:
            h.update(f.read())
    return h.hexdigest()


def counter_traffic(kernel, workload, prec):
    """HBM bytes per launch of `kernel` from a counter record under profiles/
    (a line 'traffic-record kernel=... workload=... precision=...
    source-sha256=... read_bytes=... write_bytes=...', written from two
    rocprofv3 --pmc runs, FETCH_SIZE then WRITE_SIZE, each scaled by a plain
    copy of known size), or None when no record matches the current
    sources."""
    digest = kernel_source_digest()
    pdir = os.path.join(ROOT, "profiles")
    if not os.path.isdir(pdir):
        return None
    for name in sorted(os.listdir(pdir)):
        if not name.endswith((".md", ".txt")):
            continue
        with open(os.path.join(pdir, name)) as f:
            for line in f:
                if "traffic-record" not in line:
                    continue
                kv = dict(tok.split("=", 1) for tok in line.split() if "=" in tok)
                if (kv.get("kernel") == kernel and kv.get("workload") == workload and
                        kv.get("precision") == prec and kv.get("source-sha256") == digest):
                    return int(kv["read_bytes"]) + int(kv["write_bytes"])
    return None


def roofline(res):
    """HBM roofline of the dominant single-launch kernel: algorithmic bytes of
    its launch over its HIP-event duration (averaged over the timed steps).
    The alpha tile kernel exists only when alpha is materialised; with the
    fused sweeps its timer entry brackets the block seeds instead, so the
    candidate there is the Gamma tile alone."""
    n, prec, ph = res["n"], res["precision"], res["phases_ms"]
    cands = [k for k in SINGLE_LAUNCH if not (k == "alpha_tile" and res.get("fused"))]
    dom = max(cands, key=lambda k: ph[k])
    b = kernel_bytes(dom, n, prec)
    ach = b / (ph[dom] * 1e-3) / 1e9
    traffic = counter_traffic(SINGLE_LAUNCH[dom], res["workload"], prec)
    return dict(kernel=SINGLE_LAUNCH[dom], ms=ph[dom], bound="hbm", achieved=ach,
                peak=HBM_PEAK_GBS, unit="GB/s", frac=ach / HBM_PEAK_GBS, traffic=traffic,
                algorithmic_bytes=b,
                achieved_counted=None if traffic is None else traffic / (ph[dom] * 1e-3) / 1e9)


def solve_bytes(res):
    """Algorithmic HBM bytes of one whole solve, E bytes per stored value:
    with alpha materialised, E (2.5 n 2^n + 4 2^n) (alpha written once and
    read by both sweeps, the L and Rp halves read for every Gamma endpoint,
    L and Rp written and read); with the fused sweeps the alpha terms are
    gone and the block seeds are written once and read by both sweeps."""
    n, d, E = res["n"], res["d"], STORE_BYTES[res["precision"]]
    mat = E * (2.5 * n * 2 ** n + 4 * 2 ** n)
    if not res.get("fused"):
        return mat, mat
    ks9 = sum(math.comb(9, k) for k in range(d))
    seeds = 3 * 8 * n * 2 ** (n - 10) * ks9      # 8-byte seeds, written once, read twice
    return mat, E * (n * 2 ** n + 4 * 2 ** n) + seeds


def solve_roofline(res):
    mat, method = solve_bytes(res)
    sec = res["ms_per_step"] * 1e-3
    return dict(ms=res["ms_per_step"], bytes_method=method, GBs_method=method / sec / 1e9,
                frac_method=method / sec / 1e9 / HBM_PEAK_GBS,
                bytes_materialised_accounting=mat,
                GBs_materialised_accounting=mat / sec / 1e9,
                frac_materialised_accounting=mat / sec / 1e9 / HBM_PEAK_GBS)


def copy_calibration(nbytes):
    """One device-to-device copy of nbytes (torch's copy kernel): the known
    traffic that scales the FETCH_SIZE / WRITE_SIZE counters."""
    import torch
    src = torch.ones(nbytes // 4, dtype=torch.float32, device="cuda")
    dst = torch.empty_like(src)
    torch.cuda.synchronize()
    dst.copy_(src)
    torch.cuda.synchronize()
    print(json.dumps({"copy_bytes_read": nbytes, "copy_bytes_written": nbytes}), flush=True)


def mfma_experiment(bn, torch):
    """One in-tile zeta step (4 bits, FP64) as register add steps against the
    blocked 0/1 contraction on the FP64 matrix cores (bn_zeta4_probe): one
    HBM pass over 2^28 doubles, then the arithmetic alone (256 repetitions on
    2^24 doubles held in registers). Each figure is the best of three."""
    out = {}
    for label, count, reps in (("hbm_pass", 1 << 28, 1), ("arithmetic", 1 << 24, 256)):
        x = torch.rand(count, dtype=torch.float64, device="cuda")
        y = torch.empty_like(x)
        for method in ("valu", "mfma"):
            bn.zeta4_probe(x, y, method, reps)               # warm-up
            ms = min(bn.zeta4_probe(x, y, method, reps) for _ in range(3))
            # values transformed per second (each value once per repetition)
            rate = count * reps / (ms * 1e-3)
            out[f"{label}_{method}"] = dict(ms=ms, values_per_s=rate,
                                            GBs=16 * count / (ms * 1e-3) / 1e9 if reps == 1
                                            else None)
        out[f"{label}_mfma_over_valu_time"] = (out[f"{label}_mfma"]["ms"] /
                                               out[f"{label}_valu"]["ms"])
        del x, y
        torch.cuda.empty_cache()
    return out


def serving(bn, datagen, num=512, check=512):
    """Serving stream: 512 requests, n ~ U{10..22}, m ~ U{100..2000}, arity
    in {2,3}, d = 3, FP32-scaled, on one server. A first closed-loop pass
    (all requests at t = 0) warms the server (kernel code loaded on first
    use, the device arena grown) and is reported as the cold start; then the
    timed closed-loop saturation pass, then open-loop Poisson arrivals at 0.5
    and 0.8 of that rate; latency = arrival (submit) -> completion observed
    by the server."""
    import threading

    import numpy as np

    reqs = datagen.serving_stream(num, seed=4)
    data = [datagen.request_dataset(r) for r in reqs]
    srv = bn.Server(mem_budget_bytes=0, max_active=16)

    def run(arrivals):
        tickets = [None] * num
        t0 = time.perf_counter()

        def submitter():
            for j, (ds, r) in enumerate(zip(data, reqs)):
                if arrivals is not None:
                    delay = t0 + arrivals[j] - time.perf_counter()
                    if delay > 0:
                        time.sleep(delay)
                tickets[j] = srv.submit(ds.data, ds.arity, r["d"], precision="fp32",
                                        ess=r["ess"])

        th = threading.Thread(target=submitter)
        th.start()
        lat, posts = [], []
        for j in range(num):
            while tickets[j] is None:
                time.sleep(1e-4)
            s, post, rep = srv.poll(tickets[j], timeout_us=-1)
            assert s == bn.BN_OK, s
            lat.append(rep["ms_latency"])
            if j < check:
                posts.append(post)
        th.join()
        wall = time.perf_counter() - t0
        lat = np.array(lat)
        return dict(seconds=wall, solves_per_s=num / wall, p50_ms=float(np.percentile(lat, 50)),
                    p99_ms=float(np.percentile(lat, 99))), posts

    cold, _ = run(None)
    sat, posts = run(None)
    # every request of the closed-loop mix against the same problem solved
    # alone (bitwise: the kernels reduce in a fixed order)
    same, ndiff, maxdiff = True, 0, 0.0
    for j in range(check):
        alone, _ = bn.edge_posteriors(data[j].data, data[j].arity, reqs[j]["d"], precision="fp32",
                                      ess=reqs[j]["ess"])
        eq = bool(np.array_equal(alone, posts[j]))
        same = same and eq
        if not eq:
            ndiff += 1
            maxdiff = max(maxdiff, float(np.abs(alone - posts[j]).max()))
    rng = np.random.default_rng(4)
    out = dict(requests=num, workload="512 requests, n~U{10..22}, m~U{100..2000}, arity~U{2,3}, "
                                       "d=3, FP32-scaled",
               cold_start=cold, closed_loop=sat, open_loop=[], served_equals_alone=same,
               checked=check, differing=ndiff, max_abs_diff=maxdiff,
               mean_cells=float(np.mean([r["n"] * 2 ** r["n"] for r in reqs])))
    out["cells_per_s"] = out["mean_cells"] * sat["solves_per_s"]
    for frac in (0.5, 0.8):
        rate = frac * sat["solves_per_s"]
        gaps = rng.exponential(1.0 / rate, size=num)
        res, _ = run(np.cumsum(gaps))
        res["offered_rate"] = rate
        out["open_loop"].append(res)
    srv.close()
    return out


def subset_bench(bn, torch, datagen, nbits=30, steps=5):
    """Generic subset transforms in place on 2^nbits entries: FP64 (8 GiB at
    30 bits: upward zeta, upward zeta with |S| <= 3, downward zeta, upward
    Moebius) and the FP32-scaled storage (5 GiB: the zeta kinds). Each step
    restores the input (untimed) and times one transform with events on the
    current stream. Algorithmic bytes: one read and one write of every entry
    (16 B per entry in FP64, 10 B in the FP32-scaled form); the kernels make
    `passes` such sweeps over the array, so the bytes they move are passes
    times that."""
    passes = 1 + max(0, math.ceil((nbits - 12) / 9))
    out = dict(nbits=nbits, entries=1 << nbits, steps=steps, passes=passes, fp64={}, x32={})

    def timed(call, restore):
        tot = 0.0
        for k in range(steps + 1):
            restore()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            call()
            e1.record()
            e1.synchronize()
            if k > 0:     # the first call is a warmup
                tot += e0.elapsed_time(e1)
        return tot / steps

    def entry(ms, per_entry, d=-1):
        # moved: dense passes; a truncated transform skips rows without inputs
        alg = per_entry * (1 << nbits)
        return dict(ms=ms, algorithmic_bytes=alg, GB_s=alg / (ms * 1e-3) / 1e9,
                    frac=alg / (ms * 1e-3) / 1e9 / HBM_PEAK_GBS,
                    moved_GB_s=passes * alg / (ms * 1e-3) / 1e9 if d < 0 else None)

    base = torch.from_numpy(datagen.subset_values(nbits, 30, "uniform")).cuda()
    xt = torch.empty_like(base)
    for kind, d in [("zeta_up", -1), ("zeta_up", 3), ("zeta_down", -1), ("mobius_up", -1)]:
        ms = timed(lambda: bn.subset_transform(xt, kind, d), lambda: xt.copy_(base))
        out["fp64"][f"{kind}" + (f"_d{d}" if d >= 0 else "")] = entry(ms, 16, d)
    del base, xt
    torch.cuda.empty_cache()
    f = torch.empty(1 << nbits, dtype=torch.float32, device="cuda")
    b = torch.empty(1 << nbits, dtype=torch.uint8, device="cuda")

    def restore_x32():
        f.fill_(1.5)
        b.fill_(200)
    for kind, d in [("zeta_up", -1), ("zeta_up", 3), ("zeta_down", -1)]:
        ms = timed(lambda: bn.subset_transform_x32(f, b, kind, d), restore_x32)
        out["x32"][f"{kind}" + (f"_d{d}" if d >= 0 else "")] = entry(ms, 10, d)
    del f, b
    torch.cuda.empty_cache()
    return out


def cpu_baseline(datagen, name, sample_n):
    from oracle import oracle as O
    ds, p = datagen.workload(name)
    ns = min(sample_n, ds.n)
    r = O.edge_posteriors(ds.data[:ns], ds.arity[:ns], p["d"], ess=p["ess"])
    return dict(value=ns * 2 ** ns / r["seconds"], unit="cells/s", cores=O.num_threads(),
                kind="oracle", seconds=r["seconds"],
                sample=f"first {ns} of the {ds.n} variables of the {name} dataset "
                       f"(same m={ds.m}, d={p['d']}): {ns}*2^{ns} cells, one solve")


def main():
    ap = argparse.ArgumentParser(description=__doc__)
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--workload", default="n30_binary_m500_d3")
    ap.add_argument("--precision", default="fp32", choices=["fp32", "fp64"])
    ap.add_argument("--compare", default="fp64@n30_binary_m500_d3:3,"
                                         "fp32+fused@n30_binary_m500_d3:3,"
                                         "fp32+nolin@n30_binary_m500_d3:2,"
                                         "fp32@n25_binary_m2000_d4:10,"
                                         "fp64@n25_binary_m2000_d4:5",
                    help="extra lines prec[+variant]@workload:steps, comma separated ('' for "
                         "none); variants: fused (alpha never materialised), mat (alpha materialised), "
                         "nolin (no linear tiles)")
    ap.add_argument("--cpu-sample-n", type=int, default=25)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-serving", action="store_true")
    ap.add_argument("--no-subset", action="store_true")
    ap.add_argument("--subset-only", action="store_true",
                    help="only time the generic subset transforms (2^30 doubles) and exit")
    ap.add_argument("--copy-calibration", type=int, default=0, metavar="BYTES",
                    help="only run one device copy of BYTES (counter calibration) and exit")
    ap.add_argument("--serving-only", action="store_true",
                    help="only run the 512-request serving stream and exit")
    ap.add_argument("--mfma-experiment", action="store_true",
                    help="only time one 4-bit zeta step as register adds and as an FP64 "
                         "matrix-core contraction, and exit")
    ap.add_argument("--source-digest", action="store_true",
                    help="print the kernel-source digest that counter records carry and exit")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py runs on one GPU only: the solve is single-GPU (multi-GPU sharding of "
              "the lattice is a design, not built); use --gpus 1", file=sys.stderr)
        sys.exit(2)

    if args.source_digest:
        print(kernel_source_digest())
        return
    if args.copy_calibration:
        copy_calibration(args.copy_calibration)
        return

    import numpy as np
    import torch

    import paper_1408_1664_amd as bn
    from paper_1408_1664_amd import datagen

    torch.cuda.set_device(0)
    if args.subset_only:
        print(json.dumps({"subset_transform": subset_bench(bn, torch, datagen)}), flush=True)
        return
    if args.mfma_experiment:
        print(json.dumps({"zeta4_step": mfma_experiment(bn, torch)}), flush=True)
        return
    if args.serving_only:
        print(json.dumps({"serving": serving(bn, datagen)}), flush=True)
        return
    head = measure(bn, torch, datagen, args.workload, args.precision, args.steps, args.warmup)
    print(f"# {args.workload} {args.precision}: {head['ms_per_step']:.2f} ms/step, "
          f"{head['cells_per_s']:.3e} cells/s, phases {head['phases_ms']}", file=sys.stderr,
          flush=True)
    comps = []
    for item in [c for c in args.compare.split(",") if c.strip()]:
        pw, st = item.split(":")
        pv, wl = pw.split("@")
        prec, _, variant = pv.partition("+")
        r = measure(bn, torch, datagen, wl, prec, int(st), 1, variant)
        line = {k: v for k, v in r.items() if k != "post"}
        if wl == args.workload:
            line["max_abs_posterior_diff_vs_headline"] = float(np.abs(r["post"] -
                                                                      head["post"]).max())
        line["roofline"] = roofline(r)
        line["solve_roofline"] = solve_roofline(r)
        comps.append(line)
        print(f"# {wl} {pv}: {r['ms_per_step']:.2f} ms/step, {r['cells_per_s']:.3e} cells/s, "
              f"phases {r['phases_ms']}", file=sys.stderr, flush=True)
    serve = None
    if not args.no_serving:
        # the lattice runs above leave their workspaces in torch's cache;
        # the server allocates its own device arena
        torch.cuda.empty_cache()
        serve = serving(bn, datagen)
        print(f"# serving: {serve['closed_loop']['solves_per_s']:.0f} solves/s saturated, "
              f"open-loop p50/p99 {[(round(o['p50_ms'], 2), round(o['p99_ms'], 2)) for o in serve['open_loop']]}",
              file=sys.stderr, flush=True)
    sub = None
    if not args.no_subset:
        sub = subset_bench(bn, torch, datagen)
        print(f"# subset transforms 2^30: " + ", ".join(
            f"{form} {k} {v['ms']:.2f} ms" for form in ("fp64", "x32") for k, v in sub[form].items()),
            file=sys.stderr, flush=True)
    cpu = None
    if not args.no_cpu_baseline:
        cpu = cpu_baseline(datagen, args.workload, args.cpu_sample_n)
    rf = roofline(head)
    out = {
        "metric": METRIC,
        "value": head["cells_per_s"],
        "unit": "cells/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": head["ms_per_step"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        # FP32-scaled: FP32 significands (with integer exponents) in storage,
        # products and sweep sums; FP64 zeta adds inside a tile and FP64
        # log-gamma scores
        "dtype": "f32+f64" if args.precision == "fp32" else "f64",
        "data": "synthetic",
        "config": {"workload": args.workload, "n": head["n"], "m": head["m"], "d": head["d"],
                   "precision": "fp32_scaled" if args.precision == "fp32" else "fp64_log",
                   "alpha": "never materialised (fused sweeps)" if head["fused"]
                            else "materialised",
                   "score": "BDeu(ess=1)", "prior": "q=1, rho_k=1/C(n-1,k)"},
        "roofline": {k: rf[k] for k in ("bound", "achieved", "peak", "unit", "frac", "traffic")},
        "roofline_kernel": rf["kernel"],
        "roofline_kernel_ms": rf["ms"],
        "roofline_achieved_counted": rf["achieved_counted"],
        "solve_roofline": solve_roofline(head),
        "workspace_bytes": head["workspace_bytes"],
        "fallback": head["fallback"],
        "cpu_baseline": cpu,
        "phases_ms": head["phases_ms"],
        "log_LV": head["log_LV"],
        "max_invariant_residual": head["max_invariant_residual"],
        "saturated": head["saturated"],
        "flushed": head["flushed"],
        "comparisons": comps,
        "serving": serve,
        "subset_transform": sub,
    }
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
