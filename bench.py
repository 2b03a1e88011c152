#!/usr/bin/env python3
"""Throughput benchmark of the interior eigensolver on one MI355X.

Metric: eigenpairs/s at ||H x - lambda x||_2 <= 1e-10.  One step solves the
whole workload once, every inner step on the GPU (apply, fold, Jacobi-PCG,
Gram, Rayleigh-Ritz, small dense eigensolves, final FP64 residual check).

Workloads (--workload):
  l24  (default) L=24 open chain, Sz=0 (n=2704156), J=Delta=1, W=4, seed 0,
       sigma at energy density 0.5, 64 eigenpairs, block 128, tol 1e-10,
       mixed precision.  One step is one whole solve (several minutes); the
       timed steps stop within a wall budget (--budget-s) and report how many
       ran, warm-up runs on a small L=12 problem.
  l22  the same at L=22 (n=705432).
  l20  L=20, Sz=0 (n=184756), W in {1,2,4,8}, one realisation per W from
       seed 0, 32 eigenpairs per W, block 64, tol 1e-10, FP64.
  l12  L=12, Sz=0 (n=924), W=8, seed 0, 8 pairs, block 16 (seconds).
  batch, serve, slices, gram, precision, cgstep: the batched, serving,
       spectrum-slice, Gram, mixed-against-FP64 and CG-step measurements (see
       their functions).

The JSON line carries a roofline entry for the dominant kernel (the fused CG
apply kernels, timed with HIP events on the solve's stream inside the timed
region), and a CPU baseline from the FP64 oracle on a bounded sample.
"""

import argparse
import hashlib
from math import comb
import json
import os
import re
import sys
import time

T_START = time.perf_counter()
ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBPS = 8000.0
APPLY_SRC = [os.path.join(ROOT, "paper_2012_00217_amd", "csrc", f)
             for f in ("apply.hip", "apply_schedules.inc", "cg_panel.hip", "cg_column.hip")]
COUNTERS = os.path.join(ROOT, "profiles", "cg_apply_{}_counters.md")  # per workload

WORKLOADS = {
    "l20": dict(L=20, Ws=[1.0, 2.0, 4.0, 8.0], seed=0, eps=0.5, nev=32, block=64, tol=1e-10,
                precision="f64",
                desc="L=20 open chain, Sz=0 (n=184756), J=Delta=1, W in {1,2,4,8}, one "
                     "realisation per W from seed 0, 32 eigenpairs nearest sigma at energy "
                     "density 0.5, LOBPCG block 64, tol 1e-10, FP64"),
    "l24": dict(L=24, Ws=[4.0], seed=0, eps=0.5, nev=64, block=128, tol=1e-10, precision="mixed",
                desc="L=24 open chain, Sz=0 (n=2704156), J=Delta=1, W=4, seed 0, 64 eigenpairs "
                     "nearest sigma at energy density 0.5, block 128, tol 1e-10, mixed precision"),
    "l22": dict(L=22, Ws=[4.0], seed=0, eps=0.5, nev=64, block=128, tol=1e-10, precision="mixed",
                desc="L=22 open chain, Sz=0 (n=705432), J=Delta=1, W=4, seed 0, 64 eigenpairs "
                     "nearest sigma at energy density 0.5, block 128, tol 1e-10, mixed precision"),
    "l12": dict(L=12, Ws=[8.0], seed=0, eps=0.5, nev=8, block=16, tol=1e-10, precision="f64",
                desc="L=12 open chain, Sz=0 (n=924), J=Delta=1, W=8, seed 0, 8 eigenpairs "
                     "nearest sigma at energy density 0.5, block 16, tol 1e-10, FP64"),
}


def apply_src_hash():
    """Hash of the CG kernel sources and the compiled-in launch schedules."""
    h = hashlib.sha256()
    for path in APPLY_SRC:
        with open(path, "rb") as f:
            h.update(f.read())
    return h.hexdigest()[:16]


def cg_launch_widths(steps, column_steps, block, nev):
    """CG launches per column width of a solve whose CG runs on all `block`
    columns until the guard columns stop, then on the `nev` wanted ones:
    x + y = steps, block x + nev y = column_steps.  {} if the counts do not
    fit that pattern."""
    y = (block * steps - column_steps) / float(block - nev) if block > nev else 0.0
    if abs(y - round(y)) > 1e-6 or not 0 <= y <= steps:
        return {}
    y = int(round(y))
    return {block: steps - y, **({nev: y} if y > 0 else {})}


def column_cg(n):
    """The CG of a sector of n rows runs one workgroup per column (every sector of the
    workloads with at most 13,312 rows, unless the environment asks for a kernel)."""
    return n <= 13312 and not any(k.startswith(("MBL_APPLY_", "MBL_PCG_CACHE_MB"))
                                  for k in os.environ)


def read_traffic(kernel, workload, precision, width=None):
    """HBM bytes per launch from the committed counter summary, or None if the
    summary is missing, covers another workload or precision, or was taken
    from a different kernel source.  `width`: the launch's column count (the
    summary holds one value per width the counters were taken at)."""
    path = COUNTERS.format(workload)
    if not os.path.exists(path):
        return None
    txt = open(path).read()
    m = re.search(r"counters_workload:\s*(\S+)", txt)
    if not m or m.group(1) != workload:
        return None
    m = re.search(r"counters_precision:\s*(\S+)", txt)
    if not m or m.group(1) != precision:
        return None
    m = re.search(r"apply_src_sha256_16:\s*([0-9a-f]+)", txt)
    if not m or m.group(1) != apply_src_hash():
        return None
    key = f"{kernel}_hbm_bytes_per_launch" + (f"_w{width}" if width else "")
    m = re.search(rf"{key}:\s*([0-9.eE+]+)", txt)
    return float(m.group(1)) if m else None


class OracleLeg:
    """The FP64 oracle's work of one bench run, on a host thread.

    While the GPU solves (its calls release the GIL), the thread builds the
    sector matrix of every realisation (scipy CSR, FP64) and times the
    cpu_baseline sample: the oracle's step-by-step Jacobi-PCG on the fold of
    the first realisation, `steps` CG steps on a random n x block block (two
    sparse block applies each) plus one sparse apply, on this one core; the
    per-step time is projected with the GPU solve's own CG-step and apply
    counts (a projection: the oracle cannot solve these sectors itself).
    After the solve, check() recomputes every returned pair's residual with the
    oracle's CSR matrix.
    """

    def __init__(self, wl, sigmas, steps=4, verbose=False):
        import threading
        self.wl, self.sigmas, self.steps, self.verbose = wl, sigmas, steps, verbose
        self.mats, self.timing, self.error = {}, None, None
        self.thread = threading.Thread(target=self._run, daemon=True)
        self.thread.start()

    def note(self, msg):
        if self.verbose:
            print(f"[oracle] {msg}", file=sys.stderr, flush=True)

    def _run(self):
        try:
            import numpy as np
            from oracle import hamiltonian, pcg
            from paper_2012_00217_amd import workloads
            wl = self.wl
            L, b = wl["L"], wl["block"]
            st = None
            t_setup = None
            for W in wl["Ws"]:
                h = workloads.disorder(L, W, wl["seed"])
                t0 = time.perf_counter()
                st, H = hamiltonian.sector_matrix(L, L // 2, 1.0, 1.0, h, states=st)
                self.mats[W] = H
                if t_setup is None:
                    t_setup = time.perf_counter() - t0
                self.note(f"sector matrix W={W:g}: {time.perf_counter() - t0:.1f} s")
            W0 = wl["Ws"][0]
            H, sigma = self.mats[W0], self.sigmas[W0]
            t0 = time.perf_counter()
            d = hamiltonian.fold_diagonal(H, sigma)
            t_setup += time.perf_counter() - t0
            R = workloads.random_block(H.shape[0], b, seed=1)
            t0 = time.perf_counter()
            pcg.pcg_fold(H, sigma, d, R, self.steps)
            t_step = (time.perf_counter() - t0) / self.steps
            t0 = time.perf_counter()
            hamiltonian.apply_shifted(H, R, sigma)
            t_apply = time.perf_counter() - t0
            self.timing = dict(t_setup=t_setup, t_step=t_step, t_apply=t_apply, n=H.shape[0])
            self.note(f"{self.steps} CG steps: {t_step:.2f} s per step")
        except Exception as e:  # reported in the JSON line, never fatal
            self.error = repr(e)

    def check(self, W, evals, evecs):
        """Oracle FP64 residuals of the returned pairs (None if unavailable)."""
        from oracle import linalg
        self.thread.join()
        if W not in self.mats:
            return None
        return linalg.residual_norms(self.mats[W], evals, evecs)

    def baseline(self, run):
        """cpu_baseline entry from the GPU solve's counts (None if unavailable)."""
        self.thread.join()
        if self.timing is None:
            return None
        wl, tm = self.wl, self.timing
        other = run["applies"] - 2 * run["pcg_steps"]
        # the guard columns run fewer CG steps: charge the oracle per column-step
        col_steps = run["pcg_columns"] / float(wl["block"])
        t_proj = tm["t_setup"] + tm["t_step"] * col_steps + tm["t_apply"] * other
        nev = wl["nev"]
        return {
            "value": nev / t_proj,
            "unit": "eigenpairs/s",
            "cores": 1,
            "kind": "oracle",
            "sample": (f"oracle Jacobi-PCG on the fold, {self.steps} steps (2 CSR block applies "
                       f"each) on the L={wl['L']} W={wl['Ws'][0]:g} sector (n={tm['n']}, block "
                       f"{wl['block']}), {tm['t_step']:.3f} s/step on one core, projected with "
                       f"the GPU solve's {col_steps:.0f} full-block-equivalent CG steps and "
                       f"{other} other applies: {t_proj:.0f} s for {nev} pairs"),
            "host_cpu": _cpu_model(),
            "host_cores_available": len(os.sched_getaffinity(0)),
        }


def _cpu_model():
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def run_batch(args):
    """256 disorder realisations of mixed L (the batched workload): one step is
    one mbl_batch_solve over all problems, `--concurrency` at a time; the same
    problems one at a time give the single-solve comparison."""
    import numpy as np
    import torch
    from paper_2012_00217_amd import api, workloads

    probs = []
    for p in workloads.batch_problems(args.count):
        probs.append({"L": p["L"], "h": p["h"], "eps": 0.5, "nev": 16, "block": 32, "tol": 1e-10,
                      "precision": "f64", "seed": 7})
    torch.cuda.init()
    api.batch_solve(probs[:2], concurrency=2)  # load kernels
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    res = api.batch_solve(probs, concurrency=args.concurrency)
    torch.cuda.synchronize()
    el = time.perf_counter() - t0
    pairs = sum(int(np.sum(r["resid"] <= 1e-10)) for r in res if r["status"] == "MBL_OK")
    out = {"metric": "eigenpairs/s at resid<=1e-10 (batched)", "value": round(pairs / el, 3),
           "unit": "eigenpairs/s", "n_gpus": 1, "steps": 1, "warmup": 0,
           "ms_per_step": round(el * 1e3, 1), "higher_is_better": True, "scaling": "weak",
           "vs_baseline": None, "dtype": "f64", "data": "synthetic",
           "config": {"workload": f"{args.count} realisations, L in {{14,16,18}} (Sz=0), W in "
                                  "{2,4,6,8} from seed j, 16 pairs nearest energy density 0.5, "
                                  "block 32, tol 1e-10, FP64",
                      "concurrency": args.concurrency, "pairs": pairs,
                      "failed": sum(r["status"] != "MBL_OK" for r in res)}}
    if args.plain:
        t0 = time.perf_counter()
        res1 = api.batch_solve(probs, concurrency=1)
        el1 = time.perf_counter() - t0
        p1 = sum(int(np.sum(r["resid"] <= 1e-10)) for r in res1 if r["status"] == "MBL_OK")
        same = all(np.array_equal(a["evals"], b["evals"]) for a, b in zip(res, res1))
        out["plain"] = {"value": round(p1 / el1, 3), "ms": round(el1 * 1e3, 1),
                        "identical_results": same}
    print(json.dumps(out), flush=True)


def run_precision(args):
    """Mixed precision against FP64 on one problem (--precision-L, default 22;
    W=4, seed 0, 64 pairs, block 128, tol 1e-10, sigma at energy density 0.5):
    the same sigma and starting block in both runs; iterations, CG steps and
    time of each, the oracle's FP64 residual of every pair of both, and per
    pair the eigenvalue difference and the largest principal angle per
    near-degenerate cluster."""
    import numpy as np
    import scipy.linalg as sla
    import torch
    from oracle import hamiltonian, linalg
    from paper_2012_00217_amd import api, workloads

    L, nev, b, tol = args.precision_L, 64, 128, 1e-10
    h = workloads.disorder(L, 4.0, 0)
    torch.cuda.init()
    H = api.Hamiltonian(L, h)
    lo, hi = H.spectrum_bounds(1e-12)
    sigma = lo + 0.5 * (hi - lo)
    runs = {}
    for prec in ("mixed", "f64"):
        t0 = time.perf_counter()
        ev, V, rs, info = H.solve(sigma, nev, b, tol=tol, precision=prec, verbose=args.verbose,
                                  raise_on_noconv=False, guard_cg=args.guard_cg)
        el = time.perf_counter() - t0
        runs[prec] = dict(ev=ev, V=V.cpu().numpy(), s=el, info=info)
        del V
        torch.cuda.empty_cache()
        print(f"[precision] {prec}: {el:.1f} s, {info['iters']} iterations", file=sys.stderr,
              flush=True)
    st, Ho = hamiltonian.sector_matrix(L, L // 2, 1.0, 1.0, h)
    for r in runs.values():
        r["res"] = linalg.residual_norms(Ho, r["ev"], r["V"])
    em, ed = runs["mixed"]["ev"], runs["f64"]["ev"]
    dev = np.abs(em - ed)
    worst = max(runs["mixed"]["res"].max(), runs["f64"]["res"].max())
    cl = linalg.clusters(ed, 1e3 * worst)
    angles = [float(np.max(sla.subspace_angles(runs["mixed"]["V"][:, c], runs["f64"]["V"][:, c])))
              for c in cl]
    out = {"workload": f"L={L}, Sz=0 (n={H.n}), W=4, seed 0, {nev} pairs nearest sigma at "
                       f"energy density 0.5, block {b}, tol {tol:g}",
           "sigma": sigma,
           "runs": {p: {"seconds": round(r["s"], 1), "iters": r["info"]["iters"],
                        "iters_fp64": r["info"]["iters_fp64"],
                        "pcg_steps": r["info"]["pcg_steps"], "status": r["info"]["status"],
                        "oracle_max_resid": float(r["res"].max()),
                        "oracle_pairs_le_tol": int(np.sum(r["res"] <= tol))}
                    for p, r in runs.items()},
           "eig_absdiff_max": float(dev.max()), "eig_absdiff_median": float(np.median(dev)),
           "min_gap": float(np.diff(np.sort(ed)).min()), "clusters": len(cl),
           "max_angle": max(angles), "median_angle": float(np.median(angles))}
    print(json.dumps(out), flush=True)


def run_cgstep(args):
    """Time of one block Jacobi-PCG step and of one plain apply (H - sigma) X,
    per kernel path: `--cases` lists L:block:dtype (W=4, seed 0, Sz=0), and
    `--modes` the apply kernels (onepass: those that the library picks, split:
    the two-pass kernel, MBL_APPLY_SPLIT=1).  The CG step time is the
    difference of two PCG calls of m1 and m2 steps over m2 - m1 (setup and
    the first steps cancel); algorithmic bytes of a CG step: apply1 2nbs,
    apply2 6nbs, p update 3nbs (11nbs, plus per-row tables) with the gather
    kernels, 2nbs, 3nbs and 5nbs (10nbs) with the panels; reported at 11nbs."""
    import torch
    from paper_2012_00217_amd import api, workloads

    def timeit(fn, reps):
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / reps

    torch.cuda.init()
    out = []
    for case in args.cases.split(","):
        L, b, dt = case.split(":")
        L, b = int(L), int(b)
        dtype = torch.float32 if dt == "f32" else torch.float64
        s = 4 if dt == "f32" else 8
        H = api.Hamiltonian(L, workloads.disorder(L, 4.0, 0))
        n = H.n
        g = torch.Generator(device="cuda")
        g.manual_seed(1)
        R = torch.randn(n, b, dtype=dtype, device="cuda", generator=g)
        Y = torch.empty_like(R)
        res = {"L": L, "block": b, "dtype": dt, "n": n}
        for mode in args.modes.split(","):
            os.environ["MBL_APPLY_SPLIT"] = "1" if mode == "split" else "0"
            H.pcg(R, -0.5, 8)
            m1, m2 = 10, 60
            t1 = timeit(lambda: H.pcg(R, -0.5, m1), 2)
            t2 = timeit(lambda: H.pcg(R, -0.5, m2), 2)
            step = (t2 - t1) / (m2 - m1)
            H.apply(R, -0.5, out=Y)
            ta = timeit(lambda: H.apply(R, -0.5, out=Y), 10)
            res[mode] = {"cg_step_ms": round(step, 4),
                         "cg_alg_GBps": round(11 * n * b * s / step / 1e6, 1),
                         "apply_ms": round(ta, 4),
                         "apply_alg_GBps": round(2 * n * b * s / ta / 1e6, 1)}
        os.environ.pop("MBL_APPLY_SPLIT", None)
        print(json.dumps(res), flush=True)
        out.append(res)
        del R, Y
        H.close()
        torch.cuda.empty_cache()
    return out


def run_serve(args):
    """Open-loop request stream: Poisson arrivals of solves with mixed L, W and
    energy density, served with continuous batching; p50/p99 latency."""
    import numpy as np
    import torch
    from paper_2012_00217_amd import api, workloads

    Ls = tuple(int(x) for x in args.serve_L.split(","))
    reqs = workloads.request_stream(args.count, rate_hz=1.0, Ls=Ls)
    probs = [{"L": r["L"], "h": r["h"], "eps": r["eps"], "nev": 16, "block": 32, "tol": 1e-10,
              "precision": args.serve_precision, "seed": 7} for r in reqs]
    def note(msg):
        print(f"[serve] {msg}", file=sys.stderr, flush=True)

    torch.cuda.init()
    api.batch_solve(probs[:2], concurrency=2)
    # closed-loop capacity: all requests submitted at once
    def drain(srv, pending, t0, tag, results=None):
        # collect results in completion order, one progress line per request
        while pending:
            for i, t in list(pending.items()):
                r = srv.wait(t, timeout=0.02)
                if r is None:
                    continue
                del pending[i]
                if results is not None:
                    results[i] = r
                note(f"{tag}: request {i} (L={probs[i]['L']}) done at "
                     f"{time.perf_counter() - t0:.1f} s, latency {r['latency']:.2f} s")

    with api.Server(max_slots=args.concurrency) as srv:
        t0 = time.perf_counter()
        drain(srv, {i: srv.submit(d) for i, d in enumerate(probs)}, t0, "closed loop")
        cap = len(probs) / (time.perf_counter() - t0)
    rate = args.load * cap
    gaps = np.random.default_rng(args.count).exponential(1.0 / rate, len(probs))
    results = [None] * len(probs)
    # the open loop keeps every request's eigenvectors (copied out at
    # completion) so that the oracle can re-check every served pair afterwards
    served = [dict(d, want_vectors=True) for d in probs]
    vecs = [None] * len(probs)
    with api.Server(max_slots=args.concurrency) as srv:
        t0 = time.perf_counter()
        arrive = np.cumsum(gaps)
        pending, nxt = {}, 0
        while nxt < len(probs) or pending:
            now = time.perf_counter() - t0
            while nxt < len(probs) and arrive[nxt] <= now:
                pending[nxt] = srv.submit(served[nxt])
                vecs[nxt] = torch.empty((comb(probs[nxt]["L"], probs[nxt]["L"] // 2),
                                         probs[nxt]["nev"]), dtype=torch.float64, device="cuda")
                note(f"open loop: request {nxt} (L={probs[nxt]['L']}) arrived at {now:.1f} s")
                nxt += 1
            if pending:
                drain_once = dict(pending)
                for i, t in drain_once.items():
                    r = srv.wait(t, timeout=0.02, vectors_out=vecs[i])
                    if r is not None:
                        del pending[i]
                        results[i] = r
                        note(f"open loop: request {i} (L={probs[i]['L']}) done at "
                             f"{time.perf_counter() - t0:.1f} s, latency {r['latency']:.2f} s")
            else:
                time.sleep(min(0.05, max(0.0, arrive[nxt] - now)))
        el = time.perf_counter() - t0
        st = srv.stats()
    lat = np.array([r["latency"] for r in results])
    pairs = sum(int(np.sum(r["resid"] <= 1e-10)) for r in results if r["status"] == "MBL_OK")
    # the oracle's FP64 CSR residual of every served pair (after the timed loop)
    from oracle import hamiltonian, linalg
    checked, worst = 0, 0.0
    for i, r in enumerate(results):
        if r["status"] != "MBL_OK":
            continue
        L = probs[i]["L"]
        _, Ho = hamiltonian.sector_matrix(L, L // 2, 1.0, 1.0, probs[i]["h"])
        rc = linalg.residual_norms(Ho, r["evals"], vecs[i].cpu().numpy())
        checked += int(np.sum(rc <= 1e-10))
        worst = max(worst, float(rc.max()))
        vecs[i] = None
    note(f"oracle: {checked} of {pairs} served pairs at <= 1e-10 (largest residual {worst:.3g})")
    out = {"metric": "p99 ms (serving)", "value": round(float(np.percentile(lat, 99)) * 1e3, 1),
           "unit": "ms", "higher_is_better": False, "n_gpus": 1, "steps": 1, "warmup": 0,
           "ms_per_step": round(el * 1e3, 1), "scaling": "weak", "vs_baseline": None,
           "dtype": args.serve_precision, "data": "synthetic",
           "config": {"workload": f"{len(probs)} Poisson requests at {args.load:g} x closed-loop "
                                  f"capacity ({rate:.3f}/s), L in {Ls} (Sz=0), W~U[1,10], "
                                  "energy density in {0.1,0.5,0.9}, 16 pairs, block 32, tol 1e-10",
                      "concurrency": args.concurrency},
           "p50_ms": round(float(np.percentile(lat, 50)) * 1e3, 1),
           "throughput_pairs_per_s": round(pairs / el, 3),
           "oracle_checked_pairs": checked, "oracle_max_resid": worst,
           "capacity_req_per_s": round(cap, 4),
           "server_stats": {k: st[k] for k in ("completed", "rejected", "peak_bytes")}}
    if args.plain:
        # the plain path: the same requests solved one at a time in FP64, each
        # latency being its own solve time (no queueing counted)
        fp64 = [dict(d, precision="f64") for d in probs]
        t0 = time.perf_counter()
        res1 = api.batch_solve(fp64, concurrency=1)
        el1 = time.perf_counter() - t0
        note(f"plain FP64 one at a time: {el1:.1f} s")
        lat1 = np.array([r["seconds"] for r in res1])
        p1 = sum(int(np.sum(r["resid"] <= 1e-10)) for r in res1 if r["status"] == "MBL_OK")
        # the same arrivals served first come first served, one solve at a
        # time: latency = finish - arrival with finish_i = max(arrival_i,
        # finish_{i-1}) + solve_i (exact for one server, from the measured
        # solve times)
        fin, qlat = 0.0, []
        for a, d in zip(arrive, lat1):
            fin = max(a, fin) + d
            qlat.append(fin - a)
        qlat = np.array(qlat)
        out["plain_f64_one_at_a_time"] = {
            "solve_p50_ms": round(float(np.percentile(lat1, 50)) * 1e3, 1),
            "solve_p99_ms": round(float(np.percentile(lat1, 99)) * 1e3, 1),
            "queued_p50_ms": round(float(np.percentile(qlat, 50)) * 1e3, 1),
            "queued_p99_ms": round(float(np.percentile(qlat, 99)) * 1e3, 1),
            "capacity_req_per_s": round(len(probs) / el1, 4),
            "throughput_pairs_per_s": round(p1 / el1, 3), "ms": round(el1 * 1e3, 1)}
    print(json.dumps(out), flush=True)


def run_gram(args):
    """The MFMA Gram kernel alone on the Rayleigh-Ritz shapes of the solves:
    C = S^T S for S of n rows and m = 3 x block columns.  Algorithmic flops of a
    symmetric product: n m (m + 1) (the kernel forms the 64 x 64 tiles on and
    above the diagonal); TFLOP/s against the dtype's dense MFMA peak."""
    import torch
    from paper_2012_00217_amd import api

    shapes = [("L=20 Rayleigh-Ritz (block 64), FP64", 184756, 192, torch.float64),
              ("L=24 Rayleigh-Ritz (block 128), FP32", 2704156, 384, torch.float32),
              ("L=24 Rayleigh-Ritz (block 128), FP64", 2704156, 384, torch.float64),
              ("batch L=18 Rayleigh-Ritz (block 32), FP64", 48620, 96, torch.float64)]
    torch.cuda.init()
    res = []
    for name, n, m, dt in shapes:
        g = torch.Generator(device="cuda")
        g.manual_seed(n + m)
        S = torch.randn(n, m, dtype=dt, device="cuda", generator=g)
        for _ in range(2):
            api.gram(S, S)
        torch.cuda.synchronize()
        reps = 20
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            api.gram(S, S)
        e1.record()
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / reps
        tf = float(n) * m * (m + 1) / (ms * 1e-3) / 1e12
        peak = 157.3 if dt == torch.float32 else 78.6  # dense MFMA peaks of the MI355X
        res.append({"shape": name, "n": n, "m": m, "ms": round(ms, 4), "tflops": round(tf, 2),
                    "peak_tflops": peak, "frac": round(tf / peak, 4)})
        del S
        torch.cuda.empty_cache()
    top = max(res, key=lambda r: r["ms"])
    out = {"metric": "Gram TFLOP/s (MFMA)", "value": top["tflops"], "unit": "TFLOP/s", "n_gpus": 1,
           "steps": 20, "warmup": 2, "ms_per_step": top["ms"], "higher_is_better": True,
           "scaling": "weak", "vs_baseline": None,
           "dtype": "f32" if "FP32" in top["shape"] else "f64", "data": "synthetic",
           "config": {"workload": "Gram C = S^T S of the solvers' Rayleigh-Ritz blocks"},
           "roofline": {"bound": "mfma", "achieved": top["tflops"], "peak": top["peak_tflops"],
                        "unit": "TFLOP/s", "frac": top["frac"], "traffic": None},
           "shapes": res}
    print(json.dumps(out), flush=True)


def run_slices(args):
    """Spectrum slices and MBL observables: one L=18 realisation at W=1
    (ergodic side) and at W=8 (localised side); the 16 pairs nearest each of 9
    shifts at energy densities 0.1 ... 0.9 solved `--concurrency` at a time on
    one handle (one step = both realisations); then, outside the timed region,
    the mean adjacent gap ratio of each slice's levels and the half-chain
    entanglement entropy of the eps = 0.5 eigenvectors."""
    import numpy as np
    import torch
    from paper_2012_00217_amd import api, workloads

    L, nev, b, tol = 18, 16, 32, 1e-10
    Ws = (1.0, 8.0)
    eps = [round(0.1 * k, 1) for k in range(1, 10)]
    hams = {}
    for W in Ws:
        H = api.Hamiltonian(L, workloads.disorder(L, W, 0))
        lo, hi = H.spectrum_bounds(1e-12)
        hams[W] = (H, [lo + e * (hi - lo) for e in eps])
    H0, s0 = hams[Ws[0]]
    H0.solve(s0[4], 4, 8, tol=1e-8, want_vectors=False)  # load kernels
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    out = {W: H.solve_slices(sig, nev, b, tol=tol, concurrency=args.concurrency)
           for W, (H, sig) in hams.items()}
    elapsed = time.perf_counter() - t0
    pairs = sum(int(np.sum(rs <= tol)) for _, rs in out.values())
    obs = {}
    for W, (H, sig) in hams.items():
        ev, rs = out[W]
        _, V, _, _ = H.solve(sig[4], nev, b, tol=tol)
        torch.cuda.synchronize()
        te = time.perf_counter()
        S = H.entanglement_entropy(V)
        te = time.perf_counter() - te
        obs[str(W)] = {"mean_gap_ratio": round(float(np.mean([api.gap_ratio(e) for e in ev])), 4),
                       "ratios": int(len(eps) * (nev - 2)),
                       "mean_half_chain_entropy_eps0.5": round(float(np.mean(S)), 4),
                       "entropy_ms_16_vectors": round(te * 1e3, 3),
                       "max_resid": float(np.max(rs))}
    line = {"metric": "eigenpairs/s at resid<=1e-10 (spectrum slices)",
            "value": round(pairs / elapsed, 3), "unit": "eigenpairs/s", "n_gpus": 1, "steps": 1,
            "warmup": 0, "ms_per_step": round(elapsed * 1e3, 1), "higher_is_better": True,
            "scaling": "weak", "vs_baseline": None, "dtype": "f64", "data": "synthetic",
            "config": {"workload": f"L=18 open chain, Sz=0 (n=48620), J=Delta=1, W in {{1,8}} "
                                   f"from seed 0, 16 pairs nearest each of 9 shifts at energy "
                                   f"density 0.1..0.9, block 32, tol 1e-10, FP64",
                       "concurrency": args.concurrency, "pairs": pairs},
            "observables": obs}
    print(json.dumps(line), flush=True)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=1)
    ap.add_argument("--warmup", type=int, default=0)
    ap.add_argument("--workload", default="l24",
                    choices=sorted(WORKLOADS) + ["batch", "serve", "gram", "slices", "precision",
                                                 "cgstep"])
    ap.add_argument("--count", type=int, default=0,
                    help="batch/serve: number of problems (default 256 for batch, 40 for serve)")
    ap.add_argument("--concurrency", type=int, default=8,
                    help="batch/serve/slices: concurrent solves")
    ap.add_argument("--plain", action="store_true",
                    help="batch/serve: also solve the same problems one at a time (serve: in FP64)")
    ap.add_argument("--serve-L", default="16,18,20")
    ap.add_argument("--serve-precision", default="mixed")
    ap.add_argument("--load", type=float, default=0.8, help="serve: arrival rate / capacity")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--verbose", type=int, default=1,
                    help="progress on stderr: 0 none, 1 one line per outer iteration, 2 detail")
    ap.add_argument("--max-iter", type=int, default=400, help="outer LOBPCG iterations per solve")
    ap.add_argument("--precision", default="", choices=["", "f64", "pcg32", "mixed"],
                    help="override the workload's precision")
    ap.add_argument("--pcg-iters", type=int, default=0,
                    help="CG steps per outer iteration (0: the library default)")
    ap.add_argument("--lock", action="store_true",
                    help="single solves: soft locking of converged pairs (mbl_solve_opts.lock)")
    ap.add_argument("--cg-only", type=int, default=0,
                    help="counter runs: only run this many CG steps per realisation")
    ap.add_argument("--cg-widths", default="",
                    help="counter runs: block widths of the CG calls (default: the block, "
                         "then nev when the solve narrows the CG to the wanted columns)")
    ap.add_argument("--budget-s", type=float, default=560.0,
                    help="wall seconds of the whole command (the timed steps stop in time)")
    ap.add_argument("--cases", default="24:128:f32,22:128:f32,20:64:f64",
                    help="cgstep: L:block:dtype list")
    ap.add_argument("--modes", default="onepass,split", help="cgstep: apply kernels to time")
    ap.add_argument("--precision-L", type=int, default=22,
                    help="precision: chain length of the mixed-against-FP64 comparison")
    ap.add_argument("--nev", type=int, default=0, help="single solves: override the pair count")
    ap.add_argument("--block", type=int, default=0, help="single solves: override the block width")
    ap.add_argument("--guard-cg", type=float, default=0.0,
                    help="CG steps of the guard columns as a fraction (0: library default)")
    args = ap.parse_args()
    if args.count <= 0:
        args.count = 40 if args.workload == "serve" else 256
    if args.gpus != 1:
        print(f"bench.py measures one GPU only; --gpus {args.gpus} is not supported "
              "(the library solves on one GPU; sharding one solve over several GPUs is not "
              "implemented)", file=sys.stderr)
        sys.exit(2)

    if args.workload == "batch":
        return run_batch(args)
    if args.workload == "gram":
        return run_gram(args)
    if args.workload == "serve":
        return run_serve(args)
    if args.workload == "slices":
        return run_slices(args)
    if args.workload == "precision":
        return run_precision(args)
    if args.workload == "cgstep":
        return run_cgstep(args)

    import numpy as np
    import torch
    from paper_2012_00217_amd import api, workloads

    wl = dict(WORKLOADS[args.workload])
    if args.precision and args.precision != wl["precision"]:
        wl["desc"] = wl["desc"].rsplit(", ", 1)[0] + f", precision {args.precision}"
        wl["precision"] = args.precision
    if args.nev or args.block:
        wl["nev"] = args.nev or wl["nev"]
        wl["block"] = args.block or wl["block"]
        wl["desc"] += f" (overridden: {wl['nev']} pairs, block {wl['block']})"
    L = wl["L"]

    def note(msg):
        if args.verbose:
            print(f"[bench {time.perf_counter() - T_START:6.1f} s] {msg}", file=sys.stderr,
                  flush=True)

    torch.cuda.init()
    hams, sigmas = {}, {}
    for W in wl["Ws"]:
        H = api.Hamiltonian(L, workloads.disorder(L, W, wl["seed"]))
        lo, hi = H.spectrum_bounds(1e-12)
        hams[W], sigmas[W] = H, lo + wl["eps"] * (hi - lo)
        note(f"L={L} W={W:g}: n={H.n}, spectrum [{lo:.6f}, {hi:.6f}], sigma {sigmas[W]:.6f}")
    n = hams[wl["Ws"][0]].n
    s = 8 if wl["precision"] == "f64" else 4

    if args.cg_only:
        # calibration for HBM byte counters: an elementwise kernel that reads a
        # 2 GiB buffer and writes another (well beyond the 256 MB last-level
        # cache): exactly 2 GiB fetched and 2 GiB written per launch
        src = torch.ones(1 << 29, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(3):
            torch.mul(src, 1.5, out=dst)
        torch.cuda.synchronize()
        del src, dst
        # the CG widths of the solve: every column, then the wanted ones alone
        # when the guard columns stop early (n >= 500000 and nev >= 64, see the
        # library)
        widths = ([int(x) for x in args.cg_widths.split(",")] if args.cg_widths else
                  [wl["block"]] + ([wl["nev"]] if n >= 500000 and 64 <= wl["nev"] < wl["block"]
                                   and args.guard_cg != 1.0 else []))
        for W, H in hams.items():
            for w in widths:
                R = torch.randn(n, w, dtype=torch.float64 if s == 8 else torch.float32,
                                device="cuda")
                H.pcg(R, sigmas[W], args.cg_only)
                del R
        torch.cuda.synchronize()
        print(json.dumps({"cg_only": args.cg_only, "n": n, "widths": widths}))
        return

    oracle = None if args.no_cpu_baseline else OracleLeg(wl, sigmas, verbose=args.verbose)

    def one_step(record, max_seconds):
        out = {}
        for W, H in hams.items():
            ev, V, rs, info = H.solve(sigmas[W], wl["nev"], wl["block"], tol=wl["tol"],
                                      precision=wl["precision"], timing=True,
                                      raise_on_noconv=False, verbose=args.verbose,
                                      max_iter=args.max_iter, pcg_iters=args.pcg_iters,
                                      lock=args.lock, max_seconds=max_seconds,
                                      guard_cg=args.guard_cg)
            if record:
                out[W] = dict(info=info, evals=ev, resid=rs, V=V)
        return out

    # warm-up on the small L=12 problem (loads every kernel); the timed steps
    # are the workload itself
    small = api.Hamiltonian(12, workloads.disorder(12, 8.0, 0))
    lo12, hi12 = small.spectrum_bounds(1e-12)
    for _ in range(max(1, args.warmup)):
        small.solve(lo12 + 0.5 * (hi12 - lo12), 8, 16, tol=1e-10, precision=wl["precision"])
    small.close()
    torch.cuda.synchronize()
    note("warm-up done; timed steps start")

    # Wall budget: the driver stops the whole command at its limit, so the
    # timed steps stop early enough to leave time for the checks below; a
    # solve that would run past the budget stops at its own time limit and
    # returns its best pairs (only those the oracle confirms are counted).
    reserve = 20.0
    t0 = time.perf_counter()
    runs, elapsed = [], 0.0
    while len(runs) < args.steps:
        left = args.budget_s - (time.perf_counter() - T_START) - reserve
        if runs and left < elapsed / len(runs):
            break
        runs.append(one_step(True, max(1.0, left)))
        torch.cuda.synchronize()
        elapsed = time.perf_counter() - t0
        note(f"step {len(runs)} done: {elapsed:.1f} s timed so far")
    steps = len(runs)

    # every returned pair of the last step re-checked by the oracle (the steps
    # are the same deterministic computation)
    last = runs[-1]
    verified = {}
    for W, r in last.items():
        rc = None
        if oracle is not None:
            try:
                rc = oracle.check(W, r["evals"], r["V"].cpu().numpy())
            except Exception as e:  # the line is still printed; pairs then counted by the library
                oracle.error = oracle.error or repr(e)
        verified[str(W)] = int(np.sum(rc <= wl["tol"])) if rc is not None else None
        r["oracle_resid"] = rc
    if oracle is not None and all(v is not None for v in verified.values()):
        pairs_per_step = sum(verified.values())
        counted_by = "oracle"
    else:
        pairs_per_step = sum(int(np.sum(r["resid"] <= wl["tol"])) for r in last.values())
        counted_by = "library"
    value = pairs_per_step * steps / elapsed
    # dominant kernel from the live event timings: every CG launch of the
    # timed solves, its device time estimated per inner CG call from the
    # event-timed sample of that call (the library's *_all fields)
    k = 0 if s == 8 else 1
    tot = {"apply1": [0, 0.0, 0.0, 0, 0.0], "apply2": [0, 0.0, 0.0, 0, 0.0]}
    steps_cg, cols_cg = 0, 0
    for step in runs:
        for r in step.values():
            i = r["info"]
            for kk in ("apply1", "apply2"):
                tot[kk][0] += i["cg_launches_all"][k]
                tot[kk][1] += i[f"cg_{kk}_ms_all"][k]
                tot[kk][2] += i[f"cg_{kk}_bytes_all"][k]
                tot[kk][3] += i[f"cg_{kk}_launches"][k]
                tot[kk][4] += i[f"cg_{kk}_ms"][k]
            steps_cg += i["pcg_steps"]
            cols_cg += i["pcg_columns"]
    # Algorithmic bytes per launch over w columns of s-byte scalars (summed by
    # the library over the launches):
    #   apply1  T = (H - sigma) p, |T|^2: read p, write T, state word and
    #           diagonal per row                     -> 2 n w s + 12 n
    #   apply2  q = (H - sigma) T, x += alpha p, r -= alpha q, r.M^-1 r: read
    #           T, p, x, r, write x, r, state, diagonal, Jacobi diagonal
    #                                                -> 6 n w s + (12 + s) n
    # and of the panel CG (sectors above 13,312 rows near half filling), whose x
    # update is elsewhere and whose per-row tables are those of the two halves:
    #   apply1  read p, write T                      -> 2 n w s
    #   apply2  read T, r, write r                   -> 3 n w s
    # dominant: the larger total time (both kernels run once per CG step)
    dom = max(tot, key=lambda kk: tot[kk][1])
    nl, ms_all, bytes_all, nsample, ms_sample = tot[dom]
    kb = bytes_all / max(1, nl)
    avg_ms = ms_all / max(1, nl)
    achieved = kb / (avg_ms * 1e-3) / 1e9
    b_ = wl["block"]
    widths = None if args.lock else (
        cg_launch_widths(steps_cg, cols_cg, b_, wl["nev"]) if nl == steps_cg else {})
    traffic = None
    if widths:
        per_w = {w: read_traffic(dom, args.workload, wl["precision"], w) for w in widths}
        if len(widths) == 1 and per_w[b_] is None:
            per_w[b_] = read_traffic(dom, args.workload, wl["precision"])
        if all(v is not None for v in per_w.values()):
            traffic = sum(per_w[w] * c for w, c in widths.items()) / sum(widths.values())
    roofline = {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBPS,
                "unit": "GB/s", "frac": round(achieved / HBM_PEAK_GBPS, 4),
                "traffic": traffic,
                "kernel": f"fused CG {dom} ({'FP64' if s == 8 else 'FP32'}, "
                          + (", ".join(f"{c} launches over {w} columns"
                                       for w, c in widths.items()) if widths else
                             f"{wl['block']}-column block, narrower once pairs lock"
                             if args.lock else f"{wl['block']}-column block") + ")",
                "algorithmic_bytes_per_launch": kb, "avg_launch_us": round(avg_ms * 1e3, 2),
                "launches": nl, "timed_launches": nsample,
                "timed_avg_launch_us": round(ms_sample / max(1, nsample) * 1e3, 2)}

    if column_cg(n):
        # the CG vectors never leave the CU: a memory rate would mean nothing
        roofline = {"bound": "latency", "achieved": None, "peak": None, "unit": None,
                    "frac": None, "traffic": None,
                    "kernel": f"one workgroup per CG column, every step in one launch "
                              f"({'FP64' if s == 8 else 'FP32'}, {wl['block']} columns)",
                    "cg_steps": nl,
                    **{f"{kk}_us_per_step": round(t[1] / max(1, t[0]) * 1e3, 2)
                       for kk, t in tot.items()}}

    # H X bandwidth of the plain apply (after the timed region)
    H0 = hams[wl["Ws"][0]]
    dt = torch.float64 if s == 8 else torch.float32
    nset = max(2, int(np.ceil(1.5e9 / (2 * n * wl["block"] * s))))
    Xs = [torch.randn(n, wl["block"], dtype=dt, device="cuda") for _ in range(nset)]
    Ys = [torch.empty_like(Xs[0]) for _ in range(nset)]
    for i in range(2):
        H0.apply(Xs[i % nset], sigmas[wl["Ws"][0]], out=Ys[i % nset])
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    reps = 20
    e0.record()
    for i in range(reps):
        H0.apply(Xs[i % nset], sigmas[wl["Ws"][0]], out=Ys[i % nset])
    e1.record()
    torch.cuda.synchronize()
    hx_ms = e0.elapsed_time(e1) / reps
    hx_gbps = 2 * n * wl["block"] * s / (hx_ms * 1e-3) / 1e9
    # the same buffers every time: in cache when X and Y fit the 256 MB last-level cache
    e0.record()
    for i in range(reps):
        H0.apply(Xs[0], sigmas[wl["Ws"][0]], out=Ys[0])
    e1.record()
    torch.cuda.synchronize()
    hx_cache_gbps = 2 * n * wl["block"] * s / (e0.elapsed_time(e1) / reps * 1e-3) / 1e9
    del Xs, Ys
    # a plain 1 GiB device-to-device tensor copy (1 GiB read + 1 GiB written),
    # timed as a reference point beside the published HBM peak
    src = torch.empty(1 << 28, dtype=torch.float32, device="cuda")
    dst = torch.empty_like(src)
    dst.copy_(src)
    torch.cuda.synchronize()
    e0.record()
    for _ in range(5):
        dst.copy_(src)
    e1.record()
    torch.cuda.synchronize()
    copy_gbps = 2 * src.numel() * 4 / (e0.elapsed_time(e1) / 5 * 1e-3) / 1e9
    del src, dst
    roofline["measured_copy_GBps"] = round(copy_gbps, 1)

    per_w = {}
    for W, r in last.items():
        i = r["info"]
        per_w[str(W)] = {"sigma": sigmas[W], "iters": i["iters"], "applies": i["applies"],
                         "pcg_steps": i["pcg_steps"], "pcg_columns": i["pcg_columns"],
                         "seconds": round(i["seconds"], 3), "t_pcg": round(i["t_pcg"], 3),
                         "t_apply": round(i["t_apply"], 4), "t_gram": round(i["t_gram"], 4),
                         "t_small": round(i["t_small"], 4),
                         "max_resid": float(np.max(r["resid"])), "status": i["status"],
                         "oracle_pairs_le_tol": verified[str(W)],
                         "oracle_max_resid": (float(np.max(r["oracle_resid"]))
                                              if r["oracle_resid"] is not None else None)}
    cpu = None
    if oracle is not None:
        run0 = last[wl["Ws"][0]]["info"]
        cpu = oracle.baseline({"applies": run0["applies"], "pcg_steps": run0["pcg_steps"],
                               "pcg_columns": run0["pcg_columns"]})
        if cpu is None:
            cpu = {"error": oracle.error}
    line = {
        "metric": "eigenpairs/s at resid<=1e-10",
        "value": round(value, 4),
        "unit": "eigenpairs/s",
        "n_gpus": 1,
        "steps": steps,
        "warmup": max(1, args.warmup),
        "ms_per_step": round(elapsed / steps * 1e3, 1),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64" if wl["precision"] == "f64" else "f32+f64",
        "data": "synthetic",
        "config": {"workload": wl["desc"], "L": L, "n": n, "nev": wl["nev"],
                   "block": wl["block"], "tol": wl["tol"], "precision": wl["precision"],
                   "W": wl["Ws"], "pairs_per_step": pairs_per_step,
                   "pairs_counted_by": counted_by, "steps_requested": args.steps,
                   "warmup_workload": "L=12, W=8, 8 pairs, block 16 (kernel load)",
                   **({"soft_locking": True} if args.lock else {})},
        "roofline": roofline,
        "cpu_baseline": cpu,
        "hx_GBps": round(hx_gbps, 1),
        "hx_same_buffers_GBps": round(hx_cache_gbps, 1),
        "hx_ms": round(hx_ms, 4),
        "cg_steps": steps_cg,
        "per_W": per_w,
        "wall_s": round(time.perf_counter() - T_START, 1),
    }
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
