#!/usr/bin/env python3
"""Benchmark of the algebraic Awerbuch-Shiloach MSF hot path on one MI355X.

Headline: MSF edges/s on an R-MAT graph of scale 22 (4,194,304 vertices,
edge factor 16, a/b/c/d = .57/.19/.19/.05, permuted ids, duplicates and
self-loops removed, float32 weights), one step = one msf_solve from
device-resident COO edges to device-resident forest ids (validation, every
round, output compaction and the exact total).

Also reported on the same JSON line:
  roofline      the dominant unit of the solve (most device time per step
                among the selection of the light edges, the first round and
                all later rounds; with an adjacency matrix among its build,
                the run sort and the head sweeps): its algorithmic
                bytes per launch over its average
                launch time, both taken inside the timed steps from device
                events (contracted rounds: stamps of the device's
                clock) that the library records on the stream those kernels
                run on; `traffic` is the counter-measured bytes per launch
                from the committed profile, reported only when the sources
                built here are the ones that profile was taken on (else
                null);
  cpu_baseline  the CPU oracle (sort + union-find, one thread) on the same
                graph, timed on this host;
  batched       10^4 uneven Erdos-Renyi graphs (n log-uniform in [64, 65536),
                average degree 8) in one batched solve vs one msf_solve per
                graph;
  served        continuous-batching server: p50/p99 latency and graphs/s of
                a Poisson stream of mixed graphs at several rates, vs a plain
                one-at-a-time FIFO, and the CPU oracle's service rate on the
                same pool (one thread and the host's cores);
  multilinear_ablation
                the all-at-once multilinear kernel vs the pairwise
                formulation (pairs (a_ij, p_j) stored first, then reduced) on
                R-MAT scale 17 edge factor 8 and on the scale-22 graph, for
                the identity parent vector (round 1) and a forest of stars;
                wall time per call, both forms paying the same parent check;
  shortcut_study
                complete shortcutting by full passes, by the frontier and by a
                switch between them, on the parent forest of round 1's hooks
                on the 256^3 grid and on a random recursive tree of the same
                size: wall time per call and passes;
  components    connected components by the connectivity variant on the
                same kernels, on R-MAT scale 22 and the 256^3 grid: wall time
                per call (from a built graph) and rounds;
  starcheck     the original AS rounds (star check, one-step shortcut) on the
                same graphs: wall time per call and rounds, beside msf_solve's
                rounds with complete shortcutting.

Usage: python bench.py [--gpus 1] [--steps K] [--warmup W] [--no-cpu] [--no-extras]
                       [--no-ablation] [--ablation-only] [--shortcut-only]
                       [--components-only] [--starcheck-only]
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0  # MI355X HBM3E peak, GB/s
PROFILE = os.path.join(ROOT, "profiles", "rmat_s22_solve.md")
PROFILE_ML = os.path.join(ROOT, "profiles", "multilinear_rmat_s22_round1.md")
# timed kernels: label -> (kernel name, sources its code comes from)
# (the sources are the files holding the kernels' code; a committed counter
# profile counts only while they are unchanged)
KERNELS = {
    "place": ("k_tl_place (two-level build, placement)", ("kernels_build2.hip",)),
    "sort": ("k_sort_chunks (run sort of the head sweep)", ("kernels_heads.hip",)),
    "part2": ("k_part_sub (two-level build, level-2 partition)", ("kernels_build2.hip",)),
    "part1": ("k_part_edges (two-level build, level-1 partition)", ("kernels_build2.hip",)),
    "sweep": ("k_sweep (multilinear + projection)", ("kernels_sweep.hip",)),
    "heads": ("k_heads + k_heads_rest (head sweep)", ("kernels_heads.hip",)),
    "build": ("adjacency build (two-level)", ("kernels_build2.hip", "kernels_build.hip")),
}


def source_hash(label):
    import hashlib

    h = hashlib.sha256()
    for f in KERNELS[label][1]:
        with open(os.path.join(ROOT, "paper_2110_04865_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def measured_traffic(label, profile=None):
    """HBM bytes per launch of the kernel `label` from a committed counter
    profile (calibrated FETCH_SIZE + WRITE_SIZE), or None when the profile
    holds none or was taken on different sources than the ones built here."""
    try:
        with open(profile or PROFILE) as fh:
            lines = fh.read().splitlines()
    except OSError:
        return None
    keys = (f"{label}_traffic_bytes:", f"{label}_source_sha256:")
    vals = {}
    for ln in lines:
        for k in keys:
            if ln.strip().startswith(k):
                vals[k] = ln.strip()[len(k):].strip().strip("`")
    if vals.get(keys[1]) != source_hash(label):
        return None
    try:
        return float(vals[keys[0]])
    except (KeyError, ValueError):
        return None


def log(*a):
    print("[bench]", *a, file=sys.stderr, flush=True)


def bench_rmat(ctx, pkg, torch, steps, warmup):
    import numpy as np
    import gen

    t = time.perf_counter()
    n, e, w = gen.workload_rmat_s22()
    m = len(e)
    log(f"generated R-MAT s22: n={n} m={m} in {time.perf_counter() - t:.1f}s")
    de = torch.from_numpy(e.reshape(-1).copy()).to("cuda:0")
    dw = torch.from_numpy(w.copy()).to("cuda:0")
    out = torch.empty(n, dtype=torch.int32, device="cuda:0")
    for i in range(warmup):
        ctx.solve(n, de, dw, wtype=pkg.W_F32, out=out)
        log(f"warmup {i + 1}/{warmup} done")
    torch.cuda.synchronize()
    # per timed kernel: [device ms, algorithmic bytes, launches] over the steps
    kt = {k: [0.0, 0.0, 0] for k in KERNELS}
    build_ms = rounds_ms = adj_ms = 0.0
    t0 = time.perf_counter()
    for k in range(steps):
        ids, cnt, tot = ctx.solve(n, de, dw, wtype=pkg.W_F32, out=out)
        st = ctx.stats()
        first = st["rounds"] - st["head_sweeps"]  # rounds before the head sweep takes over
        for i, (t_ms, b) in enumerate(zip(st["sweep_ms"], st["sweep_bytes"])):
            if b > 0:  # round 1's minima come from the build: no sweep launch
                kt["sweep"][0] += t_ms
                kt["sweep"][1] += b
                kt["sweep"][2] += 1
            elif st["head_sweeps"] and i >= first:
                # descriptors: head key, column and row (16), p of the row and
                # of the head column (8) per run
                kt["heads"][0] += t_ms
                kt["heads"][1] += 24.0 * st["runs"]
                kt["heads"][2] += 1
        for q, lab in enumerate(("place", "sort", "part2", "part1")):
            if st["pass_ms"][q] > 0:
                kt[lab][0] += st["pass_ms"][q]
                kt[lab][1] += st["pass_bytes"][q]
                kt[lab][2] += 1
        build_ms += st["build_ms"]
        rounds_ms += st["rounds_ms"]
        adj_ms += st["adjacency_ms"]
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    log(f"timed {steps} steps in {t1 - t0:.3f}s; last stats {st}")
    ms = (t1 - t0) * 1000.0 / steps
    res = dict(n=n, m=m, e=e, w=w, ms=ms, count=cnt, total=tot, stats=st,
               ids=ids.cpu().numpy().astype(np.int64),
               kernels=kt, build_ms=build_ms / steps, rounds_ms=rounds_ms / steps,
               adjacency_ms=adj_ms / steps)
    return res


def bench_multilinear(ctx, pkg, torch, graphs, reps=10):
    """All-at-once vs pairwise multilinear kernel, per graph and parent vector."""
    import numpy as np

    out = {}
    for label, (n, e, w) in graphs.items():
        g = pkg.Graph(ctx, n, e, w, wtype=pkg.W_F32)
        rng = np.random.default_rng(17)
        roots = rng.choice(n, size=max(1, n // 16), replace=False).astype(np.uint32)
        star = roots[rng.integers(0, len(roots), n)]
        star[roots] = roots
        parents = {"identity": np.arange(n, dtype=np.uint32), "stars_n/16": star}
        r1 = torch.empty(n, dtype=torch.int64, device="cuda:0")
        r2 = torch.empty(n, dtype=torch.int64, device="cuda:0")
        res = {"n": n, "m": len(w)}
        for pk, p in parents.items():
            dp = torch.from_numpy(p.view(np.int32)).to("cuda:0")
            row = {}
            for form, fn, r in (("all_at_once", ctx.multilinear, r1),
                                ("pairwise", ctx.multilinear_pairwise, r2)):
                fn(g, dp, r)  # warm-up (and the pair array's allocation)
                torch.cuda.synchronize()
                t = time.perf_counter()
                for _ in range(reps):
                    fn(g, dp, r)
                torch.cuda.synchronize()
                row[form + "_ms"] = (time.perf_counter() - t) * 1000.0 / reps
            row["pairwise_over_all_at_once"] = row["pairwise_ms"] / row["all_at_once_ms"]
            row["same_r"] = bool(torch.equal(r1, r2))
            res[pk] = row
        g.close()
        out[label] = res
        log(f"multilinear ablation {label}: {res}")
    return out


def round1_forest(ctx, pkg, torch, n, e, w, wtype):
    """Parent forest after round 1's hooks and tie break: every vertex hooks
    to the other end of its minimum-key edge; of a mutual pair the smaller id
    stays root.  Minima from msf_multilinear with the identity; the rest on
    the host."""
    import numpy as np

    g = pkg.Graph(ctx, n, e, w, wtype=wtype)
    r = torch.empty(n, dtype=torch.int64, device="cuda:0")
    ctx.multilinear(g, torch.arange(n, dtype=torch.int32, device="cuda:0"), r)
    torch.cuda.synchronize()
    g.close()
    key = r.cpu().numpy().view(np.uint64)
    ids = np.arange(n, dtype=np.int64)
    has = key != np.uint64(0xFFFFFFFFFFFFFFFF)
    eid = (key & np.uint64(0xFFFFFFFF)).astype(np.int64)
    a = np.where(has, e[np.where(has, eid, 0), 0], ids)
    b = np.where(has, e[np.where(has, eid, 0), 1], ids)
    h = np.where(a == ids, b, a).astype(np.int64)
    mutual = (h[h] == ids) & (ids < h)
    h[mutual] = ids[mutual]
    return h.astype(np.uint32)


def bench_shortcut(ctx, pkg, torch, reps=5):
    """Shortcut strategies on round 1's forest of the 256^3 grid and on a
    random recursive tree of the same size."""
    import numpy as np
    import gen

    n, e, w = gen.workload_grid_256()
    forests = {"grid256_round1": round1_forest(ctx, pkg, torch, n, e, w, pkg.W_U32)}
    rng = np.random.default_rng(23)
    par = (rng.random(n) * np.arange(n)).astype(np.int64)  # parent uniform below
    perm = rng.permutation(n)
    rrt = np.empty(n, dtype=np.uint32)
    rrt[perm] = perm[par]
    forests["random_recursive_tree"] = rrt
    strategies = [("frontier", pkg.SHORTCUT_FRONTIER, 0.0), ("full", pkg.SHORTCUT_FULL, 0.0),
                  ("switch_0.25", pkg.SHORTCUT_SWITCH, 0.25),
                  ("switch_0.05", pkg.SHORTCUT_SWITCH, 0.05)]
    out = {}
    for fname, p in forests.items():
        src = torch.from_numpy(p.view(np.int32)).to("cuda:0")
        dp = torch.empty_like(src)
        res = {"n": n, "non_roots": int((p != np.arange(n)).sum())}
        for sname, st, frac in strategies:
            dp.copy_(src)
            ctx.shortcut_strategy(dp, st, frac)  # warm-up (workspace)
            total = 0.0
            for _ in range(reps):
                dp.copy_(src)
                torch.cuda.synchronize()
                t = time.perf_counter()
                passes = ctx.shortcut_strategy(dp, st, frac)
                total += time.perf_counter() - t
            res[sname] = {"ms": total * 1000.0 / reps, "passes": passes}
        out[fname] = res
        log(f"shortcut study {fname}: {res}")
    return out


def bench_components(ctx, pkg, torch, graphs, reps=3):
    """msf_components on built graphs: wall time per call and rounds."""
    out = {}
    for label, (n, e, w, wt) in graphs.items():
        g = pkg.Graph(ctx, n, e, w, wtype=wt)
        lab = torch.empty(n, dtype=torch.int32, device="cuda:0")
        rounds = ctx.components(g, lab)  # warm-up (workspace)
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(reps):
            rounds = ctx.components(g, lab)
        ms = (time.perf_counter() - t) * 1000.0 / reps
        ncomp = int(torch.unique(lab).numel())
        g.close()
        out[label] = {"n": n, "m": len(w), "ms": ms, "rounds": rounds, "components": ncomp,
                      "edges_per_s": len(w) / (ms / 1000.0)}
        log(f"components {label}: {out[label]}")
    return out


def bench_starcheck(ctx, pkg, torch, graphs, reps=3):
    """msf_solve_starcheck on built graphs vs the rounds of msf_solve."""
    out = {}
    for label, (n, e, w, wt) in graphs.items():
        de = torch.from_numpy(e.reshape(-1).copy()).to("cuda:0")
        dw = torch.from_numpy(w.copy()).to("cuda:0")
        ctx.solve(n, de, dw, wtype=wt)
        solve_rounds = ctx.stats()["rounds"]
        del de, dw
        g = pkg.Graph(ctx, n, e, w, wtype=wt)
        flags = torch.empty(len(w), dtype=torch.uint8, device="cuda:0")
        rounds = ctx.solve_starcheck(g, flags)  # warm-up (workspace)
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(reps):
            rounds = ctx.solve_starcheck(g, flags)
        ms = (time.perf_counter() - t) * 1000.0 / reps
        g.close()
        out[label] = {"n": n, "m": len(w), "ms": ms, "rounds": rounds,
                      "complete_shortcut_rounds": solve_rounds}
        log(f"starcheck {label}: {out[label]}")
    return out


def cpu_baseline(n, e, w, wtype=1):
    import oracle

    t = time.perf_counter()
    ids, cnt, tot = oracle.msf(n, e, w, wtype)
    dt = time.perf_counter() - t
    return dict(seconds=dt, count=cnt, total=tot, ids=ids)


def same_forest(gpu_ids, cnt, tot, cb, wtype):
    """Element-wise parity of a GPU result with the oracle's: ids, count,
    and the totals (exact)."""
    import numpy as np

    return (cnt == cb["count"] and np.array_equal(np.asarray(gpu_ids, dtype=np.int64), cb["ids"])
            and tot[1] == cb["total"][1] and (wtype == 1 or tot[0] == cb["total"][0]))


def host_info():
    """CPU model and the cores this process may use (for the CPU baseline)."""
    model = "unknown"
    try:
        with open("/proc/cpuinfo") as fh:
            for ln in fh:
                if ln.startswith("model name"):
                    model = ln.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    try:
        usable = len(os.sched_getaffinity(0))
    except AttributeError:
        usable = os.cpu_count()
    return {"cpu_model": model, "nproc": usable, "os_cpu_count": os.cpu_count()}


def bench_plain(ctx, pkg, torch, label, n, e, w, wt, steps=5, cpu=True):
    """One configuration's plain msf_solve from device-resident COO: time
    per solve, edges/s, rounds, element-wise parity with the oracle and the
    oracle's own time on the host (one thread)."""
    import numpy as np

    de = torch.from_numpy(e.reshape(-1).copy()).to("cuda:0")
    dw = torch.from_numpy(w.view(np.int32).copy()).to("cuda:0")
    out = torch.empty(max(n, 1), dtype=torch.int32, device="cuda:0")
    for _ in range(2):
        ctx.solve(n, de, dw, wtype=wt, out=out)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        ids, cnt, tot = ctx.solve(n, de, dw, wtype=wt, out=out)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1000.0 / steps
    st = ctx.stats()
    res = {"workload": label, "n": n, "m": len(w), "ms_per_solve": ms,
           "edges_per_s": len(w) / (ms / 1000.0), "rounds": st["rounds"],
           "hooks_per_round": st["hooks"], "build_ms": st["build_ms"],
           "rounds_ms": st["rounds_ms"], "head_sweeps": st["head_sweeps"]}
    if cpu:
        cb = cpu_baseline(n, e, w, wt)
        res["parity"] = bool(same_forest(ids.cpu().numpy(), cnt, tot, cb, wt))
        res["cpu_oracle_s"] = cb["seconds"]
        res["cpu_oracle_edges_per_s"] = len(w) / cb["seconds"]
    log(f"plain {label}: {res}")
    return res


def parents_after_round1(ctx, pkg, torch, n, e, w, wtype):
    """The parent vector at the start of round 2 of msf_solve: round 1's
    hooks and tie break (round1_forest), completed by msf_shortcut."""
    import numpy as np

    h = round1_forest(ctx, pkg, torch, n, e, w, wtype)
    p = torch.from_numpy(h.view(np.int32)).to("cuda:0")
    ctx.shortcut(p)
    torch.cuda.synchronize()
    return p


def bench_multilinear_round1(ctx, pkg, torch, n, e, w, wtype, reps=25):
    """msf_multilinear on the full adjacency with the parents after round 1:
    median device time of the sweep kernel (events the library records on
    its stream around that launch) over `reps` calls, against the streamed
    bytes 12 nnz + 4 (rows + 1) + 4 rows + 8 roots written."""
    import numpy as np

    p = parents_after_round1(ctx, pkg, torch, n, e, w, wtype)
    g = pkg.Graph(ctx, n, e, w, wtype=wtype)
    r = torch.empty(n, dtype=torch.int64, device="cuda:0")
    for _ in range(3):
        ctx.multilinear(g, p, r)
    times, gtimes = [], []
    for _ in range(reps):
        ctx.multilinear(g, p, r)
        st = ctx.stats()  # waits for the sweep's end event
        times.append(st["sweep_ms"][0])
        gtimes.append(st["pass_ms"][0])
    torch.cuda.synchronize()
    rk = r.cpu().numpy().view(np.uint64)
    roots_written = int((rk != np.uint64(0xFFFFFFFFFFFFFFFF)).sum())
    deg = np.bincount(e[e[:, 0] != e[:, 1]].reshape(-1), minlength=n)
    rows = int((deg > 0).sum())
    nnz = int(deg.sum())
    pn = p.cpu().numpy()
    shares = bench_row_shares(ctx, pkg, torch, g, p, r, n, deg, reps)
    g.close()
    med = float(np.median(times))
    b = 12.0 * nnz + 4.0 * (rows + 1) + 4.0 * rows + 8.0 * roots_written
    gb_s = b / 1e9 / (med / 1e3)
    return {"kernel": "k_sweep (msf_multilinear: multilinear kernel + projection)",
            "parents": "after round 1 of msf_solve (hooks, tie break, complete shortcut)",
            "roots": int((pn == np.arange(n)).sum()), "roots_written": roots_written,
            "nnz": nnz, "rows": rows, "reps": reps, "median_ms": med,
            "min_ms": float(np.min(times)), "max_ms": float(np.max(times)),
            "bytes": b, "achieved": gb_s, "peak": HBM_PEAK_GBS, "unit": "GB/s",
            "frac": gb_s / HBM_PEAK_GBS, "target_frac": 0.40,
            "traffic": measured_traffic("sweep", PROFILE_ML),
            "gather_bytes_if_every_entry": 4.0 * nnz,
            "order_gather_ms": float(np.median(gtimes)),
            "call_frac": b / 1e9 / ((med + float(np.median(gtimes))) / 1e3) / HBM_PEAK_GBS,
            "note": "median_ms is the sweep kernel alone; order_gather_ms is the kernel that "
                    "gathers p into the graph's degree order before it (12 B per vertex)",
            "row_shares": shares}


def bench_row_shares(ctx, pkg, torch, g, p, r, n, deg, reps, parts=8):
    """One device's share of the sweep when the rows of A are split `parts`
    ways with the whole p on every device (the sharding of the design notes):
    msf_multilinear_rows over entry-balanced ranges of stored rows, median
    sweep time per range, bytes as for the whole kernel over the range."""
    import numpy as np

    od = torch.empty(n, dtype=torch.int32, device="cuda:0")
    ctx.graph_order(g, od)
    order = od.cpu().numpy().astype(np.int64)
    sdeg = deg[order]
    pre = np.concatenate([[0], np.cumsum(sdeg)])
    tot = int(pre[-1])
    cuts = [0] + [int(np.searchsorted(pre, tot * k // parts)) for k in range(1, parts)] + [n]
    out = []
    for lo, hi in zip(cuts, cuts[1:]):
        for _ in range(2):
            ctx.multilinear_rows(g, p, r, lo, hi)
        ts = []
        for _ in range(reps):
            ctx.multilinear_rows(g, p, r, lo, hi)
            ts.append(ctx.stats()["sweep_ms"][0])
        torch.cuda.synchronize()
        rk = r.cpu().numpy().view(np.uint64)
        written = int((rk != np.uint64(0xFFFFFFFFFFFFFFFF)).sum())
        nnz_s = int(pre[hi] - pre[lo])
        rows_s = int((sdeg[lo:hi] > 0).sum())
        b = 12.0 * nnz_s + 4.0 * (rows_s + 1) + 4.0 * rows_s + 8.0 * written
        med = float(np.median(ts))
        out.append({"rows": [lo, hi], "nnz": nnz_s, "rows_with_entries": rows_s,
                    "roots_written": written, "median_ms": med, "bytes": b,
                    "achieved": b / 1e9 / (med / 1e3)})
    slow = max(out, key=lambda x: x["median_ms"])
    return {"parts": parts, "order": "stored (degree-class) order, ranges balanced by entries",
            "slowest_ms": slow["median_ms"], "slowest_rows": slow["rows"],
            "sum_ms": float(sum(x["median_ms"] for x in out)),
            "frac_of_slowest": slow["achieved"] / HBM_PEAK_GBS, "unit": "GB/s",
            "shares": out}


def bench_batched(ctx, pkg, torch, G=10000, cpu=True):
    import numpy as np
    import gen

    vo, eo, e, w = gen.workload_batch_10k(G)
    de = torch.from_numpy(e.reshape(-1).copy()).to("cuda:0")
    dw = torch.from_numpy(w.view(np.int32).copy()).to("cuda:0")
    out = torch.empty(int(vo[-1]), dtype=torch.int32, device="cuda:0")
    ctx.solve_batched(vo, eo, de, dw, wtype=pkg.W_U32, out=out)  # warm (and tune)
    torch.cuda.synchronize()
    reps = 5
    t = time.perf_counter()
    for _ in range(reps):
        ids, counts, totals = ctx.solve_batched(vo, eo, de, dw, wtype=pkg.W_U32, out=out)
    torch.cuda.synchronize()
    tb = (time.perf_counter() - t) / reps
    st = ctx.stats()
    cfgs = pkg.batch_configs()
    kernel_ms = st["batch_ms"]
    # the same batch through the disjoint union and the round loop
    old = os.environ.get("MSF_BATCH_MODE")
    os.environ["MSF_BATCH_MODE"] = "0"
    try:
        cu = pkg.Context(0)
    finally:
        if old is None:
            os.environ.pop("MSF_BATCH_MODE", None)
        else:
            os.environ["MSF_BATCH_MODE"] = old
    cu.solve_batched(vo, eo, de, dw, wtype=pkg.W_U32, out=out)
    torch.cuda.synchronize()
    t = time.perf_counter()
    cu.solve_batched(vo, eo, de, dw, wtype=pkg.W_U32, out=out)
    torch.cuda.synchronize()
    t_union = time.perf_counter() - t
    cu.close()
    ids, counts, totals = ctx.solve_batched(vo, eo, de, dw, wtype=pkg.W_U32, out=out)
    # plain: one msf_solve per graph on the same context and stream (sample
    # of graphs, scaled to the batch by its edge share)
    step = max(1, G // 500)
    sample = list(range(0, G, step))
    one = torch.empty(65536, dtype=torch.int32, device="cuda:0")
    ee = [de[2 * eo[g]:2 * eo[g + 1]] for g in sample]
    ww = [dw[eo[g]:eo[g + 1]] for g in sample]
    for g_i, g in enumerate(sample[:20]):
        ctx.solve(int(vo[g + 1] - vo[g]), ee[g_i], ww[g_i], wtype=pkg.W_U32, out=one)
    torch.cuda.synchronize()
    t = time.perf_counter()
    for g_i, g in enumerate(sample):
        ctx.solve(int(vo[g + 1] - vo[g]), ee[g_i], ww[g_i], wtype=pkg.W_U32, out=one)
    torch.cuda.synchronize()
    tp = (time.perf_counter() - t) / len(sample)  # seconds per graph
    ci = st["batch_config"]
    res = {"graphs": G, "vertices": int(vo[-1]), "edges": int(eo[-1]),
           "batched_s": tb, "batched_graphs_per_s": G / tb,
           "batched_edges_per_s": float(eo[-1]) / tb,
           "persistent_kernel_ms": kernel_ms,
           "config": {"index": ci, "threads": cfgs[ci][0], "edges_per_thread": cfgs[ci][1],
                      "lds_bytes": cfgs[ci][2], "workgroups": st["batch_grid"]}
           if ci >= 0 else None,
           "union_path_s": t_union, "union_path_graphs_per_s": G / t_union,
           "plain_graphs_per_s": 1.0 / tp, "plain_sample_graphs": len(sample),
           "speedup": (G / tb) * tp}
    if cpu:
        res.update(batched_cpu(vo, eo, e, w, ids.cpu().numpy(), counts, totals, sample))
    return res


def batched_cpu(vo, eo, e, w, ids, counts, totals, sample):
    """The oracle on the batch's graphs: one thread over a sample (graphs/s,
    and element-wise parity of the batched result on those graphs), and
    every graph spread over the host's cores by a thread pool (the oracle's
    sort and union-find run outside the interpreter lock)."""
    import concurrent.futures as cf
    import numpy as np
    import oracle

    def one(g):
        n = int(vo[g + 1] - vo[g])
        return oracle.msf(n, e[eo[g]:eo[g + 1]], w[eo[g]:eo[g + 1]], oracle.W_U32)

    t = time.perf_counter()
    ok = True
    for g in sample:
        wi, wc, wt = one(g)
        ok &= bool(counts[g] == wc and np.array_equal(ids[vo[g]:vo[g] + wc].astype(np.int64), wi)
                   and totals[g][0] == wt[0])
    t1 = time.perf_counter() - t
    G = len(vo) - 1
    workers = min(16, len(os.sched_getaffinity(0)))
    t = time.perf_counter()
    with cf.ThreadPoolExecutor(workers) as ex:
        for _ in ex.map(one, range(G), chunksize=16):
            pass
    tall = time.perf_counter() - t
    return {"cpu_baseline": {"value": len(sample) / t1, "unit": "graphs/s", "cores": 1,
                             "kind": "oracle",
                             "sample": f"{len(sample)} of the {G} graphs (every "
                                       f"{sample[1] - sample[0]}th), one thread"},
            "cpu_parallel": {"value": G / tall, "unit": "graphs/s", "cores": workers,
                             "kind": "oracle", "sample": f"all {G} graphs, {workers} threads"},
            "parity_sample": ok}


def run_fifo(ctx, pkg, pool, arrivals, picks):
    """The plain FIFO actually run: one msf_solve at a time (host arrays in
    and out, as a served request), each request starting when it has
    arrived and the previous one is done.  Returns the latencies (s) and
    the time the last one finished."""
    import numpy as np

    lat = []
    t0 = time.perf_counter()
    for a, g in zip(arrivals, picks):
        now = time.perf_counter() - t0
        if now < a:
            time.sleep(a - now)
        n, e, w, kind = pool[g]
        ctx.solve(n, e, w, wtype=pkg.W_F32)
        lat.append(time.perf_counter() - t0 - a)
    return np.array(lat), time.perf_counter() - t0


def serve_stream(srv, pkg, pool, arrivals, picks):
    """Submit a Poisson stream to a server, collecting each result as soon
    as it is ready (while submitting), as a serving front end would.
    Returns the latencies (s, submit to ready) and the elapsed time."""
    import numpy as np

    pending = []
    lat = []

    def collect():
        keep = []
        for tk, n in pending:
            if srv.poll(tk):
                lat.append(srv.latency(tk))
                srv.result(tk, n)
            else:
                keep.append((tk, n))
        pending[:] = keep

    t0 = time.perf_counter()
    for a, g in zip(arrivals, picks):
        while True:
            collect()
            now = time.perf_counter() - t0
            if a <= now:
                break
            time.sleep(min(a - now, 0.0005))
        n, e, w, kind = pool[g]
        pending.append((srv.submit(n, e, w, wtype=pkg.W_F32), n))
    while pending:
        collect()
        if pending:
            time.sleep(0.0005)
    return np.array(lat), time.perf_counter() - t0


def bench_served(ctx, pkg, torch, requests_per_rate=2000, warm_requests=100,
                 rates=(0.25, 0.5, 1.0, 2.0, 4.0), budget=32 << 30,
                 budget_sweep=(8 << 30, 128 << 30), seed=5, cpu=False):
    """Poisson request stream over a pool of mixed graphs (half R-MAT with
    edge factor 16, half cubic grids with 5% of edges dropped, n log-uniform
    in [2^10, 2^22], float32 weights).  The rate is a multiple of the plain
    sequential throughput mu (one msf_solve per request, host arrays in and
    out, timed here).  At every rate the same arrivals also go through a
    plain FIFO that is actually run (one msf_solve at a time); the first
    `warm_requests` of each stream are not counted.  At the plain rate the
    server also runs under the budgets of `budget_sweep`.  With `cpu`, the
    oracle's service rate on the same pool is added (served_cpu)."""
    import numpy as np
    import gen

    t = time.perf_counter()
    pool = gen.serve_pool(64, seed=seed)
    log(f"served pool generated in {time.perf_counter() - t:.1f}s "
        f"({sum(len(p[1]) for p in pool)} edges)")
    svc = []
    for n, e, w, kind in pool:
        ctx.solve(n, e, w, wtype=pkg.W_F32)  # warm the workspace
    for n, e, w, kind in pool:
        t = time.perf_counter()
        ctx.solve(n, e, w, wtype=pkg.W_F32)
        svc.append(time.perf_counter() - t)
    mu = 1.0 / float(np.mean(svc))
    rng = np.random.default_rng(seed)
    total = warm_requests + requests_per_rate
    out = {"pool_graphs": len(pool), "requests_per_rate": requests_per_rate,
           "warm_requests_not_counted": warm_requests, "budget_bytes": budget,
           "plain_graphs_per_s": mu, "rates": [], "budgets": []}

    def stats(lat, elapsed, arrivals):
        lat = lat[warm_requests:]
        span = elapsed - arrivals[warm_requests]
        return {"p50_ms": 1e3 * float(np.percentile(lat, 50)),
                "p99_ms": 1e3 * float(np.percentile(lat, 99)),
                "graphs_per_s": requests_per_rate / span}

    servers = {}

    def server(b):
        if b not in servers:
            srv = pkg.Server(ctx, b)
            # warm: the whole pool at once, so slots, the device memory pool
            # and the pinned staging buffers reach their working set
            warm = [srv.submit(*p[:3], wtype=pkg.W_F32) for p in pool]
            for i, tk in enumerate(warm):
                srv.result(tk, pool[i][0])
            servers[b] = srv
        return servers[b]

    for mult in rates:
        lam = mult * mu
        arrivals = np.cumsum(rng.exponential(1.0 / lam, total))
        picks = rng.integers(0, len(pool), total)
        lat, el = serve_stream(server(budget), pkg, pool, arrivals, picks)
        sv = stats(lat, el, arrivals)
        flat, fel = run_fifo(ctx, pkg, pool, arrivals, picks)
        fv = stats(flat, fel, arrivals)
        row = {"rate_x_plain": mult, "arrival_per_s": lam,
               "served_p50_ms": sv["p50_ms"], "served_p99_ms": sv["p99_ms"],
               "served_graphs_per_s": sv["graphs_per_s"],
               "fifo_p50_ms": fv["p50_ms"], "fifo_p99_ms": fv["p99_ms"],
               "fifo_graphs_per_s": fv["graphs_per_s"]}
        out["rates"].append(row)
        log(f"served x{mult}: {row}")
        if mult == 1.0:
            for b in budget_sweep:
                lat, el = serve_stream(server(b), pkg, pool, arrivals, picks)
                bv = stats(lat, el, arrivals)
                out["budgets"].append({"budget_bytes": b, "rate_x_plain": mult,
                                       "served_p50_ms": bv["p50_ms"],
                                       "served_p99_ms": bv["p99_ms"],
                                       "served_graphs_per_s": bv["graphs_per_s"]})
                log(f"served x{mult} budget {b >> 30} GiB: {out['budgets'][-1]}")
                servers.pop(b).close()
    for srv in servers.values():
        srv.close()
    if cpu:
        log("served: the oracle on the pool")
        out.update(served_cpu(pool))
    return out


def served_cpu(pool):
    """The oracle's service rate on the served pool: every pool graph solved
    once by the oracle on one thread and on the host's cores (a thread pool;
    the oracle's sort and union-find run outside the interpreter lock), as
    graphs/s over the pool's size mix."""
    import concurrent.futures as cf
    import oracle

    def one(p):
        n, e, w, kind = p
        return oracle.msf(n, e, w, oracle.W_F32)

    t = time.perf_counter()
    for p in pool:
        one(p)
    t1 = time.perf_counter() - t
    workers = min(16, len(os.sched_getaffinity(0)))
    t = time.perf_counter()
    with cf.ThreadPoolExecutor(workers) as ex:
        for _ in ex.map(one, pool):
            pass
    tall = time.perf_counter() - t
    return {"cpu_baseline": {"value": len(pool) / t1, "unit": "graphs/s", "cores": 1,
                             "kind": "oracle",
                             "sample": f"the {len(pool)} pool graphs once each, one thread"},
            "cpu_parallel": {"value": len(pool) / tall, "unit": "graphs/s", "cores": workers,
                             "kind": "oracle",
                             "sample": f"the {len(pool)} pool graphs once each, {workers} "
                                       "threads"}}


def main():
    ap = argparse.ArgumentParser(description=__doc__.split("\n")[0])
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU oracle baseline")
    ap.add_argument("--no-extras", action="store_true",
                    help="skip the batched (10^4 graphs), served (Poisson stream) and "
                         "multilinear comparison legs")
    ap.add_argument("--no-ablation", action="store_true",
                    help="skip the all-at-once vs pairwise multilinear comparison")
    ap.add_argument("--ablation-only", action="store_true",
                    help="run only the multilinear comparison (prints its JSON alone)")
    ap.add_argument("--shortcut-only", action="store_true",
                    help="run only the shortcut-strategy study (prints its JSON alone)")
    ap.add_argument("--components-only", action="store_true",
                    help="run only the connected-components leg (prints its JSON alone)")
    ap.add_argument("--starcheck-only", action="store_true",
                    help="run only the original-AS-rounds leg (prints its JSON alone)")
    ap.add_argument("--multilinear-only", action="store_true",
                    help="run only msf_multilinear on R-MAT s22 with the parents after round 1")
    ap.add_argument("--served-only", action="store_true",
                    help="run only the served leg (prints its JSON alone)")
    ap.add_argument("--headline-only", action="store_true",
                    help="time only the R-MAT s22 solves and print the line without the "
                         "multilinear, plain, CPU and other legs (for profiling)")
    ap.add_argument("--plain-only", action="store_true",
                    help="run only the plain solves of the small Erdos-Renyi graph and the "
                         "256^3 grid (prints their JSON alone)")
    ap.add_argument("--batched-only", action="store_true",
                    help="run only the batched leg (prints its JSON alone)")
    ap.add_argument("--served-requests", type=int, default=2000,
                    help="requests per arrival rate in the served leg (after 100 not counted)")
    ap.add_argument("--copy-calibration", type=int, default=0, metavar="MIB",
                    help="first run a plain device copy of MIB MiB (a reference kernel "
                         "of known traffic for hardware byte counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on exactly one GPU; --gpus {args.gpus} is not supported "
              "(the hot path here is single-GPU; see the sharding notes in DESIGN.md)",
              file=sys.stderr)
        sys.exit(2)

    import torch

    import paper_2110_04865_amd as pkg

    if not torch.cuda.is_available():
        print("no GPU visible", file=sys.stderr)
        sys.exit(1)
    torch.cuda.set_device(0)
    if args.copy_calibration > 0:
        nbytes = args.copy_calibration << 20
        src = torch.ones(nbytes // 4, dtype=torch.int32, device="cuda:0")
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        log(f"calibration copy: {nbytes} bytes read, {nbytes} bytes written")
        del src, dst
    ctx = pkg.Context(0)
    if args.ablation_only:
        import gen

        n17, e17, w17 = gen.rmat(17, 8)
        n22, e22, w22 = gen.workload_rmat_s22()
        ab = bench_multilinear(ctx, pkg, torch, {"rmat_s17_e8": (n17, e17, w17),
                                                 "rmat_s22_e16": (n22, e22, w22)})
        print(json.dumps({"multilinear_ablation": ab}), flush=True)
        return
    if args.components_only:
        import gen

        n22, e22, w22 = gen.workload_rmat_s22()
        ng, eg, wg = gen.workload_grid_256()
        print(json.dumps({"components": bench_components(
            ctx, pkg, torch, {"rmat_s22_e16": (n22, e22, w22, pkg.W_F32),
                              "grid256": (ng, eg, wg, pkg.W_U32)})}), flush=True)
        return
    if args.starcheck_only:
        import gen

        n22, e22, w22 = gen.workload_rmat_s22()
        ng, eg, wg = gen.workload_grid_256()
        print(json.dumps({"starcheck": bench_starcheck(
            ctx, pkg, torch, {"rmat_s22_e16": (n22, e22, w22, pkg.W_F32),
                              "grid256": (ng, eg, wg, pkg.W_U32)})}), flush=True)
        return
    if args.multilinear_only:
        import gen

        n22, e22, w22 = gen.workload_rmat_s22()
        print(json.dumps({"multilinear": bench_multilinear_round1(ctx, pkg, torch, n22, e22, w22,
                                                                  pkg.W_F32)}), flush=True)
        return
    if args.served_only:
        print(json.dumps({"served": bench_served(ctx, pkg, torch, args.served_requests)}),
              flush=True)
        return
    if args.batched_only:
        print(json.dumps({"batched": bench_batched(ctx, pkg, torch, cpu=not args.no_cpu)}),
              flush=True)
        return
    if args.plain_only:
        import gen

        n1, e1, w1 = gen.workload_er_4096()
        plain = {"er4096": bench_plain(ctx, pkg, torch, "Erdos-Renyi n=4096 m=32768, uint32 "
                                       "weights", n1, e1, w1, pkg.W_U32, steps=50,
                                       cpu=not args.no_cpu)}
        n3, e3, w3 = gen.workload_grid_256()
        plain["grid256"] = bench_plain(ctx, pkg, torch, "3D grid 256^3, 5% of edges dropped, "
                                       "uint32 weights", n3, e3, w3, pkg.W_U32, steps=5,
                                       cpu=not args.no_cpu)
        print(json.dumps({"plain": plain}), flush=True)
        return
    if args.shortcut_only:
        print(json.dumps({"shortcut_study": bench_shortcut(ctx, pkg, torch)}), flush=True)
        return
    r = bench_rmat(ctx, pkg, torch, args.steps, args.warmup)
    m = r["m"]
    n = r["n"]
    value = m / (r["ms"] / 1000.0)
    kt = r["kernels"]
    steps = args.steps
    # the adjacency build is the dominant unit (most device time per step);
    # its bytes are what the method must move to build A (both directions
    # of every edge with its key): the edge list and weights read once
    # (12 m), column and key of every stored entry written once (12 nnz),
    # the row pointers (4 (n + 1)) and round 1's minima kept by the build
    # (8 n); its time is the device time from the solve's start to the end
    # of the placement (the run sort of the head sweep is a unit of its own,
    # and its set-up and the host step after the build belong to neither)
    nnz = 2 * m
    build_bytes = 12.0 * m + 12.0 * nnz + 4.0 * (n + 1) + 8.0 * n
    sort_ms = kt["sort"][0] / steps
    build_only_ms = r["adjacency_ms"] if r["adjacency_ms"] > 0 else r["build_ms"] - sort_ms
    units = {
        "build": (build_only_ms, build_bytes,
                  "adjacency build (k_bucket_hist, the scans, k_part_edges, k_tl_plan, "
                  "k_tl_hist2, k_part_sub, k_tl_fstart, k_tl_order, k_tl_place)"),
        "sort": (sort_ms, kt["sort"][1] / max(1, kt["sort"][2]),
                 "k_sort_chunks (run sort of the head sweep; 13 B per stored entry: key and "
                 "column read, order byte written; 16 B per run, 4 B per chunk)"),
        "heads": (kt["heads"][0] / steps, kt["heads"][1] / steps,
                  "k_heads + k_heads_rest (head sweeps of one solve; 24 B per run and sweep)"),
    }
    if r["stats"]["path"] == 4:
        # rounds over a contracted edge list: no adjacency is built.  The
        # selection reads the input once (12 m) and writes 16 bytes an edge of
        # the first list; what follows the first round reads the input's ends
        # once more (8 m) and, a round, 16 bytes an edge still on the list.
        on_list = [x / 2 for x in r["stats"]["active_nnz"]]
        first_ms = r["build_ms"] - r["adjacency_ms"]
        units = {
            "select": (r["adjacency_ms"], 12.0 * m + 16.0 * on_list[0],
                       "k_ct_init, k_ct_select (light edges' list)"),
            "first_round": (first_ms, 16.0 * on_list[0] + 16.0 * n,
                            "k_ct_edges<true>, k_ct_hook, k_ct_chase (first round)"),
            "rounds": (r["rounds_ms"], 8.0 * m + 16.0 * sum(on_list[1:]),
                       "k_ct_edges, k_ct_hook, k_ct_chase, k_ct_compose, k_ct_between, the "
                       "output (all after the first round)"),
        }
    dom = max(units, key=lambda k: units[k][0])
    d_ms, d_bytes, d_name = units[dom]
    achieved = (d_bytes / 1e9) / (d_ms / 1e3) if d_ms > 0 else 0.0
    line = {
        "metric": "MSF edges/s at R-MAT s22 (% HBM peak); batched graphs/s vs plain; p99 latency",
        "value": value,
        "unit": "edges/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": r["ms"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "u64",
        "data": "synthetic",
        "config": {"workload": "R-MAT scale 22, edge factor 16, a/b/c/d=.57/.19/.19/.05, "
                               "permuted ids, simple graph, float32 weights",
                   "n": n, "m": m, "nnz": nnz, "rounds": r["stats"]["rounds"],
                   "build_ms": r["build_ms"], "adjacency_ms": r["adjacency_ms"],
                   "rounds_ms": r["rounds_ms"]},
        "roofline": {"bound": "hbm", "kernel": d_name,
                     "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK_GBS, "traffic": measured_traffic(dom) if dom in KERNELS else None,
                     "avg_launch_ms": d_ms, "bytes_per_launch": d_bytes,
                     "units_ms_per_step": {k: v[0] for k, v in units.items()},
                     "kernel_ms_per_step": {k: v[0] / steps for k, v in kt.items()}},
        "host": host_info(),
    }
    if args.headline_only:
        print(json.dumps(line), flush=True)
        return
    log("multilinear kernel with the parents after round 1")
    line["multilinear"] = bench_multilinear_round1(ctx, pkg, torch, n, r["e"], r["w"], pkg.W_F32)
    log(f"multilinear: {line['multilinear']}")
    if not args.no_cpu:
        log("timing the CPU oracle on the same graph")
        cb = cpu_baseline(n, r["e"], r["w"])
        line["cpu_baseline"] = {"value": m / cb["seconds"], "unit": "edges/s", "cores": 1,
                                "kind": "oracle",
                                "sample": f"the full R-MAT s22 graph ({m} edges), one "
                                          "sort + union-find solve, single thread",
                                "seconds": cb["seconds"]}
        line["parity"] = bool(same_forest(r["ids"], r["count"], r["total"], cb, 1))
    import gen

    log("plain solves of the other single-graph configurations")
    n1, e1, w1 = gen.workload_er_4096()
    plain = {"er4096": bench_plain(ctx, pkg, torch, "Erdos-Renyi n=4096 m=32768, uint32 "
                                   "weights", n1, e1, w1, pkg.W_U32, steps=50,
                                   cpu=not args.no_cpu)}
    n3, e3, w3 = gen.workload_grid_256()
    plain["grid256"] = bench_plain(ctx, pkg, torch, "3D grid 256^3, 5% of edges dropped, "
                                   "uint32 weights", n3, e3, w3, pkg.W_U32, steps=5,
                                   cpu=not args.no_cpu)
    del e3, w3
    line["plain"] = plain
    if not args.no_extras:
        log("batched: 10^4 Erdos-Renyi graphs")
        line["batched"] = bench_batched(ctx, pkg, torch, cpu=not args.no_cpu)
        log("served: Poisson stream of mixed graphs")
        sv = bench_served(ctx, pkg, torch, args.served_requests, cpu=not args.no_cpu)
        line["served"] = sv
        at1 = [r for r in sv["rates"] if r["rate_x_plain"] == 1.0]
        if at1:
            line["served_p99_ms_at_plain_rate"] = at1[0]["served_p99_ms"]
    if not args.no_extras and not args.no_ablation:
        import gen

        log("multilinear: all-at-once vs pairwise")
        n17, e17, w17 = gen.rmat(17, 8)
        line["multilinear_ablation"] = bench_multilinear(
            ctx, pkg, torch, {"rmat_s17_e8": (n17, e17, w17),
                              "rmat_s22_e16": (r["n"], r["e"], r["w"])})
        log("shortcut strategies on the 256^3 grid")
        line["shortcut_study"] = bench_shortcut(ctx, pkg, torch)
        log("connected components")
        ng, eg, wg = gen.workload_grid_256()
        line["components"] = bench_components(
            ctx, pkg, torch, {"rmat_s22_e16": (r["n"], r["e"], r["w"], pkg.W_F32),
                              "grid256": (ng, eg, wg, pkg.W_U32)})
        log("original AS rounds (star check)")
        line["starcheck"] = bench_starcheck(
            ctx, pkg, torch, {"rmat_s22_e16": (r["n"], r["e"], r["w"], pkg.W_F32),
                              "grid256": (ng, eg, wg, pkg.W_U32)})
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
