"""Benchmark: aligned reads/s for 2 x 100 bp pairs (<= 4 diffs) on one MI355X.

Workload: 100 Mbp synthetic genome (41% GC, 40% repeat copies from 500
families) and 1M read pairs 2 x 100 bp (fragment ~ N(300, 30), 1%
substitutions, 0.1% indel events), seeded.  One step = the whole path over
the batch -- align both ends, locate, pair -- with reads and index resident
in HBM before the timed region.  Three forms are timed and must agree bit
for bit: plain (one lane per read, one launch per end), batched-eager (one
persistent work-stealing launch for both ends, then locate and pair, each
call enqueued by the host) and batched (the same step captured once into a
hipGraph and replayed); `value` is the batched one.  The batched form's
residency is picked first by the autotuner on the same batch.

Prints one JSON line.  The roofline entry is for the dominant kernel (the
persistent search), timed with HIP events around it on its stream (events
captured into the graph); its bytes per launch are counter-measured
(profiles/), since the search takes most of the rank lines that the oracle's
backward search touches (reported beside it) from interval tables and the
text instead.  The CPU baseline is the oracle itself on a bounded sample of the
same pairs.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import threading
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "aligned reads/s (2x100bp, <=4 diffs) on 1 MI355X, batched vs plain; p99 ms"
HBM_PEAK_GBS = 8000.0
# 32-bit integer vector ALU: 256 CUs x 4 SIMDs x 16 lanes x 2.4 GHz, one op per lane per clock
INT_ALU_PEAK_TOPS = 256 * 4 * 16 * 2.4e9 / 1e12
# integer operations of the affine local-alignment recurrence per cell: the
# gap along the reference (2 subtractions, 1 max), the gap along the read
# (same), the substitution score (compare, select, add) and H (3 maxes)
RESCUE_OPS_PER_CELL = 12


def host_threads() -> int:
    """Threads for the oracle's timed sample: every CPU this process may run
    on, capped by the job's thread allowance when the environment sets one
    (OMP_NUM_THREADS: a shared host's share for this job)."""
    n = len(os.sched_getaffinity(0))
    cap = os.environ.get("OMP_NUM_THREADS", "")
    if cap.isdigit() and int(cap) > 0:
        n = min(n, int(cap))
    return max(n, 1)


def log(msg):
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


# sources each profiled kernel is built from; a counter summary is valid only for them
KERNEL_SOURCES = {"k_align_persistent": ("bwfm.hip", "bwfm_internal.h"),
                  "k_rescue": ("rescue.hip", "bwfm_internal.h"),
                  "k_mapq": ("mapq.hip", "bwfm_internal.h")}


def kernel_source_hash(kernel: str = "k_align_persistent") -> str:
    """Hash of a kernel's sources; byte counters are valid only for it."""
    import hashlib
    h = hashlib.sha256()
    for f in KERNEL_SOURCES[kernel]:
        with open(os.path.join(ROOT, "paper_1505_07855_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def traffic_from_profiles(kernel: str, workload: str = "c2", **match):
    """HBM-side bytes per launch of `kernel` from the committed counter summary
    (FETCH_SIZE and WRITE_SIZE per dispatch, each scaled by what the same
    counter reads for a device copy of known size), or None when the summary
    was taken on other kernel sources or with other settings.  A summary may
    hold several records (one per setting); the first whose kernel, sources
    and `match` keys all agree is used."""
    path = os.path.join(ROOT, "profiles", f"{kernel}_{workload}_bytes.md")
    if not os.path.exists(path):
        return None
    rec = None
    with open(path) as fh:
        for line in fh:
            if not line.startswith("bench-traffic:"):
                continue
            r = dict(kv.split("=", 1) for kv in line.split()[1:])
            if (r.get("kernel") == kernel and r.get("source") == kernel_source_hash(kernel)
                    and all(r.get(k) == str(v) for k, v in match.items())):
                rec = r
                break
    if rec is None:
        return None
    cb = float(rec["copy_bytes"])
    fetch = float(rec["fetch_kib"]) * 1024 * cb / (float(rec["copy_fetch_kib"]) * 1024)
    write = float(rec["write_kib"]) * 1024 * cb / (float(rec["copy_write_kib"]) * 1024)
    return fetch + write


def rescue_leg(bw, torch, ix, ends, results, prs, n, w, stream, launches, n_ref, max_diff):
    """Mate rescue, then mapping quality, over the step's pair records, each
    timed alone with HIP events on its stream; rescue work is m x window cells
    per rescued-for pair."""
    out = bw.rescue_mates(ix, ends[0], ends[1], prs, w["lo"], w["hi"], max_len=100, stream=stream)
    torch.cuda.synchronize()
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    ev0.record(stream)
    for _ in range(launches):
        bw.rescue_mates(ix, ends[0], ends[1], prs, w["lo"], w["hi"], max_len=100, stream=stream, out=out)
    ev1.record(stream)
    torch.cuda.synchronize()
    ms = ev0.elapsed_time(ev1) / launches
    res = bw.rescue_numpy(out)[:n]
    pr = bw.pairs_numpy(prs)[:n]
    f = pr["flags"]
    m1, m2 = (f & bw.PF_MAPPED1) != 0, (f & bw.PF_MAPPED2) != 0
    cand = ((f & bw.PF_PAIRED) == 0) & (m1 | m2)
    a1 = m1 & (~m2 | (pr["score1"] <= pr["score2"]))
    pa = np.where(a1, pr["pos1"], pr["pos2"]).astype(np.int64)
    la = np.where(a1, pr["len1"], pr["len2"]).astype(np.int64)
    sa = np.where(a1, pr["strand1"], pr["strand2"])
    w_fwd = np.minimum(pa + w["hi"], n_ref) - pa
    w1 = np.minimum(pa + la, n_ref)
    w_rev = w1 - np.maximum(w1 - w["hi"], 0)
    width = np.clip(np.where(sa == 0, w_fwd, w_rev), 0, None)
    lens = [np.diff(e[1].cpu().numpy()) for e in ends]
    m = np.where(a1, lens[1], lens[0])
    cells = float((m * width)[cand].sum())
    cps = cells / (ms / 1e3)
    achieved = cps * RESCUE_OPS_PER_CELL / 1e12
    # mapping quality of both ends over the same records (a streaming kernel)
    mq = bw.mapq(results[0], results[1], prs, rescue=out, max_diff=max_diff, stream=stream)
    torch.cuda.synchronize()
    ev0.record(stream)
    for _ in range(launches):
        bw.mapq(results[0], results[1], prs, rescue=out, max_diff=max_diff, stream=stream, out=mq)
    ev1.record(stream)
    torch.cuda.synchronize()
    mq_ms = ev0.elapsed_time(ev1) / launches
    # per pair: its record (24 B), rescue record (16 B), two MAPQ bytes, and per
    # end an offset (8 B), c1, c2, status (9 B) and at least one hit (16 B)
    mq_bytes = n * (24 + 16 + 2 + 2 * (8 + 9 + 16))
    mq_gbs = mq_bytes / (mq_ms / 1e3) / 1e9
    q = mq.cpu().numpy()[:n]
    return {"kernel": "k_rescue", "candidates": int(cand.sum()), "rescued": int((res["end"] != 0).sum()),
            "avg_launch_ms": ms, "launches": launches, "cells": cells, "gcups": cps / 1e9,
            "pairs_per_s": n / (ms / 1e3),
            "roofline": {"bound": "alu", "achieved": achieved, "peak": INT_ALU_PEAK_TOPS, "unit": "Tops/s",
                         "frac": achieved / INT_ALU_PEAK_TOPS, "traffic": traffic_from_profiles("k_rescue"),
                         "ops_per_cell": RESCUE_OPS_PER_CELL},
            "mapq": {"kernel": "k_mapq", "avg_launch_ms": mq_ms, "launches": launches,
                     "q60_fraction": float((q == 60).mean()), "q0_fraction": float((q == 0).mean()),
                     "roofline": {"bound": "hbm", "achieved": mq_gbs, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                                  "frac": mq_gbs / HBM_PEAK_GBS, "traffic": traffic_from_profiles("k_mapq"),
                                  "bytes_per_launch": mq_bytes}}}


def served_leg(bw, torch, ix, g, args, stream):
    """The served form on the resident index, with serving-shaped requests
    (76-150 bp pairs, 1% substitutions, 0.1% indel events, per-read budgets
    from the length rule, sizes log-uniform in [1k, 200k] pairs).

    First the same inputs through all three forms: a fixed set of requests
    aligned as one batch by the plain form (a launch per end) and by the
    batched form (both ends in one persistent launch), each followed by
    pairing, and submitted at once to the server; the pair records must be
    identical, and each form's rate is reads over the wall time to the last
    record.  Then Poisson streams at fractions rho of the server's capacity
    from that burst: request latency (submit to records on the host) p50
    and p99, and reads/s over the replay."""
    from gen import configs
    from paper_1505_07855_amd import serve

    w = configs.PAIR_WINDOW
    params = dict(configs.PARAMS["C3"])
    # same inputs, three forms
    reqs = serve.make_requests(g, args.serve_same_requests, 7001, 1000, 200_000)
    n = sum(r[4] for r in reqs)
    b1 = np.concatenate([r[0] for r in reqs])
    b2 = np.concatenate([r[2] for r in reqs])

    def cat_offsets(k):
        parts, base = [np.zeros(1, np.uint64)], np.uint64(0)
        for r in reqs:
            o = r[k].astype(np.uint64)
            parts.append(o[1:] - o[0] + base)
            base = parts[-1][-1]
        return np.concatenate(parts)

    o1, o2 = cat_offsets(1), cat_offsets(3)
    L = np.concatenate([np.diff(o1), np.diff(o2)]).astype(np.int64)
    rule = np.array([min(bw.max_diff_rule(x), 15) for x in range(513)], np.uint8)
    md = torch.from_numpy(rule[L]).cuda()
    ends = [(torch.from_numpy(b).cuda(), torch.from_numpy(o.view(np.int64)).cuda()) for b, o in ((b1, o1), (b2, o2))]
    both_b = torch.cat([ends[0][0], ends[1][0]])
    both_o = torch.from_numpy(np.concatenate([o1[:-1], o1[-1] + o2]).view(np.int64)).cuda()
    forms = {}
    recs = {}
    for name, form in (("plain", bw.FORM_PLAIN), ("batched", bw.FORM_BATCHED)):
        p = bw.Params(**params, form=form)
        best = None
        for rep in range(3):  # the first call grows workspaces
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            if form == bw.FORM_PLAIN:
                r1 = bw.align_batch(ix, ends[0][0], ends[0][1], p, max_diff=md[:n], max_len=150, stream=stream)
                r2 = bw.align_batch(ix, ends[1][0], ends[1][1], p, max_diff=md[n:], max_len=150, stream=stream)
            else:
                r = bw.align_batch(ix, both_b, both_o, p, max_diff=md, max_len=150, stream=stream)
                r1, r2 = r.window(0, n), r.window(n, 2 * n)
            prs = bw.pair_reads(ix, r1, r2, w["lo"], w["hi"], w["mu"], configs.MAX_OCC, stream=stream)
            torch.cuda.synchronize()
            dt = time.perf_counter() - t0
            best = dt if best is None else min(best, dt)
        recs[name] = bw.pairs_numpy(prs)[:n].copy()
        forms[name] = {"reads_per_s": 2 * n / best, "ms": best * 1e3}
        log(f"served leg, same inputs: {name} {best * 1e3:.1f} ms")
    srv = bw.Server(ix, bw.Params(**params), w["lo"], w["hi"], w["mu"], configs.MAX_OCC,
                    arena_bytes=args.serve_arena_mib << 20, step_pairs=args.serve_step_pairs, max_len=150,
                    budget_rule=True)
    try:
        serve.replay(srv, reqs[:2], 0.0, 1)  # warm-up: the server's first steps
        best, lat = None, None
        for rep in range(2):
            lt, wall = serve.replay(srv, reqs, 0.0, 1)
            if best is None or wall < best:
                best, lat = wall, lt
        # the records of the same burst, collected request by request
        outs = []
        tk = [srv.submit(r[0], r[1], r[2], r[3]) for r in reqs]
        for t, r in zip(tk, reqs):
            outs.append(srv.wait(t, r[4])[0])
        got = np.concatenate(outs)
        forms["served"] = {"reads_per_s": 2 * n / best, "ms": best * 1e3, "note": "burst of every request at once"}
        log(f"served leg, same inputs: served {best * 1e3:.1f} ms")
        same = (np.array_equal(recs["plain"].view(np.uint8), recs["batched"].view(np.uint8))
                and np.array_equal(got.view(np.uint8), recs["batched"].view(np.uint8)))
        if not same:
            raise SystemExit("served, batched and plain forms disagree on the same requests")
        cap_pairs = n / best
        mean_size = (200_000 - 1000) / np.log(200_000 / 1000)
        rates = []
        for k, rho in enumerate(args.serve_rates):
            rq = serve.make_requests(g, args.serve_requests, 5000 + k, 1000, 200_000)
            lam = rho * cap_pairs / mean_size
            lt, wall = serve.replay(srv, rq, lam, 77 + k)
            sm = serve.summarize(lt, wall, rq)
            sm.update({"rho": rho, "arrivals_per_s": lam})
            rates.append(sm)
            log(f"served leg: rho {rho}: p50 {sm['p50_ms']:.1f} ms, p99 {sm['p99_ms']:.1f} ms, "
                f"{sm['reads_per_s'] / 1e6:.2f} M reads/s")
            del rq
        stats = srv.stats()
    finally:
        srv.close()
    return {"workload": f"requests of 1k-200k pairs, 76-150 bp, 1% substitutions, 0.1% indel events, budgets by "
                        f"the length rule, on the resident {len(g.seq) / 1e6:.0f} Mbp index",
            "same_inputs": {"requests": len(reqs), "pairs": n, "identical_records": True, **forms},
            "capacity_pairs_per_s": cap_pairs, "step_pairs": args.serve_step_pairs, "rates": rates,
            "server": stats}


def main_se(args):
    """A single-end workload at its stated size: C1 (1 Mbp i.i.d. genome,
    10,000 reads of 36 bp, 2% substitutions, at most 2 mismatches, no gaps;
    64-byte lines of 128 rows) or C5 (the 100 Mbp genome, 2M reads of 250 bp,
    3% substitutions and 0.3% indel events, a tenth from repeat copies, at
    most 6 differences with a gap, no seed; 128-byte sub-counted lines).  One
    step aligns the whole batch and locates every reported hit; the plain
    form (one lane per read) and the batched form (one persistent launch)
    are timed and must agree (the plain form on C5 over a leading part of
    the batch only: its waves wait for their slowest reads).  The roofline is
    counter-measured; the oracle's line touches per read over a leading
    sample, which is also the CPU baseline, stand beside it."""
    import torch

    import oracle
    import paper_1505_07855_amd as bw
    from gen import configs

    torch.cuda.set_device(0)
    cfg = args.config.upper()
    t0 = time.time()
    if cfg == "C1":
        g = configs.c1_genome()
        reads = configs.c1_reads(g)
        max_len, sample = 36, reads.n
    else:
        g = configs.c2_genome()
        reads = configs.c5_reads(g)
        max_len, sample = 250, min(args.cpu_reads, reads.n)
    lay = configs.LAYOUT[cfg]
    box = {}
    th = threading.Thread(target=lambda: box.update(ox=oracle.Index(g.seq)))
    if not args.no_cpu:
        th.start()
    ix = bw.Index.build_device(g.seq, **lay)
    log(f"{cfg}: {len(g.seq)} bp genome, {reads.n} reads, device index in {time.time() - t0:.1f}s")
    b = torch.from_numpy(reads.bases).cuda()
    o = torch.from_numpy(reads.offsets.view(np.int64)).cuda()
    n = reads.n
    # the plain form, one lane per read, waits for each wave's slowest read;
    # on the stress batch that makes a launch over all 2M reads run for
    # minutes, so it is timed on a leading part of the batch there
    n_plain = n if cfg == "C1" else min(args.plain_reads, n)
    # the batched form's split budget: the one given, or on the stress batch
    # the fastest of the library's default and three smaller ones, each
    # candidate's output byte-identical to the first's (a tuning knob like
    # the layout)
    split_tune = None
    split = args.split_budget
    if split is None:
        split = 0
        if cfg == "C5":
            split_tune, ref = [], None
            for cand in (0, 4096, 1024, 512):
                p = bw.Params(**configs.PARAMS[cfg], split_budget=cand)
                r = bw.align_batch(ix, b, o, p, max_len=max_len, hit_capacity=16 * n)
                torch.cuda.synchronize()
                ts = time.perf_counter()
                r = bw.align_batch(ix, b, o, p, max_len=max_len, out=r)
                torch.cuda.synchronize()
                ms = (time.perf_counter() - ts) * 1e3
                st = r.status.cpu().numpy()
                d = [x.tobytes() for x in r.to_numpy()[:4]] + [(st & 7).tobytes()]
                if ref is not None and d != ref:
                    raise SystemExit(f"split budget {cand} changes the output")
                ref = ref or d
                split_tune.append({"split_budget": cand, "ms": ms})
                log(f"{cfg}: split budget {cand or 'default'}: {ms:.1f} ms")
            split = min(split_tune, key=lambda x: x["ms"])["split_budget"]
    out = {}
    res = {}
    for name, form in (("plain", bw.FORM_PLAIN), ("batched", bw.FORM_BATCHED)):
        p = bw.Params(**configs.PARAMS[cfg], form=form, split_budget=split if form == bw.FORM_BATCHED else 0)
        nn = n_plain if form == bw.FORM_PLAIN else n
        b_, o_ = (b, o) if nn == n else (b[:int(reads.offsets[nn])], o[:nn + 1])
        ts = time.perf_counter()
        r = bw.align_batch(ix, b_, o_, p, max_len=max_len, hit_capacity=16 * nn)
        bw.locate(ix, r, configs.MAX_OCC)
        torch.cuda.synchronize()
        log(f"{cfg} {name}: first call {(time.perf_counter() - ts) * 1e3:.1f} ms")
        for i in range(args.warmup):
            ts = time.perf_counter()
            r = bw.align_batch(ix, b_, o_, p, max_len=max_len, out=r)
            bw.locate(ix, r, configs.MAX_OCC)
            torch.cuda.synchronize()
            if cfg != "C1":
                log(f"{cfg} {name}: warmup {i + 1}/{args.warmup} {(time.perf_counter() - ts) * 1e3:.1f} ms")
        bw.timing_enable(True)
        bw.timing_reset()
        times = []
        for i in range(args.steps):
            ts = time.perf_counter()
            r = bw.align_batch(ix, b_, o_, p, max_len=max_len, out=r)
            bw.locate(ix, r, configs.MAX_OCC)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - ts)
            if cfg != "C1":
                log(f"{cfg} {name}: step {i + 1}/{args.steps} {times[-1] * 1e3:.1f} ms")
        bw.timing_enable(False)
        # the batched form's search: the D-array pre-pass (long reads), the
        # first pass, the split searches' rounds and their publication
        key = "align_plain" if form == bw.FORM_PLAIN else "align_search"
        kms, kl = bw.timing_get(key)
        if form == bw.FORM_BATCHED:
            dms, dl = bw.timing_get("dscan")
            kms += dms if dl == kl else 0.0
        st = r.status.cpu().numpy()
        aligned = int(((st & bw.ST_HIT) != 0).sum())
        ms = float(np.mean(times) * 1e3)
        out[name] = {"reads": nn, "ms_per_step": ms, "aligned_reads_per_s": aligned / (ms / 1e3),
                     "reads_per_s": nn / (ms / 1e3),
                     "aligned": aligned, "overflow_reads": int(((st & bw.ST_OVERFLOW) != 0).sum()),
                     "kernel_ms": kms / kl if kl else None}
        rv = r.window(0, n_plain).to_numpy() if nn != n_plain else r.to_numpy()
        res[name] = [x.tobytes() for x in rv[:4]] + [(rv[4] & 7).tobytes()]
        log(f"{cfg} {name}: {ms:.2f} ms per step, {aligned} aligned")
    if res["plain"] != res["batched"]:
        raise SystemExit("plain and batched forms disagree")
    # the faster form over the whole batch (the plain form only covers the
    # whole batch on C1)
    best = min(("plain", "batched"), key=lambda k: out[k]["ms_per_step"]) if n_plain == n else "batched"
    roofline, cpu = None, None
    if not args.no_cpu:
        th.join()
        ox = box["ox"]
        op = oracle.Params(**configs.PARAMS[cfg], bases_per_line=ix.info()["bases_per_line"])
        nthreads = args.cpu_threads or host_threads()
        sb, so = reads.bases[:int(reads.offsets[sample])], reads.offsets[:sample + 1]
        # the sample again until at least 5 s of host work (C1's whole batch
        # takes a fraction of a second)
        log(f"{cfg}: oracle on the first {sample} reads, {nthreads} threads")
        t0 = time.perf_counter()
        rounds, cpu_aligned = 0, 0
        while rounds == 0 or time.perf_counter() - t0 < 5.0:
            orr = oracle.align(ox, sb, so, op, threads=nthreads)
            oracle.locate(ox, orr.hits, configs.MAX_OCC)
            cpu_aligned += int(((orr.status & oracle.ST_HIT) != 0).sum())
            rounds += 1
            if cfg != "C1":
                log(f"{cfg}: oracle round {rounds} done at {time.perf_counter() - t0:.1f} s")
        cpu_s = time.perf_counter() - t0
        cpu = {"value": cpu_aligned / cpu_s, "unit": "aligned reads/s", "cores": nthreads, "kind": "oracle",
               "host_cpus_visible": len(os.sched_getaffinity(0)),
               "sample": f"first {sample} reads of the same batch, {rounds} time(s): align, locate; {cpu_s:.1f} s"}
        touches = (orr.counts["touch_s"] + orr.counts["touch_d"]).astype(np.float64)
        kms = out[best]["kernel_ms"]
        if kms:
            roofline = {"bound": "hbm", "achieved": None, "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": None,
                        "traffic": None,
                        "kernel": ("k_align_plain" if best == "plain" else
                                   "k_dscan + k_align_persistent + k_align_tasks"),
                        "reads_per_launch": n, "avg_launch_ms": kms, "line_touches_per_read": float(touches.mean()),
                        "basis": "counter-measured HBM-side bytes per step of the search"}
            if best == "batched" and cfg == "C5":
                # counter-measured bytes of the same kernels at the same split
                # budget (the budget moves work between the first pass and the
                # rounds), summed over one step's launches
                traffic = traffic_from_profiles("k_align_persistent", "c5", split=split)
                roofline["traffic"] = traffic
                if traffic:
                    rate = traffic / (kms / 1e3) / 1e9
                    roofline["achieved"] = rate
                    roofline["frac"] = rate / HBM_PEAK_GBS
    ms_step = out[best]["ms_per_step"]
    line = {
        "metric": f"aligned reads/s ({cfg} single-end) on 1 MI355X", "value": out[best]["aligned_reads_per_s"],
        "unit": "aligned reads/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms_step,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "u32", "data": "synthetic",
        "config": {"workload": (f"C1 tiny: 1 Mbp i.i.d. genome, {n} single-end 36 bp reads, 2% substitutions, "
                                "<=2 mismatches, no gaps" if cfg == "C1" else
                                f"C5 stress: 100 Mbp synthetic genome, {n} single-end 250 bp reads, 3% substitutions, "
                                "0.3% indel events, 10% from repeats, <=6 diffs with a gap, no seed"),
                   "reads": n, "form": best, "line_bytes": lay["line_bytes"], "rank_format": lay["rank_format"],
                   "split_budget": split or "default (16384)", "parallelism": "1 GPU"},
        "split_tune": split_tune,
        "plain": out["plain"], "batched": out["batched"], "roofline": roofline, "cpu_baseline": cpu,
    }
    print(json.dumps(line), flush=True)


def main_c3(args):
    """The uneven-length workload at full size (3.1 Gbp reference indexed on
    the device, 10M pairs of 36-150 bp with per-read budgets): the batched
    step (both ends in one persistent launch, locate, pair), timed as the
    default workload is.  The oracle cannot index 3.1 Gbp within a bench run,
    so there is no CPU baseline and no algorithmic byte count: the bytes come
    from the committed FETCH_SIZE summary of this workload."""
    import torch

    import paper_1505_07855_amd as bw
    from gen import configs

    torch.cuda.set_device(0)
    genome = args.genome if args.genome != 100_000_000 else 3_100_000_000
    n = args.pairs if args.pairs != 1_000_000 else 10_000_000
    t0 = time.time()
    g = configs.c2_genome(genome, seed=1003)
    ix = bw.Index.build_device(g.seq, **configs.LAYOUT["C3"], kmer_levels=args.kmer_levels)
    pairs = configs.c3_pairs(g, n)
    log(f"C3 inputs and device index in {time.time() - t0:.1f}s ({ix.info()['device_bytes'] / 1e9:.2f} GB)")
    e1, e2 = pairs.end1, pairs.end2
    L = np.concatenate([np.diff(e1.offsets), np.diff(e2.offsets)]).astype(np.int64)
    rule = np.array([bw.max_diff_rule(x) for x in range(513)], np.uint8)
    md = torch.from_numpy(rule[L]).cuda()
    bases = torch.from_numpy(np.concatenate([e1.bases, e2.bases])).cuda()
    offs = torch.from_numpy(np.concatenate([e1.offsets[:-1], e1.offsets[-1] + e2.offsets]).view(np.int64)).cuda()
    del g, pairs
    p = bw.Params(**configs.PARAMS["C3"], waves_per_simd=args.waves_per_simd)
    w = configs.PAIR_WINDOW
    state = [None, None]

    def step():
        state[0] = bw.align_batch(ix, bases, offs, p, max_diff=md, max_len=150, out=state[0], hit_capacity=16 * n)
        r1, r2 = state[0].window(0, n), state[0].window(n, 2 * n)
        state[1] = bw.pair_reads(ix, r1, r2, w["lo"], w["hi"], w["mu"], configs.MAX_OCC, out=state[1])
        return r1, r2

    for i in range(args.warmup):
        step()
        torch.cuda.synchronize()
        log(f"C3 warmup step {i + 1}/{args.warmup} done")
    bw.timing_enable(True)
    bw.timing_reset()
    times = []
    for i in range(args.steps):
        t = time.perf_counter()
        r1, r2 = step()
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t)
        log(f"C3 step {i + 1}/{args.steps}: {times[-1] * 1e3:.1f} ms")
    bw.timing_enable(False)
    # the search: the first pass, then the split searches' rounds and
    # their publication
    kms, kl = bw.timing_get("align_search")
    k_ms = kms / kl if kl else None
    st = state[0].status.cpu().numpy()
    aligned = int(((st & bw.ST_HIT) != 0).sum())
    ms_step = sum(times) / len(times) * 1e3
    value = aligned / (ms_step / 1e3)
    roofline = None
    traffic = traffic_from_profiles("k_align_persistent", "c3")
    if k_ms:
        roofline = {"bound": "hbm", "achieved": traffic / (k_ms / 1e3) / 1e9 if traffic else None,
                    "peak": HBM_PEAK_GBS, "unit": "GB/s",
                    "frac": traffic / (k_ms / 1e3) / 1e9 / HBM_PEAK_GBS if traffic else None, "traffic": traffic,
                    "kernel": "k_align_persistent + k_align_tasks", "avg_launch_ms": k_ms, "reads_per_launch": 2 * n,
                    "basis": "counter-measured HBM-side bytes per step of the search (no oracle count at 3.1 Gbp)"}
    out = {
        "metric": METRIC, "value": value, "unit": "aligned reads/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": ms_step, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "u32", "data": "synthetic",
        "config": {"workload": f"C3 batched: {genome / 1e9:.1f} Gbp synthetic genome (GC 41%, 40% repeats), {n} pairs "
                               "of 36-150 bp, per-read budgets 2-6, 1 gap open, seed 32/<=2",
                   "pairs": n, "reads": 2 * n, "form": "batched: both ends in one persistent launch, locate, pair",
                   "parallelism": "1 GPU"},
        "p50_ms": float(np.percentile(np.array(times) * 1e3, 50)),
        "p99_ms": float(np.percentile(np.array(times) * 1e3, 99)),
        "aligned_fraction": aligned / (2 * n), "overflow_reads": int(((st & bw.ST_OVERFLOW) != 0).sum()),
        "roofline": roofline, "cpu_baseline": None,
        "cpu_baseline_note": "the oracle cannot index a 3.1 Gbp reference within a bench run",
    }
    print(json.dumps(out), flush=True)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--pairs", type=int, default=1_000_000)
    ap.add_argument("--genome", type=int, default=100_000_000)
    ap.add_argument("--cpu-pairs", type=int, default=250000, help="pairs in the oracle's timed sample (~15 s of host work)")
    ap.add_argument("--cpu-threads", type=int, default=0)
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--line-bytes", type=int, default=128)
    ap.add_argument("--rank-format", type=int, default=2,
                    help="0: counts + bit planes; 1: sub-counted 64-byte lines of 160 rows; "
                         "2: sub-counted 128-byte lines of 384 rows")
    ap.add_argument("--kmer-levels", type=int, default=0,
                    help="levels of the caller's short-string interval table (0: none, -1: automatic); "
                         "the search has its own")
    ap.add_argument("--waves-per-simd", type=int, default=0, help="batched-form residency (0 = autotuned)")
    ap.add_argument("--no-tune", dest="tune", action="store_false", help="skip the autotuner (most waves that fit)")
    ap.add_argument("--no-rescue", action="store_true", help="skip the mate-rescue measurement")
    ap.add_argument("--rescue-launches", type=int, default=10)
    ap.add_argument("--no-serve", action="store_true", help="skip the served leg")
    ap.add_argument("--serve-rates", type=float, nargs="+", default=[0.3, 0.6, 0.9])
    ap.add_argument("--serve-requests", type=int, default=300, help="requests per arrival rate")
    ap.add_argument("--serve-same-requests", type=int, default=12,
                    help="requests in the same-inputs comparison of the three forms")
    ap.add_argument("--serve-step-pairs", type=int, default=131072)
    ap.add_argument("--serve-arena-mib", type=int, default=2048)
    ap.add_argument("--steps-plain", type=int, default=0, help="steps for the plain form (default: --steps)")
    ap.add_argument("--cpu-reads", type=int, default=20000, help="C5: reads in the oracle's timed sample")
    ap.add_argument("--plain-reads", type=int, default=4000, help="C5: reads the plain form is timed on")
    ap.add_argument("--split-budget", type=int, default=None,
                    help="C1/C5: the batched form's split budget (default: the library's; tuned on C5)")
    ap.add_argument("--config", choices=("c2", "c3", "c1", "c5"), default="c2",
                    help="c2: the benchmark workload (default); c3: the 3.1 Gbp uneven-length workload; "
                         "c1, c5: the single-end tiny and stress workloads at their stated sizes")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py measures one GPU only; --gpus {args.gpus} is not supported (the path would shard "
              "read pairs across GPUs with a replicated index, which is not built here)", file=sys.stderr)
        sys.exit(2)
    if args.config == "c3":
        main_c3(args)
        return
    if args.config in ("c1", "c5"):
        main_se(args)
        return

    import torch

    import gen  # noqa: F401
    import paper_1505_07855_amd as bw
    from gen import configs

    torch.cuda.set_device(0)
    t0 = time.time()
    g = configs.c2_genome(args.genome)
    pairs = configs.c2_pairs(g, args.pairs)
    log(f"inputs drawn in {time.time() - t0:.1f}s")

    ox_box = {}
    want_cpu = not args.no_cpu

    def build_oracle():
        import oracle
        ox_box["ox"] = oracle.Index(g.seq)

    th = threading.Thread(target=build_oracle)
    if want_cpu:
        th.start()
    t0 = time.time()
    ix = bw.Index(g.seq, line_bytes=args.line_bytes, sa_sample=32, rank_format=args.rank_format).upload(
        kmer_levels=args.kmer_levels)
    log(f"library index built and uploaded in {time.time() - t0:.1f}s ({ix.info()['device_bytes'] / 1e6:.1f} MB)")

    w = configs.PAIR_WINDOW
    n = args.pairs
    # device inputs: each end on its own (plain form), both ends as one batch (batched form)
    e1, e2 = pairs.end1, pairs.end2
    ends = [(torch.from_numpy(e.bases).cuda(), torch.from_numpy(e.offsets.view(np.int64)).cuda()) for e in (e1, e2)]
    both_b = torch.cat([ends[0][0], ends[1][0]])
    both_o = torch.from_numpy(np.concatenate([e1.offsets[:-1], e1.offsets[-1] + e2.offsets]).view(np.int64)).cuda()
    stream = torch.cuda.current_stream()
    p_plain = bw.Params(**configs.PARAMS["C2"], form=bw.FORM_PLAIN)
    p_batched = bw.Params(**configs.PARAMS["C2"], form=bw.FORM_BATCHED, waves_per_simd=args.waves_per_simd)
    tune = None
    if args.tune and args.waves_per_simd == 0:
        from paper_1505_07855_amd.tune import tune_batched
        # the same reference in every rank-line layout (the others built on
        # the device, which gives the host builder's bytes)
        cands = [ix]
        have = (ix.info()["line_bytes"], ix.info()["rank_format"])
        for lb, fmt in ((64, bw.RANK_PLANES), (64, bw.RANK_SUBCOUNTS), (128, bw.RANK_SUB128)):
            if (lb, fmt) != have and args.kmer_levels == 0:
                cands.append(bw.Index.build_device(g.seq, line_bytes=lb, sa_sample=32, rank_format=fmt))
        best, table = tune_batched(cands, both_b, both_o, p_batched, max_len=100, hit_capacity=8 * n, log=log)
        p_batched.waves_per_simd = best["waves_per_simd"]
        ix = cands[best["key"]]
        for c in cands:
            if c is not ix:
                c.close()
        tune = {"best": best, "table": table,
                "note": "median of 3 timed batched calls per candidate; every candidate's output identical"}
        log(f"tune: picked {best['index']}, waves_per_simd {best['waves_per_simd']}")
    state = {"plain": [None, None, None], "eager": [None, None]}

    def step_plain():
        s = state["plain"]
        for k in range(2):
            s[k] = bw.align_batch(ix, ends[k][0], ends[k][1], p_plain, max_len=100, out=s[k],
                                  hit_capacity=4 * n, stream=stream)
        s[2] = bw.pair_reads(ix, s[0], s[1], w["lo"], w["hi"], w["mu"], configs.MAX_OCC, stream=stream, out=s[2])
        return s[0], s[1], s[2]

    def step_eager():
        s = state["eager"]
        s[0] = bw.align_batch(ix, both_b, both_o, p_batched, max_len=100, out=s[0], hit_capacity=8 * n, stream=stream)
        r1, r2 = s[0].window(0, n), s[0].window(n, 2 * n)
        s[1] = bw.pair_reads(ix, r1, r2, w["lo"], w["hi"], w["mu"], configs.MAX_OCC, stream=stream, out=s[1])
        return r1, r2, s[1]

    # the batched form proper: the whole step captured once and replayed
    pipe = bw.Pipeline(ix, p_batched, w["lo"], w["hi"], w["mu"], configs.MAX_OCC, max_pairs=n, max_len=100,
                       hit_capacity=8 * n, pos_capacity=128 * n)
    pipe.set_reads(both_b, both_o, n, max_len=100, stream=stream)

    def step_graph():
        pipe.run(graph=True, stream=stream)
        st = pipe.finish(stream=stream)
        if st["error"]:
            raise SystemExit(f"pipeline capacity exceeded: {st}")
        r1, r2, prs, _, _ = pipe.results()
        return r1, r2, prs

    def run(name, fn, steps):
        for i in range(args.warmup):
            fn()
            log(f"{name}: warmup step {i + 1}/{args.warmup} done")
        torch.cuda.synchronize()
        bw.timing_enable(True)
        bw.timing_reset()
        times = []
        t_all = time.perf_counter()
        out = None
        for i in range(steps):
            ts = time.perf_counter()
            out = fn()
            torch.cuda.synchronize()
            times.append(time.perf_counter() - ts)
            log(f"{name}: step {i + 1}/{steps}: {times[-1] * 1e3:.1f} ms")
        torch.cuda.synchronize()
        total = time.perf_counter() - t_all
        bw.timing_enable(False)
        kms = {}
        for k in ("align_plain", "align_persistent", "align_slow", "compact", "locate_rows", "sort", "pair"):
            ms, cnt = bw.timing_get(k)
            if cnt:
                kms[k] = {"avg_ms": ms / cnt, "launches": cnt}
        r1, r2, po = out
        st = [r.status.cpu().numpy() for r in (r1, r2)]
        aligned = int(sum(((x & bw.ST_HIT) != 0).sum() for x in st))
        research = int(sum(((x & bw.ST_RESEARCH) != 0).sum() for x in st))
        overflow = int(sum(((x & bw.ST_OVERFLOW) != 0).sum() for x in st))
        flags = bw.pairs_numpy(po)["flags"][:n]
        ms_step = total / steps * 1e3
        return {"steps": steps, "ms_per_step": ms_step, "aligned_reads_per_s": aligned / (ms_step / 1e3), "aligned": aligned,
                "p50_ms": float(np.percentile(np.array(times) * 1e3, 50)),
                "p99_ms": float(np.percentile(np.array(times) * 1e3, 99)),
                "research_reads": research, "overflow_reads": overflow, "paired_fraction": float((flags & bw.PF_PAIRED).astype(bool).mean()),
                "kernel_ms": kms, "out": out}

    def same(a, b):
        for x, y in ((a[0], b[0]), (a[1], b[1])):
            hx, hy = x.to_numpy(), y.to_numpy()
            if not (all(np.array_equal(u.view(np.uint8), v.view(np.uint8)) for u, v in zip(hx[:4], hy[:4]))
                    and np.array_equal(hx[4] & 7, hy[4] & 7)):
                return False
        return np.array_equal(bw.pairs_numpy(a[2]).view(np.uint8), bw.pairs_numpy(b[2]).view(np.uint8))

    plain = run("plain", step_plain, args.steps_plain or args.steps)
    eager = run("batched-eager", step_eager, args.steps_plain or args.steps)
    batched = run("batched", step_graph, args.steps)

    # end to end: the same step with the reads coming from pinned host memory
    # and the results (pair records, per-read status, c1, c2) going back to it
    h_b = torch.from_numpy(np.concatenate([e1.bases, e2.bases])).pin_memory()
    h_o = torch.from_numpy(np.concatenate([e1.offsets[:-1], e1.offsets[-1] + e2.offsets]).view(np.int64)).pin_memory()
    h_out = {"pairs": torch.empty((n, 24), dtype=torch.uint8).pin_memory(),
             "status": torch.empty(2 * n, dtype=torch.uint8).pin_memory(),
             "c1": torch.empty(2 * n, dtype=torch.int32).pin_memory(),
             "c2": torch.empty(2 * n, dtype=torch.int32).pin_memory()}

    def step_e2e():
        both_b.copy_(h_b, non_blocking=True)
        both_o.copy_(h_o, non_blocking=True)
        pipe.set_reads(both_b, both_o, n, max_len=100, stream=stream)
        r1, r2, prs = step_graph()
        h_out["pairs"].copy_(prs[:n], non_blocking=True)
        for k in ("status", "c1", "c2"):
            h_out[k][:n].copy_(getattr(r1, k), non_blocking=True)
            h_out[k][n:].copy_(getattr(r2, k), non_blocking=True)
        return r1, r2, prs

    e2e = run("end-to-end", step_e2e, args.steps)
    # every form must agree exactly
    a_out, e_out, b_out, x_out = plain.pop("out"), eager.pop("out"), batched.pop("out"), e2e.pop("out")
    if not same(a_out, b_out) or not same(e_out, b_out) or not same(x_out, b_out):
        raise SystemExit("plain, eager batched and captured batched forms disagree")
    if not np.array_equal(h_out["pairs"].numpy(), bw.pairs_numpy(b_out[2])[:n].view(np.uint8).reshape(n, 24)):
        raise SystemExit("pair records copied to the host differ")
    n_reads = 2 * n
    aligned = batched["aligned"]
    ms_step = batched["ms_per_step"]
    value = batched["aligned_reads_per_s"]
    kernel_ms = batched["kernel_ms"]

    rescue = None
    if not args.no_rescue:
        rescue = rescue_leg(bw, torch, ix, ends, b_out[:2], b_out[2], n, w, stream, args.rescue_launches, len(g.seq),
                            configs.PARAMS["C2"]["max_diff"])
        log(f"rescue: {rescue['candidates']} candidates, {rescue['rescued']} rescued, "
            f"{rescue['avg_launch_ms']:.3f} ms per launch")

    served = None
    if not args.no_serve:
        served = served_leg(bw, torch, ix, g, args, stream)

    roofline = None
    cpu = None
    if want_cpu:
        th.join()
        import oracle
        ox = ox_box["ox"]
        op = oracle.Params(**configs.PARAMS["C2"], bases_per_line=ix.info()["bases_per_line"])
        nthreads = args.cpu_threads or host_threads()
        ns = min(args.cpu_pairs, args.pairs)
        sb = [(e.bases[:int(e.offsets[ns])], e.offsets[:ns + 1]) for e in (pairs.end1, pairs.end2)]
        t0 = time.perf_counter()
        ores = [oracle.align(ox, b, o, op, threads=nthreads) for b, o in sb]
        locs = [oracle.locate(ox, r.hits, configs.MAX_OCC) for r in ores]
        oracle.pair(ores[0], locs[0][0], locs[0][1], ores[1], locs[1][0], locs[1][1], w["lo"], w["hi"], w["mu"])
        cpu_s = time.perf_counter() - t0
        cpu_aligned = int(sum(((r.status & oracle.ST_HIT) != 0).sum() for r in ores))
        cpu = {"value": cpu_aligned / cpu_s, "unit": "aligned reads/s", "cores": nthreads, "kind": "oracle",
               "host_cpus_visible": len(os.sched_getaffinity(0)),
               "sample": f"first {ns} pairs of the same batch ({2 * ns} reads): align both ends, locate, pair; "
                         f"{cpu_s:.1f} s"}
        # rank lines a read touches in plain backward search (D-array scans +
        # search), same order as the kernel
        touches = np.concatenate([r.counts["touch_s"] + r.counts["touch_d"] for r in ores]).astype(np.float64)
        kf, timed_in = kernel_ms.get("align_persistent"), "batched (graph replays)"
        if not kf:
            kf, timed_in = eager["kernel_ms"].get("align_persistent"), "batched-eager (same kernel and batch)"
        if kf:
            traffic = traffic_from_profiles("k_align_persistent")
            rate = traffic / (kf["avg_ms"] / 1e3) / 1e9 if traffic else None
            roofline = {"bound": "hbm", "achieved": rate, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                        "frac": rate / HBM_PEAK_GBS if rate else None, "traffic": traffic,
                        "kernel": "k_align_persistent", "reads_per_launch": n_reads, "avg_launch_ms": kf["avg_ms"],
                        "timed_in": timed_in, "basis": "counter-measured HBM-side bytes per launch",
                        "line_touches_per_read": float(touches.mean())}

    out = {
        "metric": METRIC, "value": value, "unit": "aligned reads/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": ms_step, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "u32", "data": "synthetic",
        "config": {"workload": f"C2 mid: {args.genome / 1e6:.0f} Mbp synthetic genome (GC 41%, 40% repeats), "
                               f"{args.pairs} pairs 2x100 bp, <=4 diffs, 1 gap open, seed 32/<=2",
                   "pairs": args.pairs, "reads": n_reads, "form": "batched: align both ends in one persistent launch, locate, pair; replayed as one captured hipGraph",
                   "waves_per_simd": p_batched.waves_per_simd,
                   "line_bytes": ix.info()["line_bytes"], "rank_format": ix.info()["rank_format"],
                   "bases_per_line": ix.info()["bases_per_line"], "parallelism": "1 GPU"},
        "p50_ms": batched["p50_ms"], "p99_ms": batched["p99_ms"],
        "reads_per_s": n_reads / (ms_step / 1e3), "pairs_per_s": n / (ms_step / 1e3),
        "aligned_fraction": aligned / n_reads, "paired_fraction": batched["paired_fraction"],
        "overflow_reads": batched["overflow_reads"],
        "overflow_note": "reads with more than max_hits (256) distinct candidate hits report none (status "
                         "OVERFLOW, c1 = c2 = 0xFFFFFFFF), on the GPU and in the oracle alike",
        "plain": {k: v for k, v in plain.items()}, "batched": {k: v for k, v in batched.items()},
        "batched_eager": {k: v for k, v in eager.items()}, "autotune": tune,
        "end_to_end": {"ms_per_step": e2e["ms_per_step"], "aligned_reads_per_s": e2e["aligned_reads_per_s"],
                       "p99_ms": e2e["p99_ms"],
                       "note": "reads from pinned host memory, pair records, status, c1, c2 back to it"},
        "roofline": roofline, "cpu_baseline": cpu, "rescue": rescue, "served": served,
    }
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
