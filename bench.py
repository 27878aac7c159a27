#!/usr/bin/env python3
"""Benchmark of the per-GPU relational hot path on one MI355X.

Step = one fused star query over HBM-resident synthetic tables of the measured
shape (build 1.5M rows {key, segment}, probe 60M rows {fk, date, price}):
filter segment == 1 and date < 1200, join fk = key, GROUP BY key SUM(price),
i.e. dimension filter + hash build + one fused probe/aggregate pass over the
fact columns + group compaction.  value = probe rows per second.

Beside the headline line it reports, measured outside the timed region:
  roofline      : the fused probe kernel's algorithmic bytes / its mean HIP-event
                  duration against the 8 TB/s HBM peak (+ counter traffic when
                  a committed counter profile matches the current kernel source)
  cpu_baseline  : the CPU oracle (single thread) on a bounded sample, and the
                  threaded CPU baseline over every usable host core
  partition     : hash partition of the probe table, fanout 2 / 8 / 64
  chain         : the two-join chain query (fact 120M, Zipf s = 0 and 1)
  groupby       : GROUP BY orderkey SUM(quantity) over 60M lineitem-like rows
                  (about 14.7M groups), radix-partitioned path vs HBM hash table
  join          : the materializing join of the join microbenchmark at one GPU's
                  share (build 60M / probe 160M, hit ratio 0.5, k = 1, 4, 8
                  8-byte columns a side)
"""
import argparse
import glob
import hashlib
import json
import os
import sys
import threading
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
PROBE_ROW_BYTES = 16   # fk int32 + date int32 + price int64
BUILD_ROW_BYTES = 8    # key int32 + segment int32
GROUP_OUT_BYTES = 16   # key int64 + sum int64


KERNEL_SOURCES = {  # the files that define each profiled kernel (name patterns as rocprofv3 prints them)
    "k_fast_fact": ["fast.hip", "pyst_internal.h", "table.h", "query.h"],
    "k_fast_fact<2, 8, 2": ["fast.hip", "pyst_internal.h", "table.h", "query.h"],
    "k_direct_store": ["join.hip", "ranges.h", "pyst_internal.h", "table.h"],
    "k_direct_lookup": ["join.hip", "ranges.h", "pyst_internal.h", "table.h"],
    "k_gather_rows<4": ["ops.hip", "pyst_internal.h"],
    "k_gather<": ["ops.hip", "pyst_internal.h"],
    "k_key_range": ["agg.hip", "pyst_internal.h"],
    "k_once_hist": ["agg.hip", "pyst_internal.h"],
    "k_once_move": ["agg.hip", "pyst_internal.h"],
    "k_once_groups": ["agg.hip", "pyst_internal.h"],
    "k_move_hist_both": ["agg.hip", "pyst_internal.h"],
    "k_move_scatter": ["agg.hip", "pyst_internal.h"],
    "k_bucket_groups": ["agg.hip", "pyst_internal.h"],
    "k_bat_fact_staged": ["batch.hip", "fast.hip", "pyst_internal.h", "table.h", "query.h"],
    "k_part_hist_i32": ["ops.hip", "pyst_internal.h"],
    "k_part_scatter": ["ops.hip", "pyst_internal.h"],
}
Q18_WORKLOAD = "q18_n60000000_g15000000"
BATCH_WORKLOAD = "batch_512"
Q18_KERNELS = ("k_key_range", "k_once_hist", "k_once_move", "k_once_groups")
PAIR_KERNELS = ("k_move_hist_both", "k_move_scatter", "k_bucket_groups")
CHAIN_WORKLOAD = "chain_a3000000_b300000_f120000000"  # fact-pass counters averaged over s = 0 and 1
JOIN_WORKLOAD = "join_b60000000_p160000000_k4"  # counters of the k = 4 materializing join


def source_hash(kernel="k_fast_fact"):
    h = hashlib.sha256()
    for f in KERNEL_SOURCES[kernel]:
        h.update(open(os.path.join(ROOT, "paper_2512_02862_amd", "csrc", f), "rb").read())
    return h.hexdigest()[:16]


def _db_rows(db, sql):
    import sqlite3
    return list(sqlite3.connect(db).execute(sql))


def summarize(args):
    """Turn rocprofv3 result databases into the text summaries and traffic.json kept in profiles/.

    --summarize trace DB OUT.txt CMD...          kernel-trace statistics (top kernels)
    --summarize pmc FETCH_DB WRITE_DB COPY_FETCH_DB COPY_WRITE_DB KERNEL WORKLOAD CMD...
        per-dispatch FETCH_SIZE / WRITE_SIZE of KERNEL, scaled by the same counters of a plain
        1 GiB copy (bench.py --calibrate-copy), into profiles/traffic.json and a text summary.
    """
    kind, rest = args[0], args[1:]
    prof = os.path.join(ROOT, "profiles")
    if kind == "trace":
        db, out, cmd = rest[0], rest[1], " ".join(rest[2:])
        rows = _db_rows(db, "select name, total_calls, total_duration, average, percentage from top_kernels")
        with open(os.path.join(prof, out), "w") as fh:
            fh.write("# rocprofv3 --kernel-trace --stats\n# command: %s\n" % cmd)
            fh.write("%-90s %6s %14s %12s %7s\n" % ("kernel", "calls", "total_us", "avg_us", "pct"))
            for r in rows:
                fh.write("%-90s %6d %14.1f %12.2f %7.2f\n" % (r[0][:90], r[1], r[2], r[3], r[4]))
        return
    fdb, wdb, cfdb, cwdb, kernel, workload = rest[:6]
    cmd = " ".join(rest[6:])

    def avg(db, counter, like):
        r = _db_rows(db, "select avg(value), count(*) from counters_collection where counter_name='%s' "
                         "and kernel_name like '%%%s%%'" % (counter, like))
        return r[0]

    fetch, nf = avg(fdb, "FETCH_SIZE", kernel)
    write, nw = avg(wdb, "WRITE_SIZE", kernel)
    copy_bytes = 1 << 30
    cfetch, _ = avg(cfdb, "FETCH_SIZE", "copyBuffer")
    cwrite, _ = avg(cwdb, "WRITE_SIZE", "copyBuffer")
    ffac, wfac = copy_bytes / 1024 / cfetch, copy_bytes / 1024 / cwrite
    traffic = fetch * ffac * 1024 + write * wfac * 1024
    path = os.path.join(prof, "traffic.json")
    rec = json.load(open(path)) if os.path.exists(path) else {}
    rec[kernel + "|" + workload] = {
        "bytes_per_launch": traffic, "fetch_kib_per_dispatch": fetch, "write_kib_per_dispatch": write,
        "fetch_scale": ffac, "write_scale": wfac, "dispatches": [nf, nw], "source_hash": source_hash(kernel),
        "command": cmd}
    json.dump(rec, open(path, "w"), indent=1, sort_keys=True)
    fname = "".join(ch if ch.isalnum() else "_" for ch in kernel).strip("_")
    fname = "_".join(x for x in fname.split("_") if x)  # k_fast_fact<2, 8, 2 -> k_fast_fact_2_8_2
    with open(os.path.join(prof, "%s_%s_traffic.txt" % (fname, workload)), "w") as fh:
        fh.write("# HBM traffic of %s on %s from rocprofv3 --pmc FETCH_SIZE, then --pmc WRITE_SIZE\n" % (kernel, workload))
        fh.write("# command: %s\n" % cmd)
        fh.write("FETCH_SIZE KiB/dispatch %.1f (x%.3f from a 1 GiB copy reading %.1f KiB)\n" % (fetch, ffac, cfetch))
        fh.write("WRITE_SIZE KiB/dispatch %.1f (x%.3f from a 1 GiB copy writing %.1f KiB)\n" % (write, wfac, cwrite))
        fh.write("HBM bytes per launch %.4g\n" % traffic)


def counter_traffic(kernel, workload):
    """HBM bytes per launch from a committed rocprofv3 counter summary, if it is current."""
    path = os.path.join(ROOT, "profiles", "traffic.json")
    if not os.path.exists(path):
        return None
    try:
        rec = json.load(open(path)).get(kernel + "|" + workload)
    except ValueError:
        return None
    if not rec or rec.get("source_hash") != source_hash(kernel):
        return None
    return rec.get("bytes_per_launch")


def to_dev(d):
    import torch
    return {k: torch.from_numpy(v).cuda() for k, v in d.items()}


def hbm_ceiling(pyst):
    """The HBM peak three ways: the published figure the roofline uses, the one
    the device's properties imply, and a measured streaming copy (a 4 GiB
    device-to-device copy, 2 bytes moved per byte copied, best of 10)."""
    import torch
    clk, bits, props = pyst.device_hbm(0)
    src = torch.empty(1 << 29, dtype=torch.int64, device="cuda")
    dst = torch.empty_like(src)
    src.fill_(1)
    best = None
    for _ in range(12):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        dst.copy_(src)
        e1.record()
        e1.synchronize()
        ms = e0.elapsed_time(e1)
        best = ms if best is None else min(best, ms)
    nbytes = 2 * src.numel() * 8
    del src, dst
    torch.cuda.empty_cache()
    return {"published_gbs": HBM_PEAK_GBS, "device_props_gbs": props, "mem_clock_khz": clk, "bus_bits": bits,
            "measured_copy_gbs": nbytes / (best / 1e3) / 1e9,
            "copy": "torch device-to-device copy of 4 GiB, best of 12, read + write bytes"}


def timed_loop(fn, steps, warmup):
    import torch
    for _ in range(warmup):
        fn()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        fn()
    torch.cuda.synchronize()
    return time.perf_counter() - t0


def main():
    if len(sys.argv) > 1 and sys.argv[1] == "--summarize":
        summarize(sys.argv[2:])
        return
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--build-rows", type=int, default=1_500_000)
    ap.add_argument("--probe-rows", type=int, default=60_000_000)
    ap.add_argument("--max-load", type=float, default=0.5)
    ap.add_argument("--no-extras", action="store_true", help="skip every measurement beside the headline")
    ap.add_argument("--extras", default="partition,chain,groupby,join,batch,config4",
                    help="comma-separated extra measurements to run")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-sample-rows", type=int, default=30_000_000)
    ap.add_argument("--join-k", default="1,4,8", help="8-byte columns a side of the join microbenchmark")
    ap.add_argument("--partition-fanouts", default="2,8,64", help="fanouts of the partition extra")
    ap.add_argument("--join-legs", default="plain,partition,m2m",
                    help="parts of the join extra: the materializing join, the same with its partition leg, "
                         "the many-to-many join (counter runs take 'plain' alone)")
    ap.add_argument("--batch-fragments", type=int, default=512)
    ap.add_argument("--batch-max-rows", type=float, default=2e7, help="largest fragment probe size")
    ap.add_argument("--config4-rows", type=int, default=2_000_000_000, help="pinned host fact rows, streamed and served")
    ap.add_argument("--config4-requests", type=int, default=200)
    ap.add_argument("--config4-serve", action="store_true",
                    help="also serve the config4 requests at full size (off by default: a full-size Poisson "
                         "serving run has failed with a device memory fault whose cause is not found yet)")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="only run a plain 1 GiB device-to-device copy 5 times (counter calibration)")
    args = ap.parse_args()
    if args.calibrate_copy:
        import torch
        src = torch.ones(1 << 28, dtype=torch.int32, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(5):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"copy_bytes_per_launch": src.numel() * 4, "launches": 5}))
        return
    if args.gpus != 1:
        print("bench.py measures one GPU: this build has no multi-GPU path (the shuffle stops at the "
              "partitioned per-destination buffers); run with --gpus 1", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    import gen
    from paper_2512_02862_amd import pyst

    def log(msg):
        print("[bench] " + msg, file=sys.stderr, flush=True)

    nb, npr = args.build_rows, args.probe_rows
    log("generating star tables: build %d, probe %d" % (nb, npr))
    b_host, p_host = gen.star_tables(nb, npr, workload=1)
    b = to_dev(b_host)
    p = to_dev(p_host)
    fact = [p["fk"], p["date"], p["price"]]
    ctx = pyst.Ctx(0, 16 << 30)
    plan = pyst.star_plan(b, max_load=args.max_load)
    out_cap = nb
    keys = torch.empty(out_cap, dtype=torch.int64, device="cuda")

    def step():
        pyst.query(ctx, plan, fact, out_cap=out_cap)

    log("warmup %d, timed %d steps" % (args.warmup, args.steps))
    for _ in range(args.warmup):
        step()
    ctx.check()
    ctx.timing(True)
    elapsed = timed_loop(step, args.steps, 0)
    ctx.timing(False)
    fact_ms, launches = ctx.kernel_time("fact_pass")
    ctx.check()
    k, s, ng = pyst.query(ctx, plan, fact, out_cap=out_cap)
    ctx.check()
    n_groups = int(ng.item())
    del keys

    ms_per_step = elapsed / args.steps * 1e3
    rows_per_s = args.steps * npr / elapsed
    fact_mean_s = fact_ms / max(launches, 1) / 1e3
    fact_bytes = npr * PROBE_ROW_BYTES
    achieved = fact_bytes / fact_mean_s / 1e9
    query_bytes = npr * PROBE_ROW_BYTES + nb * BUILD_ROW_BYTES + n_groups * GROUP_OUT_BYTES
    workload = "star_b%d_p%d" % (nb, npr)
    traffic = counter_traffic("k_fast_fact", workload)

    result = {
        "metric": "probe rows/s and % HBM peak for filter+join+agg; batched p50/p99 latency",
        "value": rows_per_s,
        "unit": "probe rows/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "int64",
        "data": "synthetic (seeded splitmix64 tables of the measured shape; no dataset)",
        "config": {
            "workload": "star query, build %d rows {key, segment}, probe %d rows {fk, date, price}: "
                        "segment == 1, date < 1200, join fk = key, GROUP BY key SUM(price)" % (nb, npr),
            "build_rows": nb, "probe_rows": npr, "max_load": args.max_load, "groups": n_groups,
            "parallelism": "single GPU",
        },
        "query_hbm": {"algorithmic_bytes": query_bytes, "gbs": query_bytes / (ms_per_step / 1e3) / 1e9,
                      "frac_of_peak": query_bytes / (ms_per_step / 1e3) / 1e9 / HBM_PEAK_GBS},
        "hbm_ceiling": None if args.no_extras else hbm_ceiling(pyst),  # (kept out of --no-extras profile runs)
        "roofline": {
            "kernel": "k_fast_fact (fused filter + probe + SUM)",
            "bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
            "frac": achieved / HBM_PEAK_GBS, "traffic": traffic,
            "algorithmic_bytes_per_launch": fact_bytes, "mean_launch_us": fact_mean_s * 1e6,
            "launches": launches,
        },
    }

    extras = [] if args.no_extras else args.extras.split(",")
    def extra(name, fn, *a):
        # an extra that fails is recorded with its error; the headline line is still printed
        if name not in extras:
            return
        try:
            result[name] = fn(*a)
        except Exception as e:  # noqa: BLE001
            log("extra %s failed: %r" % (name, e))
            result[name] = {"error": repr(e)}
        torch.cuda.empty_cache()

    extra("partition", bench_partition, ctx, pyst, p, npr, log, [int(x) for x in args.partition_fanouts.split(",")])
    del b, p, fact
    torch.cuda.empty_cache()
    extra("chain", bench_chain, ctx, pyst, gen, log)
    extra("groupby", bench_groupby, ctx, pyst, gen, log)
    extra("join", bench_join, ctx, pyst, gen, log, 60_000_000, 160_000_000, [int(x) for x in args.join_k.split(",")],
          2, args.join_legs.split(","))
    extra("batch", bench_batch, ctx, pyst, gen, log, args.batch_fragments, args.batch_max_rows)
    extra("config4", bench_config4, pyst, gen, log, args.config4_rows, args.config4_requests, 64_000_000, 32 << 30,
          args.config4_serve)

    if not args.no_cpu_baseline:
        result["cpu_baseline"] = cpu_baseline(b_host, p_host, args.cpu_sample_rows, log)

    ctx.close()
    print(json.dumps(result), flush=True)


PART_WORKLOAD = "partition_f64_n60000000"  # counters of the fanout-64 partition (--partition-fanouts 64)


def bench_partition(ctx, pyst, p, npr, log, fanouts=(2, 8, 64)):
    import torch
    out = {}
    for fanout in fanouts:
        log("partition fanout %d" % fanout)

        def step():
            pyst.partition(ctx, p["fk"], [p["date"], p["price"]], fanout)

        for _ in range(2):
            step()
        ctx.check()
        ctx.timing(True)
        el = timed_loop(step, 10, 0)
        ctx.timing(False)
        sc_ms, sc_n = ctx.kernel_time("part_scatter")
        ctx.kernel_time("partition")
        ctx.check()
        alg = npr * 32  # read 16 B + write 16 B per row
        ms = el / 10 * 1e3
        out["F%d" % fanout] = {"ms": ms, "rows_per_s": npr / (ms / 1e3), "gbs": alg / (ms / 1e3) / 1e9,
                              "frac_of_peak": alg / (ms / 1e3) / 1e9 / HBM_PEAK_GBS,
                              "scatter_kernel_us": sc_ms / max(sc_n, 1) * 1e3}
        if fanout == 64:  # HBM bytes per launch from committed counters (null once the kernels changed)
            out["F64"]["counter_traffic"] = {k: counter_traffic(k, PART_WORKLOAD)
                                             for k in ("k_part_hist_i32", "k_part_scatter")}
        torch.cuda.empty_cache()
    return out


def bench_chain(ctx, pyst, gen, log):
    import torch
    na, nbd, nf = 3_000_000, 300_000, 120_000_000
    out = {}
    a_h, b_h = gen.chain_dims(na, nbd)
    a, b = to_dev(a_h), to_dev(b_h)
    for zs in (0.0, 1.0):
        log("chain query, fact %d, zipf s=%g" % (nf, zs))
        f_h = gen.chain_fact(nf, na, nbd, zs)
        f = to_dev(f_h)
        del f_h
        fact = [f[c] for c in ("a_fk", "b_fk", "date", "price", "discount")]
        plan = pyst.chain_plan(a, b)
        cap = 16_000_000

        def step():
            pyst.query(ctx, plan, fact, out_cap=cap)

        step()
        ctx.check()
        ctx.timing(True)
        el = timed_loop(step, 5, 0)
        ctx.timing(False)
        fms, fn = ctx.kernel_time("fact_pass")
        k, s, ng = pyst.query(ctx, plan, fact, out_cap=cap)
        ctx.check()
        groups = int(ng.item())
        alg = nf * 24 + na * 8 + nbd * 8 + groups * 16
        ms = el / 5 * 1e3
        out["s%g" % zs] = {"ms": ms, "fact_rows_per_s": nf / (ms / 1e3), "groups": groups,
                           "algorithmic_bytes": alg, "gbs": alg / (ms / 1e3) / 1e9,
                           "frac_of_peak": alg / (ms / 1e3) / 1e9 / HBM_PEAK_GBS,
                           "fact_pass_us": fms / max(fn, 1) * 1e3}
        del f, fact, k, s
        torch.cuda.empty_cache()
    # HBM bytes per launch of the chain's fact pass from committed counters (null
    # when the kernel's source has changed since they were taken)
    out["fact_pass_traffic"] = counter_traffic("k_fast_fact<2, 8, 2", CHAIN_WORKLOAD)
    # the pair group-by's kernels (the two moves share one name: their mean per launch)
    out["pair_groupby_traffic"] = {k: counter_traffic(k, CHAIN_WORKLOAD) for k in PAIR_KERNELS}
    out["fact_pass_algorithmic_bytes"] = nf * 24
    return out


def bench_groupby(ctx, pyst, gen, log, n=60_000_000, n_orders=15_000_000):
    """GROUP BY orderkey SUM(quantity), groups far beyond the caches: both group-by paths."""
    import torch
    li = gen.q18_lineitem(n, n_orders)
    k, v = torch.from_numpy(li["orderkey"]).cuda(), torch.from_numpy(li["quantity"]).cuda()
    del li
    out = {"rows": n, "key_range": n_orders}
    for path, hash_only in (("radix", False), ("hash", True)):
        log("group-by %d rows, path %s" % (n, path))
        ctx.groupby_hash_only(hash_only)

        def step():
            return pyst.groupby_sum(ctx, k, v, max_groups=n_orders)

        r = step()
        ctx.check()
        groups = int(r[2].item())
        del r
        ctx.timing(True)
        el = timed_loop(step, 5, 0)
        ctx.timing(False)
        g_ms, g_n = ctx.kernel_time("groupby_" + path)
        ctx.check()
        ms = el / 5 * 1e3
        alg = n * 8 + groups * 16  # key and value read once, each group written once
        out[path] = {"ms": ms, "rows_per_s": n / (ms / 1e3), "groups": groups, "algorithmic_bytes": alg,
                     "gbs": alg / (ms / 1e3) / 1e9, "frac_of_peak": alg / (ms / 1e3) / 1e9 / HBM_PEAK_GBS,
                     "region_us": g_ms / max(g_n, 1) * 1e3}
    ctx.groupby_hash_only(False)
    out["radix_speedup"] = out["hash"]["ms"] / out["radix"]["ms"]
    # HBM bytes per launch of the radix path's kernels, from committed counters
    out["radix"]["counter_traffic"] = {k: counter_traffic(k, Q18_WORKLOAD) for k in Q18_KERNELS}
    return out


def partitioned_join(ctx, pyst, bk, bc, pk, pc, fanout):
    """One GPU's whole share of the distributed join: both sides hash-partitioned
    into `fanout` destinations (the send side; the per-destination counts come
    back to the host, as the count exchange of a shuffle needs them), then each
    destination's build and probe segments joined and materialized (the receive
    side's work, here on the segments this GPU holds).  Returns per destination
    (probe, build, columns, count) of pyst_join_materialize and the offsets."""
    ob = pyst.partition(ctx, bk, bc, fanout)
    op = pyst.partition(ctx, pk, pc, fanout)
    offs_b, offs_p = ob[2].cpu().tolist(), op[2].cpu().tolist()
    res = []
    for q in range(fanout):
        b0, b1, p0, p1 = offs_b[q], offs_b[q + 1], offs_p[q], offs_p[q + 1]
        res.append(pyst.join_materialize(ctx, ob[0][b0:b1], [c[b0:b1] for c in ob[1]], op[0][p0:p1],
                                         [c[p0:p1] for c in op[1]]))
    return res, ob, op, offs_b, offs_p


def bench_partitioned_join(ctx, pyst, log, bk, bc, pk, pc, fanout, m_expect):
    """partition(build) + partition(probe) + build + probe + materialize per destination."""
    nb, npr, k = bk.numel(), pk.numel(), len(bc)
    log("join microbenchmark with the partition leg: fanout %d, k = %d" % (fanout, k))

    def step():
        return partitioned_join(ctx, pyst, bk, bc, pk, pc, fanout)

    r = step()
    ctx.check()
    m = sum(int(x[3].item()) for x in r[0])
    del r
    ctx.timing(True)
    el = timed_loop(step, 3, 0)
    ctx.timing(False)
    part_ms, part_n = ctx.kernel_time("partition")
    for name in ("part_scatter", "join_build", "join_probe", "gather", "gather_rows", "pack_rows"):
        ctx.kernel_time(name)
    ctx.check()
    ms = el / 3 * 1e3
    part_bytes = 2 * (nb + npr) * (4 + 8 * k)  # each side read and written once
    return {"fanout": fanout, "ms": ms, "matches": m, "matches_equal_unpartitioned": m == m_expect,
            "partition_ms_both_sides": part_ms / 3, "partition_bytes": part_bytes,
            "partition_gbs": part_bytes / (part_ms / 3 / 1e3) / 1e9 if part_n else None,
            "probe_rows_per_s": npr / (ms / 1e3), "output_tuples_per_s": m / (ms / 1e3)}


def bench_many_to_many(ctx, pyst, gen, log, nb, npr, ks=(1, 4)):
    """The materializing join with duplicate build keys: nb build rows over nb / 4 keys
    (uniform, about 4 rows a key), npr probe rows over 2 * nb / 4 keys, k columns a side."""
    import numpy as np
    import torch
    nkeys = nb // 4
    out = {"build_rows": nb, "probe_rows": npr, "build_keys": nkeys}
    for k in ks:
        log("many-to-many join: build %d over %d keys, probe %d, k = %d" % (nb, nkeys, npr, k))
        b_h, p_h = gen.join_tables_dup(nb, npr, k, nkeys)
        need = int(np.bincount(b_h["key"], minlength=2 * nkeys + 1)[p_h["key"]].sum())
        bk, pk = torch.from_numpy(b_h["key"]).cuda(), torch.from_numpy(p_h["key"]).cuda()
        bc = [torch.from_numpy(b_h["c%d" % c]).cuda() for c in range(k)]
        pc = [torch.from_numpy(p_h["c%d" % c]).cuda() for c in range(k)]
        del b_h, p_h

        def step():
            return pyst.join_materialize(ctx, bk, bc, pk, pc, unique_keys=False, out_cap=need)

        r = step()
        ctx.check()
        m = int(r[3].item())
        del r
        torch.cuda.empty_cache()
        ctx.timing(True)
        el = timed_loop(step, 3, 0)
        ctx.timing(False)
        b_ms, b_n = ctx.kernel_time("join_build")
        p_ms, p_n = ctx.kernel_time("join_probe")
        for name in ("gather", "gather_rows", "pack_rows"):
            ctx.kernel_time(name)
        ctx.check()
        ms = el / 3 * 1e3
        out["k%d" % k] = {"ms": ms, "matches": m, "matches_expected": need, "output_tuples_per_s": m / (ms / 1e3),
                          "probe_rows_per_s": npr / (ms / 1e3), "build_us": b_ms / max(b_n, 1) * 1e3,
                          "probe_us": p_ms / max(p_n, 1) * 1e3}
        del bk, pk, bc, pc
        torch.cuda.empty_cache()
    return out


def bench_join(ctx, pyst, gen, log, nb=60_000_000, npr=160_000_000, ks=(1, 4, 8), fanout=2,
               legs=("plain", "partition", "m2m")):
    """Build + probe + materialize of k 8-byte columns per side (one pyst_join_materialize call),
    and the same join with its partition leg (both sides partitioned first, fanout 2: two GPUs)."""
    import torch
    out = {"build_rows": nb, "probe_rows": npr, "hit_ratio": 0.5}
    for k in ks:
        log("join microbenchmark: build %d, probe %d, k = %d" % (nb, npr, k))
        b_h, p_h = gen.join_tables(nb, npr, k)
        bk, pk = torch.from_numpy(b_h["key"]).cuda(), torch.from_numpy(p_h["key"]).cuda()
        bc = [torch.from_numpy(b_h["c%d" % c]).cuda() for c in range(k)]
        pc = [torch.from_numpy(p_h["c%d" % c]).cuda() for c in range(k)]
        del b_h, p_h

        def step():
            return pyst.join_materialize(ctx, bk, bc, pk, pc)

        r = step()
        ctx.check()
        m = int(r[3].item())
        del r
        ctx.timing(True)
        el = timed_loop(step, 5, 0)
        ctx.timing(False)
        b_ms, b_n = ctx.kernel_time("join_build")
        p_ms, p_n = ctx.kernel_time("join_probe")
        g_ms, g_n = ctx.kernel_time("gather")
        r_ms, r_n = ctx.kernel_time("gather_rows")
        k_ms, k_n = ctx.kernel_time("pack_rows")
        ctx.check()
        ms = el / 5 * 1e3
        cap = 1 << (int(nb / 0.5)).bit_length()
        # algorithmic bytes: keys read once, one table slot written per build row and
        # read per probe row, the table cleared, (probe row, build row) pairs written
        # and read back, k values read and written per match and side
        gather_bytes = m * (4 + 16 * k)  # per gather launch
        alg = nb * (4 + 8) + cap * 8 + npr * (4 + 8) + m * 8 + 2 * gather_bytes
        g_us = g_ms / max(g_n, 1) * 1e3
        out["k%d" % k] = {
            "ms": ms, "matches": m, "probe_rows_per_s": npr / (ms / 1e3), "output_tuples_per_s": m / (ms / 1e3),
            "algorithmic_bytes": alg, "gbs": alg / (ms / 1e3) / 1e9,
            "frac_of_peak": alg / (ms / 1e3) / 1e9 / HBM_PEAK_GBS,
            "build_us": b_ms / max(b_n, 1) * 1e3, "probe_us": p_ms / max(p_n, 1) * 1e3,
            # column gathers: the probe side (and the build side at k = 1); packed-row
            # gathers: the build side at k > 1, after packing its columns row-major
            "gather_us": g_us, "gather_gbs": gather_bytes / (g_us / 1e6) / 1e9 if g_us > 0 else None,
            "gather_rows_us": r_ms / r_n * 1e3 if r_n else None, "pack_rows_us": k_ms / k_n * 1e3 if k_n else None}
        if "partition" in legs:
            out["k%d" % k]["with_partition"] = bench_partitioned_join(ctx, pyst, log, bk, bc, pk, pc, fanout, m)
        del bk, pk, bc, pc
        torch.cuda.empty_cache()
    if "m2m" in legs:
        out["many_to_many"] = bench_many_to_many(ctx, pyst, gen, log, nb, npr)
    # HBM bytes per launch from committed counters of the k = 4 run (null once the kernels changed)
    out["k4_counter_traffic"] = {"k_direct_store": counter_traffic("k_direct_store", JOIN_WORKLOAD),
                                 "k_direct_lookup": counter_traffic("k_direct_lookup", JOIN_WORKLOAD),
                                 "k_gather_rows": counter_traffic("k_gather_rows<4", JOIN_WORKLOAD),
                                 "k_gather": counter_traffic("k_gather<", JOIN_WORKLOAD)}
    return out


def pinned_empty(n, dtype):
    import torch
    return torch.empty(n, dtype=dtype, pin_memory=True)


def chain_fact_pinned(gen, n, na, nb, zs):
    """Chain fact columns generated straight into pinned host tensors."""
    import torch
    cols = {"a_fk": torch.int32, "b_fk": torch.int32, "date": torch.int32, "price": torch.int64,
            "discount": torch.int32}
    t = {c: pinned_empty(n, d) for c, d in cols.items()}
    gen.chain_fact(n, na, nb, zs, out={c: v.numpy() for c, v in t.items()})
    return [t[c] for c in ("a_fk", "b_fk", "date", "price", "discount")]


def h2d_peak(host_t, log):
    """Plain pinned host-to-device copy rate of a large buffer (GB/s)."""
    import torch
    d = torch.empty(host_t.numel(), dtype=host_t.dtype, device="cuda")
    d.copy_(host_t, non_blocking=True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(3):
        d.copy_(host_t, non_blocking=True)
    torch.cuda.synchronize()
    dt = (time.perf_counter() - t0) / 3
    gbs = host_t.numel() * host_t.element_size() / dt / 1e9
    log("pinned H2D copy: %.1f GB/s" % gbs)
    return gbs


def bench_batch(ctx, pyst, gen, log, nfrag, max_rows):
    """512 star fragments in one batch vs one at a time (each read back, as a sizing caller must)."""
    import torch
    sizes, builds = gen.fragment_sizes(nfrag, hi=max_rows)
    log("batch: generating %d fragments, %d probe rows" % (nfrag, int(sizes.sum())))
    frags = []
    for f, (p, b) in enumerate(zip(sizes, builds)):
        bt, pt = gen.star_tables(max(int(b), 1), int(p), workload=3, fragment=f)
        bd = to_dev(bt)
        frags.append((pyst.star_plan(bd), [torch.from_numpy(pt[c]).cuda() for c in ("fk", "date", "price")]))
    batch = pyst.Batch(ctx, frags)
    best, best_ms = batch.autotune(reps=2)
    log("autotune best %s: %.3f ms" % (best, best_ms))
    batch.run(best)
    ctx.check()
    el = timed_loop(lambda: batch.run(best), 5, 0)
    batched_s = el / 5
    # the same batch captured once as a HIP graph and replayed
    graph = batch.graph(best)
    graph.launch()
    ctx.check()
    graph_s = timed_loop(graph.launch, 5, 0) / 5
    graph.close()

    def one_at_a_time():
        for plan, fact in frags:
            k, s, ng = pyst.query(ctx, plan, fact)
            int(ng.item())

    one_at_a_time()
    t0 = time.perf_counter()
    one_at_a_time()
    seq_s = time.perf_counter() - t0
    # results of the two executions agree fragment by fragment
    res = batch.results()
    mismatches = 0
    for (k, s), (plan, fact) in zip(res, frags):
        r = pyst.query(ctx, plan, fact)
        m = int(r[2].item())
        if m != k.numel() or not torch.equal(torch.sort(k).values, torch.sort(r[0][:m]).values):
            mismatches += 1
    total_rows = int(sizes.sum())
    return {"fragments": nfrag, "probe_rows": total_rows, "tuning": {"fanout": best[0], "block": best[1],
            "max_load": best[2]}, "batched_ms": batched_s * 1e3, "sequential_ms": seq_s * 1e3,
            "batched_fragments_per_s": nfrag / batched_s, "sequential_fragments_per_s": nfrag / seq_s,
            "speedup": seq_s / batched_s, "graph_ms": graph_s * 1e3, "graph_speedup": seq_s / graph_s,
            "batched_probe_rows_per_s": total_rows / batched_s,
            "batched_gbs": total_rows * 16 / batched_s / 1e9, "result_mismatches": mismatches,
            "fact_pass_traffic": counter_traffic("k_bat_fact_staged", BATCH_WORKLOAD)}


def host_memory(log):
    """Host memory this process may still take: MemAvailable, capped by the
    cgroup limit minus its current use when one is set (bytes, and the figures)."""
    info = {}
    with open("/proc/meminfo") as f:
        for line in f:
            k, v = line.split(":", 1)
            if k in ("MemTotal", "MemAvailable"):
                info[k] = int(v.split()[0]) * 1024
    avail = info.get("MemAvailable", 0)
    for lim_p, cur_p in (("/sys/fs/cgroup/memory.max", "/sys/fs/cgroup/memory.current"),
                         ("/sys/fs/cgroup/memory/memory.limit_in_bytes", "/sys/fs/cgroup/memory/memory.usage_in_bytes")):
        try:
            lim = open(lim_p).read().strip()
            cur = int(open(cur_p).read().strip())
        except (OSError, ValueError):
            continue
        if lim.isdigit() and int(lim) < (1 << 60):
            info["cgroup_limit"] = int(lim)
            info["cgroup_used"] = cur
            avail = min(avail, int(lim) - cur)
        break
    info["usable"] = avail
    log("host memory: %s" % {k: "%.1f GB" % (v / 1e9) for k, v in info.items()})
    return avail, info


class PinnedHost:
    """Exact-size pinned host buffers from hipHostMalloc, returned to the system by
    free_all().  (torch's pinned allocator rounds sizes up to powers of two and keeps
    freed blocks, while the GPU machine pins at most about 64 GiB in all.)"""

    def __init__(self):
        import ctypes
        self.ct = ctypes
        self.hip = ctypes.CDLL("libamdhip64.so")
        self.hip.hipHostMalloc.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_size_t, ctypes.c_uint]
        self.hip.hipHostMalloc.restype = ctypes.c_int
        self.hip.hipHostFree.argtypes = [ctypes.c_void_p]
        self.hip.hipHostFree.restype = ctypes.c_int
        self.ptrs = []

    def empty(self, n, dtype):
        import numpy as np
        import torch
        ct = self.ct
        nbytes = max(int(n), 1) * torch.tensor([], dtype=dtype).element_size()
        p = ct.c_void_p()
        if self.hip.hipHostMalloc(ct.byref(p), nbytes, 0) != 0:
            raise MemoryError("hipHostMalloc of %d bytes failed" % nbytes)
        self.ptrs.append(p.value)
        npt = {torch.int32: (ct.c_int32, np.int32), torch.int64: (ct.c_int64, np.int64)}[dtype]
        arr = np.ctypeslib.as_array(ct.cast(p, ct.POINTER(npt[0])), shape=(max(int(n), 1),))[:n]
        return torch.from_numpy(arr)

    def free_all(self):
        for p in self.ptrs:
            self.hip.hipHostFree(p)
        self.ptrs = []


def _digest(k, s):
    """Order-independent fingerprint of a (keys, sums) result (wrapping int64 sums on the device)."""
    if k.numel() == 0:
        return (0, 0, 0, 0)
    return (int(k.numel()), int(k.sum()), int(s.sum()), int((k * 0x9E3779B1 + s).sum()))


def bench_config4(pyst, gen, log, want_rows, nreq, chunk, budget_total, serve_requests=False):
    """The served workload at its stated size: a 2e9-row chain fact table in
    pinned host memory streamed in 64M-row chunks under a 32 GiB device
    budget; the chain query streamed over all of it (raw and bit-packed); then
    Poisson streams of star/chain requests (sizes log-uniform in [1e6, rows])
    at 0.5 and 0.9 of the one-at-a-time capacity, FIFO against continuous
    batching, plus back-to-back bursts of both; every request of the
    continuous-batching runs compared with its FIFO (alone) result, and a
    seeded sample of requests checked against the oracle on its fact prefix.
    Without serve_requests only the streamed query runs (raw and packed)."""
    import numpy as np
    import torch

    import oracle
    na, nbd = 3_000_000, 300_000
    # Bytes a row: raw columns (pinned), and in the packed phase the packed copy (about
    # 10.2 B) pageable and pinned.  The raw table is unpinned before the packed one is
    # pinned: the box pins at most about 64 GiB.
    raw_b, packed_b = 24, 11
    pin_limit = 60 << 30
    avail, mem = host_memory(log)
    margin = 24 << 30
    fit = min((avail - margin) // (raw_b + 2 * packed_b), pin_limit // raw_b)
    nrows = int(min(want_rows, max(fit // 1_000_000 * 1_000_000, 64_000_000)))
    if nrows < want_rows:
        log("config4: host memory holds %d rows, not %d" % (nrows, want_rows))
    a_h, b_h = gen.chain_dims(na, nbd)
    a, b = to_dev(a_h), to_dev(b_h)
    t0 = time.perf_counter()
    log("config4: generating %d pinned fact rows" % nrows)
    pinned = PinnedHost()
    names = ("a_fk", "b_fk", "date", "price", "discount")
    dts = (torch.int32, torch.int32, torch.int32, torch.int64, torch.int32)
    host = [pinned.empty(nrows, d) for d in dts]
    gen.chain_fact(nrows, na, nbd, 0.0, out={c: t.numpy() for c, t in zip(names, host)})
    gen_s = time.perf_counter() - t0
    peak = h2d_peak(host[3][:min(nrows, 500_000_000)], log)
    out = {"rows": nrows, "requested_rows": want_rows, "host_memory": mem, "generate_s": gen_s,
           "chunk_rows": chunk, "device_budget_bytes": budget_total, "pinned_h2d_peak_gbs": peak}

    # --- the chain query streamed over the whole table
    ring = 2 * chunk * raw_b
    max_groups = 150_000_000
    sctx = pyst.Ctx(0, budget_total)
    plan = pyst.chain_plan(a, b, max_groups=max_groups)
    stream = {}
    for nbuf in (2, 3):
        sctx.timing(True)
        t0 = time.perf_counter()
        k, s_, ng = pyst.query_streamed(sctx, plan, host, chunk_rows=chunk, nbuf=nbuf, out_cap=max_groups)
        sctx.check()
        dt = time.perf_counter() - t0
        sctx.timing(False)
        copy_ms, copies = sctx.kernel_time("h2d_chunk")
        fact_ms, _ = sctx.kernel_time("fact_pass")
        gbs = nrows * raw_b / dt / 1e9
        stream["nbuf%d" % nbuf] = {"seconds": dt, "fact_rows_per_s": nrows / dt, "h2d_gbs": gbs,
                                   "frac_of_pinned_h2d": gbs / peak, "copy_busy_ms": copy_ms,
                                   "compute_busy_ms": fact_ms, "chunks": copies, "groups": int(ng.item())}
        stream_digest = _digest(k[:int(ng.item())], s_[:int(ng.item())])
        del k, s_
    torch.cuda.empty_cache()
    # the chunked path against the oracle: a 200M-row prefix of the same pinned
    # table streamed in the configured chunks (three full ones and a partial one)
    pre = min(nrows, 200_000_000)
    k, s_, ng = pyst.query_streamed(sctx, plan, [t[:pre] for t in host], chunk_rows=chunk, nbuf=2, out_cap=max_groups)
    sctx.check()
    m = int(ng.item())
    got_k, got_s = k[:m].cpu().numpy(), s_[:m].cpu().numpy()
    del k, s_
    t0 = time.perf_counter()
    wk, ws = oracle.chain_query(a_h, b_h, {c: t[:pre].numpy() for c, t in zip(names, host)})
    o = np.argsort(got_k)
    stream["oracle_check"] = {
        "rows": pre, "chunk_rows": chunk, "groups": int(len(wk)), "oracle_s": time.perf_counter() - t0,
        "equal": bool(len(got_k) == len(wk) and np.array_equal(got_k[o], wk) and np.array_equal(got_s[o], ws))}
    log("config4: streamed %d-row prefix equal to the oracle: %s" % (pre, stream["oracle_check"]["equal"]))
    del got_k, got_s, wk, ws
    stream["workload"] = "chain query, fact %d rows (24 B/row) from pinned host, %d-row chunks, %d GiB arena" % (
        nrows, chunk, budget_total >> 30)
    out["stream"] = stream

    # --- serving
    serve = {}
    if serve_requests:
        rows = np.minimum(gen.loguniform_i64(nreq, 1e6, nrows, gen.seed(4, 7, 0)), nrows)
        kinds = ["star" if i % 2 == 0 else "chain" for i in range(nreq)]
        srv_budget = budget_total - ring - (1 << 20)

        def plan_for(kind, r):
            if kind == "star":
                return pyst.fact_star_plan(b), nbd
            g = int(min(max(r // 8, 1024), max_groups))
            return pyst.chain_plan(a, b, max_groups=g), g

        # seeded oracle sample: two star and two chain requests small enough for the
        # single-threaded oracle (star <= 1.5e8 rows, chain <= 4e7 rows)
        rng = np.random.default_rng(gen.seed(4, 9, 0))
        small_star = [i for i in range(nreq) if kinds[i] == "star" and rows[i] <= 150_000_000]
        small_chain = [i for i in range(nreq) if kinds[i] == "chain" and rows[i] <= 40_000_000]
        sample = sorted(list(rng.choice(small_star, min(2, len(small_star)), replace=False)) +
                        list(rng.choice(small_chain, min(2, len(small_chain)), replace=False)))
        sample = [int(i) for i in sample]
        star_ids = [i for i in range(nreq) if kinds[i] == "star"]
        big_star = max(star_ids, key=lambda i: rows[i]) if star_ids else None

        def run(max_active, arrivals, packed_cols=None, keep=()):
            srv = pyst.Server(None if packed_cols else host, budget=srv_budget, max_active=max_active, nbuf=2,
                              chunk_rows=chunk, packed=packed_cols)
            for kind in ("star", "chain"):  # warm the resident dimension tables outside the trace
                p, c = plan_for(kind, 1_000_000)
                srv.wait(srv.submit(p, 1_000_000, c))
            base = srv.stats()
            t_start = time.perf_counter()
            tickets = [None] * nreq

            def producer():
                for i in range(nreq):
                    delay = t_start + arrivals[i] - time.perf_counter()
                    if delay > 0:
                        time.sleep(delay)
                    p, c = plan_for(kinds[i], int(rows[i]))
                    tickets[i] = srv.submit(p, int(rows[i]), c)

            failed = []

            def producer_checked():
                try:
                    producer()
                except BaseException as e:  # noqa: BLE001 -- reported by the consumer below
                    failed.append(e)

            th = threading.Thread(target=producer_checked)
            th.start()
            lat, digests, kept = [], [], {}
            for i in range(nreq):
                while tickets[i] is None:
                    if failed:
                        raise RuntimeError("config4 request producer failed: %r" % (failed[0],))
                    time.sleep(0.0005)
                k, s_, l_ = srv.wait(tickets[i])
                lat.append(l_)
                digests.append(_digest(k, s_))
                if i in keep:
                    kept[i] = (k.cpu().numpy(), s_.cpu().numpy())
                del k, s_
            th.join()
            makespan = time.perf_counter() - t_start
            st = srv.stats()
            srv.check()
            srv.close()
            torch.cuda.empty_cache()
            lat = np.array(lat)
            res = {"p50_ms": float(np.percentile(lat, 50, method="nearest")),
                   "p99_ms": float(np.percentile(lat, 99, method="nearest")),
                   "mean_ms": float(lat.mean()), "max_ms": float(lat.max()), "makespan_s": makespan,
                   "requests_per_s": nreq / makespan, "rows_per_s": float(rows.sum()) / makespan,
                   "chunks_copied": st["chunks_copied"] - base["chunks_copied"],
                   "h2d_gb": (st["bytes_copied"] - base["bytes_copied"]) / 1e9,
                   "max_active_seen": st["max_active_seen"],
                   "admission_waits": st["admission_waits"] - base["admission_waits"]}
            log("config4: served %d requests, max_active %d: makespan %.1f s, p50 %.0f ms, p99 %.0f ms, "
                "admission waits %d" % (nreq, max_active, makespan, res["p50_ms"], res["p99_ms"], res["admission_waits"]))
            return res, digests, kept

        serve = {}
        traces = {}
        burst_fifo, fifo_digests, _ = run(1, np.zeros(nreq))
        serve["burst_one_at_a_time"] = burst_fifo
        capacity = burst_fifo["requests_per_s"]
        burst_cb, d, kept = run(8, np.zeros(nreq), keep=set(sample + ([big_star] if big_star is not None else [])))
        burst_cb["results_equal_to_alone"] = sum(x == y for x, y in zip(d, fifo_digests))
        serve["burst_continuous_batching"] = burst_cb
        for rho in (0.5, 0.9):
            lam = rho * capacity
            arrivals = gen.poisson_arrivals(nreq, lam, gen.seed(4, 8, int(rho * 10)))
            traces[rho] = arrivals
            log("config4: Poisson rate %.2f req/s (%.1f x one-at-a-time capacity)" % (lam, rho))
            fifo, _, _ = run(1, arrivals)
            cb, d, _ = run(8, arrivals)
            cb["results_equal_to_alone"] = sum(x == y for x, y in zip(d, fifo_digests))
            serve["rho%.1f" % rho] = {"arrival_rate_per_s": lam, "one_at_a_time": fifo, "continuous_batching": cb}

        # the oracle on the sampled requests' fact prefixes (results of the burst run)
        checks = []
        for i in sample:
            pref = {c: v[:int(rows[i])].numpy() for c, v in zip(("a_fk", "b_fk", "date", "price", "discount"), host)}
            t0 = time.perf_counter()
            if kinds[i] == "star":
                wk, ws = oracle.star_query(b_h, {"fk": pref["b_fk"], "date": pref["date"], "price": pref["price"]})
            else:
                wk, ws = oracle.chain_query(a_h, b_h, pref)
            k, s_ = kept[i]
            o = np.argsort(k)
            ok = bool(len(k) == len(wk) and np.array_equal(k[o], wk) and np.array_equal(s_[o], ws))
            checks.append({"request": i, "kind": kinds[i], "rows": int(rows[i]), "groups": int(len(wk)), "equal": ok,
                           "oracle_s": time.perf_counter() - t0})
        if big_star is not None:
            i = big_star
            pref = {c: v[:int(rows[i])].numpy() for c, v in zip(("b_fk", "date", "price"), host[1:4])}
            t0 = time.perf_counter()
            wk, ws, used = oracle.star_query_threaded(b_h, {"fk": pref["b_fk"], "date": pref["date"],
                                                            "price": pref["price"]}, threads=len(os.sched_getaffinity(0)))
            k, s_ = kept[i]
            o = np.argsort(k)
            checks.append({"request": i, "kind": "star", "rows": int(rows[i]), "groups": int(len(wk)),
                           "equal": bool(np.array_equal(k[o], wk) and np.array_equal(s_[o], ws)),
                           "checked_by": "threaded baseline (%d threads; equal to the oracle by test)" % used,
                           "seconds": time.perf_counter() - t0})
        serve["oracle_checks"] = checks
        serve["result_mismatches"] = sum(not c["equal"] for c in checks)

    # --- the same table bit-packed: encoded into pageable memory, the raw table
    # unpinned, the packed one pinned; streamed and served again
    log("config4: packing %d rows" % nrows)
    t0 = time.perf_counter()
    packed_pageable = [pyst.pack(t, pinned=False) for t in host]
    pack_s = time.perf_counter() - t0
    host = None
    pinned.free_all()
    packed = []
    for (bl, w), d in zip(packed_pageable, dts):
        pb, pw = pinned.empty(bl.numel(), torch.int64).view(bl.shape), pinned.empty(w.numel(), torch.int32)
        pb.copy_(bl)
        pw.copy_(w)
        packed.append((pb, pw, nrows, d))
    del packed_pageable
    packed_bytes = sum(bl.numel() * 8 + w.numel() * 4 for bl, w, _, _ in packed)
    for nbuf in (2, 3):
        sctx.timing(True)
        t0 = time.perf_counter()
        k, s_, ng = pyst.query_streamed_packed(sctx, plan, packed, chunk_rows=chunk, nbuf=nbuf, out_cap=max_groups)
        sctx.check()
        dt = time.perf_counter() - t0
        sctx.timing(False)
        copy_ms, _ = sctx.kernel_time("h2d_chunk")
        unpack_ms, _ = sctx.kernel_time("unpack")
        fact_ms, _ = sctx.kernel_time("fact_pass")
        stream["packed_nbuf%d" % nbuf] = {
            "seconds": dt, "fact_rows_per_s": nrows / dt, "link_gbs": packed_bytes / dt / 1e9,
            "frac_of_pinned_h2d": packed_bytes / dt / 1e9 / peak, "copy_busy_ms": copy_ms,
            "unpack_busy_ms": unpack_ms, "compute_busy_ms": fact_ms, "groups": int(ng.item()),
            "equal_to_raw": _digest(k[:int(ng.item())], s_[:int(ng.item())]) == stream_digest,
            "speedup_vs_raw": stream["nbuf%d" % nbuf]["seconds"] / dt}
        del k, s_
    sctx.close()
    stream["packed"] = {"bytes": packed_bytes, "bytes_per_row": packed_bytes / nrows,
                        "ratio": nrows * raw_b / packed_bytes, "host_encode_s": pack_s}
    if serve_requests:
        cbp, d, _ = run(8, traces[0.9], packed)
        cbp["results_equal_to_alone"] = sum(x == y for x, y in zip(d, fifo_digests))
        serve["rho0.9"]["continuous_batching_packed"] = cbp
        serve.update({"requests": nreq, "server_budget_bytes": srv_budget, "ring_bytes": ring, "max_active": 8,
                      "request_rows_mean": float(rows.mean()), "request_rows_max": int(rows.max()),
                      "workload": "50/50 star and chain requests, scan sizes log-uniform in [1e6, %d]; device arena "
                                  "%d GiB in total (chunk ring of 2 x %d rows included)" % (nrows, budget_total >> 30,
                                                                                         chunk)})
    else:
        serve = {"skipped": "full-size serving runs only with --config4-serve (a full-size Poisson serving run "
                            "failed with a device memory fault whose cause is not found yet)"}
    out["serve"] = serve
    del packed
    pinned.free_all()
    return out


def host_cpu_info():
    """Cores this process may run on, the machine's count and the CPU model."""
    model = None
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    return {"affinity_cores": len(os.sched_getaffinity(0)), "cpu_count": os.cpu_count(), "model": model}


def cpu_baseline(b_host, p_host, sample_rows, log):
    """The oracle on one core over a bounded sample, and the threaded CPU
    baseline (the same algorithm over every core this process may use) on the
    whole probe table, checked equal to the oracle on the sample first."""
    import numpy as np

    import oracle
    info = host_cpu_info()
    sample_rows = min(sample_rows, len(p_host["fk"]))
    sample = {c: v[:sample_rows] for c, v in p_host.items()}
    log("cpu oracle on %d probe rows" % sample_rows)
    t0 = time.perf_counter()
    ok, osum = oracle.star_query(b_host, sample)
    dt = time.perf_counter() - t0
    out = {"value": sample_rows / dt, "unit": "probe rows/s", "cores": 1, "kind": "oracle",
           "sample": "full build table (%d rows), first %d probe rows; %.1f s single-threaded"
                     % (len(b_host["key"]), sample_rows, dt),
           "host": info}
    threads = info["affinity_cores"]
    tk, ts, used = oracle.star_query_threaded(b_host, sample, threads=threads)
    equal = bool(np.array_equal(tk, ok) and np.array_equal(ts, osum))
    n = len(p_host["fk"])
    log("threaded cpu baseline on %d probe rows, %d threads" % (n, threads))
    t0 = time.perf_counter()
    oracle.star_query_threaded(b_host, p_host, threads=threads)
    dtm = time.perf_counter() - t0
    out["threaded"] = {"value": n / dtm, "unit": "probe rows/s", "cores": used, "kind": "threaded baseline",
                       "equal_to_oracle_on_sample": equal,
                       "sample": "full build table, all %d probe rows; %.2f s on %d threads" % (n, dtm, used)}
    return out


if __name__ == "__main__":
    main()
