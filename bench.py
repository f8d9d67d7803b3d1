"""Benchmark: sliding-window streaming IVF on one MI355X.

Default workload: the sliding-window plain FP32 configuration.  The window
holds 1,000,000 vectors (d=128, integer values 0..255 stored as fp32) in 1,024
lists (k-means centroids) with slabs of 64.  Each step inserts 10,000 new
vectors, searches 10,000 queries (nprobe 32, k 10) and evicts the oldest
10,000 -- the paper's insert -> search -> delete loop.  All inputs are
synthetic, generated on the host and copied to HBM before timing (the
paper's datasets are not available).

Prints one JSON line.  value = queries answered per second of window-step
time (every step also inserts and deletes 10,000 vectors).  Reported beside
it: per-operation device rates, step-latency percentiles (eager and
HIP-graph steps), recall@10 and an nprobe sweep against exact kNN, the
roofline of the scan kernel, and the CPU oracle's rate on a bounded sample.

Other modes (not the headline line):
  --workload batched   the batched uneven form: 5M vectors over 2,048 Zipf-
                       skewed lists, 32k queries with per-query nprobe
                       U[8,128] and k in {1,10,100}, +20k / -20k random ids
                       per step, autotuned schedule, eager and graph steps
  --workload mutation  bulk mutation kernels: the 1M window inserted in one
                       call, then half of it deleted (random ids) in one call
  --workload serve     the serving form: a 50M-vector fp16 window (d=128,
                       16,384 lists, slab 128) under a Poisson stream of
                       searches, inserts and deletes through the
                       overlapping request server; p50/p99 per request type
  --storage bf16|f16   the precision form on the same window data
  --workload precision 10M unit vectors, d=96, inner product, bf16 slabs,
                       4,096 lists, slab 128, 16k queries, nprobe 64,
                       re-rank of the top 40
"""
import argparse
import hashlib
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

# FP32 VALU peak with packed FP32 off: 256 CUs x 4 SIMD x 16 lanes x 2 flop
# (fma) x 2.4 GHz.  Dense MFMA peak, BF16 / FP16: 2.5 PFLOP/s.
ALU_PEAK_TFLOPS = 256 * 4 * 16 * 2 * 2.4e9 / 1e12
MFMA16_PEAK_TFLOPS = 2500.0


HBM_PEAK_GBPS = 8000.0


def fp32_scan_roofline(evals, d, scan_ms, tile, traffic=None):
    """Roofline of the FP32 scan that ran.

    Bound: a list is read once per work item of `tile` queries, so one
    (query, list entry) evaluation moves (4d + 4) / tile bytes of slab rows and
    ids; at tile 16 that is 16 flop/B of matrix-core work against a ridge of
    2500 / 8 = 313 flop/B, so the certified scan is HBM-bound and is reported
    against the HBM peak.  The VALU scan (tiles 4
    and 8) sits at 3d*tile/(4d+4) <= 6 flop/B, under its own ridge of 9.8 only
    because packed FP32 is off, and is reported against the FP32 VALU peak on
    its 3d flops per evaluation.  The matrix-core accounting of the certified
    scan (its bf16 filter: rows rounded once, queries in two parts, so 2 * 2 *
    32 * ceil(d / 32) flops per evaluation against the bf16 MFMA peak) is kept
    beside it.  Where consecutive tiles of one list re-read its chunk
    from L2 / MALL (many queries on few long lists), the per-tile byte count
    exceeds what HBM can deliver in the measured time: the scan is then
    reported against the matrix-core peak, with the HBM model beside it."""
    exact_tf = evals * 3.0 * d / (scan_ms * 1e-3) / 1e12
    if tile == 16:
        per_eval = (4.0 * d + 4.0) / tile
        gbps = evals * per_eval / (scan_ms * 1e-3) / 1e9
        tf = evals * 4.0 * 32 * ((d + 31) // 32) / (scan_ms * 1e-3) / 1e12
        hbm = {"bound": "hbm", "kernel": "k_scan_cert", "achieved": round(gbps, 1), "peak": HBM_PEAK_GBPS,
               "unit": "GB/s", "frac": round(gbps / HBM_PEAK_GBPS, 4),
               "bytes_per_eval": per_eval, "algorithmic_bytes_per_launch": int(evals * per_eval)}
        mf = {"achieved_tflops": round(tf, 3), "peak_tflops": MFMA16_PEAK_TFLOPS,
              "frac": round(tf / MFMA16_PEAK_TFLOPS, 4), "flops_per_eval": 4 * 32 * ((d + 31) // 32)}
        if gbps <= HBM_PEAK_GBPS:
            roof = dict(hbm, mfma=mf)
        else:
            roof = {"bound": "mfma", "kernel": "k_scan_cert", "achieved": mf["achieved_tflops"],
                    "peak": MFMA16_PEAK_TFLOPS, "unit": "TFLOP/s", "frac": mf["frac"],
                    "flops_per_eval": mf["flops_per_eval"],
                    "hbm_model": dict(hbm, note="per-tile chunk reads exceed HBM peak: served from L2/MALL")}
    else:
        roof = {"bound": "alu", "kernel": "k_scan_sq", "achieved": round(exact_tf, 3),
                "peak": round(ALU_PEAK_TFLOPS, 2), "unit": "TFLOP/s", "frac": round(exact_tf / ALU_PEAK_TFLOPS, 4),
                "flops_per_eval": 3 * d}
    roof.update({"traffic": traffic,
                 "traffic_unit": "bytes per launch (DRAM, rocprofv3 FETCH_SIZE + WRITE_SIZE, copy-calibrated; "
                                 "taken from the committed counter summary while the scan source is unchanged)",
                 "evals_per_launch": evals, "exact_distance_tflops": round(exact_tf, 3),
                 "avg_launch_ms": round(scan_ms, 4)})
    return roof


STORAGE = {"f32": 0, "bf16": 1, "f16": 2}


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=30)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", default="window",
                    choices=["window", "tiny", "precision", "serve", "batched", "mutation", "tier"])
    ap.add_argument("--serve-seconds", type=float, default=5.0, help="serve: length of the arrival stream")
    ap.add_argument("--serve-rate", type=float, default=2000.0, help="serve: Poisson arrival rate (req/s)")
    ap.add_argument("--serve-n", type=int, default=50_000_000, help="serve: steady-state window size")
    ap.add_argument("--storage", default=None, choices=list(STORAGE))
    ap.add_argument("--batch", type=int, default=None, help="window/tiny: vectors inserted and evicted per step")
    ap.add_argument("--rerank", type=int, default=4, help="re-rank factor R for bf16/f16 storage")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--recall-queries", type=int, default=1000)
    ap.add_argument("--no-sweep", action="store_true", help="skip the nprobe / recall sweep")
    ap.add_argument("--schedule", default=None,
                    help="T,log2chunk,persistent: set the search schedule instead of running the autotuner")
    ap.add_argument("--latency-steps", type=int, default=1000,
                    help="window: steady-state steps of each latency leg (at B and at B=1000); 0 skips them")
    ap.add_argument("--no-forms", action="store_true",
                    help="window: skip the bf16 form and the bulk-mutation leg")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="also run a plain 1 GiB device copy (scale for DRAM byte counters)")
    return ap.parse_args()


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def recorded_traffic(name="k_scan_window_1M.md"):
    """DRAM bytes per search of the scan from the committed counter summary, or
    None when the source of its kernel changed since the counters were taken."""
    prof = os.path.join(ROOT, "profiles", name)
    src = {"k_scan_cert_window_1M.md": "scan_cert.h", "k_scan_mfma_precision_10M.md": "scan_mfma.hip"}.get(name, "search.hip")
    src = os.path.join(ROOT, "paper_2601_11808_amd", "csrc", src)
    try:
        kv = dict(l.split(": ", 1) for l in open(prof).read().splitlines() if l.startswith(("traffic_", "source_")))
        if hashlib.sha256(open(src, "rb").read()).hexdigest() != kv["source_sha256"].strip():
            return None
        return int(kv["traffic_bytes_per_launch"])
    except (OSError, KeyError, ValueError):
        return None


def exact_topk(xw, idw, q, k, metric, chunk=1 << 18):
    """Exact top-k (float64) of q over the window rows, ties by smaller id:
    squared L2 ascending, or inner product descending."""
    qd = q.astype(np.float64)
    best_s = np.full((q.shape[0], k), np.inf)
    best_i = np.full((q.shape[0], k), np.iinfo(np.int64).max, dtype=np.int64)
    for s in range(0, xw.shape[0], chunk):
        xd = xw[s:s + chunk].astype(np.float64)
        if metric == 0:
            sc = (xd * xd).sum(1)[None, :] - 2.0 * (qd @ xd.T) + (qd * qd).sum(1)[:, None]
        else:
            sc = -(qd @ xd.T)
        kk = min(k, sc.shape[1])
        part = np.argpartition(sc, kk - 1, axis=1)[:, :kk]
        cs = np.concatenate([best_s, np.take_along_axis(sc, part, 1)], 1)
        ci = np.concatenate([best_i, idw[s:s + chunk][part]], 1)
        o = np.lexsort((ci, cs), axis=1)[:, :k]
        best_s, best_i = np.take_along_axis(cs, o, 1), np.take_along_axis(ci, o, 1)
    return best_i


def copy_calibration():
    """A plain 1 GiB device-to-device copy: its DRAM byte counters scale those
    of the library's kernels (1 GiB read, 1 GiB written)."""
    import torch
    nbytes = 1 << 30
    src = torch.ones(nbytes // 4, dtype=torch.float32, device="cuda:0")
    dst = torch.empty_like(src)
    torch.cuda.synchronize()
    dst.copy_(src)
    torch.cuda.synchronize()
    del src, dst


def cpu_model():
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def cpu_baseline(w, x, ids, q, nprobe, k, n_sample_q, reps=3):
    """The CPU oracle on a bounded sample of the same workload: window steps
    (insert a batch, search a query sample, delete the oldest batch) on the
    full window, three steps, median; the search time is scaled to the full
    query batch."""
    import oracle
    ix = oracle.OracleIndex(w.dim, w.nlist, w.centroids, w.metric, w.slab, 1 << 26, ids.shape[0] + 4 * w.batch)
    t0 = time.time()
    assert ix.add(x, ids) == 0
    build_s = time.time() - t0
    rates, parts = [], []
    for t in range(1, reps + 1):
        xb, idb = w.stream_batch(t)
        old = w.oldest_ids(t)
        t0 = time.time()
        assert ix.add(xb, idb) == 0
        t_add = time.time() - t0
        t0 = time.time()
        st, _, _ = ix.search(q[:n_sample_q], k, nprobe)
        t_search = time.time() - t0
        t0 = time.time()
        st, nr = ix.remove(old)
        t_rm = time.time() - t0
        step_s = t_add + t_search * (q.shape[0] / n_sample_q) + t_rm
        rates.append(q.shape[0] / step_s)
        parts.append((t_add, t_search, t_rm))
    ix.close()
    med = int(np.argsort(rates)[len(rates) // 2])
    t_add, t_search, t_rm = parts[med]
    return {
        "value": round(float(rates[med]), 1), "unit": "queries/s", "cores": oracle.num_threads(), "kind": "oracle",
        "cpu_model": cpu_model(), "host_cpus": os.cpu_count(), "repetitions": reps,
        "all_values": [round(float(r), 1) for r in rates],
        "sample": (f"median of {reps} window steps on the full {ids.shape[0]}-vector window; median step: insert "
                   f"{w.batch} ({t_add:.2f} s), search {n_sample_q} of {q.shape[0]} queries ({t_search:.2f} s, "
                   f"scaled x{q.shape[0] / n_sample_q:.0f}), delete {w.batch} ({t_rm:.3f} s); untimed window "
                   f"build {build_s:.1f} s"),
        "insert_vec_per_s": round(w.batch / t_add, 1), "delete_vec_per_s": round(w.batch / max(t_rm, 1e-9), 1),
    }


def latency_leg(ix, pool, q, k, nprobe, first_add_id, first_old_id, n_base, B, steps, dist, lab):
    """Host wall-clock per window step (add B, search, remove the oldest B;
    synchronised at the end of each step) over `steps` steady-state steps.
    Vectors come from a device-resident pool of earlier stream batches under
    fresh ids, so the window keeps its size and distribution."""
    import torch
    dev = pool.device
    ids = torch.arange(first_add_id, first_add_id + B * steps, device=dev)
    olds = torch.arange(first_old_id, first_old_id + B * steps, device=dev)
    npool = pool.shape[0] // B
    times = []
    torch.cuda.synchronize()
    for s_ in range(steps):
        xb = pool[(s_ % npool) * B:(s_ % npool + 1) * B]
        ts = time.perf_counter()
        ix.step(xb, ids[s_ * B:(s_ + 1) * B], q, k, nprobe, olds[s_ * B:(s_ + 1) * B], out=(dist, lab))
        torch.cuda.synchronize()
        times.append((time.perf_counter() - ts) * 1e3)
    assert ix.sync() == 0
    assert ix.stats()["live"] == n_base
    v = np.sort(np.array(times))
    return {"batch": B, "steps": steps, "p50_ms": round(float(np.percentile(v, 50)), 4),
            "p99_ms": round(float(np.percentile(v, 99)), 4), "max_ms": round(float(v[-1]), 4),
            "mean_ms": round(float(v.mean()), 4)}, first_add_id + B * steps, first_old_id + B * steps


def bulk_mutation_leg(w, x, ids, reps=3):
    """Mutation kernels at bulk scale on the window data: the whole window
    inserted in one call, then half of it (uniformly random ids) deleted in
    one call; device time of each call from the library's HIP events, median
    of `reps` after one warm-up.  Algorithmic bytes per unit: insert 4d (read)
    + 4d (write) + 4 (id) + 4 (address table) per vector; delete 4 (address
    table read) + 2 (4d + 4) (a tail entry moved into the hole) + 8 (two
    address-table writes) per removed id, the upper bound the method moves."""
    import torch
    import paper_2601_11808_amd as sivf
    dev = torch.device("cuda:0")
    N, d = x.shape
    num_slabs = int(1.15 * N / w.slab) + w.nlist
    ix = sivf.Index(w.dim, w.nlist, w.centroids, metric=w.metric, slab_capacity=w.slab, num_slabs=num_slabs,
                    id_capacity=N, max_batch=N, max_queries=16, max_k=16, max_nprobe=16, device="cuda:0")
    xd, idd = torch.from_numpy(x).to(dev), torch.from_numpy(ids).to(dev)
    rng = np.random.default_rng([w.seed, 7, 0])
    add_ms, rm_ms = [], []
    for r in range(reps + 1):
        rm = torch.from_numpy(np.sort(rng.choice(N, N // 2, replace=False)).astype(np.int64)).to(dev)
        torch.cuda.synchronize()
        ix.profile_read()
        ix.profile(True)
        ix.add(xd, idd)
        assert ix.sync() == 0
        pa = ix.profile_read()
        nr = ix.remove(rm)
        assert ix.sync() == 0
        pr = ix.profile_read()
        ix.profile(False)
        assert int(nr.item()) == N // 2
        ix.remove(idd)                      # empty the index for the next repetition
        assert ix.sync() == 0 and ix.stats()["live"] == 0
        if r > 0:
            add_ms.append(pa["add"][0])
            rm_ms.append(pr["remove"][0])
    ix.close()
    del ix, xd, idd
    torch.cuda.empty_cache()
    ins_b = N * (4 * d + 4 * d + 8)
    del_b = (N // 2) * (4 + 2 * (4 * d + 4) + 8)
    am, rmm = float(np.median(add_ms)), float(np.median(rm_ms))
    ins_gbps, del_gbps = ins_b / (am * 1e-3) / 1e9, del_b / (rmm * 1e-3) / 1e9
    return {
        "insert": {"vectors": N, "ms": round(am, 4), "vec_per_s": round(N / (am * 1e-3), 1),
                   "algorithmic_bytes": ins_b, "GBps": round(ins_gbps, 1), "frac": round(ins_gbps / HBM_PEAK_GBPS, 4),
                   "bytes_per_vector": 8 * d + 8,
                   "note": "the call includes the exact coarse assignment (bf16 MFMA with the certified bound; FP64 re-check of the rows it leaves undecided)"},
        "delete": {"ids": N // 2, "ms": round(rmm, 4), "vec_per_s": round((N // 2) / (rmm * 1e-3), 1),
                   "algorithmic_bytes": del_b, "GBps": round(del_gbps, 1), "frac": round(del_gbps / HBM_PEAK_GBPS, 4),
                   "bytes_per_id": 4 + 2 * (4 * d + 4) + 8},
        "repetitions": reps,
    }


def build_window_index(sivf, w, x, ids, storage, rerank, id_cap, B, nq, nprobe, dev):
    import torch
    num_slabs = int(1.15 * (w.n_base + 2 * B) / w.slab) + w.nlist
    chunk = 65536
    ix = sivf.Index(w.dim, w.nlist, w.centroids, metric=w.metric, slab_capacity=w.slab, num_slabs=num_slabs,
                    id_capacity=id_cap, max_batch=max(chunk, B), max_queries=nq, max_k=16,
                    max_nprobe=max(128, nprobe), storage=storage, rerank_factor=rerank, device="cuda:0")
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    bulk_ms = 0.0
    for s0 in range(0, x.shape[0], 1 << 20):
        xd = torch.from_numpy(x[s0:s0 + (1 << 20)]).to(dev)
        idd = torch.from_numpy(ids[s0:s0 + (1 << 20)]).to(dev)
        torch.cuda.synchronize()
        e0.record()
        for c in range(0, xd.shape[0], chunk):
            ix.add(xd[c:c + chunk], idd[c:c + chunk])
        e1.record()
        assert ix.sync() == 0
        bulk_ms += e0.elapsed_time(e1)
    return ix, bulk_ms


def timed_steps(ix, bx, bi, bo, qd, k, nprobe, dist, lab, t_from, t_to):
    import torch
    ix.profile_read()
    ix.profile(True)
    step_ms = []
    torch.cuda.synchronize()
    t_all = time.perf_counter()
    for t in range(t_from, t_to):
        ts = time.perf_counter()
        ix.step(bx[t], bi[t], qd, k, nprobe, bo[t], out=(dist, lab))
        torch.cuda.synchronize()
        step_ms.append((time.perf_counter() - ts) * 1e3)
    elapsed = time.perf_counter() - t_all
    prof = ix.profile_read()
    ix.profile(False)
    assert ix.sync() == 0
    return elapsed, step_ms, prof


def nprobe_sweep(ix, qd, k, nq, nprobe, grid, recall_of, dist, lab):
    sweep = []
    ix.profile(True)
    for npb in grid:
        ix.search(qd, k, npb, out=(dist, lab))
        ix.sync()
        ix.profile_read()
        for _ in range(3):
            ix.search(qd, k, npb, out=(dist, lab))
        pr = ix.profile_read()
        sms = pr["search"][0] / max(pr["search"][1], 1)
        sweep.append({"nprobe": npb, "recall_at_10": round(recall_of(lab.cpu().numpy()), 4),
                      "search_qps": round(nq / (sms * 1e-3), 1)})
    ix.profile(False)
    ok95 = [r for r in sweep if r["recall_at_10"] >= 0.95]
    best95 = max(ok95, key=lambda r: r["search_qps"]) if ok95 else None
    return sweep, best95


def main():
    a = parse()
    if a.gpus != 1:
        print("bench.py runs on one GPU only: every GPU box here has a single MI355X, so --gpus must be 1 "
              "(multi-GPU sharding is a design note, not part of this build)", file=sys.stderr)
        sys.exit(2)
    if a.workload == "serve":
        return serve_main(a)
    if a.workload == "batched":
        return batched_main(a)
    if a.workload == "mutation":
        return mutation_main(a)
    if a.workload == "tier":
        return tier_main(a)
    import torch
    import paper_2601_11808_amd as sivf
    import workloads

    if not os.path.exists(sivf.LIB_PATH):
        raise SystemExit("libsivf.so is not built: run python -c 'import __graft_entry__ as g; g.build()'")
    dev = torch.device("cuda:0")
    t0 = time.time()
    w = {"window": workloads.window, "tiny": workloads.tiny, "precision": workloads.precision}[a.workload]()
    if a.batch:
        w.batch = a.batch
    storage = a.storage or ("bf16" if a.workload == "precision" else "f32")
    st_code = STORAGE[storage]
    rerank = a.rerank if st_code else 0
    x, ids = w.base()
    q = w.queries()
    B, nq, k, nprobe = w.batch, q.shape[0], w.k, w.nprobe
    T = a.warmup + a.steps
    T2 = T + a.steps
    lat_steps = a.latency_steps if a.workload == "window" else 0
    B_small = 1000
    log(f"[bench] workload {w.name}: N={w.n_base} d={w.dim} nlist={w.nlist} C={w.slab} B={B} nq={nq} "
        f"storage={storage} (generated in {time.time() - t0:.1f} s)")
    # ids: base, then T2 stream batches, then the latency legs (B and B_small per step)
    id_cap = w.n_base + B * (T2 + 2) + lat_steps * (B + B_small)
    ix, bulk_ms = build_window_index(sivf, w, x, ids, st_code, rerank, id_cap, B, nq, nprobe, dev)
    log(f"[bench] workspace {ix.workspace_bytes / 2**30:.2f} GiB; bulk load {x.shape[0]} vectors: {bulk_ms:.1f} ms "
        f"({x.shape[0] / bulk_ms * 1e3 / 1e6:.2f} M vec/s)")
    # stream batches 1..T2, resident in HBM before timing
    bx, bi, bo = [], [], []
    for t in range(1, T2 + 1):
        xb, idb = w.stream_batch(t)
        bx.append(torch.from_numpy(xb).to(dev))
        bi.append(torch.from_numpy(idb).to(dev))
        bo.append(torch.from_numpy(w.oldest_ids(t)).to(dev))
    qd = torch.from_numpy(q).to(dev)
    dist = torch.empty((nq, k), dtype=torch.float32, device=dev)
    lab = torch.empty((nq, k), dtype=torch.int64, device=dev)
    t0 = time.perf_counter()
    if a.schedule:
        tile, sh, pers = (int(v) for v in a.schedule.split(","))
        ix.set_search_schedule(tile, sh, pers)
    else:
        tile, sh, pers = ix.tune_search(qd, k, nprobe)   # search schedule for this batch shape (untimed)
    log(f"[bench] schedule: {tile} queries x 2^{sh} positions per work item, persistent={pers} "
        f"({'given' if a.schedule else 'autotuned'}, {time.perf_counter() - t0:.1f} s)")
    torch.cuda.synchronize()
    for t in range(a.warmup):
        ix.step(bx[t], bi[t], qd, k, nprobe, bo[t], out=(dist, lab))
    assert ix.sync() == 0
    elapsed, step_ms, prof = timed_steps(ix, bx, bi, bo, qd, k, nprobe, dist, lab, a.warmup, T)
    # scan roofline: distance evaluations of one search = sum over (query,
    # probe) of the probed list's length
    probes = ix.probe(qd, nprobe).cpu().numpy()
    lens = ix.dump()["list_len"].astype(np.int64)
    evals = int(lens[probes[probes >= 0]].sum())
    balanced = nq * nprobe * w.n_base / w.nlist
    scan_ms = prof["scan"][0] / max(prof["scan"][1], 1)
    log(f"[bench] {a.steps} steps in {elapsed:.3f} s; device ms per class: "
        + ", ".join(f"{kk}={v[0] / max(v[1], 1):.3f}" for kk, v in prof.items()))

    # graph mode: the same step captured once and replayed on refilled buffers
    gx = torch.empty((B, w.dim), dtype=torch.float32, device=dev)
    gi = torch.empty(B, dtype=torch.int64, device=dev)
    go = torch.empty(B, dtype=torch.int64, device=dev)
    nrem = torch.zeros(1, dtype=torch.int64, device=dev)
    g = ix.step_graph(gx, gi, qd, k, nprobe, go, dist, lab, nrem)
    gsteps = []
    for t in range(T, T2):
        torch.cuda.synchronize()
        ts = time.perf_counter()
        gx.copy_(bx[t])
        gi.copy_(bi[t])
        go.copy_(bo[t])
        g.launch()
        torch.cuda.synchronize()
        gsteps.append((time.perf_counter() - ts) * 1e3)
    g.close()
    assert ix.sync() == 0
    gsm = np.sort(np.array(gsteps))
    log(f"[bench] graph steps: p50 {np.percentile(gsm, 50):.3f} ms, p99 {np.percentile(gsm, 99):.3f} ms")

    # recall@10 and the nprobe sweep on the window after T2 steps (base ids >=
    # B*T2 plus the live part of batches 1..T2) against exact kNN (float64)
    nrq = min(a.recall_queries, nq)
    keep = ids >= B * T2
    parts_x, parts_i = [x[keep]], [ids[keep]]
    for t in range(1, T2 + 1):
        xb, idb = w.stream_batch(t)
        if idb[-1] >= B * T2:
            sel = idb >= B * T2
            parts_x.append(xb[sel])
            parts_i.append(idb[sel])
    xw, idw = np.concatenate(parts_x), np.concatenate(parts_i)
    assert xw.shape[0] == w.n_base
    t0 = time.time()
    gt = exact_topk(xw, idw, q[:nrq], k, w.metric)
    del xw, idw
    log(f"[bench] exact kNN of {nrq} queries in {time.time() - t0:.1f} s")

    def recall_of(labels):
        return float(np.mean([len(set(gt[i]) & set(labels[i])) / k for i in range(nrq)]))

    grid = [1, 2, 4, 8, 16, 32, 64] + ([128] if nprobe > 64 else [])
    sweep, best95 = nprobe_sweep(ix, qd, k, nq, nprobe, grid if not a.no_sweep else [nprobe], recall_of, dist, lab)
    recall = [r for r in sweep if r["nprobe"] == nprobe][0]["recall_at_10"]
    log(f"[bench] recall@{k} at nprobe {nprobe}: {recall:.4f}; sweep {sweep}")

    # latency legs: >= 1,000 steady-state steps at B, then at B = 1,000
    latency = {}
    if lat_steps:
        pool = torch.cat(bx[:16])
        nxt, old = w.n_base + B * T2, B * T2
        latency[f"B{B}"], nxt, old = latency_leg(ix, pool, qd, k, nprobe, nxt, old, w.n_base, B, lat_steps, dist, lab)
        log(f"[bench] latency at B={B}: {latency[f'B{B}']}")
        latency[f"B{B_small}"], nxt, old = latency_leg(ix, pool, qd, k, nprobe, nxt, old, w.n_base, B_small,
                                                       lat_steps, dist, lab)
        log(f"[bench] latency at B={B_small}: {latency[f'B{B_small}']}")
        del pool

    if a.copy_calibration:
        copy_calibration()

    add_ms = prof["add"][0] / max(prof["add"][1], 1)
    rm_ms = prof["remove"][0] / max(prof["remove"][1], 1)
    se_ms = prof["search"][0] / max(prof["search"][1], 1)
    sm = np.sort(np.array(step_ms))
    if st_code == 0:
        prof_name = ("k_scan_cert_window_1M.md" if tile == 16 else "k_scan_window_1M.md")
        roof = fp32_scan_roofline(evals, w.dim, scan_ms, tile,
                                  recorded_traffic(prof_name) if a.workload == "window" else None)
    else:
        # a list is read once per tile of 16 queries: rounded rows (2 B per dim), ids, and for L2 the
        # norms of the rounded rows
        per_eval = (2.0 * w.dim + 4 + (4 if w.metric == 0 else 0)) / 16
        gbps = evals * per_eval / (scan_ms * 1e-3) / 1e9
        flops = evals * 2.0 * 32 * ((w.dim + 31) // 32)   # MFMA work incl. padding to 32-dim blocks
        mfma_tf = flops / (scan_ms * 1e-3) / 1e12
        prof_name = "k_scan_mfma_precision_10M.md" if a.workload == "precision" else None
        roof = {"bound": "hbm", "kernel": "k_scan_mfma", "achieved": round(gbps, 1), "peak": HBM_PEAK_GBPS,
                "unit": "GB/s", "frac": round(gbps / HBM_PEAK_GBPS, 4),
                "traffic": recorded_traffic(prof_name) if prof_name else None,
                "traffic_unit": "bytes per launch (DRAM, rocprofv3 FETCH_SIZE + WRITE_SIZE, copy-calibrated)",
                "algorithmic_bytes_per_launch": int(evals * per_eval), "evals_per_launch": evals,
                "mfma_tflops": round(mfma_tf, 3), "mfma_frac": round(mfma_tf / MFMA16_PEAK_TFLOPS, 4),
                "avg_launch_ms": round(scan_ms, 4)}
        if gbps > HBM_PEAK_GBPS:
            # the per-tile reads exceed what HBM can deliver in the measured time (tiles of one list re-read
            # it from L2 / MALL): report the matrix-core bound, with the HBM model beside it
            hbm = {k: roof.pop(k) for k in ("bound", "achieved", "peak", "unit", "frac")}
            roof = dict({"bound": "mfma", "achieved": round(mfma_tf, 3), "peak": MFMA16_PEAK_TFLOPS,
                         "unit": "TFLOP/s", "frac": round(mfma_tf / MFMA16_PEAK_TFLOPS, 4)}, **roof,
                        hbm_model=dict(hbm, note="per-tile chunk reads exceed HBM peak: served from L2/MALL"))
    roof["probed_list_imbalance"] = round(evals / balanced, 3)
    res = {
        "metric": "insert/delete vectors/s; search QPS at recall@10>=0.95; p99 window-step ms",
        "value": round(nq * a.steps / elapsed, 1),
        "unit": f"queries/s (window step: +{B} insert, {nq}-query search, -{B} delete)",
        "n_gpus": 1, "steps": a.steps, "warmup": a.warmup,
        "ms_per_step": round(elapsed / a.steps * 1e3, 4),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": {"f32": "f32", "bf16": "bf16 scan + f32 re-rank", "f16": "f16 scan + f32 re-rank"}[storage],
        "data": "synthetic",
        "config": {"workload": f"{w.name}: sliding window N={w.n_base}, d={w.dim}, nlist={w.nlist}, slab={w.slab}, "
                               f"+{B}/-{B} per step, {nq} queries, nprobe={nprobe}, k={k}, "
                               f"{'L2' if w.metric == 0 else 'IP'}, storage={storage}"
                               + (f", re-rank top {rerank * k}" if rerank else ""),
                   "global_batch": nq, "parallelism": "single GPU"},
        "schedule": {"tile": tile, "chunk_positions": 1 << sh, "persistent_waves": bool(pers)},
        "recall_at_10": recall,
        "qps_at_recall95": best95,
        "nprobe_sweep": sweep,
        "search_qps": round(nq / (se_ms * 1e-3), 1),
        "insert_vec_per_s": round(B / (add_ms * 1e-3), 1),
        "delete_vec_per_s": round(B / (rm_ms * 1e-3), 1),
        "bulk_insert_vec_per_s": round(x.shape[0] / (bulk_ms * 1e-3), 1),
        "timed_steps_p50_ms": round(float(np.percentile(sm, 50)), 4),
        "timed_steps_max_ms": round(float(sm[-1]), 4),
        "graph_p50_step_ms": round(float(np.percentile(gsm, 50)), 4),
        "graph_p99_step_ms": round(float(np.percentile(gsm, 99)), 4),
        "device_ms": {kk: round(v[0] / max(v[1], 1), 4) for kk, v in prof.items()},
        "roofline": roof,
        "cpu_baseline": None,
    }
    if latency:
        res["latency"] = latency
        res["p50_step_ms"] = latency[f"B{B}"]["p50_ms"]
        res["p99_step_ms"] = latency[f"B{B}"]["p99_ms"]
        res["max_step_ms"] = latency[f"B{B}"]["max_ms"]
    ix.close()
    del ix
    torch.cuda.empty_cache()

    if a.workload == "window" and st_code == 0 and not a.no_forms:
        # the reduced-precision form on the same window data, queries and steps
        t0 = time.time()
        ixb, bulk_b = build_window_index(sivf, w, x, ids, STORAGE["bf16"], a.rerank, id_cap, B, nq, nprobe, dev)
        tb = ixb.tune_search(qd, k, nprobe)
        for t in range(a.warmup):
            ixb.step(bx[t], bi[t], qd, k, nprobe, bo[t], out=(dist, lab))
        assert ixb.sync() == 0
        el_b, st_b, prof_b = timed_steps(ixb, bx, bi, bo, qd, k, nprobe, dist, lab, a.warmup, T)
        for t in range(T, T2):      # same window as the FP32 index had for the sweep
            ixb.step(bx[t], bi[t], qd, k, nprobe, bo[t], out=(dist, lab))
        assert ixb.sync() == 0
        sweep_b, best95_b = nprobe_sweep(ixb, qd, k, nq, nprobe, grid, recall_of, dist, lab)
        smb = np.sort(np.array(st_b))
        res["bf16_form"] = {
            "value": round(nq * a.steps / el_b, 1), "unit": res["unit"], "steps": a.steps,
            "ms_per_step": round(el_b / a.steps * 1e3, 4), "p50_step_ms": round(float(np.percentile(smb, 50)), 4),
            "schedule": {"tile": tb[0], "chunk_positions": 1 << tb[1], "persistent_waves": bool(tb[2])},
            "recall_at_10": [r for r in sweep_b if r["nprobe"] == nprobe][0]["recall_at_10"],
            "qps_at_recall95": best95_b, "nprobe_sweep": sweep_b,
            "device_ms": {kk: round(v[0] / max(v[1], 1), 4) for kk, v in prof_b.items()},
            "rerank_top": a.rerank * k,
            "fp32_qps_at_recall95": best95,
        }
        log(f"[bench] bf16 form: {res['bf16_form']['value']} q/s, sweep {sweep_b} ({time.time() - t0:.1f} s)")
        ixb.close()
        del ixb
        torch.cuda.empty_cache()
        t0 = time.time()
        res["bulk_mutation"] = bulk_mutation_leg(w, x, ids)
        log(f"[bench] bulk mutation: {res['bulk_mutation']} ({time.time() - t0:.1f} s)")
    del bx, bi, bo

    if not a.no_cpu_baseline and a.workload != "precision":
        t0 = time.time()
        res["cpu_baseline"] = cpu_baseline(w, x, ids, q, nprobe, k,
                                           n_sample_q=200 if a.workload == "window" else nq)
        log(f"[bench] cpu baseline in {time.time() - t0:.1f} s")
    print(json.dumps(res), flush=True)


def exact_knn_device(ix, live_ids, q, k, metric, dev, cand=None):
    """Exact top-k over the live rows (fetched from the index in 2M-row
    chunks): candidates by fp32 scores on the device, the best `cand` of them
    re-scored in float64 on the host, ties by smaller id."""
    import torch
    cand = cand or max(32, 2 * k)
    nq = q.shape[0]
    q2 = (q * q).sum(1, keepdim=True)
    best_s = torch.full((nq, cand), float("inf"), device=dev)
    best_i = torch.full((nq, cand), -1, dtype=torch.int64, device=dev)
    for s0 in range(0, live_ids.shape[0], 1 << 21):
        idc = torch.from_numpy(live_ids[s0:s0 + (1 << 21)]).to(dev)
        rows = ix.get_rows(idc)
        sc = (q2 + (rows * rows).sum(1)[None, :] - 2.0 * (q @ rows.T)) if metric == 0 else -(q @ rows.T)
        s_c, o_c = torch.topk(sc, min(cand, sc.shape[1]), dim=1, largest=False)
        cs = torch.cat([best_s, s_c], 1)
        ci = torch.cat([best_i, idc[o_c]], 1)
        best_s, o = torch.topk(cs, cand, dim=1, largest=False)
        best_i = torch.gather(ci, 1, o)
        del rows, sc
    ci = best_i.cpu().numpy()
    rows = ix.get_rows(torch.from_numpy(ci.reshape(-1)).to(dev)).cpu().numpy().astype(np.float64)
    qd = q.cpu().numpy().astype(np.float64)
    rows = rows.reshape(nq, cand, -1)
    d64 = ((rows - qd[:, None, :]) ** 2).sum(2) if metric == 0 else -(rows * qd[:, None, :]).sum(2)
    return [ci[j][np.lexsort((ci[j], d64[j]))[:k]] for j in range(nq)]


def batched_main(a):
    """Batched uneven form: skewed lists, per-query nprobe and k, random
    deletes; window steps eager and as HIP graphs, after the autotuner."""
    import torch
    import paper_2601_11808_amd as sivf
    import workloads

    if not os.path.exists(sivf.LIB_PATH):
        raise SystemExit("libsivf.so is not built: run python -c 'import __graft_entry__ as g; g.build()'")
    dev = torch.device("cuda:0")
    w = workloads.batched()
    N, B, C, nq = w.n_base, w.batch, w.slab, w.n_queries
    steps, warm = a.steps, a.warmup
    T = warm + 2 * steps
    npq, kpq = workloads.per_query_params(nq)
    kmax = int(kpq.max())
    id_cap = N + B * (T + 2)
    num_slabs = int(1.1 * (N + 2 * B) / C) + 2 * w.nlist
    ix = sivf.Index(w.dim, w.nlist, w.centroids, metric=w.metric, slab_capacity=C, num_slabs=num_slabs,
                    id_capacity=id_cap, max_batch=1 << 16, max_queries=nq, max_k=kmax, max_nprobe=int(npq.max()),
                    device="cuda:0")
    log(f"[batched] N={N} d={w.dim} nlist={w.nlist} C={C}; {nq} queries, nprobe U[{npq.min()},{npq.max()}], "
        f"k in {sorted(set(kpq.tolist()))}; workspace {ix.workspace_bytes / 2**30:.1f} GiB")
    means = torch.from_numpy(w.means).to(dev)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for c, s0 in enumerate(range(0, N, 1 << 16)):
        n = min(1 << 16, N - s0)
        ix.add(workloads.device_sample(w, n, 1000 + c, dev, means), torch.arange(s0, s0 + n, device=dev))
    assert ix.sync() == 0
    load_s = time.perf_counter() - t0
    lens = ix.dump()["list_len"]
    log(f"[batched] bulk load {load_s:.1f} s; list lengths min {lens.min()} median {int(np.median(lens))} "
        f"max {lens.max()}")
    qd = workloads.device_sample(w, nq, 2, dev, means)
    kpq_d = torch.from_numpy(kpq).to(dev)
    npq_d = torch.from_numpy(npq).to(dev)
    t0 = time.perf_counter()
    if a.schedule:
        tile, sh, pers = (int(v) for v in a.schedule.split(","))
        ix.set_search_schedule(tile, sh, pers)
    else:
        tile, sh, pers = ix.tune_search(qd, kmax, int(npq.max()), k_per_query=kpq_d, nprobe_per_query=npq_d)
    log(f"[batched] schedule: {tile} queries x 2^{sh} positions per work item, persistent={pers} "
        f"({'given' if a.schedule else 'autotuned'}, {time.perf_counter() - t0:.1f} s)")
    # per step: B fresh vectors in, B uniformly random live ids out
    rng = np.random.default_rng([w.seed, 3, 1])
    live = np.arange(N, dtype=np.int64)
    bx, bi, bo = [], [], []
    for t in range(T):
        ids = np.arange(N + B * t, N + B * (t + 1), dtype=np.int64)
        idx = rng.choice(live.shape[0], B, replace=False)
        out = live[idx]
        live = np.concatenate([np.delete(live, idx), ids])
        bx.append(workloads.device_sample(w, B, 100 + t, dev, means))
        bi.append(torch.from_numpy(ids).to(dev))
        bo.append(torch.from_numpy(out).to(dev))
    dist = torch.empty((nq, kmax), dtype=torch.float32, device=dev)
    lab = torch.empty((nq, kmax), dtype=torch.int64, device=dev)
    np_max = int(npq.max())
    for t in range(warm):
        ix.step(bx[t], bi[t], qd, kmax, np_max, bo[t], out=(dist, lab), k_per_query=kpq_d, nprobe_per_query=npq_d)
    assert ix.sync() == 0
    ix.profile_read()
    ix.profile(True)
    step_ms = []
    torch.cuda.synchronize()
    t_all = time.perf_counter()
    for t in range(warm, warm + steps):
        ts = time.perf_counter()
        ix.step(bx[t], bi[t], qd, kmax, np_max, bo[t], out=(dist, lab), k_per_query=kpq_d, nprobe_per_query=npq_d)
        torch.cuda.synchronize()
        step_ms.append((time.perf_counter() - ts) * 1e3)
    elapsed = time.perf_counter() - t_all
    prof = ix.profile_read()
    ix.profile(False)
    assert ix.sync() == 0
    # graph mode on refilled buffers
    gx = torch.empty((B, w.dim), dtype=torch.float32, device=dev)
    gi = torch.empty(B, dtype=torch.int64, device=dev)
    go = torch.empty(B, dtype=torch.int64, device=dev)
    nrem = torch.zeros(1, dtype=torch.int64, device=dev)
    g = ix.step_graph(gx, gi, qd, kmax, np_max, go, dist, lab, nrem, k_per_query=kpq_d, nprobe_per_query=npq_d)
    gsteps = []
    for t in range(warm + steps, T):
        gx.copy_(bx[t])
        gi.copy_(bi[t])
        go.copy_(bo[t])
        torch.cuda.synchronize()
        ts = time.perf_counter()
        g.launch()
        torch.cuda.synchronize()
        gsteps.append((time.perf_counter() - ts) * 1e3)
    g.close()
    assert ix.sync() == 0
    st = ix.stats()
    assert st["live"] == live.shape[0], (st["live"], live.shape[0])
    # recall@10 of queries with k >= 10 (their own nprobe) on the final window
    sel = np.flatnonzero(kpq >= 10)[:500]
    qs = qd[torch.from_numpy(sel).to(dev)]
    gt = exact_knn_device(ix, live, qs, 10, w.metric, dev)
    _, lab_s = ix.search(qs, kmax, np_max, k_per_query=kpq_d[torch.from_numpy(sel).to(dev)],
                         nprobe_per_query=npq_d[torch.from_numpy(sel).to(dev)])
    lab_s = lab_s.cpu().numpy()
    rec = float(np.mean([len(set(gt[j]) & set(lab_s[j][:10])) / 10 for j in range(sel.shape[0])]))
    # scan roofline: distance evaluations = sum over (query, probe) of the probed list's length
    probes = ix.probe(qd, np_max).cpu().numpy()
    probes = np.where(np.arange(np_max)[None, :] < npq[:, None], probes, -1)
    lens = ix.dump()["list_len"].astype(np.int64)
    ev_q = np.where(probes >= 0, lens[np.maximum(probes, 0)], 0).sum(axis=1)   # evaluations per query
    evals = int(ev_q.sum())
    scan_ms = prof["scan"][0] / max(prof["scan"][1], 1)
    deep_ms = prof["scan_deep"][0] / max(prof["scan_deep"][1], 1)
    deep_sched = ix.search_schedule()[1]
    if prof["scan_deep"][1] > 0:
        # two passes: k <= 64 on the certified scan, k > 64 on the deep schedule
        ev_s, ev_d = int(ev_q[kpq <= 64].sum()), int(ev_q[kpq > 64].sum())
        passes = [dict(fp32_scan_roofline(ev_s, w.dim, scan_ms, tile), queries="k <= 64"),
                  dict(fp32_scan_roofline(ev_d, w.dim, deep_ms, deep_sched[0]), queries="k > 64")]
        roof = dict(passes[0] if scan_ms >= deep_ms else passes[1])
        roof["passes"] = passes
    else:
        roof = fp32_scan_roofline(evals, w.dim, scan_ms, tile)
    sm, gsm = np.sort(np.array(step_ms)), np.sort(np.array(gsteps))
    se_ms = prof["search"][0] / max(prof["search"][1], 1)
    res = {
        "metric": "batched uneven form: queries/s of window steps (per-query nprobe and k), p50/p99 step ms",
        "value": round(nq * steps / elapsed, 1), "unit": f"queries/s (window step: +{B} insert, {nq}-query "
                                                         f"search, -{B} random delete)",
        "n_gpus": 1, "steps": steps, "warmup": warm, "ms_per_step": round(elapsed / steps * 1e3, 4),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": f"batched: N={N}, d={w.dim}, Zipf(1.1) over {w.nlist} clusters, nlist={w.nlist}, "
                               f"slab={C}, {nq} queries, nprobe U[8,128], k in {{1,10,100}}, +{B}/-{B} random",
                   "parallelism": "single GPU"},
        "schedule": {"tile": tile, "chunk_positions": 1 << sh, "persistent_waves": bool(pers),
                     "deep_pass": {"tile": deep_sched[0], "chunk_positions": 1 << deep_sched[1],
                                   "persistent_waves": bool(deep_sched[2])}},
        "recall_at_10_k_ge_10": round(rec, 4),
        "search_qps": round(nq / (se_ms * 1e-3), 1),
        "p50_step_ms": round(float(np.percentile(sm, 50)), 3), "p99_step_ms": round(float(np.percentile(sm, 99)), 3),
        "graph_p50_step_ms": round(float(np.percentile(gsm, 50)), 3),
        "graph_p99_step_ms": round(float(np.percentile(gsm, 99)), 3),
        "device_ms": {kk: round(v[0] / max(v[1], 1), 4) for kk, v in prof.items()},
        "list_len": {"min": int(lens.min()), "median": int(np.median(lens)), "max": int(lens.max())},
        "roofline": roof,
        "bulk_load_vec_per_s": round(N / load_s, 1),
    }
    print(json.dumps(res), flush=True)


# PCIe 5.0 x16, one direction: the host link of an MI355X
HOST_LINK_GBPS = 64.0


def tier_main(a):
    """Host tier on the window data: the odd lists move to pinned host memory.
    Reports the offload rate and the window search with those lists scanned in
    host memory, beside the same search with every list on the device (the
    results must be identical)."""
    import torch
    import paper_2601_11808_amd as sivf
    import workloads

    if not os.path.exists(sivf.LIB_PATH):
        raise SystemExit("libsivf.so is not built: run python -c 'import __graft_entry__ as g; g.build()'")
    dev = torch.device("cuda:0")
    w = workloads.window()
    x, ids = w.base()
    q = w.queries()
    N, d = x.shape
    nq, k, nprobe = q.shape[0], w.k, w.nprobe
    num_slabs = int(1.15 * N / w.slab) + w.nlist
    ix = sivf.Index(d, w.nlist, w.centroids, metric=w.metric, slab_capacity=w.slab, num_slabs=num_slabs,
                    id_capacity=N, max_batch=65536, max_queries=nq, max_k=16, max_nprobe=nprobe,
                    delete_mode=sivf.DELETE_LAZY, device="cuda:0")
    xd, idd = torch.from_numpy(x).to(dev), torch.from_numpy(ids).to(dev)
    for c in range(0, N, 65536):
        ix.add(xd[c:c + 65536], idd[c:c + 65536])
    assert ix.sync() == 0
    ix.tier_attach(num_slabs)
    qd = torch.from_numpy(q).to(dev)
    sched = tuple(int(v) for v in a.schedule.split(",")) if a.schedule else (16, 16, 0)
    ix.set_search_schedule(*sched)
    reps = max(3, a.steps)

    def timed_search():
        for _ in range(a.warmup):
            ix.search(qd, k, nprobe)
        assert ix.sync() == 0
        ix.profile_read()
        ix.profile(True)
        for _ in range(reps):
            dist, lab = ix.search(qd, k, nprobe)
        prof = ix.profile_read()
        ix.profile(False)
        assert ix.sync() == 0
        return {kk: v[0] / max(v[1], 1) for kk, v in prof.items() if v[1] > 0}, dist, lab

    hot, d_hot, l_hot = timed_search()
    odd = np.arange(1, w.nlist, 2, dtype=np.int32)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    moved = ix.tier_offload(odd)
    off_s = time.perf_counter() - t0
    ts = ix.tier_stats()
    cold, d_cold, l_cold = timed_search()
    same = bool(torch.equal(l_hot, l_cold) and torch.equal(d_hot.view(torch.int32), d_cold.view(torch.int32)))
    # link bytes of the cold scan: every probed cold segment crosses the host link at least once per
    # search (rows and ids); re-reads by further query tiles are served from the GPU's caches
    probes = ix.probe(qd, nprobe).cpu().numpy()
    clen = ix.tier_dump()["cold_len"].astype(np.int64)
    cold_evals = int(clen[probes[probes >= 0]].sum())
    probed = np.zeros(w.nlist, bool)
    probed[probes[probes >= 0]] = True
    link_bytes = float(clen[probed].sum()) * (4.0 * d + 4.0)
    scan_cold_ms = cold.get("scan_cold", 0.0)
    res = {
        "metric": "host tier: window search with half the lists in host memory; offload rate",
        "value": round(nq / (cold["search"] * 1e-3), 1), "unit": "queries/s (half the lists cold)",
        "n_gpus": 1, "steps": reps, "warmup": a.warmup, "ms_per_step": round(cold["search"], 4),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": f"tier: window data N={N}, d={d}, nlist={w.nlist}, slab={w.slab}, lazy deletes; "
                               f"the {odd.shape[0]} odd lists offloaded; {nq} queries, nprobe {nprobe}, k {k}",
                   "parallelism": "single GPU"},
        "identical_results": same,
        "offload": {"positions": moved, "seconds": round(off_s, 4), "positions_per_s": round(moved / off_s, 1),
                    "link_GBps": round(moved * (4.0 * d + 4.0) / off_s / 1e9, 2)},
        "tier_stats": ts,
        "search_all_device_ms": {kk: round(v, 4) for kk, v in hot.items()},
        "search_half_cold_ms": {kk: round(v, 4) for kk, v in cold.items()},
        "cold_scan": {"bound": "host link", "evals_per_launch": cold_evals, "link_bytes": int(link_bytes),
                      "achieved": round(link_bytes / (scan_cold_ms * 1e-3) / 1e9, 2) if scan_cold_ms else None,
                      "peak": HOST_LINK_GBPS, "unit": "GB/s",
                      "frac": round(link_bytes / (scan_cold_ms * 1e-3) / 1e9 / HOST_LINK_GBPS, 4) if scan_cold_ms
                      else None,
                      "note": "each probed cold segment's rows and ids cross the link once per search"},
    }
    print(json.dumps(res), flush=True)


def mutation_main(a):
    """Mutation kernels at bulk scale on the window data (the bulk-mutation leg
    of the default run on its own, for kernel traces and counters)."""
    import paper_2601_11808_amd as sivf
    import workloads

    if not os.path.exists(sivf.LIB_PATH):
        raise SystemExit("libsivf.so is not built: run python -c 'import __graft_entry__ as g; g.build()'")
    w = workloads.window()
    x, ids = w.base()
    N, d = x.shape
    reps = max(1, a.steps // 10)
    m = bulk_mutation_leg(w, x, ids, reps=reps)
    if a.copy_calibration:
        copy_calibration()
    res = {
        "metric": "insert/delete vectors/s at bulk scale (whole-window insert, half-window delete)",
        "value": m["insert"]["vec_per_s"], "unit": "inserted vectors/s",
        "n_gpus": 1, "steps": reps, "warmup": 1, "ms_per_step": round(m["insert"]["ms"] + m["delete"]["ms"], 4),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": f"mutation: window data N={N}, d={d}, nlist={w.nlist}, slab={w.slab}; insert {N} "
                               f"in one call, delete {N // 2} random ids in one call", "parallelism": "single GPU"},
        **m,
    }
    print(json.dumps(res), flush=True)


def serve_main(a):
    """Serving form: the steady-state window under an open-loop Poisson
    request stream, every request submitted through the overlapping server
    at its arrival time.  Latency = completion seen by the host - arrival."""
    import torch
    import paper_2601_11808_amd as sivf
    import workloads

    if not os.path.exists(sivf.LIB_PATH):
        raise SystemExit("libsivf.so is not built: run python -c 'import __graft_entry__ as g; g.build()'")
    dev = torch.device("cuda:0")
    w = workloads.serving(n_base=a.serve_n)
    N, C, k = w.n_base, w.slab, w.k
    t0 = time.time()
    reqs = workloads.serving_requests(a.serve_seconds, rate=a.serve_rate)
    dels, live_end = workloads.serving_delete_ids(reqs, N)
    n_ins = sum(r.n for r in reqs if r.kind == "insert")
    id_cap = N + n_ins
    log(f"[serve] {len(reqs)} requests over {a.serve_seconds} s at {a.serve_rate} req/s "
        f"(+{n_ins} / -{sum(v.shape[0] for v in dels.values())} vectors) prepared in {time.time() - t0:.1f} s")
    num_slabs = int(1.3 * max(N, int(np.count_nonzero(live_end))) / C) + 2 * w.nlist
    ix = sivf.Index(w.dim, w.nlist, w.centroids, metric=w.metric, slab_capacity=C, num_slabs=num_slabs,
                    id_capacity=id_cap, max_batch=100_000, max_queries=4096, max_k=16, max_nprobe=64,
                    storage=STORAGE["f16"], rerank_factor=4, device="cuda:0")
    log(f"[serve] workspace {ix.workspace_bytes / 2**30:.1f} GiB, {num_slabs} slabs")
    means = torch.from_numpy(w.means).to(dev)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    chunk = 100_000
    for c, s0 in enumerate(range(0, N, chunk)):
        n = min(chunk, N - s0)
        xb = workloads.device_sample(w, n, 1000 + c, dev, means)
        ix.add(xb, torch.arange(s0, s0 + n, device=dev))
        if c % 50 == 49:
            assert ix.sync() == 0
            log(f"[serve] loaded {s0 + n} vectors")
    assert ix.sync() == 0
    load_s = time.perf_counter() - t0
    log(f"[serve] bulk load {N} vectors in {load_s:.1f} s ({N / load_s / 1e6:.2f} M vec/s)")
    # payloads resident before the stream starts
    pool = workloads.device_sample(w, 2_000_000, 1, dev, means)
    qpool = workloads.device_sample(w, 65536, 2, dev, means)
    ins_ids = torch.arange(N, id_cap, device=dev)
    del_all = torch.from_numpy(np.concatenate([dels[i] for i in sorted(dels)]) if dels else
                               np.zeros(0, np.int64)).to(dev)
    rng = np.random.default_rng([w.seed, 6, 0])
    plan, ioff, doff = [], 0, 0
    for i, r in enumerate(reqs):
        if r.kind == "insert":
            o = int(rng.integers(0, pool.shape[0] - r.n + 1))
            plan.append((pool[o:o + r.n], ins_ids[ioff:ioff + r.n]))
            ioff += r.n
        elif r.kind == "delete":
            m = dels[i].shape[0]
            plan.append((del_all[doff:doff + m],))
            doff += m
        else:
            o = int(rng.integers(0, qpool.shape[0] - r.n + 1))
            plan.append((qpool[o:o + r.n],))
    torch.cuda.synchronize()

    ix.profile_read()
    ix.profile(True)
    srv = sivf.Server(ix)
    queues = {"search": [], "mut": []}      # (request index, ticket) in submission order
    heads = {"search": 0, "mut": 0}
    done_t = np.zeros(len(reqs))
    sub_t = np.zeros(len(reqs))
    refused, refused_at = 0, -1
    refused_s, refused_s_at = 0, -1
    i = 0
    start = time.perf_counter() + 0.05
    while True:
        now = time.perf_counter() - start
        if i < len(reqs) and reqs[i].t <= now:
            r, pl = reqs[i], plan[i]
            if r.kind == "insert":
                t = srv.add(pl[0], pl[1])
                if t is None:           # not admitted yet: retry once something completes
                    if refused_at != i:
                        refused += 1
                        refused_at = i
                else:
                    queues["mut"].append((i, t))
            elif r.kind == "delete":
                t, _ = srv.remove(pl[0])
                queues["mut"].append((i, t))
            else:
                t, _, _ = srv.search(pl[0], k, r.nprobe)
                if t is None:           # search slots full: retry once something completes
                    if refused_s_at != i:
                        refused_s += 1
                        refused_s_at = i
                else:
                    queues["search"].append((i, t))
            if t is not None:
                sub_t[i] = time.perf_counter() - start
                i += 1
                continue
        for kq in ("search", "mut"):
            qq = queues[kq]
            while heads[kq] < len(qq) and srv.poll(qq[heads[kq]][1]):
                done_t[qq[heads[kq]][0]] = time.perf_counter() - start
                heads[kq] += 1
        if i == len(reqs) and all(heads[kq] == len(queues[kq]) for kq in queues):
            break
    end = time.perf_counter() - start
    nb_launch, nb_req = srv.batches()
    srv.close()
    assert ix.sync() == 0
    prof = ix.profile_read()
    ix.profile(False)
    st = ix.stats()
    log(f"[serve] stream done in {end:.2f} s; live {st['live']} (expected {int(np.count_nonzero(live_end))})")
    assert st["live"] == int(np.count_nonzero(live_end))
    assert st["used_slabs"] + st["free_slabs"] == num_slabs

    arr = np.array([r.t for r in reqs])
    lat = (done_t - arr) * 1e3
    per = {}
    for kind in ("search", "insert", "delete"):
        sel = np.array([r.kind == kind for r in reqs])
        if sel.any():
            v = np.sort(lat[sel])
            per[kind] = {"count": int(sel.sum()), "p50_ms": round(float(np.percentile(v, 50)), 3),
                         "p99_ms": round(float(np.percentile(v, 99)), 3), "max_ms": round(float(v[-1]), 3),
                         "mean_size": round(float(np.mean([r.n for r in reqs if r.kind == kind])), 1)}
    last_arrival = float(arr[-1]) if len(reqs) else 0.0
    # recall@10 on the final window for 256 pooled queries
    nrq = 256
    qh = qpool[:nrq]
    gt = exact_knn_device(ix, np.flatnonzero(live_end).astype(np.int64), qh, k, w.metric, dev)
    recall = {}
    for npb in (16, 32, 64):
        _, lab = ix.search(qh, k, npb)
        lab = lab.cpu().numpy()
        recall[str(npb)] = round(float(np.mean([len(set(gt[j]) & set(lab[j])) / k for j in range(nrq)])), 4)
    log(f"[serve] recall@10 on the final window: {recall}")
    nq_tot = sum(r.n for r in reqs if r.kind == "search")
    n_del = int(sum(v.shape[0] for v in dels.values()))
    res = {
        "metric": "serving: completed requests/s with p50/p99 latency per request type",
        "value": round(len(reqs) / end, 1), "unit": "requests/s",
        "n_gpus": 1, "steps": len(reqs), "warmup": 0, "ms_per_step": round(end / max(len(reqs), 1) * 1e3, 4),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f16 scan + f32 re-rank", "data": "synthetic",
        "config": {"workload": f"serving: steady window N={N}, d={w.dim}, nlist={w.nlist}, slab={C}, fp16 storage, "
                               f"Poisson {a.serve_rate} req/s for {a.serve_seconds} s, mix search 1/2 "
                               f"(1-4096 queries, nprobe 16-64, k=10), insert 1/3 (1k-50k), delete 1/6 (1k-100k)",
                   "parallelism": "single GPU"},
        "offered_req_per_s": round(len(reqs) / max(last_arrival, 1e-9), 1),
        "drain_s_after_last_arrival": round(end - last_arrival, 3),
        "latency": per,
        "insert_vec_per_s": round(n_ins / end, 1), "delete_ids_per_s": round(n_del / end, 1),
        "search_queries_per_s": round(nq_tot / end, 1),
        "inserts_refused_then_retried": refused,
        "searches_refused_then_retried": refused_s,
        "search_batches": {"launches": nb_launch, "requests": nb_req},
        # device time per request class (HIP events on the server's streams; searches and inserts overlap,
        # so the sums can exceed the wall time)
        "device_ms_mean": {kk: round(v[0] / max(v[1], 1), 3) for kk, v in prof.items()},
        "device_ms_total": {kk: round(v[0], 1) for kk, v in prof.items()},
        "recall_at_10_final_window": recall,
        "bulk_load_vec_per_s": round(N / load_s, 1),
    }
    print(json.dumps(res), flush=True)


if __name__ == "__main__":
    main()
