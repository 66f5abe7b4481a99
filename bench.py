"""Benchmark: exact k-clique counting on the R-MAT scale-18 workload, one MI355X.

One step = the whole hot path over the resident input: ebbkc_prepare on the CSR already in HBM
(validation, supports, truss-based edge ordering, rank-tagged adjacency) followed by ebbkc_count
for every k of the workload (5, 6, 7, 8, 9; the first count also builds the sub-branch arena).
value = k-cliques counted per second = (sum over k of N_k) / step time.

Wall budget.  The run is bounded by --budget-s seconds from process start (default 450).  --warmup
and --steps are upper bounds: warmup steps beyond the first run only while the timed steps still
fit, and a timed step starts only while it is expected to end before the measurement deadline
(--core-s, default 300 s from process start; at least one timed step always runs).  "steps" and
"warmup" on the JSON line are the numbers actually run, "steps_requested" / "warmup_requested" the
numbers asked for.  Every leg after the measurement runs only if its estimated time fits what is
left of the budget; a leg left out is reported as {"skipped": reason}.

Also reported on the same JSON line:
  roofline      the dominant branch-kernel launch (the bitmap width class launch with the largest
                device time in the timed steps): its algorithmic 64-bit word operations (AND +
                popcount of one candidate-bitmap word; counted by the library's per-launch work
                counters, on in the timed run: they cost under 1 %) divided by its device time
                (HIP events on the launch stream).  Bound: VALU ("alu"); peak derived from
                256 CUs x 64 int32 lanes/clock x 2.4 GHz = 39.3 T lane-ops/s, four lane-ops per
                word-op (two 32-bit ANDs, two 32-bit popcounts) -> 9.83 T word-ops/s.
                traffic: HBM bytes per launch from rocprofv3 FETCH_SIZE + WRITE_SIZE (KiB, scaled
                by the same counters on a copy kernel of known size) when the committed record
                (profiles/search_rmat18_k9_traffic.json) was taken on the current kernel source,
                else null.
  cpu_baseline  the CPU oracle (degeneracy-ordered vertex branch and bound) timed on the host
                cores on a bounded sample of the same workload (the full k = 5 and k = 6 counts),
                with the GPU's time on the same sample (from the timed steps) beside it.
  listing       every 5-clique of the workload (5.5e10 tuples, 1.1 TB) listed rank-range chunk by
                chunk into one 80 GB device buffer: tuples/s and GB/s written (HBM-write bound).
  batched       many small graphs with per-graph k: one launch per (graph, k) vs the fused
                batch (one persistent launch per width class, replayed from a HIP graph).
  served        Poisson request streams over a mixed resident catalogue against the native
                continuous-batching server: p50/p99 latency from arrival to result, k-cliques per
                second, every result equal to the same request run alone.
  ablation      (--ablation) the same engine under the paper's variants: orderings C, T and the
                edge- and node-parallel VBBkC roots, Rule (2) off, early termination off, t = 1 / 3.

Counter modes (not part of the default run):
  --traffic-run               a 1 GiB device copy (counter calibration), then the workload's k = 9
                              count after the k = 4 count that builds the arena; run it under
                              rocprofv3 --pmc FETCH_SIZE, and again under --pmc WRITE_SIZE.
  --traffic-record F W OUT    reads those two runs' counter CSVs (directories F and W) and writes
                              the per-launch HBM bytes of the search kernels to OUT, with the hash
                              of the kernel sources they belong to.
"""
from __future__ import annotations

import time

T_START = time.time()  # the wall budget counts from here, before the heavy imports

import argparse  # noqa: E402
import csv  # noqa: E402
import glob  # noqa: E402
import hashlib  # noqa: E402
import json  # noqa: E402
import os  # noqa: E402
import re  # noqa: E402
import sys  # noqa: E402

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "k-cliques counted/sec (R-MAT s18, k=5..9) vs plain kernel; p50/p99 request latency"
PEAK_WORD_OPS = 256 * 64 * 2.4e9 / 4 / 1e12  # T word-ops/s
TRAFFIC_RECORD = os.path.join(ROOT, "profiles", "search_rmat18_k9_traffic.json")
CSRC = os.path.join(ROOT, "paper_2311_13798_amd", "csrc")
COPY_BYTES = 1 << 30


def log(msg):
    print(f"[bench {time.time() - T_START:7.1f}s] {msg}", file=sys.stderr, flush=True)


def left(budget_s):
    return T_START + budget_s - time.time()


# ---------------------------------------------------------------- HBM traffic record

def code_of(text: str) -> str:
    """C++ source without comments and blank space: what the compiler sees of it."""
    text = re.sub(r"/\*.*?\*/", " ", text, flags=re.S)
    text = re.sub(r"//[^\n]*", " ", text)
    return " ".join(text.split())


def source_sha256(read=None) -> str:
    """Hash of the search kernel's code, comments left out (the traffic record is valid only for
    this code).  read(name) gives a file's text (default: the file under csrc/)."""
    if read is None:
        def read(name):
            with open(os.path.join(CSRC, name), encoding="utf-8") as fh:
                return fh.read()
    h = hashlib.sha256()
    for f in ("search.hip", "search_kernel.h", "binom.h", "build.h", "arena.h", "device_util.h", "common.h"):
        h.update(code_of(read(f) or "").encode())
    return h.hexdigest()


def traffic_for(kernel: str, k: int):
    """HBM bytes per launch of the given kernel at k, from the committed counter record, if it
    was taken on the current kernel source."""
    if not os.path.exists(TRAFFIC_RECORD):
        return None
    rec = json.load(open(TRAFFIC_RECORD))
    if rec.get("source_sha256") != source_sha256():
        return None
    e = rec.get("launches", {}).get(f"{kernel}@k={k}")
    return None if e is None else e.get("hbm_bytes")


def traffic_run(k: int = 9):
    import torch

    import paper_2311_13798_amd as ebb
    from graphgen import configs

    torch.cuda.set_device(0)
    n = COPY_BYTES // 4  # float32 elements
    src = torch.ones(n, dtype=torch.float32, device="cuda")
    dst = torch.empty_like(src)
    torch.mul(src, 2.0, out=dst)
    torch.cuda.synchronize()
    print("copy done", flush=True)
    g = configs.rmat18()
    G = ebb.Graph.from_csr(g)
    G.count(4)
    print(f"k={k} count={G.count(k)} classes_ms={G.last_timing()}", flush=True)
    G.close()


def _per_dispatch(run_dir: str, counter: str):
    """(kernel name, dispatch id) -> counter value summed over the CSV rows of that dispatch."""
    files = glob.glob(os.path.join(run_dir, "**", "*counter_collection.csv"), recursive=True)
    if not files:
        raise FileNotFoundError(f"no counter_collection.csv under {run_dir}")
    out = {}
    for f in files:
        with open(f, newline="") as fh:
            for row in csv.DictReader(fh):
                if row.get("Counter_Name") != counter:
                    continue
                key = (row["Kernel_Name"], int(row.get("Dispatch_Id", 0)))
                out[key] = out.get(key, 0.0) + float(row["Counter_Value"])
    return out


def traffic_record(fetch_dir: str, write_dir: str, out_json: str, k: int = 9, command: str = ""):
    fetch = _per_dispatch(fetch_dir, "FETCH_SIZE")
    write = _per_dispatch(write_dir, "WRITE_SIZE")

    def copy_kib(d):
        vals = [v for (name, _), v in d.items() if "elementwise" in name and "MulFunctor" in name]
        if not vals:
            raise ValueError("the copy kernel was not profiled")
        return max(vals)

    ff = COPY_BYTES / (copy_kib(fetch) * 1024.0)
    wf = COPY_BYTES / (copy_kib(write) * 1024.0)
    launches = {}
    for (name, _), fk in sorted(fetch.items(), key=lambda kv: kv[0][1]):
        mm = re.search(r"k_search<(\d), false(?:, true)?>", name)
        if not mm:
            continue
        wk = next((v for (n2, _), v in write.items() if n2 == name), None)
        if wk is None:
            continue
        key = f"ebb::k_search<{mm.group(1)}, false>@k={k}"
        launches[key] = {"fetch_KiB": fk, "write_KiB": wk,
                         "hbm_bytes": int(round(fk * 1024.0 * ff + wk * 1024.0 * wf))}
    rec = {"source_sha256": source_sha256(), "command": command,
           "copy_kernel": {"bytes_read": COPY_BYTES, "bytes_written": COPY_BYTES,
                           "fetch_KiB": copy_kib(fetch), "write_KiB": copy_kib(write),
                           "fetch_scale": ff, "write_scale": wf},
           "launches": launches}
    with open(out_json, "w") as fh:
        json.dump(rec, fh, indent=1)
    return rec


# ---------------------------------------------------------------- legs after the measurement

def full_listing(ebb, torch, rp, ci, g, k=5, cap=4_000_000_000):
    """Every k-clique of the workload listed into one reused device buffer of cap tuples (80 GB at
    k = 5), rank-range chunk by chunk: HBM-write bound, 4 k bytes per tuple."""
    from paper_2311_13798_amd.listing import list_in_chunks, plan_chunks
    G = ebb.Graph(rp, ci, g.n)
    G.count(4)  # sub-branch arena
    cuts, sizes = plan_chunks(G, k, cap)
    buf = torch.empty((cap, k), dtype=torch.int32, device="cuda")
    list_in_chunks(G, k, buf, cap, 0, cuts=cuts[:2])  # warm: first chunk
    torch.cuda.synchronize()
    t = time.perf_counter()
    total, hu, nch = list_in_chunks(G, k, buf, cap, 0, cuts=cuts)
    torch.cuda.synchronize()
    dt = time.perf_counter() - t
    G.close()
    del buf
    gbs = total * 4 * k / dt / 1e9
    log(f"listing k={k}: {total} tuples in {nch} chunks, {dt:.3f}s, {gbs:.1f} GB/s written")
    return {"k": k, "tuples": total, "chunks": nch, "buffer_tuples": cap, "seconds": round(dt, 4),
            "tuples_per_s": total / dt, "write_GB_per_s": round(gbs, 2), "bound": "hbm",
            "write_frac_of_8TBps": round(gbs / 8000.0, 5), "unordered_checksum": str(hu),
            "order": "unsorted (tuples ascending inside, buffer order by seed rank)"}


def batched_leg(ebb, torch, configs, ngraphs=512, scale=0.1):
    """One launch per (graph, k) against the fused batch on graphs of the batched workload with n
    scaled by `scale`: k-cliques/s of each, unprofiled, at identical counts."""
    params = configs.batch_params(4096)[:ngraphs]
    gs, ks = [], []
    for p in params:
        q = dict(p)
        q["n"] = max(50, int(p["n"] * scale))
        q["clique"] = min(p["clique"], q["n"])
        gs.append(configs.batch_graph(q))
        ks.append(int(p["k"]))
    Gs = [ebb.Graph.from_csr(g) for g in gs]
    torch.cuda.synchronize()
    [G.count(k) for G, k in zip(Gs, ks)]  # also builds every arena
    t = time.perf_counter()
    plain = [G.count(k) for G, k in zip(Gs, ks)]
    t_plain = time.perf_counter() - t
    B = ebb.Batch(Gs, ks)
    B.run(use_graph=True)
    t = time.perf_counter()
    got = B.run(use_graph=True)
    t_batch = time.perf_counter() - t
    B.close()
    tot = sum(plain)
    out = {"graphs": len(Gs),
           "workload": f"{ngraphs} graphs of the batched workload with n scaled by {scale} "
                       "(p U[0.005,0.2], 20% with a planted 20..40-clique, k U{3..10})",
           "kcliques": tot, "plain_s": round(t_plain, 5), "batched_s": round(t_batch, 5),
           "plain_kcliques_per_s": tot / t_plain, "batched_kcliques_per_s": tot / t_batch,
           "vs_plain": round(t_plain / t_batch, 3), "identical": got == plain}
    log(f"batched: plain {t_plain:.3f}s fused {t_batch:.3f}s identical={got == plain}")
    return out, Gs


def batch_full(ebb, torch, configs, count=4096, threads=16):
    """The batched workload at its stated size (4,096 graphs, n U{50..5000}): one launch per graph (the
    plain kernel: ebbkc_count on each prepared graph, whose first count builds its sub-branch arena;
    graphs are prepared, counted and released one at a time) against the fused batch of all graphs
    resident at once (tasks build their sub-branches in LDS, since the arenas would need about
    700 GB), both timed around the counting only, with every count checked against the oracle's
    stored value when tests/golden/batch4096.json is present."""
    import concurrent.futures as cf
    params = configs.batch_params(4096)[:count]
    gold_path = os.path.join(ROOT, "tests", "golden", "batch4096.json")
    gold = {}
    if os.path.exists(gold_path):
        gold = {r["index"]: int(r["count"]) for r in json.load(open(gold_path))["graphs"]}

    def graphs(part):
        with cf.ThreadPoolExecutor(max_workers=threads) as ex:
            return list(ex.map(configs.batch_graph, part))

    t_plain, plain, t_prep = 0.0, [], 0.0
    for i0 in range(0, len(params), 256):
        part = params[i0:i0 + 256]
        for p, g in zip(part, graphs(part)):
            t = time.perf_counter()
            G = ebb.Graph.from_csr(g)
            torch.cuda.synchronize()
            t_prep += time.perf_counter() - t
            t = time.perf_counter()
            plain.append(G.count(int(p["k"])))
            t_plain += time.perf_counter() - t
            G.close()
        log(f"batch-full plain {len(plain)} graphs: {t_plain:.1f} s counting, {t_prep:.1f} s preparing")
    Gs, ks = [], []
    for i0 in range(0, len(params), 256):
        part = params[i0:i0 + 256]
        for p, g in zip(part, graphs(part)):
            Gs.append(ebb.Graph.from_csr(g))
            ks.append(int(p["k"]))
    torch.cuda.synchronize()
    o = ebb.ebbkc_default_options()
    o.batch_build = ebb.BATCH_BUILD
    t = time.perf_counter()
    B = ebb.Batch(Gs, ks, options=o)
    t_create = time.perf_counter() - t
    B.run(use_graph=True)  # capture
    t = time.perf_counter()
    got = B.run(use_graph=True)
    t_batch = time.perf_counter() - t
    tasks = B.info()[0]
    B.close()
    m_total = sum(int(G.info.m) for G in Gs)
    for G in Gs:
        G.close()
    tot = sum(plain)
    want = [gold.get(p["index"]) for p in params]
    out = {"graphs": len(params), "edges": m_total, "tasks": tasks,
           "workload": "the batched workload at its stated size: graph i from seed splitmix64(1 ^ i), n U{50..5000}, "
                       "p U[0.005,0.2], 20% with one planted clique of U{20..40}, k U{3..10}",
           "kcliques": tot, "plain_s": round(t_plain, 4), "batched_s": round(t_batch, 4),
           "batch_create_s": round(t_create, 4), "prepare_s": round(t_prep, 4),
           "plain_kcliques_per_s": tot / t_plain, "batched_kcliques_per_s": tot / t_batch,
           "vs_plain": round(t_plain / t_batch, 3), "identical": got == plain,
           "equal_to_oracle": (got == want) if all(w is not None for w in want) else None}
    log(f"batch-full: plain {t_plain:.1f}s fused {t_batch:.1f}s identical={got == plain} oracle={out['equal_to_oracle']}")
    return out


def served_full(ebb, torch, configs, rates=(50, 100, 200, 500, 1000, 2000), count=500, cap_s=1.0,
                budget=1 << 36):
    """The served workload at its stated shape: a resident catalogue of R-MAT s12..s18, Chung-Lu
    n = 1e4, 3e4, 1e5, 3e5, 1e6 (200 n / 1e6 planted cliques, at least 2), ER(2000, 0.01) and the first
    64 graphs of the batched workload at full size; requests (graph, k) uniform over the pairs with
    3 <= k <= 12 whose standalone count takes at most cap_s (k grows per graph until a count exceeds
    it); Poisson arrivals at each rate, `count` requests each.  Every result is compared with its
    standalone count, and the standalone counts with every stored oracle value there is."""
    import concurrent.futures as cf
    from paper_2311_13798_amd.serve import Server, poisson_requests, summarize
    named = [(f"rmat{s}", lambda s=s: configs.rmat_scale(s)) for s in range(12, 19)]
    named += [(f"cl{n:g}", lambda n=n: configs.cl_planted(n)) for n in (10000, 30000, 100000, 300000, 1000000)]
    named += [("er2000", configs.er_small)]
    params = configs.batch_params(4096)[:64]
    with cf.ThreadPoolExecutor(max_workers=16) as ex:
        c4 = list(ex.map(configs.batch_graph, params))
    graphs = [(n, mk()) for n, mk in named] + [(f"batch{p['index']}", g) for p, g in zip(params, c4)]
    gold = {}  # (graph name, k) -> oracle count
    gdir = os.path.join(ROOT, "tests", "golden")

    def load(name):
        path = os.path.join(gdir, name)
        return json.load(open(path)) if os.path.exists(path) else None
    r18, cl, er, sv, b4 = (load(f) for f in ("rmat18.json", "cl1m.json", "er_small.json", "served.json", "batch4096.json"))
    for rec, name in ((r18, "rmat18"), (cl, "cl1e+06"), (er, "er2000")):
        if rec:
            for k, v in rec["counts"].items():
                gold[(name, int(k))] = int(v)
    k8 = load("rmat18_k8.json")
    if k8:
        gold[("rmat18", 8)] = int(k8["count"])
    if sv:
        for k, v in sv["graphs"]["rmat13"]["counts"].items():
            gold[("rmat13", int(k))] = int(v)
    if b4:
        for r in b4["graphs"][:64]:
            gold[(f"batch{r['index']}", int(r["k"]))] = int(r["count"])
    Gs = [ebb.Graph.from_csr(g) for _, g in graphs]
    names = [n for n, _ in graphs]
    alone, secs, pairs = {}, {}, []
    for i, G in enumerate(Gs):
        for k in range(3, 13):
            t = time.perf_counter()
            v = G.count(k)
            dt = time.perf_counter() - t
            if dt > cap_s:
                secs[f"{names[i]}@{k}"] = round(dt, 3)
                break
            alone[(i, k)] = v
            pairs.append((i, k))
        log(f"served-full catalogue {names[i]}: k <= {max(k for j, k in pairs if j == i)}")
    checked = [(names[i], k) for i, k in pairs if (names[i], k) in gold]
    oracle_ok = all(alone[(names.index(n), k)] == gold[(n, k)] for n, k in checked)
    out = {"catalogue": names, "k": "3..12, per graph up to the last k whose standalone count takes at most "
                                    f"{cap_s} s", "pairs": len(pairs), "budget_bytes": budget,
           "excluded_first_pair_seconds": secs, "pairs_checked_against_oracle": len(checked),
           "standalone_equal_to_oracle": oracle_ok, "rates": {}}
    rng_pairs = pairs
    for rate in rates:
        S = Server(Gs, budget)
        reqs = poisson_requests(rate=float(rate), count=count, n_graphs=len(rng_pairs), k_lo=3, k_hi=3, seed=rate)
        reqs = [(off, rng_pairs[j][0], rng_pairs[j][1]) for off, j, _ in reqs]
        res = S.run_stream(reqs)
        st = S.stats()
        S.close()
        sm = summarize(res)
        same = all(r["status"] == 0 and r["count"] == alone[(g, k)] for (o, g, k), r in zip(reqs, res))
        out["rates"][str(rate)] = {"requests": count, "p50_ms": round(sm["p50_ms"], 4), "p99_ms": round(sm["p99_ms"], 4),
                                   "mean_ms": round(sm["mean_ms"], 4), "makespan_s": round(sm["makespan_s"], 3),
                                   "kcliques_per_s": sm["kcliques_per_s"], "epochs": st["epochs"],
                                   "max_requests_per_epoch": st["max_epoch_requests"], "identical_to_alone": same}
        log(f"served-full {rate} req/s: p50 {sm['p50_ms']:.2f} ms p99 {sm['p99_ms']:.1f} ms "
            f"{sm['kcliques_per_s']:.3e} k-cliques/s identical={same}")
    for G in Gs:
        G.close()
    return out


def served_leg(ebb, configs, Gs, rates, budget_s, est_per_rate_s=25.0):
    """Poisson request streams over a resident catalogue (R-MAT s12, s13, Chung-Lu 1e4..3e5,
    ER(2000, 0.01) and 64 of the batched graphs), k U{3..12}; every result compared with the same
    request run alone."""
    from paper_2311_13798_amd.serve import Server, poisson_requests, summarize
    named = [("rmat12", configs.rmat_scale(12)), ("rmat13", configs.rmat_scale(13)),
             ("cl1e4", configs.cl_planted(10000)), ("cl3e4", configs.cl_planted(30000)),
             ("cl1e5", configs.cl_planted(100000)), ("cl3e5", configs.cl_planted(300000)),
             ("er2000", configs.er_small())]
    extra = [ebb.Graph.from_csr(g) for _, g in named]
    cat = extra + Gs[:64]
    alone = {(i, k): G.count(k) for i, G in enumerate(cat) for k in range(3, 13)}
    served = {"catalogue": [n for n, _ in named] + ["64 batched-workload graphs (n scaled by 0.1)"],
              "k": "U{3..12}", "budget_bytes": 1 << 34, "epochs_in_flight": 3, "rates": {}}
    for rate, count in rates:
        if left(budget_s) < est_per_rate_s:
            served["rates"][str(int(rate))] = {"skipped": "wall budget"}
            continue
        S = Server(cat, 1 << 34)
        reqs = poisson_requests(rate=rate, count=count, n_graphs=len(cat), k_lo=3, k_hi=12, seed=1)
        res = S.run_stream(reqs)
        st = S.stats()
        S.close()
        s = summarize(res)
        same = all(r["count"] == alone[(g, k)] and r["status"] == 0 for (o, g, k), r in zip(reqs, res))
        served["rates"][str(int(rate))] = {"requests": count, "p50_ms": round(s["p50_ms"], 4),
                                           "p99_ms": round(s["p99_ms"], 4), "kcliques_per_s": s["kcliques_per_s"],
                                           "epochs": st["epochs"], "max_requests_per_epoch": st["max_epoch_requests"],
                                           "identical_to_alone": same}
        log(f"served {rate:.0f} req/s: p50 {s['p50_ms']:.3f} ms p99 {s['p99_ms']:.3f} ms identical={same}")
    for G in extra:
        G.close()
    return served


def ablation(ebb, torch, configs, graphgen):
    """Variants of the path on the same engine (Section 6.2 (3)-(5), (7)): orderings H (default), C, T
    and the edge- and node-parallel VBBkC roots, Rule (2) off, early termination off, t fixed to 1..5 (the
    t sweep of Section 6.2 (6); t >= 4 through kCtPlex branching).  Times
    are wall-clock per count on the prepared graph (arena built beforehand); a variant stops at the
    first k over 10 s, and a refused count (sub-branch wider than 256) is reported as such."""
    variants = [("H", {}), ("H-no-rule2", {"rule2": 0}), ("H-no-ET", {"early_termination": 0}),
                ("H-t1", {"t_plex": 1}), ("H-t2", {"t_plex": 2}), ("H-t3", {"t_plex": 3}), ("H-t4", {"t_plex": 4}),
                ("H-t5", {"t_plex": 5}), ("C", {"ordering": 1}),
                ("VBBkC-EP", {"ordering": 2, "rule2": 0}), ("VBBkC-NP", {"ordering": 4, "rule2": 0}),
                ("T", {"ordering": 3})]
    graphs = [("R-MAT s12", lambda: graphgen.rmat(12, 16, seed=1), (6, 7, 8, 9, 10)),
              ("Chung-Lu 1e6 + planted", configs.cl_planted, (8, 10, 12)),
              ("R-MAT s18", configs.rmat18, (5, 6, 7))]
    out = {}
    for gname, mk, gks in graphs:
        g = mk()
        out[gname] = {}
        for vname, kw in variants:
            o = ebb.ebbkc_default_options()
            for key, v in kw.items():
                setattr(o, key, v)
            G = ebb.Graph.from_csr(g, options=o)
            rec = {}
            try:
                G.count(4)
                for k in gks:
                    t = time.perf_counter()
                    G.count(k)
                    dt = time.perf_counter() - t
                    rec[str(k)] = round(dt * 1e3, 2)
                    log(f"ablation {gname} {vname} k={k} {dt * 1e3:.1f} ms")
                    if dt > 10.0:
                        break
            except ebb.EbbkcError as e:
                rec["refused"] = str(e)
                log(f"ablation {gname} {vname} refused: {e}")
            G.close()
            out[gname][vname] = rec
    return {"unit": "ms per count", "variants": {v: kw for v, kw in variants}, "results": out}


# ---------------------------------------------------------------- the measurement

def plan_warmups(requested: int, done: int, step_s: float, core_left: float, steps_requested: int) -> bool:
    """Whether another warmup step runs: the first always does (if any was asked for); later ones
    only while the requested timed steps would still fit after it."""
    if done >= requested:
        return False
    if done == 0:
        return True
    return core_left > step_s * (1 + steps_requested)


def plan_timed(done: int, steps_requested: int, step_s: float, core_left: float) -> bool:
    """Whether another timed step starts: the first always does; later ones only while the step is
    expected to end before the measurement deadline."""
    if done >= steps_requested:
        return False
    if done == 0:
        return True
    return core_left > step_s


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3, help="timed steps (an upper bound under the wall budget)")
    ap.add_argument("--warmup", type=int, default=1, help="warmup steps (an upper bound under the wall budget)")
    ap.add_argument("--budget-s", type=float, default=450.0, help="wall budget of the whole run from process start")
    ap.add_argument("--core-s", type=float, default=300.0, help="deadline of the timed steps from process start")
    ap.add_argument("--ks", default="5,6,7,8,9", help="comma-separated k values counted in every step")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-systems", action="store_true", help="skip the batched and served forms")
    ap.add_argument("--no-list", action="store_true", help="skip the full k = 5 listing")
    ap.add_argument("--cpu-threads", type=int, default=0)
    ap.add_argument("--ablation", action="store_true", help="also time the ordering / rule / termination variants")
    ap.add_argument("--traffic-run", action="store_true", help="counter mode: copy calibration + k = 9 count")
    ap.add_argument("--traffic-record", nargs=3, metavar=("FETCH_DIR", "WRITE_DIR", "OUT_JSON"))
    ap.add_argument("--traffic-k", type=int, default=9)
    ap.add_argument("--traffic-command", default="")
    ap.add_argument("--batch-full", action="store_true",
                    help="only the batched workload at its stated size (4,096 graphs), plain vs fused")
    ap.add_argument("--served-full", action="store_true",
                    help="only the served workload at its stated shape (full catalogue, six rates)")
    ap.add_argument("--served-count", type=int, default=500, help="requests per rate in --served-full")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (asked for --gpus {args.gpus}); the multi-GPU sharding of this "
              "path is a design note, not a built feature", file=sys.stderr)
        sys.exit(2)
    if args.traffic_record:
        rec = traffic_record(*args.traffic_record, k=args.traffic_k, command=args.traffic_command)
        print(json.dumps(rec, indent=1))
        return
    if args.traffic_run:
        traffic_run(args.traffic_k)
        return
    if args.batch_full:
        import torch

        import paper_2311_13798_amd as ebb
        from graphgen import configs
        torch.cuda.set_device(0)
        print(json.dumps({"batched_full": batch_full(ebb, torch, configs)}), flush=True)
        return
    if args.served_full:
        import torch

        import paper_2311_13798_amd as ebb
        from graphgen import configs
        torch.cuda.set_device(0)
        print(json.dumps({"served_full": served_full(ebb, torch, configs, count=args.served_count)}), flush=True)
        return
    ks = [int(x) for x in args.ks.split(",") if x]

    import numpy as np
    import torch

    import paper_2311_13798_amd as ebb
    from graphgen import configs

    torch.cuda.set_device(0)
    g = configs.rmat18()
    rp = torch.from_numpy(g.row_ptr).cuda()
    ci = torch.from_numpy(g.col_idx).cuda()
    torch.cuda.synchronize()
    log(f"setup done: n={g.n} m={g.m}")
    opts = ebb.ebbkc_default_options()
    opts.count_work = 1

    def step(tag):
        t0 = time.perf_counter()
        G = ebb.Graph(rp, ci, g.n, options=opts)
        t_prep = time.perf_counter() - t0
        counts, kms, work, wall = {}, {}, {}, {}
        for k in ks:
            t = time.perf_counter()
            counts[k] = G.count(k)
            wall[k] = time.perf_counter() - t
            kms[k] = G.last_timing()
            work[k] = [G.last_work_class(W) for W in (1, 2, 3, 4)]
            log(f"{tag} k={k} N_k={counts[k]} {wall[k]:.3f}s")
        info = G.info
        G.close()
        torch.cuda.synchronize()
        return dict(counts=counts, kms=kms, work=work, wall=wall, prep_ms=info.prepare_ms, prep_wall=t_prep,
                    info=info, total_s=time.perf_counter() - t0)

    step_s = 0.0
    warm = 0
    while plan_warmups(args.warmup, warm, step_s, left(args.core_s), args.steps):
        r = step(f"warmup {warm}")
        step_s = max(step_s, r["total_s"])
        warm += 1
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    runs = []
    while plan_timed(len(runs), args.steps, step_s, left(args.core_s)):
        runs.append(step(f"step {len(runs)}"))
        step_s = max(step_s, runs[-1]["total_s"]) if warm else runs[-1]["total_s"]
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    nsteps = len(runs)
    counts, info = runs[-1]["counts"], runs[-1]["info"]
    assert all(r["counts"] == counts for r in runs), "counts differ between steps"
    total = sum(counts.values())
    ms_per_step = 1000.0 * elapsed / nsteps
    log(f"timed {nsteps} steps after {warm} warmup: {ms_per_step / 1e3:.2f} s per step")

    # dominant launch: the (k, width class) launch with the largest mean device time
    best = None
    for k in ks:
        per_class = np.mean([np.array(r["kms"][k]) for r in runs], axis=0)
        for W in range(1, 5):
            if best is None or per_class[W - 1] > best[2]:
                best = (k, W, float(per_class[W - 1]))
    kd, wd, dom_ms = best
    word_ops = int(np.mean([r["work"][kd][wd - 1][2] for r in runs]))
    achieved = word_ops / (dom_ms / 1e3) / 1e12 if dom_ms > 0 else 0.0
    kernel = f"ebb::k_search<{wd}, false>"
    roofline = {"bound": "alu", "kernel": kernel, "k": kd, "achieved": round(achieved, 4),
                "peak": round(PEAK_WORD_OPS, 3), "unit": "T word-ops/s", "frac": round(achieved / PEAK_WORD_OPS, 5),
                "traffic": traffic_for(kernel, kd), "word_ops_per_launch": word_ops,
                "nodes_per_launch": int(np.mean([r["work"][kd][wd - 1][1] for r in runs])),
                "tasks_per_launch": int(np.mean([r["work"][kd][wd - 1][0] for r in runs])),
                "launch_ms": round(dom_ms, 3),
                # the launch's last wave ends this long after the mean wave end
                "wave_tail_ms": round(float(np.mean([r["work"][kd][wd - 1][3] for r in runs])) / 1e6, 3)}

    line = {
        "metric": METRIC, "value": total / (ms_per_step / 1e3), "unit": "k-cliques/s", "n_gpus": 1,
        "steps": nsteps, "warmup": warm, "steps_requested": args.steps, "warmup_requested": args.warmup,
        "ms_per_step": round(ms_per_step, 3), "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "u64", "data": "synthetic",
        "config": {"workload": "R-MAT scale 18, edge factor 16, (a,b,c,d)=(0.57,0.19,0.19,0.05), seed 1, "
                               "symmetrised, deduplicated, loops dropped; step = prepare + count at k=" +
                               ",".join(map(str, ks)),
                   "n": g.n, "m": g.m, "tau": int(info.tau), "peel_rounds": int(info.rounds), "ks": ks},
        "wall_budget": {"budget_s": args.budget_s, "core_s": args.core_s},
        "counts": {str(k): v for k, v in counts.items()},
        "prepare_ms": round(float(np.mean([r["prep_ms"] for r in runs])), 3),
        "count_wall_s": {str(k): round(float(np.mean([r["wall"][k] for r in runs])), 4) for k in ks},
        # space (Section 6.2 (8)): the prepared graph's device arrays plus its sub-branch arena
        "device_bytes": int(info.device_bytes),
        "branch_ms_by_class": {str(k): [round(x, 3) for x in np.mean([np.array(r["kms"][k]) for r in runs], axis=0)]
                               for k in ks},
        "roofline": roofline,
    }

    if not args.no_cpu_baseline:
        if left(args.budget_s) < 60:
            line["cpu_baseline"] = {"skipped": "wall budget"}
        else:
            import oracle
            th = args.cpu_threads or max(1, min(16, os.cpu_count() or 1))
            got, secs = {}, {}
            for k in (5, 6):  # about 20 s of oracle work on 16 host threads
                t = time.perf_counter()
                got[k] = oracle.count(g, k, threads=th)
                secs[k] = time.perf_counter() - t
            n_all, dt = sum(got.values()), sum(secs.values())
            cb = {"value": n_all / dt, "unit": "k-cliques/s", "cores": th, "kind": "oracle",
                  "sample": "full k=5 and k=6 counts of the same graph (" +
                            ", ".join(f"N_{k}={got[k]} in {secs[k]:.2f} s" for k in got) +
                            "); degeneracy-ordered vertex branch and bound, uint64",
                  "agrees_with_gpu": all(got[k] == counts[k] for k in got if k in counts)}
            if 5 in ks and 6 in ks:
                # the GPU on the same sample, from the timed steps: the k = 5 and k = 6 counts (the
                # first includes the sub-branch arena build) with and without the prepare
                gc = float(np.mean([r["wall"][5] + r["wall"][6] for r in runs]))
                gp = float(np.mean([r["prep_wall"] for r in runs]))
                cb["gpu_same_sample"] = {"count_s": round(gc, 4), "prepare_s": round(gp, 4),
                                         "kcliques_per_s": n_all / gc, "kcliques_per_s_with_prepare": n_all / (gc + gp)}
            line["cpu_baseline"] = cb
            log(f"cpu baseline {n_all / dt:.3e} k-cliques/s on {th} threads")

    if not args.no_list:
        line["listing"] = full_listing(ebb, torch, rp, ci, g) if left(args.budget_s) > 60 else {
            "skipped": "wall budget"}

    if not args.no_systems:
        if left(args.budget_s) > 70:
            line["batched"], Gs = batched_leg(ebb, torch, configs)
            line["served"] = served_leg(ebb, configs, Gs, ((50.0, 500), (200.0, 1000), (1000.0, 2000)),
                                        args.budget_s)
            for G in Gs:
                G.close()
        else:
            line["batched"] = line["served"] = {"skipped": "wall budget"}

    if args.ablation:
        import graphgen
        line["ablation"] = ablation(ebb, torch, configs, graphgen)
    line["bench_wall_s"] = round(time.time() - T_START, 1)
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
