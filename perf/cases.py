"""The timed workloads: what a program does with this framework, through its public entry points.

A case is one of the framework's uses ("kind") on one graph family at one size:

  step       a graph comes in as CSR arrays, is prepared and counted at a few k, and is dropped
             (the bench step; a one-shot program)
  prepare    a graph is prepared and its edge order read back (ranks, levels, supports)
  count      a prepared graph that stays resident is counted at one or more k
  omega      the maximum clique size and the triangles of a resident graph
  list       every k-clique of a resident graph into a device buffer, sorted (the default)
  seeds      per-seed counts of listed edges of a resident graph
  batch      many (graph, k) counts as one fused batch, made and run once; sub-branches from the
             graphs' arenas, or built by the tasks in LDS (build = True)
  serve      a burst of requests submitted to a resident server and polled until all are done

The graph families are the repository's: Erdos-Renyi with planted cliques, R-MAT with edge factor
16 and (0.57, 0.19, 0.19, 0.05), and Chung-Lu with exponent 2.1, mean degree 30 and planted
cliques of 30..60 vertices.  They are drawn here with torch from the seed alone.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2311_13798_amd as ebb

# ---------------------------------------------------------------- inputs


def _gen(seed):
    return torch.Generator().manual_seed(int(seed) & 0x7FFFFFFFFFFFFFFF)


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _csr(n, u, v):
    """Simple undirected CSR (int32, rows ascending) of the pairs (u, v): loops and repeats dropped."""
    dev = _device()
    u, v = u.to(dev), v.to(dev)
    keep = u != v
    u, v = u[keep].long(), v[keep].long()
    key = torch.unique(torch.cat([u * n + v, v * n + u]))
    row = torch.div(key, n, rounding_mode="floor")
    rp = torch.zeros(n + 1, dtype=torch.int64, device=dev)
    rp[1:] = torch.cumsum(torch.bincount(row, minlength=n), 0)
    return rp.int(), (key - row * n).int()


def _planted(n, count, smin, smax, g):
    us, vs = [], []
    for _ in range(count):
        s = min(n, int(torch.randint(smin, smax + 1, (1,), generator=g)))
        ids = torch.randperm(n, generator=g)[:s]
        a, b = torch.triu_indices(s, s, 1)
        us.append(ids[a])
        vs.append(ids[b])
    return us, vs


def _er(n, p, plant, seed):
    """G(n, p), with one planted clique of `plant` vertices when plant > 0."""
    g = _gen(seed)
    a, b = torch.nonzero(torch.rand(n, n, generator=g).triu_(1) > 1.0 - p, as_tuple=True)
    us, vs = _planted(n, 1 if plant else 0, plant, plant, g)
    return _csr(n, torch.cat([a, *us]), torch.cat([b, *vs]))


def _rmat(n, seed):
    """16 n sampled pairs over the next power of two, those within n kept."""
    g = _gen(seed)
    scale = max(1, math.ceil(math.log2(n)))
    m = 16 * n
    u = torch.zeros(m, dtype=torch.int32)
    v = torch.zeros(m, dtype=torch.int32)
    for _ in range(scale):
        r = torch.rand(m, generator=g)
        u = 2 * u + (r >= 0.76).int()
        v = 2 * v + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95)).int()
    keep = (u < n) & (v < n)
    return _csr(n, u[keep], v[keep])


def _chung_lu(n, seed):
    """Edge (i, j) with probability min(1, w_i w_j / sum w), w_i ~ (i + i0)^(-1/1.1) and the largest
    weight sqrt(sum w): the dense core pair by pair, the rest by drawing endpoints; one planted clique
    of 30..60 vertices per 5,000 vertices."""
    g = _gen(seed)
    total = 30.0 * n
    i = np.arange(n, dtype=np.float64)
    lo, hi = 1e-3, float(n)
    for _ in range(60):  # i0 with w_0 = sqrt(total)
        i0 = math.sqrt(lo * hi)
        w = (i + i0) ** (-1.0 / 1.1)
        if total * w[0] / w.sum() > math.sqrt(total):
            lo = i0
        else:
            hi = i0
    cum = torch.from_numpy(np.cumsum(w / w.sum()))
    m = int(total / 2)
    u = torch.searchsorted(cum, torch.rand(m, generator=g, dtype=torch.float64)).clamp_(max=n - 1)
    v = torch.searchsorted(cum, torch.rand(m, generator=g, dtype=torch.float64)).clamp_(max=n - 1)
    core = min(n, 2048)
    rest = (u >= core) | (v >= core)
    wc = torch.from_numpy(w[:core] * math.sqrt(total) / w.sum())
    a, b = torch.nonzero((torch.rand(core, core, generator=g, dtype=torch.float64) < torch.outer(wc, wc)).triu_(1), as_tuple=True)
    us, vs = _planted(n, max(2, n // 5000), 30, 60, g)
    return _csr(n, torch.cat([u[rest], a, *us]), torch.cat([v[rest], b, *vs]))


def _graph(family, n, p, plant, seed):
    if family == "er":
        return _er(n, p, plant, seed)
    return _rmat(n, seed) if family == "rmat" else _chung_lu(n, seed)


def _many(count, nmax, seed):
    """Graphs of the batched workload: n ~ U{50..nmax}, p ~ U[0.005, 0.2], one in five with a
    planted clique of 20..40 vertices, k ~ U{3..10}."""
    r = np.random.Generator(np.random.PCG64(seed))
    out = []
    for i in range(count):
        n, p = int(r.integers(50, nmax + 1)), float(r.uniform(0.005, 0.2))
        k, size, s = int(r.integers(3, 11)), int(r.integers(20, 41)), int(r.integers(1 << 40))
        out.append((_er(n, p, size if i % 5 == 0 else 0, s), n, k))
    return out


# ---------------------------------------------------------------- cases


def listed():
    return [
        # the smallest call: a resident 2,000-vertex graph counted again (launches and host path)
        dict(name="count_er2k", kind="count", family="er", n=2000, p=0.05, plant=0, ks="5"),
        # a one-shot program on the small plain workload, host arrays in, one count out
        dict(name="step_er2k", kind="step", family="er", n=2000, p=0.01, plant=0, ks="4", host=True),
        # the truss order alone, as an analysis that reads ranks and levels does; n odd
        dict(name="prepare_rmat", kind="prepare", family="rmat", n=49999, p=0.0, plant=0),
        # the bench step at its graph's full size, up to the k that fits a pass
        dict(name="step_rmat18", kind="step", family="rmat", n=1 << 18, p=0.0, plant=0, ks="5,6", host=False),
        # the same graph resident, at the k where the search dominates
        dict(name="count_rmat18", kind="count", family="rmat", n=1 << 18, p=0.0, plant=0, ks="7"),
        # large cliques: early termination, odd n
        dict(name="count_cl", kind="count", family="cl", n=299999, p=0.0, plant=0, ks="8,10"),
        # omega of a graph with planted cliques: many counts, most near or past omega
        dict(name="omega_cl", kind="omega", family="cl", n=30001, p=0.0, plant=0),
        # a listing that fills a buffer, sorted
        dict(name="list_rmat", kind="list", family="rmat", n=8191, p=0.0, plant=0, k=4),
        # counts per seed edge, as chunked listings and local analyses ask for them
        dict(name="seeds_rmat", kind="seeds", family="rmat", n=65537, p=0.0, plant=0, k=6, seeds=100003),
        # the batched workload: small graphs, arenas
        dict(name="batch_small", kind="batch", count=192, nmax=500, build=False),
        # the batched workload at its stated graph sizes, every task building its sub-branch
        dict(name="batch_build", kind="batch", count=10, nmax=5000, build=True),
        # a burst of requests to a resident server
        dict(name="serve_mixed", kind="serve", count=24, nmax=500, requests=200),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _er_kmax(n, p):
    """The largest k up to 7 of which G(n, p) holds a hundred k-cliques or so."""
    return max([3] + [k for k in range(3, 8) if math.comb(n, k) * p ** (k * (k - 1) // 2) >= 100])


def draw(rng):
    kind = rng.choice(["count", "count", "count", "step", "step", "prepare", "omega", "list", "seeds", "batch", "serve"])
    if kind == "batch":
        if rng.random() < 0.5:
            return dict(kind=kind, count=_log_int(rng, 8, 192), nmax=rng.randrange(100, 501), build=rng.random() < 0.3)
        return dict(kind=kind, count=rng.randrange(2, 9), nmax=rng.randrange(1000, 4001), build=True)
    if kind == "serve":
        return dict(kind=kind, count=rng.randrange(8, 25), nmax=rng.randrange(100, 501), requests=_log_int(rng, 8, 200))
    family = rng.choice(["er", "rmat", "cl"])
    if family == "er":
        n = _log_int(rng, 200, 4000)
        p = round(rng.uniform(max(0.005, 12.0 / n), 0.1), 4)
        case = dict(kind=kind, family=family, n=n, p=p, plant=rng.choice([0, 0, rng.randrange(12, 31)]))
    elif family == "rmat":
        n = _log_int(rng, 1000, 200000)
        case = dict(kind=kind, family=family, n=n, p=0.0, plant=0)
    else:
        n = _log_int(rng, 5000, 250000)
        case = dict(kind=kind, family=family, n=n, p=0.0, plant=0)
    if kind in ("count", "step"):
        kmax = dict(cl=9, rmat=7).get(family) or _er_kmax(n, p)
        ks = sorted(rng.sample(range(3, kmax + 1), min(kmax - 2, rng.choice([1, 1, 2]))))
        case["ks"] = ",".join(map(str, ks))
        if kind == "step":
            case["host"] = rng.random() < 0.3
    elif kind == "omega":
        case["n"] = min(n, 30001)
        if family == "rmat":  # without planted cliques the search near omega is long: smaller graphs
            case["n"] = min(n, 3000)
    elif kind == "list":
        # planted cliques of 60 hold too many k-cliques to keep: R-MAT or G(n, p)
        if family == "cl":
            case.update(family="rmat")
        case["n"] = min(n, 8192)
        case["k"] = rng.choice([3, 4]) if case["family"] == "rmat" else rng.randrange(3, min(5, _er_kmax(case["n"], p)) + 1)
    elif kind == "seeds":
        case["n"] = min(n, 65537)
        case["k"] = rng.randrange(3, _er_kmax(case["n"], p) + 1) if family == "er" else rng.randrange(4, 7)
        case["seeds"] = _log_int(rng, 100, 100000)
    return case


# ---------------------------------------------------------------- state and pass


class _Server:
    """A resident server; destroyed with the state."""

    def __init__(self, graphs, budget):
        self.graphs = graphs
        self.handle = ebb.ebbkc_server_create([G.handle for G in graphs], budget)

    def __del__(self):
        try:
            ebb.ebbkc_server_destroy(self.handle)
        except Exception:
            pass


def _edge_room(case):
    """More edges than a graph of the case has."""
    n = case["n"]
    if case["family"] == "er":
        return int(case["p"] * n * n / 2 + 4 * math.sqrt(case["p"]) * n) + case["plant"] ** 2 + 100
    return 16 * n if case["family"] == "rmat" else 17 * n + 10000


def _list_room(case):
    """Tuples of a buffer that holds every k-clique of a graph of the case."""
    n, k = case["n"], case["k"]
    if case["family"] == "er":
        mean = math.comb(n, k) * case["p"] ** (k * (k - 1) // 2)
        return int(1.5 * mean) + math.comb(case["plant"], k) * 2 + 10000
    return int((1.5e5 * (n / 1000) ** 1.34) if k == 3 else (9e5 * (n / 1000) ** 1.7))


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("batch", "serve"):
        many = _many(case["count"], case["nmax"], seed)
        opt = ebb.ebbkc_default_options()
        if case.get("build"):
            opt.batch_build = ebb.BATCH_BUILD
        graphs = [ebb.Graph(rp, ci, n) for (rp, ci), n, _ in many]
        state = dict(kind=kind, graphs=graphs, ks=[k for _, _, k in many], opt=opt)
        if kind == "serve":
            r = np.random.Generator(np.random.PCG64(seed + 1))
            state["server"] = _Server(graphs, 16 << 30)
            state["requests"] = [(int(r.integers(len(graphs))), int(r.integers(3, 9))) for _ in range(case["requests"])]
        return state
    rp, ci = _graph(case["family"], case["n"], case["p"], case["plant"], seed)
    state = dict(kind=kind, n=case["n"], ks=[int(k) for k in case.get("ks", "").split(",") if k])
    if kind in ("step", "prepare"):
        if case.get("host"):
            rp, ci = rp.cpu().numpy(), ci.cpu().numpy()
        state.update(rp=rp, ci=ci)
        if kind == "prepare":  # rank, level and support of every edge are read back into these
            state["arrays"] = torch.zeros(3, _edge_room(case), dtype=torch.int32, device="cuda")
        return state
    G = ebb.Graph(rp, ci, case["n"])
    state["graph"] = G
    if kind == "list":
        state["k"] = case["k"]
        state["cap"] = _list_room(case)
        state["buf"] = torch.zeros(state["cap"], case["k"], dtype=torch.int32, device="cuda")
    if kind == "seeds":
        state["k"] = case["k"]
        m = int(G.info.m)
        e = torch.randperm(m, generator=_gen(seed + 1))[: min(m, case["seeds"])]
        state["eids"] = e.numpy().astype(np.int64)
    return state


def _whole(values):
    """Unsigned 64-bit results, bit for bit."""
    return np.array(values, dtype=np.uint64).view(np.int64)


def run(state):
    kind = state["kind"]
    if kind == "count":
        return _whole([state["graph"].count(k) for k in state["ks"]])
    if kind == "omega":
        return int(state["graph"].max_clique_size()), _whole([state["graph"].count(3)])
    if kind == "list":
        written, ordered, unordered = ebb.ebbkc_list(state["graph"].handle, state["k"], state["buf"], state["cap"])
        return written, _whole([ordered, unordered]), state["buf"]
    if kind == "seeds":
        out = np.zeros(len(state["eids"]), np.uint64)
        ebb.ebbkc_count_seeds(state["graph"].handle, state["k"], state["eids"], out)
        return out.view(np.int64)
    if kind == "batch":
        b = ebb.Batch(state["graphs"], state["ks"], state["opt"])
        counts = b.run()
        b.close()
        return _whole(counts)
    if kind == "serve":
        s = state["server"].handle
        ids = [ebb.ebbkc_server_submit(s, g, k) for g, k in state["requests"]]
        got = {}
        while len(got) < len(ids):
            for r in ebb.ebbkc_server_poll(s, wait=True):
                got[r["id"]] = (r["status"], r["count"])
        return [got[i][0] for i in ids].count(ebb.OK), _whole([got[i][1] for i in ids])
    G = ebb.Graph(state["rp"], state["ci"], state["n"])
    if kind == "step":
        out = _whole([G.count(k) for k in state["ks"]])
    else:
        arrays = state["arrays"]
        for row, which in zip(arrays, (ebb.ARR_RANK, ebb.ARR_LEVEL, ebb.ARR_SUPPORT)):
            ebb.ebbkc_export(G.handle, which, row)
        out = arrays, int(G.info.tau), int(G.info.m)
    G.close()
    return out


def _edges(family, n, p, plant):
    """About how many edges a graph of the family has after loops and repeats are dropped."""
    if family == "er":
        return p * n * n / 2 + plant * plant / 2
    return 14.5 * n if family == "rmat" else 15.0 * n


def work(case):
    """Bytes: every graph's CSR read once (both directions), the outputs written once.  Operations:
    one test per edge and counted k (a lower bound on any exact count)."""
    kind = case["kind"]
    if kind in ("batch", "serve"):
        m = case["count"] * 0.1 * case["nmax"] ** 2 / 6
        return {"bytes": 8 * m + 4 * case["count"] * case["nmax"] / 2, "flops": m}
    n = case["n"]
    m = _edges(case["family"], n, case["p"], case["plant"])
    read, counts = 4 * (n + 1) + 8 * m, max(1, len(case.get("ks", "").split(",")))
    if kind == "prepare":
        return {"bytes": read + 12 * m, "flops": m}
    if kind == "list":
        return {"bytes": read + 4 * case["k"] * m, "flops": m}
    if kind == "seeds":
        return {"bytes": read + 16 * case["seeds"], "flops": m}
    return {"bytes": read + 8 * counts, "flops": m * counts}


def exact(case, seed):
    """Plain counts with Python integers as bit sets, where the graph is small enough; the numbers
    are whole, so there is nothing between them and the exact value."""
    if case["kind"] not in ("count", "step") or case["family"] != "er" or case["n"] > 2500 or case["plant"]:
        return None
    ks = [int(k) for k in case["ks"].split(",")]
    if max(ks) > 5 or case["p"] > 0.05:
        return None
    rp, ci = (t.cpu().numpy() for t in _er(case["n"], case["p"], 0, seed))
    later = [0] * case["n"]
    for u in range(case["n"]):
        for w in ci[rp[u]:rp[u + 1]]:
            if w > u:
                later[u] |= 1 << int(w)

    def count(cand, left):
        if left == 1:
            return bin(cand).count("1")
        total = 0
        while cand:
            low = cand & -cand
            cand ^= low
            total += count(cand & later[low.bit_length() - 1], left - 1)
        return total

    return np.array([count((1 << case["n"]) - 1, k) for k in ks], dtype=np.int64)
