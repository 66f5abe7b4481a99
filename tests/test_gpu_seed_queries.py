"""Per-seed counts of more than 2,048 listed edges are looked up and sorted on the device: against counts of single
ranks and whole counts, over all width classes, repeated and unordered ids, list lengths at the edges
of the sort tiles, more ids than one pass takes, and host and device arrays."""
import math

import numpy as np
import pytest

import graphgen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ebb():
    import torch
    import paper_2311_13798_amd as m
    torch.cuda.set_device(0)
    return m


def query(ebb, G, k, eids):
    out = np.full(len(eids), 77, np.uint64)
    ebb.ebbkc_count_seeds(G.handle, k, np.ascontiguousarray(eids, np.int64), out)
    return out


@pytest.mark.parametrize("name", ["k67", "k131", "k195", "k258", "er", "path"])
def test_all_edges_then_some(ebb, name):
    g = {"er": lambda: graphgen.er_planted(300, 0.1, 1, 30, 30, 4), "path": lambda: graphgen.er_planted(50, 0.03, 0, 2, 2, 1)}.get(
        name, lambda: graphgen.complete(int(name[1:])))()
    G = ebb.Graph.from_csr(g)
    m = G.info.m
    rank = np.zeros(m, np.int32)
    ebb.ebbkc_export(G.handle, ebb.ARR_RANK, rank)
    rng = np.random.default_rng(5)
    for k in (3, 4, 5, 8):
        print(f"case {name} k={k}", flush=True)
        if name.startswith("k") and math.comb(int(name[1:]), k) >= 2**64:
            continue
        perm = rng.permutation(m)
        full = query(ebb, G, k, perm)
        assert int(full.sum()) == G.count(k), k
        by_edge = np.zeros(m, np.uint64)
        by_edge[perm] = full
        for e in rng.choice(m, min(m, 25), replace=False):
            r = int(rank[e])
            assert int(by_edge[e]) == G.count_range(k, r, r + 1), (k, e)
        for n in (1, 2, 255, 2047, 2048, 2049, 4096, 4097):
            e = rng.integers(0, m, n)
            assert np.array_equal(query(ebb, G, k, e), by_edge[e]), (k, n)
    G.close()


def test_refused_ids_and_long_lists(ebb):
    import torch
    g = graphgen.er_planted(120, 0.2, 1, 12, 12, 9)
    G = ebb.Graph.from_csr(g)
    m = G.info.m
    by_edge = query(ebb, G, 5, np.arange(m))
    for bad in (-1, m, 1 << 40):
        for n in (3, 3000):  # looked up on the host, on the device
            ids = np.arange(n, dtype=np.int64) % m
            ids[1] = bad
            out = np.full(n, 77, np.uint64)
            with pytest.raises(Exception):
                ebb.ebbkc_count_seeds(G.handle, 5, ids, out)
            assert (out == 77).all()
    n = (1 << 22) + 3  # one pass takes 2^22 ids
    e = np.arange(n, dtype=np.int64) % m
    assert np.array_equal(query(ebb, G, 5, e), by_edge[e])
    d = torch.arange(m, device="cuda", dtype=torch.int64).flip(0)
    o = torch.zeros(m, device="cuda", dtype=torch.int64)
    ebb.ebbkc_count_seeds(G.handle, 5, d, o)
    assert np.array_equal(o.cpu().numpy().view(np.uint64), by_edge[::-1])
    G.close()


@pytest.mark.parametrize("n", [1023, 1024, 1025])
def test_the_longest_list_looked_up_on_the_host(ebb, n):
    g = graphgen.er_planted(200, 0.2, 1, 20, 20, 3)
    G = ebb.Graph.from_csr(g)
    by_edge = query(ebb, G, 5, np.arange(G.info.m))
    assert int(by_edge.sum()) == G.count(5)
    e = np.random.default_rng(n).integers(0, G.info.m, n)
    assert np.array_equal(query(ebb, G, 5, e), by_edge[e])
    rank = np.zeros(G.info.m, np.int32)
    ebb.ebbkc_export(G.handle, ebb.ARR_RANK, rank)
    for i in (0, n // 2, n - 1):
        r = int(rank[e[i]])
        assert int(by_edge[e[i]]) == G.count_range(5, r, r + 1)
    G.close()
