"""Supports, truss levels, ranks and sub-branch sizes at the edges of the triangle kernels' row
classes (out-rows of 32 / 33, 512 / 513 and more than 2,816 entries) and of the peel's edge classes
(256 / 257 triangles and more than a workgroup's worth), against the oracle."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ebb():
    import torch
    import paper_2311_13798_amd as m
    torch.cuda.set_device(0)
    m.load_library()
    return m


def check(ebb, g, what, n3=None):
    print(f"case {what} n={g.n} m={g.m}", flush=True)
    G = ebb.Graph.from_csr(g)
    tr = oracle.truss_levelsync(g)
    assert (G.info.tau, G.info.rounds) == (tr["tau"], tr["rounds"])
    assert (G.export(ebb.ARR_SUPPORT) == oracle.edge_support(g)).all()
    assert (G.export(ebb.ARR_LEVEL) == tr["level"]).all()
    assert (G.export(ebb.ARR_RANK) == tr["rank"]).all()
    assert (G.export(ebb.ARR_SUBSIZE) == oracle.seed_sizes(g, tr["rank"])).all()
    if n3 is not None:
        assert G.count(3) == n3
    G.close()


def book(pages, spines=1):
    """`spines` disjoint edges, each with `pages` common neighbours of its own."""
    edges = []
    for s in range(spines):
        o = s * (pages + 2)
        p = np.arange(o + 2, o + 2 + pages)
        edges += [np.array([[o, o + 1]]), np.stack([np.full(pages, o), p], 1), np.stack([np.full(pages, o + 1), p], 1)]
    return graphgen.from_edges(spines * (pages + 2), np.concatenate(edges))


@pytest.mark.parametrize("pages", [1, 16, 255, 256, 257, 1023, 1024, 1025, 5000])
def test_edges_with_many_triangles(ebb, pages):
    check(ebb, book(pages), f"book{pages}", pages)


def test_many_long_edges_in_one_round(ebb):
    # the spines all leave in the second round
    check(ebb, book(257, 1500), "books", 257 * 1500)


@pytest.mark.parametrize("n", [32, 33, 34, 100, 513, 514])
def test_out_rows_at_class_edges(ebb, n):
    # K_n: vertex i has n - 1 - i out-neighbours; every edge leaves in one round (K_514: 131,841 edges
    # of 512 triangles, more than the workgroups' lists of long edges hold)
    check(ebb, graphgen.complete(n), f"K{n}", n * (n - 1) * (n - 2) // 6)


def test_out_rows_searched_in_place(ebb):
    # complete bipartite with interleaved sides (out-rows of up to 3,000 entries) and a few edges
    # inside one side, so that triangles are found at the long rows
    s = 2950
    a, b = np.meshgrid(2 * np.arange(s), 2 * np.arange(s) + 1, indexing="ij")
    inner = np.array([[0, 2], [0, 4], [2, 4], [6, 4], [0, 5000], [5000, 5002]])
    g = graphgen.from_edges(2 * s, np.concatenate([np.stack([a.ravel(), b.ravel()], 1), inner]))
    print(f"case bipartite n={g.n} m={g.m}", flush=True)
    G = ebb.Graph.from_csr(g)
    deg = np.bincount(inner.ravel(), minlength=g.n)  # inside side A
    e = g.edges()
    side = e % 2
    cross = side[:, 0] != side[:, 1]
    want = np.where(cross, np.where(side[:, 0] == 0, deg[e[:, 0]], deg[e[:, 1]]), s)
    for u, v in ((0, 2), (0, 4), (2, 4)):  # the one triangle inside A
        want[(e[:, 0] == u) & (e[:, 1] == v)] += 1
    assert (G.export(ebb.ARR_SUPPORT) == want).all()
    assert G.count(3) == len(inner) * s + 1
    assert G.count(4) == s
    assert G.count(5) == 0
    G.close()
