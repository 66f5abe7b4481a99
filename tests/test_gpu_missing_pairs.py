"""4-cliques from missing pairs on the matrix cores at the edges of its tiles (sets of 4 .. 193
vertices around every multiple of 16), of its words, and of the ranges of split roots searched on
narrower rows: graphs whose missing pairs form disjoint random blocks, so that N_k is a coefficient
of the product of the blocks' independence polynomials."""
import itertools

import numpy as np
import pytest

import graphgen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ebb():
    import torch
    import paper_2311_13798_amd as m
    torch.cuda.set_device(0)
    m.load_library()
    return m


def blocks_graph(n, block, density, seed):
    """(graph, [N_0, N_1, ...]) of K_n minus random graphs of the given density on disjoint blocks."""
    r = np.random.Generator(np.random.PCG64(seed))
    perm = r.permutation(n)
    adj = ~np.eye(n, dtype=bool)
    poly = [1]
    for b in range(0, n, block):
        ids = perm[b:b + block]
        s = len(ids)
        miss = np.triu(r.random((s, s)) < density, 1)
        miss |= miss.T
        adj[np.ix_(ids, ids)] &= ~miss
        ind = [0] * (s + 1)
        masks = [int(sum(1 << j for j in range(s) if miss[i, j])) for i in range(s)]
        for sub in range(1 << s):
            if not any((sub >> i) & 1 and (sub & masks[i]) for i in range(s)):
                ind[bin(sub).count("1")] += 1
        poly = [sum(poly[i] * ind[j - i] for i in range(max(0, j - s), min(j, len(poly) - 1) + 1))
                for j in range(len(poly) + s)]
    iu = np.stack(np.triu_indices(n, 1), 1)
    return graphgen.from_edges(n, iu[adj[iu[:, 0], iu[:, 1]]], f"blocks{n}"), poly


def test_expected_values_on_a_small_graph():
    g, poly = blocks_graph(12, 5, 0.5, 3)
    adj = np.zeros((12, 12), bool)
    e = g.edges()
    adj[e[:, 0], e[:, 1]] = adj[e[:, 1], e[:, 0]] = True
    for k in (3, 4, 5):
        assert poly[k] == sum(all(adj[a, b] for a, b in itertools.combinations(c, 2))
                              for c in itertools.combinations(range(12), k))


@pytest.mark.parametrize("n", [6, 16, 17, 18, 19, 33, 34, 35, 50, 65, 66, 67, 81, 98, 130, 131, 146, 194, 195])
@pytest.mark.parametrize("density", [0.3, 0.8])
def test_dense_sets_at_tile_edges(ebb, n, density):
    g, poly = blocks_graph(n, 9, density, n)
    # the range split threshold at its default (ranges on narrower rows past about 60 vertices at
    # k = 7) and never; early termination off, so that every leaf is counted from its sets
    for split in (0, -1):
        opt = ebb.ebbkc_default_options()
        opt.early_termination = 0
        opt.split_threshold = split
        G = ebb.Graph.from_csr(g, options=opt)
        for k in (5, 6, 7) if n > 70 else (5, 6, 7, 8, 9):
            print(f"case blocks n={n} density={density} split={split} k={k}", flush=True)
            assert G.count(k) == (poly[k] if k < len(poly) else 0), (n, k)
        G.close()
