"""Whole-graph counts and listings take their tasks from the arena's slot order; rank ranges build
a task list.  Both against closed forms and each other at the edges of the width classes, of the
scan tiles (2,048 edges) and of root splitting."""
import math

import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ebb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2311_13798_amd as ebb
    torch.cuda.set_device(0)
    return ebb


@pytest.mark.parametrize("n", [3, 5, 64, 65, 66, 67, 130, 131, 194, 195, 257, 258])
def test_complete_graph_at_class_edges(ebb, n):
    # sub-branches of 0 .. n - 2 vertices: every size up to the class edge
    G = ebb.Graph.from_csr(graphgen.complete(n))
    m = n * (n - 1) // 2
    for k in (4, 5, 6):
        print(f"case complete n={n} k={k}", flush=True)
        assert G.count(k) == math.comb(n, k), (n, k)
        assert sum(G.count_range(k, a, b) for a, b in ((0, m // 3), (m // 3, m))) == math.comb(n, k), (n, k)
    G.close()


@pytest.mark.parametrize("m", [2047, 2048, 2049, 4096, 4097])
def test_slots_at_tile_edges(ebb, m):
    # m edges, all in one graph: a dense core plus pendant edges (no sub-branch) up to m
    core = graphgen.er_planted(60, 0.7, 0, 2, 2, 5)
    e = core.edges()
    extra = m - len(e)
    assert extra > 0
    pend = np.stack([np.arange(extra) % 60, 60 + np.arange(extra)], 1).astype(np.int32)
    g = graphgen.from_edges(60 + extra, np.concatenate([e, pend]), f"tile{m}")
    assert g.m == m
    G = ebb.Graph.from_csr(g)
    for k in (3, 4, 5, 7):
        print(f"case tile m={m} k={k}", flush=True)
        assert G.count(k) == oracle.count(core, k), (m, k)
    G.close()


@pytest.mark.parametrize("split", [0, 1, 50, 5000, -1])
def test_split_roots_and_whole_roots(ebb, split):
    import torch
    g = graphgen.er_planted(220, 0.5, 1, 24, 24, 11)
    opt = ebb.ebbkc_default_options()
    opt.split_threshold = split
    G = ebb.Graph.from_csr(g, options=opt)
    for k in (5, 6, 7, 8):
        print(f"case split={split} k={k}", flush=True)
        want = oracle.count(g, k)
        cuts = [0, G.info.m // 5, G.info.m // 2, G.info.m]
        assert G.count(k) == want, (split, k)
        assert sum(G.count_range(k, a, b) for a, b in zip(cuts[:-1], cuts[1:])) == want, (split, k)
    n6 = oracle.count(g, 6)
    buf = torch.empty(n6, 6, dtype=torch.int32, device="cuda")
    whole = ebb.ebbkc_list(G.handle, 6, buf, n6, 0)
    rows = torch.unique(buf, dim=0)
    assert whole[0] == n6 and len(rows) == n6
    hu = 0
    for a, b in zip(cuts[:-1], cuts[1:]):
        hu = (hu + ebb.ebbkc_list(G.handle, 6, buf, n6, 0, a, b)[2]) % (1 << 64)
    assert hu == whole[2]
    G.close()
