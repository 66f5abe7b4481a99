"""The task list of a batch over arenas is planned from the slots' sizes; one over sub-branches built
in LDS has a task per edge.  Both against closed forms at the edges of the width classes, with roots
split often, rarely and never, one graph under several k, and through the calls of a batch that
launches first and then replays."""
import math

import pytest

import graphgen

pytestmark = pytest.mark.gpu

SIZES = [3, 10, 66, 67, 130, 131, 194, 195, 258]
KS = {n: [3, 4, 5] + ([7, 8, 9, n - 2, n - 1, n, n + 1] if n <= 67 else []) for n in SIZES}


@pytest.fixture(scope="module")
def cliques():
    import torch
    import paper_2311_13798_amd as ebb
    torch.cuda.set_device(0)
    G = {n: ebb.Graph.from_csr(graphgen.complete(n)) for n in SIZES}
    empty = ebb.Graph.from_csr(graphgen.empty(5))
    yield ebb, G, empty
    for g in [*G.values(), empty]:
        g.close()


@pytest.mark.parametrize("split", [-1, 0, 1, 1 << 16])
@pytest.mark.parametrize("build", [False, True])
def test_cliques_of_cliques(cliques, split, build):
    ebb, G, empty = cliques
    cases = [(n, k) for n in SIZES for k in KS[n] if 1 <= k]
    cases = [(n, k) for n, k in cases if math.comb(n, k) < 2**64]
    graphs = [G[n] for n, _ in cases] + [empty, empty]
    ks = [k for _, k in cases] + [3, 1]
    want = [math.comb(n, k) for n, k in cases] + [0, 5]
    o = ebb.ebbkc_default_options()
    o.split_threshold = split
    o.batch_build = ebb.BATCH_BUILD if build else ebb.BATCH_ARENA
    print(f"case split={split} build={build}", flush=True)
    B = ebb.Batch(graphs, ks, options=o)
    for rep, use_graph in enumerate((True, True, False, True)):
        assert B.run(use_graph=use_graph) == want, rep
    B.close()


@pytest.mark.parametrize("p", [0.03, 0.3, 0.7])
def test_built_sub_branches_of_every_density(cliques, p):
    # tasks that build: with and without colours (a search that does not branch colours the dense
    # ones), edges alone at k = 4, rows of G up to and beyond the 64 entries of one search step
    ebb, _, _ = cliques
    n = 180 if p < 0.7 else 90
    graphs = [ebb.Graph.from_csr(graphgen.er_planted(n + d, p, 1, 20, 20, 11 + d)) for d in range(3)]
    ks = [3, 4, 5, 6, 7, 8]
    o = ebb.ebbkc_default_options()
    o.batch_build = ebb.BATCH_BUILD
    print(f"case p={p}", flush=True)
    B = ebb.Batch([g for g in graphs for _ in ks], ks * 3, options=o)
    assert B.run() == [g.count(k) for g in graphs for k in ks]
    B.close()
    for g in graphs:
        g.close()
