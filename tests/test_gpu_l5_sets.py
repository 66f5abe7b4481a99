"""One-word l = 5 nodes: sets of at least 24 vertices are taken by the wave, smaller ones are queued.  Dense
graphs whose sets lie on both sides of the line, with none, few and many missing pairs, against the oracle."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [24, 26, 27, 28, 29, 31, 40, 66])
@pytest.mark.parametrize("missing", [0.0, 0.02, 0.15])
def test_sets_on_both_sides_of_the_line(n, missing):
    import torch
    import paper_2311_13798_amd as ebb
    torch.cuda.set_device(0)
    u, v = np.triu_indices(n, 1)
    keep = np.random.default_rng(n).random(len(u)) >= missing
    g = graphgen.from_edges(n, np.stack([u[keep], v[keep]], 1))
    G = ebb.Graph.from_csr(g)
    for k in (7, 9) if n <= 40 else (7,):
        print(f"case l5 n={n} missing={missing} k={k}", flush=True)
        assert G.count(k) == oracle.count(g, k)
    G.close()
