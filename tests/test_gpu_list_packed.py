"""Sorted listings pack whole tuples into 64-bit keys where they fit: tuples, order and checksums at
the last k that fits and the first that does not, from one tuple up, against the oracle's hash and
the combinations themselves."""
import itertools
import math

import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


# (n, k): bits of a vertex id times k on both sides of 64, and a single tuple
@pytest.mark.parametrize("n,k", [(12, 12), (16, 15), (16, 16), (17, 12), (17, 13), (17, 17), (18, 12), (18, 13), (22, 4)])
def test_cliques_of_a_clique(n, k):
    import torch
    import paper_2311_13798_amd as ebb
    torch.cuda.set_device(0)
    g = graphgen.complete(n)
    G = ebb.Graph.from_csr(g)
    N = math.comb(n, k)
    buf = torch.full((N, k), -1, dtype=torch.int32, device="cuda")
    print(f"case n={n} k={k}", flush=True)
    w, ho, hu = ebb.ebbkc_list(G.handle, k, buf, N, ebb.LIST_SORTED)
    assert w == N
    assert np.array_equal(buf.cpu().numpy(), np.array(list(itertools.combinations(range(n), k)), dtype=np.int32))
    c, oho, ohu, _ = oracle.list_lex(g, k)
    assert (c, oho, ohu) == (N, ho, hu)
    G.close()
