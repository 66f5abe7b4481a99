"""Searches deeper than the frames in LDS with more tasks than the widest class runs waves: per-seed counts
of near-maximum cliques of K_n without early termination, by more listed seeds than one launch has waves,
against binomials."""
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
    m.load_library()
    return m


@pytest.mark.parametrize("n,k", [(40, 38), (72, 70), (140, 138), (200, 198)])
@pytest.mark.parametrize("seeds", [2048, 2049, 5000])
def test_listed_seeds(ebb, n, k, seeds):
    print(f"case K{n} k={k} seeds={seeds}", flush=True)
    o = ebb.ebbkc_default_options()
    o.early_termination = 0
    G = ebb.Graph.from_csr(graphgen.complete(n), options=o)
    assert (G.export(ebb.ARR_RANK) == np.arange(G.info.m)).all()  # one round: ranks by edge id
    j = 1 + np.arange(seeds) % 6  # edge (0, j) seeds the cliques of 0, j and k - 2 later vertices
    out = np.zeros(seeds, np.uint64)
    ebb.ebbkc_count_seeds(G.handle, k, (j - 1).astype(np.int64), out)
    want = np.array([math.comb(n - 1 - i, k - 2) for i in j], np.uint64)
    assert (out == want).all()
    G.close()
