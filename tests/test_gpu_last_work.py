"""Work and time figures of the last count: one count's, over all its passes."""
import numpy as np
import pytest

import graphgen

pytestmark = pytest.mark.gpu


def options(ebb):
    o = ebb.ebbkc_default_options()
    o.count_work = 1
    return o


def test_seed_lists_of_several_passes():
    import torch
    import paper_2311_13798_amd as ebb
    torch.cuda.set_device(0)
    G = ebb.Graph.from_csr(graphgen.er_planted(120, 0.2, 1, 12, 12, 9), options=options(ebb))
    m, k = G.info.m, 6
    out = np.zeros(m, np.uint64)
    ebb.ebbkc_count_seeds(G.handle, k, np.arange(m, dtype=np.int64), out)
    once, cls = list(G.last_work()), [list(G.last_work_class(W)) for W in (1, 2, 3, 4)]
    assert once[0] > 0 and once[1] > 0 and once[2] > 0
    reps = (1 << 22) // m + 2  # one pass takes 2^22 ids: the second one here is short
    ids = np.tile(np.arange(m, dtype=np.int64), reps)
    assert len(ids) > 1 << 22
    full = np.zeros(len(ids), np.uint64)
    ebb.ebbkc_count_seeds(G.handle, k, ids, full)
    assert np.array_equal(full.reshape(reps, m), np.tile(out, (reps, 1)))
    assert list(G.last_work())[:3] == [reps * x for x in once[:3]]
    for W in (1, 2, 3, 4):
        assert list(G.last_work_class(W))[:3] == [reps * x for x in cls[W - 1][:3]]
    G.close()


@pytest.mark.parametrize("seeds", [3, 3000])  # looked up on the host, on the device
def test_classes_that_did_not_run_are_zero(seeds):
    import torch
    import paper_2311_13798_amd as ebb
    torch.cuda.set_device(0)
    # K_100 and, apart from it, K_12: two width classes
    G = ebb.Graph.from_csr(graphgen.disjoint_cliques([100, 12]), options=options(ebb))
    G.count(5)
    t, w = list(G.last_timing()), [list(G.last_work_class(W)) for W in (1, 2)]
    assert t[0] > 0 and t[1] > 0 and w[0][0] > 0 and w[1][0] > 0
    rank = np.zeros(G.info.m, np.int32)
    ebb.ebbkc_export(G.handle, ebb.ARR_RANK, rank)
    counts = [G.count_range(7, r, r + 1) for r in range(G.info.m)]
    # seeds of at most 64 candidates hold fewer than C(64, 5) 7-cliques of their own
    small = int(np.flatnonzero([0 < counts[r] <= 252 for r in rank])[0])
    G.count(5)
    out = np.zeros(seeds, np.uint64)
    ebb.ebbkc_count_seeds(G.handle, 7, np.full(seeds, small, np.int64), out)
    assert (out == counts[rank[small]]).all()
    assert G.last_timing()[0] > 0 and list(G.last_timing())[1:] == [0, 0, 0]
    assert list(G.last_work_class(2)) == [0, 0, 0, 0]
    G.close()
