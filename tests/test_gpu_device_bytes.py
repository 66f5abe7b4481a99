"""The device memory ebbkc_info_get reports: every array a handle holds, after prepare, after the edge
sub-branches and after the vertex sub-branches are built."""
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


def slots(sizes, per_slot):
    """Bytes of the sub-branches of these sizes: rows, ids and colours of the vertices, per_slot a slot."""
    c = sizes[sizes > 0].astype(np.int64)
    return int((c * ((c + 63) // 64) * 8 + 6 * c).sum()) + per_slot * len(c)


@pytest.mark.parametrize("ordering", range(5))
@pytest.mark.parametrize("adj_max_n", [0, -1])
def test_every_held_array_is_counted(ebb, ordering, adj_max_n):
    g = graphgen.er_planted(700, 0.05, 1, 70, 70, 4)
    o = ebb.ebbkc_default_options()
    o.ordering, o.adj_max_n = ordering, adj_max_n
    G = ebb.Graph.from_csr(g, options=o)
    n, m = g.n, g.m
    bytes_now = lambda: ebb.ebbkc_info_get(G.handle).device_bytes
    # offsets, ids, ranks and rank-sorted rows; seven arrays per edge and the oriented rows
    want = 4 * (2 * (n + 1) + 2 * 2 * m + 7 * m) + 8 * (2 * m + m)
    want += {1: 8, 2: 4, 4: 4}.get(ordering, 0) * n  # vertex positions and colours
    if adj_max_n == 0:
        want += n * ((n + 63) // 64) * 10  # adjacency bitmap and its counts
    assert bytes_now() == want
    sizes = G.export(ebb.ARR_SUBSIZE)
    assert bytes_now() == want
    ebb.ebbkc_count_range(G.handle, 4, 0, m // 2)  # the edge sub-branches
    want += slots(sizes, 36)
    assert bytes_now() == want
    if ordering == 4:
        G.count(4)  # the vertex sub-branches: later neighbours in the vertex order
        pos = G.export(ebb.ARR_VERTEX_POS)
        e = g.edges()
        first = np.where(pos[e[:, 0]] < pos[e[:, 1]], e[:, 0], e[:, 1])
        want += slots(np.bincount(first, minlength=n), 40)
        assert bytes_now() == want
    G.close()
