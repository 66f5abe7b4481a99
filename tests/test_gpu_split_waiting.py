"""Runtime splitting with more waves than may wait for nodes: counts where nearly every wave runs out of
tasks early, with splitting off, on demand at several bounds and forced, on full and on small grids."""
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


@pytest.mark.parametrize("name,ks", [("rmat12", (26, 32)), ("er", (10, 12, 14)), ("planted", (12, 20))])
def test_every_setting_gives_the_same_count(ebb, name, ks):
    g = {"rmat12": lambda: graphgen.rmat(12), "er": lambda: graphgen.er(220, 0.6),
         "planted": lambda: graphgen.er_planted(500, 0.2, 2, 40, 60, 7)}[name]()
    want = {}
    for split in (-1, 0, 1, 2, 1 << 14):
        for blocks in (0, 1):
            o = ebb.ebbkc_default_options()
            o.node_split, o.blocks_per_cu = split, blocks
            G = ebb.Graph.from_csr(g, options=o)
            for k in ks:
                print(f"case {name} k={k} split={split} blocks={blocks}", flush=True)
                got = G.count128(k)
                assert got == want.setdefault(k, got), (k, split, blocks)
            G.close()
