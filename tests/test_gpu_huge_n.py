"""Graphs of 1.7e9 vertices, nearly all of them isolated: row numbers past 2^30, whose sums pass 2^31, and
more vertices than one pass of a grid covers."""
import pytest

pytestmark = pytest.mark.gpu

N = 1_700_000_000


@pytest.fixture(scope="module")
def ebb():
    import torch
    import paper_2311_13798_amd as m
    torch.cuda.set_device(0)
    m.load_library()
    return m


def clique_at_the_end(size):
    import torch
    rp = torch.zeros(N + 1, dtype=torch.int32, device="cuda")
    rp[N - size:] = torch.arange(size + 1, dtype=torch.int32, device="cuda") * (size - 1)
    ids = torch.arange(N - size, N, dtype=torch.int32, device="cuda")
    ci = torch.stack([ids[ids != v] for v in ids]).ravel()
    return rp, ci.contiguous()


def test_a_clique_of_the_last_vertices(ebb):
    import torch
    if torch.cuda.mem_get_info()[0] < 120 << 30:
        pytest.skip("needs 120 GiB of free device memory")
    print(f"case n={N}", flush=True)
    rp, ci = clique_at_the_end(6)
    G = ebb.Graph(rp, ci, N)
    assert (G.info.m, G.info.tau, G.info.max_degree) == (15, 4, 5)
    assert [G.count(k) for k in (1, 2, 3, 4, 5, 6, 7)] == [N, 15, 20, 15, 6, 1, 0]
    G.close()
    rp[N] = 31  # more entries than there are
    with pytest.raises(ebb.EbbkcError) as e:
        ebb.Graph(rp, ci, N)
    assert e.value.status == ebb.E_BAD_CSR
    rp[N] = 30
    rp[N - 3] = 2  # offsets that fall
    with pytest.raises(ebb.EbbkcError) as e:
        ebb.Graph(rp, ci, N)
    assert e.value.status == ebb.E_BAD_CSR
    del rp, ci
    torch.cuda.empty_cache()
