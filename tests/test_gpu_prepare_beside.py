"""Graphs prepared while other streams keep the device busy: the truss order's workgroups wait for each
other, so they have to find room beside counts that fill the device and beside other preparations."""
import threading

import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ebb():
    import torch
    import paper_2311_13798_amd as m
    torch.cuda.set_device(0)
    m.load_library()
    return m


@pytest.fixture(scope="module")
def graphs():
    gs = [graphgen.rmat(12), graphgen.er(2000, 0.02), graphgen.complete(90), graphgen.er_planted(900, 0.05, 2, 15, 30, 3)]
    return [(g, oracle.truss_levelsync(g), oracle.edge_support(g)) for g in gs]


def prepare_and_check(ebb, graphs, stream):
    for g, tr, sup in graphs:
        h = ebb.ebbkc_prepare(np.ascontiguousarray(g.row_ptr, np.int32), np.ascontiguousarray(g.col_idx, np.int32), g.n,
                              g.nnz, None, stream)
        info = ebb.ebbkc_info_get(h)
        assert (info.tau, info.rounds) == (tr["tau"], tr["rounds"])
        for which, want in ((ebb.ARR_SUPPORT, sup), (ebb.ARR_LEVEL, tr["level"]), (ebb.ARR_RANK, tr["rank"])):
            out = np.zeros(g.m, np.int32)
            ebb.ebbkc_export(h, which, out, stream)
            assert (out == want).all()
        ebb.ebbkc_destroy(h)


def run(threads):
    errors = []

    def guarded(f):
        def body():
            try:
                f()
            except BaseException as e:  # reported by the test's own thread
                errors.append(e)
        return body

    ts = [threading.Thread(target=guarded(f)) for f in threads]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    if errors:
        raise errors[0]


def test_beside_a_count(ebb, graphs):
    import torch
    print("case prepare beside counts", flush=True)
    G = ebb.Graph.from_csr(graphgen.er(400, 0.6))
    want = G.count(8)
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    stop = threading.Event()

    def count():
        while not stop.is_set():
            assert ebb.ebbkc_count(G.handle, 8, streams[0].cuda_stream) == want

    def prepare():
        try:
            for _ in range(3):
                prepare_and_check(ebb, graphs, streams[1].cuda_stream)
        finally:
            stop.set()

    run([count, prepare])
    G.close()


def test_beside_other_preparations(ebb, graphs):
    import torch
    print("case three prepare at once", flush=True)
    streams = [torch.cuda.Stream() for _ in range(3)]
    torch.cuda.synchronize()
    run([lambda s=s: prepare_and_check(ebb, graphs * 3, s.cuda_stream) for s in streams])
