"""The stable sort of (key, value) pairs with short and with long tiles, around the lengths where one more
tile begins, against torch's stable sort."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import torch
    import paper_2311_13798_amd as m
    torch.cuda.set_device(0)
    m.load_library()
    return ctypes.CDLL(m.LIB_PATH)


def internal(lib, name, restype, *argtypes):
    f = getattr(lib, name)
    f.restype, f.argtypes = restype, argtypes
    return f


@pytest.mark.parametrize("n", [2, 1023, 1024, 1025, 4095, 4096, 4097, 100_003, 1 << 20, (1 << 20) + 1])
@pytest.mark.parametrize("small_hist", [False, True])
def test_sort(lib, n, small_hist):
    import torch
    print(f"case n={n} small_hist={small_hist}", flush=True)
    vp, i64 = ctypes.c_void_p, ctypes.c_int64
    hist_elems = internal(lib, "_ZN3ebb16radix_hist_elemsElb", i64, i64, ctypes.c_bool)
    scan_elems = internal(lib, "_ZN3ebb14scan_tmp_elemsEl", i64, i64)
    sort = internal(lib, "_ZN3ebb14radix_sort_u64EPmPjS0_S1_liPlS2_P12ihipStream_tb", ctypes.c_int, vp, vp, vp, vp, i64,
                    ctypes.c_int, vp, vp, vp, ctypes.c_bool)
    bits = 10
    keys = torch.from_numpy(np.random.default_rng(n).integers(0, 1 << bits, n)).cuda()
    vals = torch.arange(n, dtype=torch.int32, device="cuda")
    want_k, want_v = torch.sort(keys, stable=True)
    keys2, vals2 = torch.empty_like(keys), torch.empty_like(vals)
    hn = hist_elems(n, small_hist)
    guard = 1 << 62  # behind the histograms: not written
    hist = torch.full((hn + 256,), guard, dtype=torch.int64, device="cuda")
    tmp = torch.empty(scan_elems(hn) + 64, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    assert sort(keys.data_ptr(), vals.data_ptr(), keys2.data_ptr(), vals2.data_ptr(), n, bits, hist.data_ptr(),
                tmp.data_ptr(), None, small_hist) == 0
    torch.cuda.synchronize()
    assert torch.equal(keys, want_k) and torch.equal(vals.long(), want_v)
    assert (hist[hn:] == guard).all()
