"""Host arithmetic of the launches (no GPU calls), through the library's internal functions: where each
width class's root ranges start in one task list of up to 2^32 entries, and the frames of deep searches."""
import ctypes
import math
import os

import pytest

import paper_2311_13798_amd as ebb

pytestmark = pytest.mark.skipif(not os.path.exists(ebb.LIB_PATH), reason="libebbkc.so not built")

MAX_W = 4


def internal(name, restype, *argtypes):
    f = getattr(ctypes.CDLL(ebb.LIB_PATH), name)
    f.restype, f.argtypes = restype, argtypes
    return f


def root_ranges(c, l0, log_threshold):
    """Root ranges of a slot of c vertices, by class of the vertices a range can use."""
    lb = lambda n, r: math.lgamma(n + 1) - math.lgamma(r + 1) - math.lgamma(n - r + 1)
    if not (l0 >= 4 and c >= l0 + 8 and lb(c, l0) > log_threshold):
        return [0] * MAX_W
    n, x0, acc = [0] * MAX_W, 0, 0.0
    for x in range(c - l0 + 1):
        acc += math.exp(lb(c - 1 - x, l0 - 1) - lb(c - 1, l0 - 1))
        if acc >= 0.999 or x == c - l0:
            n[(c - x0 + 63) // 64 - 1] += 1
            x0, acc = x + 1, 0.0
    return n


# the second: ranges of the one-word class alone reach 2^31, the third: their sum is refused
@pytest.mark.parametrize("sizes", [{200: 3, 100: 5, 40: 7}, {60: 180_000_000, 100: 10_000_000, 200: 1_000},
                                   {256: 90_000_000}])
def test_classes_start_where_the_ones_before_end(sizes):
    f = internal("_ZN3ebb11plan_rangesERK10SizeCountsidPl", ctypes.c_int64, ctypes.c_void_p, ctypes.c_int, ctypes.c_double,
                 ctypes.c_void_p)
    l0, thr = 4, math.log(1000.0)
    n = (ctypes.c_int64 * 257)()
    want = [0] * MAX_W
    for c, slots in sizes.items():
        n[c] = slots
        for w, r in enumerate(root_ranges(c, l0, thr)):
            want[w] += slots * r
    first = (ctypes.c_int64 * MAX_W)()
    total = f(n, l0, thr, first)
    assert total == (sum(want) if sum(want) < 2**32 else -1)
    if total >= 0:
        assert list(first) == [sum(want[:w]) for w in range(MAX_W)]



@pytest.mark.parametrize("waves", [(4096, 4096, 3072, 2048), (2048, 2048, 2048, 2048), (4, 4, 4, 4), (1024, 8192, 1024, 512),
                                   (512, 512, 4096, 256)])
def test_deep_frames_serve_every_class(waves):
    # a wave's frames start at its number times the class's frame size, whatever class is launched
    frame = internal("_ZN3ebb18search_frame_bytesEi", ctypes.c_size_t, ctypes.c_int)
    total = internal("_ZN3ebb16frames_for_wavesEPKl", ctypes.c_size_t, ctypes.c_void_p)((ctypes.c_int64 * MAX_W)(*waves))
    per_wave = 124  # GLOBAL_FRAMES
    for w in range(MAX_W):
        assert total >= waves[w] * per_wave * frame(w + 1), w + 1


def test_deep_frames_of_an_unknown_device():
    f = internal("_ZN3ebb16frames_for_wavesEPKl", ctypes.c_size_t, ctypes.c_void_p)
    assert f((ctypes.c_int64 * MAX_W)(4, -1, 4, 4)) == 0
