"""The library without a GPU: host arithmetic of the launches, through internal functions (where each width
class's root ranges start in one task list of up to 2^32 entries, the frames of deep searches, the workgroups
of the peel, the bytes of task lists and of preparing), and its kernels."""
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


@pytest.mark.parametrize("m", [1, 1024, 1025, 100_000, (1 << 20) - 1, 1 << 20, 1 << 30])
@pytest.mark.parametrize("resident", [0, 1, 20, 38, 64, 100, 128, 256])
def test_the_peel_fits_the_device(m, resident):
    # its workgroups wait for each other: no more than run side by side
    grid = internal("_ZN3ebb9peel_gridEll", ctypes.c_int64, ctypes.c_int64, ctypes.c_int64)(m, resident)
    assert 1 <= grid <= max(1, resident)
    assert grid == max(1, min(resident, 128 if m >= 1 << 20 else 64, ((m + 1023) // 1024 + 1) // 2))


@pytest.mark.parametrize("grid,room,tried", [(128, 128, [128]), (128, 100, [128, 32]), (64, 5, [64, 16, 4]),
                                             (64, 1, [64, 16, 4, 1]), (3, 1, [3, 1]), (2, 1, [2, 1]), (1, 1, [1])])
def test_a_peel_without_room_starts_over_with_fewer(grid, room, tried):
    CB = ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_void_p, ctypes.c_int64)
    f = internal("_ZN3ebb13peel_attemptsElPFiPvlES0_", ctypes.c_int, ctypes.c_int64, CB, ctypes.c_void_p)
    seen = []

    def attempt(_, g):
        seen.append(g)
        return 0 if g <= room else 1

    assert f(grid, CB(attempt), None) == 0 and seen == tried
    # an error is final, and so is one workgroup that gives up
    assert f(grid, CB(lambda _, g: ebb.E_OOM), None) == ebb.E_OOM
    assert f(grid, CB(lambda _, g: 1), None) == ebb.E_HIP


@pytest.mark.parametrize("slots,tasks", [(1, 1), (10**6, 10**6), (21_000_000, 1 << 20), (20_900_000, 100_000), (1, 6_000_000)])
def test_sorting_few_tasks_needs_no_more_scratch_than_many(slots, tasks):
    # the task list of a count that may not allocate: 12 bytes a slot, 40 a task, and one histogram of 256
    # for every 4,096 tasks (2 KB); shorter tiles only where there is room for their histograms
    rnd = lambda b: (b + 255) // 256 * 256
    scan = lambda n: (n + 2047) // 2048 + 65
    hist = 256 * ((tasks + 4095) // 4096) + 1
    want = (rnd(4 * slots) + rnd(8 * (slots + 1)) + rnd(8 * scan(slots + 1)) + 4 * rnd(8 * tasks) + 2 * rnd(4 * tasks) +
            rnd(8 * hist) + rnd(8 * scan(hist)) + 4096)
    f = internal("_ZN3ebb10task_bytesEllb", ctypes.c_size_t, ctypes.c_int64, ctypes.c_int64, ctypes.c_bool)
    assert f(slots, tasks, True) == want <= f(slots, tasks, False)


def test_every_kernel_is_compiled_once():
    # two copies of a kernel would each have binomial tables of their own, of which one is filled; a code
    # object names a kernel's descriptor twice, in its two symbol tables
    import re
    data = open(ebb.LIB_PATH, "rb").read()
    names = {n for n in re.findall(rb"_Z[A-Za-z0-9_]+\.kd", data) if b"_GLOBAL__N_1" not in n}
    assert sum(b"k_search" in n for n in names) >= 16
    assert [n for n in names if data.count(n + b"\0") != 2] == []


def test_prepare_takes_184_bytes_an_edge():
    # beside the triangle incidence; arrays of one entry a vertex and the sort's histograms come on top
    f = internal("_ZN3ebb13prepare_sizesEilPNS_8SlabSizeE", None, ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p)
    size = (ctypes.c_size_t * 2)()
    n, m = 1 << 20, 1 << 29
    f(n, 2 * m, size)
    assert 68 * m <= size[0] <= 68 * m + 16 * n + 4096
    assert size[0] + size[1] <= 188 * m
    f(1, 0, size)
    assert 0 < size[0] + size[1] < 4 << 20
