"""The kernel and split that a default tile runs (``default_geometry`` of ``rt_api.hip``, called in
the built library without a GPU): on both sides of its lines, and what it reserves."""
import ctypes as ct

import pytest

from paper_2203_02293_amd import rt

LAYER, DEEP, STREAM = 2, 3, 4
N_CU, LDS = 256, 160 * 1024


class Geometry(ct.Structure):
    _fields_ = [(n, ct.c_int) for n in ("kernel", "K", "PC", "CH", "threads", "blocks")] + [
        ("lanes", ct.c_longlong), ("lds", ct.c_size_t), ("scratch", ct.c_size_t), ("us", ct.c_double)]


class Limits(ct.Structure):
    _fields_ = [("n_cu", ct.c_int), ("lds", ct.c_size_t)]


DEV = Limits(N_CU, LDS)


def _fn(name):
    f = getattr(rt.lib(), name)
    f.restype = Geometry
    return f


def default(C, N, NB, mixed=False, may_deep=True, NG=1):
    return _fn("_ZN3rtk16default_geometryEiiiibiRKNS_12DeviceLimitsE")(C, N, NB, NG, ct.c_bool(may_deep), int(mixed), ct.byref(DEV))


def layer(C, N, NB, mixed=False, NG=1):
    return _fn("_ZN3rtk14solve_geometryEiiiiiiRKNS_12DeviceLimitsEi")(C, N, NB, 0, LAYER, int(mixed), ct.byref(DEV), NG)


def deep(C, N, NB):
    return _fn("_ZN3rtk13deep_geometryEiiiRKNS_12DeviceLimitsE")(C, N, NB, ct.byref(DEV))


# (columns, slabs, lanes, mixed) -> kernel, segments per column.  The measured sides of each line
# stand beside the rules.
LINES = [((42, 12, 7, 0), STREAM, 4), ((162, 40, 30, 0), STREAM, 8), ((2562, 40, 30, 0), STREAM, 2),
         ((2562, 40, 30, 1), STREAM, 2), ((2562, 80, 30, 1), STREAM, 2), ((517, 61, 100, 0), STREAM, 2),
         ((10242, 80, 300, 1), STREAM, 1), ((1, 1, 1, 0), STREAM, 1),
         # 4 to 8 layers: the layer kernel on small grids, one segment on larger ones
         ((20, 5, 30, 0), LAYER, 0), ((20, 5, 30, 1), LAYER, 0), ((162, 5, 100, 0), LAYER, 0), ((2562, 5, 30, 0), STREAM, 1),
         ((20, 3, 30, 0), STREAM, 1), ((20, 12, 30, 0), STREAM, 4),
         # few lanes per column, padded to eight, on large grids
         ((10242, 40, 2, 0), LAYER, 0), ((10242, 120, 3, 1), LAYER, 0), ((30000, 120, 1, 1), LAYER, 0), ((600, 40, 3, 0), STREAM, 8),
         # level sums that fill the LDS
         ((10242, 120, 10, 1), LAYER, 0), ((20000, 120, 5, 1), LAYER, 0), ((1000, 300, 30, 0), STREAM, 4),
         # workgroups of eight wavefronts that do not all run at once
         ((162, 20, 100, 0), STREAM, 4), ((100, 20, 100, 0), STREAM, 8),
         # deep columns
         ((1, 4096, 30, 0), DEEP, 0), ((16, 1000, 30, 1), DEEP, 0), ((16, 40, 30, 1), DEEP, 0), ((64, 87, 30, 0), STREAM, 16),
         ((64, 88, 30, 0), DEEP, 0), ((3, 47, 40, 0), STREAM, 8), ((3, 48, 40, 0), DEEP, 0),
         # FP64 above a quarter of the compute units, or 3200 lanes: by the layers
         ((96, 2000, 30, 0), STREAM, 16), ((65, 4096, 30, 0), DEEP, 0), ((16, 1000, 300, 0), STREAM, 8), ((16, 4096, 300, 0), DEEP, 0),
         ((11, 400, 300, 0), STREAM, 8), ((11, 1000, 300, 0), DEEP, 0), ((40, 4096, 100, 0), DEEP, 0), ((128, 1000, 100, 0), STREAM, 8)]


@pytest.mark.parametrize("shape,kernel,S", LINES, ids=["x".join(map(str, c[0])) for c in LINES])
def test_lines(shape, kernel, S):
    g = default(*shape)
    assert g.kernel == kernel
    if kernel == STREAM:
        assert g.PC == S


def test_gpu_shapes_reach_every_split():
    """What the GPU tests of the default tile run: one segment and every split by the stream kernel, and
    AUTO on both sides of its FP64 line."""
    from tests.test_gpu_stream import CASES, SEGMENTS, columns
    for mixed in (False, True):
        got = [default(C, N, NB, mixed, False) for NB, N, C in SEGMENTS]
        assert {g.PC for g in got if g.kernel == STREAM} == {1, 2, 3, 4, 8, 16}
        assert {g.kernel for g in got} == {LAYER, STREAM}
    for NB, N in CASES:
        g = default(columns(NB), N, NB, False, False)
        assert (g.kernel, g.PC) == (STREAM, 1), (NB, N)
    for shape, kernel in (((64, 87, 30), STREAM), ((64, 88, 30), DEEP), ((65, 88, 30), STREAM), ((3, 47, 40), STREAM),
                          ((3, 48, 40), DEEP), ((32, 89, 100), DEEP)):
        assert default(*shape).kernel == kernel, shape


def test_bench_names_the_kernels_it_runs():
    """bench.py's workloads run the kernels that it names: the stream kernel for a default tile, the
    deep path's four launches for a deep column of up to 64 lanes."""
    import bench
    for C, N, NB, NG in ((2562, 40, 30, 1), (2562, 80, 30, 1), (2562, 40, 600, 20), (2562, 80, 600, 20), (10242, 80, 300, 1)):
        for mixed in (False, True):
            assert default(C, N, NB, mixed, NG=NG).kernel == STREAM
    assert default(1, 4096, 30).kernel == DEEP and default(16, 1000, 30, True).kernel == DEEP
    assert bench.KERNEL_NAMES[2] == "k_solve_stream" and bench.KERNEL_NAMES[3] == "k_cascade_*"


def test_reservation_is_the_former_kernels():
    """A default tile asks for the work buffer that the layer or deep kernel asked for at this size, so
    what fitted a budget or the static buffer still does."""
    for C in (1, 3, 60, 128, 129, 777, 2562, 20000):
        for N in (1, 4, 39, 40, 87, 200, 1000, 4096):
            for NB, NG in ((1, 1), (7, 1), (30, 1), (64, 1), (65, 1), (300, 1), (768, 3)):
                for mixed in (False, True):
                    g, former = default(C, N, NB, mixed, NG=NG), layer(C, N, NB, mixed, NG)
                    if N >= 40 and 2 * C <= N_CU:
                        former = deep(C, N, NB)
                    assert (g.threads > 0) == (former.threads > 0)
                    assert g.scratch == former.scratch and g.lds <= LDS, (C, N, NB, NG, mixed)


def test_tuned_entries_follow_the_line():
    """The autotuner's table, applied to shapes around its entries, sends no FP64 request to the other
    side of AUTO's line between the deep and the stream kernel."""
    for NB in (30, 100, 300):
        for C in (1, 8, 20, 40, 64, 65, 100, 128, 129):
            for N in (40, 60, 100, 150, 250, 300, 400, 1000, 4096):
                kernel, K = rt.tuned_launch(NB, rt.RT_FP64, C, N)
                if kernel != rt.RT_KERNEL_AUTO:
                    assert K == 0 and (kernel == rt.RT_KERNEL_DEEP) == (default(C, N, NB).kernel == DEEP), (C, N, NB, kernel)
