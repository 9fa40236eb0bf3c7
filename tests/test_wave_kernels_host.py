"""The wavefront kernels (``csrc/rt_stream.hip``, ``csrc/rt_cascade.hip``) run on the CPU
through their host build (``tests/host_emu/wave_build.py``: a fiber per GPU thread,
wavefront and workgroup barriers, work buffer and LDS each ending at an inaccessible
page) against the oracle.  The compute-unit count moves the split into segments.
Host arithmetic differs from the device's in the reciprocal only, so the GPU parity bars
apply."""
import numpy as np
import pytest

import oracle as O
from paper_2203_02293_amd import synth
from tests.parity import FLOOR, FLOOR_BIN, errors

run = pytest.importorskip("tests.host_emu.wave_run")


def work(C, N, NB, seed, cloud="night", **kw):
    mu = np.linspace(-0.4, 0.95, C) if C > 1 else np.array([0.6])
    return synth.make(synth.Spec(name="w", g_level=3, n_layers=N, n_bins=NB, cloud=cloud, seed=seed, **kw),
                      n_cols=C, mu_star=mu)


def compare(w, out, mixed, opts=None):
    ref = (O.solve_sublayer if w.get("sublayer", False) else O.solve)(w, opts, per_bin=True, extended=True)
    e = errors(out, ref, w["p_iface"], floor=FLOOR[int(mixed)], floor_bin=FLOOR_BIN[int(mixed)])
    bad = {k: v for k, v in e.items() if not v <= (1e-5 if mixed else 1e-10)}
    assert not bad, bad
    np.testing.assert_array_equal(out["flags"], ref["flags"])


# (columns, layers, lanes, compute units) -> segments per column: padding of 8 to 64 lanes, wide
# columns, ragged last workgroups, odd and uneven segments
STREAM = [((9, 3, 1, 1), 1), ((55, 11, 7, 1), 1), ((30, 16, 16, 1), 1), ((7, 17, 33, 1), 1), ((4, 9, 65, 1), 1), ((3, 8, 130, 1), 1),
          ((37, 8, 5, 1), 2), ((21, 9, 16, 1), 2), ((6, 17, 33, 1), 2), ((4, 8, 65, 2), 2), ((6, 23, 65, 2), 2),
          ((29, 17, 5, 1), 3), ((15, 13, 9, 1), 3), ((7, 17, 30, 1), 3), ((4, 13, 100, 2), 3),
          ((1, 7, 5, 1), 4), ((5, 9, 30, 256), 4), ((7, 13, 7, 256), 4), ((2, 19, 100, 256), 4),
          ((3, 23, 30, 256), 8), ((9, 25, 5, 256), 8), ((1, 21, 70, 256), 8),
          ((3, 57, 7, 256), 16), ((2, 61, 30, 256), 16)]


@pytest.mark.parametrize("mixed", [False, True], ids=["fp64", "mixed"])
@pytest.mark.parametrize("shape,S", STREAM, ids=["x".join(map(str, s)) for s, _ in STREAM])
def test_stream(shape, S, mixed):
    C, N, NB, ncu = shape
    w = work(C, N, NB, 40 + N)
    out, g = run.solve_stream(w, mixed, ncu=ncu)
    assert g["S"] == S
    compare(w, out, mixed)


@pytest.mark.parametrize("mixed", [False, True], ids=["fp64", "mixed"])
def test_stream_grids_and_modes(mixed):
    from tests.test_gpu_parity import edge_workload
    w = synth.make_sublayer(synth.Spec(name="s", g_level=3, n_layers=11, n_bins=5, cloud="night", seed=81), n_cols=3)
    compare(w, run.solve_stream(w, mixed)[0], mixed)
    for NB, NG in ((5, 4), (9, 8)):   # narrow and wide columns of Gaussian points
        w = synth.make_kdist(synth.Spec(name="k", g_level=3, n_layers=21, n_bins=NB, cloud="night", seed=82), n_cols=2, n_gauss=NG)
        compare(w, run.solve_stream(w, mixed)[0], mixed)
    if not mixed:
        w = edge_workload()
        for opts in (O.Options(), O.Options(improved=0), O.Options(noniso=0)):
            compare(w, run.solve_stream(w, mixed, opts=opts)[0], mixed, opts)


@pytest.mark.parametrize("mixed", [False, True], ids=["fp64", "mixed"])
@pytest.mark.parametrize("NB", [7, 70])
def test_stream_batch_equals_single(NB, mixed):
    """Requests of other sizes in one batched launch: each its own single launch's results."""
    works = [work(C, N, NB, 50 + C) for C, N in ((3, 23), (1, 21), (5, 30))]
    for w, out in zip(works, run.solve_stream_batch(works, mixed)):
        one = run.solve_stream(w, mixed)[0]
        for k in one:
            if k != "status":
                np.testing.assert_array_equal(out[k], one[k], err_msg=k)


@pytest.mark.parametrize("mixed", [False, True], ids=["fp64", "mixed"])
def test_served_wide_columns_launch_within_lds(mixed):
    """A served request of wide columns launches at every layer count: neither of its two
    kernels asks for more LDS than it is set up for, also where the solve's fills it."""
    full = 0
    for C, NB in ((64, 100), (129, 100), (129, 300), (1, 65), (700, 768)):
        for N in (*range(1, 4096, 17), *range(3800, 4097)):
            g = run.stream_geometry(C, N, NB, mixed=mixed)
            full += g["lds"] > run.LDS - 1024
            if g["threads"]:
                assert run.batch_launches(C, N, NB, mixed), (C, N, NB, g)
    assert full


# (columns, layers, lanes, compute units): parts of 6 slabs, ragged last segments and parts, 8 to 64
# lanes, several wavefronts per segment
CASCADE = [(1, 300, 6, 4), (3, 77, 7, 4), (2, 61, 30, 8), (1, 41, 64, 8), (5, 19, 9, 2), (2, 130, 33, 4)]


@pytest.mark.parametrize("mixed", [False, True], ids=["fp64", "mixed"])
@pytest.mark.parametrize("shape", CASCADE, ids=["x".join(map(str, s)) for s in CASCADE])
def test_cascade(shape, mixed):
    C, N, NB, ncu = shape
    w = work(C, N, NB, 60 + N)
    compare(w, run.solve_cascade(w, mixed, ncu=ncu), mixed)


@pytest.mark.parametrize("mixed", [False, True], ids=["fp64", "mixed"])
def test_cascade_grids(mixed):
    w = synth.make_sublayer(synth.Spec(name="s", g_level=3, n_layers=32, n_bins=5, cloud="night", seed=83), n_cols=2)
    compare(w, run.solve_cascade(w, mixed, ncu=2), mixed)
    w = synth.make_kdist(synth.Spec(name="k", g_level=3, n_layers=40, n_bins=5, cloud="night", seed=84), n_cols=2, n_gauss=4)
    compare(w, run.solve_cascade(w, mixed, ncu=2), mixed)
