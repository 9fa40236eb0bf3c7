"""GPU parity of the wavefront-per-lanes solve, the default tile's: lane counts on both sides of every padding step (8,
16, 32, 64 lanes per column, several wavefronts per column), layer counts around
its chunks of eight and its pairs, ragged last workgroups, Gaussian points and
the sub-layer grid, on grids that fill the chip (one segment per column) and on
smaller ones (2 to 16 segments).  Bars as in ``test_gpu_parity.py``: FP64 <= 1e-10, mixed <=
1e-5 against the oracle's extended-precision build on a sample of columns."""
import numpy as np
import pytest

import oracle as O
from paper_2203_02293_amd import synth
from tests.parity import FLOOR, FLOOR_BIN, TOL, assert_close, subset
from tests.test_gpu_parity import rt, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def columns(lanes: int) -> int:
    """Columns that give a little more than six wavefronts per compute unit."""
    per = max(1, 64 // max(8, 1 << (lanes - 1).bit_length())) if lanes <= 64 else 1
    waves = -(-lanes // 64) if lanes > 64 else 1
    return (1536 * per) // waves + 3


CASES = [(1, 1), (8, 2), (9, 7), (16, 8), (17, 9), (32, 16), (33, 10), (64, 5), (65, 8), (128, 3), (130, 17), (511, 4)]


def run(rt, torch, w, cols, sub=False, gw=None):
    ws = subset(w, cols)
    ref = (O.solve_sublayer if sub else O.solve)(ws, per_bin=True, extended=True)
    s = rt.Solver(w["lambda_edges"], w["F_star"], gauss_weights=gw)
    for prec in (rt.RT_FP64, rt.RT_MIXED):
        inp = rt.to_device(w)
        out = s.solve(inp, precision=prec, per_bin=True, kernel=rt.RT_KERNEL_LAYER, cols_per_block=0)
        torch.cuda.synchronize()
        res = {k: v.cpu().numpy() for k, v in out.items()}
        res["flags"] = res["flags"].view(np.uint32)
        e = assert_close(res, ref, ws["p_iface"], TOL[prec], floor=FLOOR[prec], floor_bin=FLOOR_BIN[prec], cols=cols)
        print(f"  precision={prec} errors={e}", flush=True)
        np.testing.assert_array_equal(res["flags"][cols], ref["flags"])
    s.close()


@pytest.mark.parametrize("NB,N", CASES)
def test_stream_lane_and_layer_edges(rt, torch, NB, N):
    C = columns(NB)
    print(f"\n[stream] {C}x{N}x{NB}", flush=True)
    w = synth.make(synth.Spec(name="st", g_level=4, n_layers=N, n_bins=NB, cloud="night", seed=700 + NB), n_cols=C)
    run(rt, torch, w, np.unique(np.array([0, 1, C // 2, C - 2, C - 1])))


@pytest.mark.parametrize("NB,NG", [(5, 4), (30, 20)])
def test_stream_gauss_points(rt, torch, NB, NG):
    C = columns(NB * NG)
    w = synth.make_kdist(synth.Spec(name="st", g_level=4, n_layers=9, n_bins=NB, cloud="night", seed=731),
                         n_cols=C, n_gauss=NG)
    run(rt, torch, w, np.array([0, C // 2, C - 1]), gw=w["gauss_w"])


def test_stream_sublayer_grid(rt, torch):
    C = columns(30)
    w = synth.make_sublayer(synth.Spec(name="st", g_level=4, n_layers=5, n_bins=30, cloud="night", seed=741), n_cols=C)
    run(rt, torch, w, np.array([0, C // 2, C - 1]), sub=True)


# (lanes, layers, columns) by segments per column: the fewest layers of each rule, uneven
# splits, ragged last workgroups, a segment's groups within and across wavefronts, wide
# columns; then grids whose size sets the number
SEGMENTS = [(7, 57, 3), (16, 56, 5), (30, 61, 2),          # 16
            (30, 20, 3), (30, 41, 5), (64, 23, 2), (65, 55, 2), (300, 21, 1), (5, 25, 9),   # 8
            (30, 8, 5), (7, 12, 11), (100, 19, 2),         # 4
            (30, 7, 3), (9, 6, 9),                         # 3
            (30, 4, 3), (8, 5, 17),                        # 2
            (30, 40, 1500), (30, 41, 1800), (30, 43, 2501), (100, 11, 700)]


@pytest.mark.parametrize("NB,N,C", SEGMENTS)
def test_stream_segments(rt, torch, NB, N, C):
    print(f"\n[stream] {C}x{N}x{NB}", flush=True)
    w = synth.make(synth.Spec(name="sg", g_level=4, n_layers=N, n_bins=NB, cloud="night", seed=760 + N), n_cols=C)
    run(rt, torch, w, np.unique(np.array([0, C // 2, C - 1])))


@pytest.mark.parametrize("NB,NG,N", [(5, 4, 21), (9, 8, 13)])
def test_stream_segments_gauss_points(rt, torch, NB, NG, N):
    w = synth.make_kdist(synth.Spec(name="sg", g_level=4, n_layers=N, n_bins=NB, cloud="night", seed=781),
                         n_cols=5, n_gauss=NG)
    run(rt, torch, w, np.arange(5), gw=w["gauss_w"])


def test_stream_segments_sublayer_grid(rt, torch):
    w = synth.make_sublayer(synth.Spec(name="sg", g_level=4, n_layers=23, n_bins=30, cloud="night", seed=791), n_cols=5)
    run(rt, torch, w, np.arange(5), sub=True)
