"""Drive the host build of the wavefront kernels (``wave_build.py``) on a workload dict.
Test infrastructure only."""
import ctypes as ct

import numpy as np

from . import wave_build as _build
from .run import Args, _Guarded, _args

_L = None
NCU, LDS = 256, 160 * 1024


def lib():
    global _L
    if _L is None:
        _L = ct.CDLL(str(_build.build()))
        _L.emu_deep_scratch.restype = ct.c_longlong
    return _L


def stream_geometry(C, N, NB, NG=1, mixed=False, ncu=NCU, lds=LDS):
    v = (ct.c_longlong * 7)()
    lib().emu_stream_geometry(C, N, NB, NG, int(mixed), ncu, lds, v)
    return dict(K=v[0], S=v[1], LPT=v[2], threads=v[3], blocks=v[4], lds=v[5], scratch=v[6])


def _shape(w):
    NG = int(w.get("n_gauss", 1)) if w.get("gauss_w") is not None else 1
    sub = w.get("T_center") is not None and w.get("sublayer", False)
    return w["n_cols"], (2 if sub else 1) * w["n_layers"], w["n_bins"] * NG, NG


def solve_stream(w, mixed, opts=None, ncu=NCU, lds=LDS, per_bin=True):
    C, N, NB, NG = _shape(w)
    g = stream_geometry(C, N, NB, NG, mixed, ncu, lds)
    buf = _Guarded(g["scratch"])
    out, a, keep = _args(w, opts, per_bin, buf.ptr)
    rc = lib().emu_stream_solve(ct.byref(a), int(mixed), ncu, lds)
    assert rc == 0, (rc, g)
    return out, g


def solve_stream_batch(works, mixed, opts=None, ncu=NCU, lds=LDS):
    """Several requests in one batched launch; their outputs."""
    bufs, outs, reqs, keep = [], [], (Args * len(works))(), []
    for k, w in enumerate(works):
        C, N, NB, NG = _shape(w)
        bufs.append(_Guarded(stream_geometry(C, N, NB, NG, mixed, ncu, lds)["scratch"]))
        out, a, kp = _args(w, opts, True, bufs[-1].ptr)
        reqs[k] = a
        outs.append(out)
        keep.append(kp)
    rc = lib().emu_stream_batch(reqs, len(works), int(mixed), ncu, lds, 0)
    assert rc == 0, rc
    return outs


def batch_launches(C, N, NB, mixed, ncu=NCU, lds=LDS):
    """Whether a served request of this shape launches: its kernels' LDS against the
    limits they are set up for (nothing is run)."""
    a = Args(C=C, N=N, NB=NB, NG=1)
    return lib().emu_stream_batch(ct.byref(a), 1, int(mixed), ncu, lds, 1) == 0


def solve_cascade(w, mixed, opts=None, ncu=NCU, lds=LDS, per_bin=True):
    C, N, NB, NG = _shape(w)
    buf = _Guarded(lib().emu_deep_scratch(C, N, NB, ncu, lds))
    out, a, keep = _args(w, opts, per_bin, buf.ptr)
    rc = lib().emu_cascade_solve(ct.byref(a), int(mixed), ncu, lds)
    assert rc == 0, rc
    return out
