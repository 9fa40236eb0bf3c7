"""An FP64 layer's coefficients as segments keep them for their second elimination
(``store_layer``, ``load_layer`` of ``rt_physics.hpp``), built for the host: the two that are not
the largest are kept bit for bit; the largest, 1 - p - q (at least 1/3), is off from
``layer_terms``'s formulas in long double by no more than those two are and two roundings of
numbers up to 1, and 1 - r = t + A by no more than t and A are and one more (u = 2^-53, half
of it per rounding; the long double formulas round their input, at most as much again)."""
import ctypes as ct
import pathlib
import subprocess

import numpy as np
import pytest

CSRC = pathlib.Path(__file__).resolve().parents[1] / "paper_2203_02293_amd" / "csrc"
SRC = r'''
#include "rt_physics.hpp"
using namespace rtk;
// out [n][12]: t, r, 1 - r, A of the layer, as kept, in long double
extern "C" void layers(int n, const double *dtau, const double *w0, const double *g0, double *out)
{
    Opts o{};
    o.improved = o.noniso = o.e_clamp = 1;
    for (int i = 0; i < n; ++i) {
        uint32_t fl = 0;
        const double w = w0[i], g = g0[i], E = efit_exact(w, g, o, fl);
        Layer<double> L;
        layer_terms<double>(dtau[i], w, g, E, 1.0 - w, E - w, 1.0 - w * g, false, 0, 0, 0, false, 0, 0, 1, 1, false, 1.5, L);
        double *q = out + 12 * i;
        q[0] = L.t, q[1] = L.r, q[2] = L.omr, q[3] = L.A;
        load_layer(store_layer(L.t, L.r, L.A), q[4], q[5], q[6], q[7]);
        // layer_terms's own s and optical path, without further rounding
        const double s2 = (E - w) * (1.0 / (E * (1.0 - w * g))), is = s2 > 0.0 ? rsqrt_pos(s2) : 0.0, sd = s2 * is;
        const long double s = sd, kap = 2 * (E * (1.0 - w * g)), u = (double)((double)kap * sd) * dtau[i];
        const long double T = expl(-u), omT = -expm1l(-u), p = s > 0 ? omT / s : kap * dtau[i];
        const long double zp = (1 + s) / 2, zm = (1 - s) / 2, qq = p * (1 + T), id = 1 / (1 + zm * zm * qq);
        q[8] = T * id, q[9] = zp * zm * qq * id, q[10] = (zp + zm * T * T) * id, q[11] = omT * (zp - zm * T) * id;
    }
}
'''


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("store")
    (d / "p.cpp").write_text(SRC)
    r = subprocess.run(["hipcc", "-O1", "-std=c++20", "-fPIC", "-shared", f"-I{CSRC.parents[1] / 'include'}",
                        f"-I{CSRC}", str(d / "p.cpp"), "-o", str(d / "p.so")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return ct.CDLL(str(d / "p.so"))


def test_kept_layers_are_whole(lib):
    rng = np.random.default_rng(5)
    n = 40000
    dtau = np.exp(rng.uniform(np.log(1e-14), np.log(1e4), n))
    w0 = np.where(rng.random(n) < 0.5, rng.uniform(0.0, 1.0, n), 1.0 - np.exp(rng.uniform(np.log(1e-12), 0.0, n)))
    g0 = rng.uniform(-0.99, 0.99, n)
    w0[::50], w0[1::50], dtau[2::50], dtau[3::50] = 0.0, 1.0, 0.0, 1e8
    w0[4::50], g0[4::50] = 0.05, 1.0 - 1e-16 * rng.integers(2, 9, n // 50)   # s next to 1, r next to 0
    out = np.empty((n, 12))
    lib.layers(ct.c_int(n), *(a.ctypes.data_as(ct.c_void_p) for a in (dtau, w0, g0, out)))
    own, kept, ref = out[:, 0:4], out[:, 4:8], out[:, 8:12]
    three = [0, 1, 3]   # t, r, A: all but the largest, up to the sign of a rounded zero
    top = np.argmax(own[:, three], axis=1)
    whole = np.abs(own[:, three]) == kept[:, three]
    whole[np.arange(n), top] = True
    assert np.all(whole)
    u = 2.0**-53
    err, err_kept = np.abs(own - ref), np.abs(kept - ref)
    left = np.take_along_axis(err_kept[:, three], top[:, None], 1)[:, 0]
    others = err[:, three].sum(1) - np.take_along_axis(err[:, three], top[:, None], 1)[:, 0]
    assert np.all(left <= others + 2 * u)
    assert np.all(err_kept[:, 2] <= err_kept[:, 0] + err_kept[:, 3] + 2 * u)
