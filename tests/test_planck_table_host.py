"""Table form of the FP64 Planck edge integral (``rt_planck.hpp``), built for the host:
against the oracle's extended-precision sum over the arguments of every cell, at the
cells' edges and beyond the table.  Bar: 6 units of roundoff (2^-53) of the integral, the
rounding of its evaluation (12 Horner steps damped by the cell's width, e^-x and two
products)."""
import ctypes as ct
import pathlib
import subprocess

import numpy as np
import pytest

CSRC = pathlib.Path(__file__).resolve().parents[1] / "paper_2203_02293_amd" / "csrc"
SRC = r'''
#include "rt_planck.hpp"
extern "C" void lookup(int n, const double *x, double *out)
{
    alignas(16) static double table[rtk::kPlanckTable];
    rtk::planck_table(table);
    for (int i = 0; i < n; ++i) out[i] = rtk::planck_lookup(x[i], table);
}
// P(x) or Q(x) in long double: sums of their own terms until they no longer count
extern "C" void exact(int n, const double *x, double *out)
{
    for (int i = 0; i < n; ++i) {
        const long double v = x[i];
        long double s = 0.0L;
        if (v >= 3.0L) {
            for (int m = 1; m <= 60; ++m) {
                const long double k = 1.0L / m;
                s -= expl(-m * v) * (((v * k + 3 * k * k) * v + 6 * k * k * k) * v + 6 * k * k * k * k);
            }
        } else {   // integral of t^3 / (e^t - 1): composite Gauss-Legendre, 5 points on 400 panels
            const long double g[] = {0.0L, 0.538469310105683091036314420700208805L, 0.906179845938663992797626878299392965L};
            const long double w[] = {0.568888888888888888888888888888888889L, 0.478628670499366468041291514835638193L,
                                     0.236926885056189087514264040719917363L};
            const long double h = v / 800;
            for (int p = 0; p < 400; ++p)
                for (int q = -2; q <= 2; ++q) {
                    const int a = q < 0 ? -q : q;
                    const long double t = h * (2 * p + 1) + (q < 0 ? -h : h) * g[a];
                    s += w[a] * h * t * t * t / expm1l(t);
                }
        }
        out[i] = (double)s;
    }
}
'''


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("planck")
    (d / "p.cpp").write_text(SRC)
    r = subprocess.run(["hipcc", "-O1", "-std=c++20", "-fPIC", "-shared", f"-I{CSRC.parents[1] / 'include'}",
                        f"-I{CSRC}", str(d / "p.cpp"), "-o", str(d / "p.so")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return ct.CDLL(str(d / "p.so"))


def values(lib, name, x):
    out = np.empty_like(x)
    getattr(lib, name)(ct.c_int(x.size), x.ctypes.data_as(ct.c_void_p), out.ctypes.data_as(ct.c_void_p))
    return out


def test_lookup_matches_exact(lib):
    edges = np.concatenate([[1.0], *(2.0**k * (1 + 0.25 * np.arange(4)) for k in range(6)), [64.0]])
    x = np.concatenate([np.geomspace(1e-6, 700.0, 6000), edges, np.nextafter(edges, 0), np.nextafter(edges, 99)])
    got, ref = values(lib, "lookup", x), values(lib, "exact", x)
    assert np.all(np.abs(got - ref) <= 6 * 2.0**-53 * np.abs(ref))


def test_lookup_ends(lib):
    x = np.array([0.0, 800.0, np.inf, np.nan])
    np.testing.assert_array_equal(values(lib, "lookup", x), 0.0)
