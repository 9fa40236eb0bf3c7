// rt_optics.hip -- optical properties of the slabs: the step before the solve.
//
// Paper: Deitrick et al., "The THOR+HELIOS general circulation model"
// (arXiv 2203.02293): Section 2.1.3 (pre-mixed k-tables over temperature and
// log pressure, Gaussian points per bin), Section 2.2.3 (mixing of gas and
// condensate scattering into w0 and g0), Section 2.2.1 (sub-layer values are
// means of centre and interface values), Appendix C (Rayleigh cross
// sections of H2 and He).
//
// The outputs are three doubles per cell and (bin, Gaussian point), and the time that
// writing them takes is the floor.  A workgroup takes a run of slabs of one column, a
// thread one output of each, the point index fastest: consecutive lanes read
// consecutive k-table entries of the same (T, p) cell and write consecutive outputs, a
// slab's row is written at once, and neighbouring columns share an XCD.  The first
// wavefront finds the k-table brackets of all its levels, one lane each; a bin's
// constants stay in registers over the slabs, and a sub-layer takes the values of its
// upper level from the slab below it.  2562 columns, 40 layers on the sub-layer grid, 600
// outputs (2.95 GB): 630 us; a wavefront per cell, which evaluated every level twice,
// took 1070.  FP64 throughout.
#include "rt_internal.hpp"

#include <algorithm>
#include <cmath>
#include <vector>

namespace rtk {
namespace {

__device__ __forceinline__ int bracket(const double *grid, int n, double &x)
{
    // last i with grid[i] <= x, in [0, n-2]; x held inside the grid
    if (x < grid[0]) x = grid[0];
    if (x > grid[n - 1]) x = grid[n - 1];
    int lo = 0, hi = n - 2;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (grid[mid] <= x) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// A (T, p) point's k-table cell: lower corner (i, j) and weights (t, u).
struct Cell {
    int i, j;
    double t, u;
};

__device__ __forceinline__ Cell cell_at(const OpticsArgs &a, double T, double p)
{
    double x = T, y = log10(p);
    Cell q;
    q.i = bracket(a.temp, a.nT, x);
    q.j = bracket(a.log10p, a.nP, y);
    q.t = (x - a.temp[q.i]) / (a.temp[q.i + 1] - a.temp[q.i]);
    q.u = (y - a.log10p[q.j]) / (a.log10p[q.j + 1] - a.log10p[q.j]);
    return q;
}

constexpr int kOpticsThreads = 768;   // workgroup size bound: the most lanes of a column
constexpr int kOpticsColumns = 1 << 20;   // of one z of the grid (its threads along x: below 2^32)
constexpr int kOpticsLevels = 64;   // of a workgroup: a lane of its first wavefront each

// L slabs of a column per workgroup, an output of each per thread; ONE: a single wavefront
// takes them all, 64 at a time
template <bool SUB, bool ONE>
__global__ void __launch_bounds__(kOpticsThreads) k_optics(const OpticsArgs a, const int L)
{
    // each XCD takes a run of the columns of this blockIdx.z; of a few columns, another one
    // for the next slabs, so that all XCDs have work (1 column, 400 slabs, 600 outputs: 19.2
    // to 11.2 us; of many columns the sub-layer grid would lose 6 percent)
    const int per = gridDim.x / kXcds, turn = a.C < 8 * kXcds ? blockIdx.y : 0;
    const int c = blockIdx.z * kOpticsColumns + (blockIdx.x + turn) % kXcds * per + blockIdx.x / kXcds;
    if (c >= a.C) return;
    const int s0 = blockIdx.y * L, n = min(L, a.S - s0);
    const long long row = (long long)a.nT * a.NBG;
    // levels of the slabs, one lane each: centres, or on the sub-layer grid the lower
    // level and then the upper ones (even levels interfaces, odd ones centres)
    __shared__ struct Level {
        double w00, w10, w01, w11;   // weights of the k-table cell's corners
        long long at;                // its lower corner
        double scale;                // optical depth of the slab above per extinction
    } levels[kOpticsLevels];
    if (threadIdx.x < 64) {
        const int ln = threadIdx.x, l = s0 + min(ln, SUB ? n : n - 1);
        const long long o = (long long)(SUB ? l >> 1 : l) * a.C + c;
        double T, p, dp;
        if constexpr (SUB) {
            T = (l & 1) ? a.Tc[o] : a.T[o];
            p = (l & 1) ? a.pc[o] : a.p[o];
            dp = 0.5 * (p - __shfl_down(p, 1));   // of both levels' mean
        } else {
            T = a.Tc[o];
            p = a.pc[o];
            dp = a.p[o] - a.p[o + a.C];
        }
        const Cell q = cell_at(a, T, p);
        levels[ln] = {(1 - q.t) * (1 - q.u), q.t * (1 - q.u), (1 - q.t) * q.u, q.t * q.u,
                      q.j * row + (long long)q.i * a.NBG, dp / a.gravity / a.m_mean};
    }
    if constexpr (ONE) __syncthreads();
    // this thread's output; the padding takes the last one and stores the same values
    auto output = [&](const int bg) {
        const int b = bg / a.NG;
        const double ss = a.sig_cl_scat[b], sa = a.sig_cl_abs[b], scat = a.sig_gas[b] + ss;
        const double g0 = scat > 0.0 ? ss * a.g0_cl[b] / scat : 0.0;
        struct Corners {
            double k00, k10, k01, k11;
        };
        auto load = [&](int k) -> Corners {
            const int kc = SUB ? min(k, n) : min(k, n - 1);
            const long long e = levels[kc].at;
            const double *k0 = a.kappa + ((long long)__builtin_amdgcn_readfirstlane((int)(e >> 32)) << 32 |
                                          (unsigned)__builtin_amdgcn_readfirstlane((int)e));
            return {k0[bg], (k0 + a.NBG)[bg], (k0 + row)[bg], (k0 + row + a.NBG)[bg]};
        };
        // extinction per gas molecule and albedo at level k: bilinear opacity, then the
        // mixing of gas and condensate extinction and scattering
        double ext_lo = 0.0, w0_lo = 0.0;
        auto level = [&](int k, const Corners &v, double &ext, double &w0) {
            const Level &m = levels[k];
            const double kap = m.w00 * v.k00 + m.w10 * v.k10 + m.w01 * v.k01 + m.w11 * v.k11;
            ext = scat + kap * a.m_mean + sa;
            w0 = ext > 0.0 ? scat / ext : 0.0;
        };
        auto store = [&](int k, double dtau, double w0) {
            const long long e = ((long long)(s0 + k) * a.C + c) * a.NBG;
            (a.dtau + e)[bg] = dtau;
            (a.w0 + e)[bg] = w0;
            (a.g0 + e)[bg] = g0;
        };
        // slab k from level k + SUB's opacities; the next but one level's loads go out
        // before this slab's stores, into the same registers
        auto slab = [&](int k, Corners &v) {
            double ext, w0;
            level(k + SUB, v, ext, w0);
            v = load(k + SUB + 2);
            if constexpr (SUB) {
                store(k, (ext_lo + ext) * levels[k].scale, 0.5 * (w0_lo + w0));
                ext_lo = ext;
                w0_lo = w0;
            } else {
                store(k, ext * levels[k].scale, w0);
            }
        };
        if constexpr (!ONE) __syncthreads();
        Corners x = load(0), y = load(1);
        if constexpr (SUB) {
            level(0, x, ext_lo, w0_lo);
            x = load(2);
            int k = 0;
            for (; k + 2 <= n; k += 2) {
                slab(k, y);
                slab(k + 1, x);
            }
            if (k < n) slab(k, y);
        } else {
            int k = 0;
            for (; k + 2 <= n; k += 2) {
                slab(k, x);
                slab(k + 1, y);
            }
            if (k < n) slab(k, x);
        }
    };
    if constexpr (ONE)
        for (int bg = threadIdx.x; bg < (a.NBG + 63) / 64 * 64; bg += 64) output(min(bg, a.NBG - 1));
    else output(min((int)threadIdx.x, a.NBG - 1));
}

// Gauss-Legendre nodes and weights on [-1, 1] by Newton iteration on the
// Legendre recurrence.
void gauss_legendre(int n, std::vector<double> &x, std::vector<double> &w)
{
    x.assign(n, 0.0);
    w.assign(n, 0.0);
    for (int i = 0; i < n; ++i) {
        double z = std::cos(M_PI * (i + 0.75) / (n + 0.5)), dp = 0.0;
        for (int it = 0; it < 100; ++it) {
            double p0 = 1.0, p1 = z;
            for (int k = 2; k <= n; ++k) {
                const double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
                p0 = p1;
                p1 = p2;
            }
            dp = n * (z * p1 - p0) / (z * z - 1.0);
            const double dz = p1 / dp;
            z -= dz;
            if (std::fabs(dz) < 1e-16) break;
        }
        x[i] = z;
        w[i] = 2.0 / ((1.0 - z * z) * dp * dp);
    }
}

// Rayleigh cross section per molecule (m^2) from the Lorentz-Lorenz form of
// Appendix C, evaluated in the printed CGS units.
double rayleigh_cgs_to_si(double lam_m, double n_ref_cm3, double n_r)
{
    const double lam_cm = lam_m * 100.0;
    const double ll = (n_r * n_r - 1.0) / (n_r * n_r + 2.0);
    const double pi3 = M_PI * M_PI * M_PI;
    return 1e-4 * 24.0 * pi3 / (n_ref_cm3 * n_ref_cm3 * lam_cm * lam_cm * lam_cm * lam_cm) * ll * ll;
}

double sigma_h2(double lam_m)
{
    const double l2 = (lam_m * 1e6) * (lam_m * 1e6);
    return rayleigh_cgs_to_si(lam_m, 2.68678e19, 1.0 + 1.358e-4 * (1.0 + 7.52e-3 / l2));
}

double sigma_he(double lam_m)
{
    const double l2 = (lam_m * 1e6) * (lam_m * 1e6);
    return rayleigh_cgs_to_si(lam_m, 2.546899e19,
                              1.0 + 1e-8 * (2283.0 + 1.8102e13 / (1.5342e10 - 1.0 / l2)));
}

}  // namespace

double rayleigh_bin_average(double lam_lo, double lam_hi, double x_h2, double x_he)
{
    // mean over the bin in wavenumber: 16 Gauss-Legendre points on 24 panels
    static std::vector<double> gx, gw;
    if (gx.empty()) gauss_legendre(16, gx, gw);
    const double nu0 = 1.0 / lam_hi, nu1 = 1.0 / lam_lo;
    const int panels = 24;
    const double h = (nu1 - nu0) / panels;
    double sum = 0.0;
    for (int pnl = 0; pnl < panels; ++pnl) {
        const double m = nu0 + (pnl + 0.5) * h;
        for (size_t i = 0; i < gx.size(); ++i) {
            const double lam = 1.0 / (m + 0.5 * h * gx[i]);
            sum += 0.5 * h * gw[i] * (x_h2 * sigma_h2(lam) + x_he * sigma_he(lam));
        }
    }
    return sum / (nu1 - nu0);
}

hipError_t launch_optics(const OpticsArgs &a, const DeviceLimits &dev, hipStream_t s)
{
    if ((long long)a.S * a.C == 0 || a.NBG == 0) return hipSuccess;
    // Slabs per workgroup, in even runs of at most 16: longer ones spread the stores in
    // flight over more of the memory's pages (2562 columns, 80 slabs x 600 outputs, us by
    // slabs: 4: 905, 8: 716, 16: 642, 27: 724, 40: 783; stores alone 562, 631, 700, -, 760),
    // shorter ones pay for a workgroup's start, about 6 us, too often (30 outputs: 4: 91,
    // 16: 57, 40: 54).  Fewer, from 4 on, where that leaves the chip idle: six wavefronts per
    // CU, and three workgroups per two CUs (162 columns, 30 outputs: 4: 10.4, 8: 9.4, 16:
    // 10.2, 40: 14.3).
    // One or two slabs of many columns do not pay for a workgroup of ten wavefronts that
    // waits for its brackets (10242 columns x 512 outputs, 1 slab: 54 us, 42 in single ones).
    const bool one = a.S <= 2 && a.C >= (a.sub ? 4096 : 1024);
    const int waves = one ? 1 : (a.NBG + 63) / 64;
    const long long n_cu = dev.n_cu > 0 ? dev.n_cu : 256, want = std::max(n_cu * 6 / waves, n_cu * 3 / 2);
    const long long least = std::min<long long>((a.S + 3) / 4, (want + a.C - 1) / a.C);
    const int runs = (int)std::max<long long>((a.S + 15) / 16, least), L = (a.S + runs - 1) / runs;
    const int columns = std::min(a.C, kOpticsColumns);
    const dim3 grid((columns + kXcds - 1) / kXcds * kXcds, (a.S + L - 1) / L, (a.C + kOpticsColumns - 1) / kOpticsColumns);
    if (a.sub && one) hipLaunchKernelGGL((k_optics<true, true>), grid, dim3(64), 0, s, a, L);
    else if (a.sub) hipLaunchKernelGGL((k_optics<true, false>), grid, dim3(64 * waves), 0, s, a, L);
    else if (one) hipLaunchKernelGGL((k_optics<false, true>), grid, dim3(64), 0, s, a, L);
    else hipLaunchKernelGGL((k_optics<false, false>), grid, dim3(64 * waves), 0, s, a, L);
    return hipGetLastError();
}

}  // namespace rtk
