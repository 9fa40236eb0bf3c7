// rt_lanes.hpp -- what the wavefront-per-lanes kernels share (device code):
// the layout of columns over a wavefront's lanes, Planck radiances from edge
// integrals in LDS, and the outputs of a workgroup's columns from its level sums.
#pragma once

#include "rt_internal.hpp"
#include "rt_math.hpp"
#include "rt_physics.hpp"
#include "rt_planck.hpp"
#include "rt_wave.hpp"

#include <type_traits>

namespace rtk {

// This source file's copy of the Planck table on each device (filled by
// upload_planck_table before the device's first launch from the file).
static __device__ __attribute__((aligned(16))) double planck_values[kPlanckTable];

static hipError_t upload_planck_table()
{
    static double host[kPlanckTable];
    static const bool built = (planck_table(host), true);
    (void)built;
    return hipMemcpyToSymbol(HIP_SYMBOL(planck_values), host, sizeof host);
}

// Planck edge integral at x (planck_edge's sign convention); tab: the table in LDS (FP64).
template <class R>
__device__ __forceinline__ R edge_integral(double x, const double *tab)
{
    if constexpr (sizeof(R) == 8) return planck_lookup(x, tab);
    else return planck_edge<R>(x);
}

// n / d for 0 <= n < 2^20, 0 < d (no integer division)
__device__ __forceinline__ int small_div(int n, int d)
{
    return (int)(((float)n + 0.5f) * (1.0f / (float)d));
}

// Lane layout of a problem over wavefronts: up to 64 lanes per column, gw columns
// per wavefront, each padded to NBp lanes (a power of two from 8 to 64); or a wider
// column over NBw wavefronts, slices of NBs lanes each (the last one may hold fewer).
struct LaneLayout {
    int NBp, gw, NBw, NBs;
};
__host__ __device__ __forceinline__ LaneLayout lane_layout(int NB)
{
    LaneLayout l;
    int p = 8;
    while (p < NB && p < 64) p *= 2;
    l.NBp = p;
    l.gw = NB > 64 ? 1 : 64 / p;
    l.NBw = (NB + 63) / 64;
    l.NBs = (NB + l.NBw - 1) / l.NBw;
    return l;
}

// Planck edges that one wavefront needs at most: its lanes' bins and one more.
__host__ __device__ __forceinline__ int wave_edges(int NB, int NG)
{
    const int NBR = NB / NG, NBs = lane_layout(NB).NBs;
    const int most = NG == 1 ? NBs : (NBs + NG - 2) / NG + 1;
    return (most < NBR ? most : NBR) + 1;
}

// base + off bytes: a wavefront-uniform base and a 32-bit offset per lane
template <class T>
__device__ __forceinline__ T &at(T *base, unsigned off)
{
    return *reinterpret_cast<T *>(reinterpret_cast<char *>(const_cast<typename std::remove_const<T>::type *>(base)) + off);
}

// A wavefront-uniform value kept in scalar registers from here on (not read
// again from memory at its uses).
template <class T>
__device__ __forceinline__ void uniform_value(T &x)
{
    asm volatile("" : "+s"(x));
}

// A value that all lanes hold, in scalar registers.
__device__ __forceinline__ double first_lane(double x)
{
    return __hiloint2double(wave_uniform(__double2hiint(x)), wave_uniform(__double2loint(x)));
}

// The options used per layer, read anew here and kept in scalar registers.
__device__ __forceinline__ Opts uniform_options(ArgsK ap)
{
    Opts o = ((const SolveArgs *)ap)->o;
    uniform_value(o.e_tau);
    uniform_value(o.g_guard);
    uniform_value(o.improved);
    uniform_value(o.noniso);
    uniform_value(o.e_clamp);
    return o;
}

// LDS values written by lanes of this wavefront are read by others of it.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Temperature of level l of column cc: on the sub-layer grid even levels are
// interfaces and odd levels layer centres.
__device__ __forceinline__ double level_T(const SolveArgs &a, bool sub, int l, int cc)
{
    const double *T_if = a.T, *T_ce = sub ? a.Tc : a.T;
    const double *base = (sub && (l & 1)) ? T_ce : T_if;
    return base[(long long)(sub ? (l >> 1) : l) * a.C + cc];
}

// What the bin radiances take of a level's temperature, worked out once per level: the
// Planck prefactor; in mixed precision 1 / T as well, for the narrow bins.
template <bool MIXED>
struct LevelValue {
    double prefactor;
    __device__ __forceinline__ static LevelValue of(double T) { return {kPref * (T * T) * (T * T)}; }
};
template <>
struct LevelValue<true> {
    double iT;
    float iTf, prefactor;
    __device__ __forceinline__ static LevelValue of(double T)
    {
        const float Tf = float(T), T2 = Tf * Tf;
        return {rcp(T), rcp(Tf), float(kPref) * T2 * T2};
    }
};

// Bin radiance at a level from the edge integrals re[0], re[1] of the bin; c2b, c2a: c2 /
// lambda at its edges (LDS), fb, fa the same in FP32.  narrow (MIXED): all bins are
// (planck_narrow), and there are no edge integrals.
template <bool MIXED, class R>
__device__ __forceinline__ R bin_radiance(const R *re, const LevelValue<MIXED> &lv, float fb, float fa, const double *c2,
                                          bool narrow)
{
    if constexpr (!MIXED) {
        return lv.prefactor * planck_combine<R>(re[0], re[1]);
    } else {
        R I = R(0);
        if (!narrow) I = planck_combine<R>(re[0], re[1]);
        const R xb = fb * lv.iTf, xa = fa * lv.iTf;
        if (narrow || planck_narrow(xa, xb)) I = planck_gl3(c2[1] * lv.iT, c2[0] * lv.iT);
        return lv.prefactor * I;
    }
}

// The elimination's map of (c, eps = 1 - c, d) over a run of layers.  With den = (1 - r)
// + r eps, elim_step (rt_physics.hpp) takes w (1, eps, c, d) to w' (1, eps', c', d'), w' =
// w den, linearly in (w, e, c, d) = w (1, eps, c, d):
//   w' = (1-r) w + r e,  e' = A (1-r+t) w + (r (1-r) + t^2) e,
//   c' = r w' + t^2 c,   d' = S_dn w' + t (d + S_up c),
// so a run is the product of its layers' matrices.  The columns of w, e and c are
// non-negative: no digit is lost.  m: w and e from (e, w); c from (c, e, w); d from (d,
// c, e, w) at the top.
struct StateMap {
    double m[11] = {0, 1, 1, 0, 1, 0, 0, 1, 0, 0, 0};
    __device__ __forceinline__ void step(double t, double r, double omr, double A, double Sup, double Sdn)
    {
        const double tt = t * t, a1 = A * (omr + t), a2 = fma(r, omr, tt);
        const double we = fma(omr, m[0], r * m[2]), ww = fma(omr, m[1], r * m[3]);
        m[2] = fma(a1, m[0], a2 * m[2]);
        m[3] = fma(a1, m[1], a2 * m[3]);
        m[0] = we;
        m[1] = ww;
        m[7] *= t;
        m[8] = t * fma(Sup, m[4], m[8]);
        m[9] = fma(Sdn, we, t * fma(Sup, m[5], m[9]));
        m[10] = fma(Sdn, ww, t * fma(Sup, m[6], m[10]));
        m[4] *= tt;
        m[5] = fma(r, we, tt * m[5]);
        m[6] = fma(r, ww, tt * m[6]);
    }
    // by a power of two, so that w stays in range (every few layers: w' >= w (1 - r))
    __device__ __forceinline__ void rescale()
    {
        const int e = -ilogb_pos(m[0] + m[1]);
#pragma unroll
        for (int v = 0; v < 11; ++v) m[v] = ldexp(m[v], e);
    }
    __device__ __forceinline__ ElimState state() const { return {m[0], m[1], m[2]}; }
    __device__ __forceinline__ void set_state(const ElimState &s) { m[0] = s.c, m[1] = s.eps, m[2] = s.d; }
    // the map to a given state
    __device__ __forceinline__ static StateMap constant(const ElimState &s)
    {
        return {{0, 1, 0, s.eps, 0, 0, s.c, 0, 0, 0, s.d}};
    }
    __device__ __forceinline__ static int ilogb_pos(double x) { return x > 0.0 ? __builtin_amdgcn_frexp_exp(x) : 0; }
    __device__ __forceinline__ void apply(ElimState &s) const
    {
        const double i = 1.0 / fma(m[0], s.eps, m[1]);
        const double c = fma(m[4], s.c, fma(m[5], s.eps, m[6]));
        const double d = fma(m[7], s.d, fma(m[8], s.c, fma(m[9], s.eps, m[10])));
        s.eps = fma(m[2], s.eps, m[3]) * i;
        s.c = c * i;
        s.d = d * i;
    }
};

// Outputs of the K columns from c0 on from their level sums, sum(level, 0: up, 1:
// down or 2: beam, column): the bin-summed fluxes, the net flux, the heating and the
// flags.  All threads of the workgroup; the sums and s_flag [K] are complete.
template <class Sum>
__device__ __forceinline__ void write_columns(ArgsK ap, int c0, int K, uint32_t *s_flag, Sum sum)
{
    opaque_args(ap);
    auto args = [&]() -> const SolveArgs & { return *(const SolveArgs *)ap; };
    const int C = args().C, N = args().N;
    const bool sub = args().sub != 0;
    const int tid = threadIdx.x;
    auto out_at = [&](double *iface, double *centre, int l, int cc) -> double * {
        if (sub) return ((l & 1) ? centre : iface) + (long long)(l >> 1) * C + cc;
        return iface + (long long)l * C + cc;
    };
    for (int t = tid; t < (N + 1) * K; t += blockDim.x) {
        const int lev = K == 1 ? t : small_div(t, K), k = t - lev * K, cc = c0 + k;
        if (cc >= C) continue;
        const bool dk = args().mu[cc] > 0.0;   // (night columns have no beam sums)
        auto net = [&](int l, double &su, double &sd, double &sb) -> double {
            su = sum(l, 0, k);
            sd = sum(l, 1, k);
            sb = dk ? sum(l, 2, k) : 0.0;
            return su - sd - sb;
        };
        double su, sd, sb, x, y, z;
        const double fn = net(lev, su, sd, sb);
        *out_at(args().F_up, args().F_up_c, lev, cc) = su;
        *out_at(args().F_dn, args().F_dn_c, lev, cc) = sd;
        *out_at(args().F_beam, args().F_beam_c, lev, cc) = sb;
        *out_at(args().F_net, args().F_net_c, lev, cc) = fn;
        if (!isfinite(fn)) atomicOr(&s_flag[k], (uint32_t)F_NONFIN);
        const int up = sub ? lev + 2 : lev + 1;   // the interface above
        if (up > N || (sub && (lev & 1))) continue;
        const int j = sub ? lev >> 1 : lev;
        const double fnu = net(up, x, y, z);
        const long long o = (long long)j * C + cc;
        const double p0 = args().p[o], p1 = args().p[o + C];
        const double dp = p0 - p1;
        bool bad = !(dp > 0.0);
        if (sub) {
            const double pm = args().pc[o];
            bad = bad || !(p0 > pm && pm > p1);
        }
        if (bad) atomicOr(&s_flag[k], (uint32_t)F_INVALID);
        const double qh = args().o.gravity * (fn - fnu) / dp;
        args().heat[o] = qh;
        if (args().dTdt) args().dTdt[o] = qh / args().o.cp;
    }
    __syncthreads();
    for (int k = tid; k < K; k += blockDim.x) {
        if (c0 + k >= C) continue;
        if (args().flags) args().flags[c0 + k] = s_flag[k];
        const uint32_t bad = status_bits(s_flag[k]);
        if (args().status && bad) atomicOr(args().status, bad);
    }
}

}  // namespace rtk
