// rt_cascade.hip -- layer-parallel solve for deep columns and few columns of up to 64 lanes.
//
// Paper: Deitrick et al., "The THOR+HELIOS general circulation model"
// (arXiv 2203.02293): the same per-layer arithmetic as the other solve kernels
// (Section 2.2.1, Appendix B, `rt_physics.hpp`) and the same Thomas recurrence (Section
// 2.2.2).  The segments of a column are those of rt_deep.hip, a workgroup each; here a
// segment's layers are split again, into parts of kPart, a group of lanes of a wavefront
// each, and what one lane walked through (the elimination, the optical depth, the
// back-substitution) runs in all parts at once:
//
//   k_cascade_tau    optical depth of each segment
//   k_cascade_items  Planck, beam and the layer coefficients; each part's map of the
//                    elimination (StateMap) and upward emission, and those of the segment;
//                    the beam's sums
//   k_cascade_scan   per lane, tree scans over the segments: c and eps at every segment's
//                    top (the 2x2 maps of rt_deep.hip, rescaled to c + eps = 1), d
//                    there, the BOA condition, F_up at every segment's bottom
//   k_cascade_back   per part: the state at its top, the elimination and the
//                    back-substitution with its records in registers; sums, net flux, heating
//
// Seen from outside a run of layers is one layer, F_up at its top = T F_up at its bottom + R
// F_dn + S (the adding method), with F_dn = c F_up + d from above: with the map's w = kappa
// (1 - R c), m7 = kappa T, m0 = kappa R and sigma = kappa S,
//   F_up(top) = (m7 F_up(bottom) + m0 d + sigma) / w.
// What bounds it is the latency of one part's chain, about 2500 cycles a layer, and of four
// launches: 1 x 4096 x 30 FP64 44 us and 16 x 1000 x 30 mixed 56, by the seven launches
// of rt_deep.hip 52 and 82, which wider columns take, sub-layer columns with an odd number of slabs
// per segment, and columns of a few lanes whose parts would not fit its work buffer (cascade_fits).
#include "rt_lanes.hpp"

#include <algorithm>
#include <type_traits>

namespace rtk {
namespace {

// Slabs per part: with T_int's and the top level's, a group's Planck rows are the eight of
// one pass.
constexpr int kPart = 6;
constexpr int kRows = 8, kStride = 65;

// Work buffer, L = C NB lanes, S segments of Ls slabs, T parts:
//   coef [column][segment][wavefront][kPart][2][64] double2   the layers' coefficients
//   part [12][T][L]   each part's map and sigma
//   seg  [kFields][S][L]
//   tau [S][L], lane [2][L]
enum SegField : int { SF_SIGMA = 11, SF_P00, SF_P01, SF_P10, SF_P11, SF_C, SF_EPS, SF_D, SF_FBOT, kFields };
struct CascadeLayout {
    int S, Ls, parts, T;      // segments, their slabs, parts per segment, parts of a column
    int gw, lNBp, waves;      // groups per wavefront, log2 of their lanes, wavefronts per segment
    long long L;
    double2 *coef;
    double *part, *seg, *tau, *lane;
};
__host__ __device__ __forceinline__ CascadeLayout cascade_layout(int C, int N, int NB, int S, int Ls, double *scratch)
{
    CascadeLayout d;
    d.S = S;
    d.Ls = Ls;
    d.parts = (Ls + kPart - 1) / kPart;
    d.T = (S - 1) * d.parts + (N - (S - 1) * Ls + kPart - 1) / kPart;
    d.lNBp = 3;
    while (1 << d.lNBp < NB) ++d.lNBp;
    d.gw = 64 >> d.lNBp;
    d.waves = (d.parts + d.gw - 1) / d.gw;
    d.L = (long long)C * NB;
    d.coef = reinterpret_cast<double2 *>(scratch);
    d.part = scratch + (long long)C * S * d.waves * (kPart * 2 * 64 * 2);
    d.seg = d.part + 12 * d.T * d.L;
    d.tau = d.seg + (long long)kFields * S * d.L;
    d.lane = d.tau + S * d.L;
    return d;
}
__host__ __device__ __forceinline__ size_t cascade_doubles(int C, int N, int NB, int S, int Ls)
{
    const CascadeLayout d = cascade_layout(C, N, NB, S, Ls, nullptr);
    return (size_t)(d.lane - (double *)nullptr) + 2 * d.L;
}
__device__ __forceinline__ CascadeLayout cascade_layout(const SolveArgs &a)
{
    return cascade_layout(a.C, a.N, a.NB, a.K, a.PC, a.scratch);
}

// Part j of segment s (past the last: the last): its slabs from the TOA [e, e1); all parts run
// kPart steps, from slab e1 - kPart on, a shorter one's first `skip` are other parts'.
struct Part {
    int s, j, i, n, e, e1, skip;   // i: of the column, n: parts of the segment
};
__device__ __forceinline__ Part part_at(const SolveArgs &a, const CascadeLayout &d, int s, int j)
{
    Part p;
    p.s = s;
    const int slabs = min(d.Ls, a.N - s * d.Ls);
    p.n = (slabs + kPart - 1) / kPart;
    p.j = min(j, p.n - 1);
    p.i = s * d.parts + p.j;
    p.e = s * d.Ls + p.j * kPart;
    p.e1 = s * d.Ls + min((p.j + 1) * kPart, slabs);
    p.skip = kPart - (p.e1 - p.e);
    return p;
}

// ---------------------------------------------------------------- tau
// The optical depth in the order of rt_deep.hip's sums: the mixed path rounds the beam's
// exponential to FP32, and an optical depth off in its last bit changes a layer's heating
// by that rounding.
// Sum of p[k stride], k = 0 .. n - 1 in that order, eight loads at a time.
template <class InT>
__device__ __forceinline__ double sum_in_order(const InT *p, long long stride, int n)
{
    double t = 0.0;
    for (int k = 0; k < n; k += 8) {
        double v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = double(p[min(k + q, n - 1) * stride]);
#pragma unroll
        for (int q = 0; q < 8; ++q) t += k + q < n ? v[q] : 0.0;
    }
    return t;
}

// tau: sum of each segment's slabs.
template <class InT>
__global__ void __launch_bounds__(64) k_cascade_tau(const SolveArgs a)
{
    const CascadeLayout d = cascade_layout(a);
    const int s = blockIdx.x, c = blockIdx.y, b = threadIdx.x;
    if (a.flags && s == 0 && b == 0) a.flags[c] = 0u;
    if (b >= a.NB) return;
    const int top = a.N - s * d.Ls, slabs = min(d.Ls, top);
    const long long l = (long long)c * a.NB + b;
    d.tau[s * d.L + l] = sum_in_order(reinterpret_cast<const InT *>(a.dtau) + (top - 1) * d.L + l, -d.L, slabs);
}

// The coefficients of a mixed-precision layer in FP64: t and 1 - r from whichever of a
// value and its complement is the smaller (both relatively exact): thin layers keep 1 - t
// and r to the coefficients' relative precision, so FP32 rounding of t near 1 does not
// accumulate along the column's transmission.  Packed: t or, negative, 1 - t; r; 1 - r; A.
__device__ __forceinline__ double2 pack_mixed(float t, float omt, float r, float omr, float A)
{
    const float v = t < 0.5f ? t : -omt;
    return make_double2(__hiloint2double(__float_as_int(r), __float_as_int(v)),
                        __hiloint2double(__float_as_int(A), __float_as_int(omr)));
}
__device__ __forceinline__ void unpack_mixed(double2 x, double &t, double &r, double &omr, double &A)
{
    const float v = __int_as_float(__double2loint(x.x)), rf = __int_as_float(__double2hiint(x.x));
    t = signbit(v) ? 1.0 + double(v) : double(v);
    r = double(rf);
    omr = rf < 0.5f ? 1.0 - r : double(__int_as_float(__double2loint(x.y)));
    A = double(__int_as_float(__double2hiint(x.y)));
}

// ---------------------------------------------------------------- items
constexpr int kShared = 16;   // values a group leaves for the others of its segment
struct ItemsLds {
    int estride;
    size_t tab, c2, above, per_wave, temp, val, edge, total;   // temp, val, edge in a wavefront's region
};
__host__ __device__ __forceinline__ ItemsLds items_lds(int gw, int waves, int NBR, int QL, bool mixed)
{
    ItemsLds o;
    o.estride = (NBR + 1) | 1;
    o.tab = 0;
    o.c2 = mixed ? 0 : kPlanckTable * 8;
    o.temp = 0;
    o.val = (size_t)gw * kRows * (mixed ? 16 : 8);
    o.edge = o.val + kRows * kStride * 8;
    o.per_wave = (o.edge + (size_t)gw * kRows * o.estride * (mixed ? 4 : 8) + 15) & ~size_t(15);
    if (o.per_wave < kShared * 64 * 8) o.per_wave = kShared * 64 * 8;
    o.above = (o.c2 + (size_t)(NBR + 1) * 8 + 15) & ~size_t(15);   // double [QL][64 / gw]
    o.total = o.above + (size_t)QL * (64 / gw) * 8 + waves * o.per_wave;
    return o;
}

// Sums of a group's lanes of row q = ln % 8 (stored [8][kStride]); every lane of the group
// part p = ln / 8 ends with the sum of its group.
__device__ __forceinline__ double group_sum(const double *v, int lNBp)
{
    wave_sync();
    const int ln = threadIdx.x & 63;
    const double *r = v + (ln & 7) * kStride + (ln >> 3) * 8;
    double s = r[0];
#pragma unroll
    for (int k = 1; k < 8; ++k) s += r[k];
    if (lNBp > 3) s += __shfl_xor(s, 8);
    if (lNBp > 4) s += __shfl_xor(s, 16);
    if (lNBp > 5) s += __shfl_xor(s, 32);
    wave_sync();
    return s;
}

__device__ __forceinline__ double *level_out(const SolveArgs &a, double *iface, double *centre, int l, int c)
{
    if (a.sub) return ((l & 1) ? centre : iface) + (long long)(l >> 1) * a.C + c;
    return iface + (long long)l * a.C + c;
}

__device__ __forceinline__ StateMap compose(const StateMap &A, const StateMap &B)   // A above B
{
    StateMap m;
    const double *x = A.m, *y = B.m;
    m.m[0] = fma(y[0], x[2], y[1] * x[0]);
    m.m[1] = fma(y[0], x[3], y[1] * x[1]);
    m.m[2] = fma(y[2], x[2], y[3] * x[0]);
    m.m[3] = fma(y[2], x[3], y[3] * x[1]);
    m.m[4] = y[4] * x[4];
    m.m[5] = fma(y[4], x[5], fma(y[5], x[2], y[6] * x[0]));
    m.m[6] = fma(y[4], x[6], fma(y[5], x[3], y[6] * x[1]));
    m.m[7] = y[7] * x[7];
    m.m[8] = fma(y[7], x[8], y[8] * x[4]);
    m.m[9] = fma(y[7], x[9], fma(y[8], x[5], fma(y[9], x[2], y[10] * x[0])));
    m.m[10] = fma(y[7], x[10], fma(y[8], x[6], fma(y[9], x[3], y[10] * x[1])));
    m.rescale();
    return m;
}


// Upward emission of a run of layers (map m, sigma) with another one (b, sb) below it, per w
// of the reference state c = 0, eps = 1, d = 0; times the joint map's w it is its sigma.
__device__ __forceinline__ double emission(const StateMap &m, double sigma, const StateMap &b, double sb)
{
    const double iw = rcp(m.m[0] + m.m[1]);
    const double eps = (m.m[2] + m.m[3]) * iw, dd = (m.m[9] + m.m[10]) * iw;
    return iw * fma(m.m[7], fma(b.m[0], dd, sb) * rcp(fma(b.m[0], eps, b.m[1])), sigma);
}

template <bool MIXED, bool IN32>
__global__ void __launch_bounds__(512, 2) k_cascade_items(const SolveArgs a)
{
    using R = typename std::conditional<MIXED, float, double>::type;
    using InT = typename std::conditional<IN32, float, double>::type;
    extern __shared__ double smem[];
    char *lds = reinterpret_cast<char *>(smem);
    const CascadeLayout d = cascade_layout(a);
    const int NB = a.NB, NG = a.NG, NBR = NB / NG, N = a.N, tid = threadIdx.x, W = blockDim.x, c = blockIdx.y, s = blockIdx.x;
    const int wave = wave_uniform(tid >> 6), ln = tid & 63, NBp = 1 << d.lNBp;
    const int gl = ln >> d.lNBp, g0 = wave * d.gw;
    const Part me = part_at(a, d, s, g0 + gl);
    const int yb = ln & (NBp - 1), b = min(yb, NB - 1);
    const bool act = g0 + gl < me.n && yb < NB;
    const ItemsLds lo = items_lds(d.gw, W >> 6, NBR, a.CH, MIXED);
    double *s_tab = reinterpret_cast<double *>(lds + lo.tab), *s_c2 = reinterpret_cast<double *>(lds + lo.c2);
    char *regions = lds + lo.total - (W >> 6) * lo.per_wave, *own = regions + wave * lo.per_wave;
    LevelValue<MIXED> *s_level = reinterpret_cast<LevelValue<MIXED> *>(own + lo.temp);
    double *s_val = reinterpret_cast<double *>(own + lo.val);
    R *s_edge = reinterpret_cast<R *>(own + lo.edge);
    const long long l = (long long)c * NB + b;
    const int a0 = me.e1 - kPart;   // slab (from the TOA) of the first step

    InT dt[kPart], w0[kPart], g0s[kPart];
#pragma unroll
    for (int q = 0; q < kPart; ++q) {
        const long long o = (long long)(N - 1 - a0 - q) * d.L + l;
        dt[q] = reinterpret_cast<const InT *>(a.dtau)[o];
        w0[q] = reinterpret_cast<const InT *>(a.w0)[o];
        g0s[q] = reinterpret_cast<const InT *>(a.g0)[o];
    }
    // the row of this lane's Planck edges: T_int, the level at the top, the lower levels
    const int lrows = 9 - d.lNBp, row = ln & ((1 << lrows) - 1), e0 = ln >> lrows, epr = 64 >> lrows, rq = row & (kRows - 1);
    const Part rs = part_at(a, d, s, g0 + row / kRows);
    const double T = rq == 0 ? a.Tint[c] : level_T(a, a.sub != 0, N - (rs.e1 - kPart) - (rq - 1), c);
    if constexpr (!MIXED) {
        constexpr int n = (kPlanckTable + 63) / 64;
        double v[n];
#pragma unroll
        for (int i = 0; i < n; ++i) v[i] = planck_values[min(tid + i * W, kPlanckTable - 1)];
#pragma unroll
        for (int i = 0; i < n; ++i) s_tab[min(tid + i * W, kPlanckTable - 1)] = v[i];
    }
    for (int e = tid; e <= NBR; e += W) s_c2[e] = a.c2_over_lam[e];
    // the optical depth above the segment: CH partial sums of the segments above; then that
    // above the part
    double *s_above = reinterpret_cast<double *>(lds + lo.above);
    for (int g = g0 + gl; g < a.CH; g += (W >> 6) * d.gw)
        s_above[(g << d.lNBp) + yb] =
            g < s ? sum_in_order(d.tau + g * d.L + l, a.CH * d.L, (s - g + a.CH - 1) / a.CH) : 0.0;
    double above[8];   // the part's segment from its top, loads first
    const int before = me.e - s * d.Ls;
    const InT *p_above = reinterpret_cast<const InT *>(a.dtau) + (long long)(N - 1 - s * d.Ls) * d.L + l;
#pragma unroll
    for (int q = 0; q < 8; ++q) above[q] = double(p_above[-min(q, max(before - 1, 0)) * d.L]);

    uint32_t fl = 0u;
    const int bin = NG == 1 ? b : b / NG;
    const double mu = a.mu[c], Ti = a.Tint[c];
    const bool day = mu > 0.0;
    if (!isfinite(mu) || !(Ti >= 0.0) || !isfinite(Ti)) fl |= F_INVALID;
    if (rq > 0 && (!(T > 0.0) || !isfinite(T))) fl |= F_INVALID;
    const double inv_mu = day ? 1.0 / mu : 0.0;
    const double muF = day ? mu * a.F_star[bin] : 0.0;
    const double inv_eps2 = 1.0 / a.o.eps2;
    const double wgt = act ? (NG == 1 ? 1.0 : a.wg[b % NG]) : 0.0;
    float c2fb = 0.0f, c2fa = 0.0f;
    if constexpr (MIXED) {
        c2fb = a.c2_over_lam_f[bin];
        c2fa = a.c2_over_lam_f[bin + 1];
    }
    __syncthreads();
    double tau = 0.0;
    for (int g = 0; g < a.CH; ++g) tau += s_above[(g << d.lNBp) + yb];
    for (int k = 0; k < before; k += 8) {
        if (k > 0) {
#pragma unroll
            for (int q = 0; q < 8; ++q) above[q] = double(p_above[-min(k + q, before - 1) * d.L]);
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) tau += k + q < before ? above[q] : 0.0;
    }
    const double iT = rcp(T);
    if (e0 == 0) s_level[row] = LevelValue<MIXED>::of(T);
    R *re = s_edge + row * lo.estride;
    for (int i = 0; i <= NBR; i += 2 * epr) {
        const int e1 = min(i + e0, NBR), e2 = min(i + epr + e0, NBR);
        const R v1 = edge_integral<R>(s_c2[e1] * iT, s_tab), v2 = edge_integral<R>(s_c2[e2] * iT, s_tab);
        re[e1] = v1;
        re[e2] = v2;
    }
    wave_sync();
    auto bin_B = [&](int r) -> R {
        const int rw = gl * kRows + r;
        return bin_radiance<MIXED, R>(s_edge + rw * lo.estride + bin, s_level[rw], c2fb, c2fa, s_c2 + bin, false);
    };

    double Fb_up = day ? (me.i == 0 ? muF : beam_at<MIXED>(muF, tau, inv_mu)) : 0.0;
    const bool boa = me.i == d.T - 1;
    double Fboa = 0.0;
    if (wave_any(boa)) Fboa = double(kPI) * double(bin_B(0));
    R Bup = bin_B(1);
    StateMap map;
    double y = 0.0;   // sigma
    double P00 = 1.0, P01 = 0.0, P10 = 0.0, P11 = 1.0;
    const Opts o = a.o;
    double2 *coef = d.coef + (((long long)c * d.S + s) * d.waves + wave) * (kPart * 2 * 64) + ln;
    s_val[kPart * kStride + ln] = wgt * muF;   // beam at the TOA
#pragma unroll 1
    for (int q = 0; q < kPart; ++q) {
        double dq = 0.0, wq = 0.0, gq = 0.0;   // (uniform index into registers)
#pragma unroll
        for (int k = 0; k < kPart; ++k)
            if (q == k) {
                dq = double(dt[k]);
                wq = double(w0[k]);
                gq = double(g0s[k]);
            }
        const R B = bin_B(2 + q);
        double Fb_lo = 0.0;
        if (day) {
            if (q >= me.skip) tau += dq;   // (before them: the part's top)
            Fb_lo = beam_at<MIXED>(muF, tau, inv_mu);
        }
        const Layer<R> Ly = layer_item<MIXED, R, MIXED>(dq, wq, gq, day, mu, inv_mu, Fb_up, Fb_lo, B, Bup, o, inv_eps2, fl);
        const double Sup = double(Ly.Sup), Sdn = double(Ly.Sdn);
        double t, r, omr, A;
        double2 x;
        if constexpr (MIXED) {
            x = pack_mixed(Ly.t, Ly.omt, Ly.r, Ly.omr, Ly.A);
            unpack_mixed(x, t, r, omr, A);
        } else {
            t = Ly.t, r = Ly.r, A = Ly.A, omr = Ly.omr;
            const StoredLayer v = store_layer(t, r, A);
            x = make_double2(v.p, v.q);
        }
        // upward emission of the part with this layer below it
        const double w = map.m[0] + map.m[1], e = map.m[2] + map.m[3], D = map.m[9] + map.m[10];
        const double w1 = fma(omr, w, r * e);
        y = fma(y, w1, map.m[7] * fma(r, D, Sup * w)) * rcp(w);
        map.step(t, r, omr, A, Sup, Sdn);
        const double rt = fma(r, omr, t * t), at = A * (omr + t);
        const double q00 = fma(rt, P00, r * P10), q01 = fma(rt, P01, r * P11);
        P10 = fma(at, P00, (at + rt) * P10);
        P11 = fma(at, P01, (at + rt) * P11);
        P00 = q00;
        P01 = q01;
        if (q < me.skip) {   // (another part's)
            map = StateMap();
            y = 0.0;
            P00 = P11 = 1.0;
            P01 = P10 = 0.0;
        }
        coef[q * 128] = x;
        if constexpr (MIXED)
            coef[q * 128 + 64].x = __hiloint2double(__float_as_int(Ly.Sdn), __float_as_int(Ly.Sup));
        else coef[q * 128 + 64] = make_double2(Sup, Sdn);
        s_val[q * kStride + ln] = wgt * Fb_lo;
        Fb_up = Fb_lo;
        Bup = B;
    }
    {
        const int e = -StateMap::ilogb_pos(map.m[0] + map.m[1]);
#pragma unroll
        for (int v = 0; v < 11; ++v) map.m[v] = ldexp(map.m[v], e);
        y = ldexp(y, e);
    }
    if (act) {
#pragma unroll
        for (int v = 0; v < 11; ++v) d.part[((long long)v * d.T + me.i) * d.L + l] = map.m[v];
        d.part[(11ll * d.T + me.i) * d.L + l] = y;
        if (boa) {
            d.lane[l] = Fboa;
            d.lane[d.L + l] = Fb_up;
        }
    }
    // beam sums of the levels below the steps, and of the TOA
    {
        const int q = ln & 7, gs = ln >> d.lNBp;
        const double sum = group_sum(s_val, d.lNBp);
        const Part sg = part_at(a, d, s, g0 + gs);
        if ((ln >> 3 & ((NBp >> 3) - 1)) == 0 && g0 + gs < sg.n) {
            const int p = sg.e1 - kPart + q;   // slab
            const int lev = q < kPart ? (q >= sg.skip ? N - 1 - p : -1) : (q == kPart && sg.i == 0 ? N : -1);
            if (lev >= 0) *level_out(a, a.F_beam, a.F_beam_c, lev, c) = day ? sum : 0.0;
        }
    }
    if (fl) {   // (the padding's rows as well)
        if (a.flags) atomicOr(&a.flags[c], fl);
        const uint32_t bad = status_bits(fl);
        if (a.status && bad) atomicOr(a.status, bad);
    }
    // the segment's maps
    auto shared_at = [&](int v, int t) -> double & {   // value v of thread t
        return *reinterpret_cast<double *>(regions + (t >> 6) * lo.per_wave + (v * 64 + (t & 63)) * 8);
    };
    __syncthreads();   // (the rows' place is free)
#pragma unroll
    for (int v = 0; v < 11; ++v) shared_at(v, tid) = map.m[v];
    shared_at(11, tid) = y;
    shared_at(12, tid) = P00;
    shared_at(13, tid) = P01;
    shared_at(14, tid) = P10;
    shared_at(15, tid) = P11;
    __syncthreads();
    if (!act || me.j != 0) return;
    for (int k = 1; k < me.n; ++k) {
        const int t = tid + (k << d.lNBp);
        StateMap b;
#pragma unroll
        for (int v = 0; v < 11; ++v) b.m[v] = shared_at(v, t);
        const double em = emission(map, y, b, shared_at(11, t));
        map = compose(map, b);
        y = em * (map.m[0] + map.m[1]);
        const double m00 = shared_at(12, t), m01 = shared_at(13, t), m10 = shared_at(14, t), m11 = shared_at(15, t);
        const double q00 = fma(m00, P00, m01 * P10), q01 = fma(m00, P01, m01 * P11);
        const double q10 = fma(m10, P00, m11 * P10), q11 = fma(m10, P01, m11 * P11);
        const double mx = fmax(fmax(q00, q01), fmax(q10, q11)), sc = mx > 0.0 ? rcp(mx) : 1.0;
        P00 = q00 * sc;
        P01 = q01 * sc;
        P10 = q10 * sc;
        P11 = q11 * sc;
    }
    auto seg = [&](int f) -> double & { return d.seg[((long long)f * d.S + s) * d.L + l]; };
#pragma unroll
    for (int v = 0; v < 11; ++v) seg(v) = map.m[v];
    seg(SF_SIGMA) = y;
    seg(SF_P00) = P00;
    seg(SF_P01) = P01;
    seg(SF_P10) = P10;
    seg(SF_P11) = P11;
}

// ---------------------------------------------------------------- scan
// A group of Sp threads (a power of two >= S) per lane, thread k of it segment k; inclusive
// scans in LDS, at distance h = 1, 2, 4, ...
constexpr int kScanThreads = 256;
__host__ __device__ __forceinline__ int scan_threads(int S)
{
    int p = 1;
    while (p < S) p <<= 1;
    return p;
}
__global__ void __launch_bounds__(kScanThreads) k_cascade_scan(const SolveArgs a)
{
    __shared__ double s_x[4][kScanThreads];
    const CascadeLayout d = cascade_layout(a);
    const int Sp = scan_threads(d.S), tid = threadIdx.x, k = tid & (Sp - 1);
    const long long lane = (long long)blockIdx.x * (kScanThreads / Sp) + tid / Sp;
    const bool act = lane < d.L && k < d.S;
    const long long l = lane < d.L ? lane : d.L - 1;
    auto seg = [&](int f) -> double & { return d.seg[((long long)f * d.S + min(k, d.S - 1)) * d.L + l]; };
    double x00 = seg(SF_P00), x01 = seg(SF_P01), x10 = seg(SF_P10), x11 = seg(SF_P11);
    StateMap m;
#pragma unroll
    for (int v = 0; v < 11; ++v) m.m[v] = seg(v);
    const double sigma = seg(SF_SIGMA);
    if (k >= d.S) {
        x00 = x11 = 1.0;
        x01 = x10 = 0.0;
        m = StateMap();
    }
    // c and eps
    auto put = [&](double a0, double a1, double a2, double a3) {
        __syncthreads();
        s_x[0][tid] = a0;
        s_x[1][tid] = a1;
        s_x[2][tid] = a2;
        s_x[3][tid] = a3;
        __syncthreads();
    };
    for (int h = 1; h < Sp; h <<= 1) {
        put(x00, x01, x10, x11);
        if (k >= h) {
            const double y00 = s_x[0][tid - h], y01 = s_x[1][tid - h], y10 = s_x[2][tid - h], y11 = s_x[3][tid - h];
            const double q00 = fma(x00, y00, x01 * y10), q01 = fma(x00, y01, x01 * y11);
            const double q10 = fma(x10, y00, x11 * y10), q11 = fma(x10, y01, x11 * y11);
            const double mx = fmax(fmax(q00, q01), fmax(q10, q11)), sc = mx > 0.0 ? rcp(mx) : 1.0;
            x00 = q00 * sc;
            x01 = q01 * sc;
            x10 = q10 * sc;
            x11 = q11 * sc;
        }
    }
    put(x01, x11, 0.0, 0.0);
    ElimState st = elim_top(a.Ftoa ? a.Ftoa[l] : 0.0);
    const double d_toa = st.d;
    if (k > 0) {
        const double i = rcp(s_x[0][tid - 1] + s_x[1][tid - 1]);
        st.c = s_x[0][tid - 1] * i;
        st.eps = s_x[1][tid - 1] * i;
    }
    // d: affine maps of the segments, later after earlier
    const double iw = rcp(fma(m.m[0], st.eps, m.m[1]));
    double g = m.m[7] * iw, v = fma(m.m[8], st.c, fma(m.m[9], st.eps, m.m[10])) * iw;
    const double gam = g;
    for (int h = 1; h < Sp; h <<= 1) {
        put(g, v, 0.0, 0.0);
        if (k >= h) {
            v = fma(g, s_x[1][tid - h], v);
            g *= s_x[0][tid - h];
        }
    }
    put(fma(g, d_toa, v), 0.0, 0.0, 0.0);   // d at the segment's bottom
    if (k > 0) st.d = s_x[0][tid - 1];
    // the BOA condition at the last segment's bottom, F_up from there
    ElimState bot = st;
    m.apply(bot);
    double Fu, Fd;
    elim_boa(bot, d.lane[l], d.lane[d.L + l], Fu, Fd);
    double e = fma(m.m[0], st.d, k < d.S ? sigma : 0.0) * iw;
    g = gam;
    put(Fu, 0.0, 0.0, 0.0);
    const double F0 = s_x[0][tid - k + d.S - 1];
    for (int h = 1; h < Sp; h <<= 1) {   // upward: the segments k, k + 1, ...
        put(g, e, 0.0, 0.0);
        if (k + h < Sp) {
            e = fma(g, s_x[1][tid + h], e);
            g *= s_x[0][tid + h];
        }
    }
    put(fma(g, F0, e), 0.0, 0.0, 0.0);   // F_up at the segment's top
    if (!act) return;
    seg(SF_C) = st.c;
    seg(SF_EPS) = st.eps;
    seg(SF_D) = st.d;
    seg(SF_FBOT) = k + 1 < d.S ? s_x[0][tid + 1] : F0;
}

// ---------------------------------------------------------------- back
template <bool MIXED>
__global__ void __launch_bounds__(512) k_cascade_back(const SolveArgs a)
{
    extern __shared__ double smem[];   // per wavefront [13][64]: rows of sums, before them maps
    const CascadeLayout d = cascade_layout(a);
    const int NB = a.NB, NG = a.NG, N = a.N, tid = threadIdx.x, c = blockIdx.y, s = blockIdx.x;
    const int wave = wave_uniform(tid >> 6), ln = tid & 63, NBp = 1 << d.lNBp, gl = ln >> d.lNBp, g0 = wave * d.gw;
    const Part me = part_at(a, d, s, g0 + gl);
    const int yb = ln & (NBp - 1), b = min(yb, NB - 1);
    const bool act = g0 + gl < me.n && yb < NB;
    const long long l = (long long)c * NB + b;
    auto shared_at = [&](int v, int t) -> double & { return smem[(t >> 6) * (13 * 64) + v * 64 + (t & 63)]; };
    double *s_val = smem + wave * (13 * 64), *s_net = s_val + 9 * 64;   // [8][kStride], [group][8]
    const double2 *coef = d.coef + (((long long)c * d.S + s) * d.waves + wave) * (kPart * 2 * 64) + ln;
    double2 x[kPart], y[kPart];
#pragma unroll
    for (int q = 0; q < kPart; ++q) {
        x[q] = coef[q * 128];
        if constexpr (MIXED) y[q].x = coef[q * 128 + 64].x;
        else y[q] = coef[q * 128 + 64];
    }
    StateMap m;
#pragma unroll
    for (int v = 0; v < 11; ++v) m.m[v] = d.part[((long long)v * d.T + me.i) * d.L + l];
    const double sigma = d.part[(11ll * d.T + me.i) * d.L + l];
    auto seg = [&](int f) -> double { return d.seg[((long long)f * d.S + s) * d.L + l]; };
    ElimState st = {seg(SF_C), seg(SF_EPS), seg(SF_D)};
    double Fu = seg(SF_FBOT);
    auto below = [&](int f) -> double { return d.seg[((long long)f * d.S + min(s + 1, d.S - 1)) * d.L + l]; };
    const double c_below = below(SF_C), d_below = below(SF_D);
    const double wgt = act ? (NG == 1 ? 1.0 : a.wg[b % NG]) : 0.0;
    // this thread's output: row q8 (level) of group gs
    const int q8 = ln & 7, gs = ln >> d.lNBp;
    const Part sg = part_at(a, d, s, g0 + gs);
    const bool out = (ln >> 3 & ((NBp >> 3) - 1)) == 0 && g0 + gs < sg.n;
    const bool sub = a.sub != 0;
    const int lev = N - sg.e1 + q8;   // row 0: the part's lowest level
    const int n = sg.e1 - sg.e, levc = min(lev, N);
    const double beam = *level_out(a, a.F_beam, a.F_beam_c, levc, c);
    const int j = min(sub ? levc >> 1 : levc, (sub ? N >> 1 : N) - 1);
    const long long oj = (long long)j * a.C + c;
    const double p0 = a.p[oj], p1 = a.p[oj + a.C], pm = sub ? a.pc[oj] : 0.0;

    // the state at the part's top, F_up at its bottom
#pragma unroll
    for (int v = 0; v < 11; ++v) shared_at(v, tid) = m.m[v];
    __syncthreads();
    for (int k = me.j; k > 0; --k) {
        StateMap up;
#pragma unroll
        for (int v = 0; v < 11; ++v) up.m[v] = shared_at(v, tid - (k << d.lNBp) - ((g0 + gl - me.j) << d.lNBp));
        up.apply(st);
    }
    const double iw = rcp(fma(m.m[0], st.eps, m.m[1]));
    shared_at(11, tid) = m.m[7] * iw;
    shared_at(12, tid) = fma(m.m[0], st.d, sigma) * iw;
    __syncthreads();
    for (int k = me.n - 1 - me.j; k > 0; --k) {
        const int t = tid + (k << d.lNBp);
        Fu = fma(shared_at(11, t), Fu, shared_at(12, t));
    }
    __syncthreads();

    // the part's records, in place of its coefficients; other parts' steps are layers that
    // change nothing
#pragma unroll
    for (int q = 0; q < kPart; ++q) {
        double t, r, omr, A, Sup, Sdn;
        if constexpr (MIXED) {
            unpack_mixed(x[q], t, r, omr, A);
            Sup = double(__int_as_float(__double2loint(y[q].x)));
            Sdn = double(__int_as_float(__double2hiint(y[q].x)));
        } else {
            load_layer({x[q].x, x[q].y}, t, r, omr, A);
            Sup = y[q].x, Sdn = y[q].y;
        }
        ElimState nx = st;
        const BackRec rec = elim_step(nx, t, r, omr, A, Sup, Sdn);
        const bool own = q >= me.skip;
        x[q] = own ? make_double2(rec.G, rec.H) : make_double2(1.0, 0.0);
        y[q] = own ? make_double2(rec.c, rec.d) : make_double2(0.0, 0.0);
        if (own) st = nx;
    }
    // F_dn at the part's bottom: at a segment's, by the state that the next one starts from
    // (mixed precision: its c and eps are rescaled to 1, the elimination's are not)
    const bool last = me.j == me.n - 1 && s < d.S - 1;
    double Fd = fma(last ? c_below : st.c, Fu, last ? d_below : st.d);
    double up[kPart + 1], dn[kPart + 1];
    up[0] = Fu;
    dn[0] = Fd;
#pragma unroll
    for (int q = 0; q < kPart; ++q) {
        const double2 xg = x[kPart - 1 - q], yc = y[kPart - 1 - q];
        back_step(xg.x, xg.y, yc.x, yc.y, Fu, Fd);
        up[q + 1] = Fu;
        dn[q + 1] = Fd;
    }
    const int bot = N - me.e1, own = me.e1 - me.e;
    const bool low = me.i == d.T - 1;
    if (act && (a.F_up_bin || a.F_dn_bin)) {
#pragma unroll
        for (int r = 0; r <= kPart; ++r) {
            if (r > own || (r == 0 && !low)) continue;
            if (a.F_up_bin) a.F_up_bin[(long long)(bot + r) * d.L + l] = up[r];
            if (a.F_dn_bin) a.F_dn_bin[(long long)(bot + r) * d.L + l] = dn[r];
        }
    }
#pragma unroll
    for (int r = 0; r <= kPart; ++r) s_val[r * kStride + ln] = wgt * up[r];
    const double su = group_sum(s_val, d.lNBp);
#pragma unroll
    for (int r = 0; r <= kPart; ++r) s_val[r * kStride + ln] = wgt * dn[r];
    const double sd = group_sum(s_val, d.lNBp);
    const double fn = su - sd - beam;
    if (out) s_net[gs * 8 + q8] = fn;
    wave_sync();
    if (out && q8 <= n) {
        uint32_t fl = 0u;
        if (q8 > 0 || sg.i == d.T - 1) {
            *level_out(a, a.F_up, a.F_up_c, lev, c) = su;
            *level_out(a, a.F_dn, a.F_dn_c, lev, c) = sd;
            *level_out(a, a.F_net, a.F_net_c, lev, c) = fn;
            if (!isfinite(fn)) fl |= F_NONFIN;
        }
        const int step = sub ? 2 : 1;
        if (q8 + step <= n && !(sub && (lev & 1))) {
            const double dp = p0 - p1;
            bool bad = !(dp > 0.0);
            if (sub) bad = bad || !(p0 > pm && pm > p1);
            if (bad) fl |= F_INVALID;
            const double qh = a.o.gravity * (fn - s_net[gs * 8 + q8 + step]) / dp;
            a.heat[oj] = qh;
            if (a.dTdt) a.dTdt[oj] = qh / a.o.cp;
        }
        if (fl) {
            if (a.flags) atomicOr(&a.flags[c], fl);
            const uint32_t bad = status_bits(fl);
            if (a.status && bad) atomicOr(a.status, bad);
        }
    }
    if (a.F_up_toa_bin && s == 0 && wave == 0) {   // (part 0: group 0)
        wave_sync();
        if (NG == 1) {
            if (act && me.i == 0) a.F_up_toa_bin[l] = up[kPart];
        } else {
            if (gl == 0) s_val[ln] = up[kPart];
            wave_sync();
            const int NBR = NB / NG;
            for (int r = ln; r < NBR; r += 64) {
                double t = 0.0;
                for (int g = 0; g < NG; ++g) t += a.wg[g] * s_val[r * NG + g];
                a.F_up_toa_bin[(long long)c * NBR + r] = t;
            }
        }
    }
}

}  // namespace

// Segments of an even number of slabs on the sub-layer grid (a part's layers are whole).
bool cascade_fits(const Geometry &g, int C, int N, int NB, int NG, bool sub, const DeviceLimits &dev)
{
    const int S = g.K, Ls = g.PC;
    if (NB > 64 || N < kPart || Ls < kPart || S > kScanThreads || C > 65535 || (sub && Ls % 2)) return false;
    const CascadeLayout d = cascade_layout(C, N, NB, S, Ls, nullptr);
    return d.waves <= 8 && cascade_doubles(C, N, NB, S, Ls) * sizeof(double) <= g.scratch &&
           items_lds(d.gw, d.waves, NB / NG, deep_items_rows(Ls, NB, NB / NG, true), false).total <= dev.lds;
}

hipError_t launch_cascade(const SolveArgs &a0, const Geometry &g, int precision, hipStream_t s)
{
    SolveArgs a = a0;
    a.K = g.K;    // segments per column
    a.PC = g.PC;  // slabs per segment
    const CascadeLayout d = cascade_layout(a.C, a.N, a.NB, a.K, a.PC, a.scratch);
    const bool mixed = precision == 1;
    a.CH = deep_items_rows(g.PC, a.NB, a.NB / a.NG, mixed);   // partial sums of the optical depth
    const size_t lds = items_lds(d.gw, d.waves, a.NB / a.NG, a.CH, mixed).total, lds_back = d.waves * 13 * 64 * sizeof(double);
    const dim3 segments(d.S, a.C), threads(64 * d.waves);
    if (a.in_f32) hipLaunchKernelGGL(k_cascade_tau<float>, segments, dim3(64), 0, s, a);
    else hipLaunchKernelGGL(k_cascade_tau<double>, segments, dim3(64), 0, s, a);
    if (!mixed) hipLaunchKernelGGL((k_cascade_items<false, false>), segments, threads, lds, s, a);
    else if (a.in_f32) hipLaunchKernelGGL((k_cascade_items<true, true>), segments, threads, lds, s, a);
    else hipLaunchKernelGGL((k_cascade_items<true, false>), segments, threads, lds, s, a);
    const int lanes = kScanThreads / scan_threads(d.S);
    hipLaunchKernelGGL(k_cascade_scan, dim3((unsigned)((d.L + lanes - 1) / lanes)), dim3(kScanThreads), 0, s, a);
    if (mixed) hipLaunchKernelGGL(k_cascade_back<true>, segments, threads, lds_back, s, a);
    else hipLaunchKernelGGL(k_cascade_back<false>, segments, threads, lds_back, s, a);
    return hipGetLastError();
}

hipError_t prepare_cascade_kernels(const DeviceLimits &dev)
{
    const void *fns[] = {reinterpret_cast<const void *>(&k_cascade_items<false, false>),
                         reinterpret_cast<const void *>(&k_cascade_items<true, false>),
                         reinterpret_cast<const void *>(&k_cascade_items<true, true>)};
    for (const void *f : fns) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dev.lds);
        if (e != hipSuccess) return e;
    }
    return upload_planck_table();
}

}  // namespace rtk
