// rt_stream.hip -- the wavefront-per-lanes solve for grids that fill the chip.
//
// Paper: Deitrick et al., "The THOR+HELIOS general circulation model"
// (arXiv 2203.02293): the same per-layer arithmetic as the other solve kernels
// (Section 2.2.1, Appendix B, `rt_physics.hpp`) and the same Thomas recurrence
// (Section 2.2.2).
//
// A wavefront owns 64 lanes ((column, bin) pairs) for the whole sweep: whole
// columns of up to 64 lanes, each padded to a power of two, or 64 lanes of one
// wider column.  It walks its layers from the TOA without a barrier: Planck
// edge integrals of a few levels at a time go through LDS rows of its own, and
// the layer coefficients feed the elimination in registers, so no item is
// handed between threads.  The back-substitution records (32 bytes per layer
// and lane) go through memory; the bin sums of each level are wavefront sums,
// kept in LDS until the workgroup's one barrier before the outputs.
#include "rt_internal.hpp"
#include "rt_math.hpp"
#include "rt_physics.hpp"
#include "rt_wave.hpp"

#include <algorithm>
#include <type_traits>

namespace rtk {
namespace {

constexpr int kStreamThreads = 768;   // workgroup size bound: twelve wavefronts of a column of 768 lanes

// Levels of one chunk: their Planck edge integrals share a pass, and so do their
// column sums.
constexpr int kChunk = 8;
constexpr int kSumStride = 65;   // doubles per row of lane values to be summed (odd: rows start in different banks)

// Lane layout of a problem: NBp padded lanes per column (a power of two from 8
// to 64, or a multiple of 64), gw columns per wavefront, NBw wavefronts per column.
struct LaneLayout {
    int NBp, gw, NBw;
};
__host__ __device__ __forceinline__ LaneLayout lane_layout(int NB)
{
    LaneLayout l;
    int p = 8;
    while (p < NB && p < 64) p *= 2;
    l.NBp = NB > 64 ? (NB + 63) / 64 * 64 : p;
    l.gw = NB > 64 ? 1 : 64 / p;
    l.NBw = NB > 64 ? l.NBp / 64 : 1;
    return l;
}

// Planck edges that one wavefront needs at most: its lanes' bins and one more.
__host__ __device__ __forceinline__ int wave_edges(int NB, int NG)
{
    const int NBR = NB / NG;
    const int most = NB > 64 ? (NG == 1 ? 64 : 63 / NG + 2) : NBR;
    return (most < NBR ? most : NBR) + 1;
}

struct StreamLds {
    int estride;                         // edge values per row (odd: rows start in different banks)
    size_t wave, per_wave;               // a wavefront's own region: its start and size
    size_t edge, val, temp;              // in it: R [gw kChunk][estride]; double [kChunk][kSumStride], twice
                                         // (the second one in place of the edges); double [gw kChunk]
    size_t c2, sum, top, flag, total;
};
__host__ __device__ __forceinline__ StreamLds stream_lds(int N, int NB, int NG, int K, int waves, bool mixed)
{
    const LaneLayout ll = lane_layout(NB);
    StreamLds o;
    o.estride = wave_edges(NB, NG) | 1;
    const size_t rows = (size_t)ll.gw * kChunk, buf = kChunk * kSumStride * 8;
    const size_t e = (rows * o.estride * (mixed ? 4 : 8) + 7) & ~size_t(7);
    o.temp = 0;
    o.val = rows * 8;
    o.edge = o.val + buf;
    o.per_wave = o.edge + (e > buf ? e : buf);
    o.wave = 0;
    o.c2 = (size_t)waves * o.per_wave;                                  // double [NBR+1]
    o.sum = o.c2 + (size_t)(NB / NG + 1) * 8;                           // double [N+1][3][NBw][K]
    o.top = o.sum + (size_t)(N + 1) * 3 * ll.NBw * K * 8;               // double [K][NB] (NG > 1)
    o.flag = o.top + (NG > 1 ? (size_t)K * NB * 8 : 0);                 // uint32 [K]
    o.total = (o.flag + 4 * (size_t)K + 15) & ~size_t(15);
    return o;
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

// LDS values written by lanes of this wavefront are read by others of it.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <bool MIXED, bool IN32>
__device__ __forceinline__ void solve_tile_stream(ArgsK ap, const int tile)
{
    using R = typename std::conditional<MIXED, float, double>::type;
    using InT = typename std::conditional<IN32, float, double>::type;
    extern __shared__ double smem[];
    char *lds = reinterpret_cast<char *>(smem);
    // the arguments, re-read in each phase (ArgsK)
    auto args = [&]() -> const SolveArgs & { return *(const SolveArgs *)ap; };
    const int NB = args().NB, NG = args().NG, C = args().C, N = args().N, K = args().K;
    const int tid = threadIdx.x, wave = wave_uniform(tid >> 6), ln = tid & 63;
    const LaneLayout ll = lane_layout(NB);
    const StreamLds lo = stream_lds(N, NB, NG, K, blockDim.x >> 6, MIXED);
    const int c0 = tile * K, NBR = NB / NG;
    // this thread's column of the tile and lane of the column; the padding takes
    // the values of the last lane or column and writes nothing
    const int grp = ll.gw == 1 ? 0 : ln / ll.NBp;
    const int kk = NB > 64 ? 0 : wave * ll.gw + grp;
    const int yb = NB > 64 ? tid : ln - grp * ll.NBp;
    const int c = min(c0 + kk, C - 1), b = min(yb, NB - 1);
    const bool act = yb < NB && c0 + kk < C;
    const int lane0 = NB > 64 ? wave * 64 : 0;              // first lane of the wavefront's column slice
    const int bin0 = NG == 1 ? lane0 : lane0 / NG;
    const int lastl = min(NB > 64 ? lane0 + 63 : NB - 1, NB - 1);
    const int ne = (NG == 1 ? lastl : lastl / NG) - bin0 + 2;   // edges of the wavefront's bins
    const int bin = NG == 1 ? b : b / NG, rb = bin - bin0;
    const bool sub = args().sub != 0;

    char *own = lds + lo.wave + (size_t)wave * lo.per_wave;
    R *s_edge = reinterpret_cast<R *>(own + lo.edge);
    double *s_val = reinterpret_cast<double *>(own + lo.val), *s_val2 = reinterpret_cast<double *>(own + lo.edge);
    double *s_T = reinterpret_cast<double *>(own + lo.temp);
    double *s_c2 = reinterpret_cast<double *>(lds + lo.c2);
    double *s_sum = reinterpret_cast<double *>(lds + lo.sum);
    double *s_top = reinterpret_cast<double *>(lds + lo.top);
    uint32_t *s_flag = reinterpret_cast<uint32_t *>(lds + lo.flag);

    for (int k = tid; k < K; k += blockDim.x) s_flag[k] = 0u;
    for (int e = tid; e <= NBR; e += blockDim.x) s_c2[e] = args().c2_over_lam[e];
    const long long LB = (long long)C * NB;
    const unsigned lane = (unsigned)c * NB + b;   // of a [C][NB] plane
    uint32_t fl = 0u;
    const double mu = args().mu[c];
    const double Ti = args().Tint[c];
    const bool day = mu > 0.0, wday = wave_any(day);
    if (!isfinite(mu) || !(Ti >= 0.0) || !isfinite(Ti)) fl |= F_INVALID;
    const double inv_mu = day ? 1.0 / mu : 0.0;
    const double muF = day ? mu * args().F_star[bin] : 0.0;
    const double inv_eps2 = 1.0 / args().o.eps2;
    const double wgt = act ? (NG == 1 ? 1.0 : args().wg[b % NG]) : 0.0;
    float c2fb = 0.0f, c2fa = 0.0f;   // c2 / lambda at this lane's bin edges
    if constexpr (MIXED) {
        c2fb = args().c2_over_lam_f[bin];
        c2fa = args().c2_over_lam_f[bin + 1];
    }
    ElimState st = elim_top(args().Ftoa ? args().Ftoa[lane] : 0.0);
    __syncthreads();

    auto T_at = [&](int l, int cc) -> double {
        const double *T_if = args().T, *T_ce = sub ? args().Tc : args().T;
        const double *base = (sub && (l & 1)) ? T_ce : T_if;
        return base[(long long)(sub ? (l >> 1) : l) * C + cc];
    };
    // Planck edge integrals of a chunk of n levels into rows (column of the
    // wavefront, level): this lane keeps one row and steps through its edges, so
    // a wavefront's lanes sit in neighbouring edges (one series regime mostly) and
    // the row's temperature stays in a register.  Its row's column and level:
    const int lrows = 31 - __builtin_clz(ll.gw * kChunk);
    const int row = ln & (ll.gw * kChunk - 1), e0 = ln >> lrows, epr = 64 >> lrows;
    const int rq = row & (kChunk - 1), rk = NB > 64 ? 0 : wave * ll.gw + row / kChunk;
    const int rc = min(c0 + rk, C - 1);
    auto edges = [&](double T, int n) {
        if (rq < n) {
            const double iT = rcp(T);
            if (e0 == 0) s_T[row] = T;
            for (int e = e0; e < ne; e += epr) s_edge[row * lo.estride + e] = planck_edge<R>(s_c2[bin0 + e] * iT);
        }
        wave_sync();
    };
    auto bin_B = [&](int q) -> R {
        const int rw = grp * kChunk + q;
        const double Td = s_T[rw];
        const R Tr = R(Td), T2 = Tr * Tr;
        const R *re = s_edge + rw * lo.estride + rb;
        R I = planck_combine<R>(re[0], re[1]);
        if constexpr (MIXED) {
            const R iT = rcp(Tr);
            const R xb = c2fb * iT, xa = c2fa * iT;
            if (planck_narrow(xa, xb)) {
                const double iTd = rcp(Td);
                I = planck_gl3(s_c2[bin + 1] * iTd, s_c2[bin] * iTd);
            }
        }
        return R(kPref) * T2 * T2 * I;
    };
    // Column sums of n rows of lane values v (LDS, kSumStride apart) into the sums
    // of levels l0, l0 + dl, ...: lane (q, p) = (ln % 8, ln / 8) adds the 8 lanes
    // p of row q, then the parts of a column are added.  Fixed order.
    const int sstep = ll.NBw * K;
    double *const sum0 = s_sum + (size_t)(NB > 64 ? wave : 0) * K;
    auto sum_rows = [&](const double *v, int which, int l0, int dl, int n) {
        wave_sync();
        const int q = ln & 7, p = ln >> 3;
        const double *r = v + q * kSumStride + p * 8;
        double s = r[0];
#pragma unroll
        for (int k = 1; k < 8; ++k) s += r[k];
        if (ll.NBp > 8) s += __shfl_xor(s, 8);
        if (ll.NBp > 16) s += __shfl_xor(s, 16);
        if (ll.NBp > 32) s += __shfl_xor(s, 32);
        const int np = ll.NBp >= 64 ? 8 : ll.NBp >> 3, g = p / np;
        if (q < n && p == g * np)
            sum0[(size_t)(3 * (l0 + dl * q) + which) * sstep + (NB > 64 ? 0 : wave * ll.gw + g)] = s;
        wave_sync();
    };

    // T_int, level N and, where the number of layers is odd, level N - 1: rows
    // 0, 1 and 2 of a chunk of their own
    const int odd = N & 1;
    double Tc_ = rq == 0 ? args().Tint[rc] : T_at(max(N + 1 - rq, 0), rc);
    double Tn_ = T_at(max(N - 1 - odd - rq, 0), rc);
    auto check_T = [&](double T, bool in) {
        if (in && (!(T > 0.0) || !isfinite(T))) atomicOr(&s_flag[rk], (uint32_t)F_INVALID);
    };
    check_T(Tc_, rq == 1 || (rq == 2 && odd));
    edges(Tc_, 2 + odd);
    const double Fboa = double(kPI) * double(bin_B(0));
    R Bup = bin_B(1);
    double Fb_up = muF, tau = 0.0;
    const unsigned o_in = lane * (unsigned)sizeof(InT), o_rec = lane * 16u;
    // The inputs of a layer are loaded two layers ahead, into the registers that
    // the layer before has just used (a copy between registers would wait for
    // the load, and with it for the record stores before it).
    InT dt0, w0, g0, dt1, w1, g1;
    auto load = [&](int i, InT &dt, InT &w, InT &g) {   // (past the last layer: layer 0 again, unused)
        const long long o = (long long)max(i, 0) * LB;
        dt = at(reinterpret_cast<const InT *>(args().dtau) + o, o_in);
        w = at(reinterpret_cast<const InT *>(args().w0) + o, o_in);
        g = at(reinterpret_cast<const InT *>(args().g0) + o, o_in);
    };
    load(N - 1 - odd, dt0, w0, g0);
    load(N - 2 + odd, dt1, w1, g1);   // (odd: layer N - 1, then layer N - 3 in its place)
    Opts o;
    auto options = [&]() {   // (read anew in each chunk)
        opaque_args(ap);
        o = args().o;
        uniform_value(o.e_tau);
        uniform_value(o.g_guard);
        uniform_value(o.improved);
        uniform_value(o.noniso);
        uniform_value(o.e_clamp);
    };
    // layer i, its lower level's Planck edges in row q, its beam value into row v.
    // (The padding stores its lane's record again: same values, and the loads'
    // waits then pass the stores, whose number is the same for every wavefront.)
    auto layer = [&](int i, int q, int v, InT &dt_, InT &w_, InT &g_) {
        const R B = bin_B(q);
        double Fb_lo = 0.0;
        const double dt = double(dt_);
        if (day) {
            tau += dt;   // summed from the TOA, as the optical depth is defined
            Fb_lo = beam_at<MIXED>(muF, tau, inv_mu);
        }
        const Layer<R> Ly = layer_item<MIXED, R, MIXED>(dt, double(w_), double(g_), day, mu, inv_mu, Fb_up, Fb_lo,
                                                        B, Bup, o, inv_eps2, fl);
        load(i - 2, dt_, w_, g_);
        const BackRec rec = elim_step(st, double(Ly.t), double(Ly.r), double(Ly.omr), double(Ly.A),
                                      double(Ly.Sup), double(Ly.Sdn));
        double2 *p_rec = reinterpret_cast<double2 *>(args().scratch) + (long long)i * 2 * LB;
        at(p_rec, o_rec) = make_double2(rec.G, rec.H);
        at(p_rec + LB, o_rec) = make_double2(rec.c, rec.d);
        if (wday) s_val[v * kSumStride + ln] = wgt * Fb_lo;
        Fb_up = Fb_lo;
        Bup = B;
    };
    options();
    if (wday) s_val[ln] = wgt * muF;   // beam at level N
    if (odd) layer(N - 1, 2, 1, dt1, w1, g1);
    if (wday) sum_rows(s_val, 2, N, -1, 1 + odd);
    // chunks of an even number of layers, in pairs
    for (int hi = N - 1 - odd; hi >= 0; hi -= kChunk) {
        const int n = min(kChunk, hi + 1);
        options();
        Tc_ = Tn_;
        check_T(Tc_, rq < n);
        edges(Tc_, n);
        Tn_ = T_at(max(hi - kChunk - rq, 0), rc);   // (the chunk after this one's)
#pragma unroll 1
        for (int q = 0; q < n; q += 2) {
            layer(hi - q, q, q, dt0, w0, g0);
            layer(hi - q - 1, q + 1, q + 1, dt1, w1, g1);
        }
        if (wday) sum_rows(s_val, 2, hi, -1, n);
    }
    if (fl) atomicOr(&s_flag[kk], fl);

    double Fu, Fd, Fu_toa = 0.0;
    elim_boa(st, Fboa, Fb_up, Fu, Fd);
    // back-substitution in chunks of levels; a lane's records are loaded RD
    // levels ahead of their use.  Every chunk runs whole (past level N on the last
    // record again, into rows that are not summed), so no load is under a branch.
    constexpr int RD = MIXED ? 4 : 8;
    opaque_args(ap);
    const double2 *q_rec = reinterpret_cast<const double2 *>(args().scratch);
    double2 r0[RD], r1[RD];
    int jn = 0;   // next record
    auto ld = [&](int k) {
        r0[k] = at(q_rec, o_rec);
        r1[k] = at(q_rec + LB, o_rec);
        q_rec += ++jn < N ? 2 * LB : 0;
    };
    r0[0] = make_double2(1.0, 0.0);   // level 0: the fluxes stay as they are
    r1[0] = make_double2(0.0, Fd);
#pragma unroll
    for (int k = 1; k < RD; ++k) ld(k);
    const bool bins = args().F_up_bin || args().F_dn_bin;
    for (int i0 = 0; i0 <= N; i0 += kChunk) {
        opaque_args(ap);
#pragma unroll
        for (int k = 0; k < kChunk; ++k) {
            const int i = i0 + k;
            back_step(r0[k % RD].x, r0[k % RD].y, r1[k % RD].x, r1[k % RD].y, Fu, Fd);
            ld(k % RD);
            s_val[k * kSumStride + ln] = wgt * Fu;
            s_val2[k * kSumStride + ln] = wgt * Fd;
            if (i == N) Fu_toa = Fu;
            if (bins && act && i <= N) {
                if (args().F_up_bin) args().F_up_bin[i * LB + lane] = Fu;
                if (args().F_dn_bin) args().F_dn_bin[i * LB + lane] = Fd;
            }
        }
        const int n = min(kChunk, N + 1 - i0);
        sum_rows(s_val, 0, i0, 1, n);
        sum_rows(s_val2, 1, i0, 1, n);
    }
    if (act && args().F_up_toa_bin) {
        if (NG == 1) args().F_up_toa_bin[lane] = Fu_toa;
        else s_top[kk * NB + b] = Fu_toa;
    }
    __syncthreads();

    // outputs: the column sums of each level (over a wide column's wavefronts, in
    // order), net flux and heating
    opaque_args(ap);
    auto col_sum = [&](int lev, int v, int k) -> double {
        const double *p = s_sum + (size_t)(3 * lev + v) * sstep + k;
        double s = p[0];
        for (int w = 1; w < ll.NBw; ++w) s += p[(size_t)w * K];
        return s;
    };
    auto out_at = [&](double *iface, double *centre, int l, int cc) -> double * {
        if (sub) return ((l & 1) ? centre : iface) + (long long)(l >> 1) * C + cc;
        return iface + (long long)l * C + cc;
    };
    for (int t = tid; t < (N + 1) * K; t += blockDim.x) {
        const int lev = t / K, k = t - lev * K, cc = c0 + k;
        if (cc >= C) continue;
        const bool dk = args().mu[cc] > 0.0;   // (night columns have no beam sums)
        auto net = [&](int l, double &su, double &sd, double &sb) -> double {
            su = col_sum(l, 0, k);
            sd = col_sum(l, 1, k);
            sb = dk ? col_sum(l, 2, k) : 0.0;
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
    if (NG > 1 && args().F_up_toa_bin) {
        for (int t = tid; t < K * NBR; t += blockDim.x) {
            const int k = t / NBR, r = t - k * NBR, cc = c0 + k;
            if (cc >= C) continue;
            const double *f = s_top + k * NB + r * NG;
            double s = 0.0;
            for (int g = 0; g < NG; ++g) s += args().wg[g] * f[g];
            args().F_up_toa_bin[(long long)cc * NBR + r] = s;
        }
    }
    __syncthreads();
    for (int k = tid; k < K; k += blockDim.x) {
        if (c0 + k >= C) continue;
        if (args().flags) args().flags[c0 + k] = s_flag[k];
        const uint32_t bad = status_bits(s_flag[k]);
        if (args().status && bad) atomicOr(args().status, bad);
    }
}

template <bool MIXED, bool IN32 = false>
__global__ void __launch_bounds__(kStreamThreads, MIXED ? 4 : 3) k_solve_stream(const SolveArgs a)
{
    solve_tile_stream<MIXED, IN32>(kernel_args(a), blockIdx.x);
}

// Workgroup of request r with first[r] <= g < first[r+1] (batched launches).
__device__ __forceinline__ int batch_slot(const int *first, int n, int g)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (first[mid] <= g) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

template <bool MIXED, bool IN32 = false>
__global__ void __launch_bounds__(kStreamThreads, MIXED ? 4 : 3)
k_solve_stream_batch(const SolveArgs *__restrict__ reqs, const int *__restrict__ first, int n)
{
    const int r = batch_slot(first, n, blockIdx.x);
    solve_tile_stream<MIXED, IN32>((ArgsK)(reqs + r), blockIdx.x - first[r]);
}

}  // namespace

Geometry stream_geometry(int C, int N, int NB, int NG, bool mixed, const DeviceLimits &dev)
{
    Geometry g{};
    // 32-bit byte offsets of a lane's record in a plane of lanes
    if ((long long)C * NB >= (1ll << 28)) return g;
    const LaneLayout ll = lane_layout(NB);
    // A wavefront's sweep takes as long however few others there are, so the grid
    // has to bring more than one per SIMD: at five per compute unit (2562 columns
    // x 40 layers x 30 bins: 1284 on 256) it is even with the layer kernel, whose
    // time falls with the columns (FP64 131 against 140 us, mixed 93 against 96).
    const long long all_waves = NB > 64 ? (long long)C * ll.NBw : (C + ll.gw - 1) / ll.gw;
    if (all_waves < 5ll * (dev.n_cu > 0 ? dev.n_cu : 256)) return g;
    int waves = NB > 64 ? ll.NBw : 4;
    g.kernel = KERNEL_STREAM;
    for (;; waves /= 2) {
        g.K = NB > 64 ? 1 : waves * ll.gw;
        g.lds = stream_lds(N, NB, NG, g.K, waves, mixed).total;
        if (g.lds <= dev.lds) break;
        if (NB > 64 || waves == 1) return Geometry{};
    }
    g.threads = waves * 64;
    g.blocks = (C + g.K - 1) / g.K;
    g.lanes = (long long)C * NB;
    g.scratch = (size_t)N * 4 * (size_t)g.lanes * sizeof(double);
    return g;
}

hipError_t launch_stream(const SolveArgs &a, const Geometry &g, int precision, hipStream_t s)
{
    SolveArgs b = a;
    b.K = g.K;
    b.L = g.lanes;
    const dim3 grid(g.blocks), block(g.threads);
    if (precision != 1) hipLaunchKernelGGL((k_solve_stream<false>), grid, block, g.lds, s, b);
    else if (a.in_f32) hipLaunchKernelGGL((k_solve_stream<true, true>), grid, block, g.lds, s, b);
    else hipLaunchKernelGGL((k_solve_stream<true>), grid, block, g.lds, s, b);
    return hipGetLastError();
}

hipError_t launch_stream_batch(const SolveArgs *d_reqs, const int *d_first, int n, int total_blocks,
                               const Geometry &g, int precision, int in_f32, hipStream_t s)
{
    const dim3 grid(total_blocks), block(g.threads);
    if (precision != 1) hipLaunchKernelGGL((k_solve_stream_batch<false>), grid, block, g.lds, s, d_reqs, d_first, n);
    else if (in_f32) hipLaunchKernelGGL((k_solve_stream_batch<true, true>), grid, block, g.lds, s, d_reqs, d_first, n);
    else hipLaunchKernelGGL((k_solve_stream_batch<true>), grid, block, g.lds, s, d_reqs, d_first, n);
    return hipGetLastError();
}

hipError_t prepare_stream_kernels(const DeviceLimits &dev)
{
    const void *fns[] = {reinterpret_cast<const void *>(&k_solve_stream<false>),
                         reinterpret_cast<const void *>(&k_solve_stream<true>),
                         reinterpret_cast<const void *>(&k_solve_stream<true, true>),
                         reinterpret_cast<const void *>(&k_solve_stream_batch<false>),
                         reinterpret_cast<const void *>(&k_solve_stream_batch<true>),
                         reinterpret_cast<const void *>(&k_solve_stream_batch<true, true>)};
    for (const void *f : fns) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dev.lds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace rtk
