// rt_stream.hip -- the wavefront-per-lanes solve: the default tile of the layer
// kernel.
//
// Paper: Deitrick et al., "The THOR+HELIOS general circulation model"
// (arXiv 2203.02293): the same per-layer arithmetic as the other solve kernels
// (Section 2.2.1, Appendix B, `rt_physics.hpp`) and the same Thomas recurrence
// (Section 2.2.2).
//
// A wavefront owns up to 64 lanes ((column, bin) pairs, rt_lanes.hpp) and walks
// their layers from the TOA without a barrier: Planck edge integrals of eight
// levels at a time go through LDS rows of its own, and the layer coefficients feed
// the elimination in registers, so no item is handed between threads.  The
// back-substitution records (32 bytes per layer and lane) go through memory, where
// the L2 still holds most of them when they are read back; the level sums are taken
// eight levels at a time.  One wavefront is one workgroup (four in one kept registers and
// LDS until the slowest ended: 17 percent of the time).  2562 x 40 x 30 x 20 lanes FP64: 2.91 ms
// by the layer kernel, 1.01 here; 10242 x 80 x 300 mixed: 7.42 and 4.23, both at about the
// rate of memory for inputs and records.
//
// Where a grid brings fewer wavefronts than the chip runs (SEG), a wavefront's own
// chain of dependent FP64 operations (about 2 us per layer) is the time.  Each
// column's layers are then split into S segments from the TOA, one group of lanes each,
// in the same wavefront (while a column's lanes fill at most half of one) or in several
// of one workgroup.  Each segment composes the elimination's map over its layers on
// the way and leaves their coefficients in the records' place; the maps give the state
// at every segment's top, from which all segments eliminate, and compose their maps of
// F_up, with which all substitute back (StateMap; 64 bytes more per layer and lane).  162 x 40 x
// 30 FP64: 50 us by the layer kernel, 83 in one segment, 25 in eight; 2562 x 40 x 30: 140, 111
// and 95 in two.  (Handing the elimination from segment to segment instead, without the
// maps, took 34 us and 138.)
#include "rt_lanes.hpp"

#include <algorithm>
#include <type_traits>

namespace rtk {
namespace {

// Levels of one chunk: their Planck edge integrals share a pass, and so do their
// column sums.
constexpr int kChunk = 8;
constexpr int kSumStride = 65;        // doubles per row of lane values to be summed (odd: rows start in different banks)
constexpr int kStreamThreads = 768;   // workgroup size bound

// What the kernel needs of a problem's layout beside its sizes, worked out on the
// host (SolveArgs::CH and L): integer divisions cost a wavefront about a thousand cycles
// in its first microsecond.
struct StreamShape {
    int LPT;          // layers per segment, rounded up
    int NBR;          // bins: lanes per column / points per bin
    int NBw, NBs;     // LaneLayout
    int edges;        // wave_edges
    __host__ __device__ __forceinline__ long long pack() const
    {
        return (long long)NBR | (long long)NBw << 16 | (long long)NBs << 24 | (long long)edges << 32;
    }
    __host__ __device__ __forceinline__ static StreamShape unpack(int LPT, long long v)
    {
        return {LPT, (int)(v & 0xffff), (int)(v >> 16 & 0xff), (int)(v >> 24 & 0xff), (int)(v >> 32 & 0xff)};
    }
};
__host__ StreamShape stream_sizes(int N, int NB, int NG, int S)
{
    const LaneLayout ll = lane_layout(NB);
    return {(N + S - 1) / S, NB / NG, ll.NBw, ll.NBs, wave_edges(NB, NG)};
}

struct StreamLds {
    int estride;                         // edge values per row (odd: rows start in different banks)
    size_t per_wave;                     // a wavefront's own region
    size_t edge, val, temp;              // in it: R [gw kChunk][estride]; double [kChunk][kSumStride], twice
                                         // (the second one in place of the edges); LevelValue [gw kChunk]
    size_t tab, c2, sum, top, flag, total;
};
// K columns of S segments each on `waves` wavefronts: K S = gw waves
__host__ __device__ __forceinline__ StreamLds stream_lds(const StreamShape &sh, int N, int NB, int NG, int K, int gw,
                                                         int waves, bool mixed)
{
    StreamLds o;
    o.estride = sh.edges | 1;
    const size_t rows = (size_t)gw * kChunk, buf = kChunk * kSumStride * 8;
    const size_t e = (rows * o.estride * (mixed ? 4 : 8) + 7) & ~size_t(7);
    o.temp = 0;
    o.val = rows * (mixed ? 16 : 8);
    o.edge = o.val + buf;
    o.per_wave = o.edge + (e > buf ? e : buf);
    o.tab = 0;                                                                  // FP64: the Planck table
    o.c2 = (mixed ? 0 : kPlanckTable * 8) + (size_t)waves * o.per_wave;         // double [edges]
    o.sum = o.c2 + (size_t)sh.edges * 8;                                        // double [N+1][3][K]
    o.top = o.sum + (size_t)(N + 1) * 3 * K * 8;                                // double [K][NB] (NG > 1, NB <= 64)
    o.flag = o.top + (NG > 1 && NB <= 64 ? (size_t)K * NB * 8 : 0);             // uint32 [K]
    o.total = (o.flag + 4 * (size_t)K + 15) & ~size_t(15);
    return o;
}

// Back-substitution records: a workgroup's lanes (K columns, or a slice of one) hold
// theirs in one block, [layer][2][lane] double2, in the order of the lanes.  (In planes of
// all lanes the stores of thousands of wavefronts, each at its own layer, spread over
// the memory's pages: 10242 x 80 x 300 mixed, 7.9 GB of records, took 4.8 ms in place of 4.3.)  A slice of a
// wide column leaves its level sums (up, down, beam of each level) and flags for
// k_stream_columns at the start of its block, its lanes' F_up at the TOA in the last plane.
__device__ __forceinline__ double2 *record_block(double *scratch, int N, int NB, int c, int lane0)
{
    return reinterpret_cast<double2 *>(scratch) + ((long long)c * NB + lane0) * 2 * N;
}

template <bool MIXED, bool IN32, bool SEG>
__device__ __forceinline__ void solve_tile_stream(ArgsK ap, const int tile)
{
    using R = typename std::conditional<MIXED, float, double>::type;
    using InT = typename std::conditional<IN32, float, double>::type;
    extern __shared__ double smem[];
    char *lds = reinterpret_cast<char *>(smem);
    // the arguments, re-read in each phase (ArgsK)
    auto args = [&]() -> const SolveArgs & { return *(const SolveArgs *)ap; };
    const int NB = args().NB, NG = args().NG, C = args().C, N = args().N, K = args().K;
    const int S = SEG ? args().PC : 1;
    const StreamShape sh = StreamShape::unpack(args().CH, args().L);
    const int tid = threadIdx.x, wave = SEG ? wave_uniform(tid >> 6) : 0, ln = tid & 63;
    const int W = SEG ? blockDim.x : 64;
    const bool wide = NB > 64;
    int lNBp = 3;   // log2 of a group's lanes
    while (lNBp < 6 && 1 << lNBp < NB) ++lNBp;
    const int NBp = 1 << lNBp, gw = 64 >> lNBp;
    const StreamLds lo = stream_lds(sh, N, NB, NG, K, gw, W >> 6, MIXED);
    const int c0 = wide ? tile / sh.NBw : tile * K, slice = wide ? tile - c0 * sh.NBw : 0;
    // group g of the workgroup's lanes: segment g / K, column g % K, its layers at
    // positions [e, e1) from the TOA.  All segments run LPT steps, from position a = e1 -
    // LPT on (a shorter one repeats the last layer of the one above).
    const int LPT = SEG ? sh.LPT : N, shorter = SEG && S * LPT != N ? LPT - 1 : LPT, longer = SEG ? N - S * shorter : 0;
    struct Group {
        int kk, s, a, e, e1;
    };
    auto group = [&](int g) -> Group {
        Group r;
        if constexpr (SEG) {
            r.s = K == 1 ? g : small_div(g, K);
            r.kk = g - r.s * K;
            r.e = r.s * shorter + min(r.s, longer);
            r.e1 = r.e + shorter + (r.s < longer ? 1 : 0);
            r.a = r.e1 - LPT;
        } else {
            r.kk = g;
            r.s = r.e = r.a = 0;
            r.e1 = N;
        }
        return r;
    };
    const int gl = ln >> lNBp, g0 = SEG ? wave * gw : 0;
    const Group me = group(g0 + gl);
    // a wavefront of first segments alone eliminates as it goes
    const bool direct = SEG && K == gw && wave == 0;
    // this thread's lane of its column; the padding takes the values of the last lane
    // or column and writes nothing but the same records
    const int lane0 = slice * sh.NBs, nlane = wide ? min(sh.NBs, NB - lane0) : NB;
    const int yb = ln & (NBp - 1), b = lane0 + min(yb, nlane - 1), c = min(c0 + me.kk, C - 1);
    const bool act = yb < nlane && c0 + me.kk < C;
    const int bin0 = NG == 1 ? lane0 : lane0 / NG, lastl = lane0 + nlane - 1;
    const int ne = (NG == 1 ? lastl : lastl / NG) - bin0 + 2;   // edges of the wavefront's bins
    const int bin = NG == 1 ? b : b / NG, rb = bin - bin0;
    const bool sub = args().sub != 0;

    double *s_tab = reinterpret_cast<double *>(lds + lo.tab);
    char *own = lds + (MIXED ? 0 : kPlanckTable * 8) + (size_t)wave * lo.per_wave;
    R *s_edge = reinterpret_cast<R *>(own + lo.edge);
    double *s_val = reinterpret_cast<double *>(own + lo.val), *s_val2 = reinterpret_cast<double *>(own + lo.edge);
    LevelValue<MIXED> *s_level = reinterpret_cast<LevelValue<MIXED> *>(own + lo.temp);
    double *s_c2 = reinterpret_cast<double *>(lds + lo.c2) - bin0;
    double *s_sum = reinterpret_cast<double *>(lds + lo.sum);
    double *s_top = reinterpret_cast<double *>(lds + lo.top);
    // SEG: values a group leaves for the other groups of its column, in place of its
    // rows: value v of the group d above (d < 0: below) this lane's
    auto shared_at = [&](int v, int d) -> double & {
        const int t = tid + d * K * NBp;
        return *reinterpret_cast<double *>(lds + (MIXED ? 0 : kPlanckTable * 8) + (size_t)(t >> 6) * lo.per_wave +
                                           lo.val + (v * 64 + (t & 63)) * 8);
    };
    uint32_t *s_flag = reinterpret_cast<uint32_t *>(lds + lo.flag);
    auto sync = [&]() {
        if (SEG && W > 64) __syncthreads();
        else wave_sync();
    };

    const long long LB = (long long)C * NB;
    const unsigned lane = (unsigned)c * NB + b;   // of a [C][NB] plane
    auto records = [&]() -> double2 * { return record_block(args().scratch, N, NB, c0, lane0); };
    // byte offsets of this lane's layers from those of the lowest segment (32 bits: stream_geometry)
    const int a_last = SEG ? N - LPT : 0;
    // records: lanes of the workgroup's block, this one's place in it
    const int RB = wide ? nlane : min(K, C - c0) * NB;
    const unsigned rlane = wide ? b - lane0 : (c - c0) * NB + b;
    const unsigned rlay = SEG ? (unsigned)(a_last - me.a) * (unsigned)RB : 0u;
    const unsigned lay = SEG ? (unsigned)(a_last - me.a) * (unsigned)LB : 0u;
    const unsigned o_in = (lane + lay) * (unsigned)sizeof(InT), o_rec = rlane * 16u + rlay * 32u;
    auto in_at = [&](const double *base, int q) -> InT {   // step q's (past the last: one of the lowest layers, unused)
        return at(reinterpret_cast<const InT *>(base) + (long long)max(N - 1 - a_last - q, 0) * LB, o_in);
    };
    // The inputs of a layer are loaded two layers ahead, into the registers that
    // the layer before has just used (a copy between registers would wait for
    // the load, and with it for the record stores before it), from pointers that move
    // with the layers (addresses worked out anew take twenty scalar instructions of a
    // layer's 600, and argument loads that the wavefront waits for).
    InT dt0, w0, g0_, dt1, w1, g1;
    auto load = [&](int q, InT &dt, InT &w, InT &g) {
        dt = in_at(args().dtau, q);
        w = in_at(args().w0, q);
        g = in_at(args().g0, q);
    };
    const int odd = LPT & 1;
    const bool uneven = SEG && N % S != 0;   // some segments repeat a layer
    load(odd, dt0, w0, g0_);
    load(1 - odd, dt1, w1, g1);   // (odd: the first step, then the third in its place)
    int left = N - 1 - a_last - 2;   // layers below that of the next load (step 2)
    const InT *p_dt = reinterpret_cast<const InT *>(args().dtau) + (long long)max(left, 0) * LB;
    const InT *p_w = reinterpret_cast<const InT *>(args().w0) + (long long)max(left, 0) * LB;
    const InT *p_g = reinterpret_cast<const InT *>(args().g0) + (long long)max(left, 0) * LB;
    auto load_next = [&](InT &dt, InT &w, InT &g) {
        dt = at(p_dt, o_in);
        w = at(p_w, o_in);
        g = at(p_g, o_in);
        const long long step = left > 0 ? LB : 0;   // (at the lowest layer: again)
        --left;
        p_dt -= step;
        p_w -= step;
        p_g -= step;
    };
    // Planck edge integrals of a chunk of levels: rows (group of the wavefront, row of
    // the chunk); a lane keeps one row and steps through its edges, so a wavefront's
    // lanes sit in neighbouring edges and the row's temperature stays in a register.
    // The first chunk's rows are T_int, the level the group starts at, the lower
    // level of the odd first step if there is one (and one row unused, so that the
    // chunks hold pairs of layers), then lower levels like the other chunks' rows.
    const int lrows = 9 - lNBp;   // log2 of gw kChunk
    const int row = ln & ((1 << lrows) - 1), e0 = ln >> lrows, epr = 64 >> lrows;
    const int rq = row & (kChunk - 1);
    const Group rg = group(g0 + row / kChunk);
    const int rc = min(c0 + rg.kk, C - 1);
    const int head = 2 + 2 * odd;   // rows of the first chunk before its pairs of layers
    auto T_at = [&](int p) -> double { return level_T(args(), sub, max(N - p, 0), rc); };   // level p from the TOA
    double Tc_ = rq == 0 ? args().Tint[rc] : T_at(rg.a + (rq < head ? min(rq - 1, odd) : rq - head + 1 + odd));
    double Tn_ = T_at(rg.a + rq + kChunk - head + 1 + odd);

    for (int k = tid; k < K; k += W) s_flag[k] = 0u;
    for (int e = tid; e < ne; e += W) s_c2[bin0 + e] = args().c2_over_lam[bin0 + e];
    if constexpr (!MIXED) {   // (all loads before the first store; past the end: the last value again)
        constexpr int n = (kPlanckTable + 63) / 64;
        double v[n];
#pragma unroll
        for (int i = 0; i < n; ++i) v[i] = planck_values[min(tid + i * W, kPlanckTable - 1)];
#pragma unroll
        for (int i = 0; i < n; ++i) s_tab[min(tid + i * W, kPlanckTable - 1)] = v[i];
    }
    uint32_t fl = 0u;
    const double mu = args().mu[c], Ti = args().Tint[c];
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
    ElimState st;
    StateMap map;   // (SEG; m[0..2]: the state, where direct)
    auto top_state = [&]() { return elim_top(args().Ftoa ? args().Ftoa[lane] : 0.0); };
    if (!SEG || direct) st = top_state();
    if (direct) map.set_state(st);
    double Fb_up = muF, tau = 0.0;   // beam and optical depth at the current level
    if constexpr (SEG) {
        // the optical depth above each segment: sums over [a, the next one's a)
        if (wday && me.s < S - 1) {
            const int n = group(g0 + gl + K).a - me.a;
            double ts = 0.0;
            for (int q = 0; q < LPT + 1; q += 8) {
                InT v[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = in_at(args().dtau, q + k);
#pragma unroll
                for (int k = 0; k < 8; ++k) ts += q + k < n ? double(v[k]) : 0.0;
            }
            shared_at(0, 0) = ts;
        }
        sync();
        if (day && me.s > 0) {
            for (int s = me.s; s > 0; --s) tau += shared_at(0, -s);
            Fb_up = beam_at<MIXED>(muF, tau, inv_mu);
        }
        sync();
    } else {
        sync();
    }

    // Mixed: temperatures at which every bin of the wavefront takes the narrow bins'
    // quadrature; a chunk of such levels needs no edge integrals (10242 x 80 x 300: 380
    // vector instructions per layer in place of 434; 369 now, with the later steps).
    double narrow_lo = 0.0, narrow_hi = 0.0;
    bool narrow = false;
    if constexpr (MIXED) {
        const PlanckNarrow r = planck_narrow_range(args().c2_over_lam[bin + 1], args().c2_over_lam[bin]);
        narrow_lo = r.lo;
        narrow_hi = r.hi;
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) {
            narrow_lo = fmax(narrow_lo, __shfl_xor(narrow_lo, m));
            narrow_hi = fmin(narrow_hi, __shfl_xor(narrow_hi, m));
        }
        narrow_lo = first_lane(narrow_lo);
        narrow_hi = first_lane(narrow_hi);
    }
    auto edges = [&](double T, int from, int n, bool check) {
        if constexpr (MIXED) narrow = !wave_any(!(T >= narrow_lo && T <= narrow_hi));
        if (rq >= from && rq < n) {
            if (check && (!(T > 0.0) || !isfinite(T))) atomicOr(&s_flag[rg.kk], (uint32_t)F_INVALID);
            const double iT = rcp(T);
            if (e0 == 0) s_level[row] = LevelValue<MIXED>::of(T);
            if (!MIXED || !narrow) {
            // two at a time (past the last edge: that one again), so that their chains overlap
            R *re = s_edge + row * lo.estride;
            for (int i = 0; i < ne; i += 2 * epr) {
                const int e1 = min(i + e0, ne - 1), e2 = min(i + epr + e0, ne - 1);
                const R v1 = edge_integral<R>(s_c2[bin0 + e1] * iT, s_tab), v2 = edge_integral<R>(s_c2[bin0 + e2] * iT, s_tab);
                re[e1] = v1;
                re[e2] = v2;
            }
            }
        }
        wave_sync();
    };
    auto bin_B = [&](int q) -> R {
        const int rw = gl * kChunk + q;
        return bin_radiance<MIXED, R>(s_edge + rw * lo.estride + rb, s_level[rw], c2fb, c2fa, s_c2 + bin, narrow);
    };
    // Column sums of n rows of lane values v (LDS, kSumStride apart) into the sums of
    // levels lev(group, row): lane (q, p) = (ln % 8, ln / 8) adds the 8 lanes p of row
    // q, then the parts of a group are added.  Fixed order.
    const Group sg = group(g0 + (ln >> lNBp));   // (p >> (lNBp - 3))
    const bool sumout = (ln >> 3 & ((NBp >> 3) - 1)) == 0;
    auto sum_rows = [&](const double *v, int which, auto lev) {
        wave_sync();
        const int q = ln & 7, p = ln >> 3;
        const double *r = v + q * kSumStride + p * 8;
        double s = r[0];
#pragma unroll
        for (int k = 1; k < 8; ++k) s += r[k];
        if (lNBp > 3) s += __shfl_xor(s, 8);
        if (lNBp > 4) s += __shfl_xor(s, 16);
        if (lNBp > 5) s += __shfl_xor(s, 32);
        const int l = lev(sg, q);
        if (l >= 0 && sumout) s_sum[(3 * l + which) * K + sg.kk] = s;
        wave_sync();
    };

    // records: the layer that a shorter segment repeats is another's, so an uneven split's
    // first step stores in the place of its next one, whose records follow
    double2 *p_rec = records() + (long long)(N - 1 - a_last - (uneven ? 1 : 0)) * 2 * RB;
    int rec_step = uneven ? 0 : 2 * RB;
    unsigned o_st = o_rec + (uneven && me.a == me.e ? (unsigned)RB * 32u : 0u);
    Opts o;
    auto options = [&]() {   // (read anew in each chunk)
        opaque_args(ap);
        o = uniform_options(ap);
    };
    // step q, its lower level's Planck edges in row r, its beam value into row v.
    // (The padding stores its lane's record again: same values, and the loads'
    // waits then pass the stores, whose number is the same for every wavefront.)
    auto layer = [&](int q, int r, int v, InT &dt_, InT &w_, InT &g_, R &Bup) {
        const R B = bin_B(r);
        double Fb_lo = 0.0;
        const double dt = double(dt_);
        if (day) {
            tau += dt;   // summed from the TOA, as the optical depth is defined
            Fb_lo = beam_at<MIXED>(muF, tau, inv_mu);
        }
        const Layer<R> Ly = layer_item<MIXED, R, MIXED>(dt, double(w_), double(g_), day, mu, inv_mu, Fb_up, Fb_lo,
                                                        B, Bup, o, inv_eps2, fl);
        load_next(dt_, w_, g_);
        double2 x, y;
        if constexpr (!SEG) {
            const BackRec rec = elim_step(st, double(Ly.t), double(Ly.r), double(Ly.omr), double(Ly.A),
                                          double(Ly.Sup), double(Ly.Sdn));
            x = make_double2(rec.G, rec.H);
            y = make_double2(rec.c, rec.d);
        } else if (direct) {
            st = map.state();
            const BackRec rec = elim_step(st, double(Ly.t), double(Ly.r), double(Ly.omr), double(Ly.A),
                                          double(Ly.Sup), double(Ly.Sdn));
            map.set_state(st);
            x = make_double2(rec.G, rec.H);
            y = make_double2(rec.c, rec.d);
        } else if constexpr (MIXED) {
            map.step(double(Ly.t), double(Ly.r), double(Ly.omr), double(Ly.A), double(Ly.Sup), double(Ly.Sdn));
            x = make_double2(__hiloint2double(__float_as_int(Ly.r), __float_as_int(Ly.t)),
                             __hiloint2double(__float_as_int(Ly.A), __float_as_int(Ly.omr)));
            y = make_double2(__hiloint2double(__float_as_int(Ly.Sdn), __float_as_int(Ly.Sup)), 0.0);
        } else {
            map.step(Ly.t, Ly.r, Ly.omr, Ly.A, Ly.Sup, Ly.Sdn);
            const StoredLayer c = store_layer(Ly.t, Ly.r, Ly.A);
            x = make_double2(c.p, c.q);
            y = make_double2(Ly.Sup, Ly.Sdn);
        }
        at(p_rec, o_st) = x;
        at(p_rec + RB, o_st) = y;
        p_rec -= rec_step;
        rec_step = 2 * RB;
        o_st = o_rec;
        if (wday) s_val[v * kSumStride + ln] = wgt * Fb_lo;
        Fb_up = Fb_lo;
        Bup = B;
        if constexpr (SEG)
            if (uneven && q == 0 && me.a != me.e) map = StateMap();
    };
    options();
    edges(Tc_, 0, min(kChunk, LPT + head - odd), rq > 0);
    const double Fboa = double(kPI) * double(bin_B(0));
    R Bup = bin_B(1);
    if (wday) s_val[ln] = wgt * muF;   // beam at level N
    if (odd) layer(0, 2, 1, dt1, w1, g1, Bup);
    if (wday)
        sum_rows(s_val, 2, [&](const Group &g, int q) {
            return q == 0 ? (g.s == 0 ? N : -1) : (q == 1 && odd && g.a == g.e ? N - 1 - g.a : -1);
        });
    // chunks of pairs of layers: steps q0 .. q0 + n - 1 in rows r0 ..
    for (int q0 = odd, r0 = head; q0 < LPT;) {
        const int n = min(kChunk - r0, LPT - q0);
#pragma unroll 1
        for (int k = 0; k < n; k += 2) {
            layer(q0 + k, r0 + k, k, dt0, w0, g0_, Bup);
            layer(q0 + k + 1, r0 + k + 1, k + 1, dt1, w1, g1, Bup);
        }
        if (wday)
            sum_rows(s_val, 2, [&](const Group &g, int q) {
                return q < n && q0 + q >= g.e - g.a ? N - 1 - g.a - q0 - q : -1;
            });
        q0 += n;
        r0 = 0;
        if (q0 < LPT) {
            if (SEG && !direct) map.rescale();
            options();
            Tc_ = Tn_;
            edges(Tc_, 0, min(kChunk, LPT - q0), true);
            Tn_ = T_at(rg.a + q0 + kChunk + rq + 1);   // (the chunk after this one's)
        }
    }
    if (fl) atomicOr(&s_flag[me.kk], fl);

    double Fu = 0.0, Fd = 0.0;
    if constexpr (!SEG) {
        elim_boa(st, Fboa, Fb_up, Fu, Fd);
    } else {
        // the state at the segment's top, from the maps of the ones above
        if (direct) map = StateMap::constant(map.state());
        sync();   // (the rows' place is free)
#pragma unroll
        for (int v = 0; v < 11; ++v) shared_at(v, 0) = map.m[v];
        sync();
        st = top_state();
        for (int d = -me.s; d < 0; ++d) {
            StateMap up;
#pragma unroll
            for (int v = 0; v < 11; ++v) up.m[v] = shared_at(v, d);
            up.apply(st);
        }
        // the elimination of all segments: coefficients become records in place, and
        // the segment's map of F_up is composed
        constexpr int RC = 4;
        double2 x[RC], y[RC];
        auto ld = [&](int q, int k) {
            const double2 *r = records() + (long long)(N - 1 - a_last - min(q, LPT - 1)) * 2 * RB;
            x[k] = at(r, o_rec);
            if constexpr (MIXED) y[k].x = at(r + RB, o_rec).x;
            else y[k] = at(r + RB, o_rec);
        };
        double gam = 1.0, eta = 0.0;
        auto step = [&](int q, int k) {
            BackRec rec;
            if constexpr (MIXED) {
                auto lo_f = [](double v) { return double(__int_as_float(__double2loint(v))); };
                auto hi_f = [](double v) { return double(__int_as_float(__double2hiint(v))); };
                rec = elim_step(st, lo_f(x[k].x), hi_f(x[k].x), lo_f(x[k].y), hi_f(x[k].y), lo_f(y[k].x), hi_f(y[k].x));
            } else {
                double t, r, omr, A;
                load_layer({x[k].x, x[k].y}, t, r, omr, A);
                rec = elim_step(st, t, r, omr, A, y[k].x, y[k].y);
            }
            double2 *r = records() + (long long)(N - 1 - a_last - q) * 2 * RB;
            at(r, o_rec) = make_double2(rec.G, rec.H);
            at(r + RB, o_rec) = make_double2(rec.c, rec.d);
            eta = fma(gam, rec.H, eta);
            gam *= rec.G;
        };
        // (not for the padding's columns: another wavefront may have been through the
        // last column's coefficients already)
        if (!direct && c0 + me.kk < C) {
            int q = 0;
            if (uneven) {   // a shorter segment's first step is not its own
                ld(0, 0);
                if (me.a == me.e) step(0, 0);
                q = 1;
            }
#pragma unroll
            for (int k = 0; k < RC; ++k) ld(q + k, k);
            for (; q + RC <= LPT; q += RC) {
#pragma unroll
                for (int k = 0; k < RC; ++k) {
                    step(q + k, k);
                    ld(q + k + RC, k);
                }
            }
#pragma unroll
            for (int k = 0; k < RC; ++k)
                if (q + k < LPT) step(q + k, k);
        }
        shared_at(11, 0) = gam;
        shared_at(12, 0) = eta;
        if (me.s == S - 1) {
            elim_boa(st, Fboa, Fb_up, Fu, Fd);
            shared_at(13, 0) = Fu;
        }
        sync();
        // F_up at the bottom of the segment, from the one at the BOA upward
        if (me.s < S - 1) {
            const int down = S - 1 - me.s;
            Fu = shared_at(13, down);
            for (int d = down; d > 0; --d) Fu = fma(shared_at(11, d), Fu, shared_at(12, d));
        }
        sync();
    }
    // back-substitution in chunks of levels, from the group's first one on (level 0,
    // or the one above its lowest layer); a lane's records are loaded RD levels
    // ahead of their use.  Every chunk runs whole (past the group's last level on its
    // last record again, into rows that are not summed), so no load is under a branch.
    constexpr int RD = MIXED ? 4 : 8;
    opaque_args(ap);
    const bool low = me.s == S - 1;
    const int ilo = N - me.e1, first = low ? 0 : ilo + 1;   // its lowest layer, its first level
    const int last = N - me.e;                              // its last level
    double2 r0[RD], r1[RD];
    // next record: that of the layer below the level (past the last: the last again)
    int jn = first - 1;
    const double2 *p_back = records();
    unsigned o_back = rlane * 16u;
    if constexpr (SEG) o_back += (unsigned)max(jn, 0) * (unsigned)RB * 32u;
    auto ld = [&](int k) {
        r0[k] = at(p_back, o_back);
        r1[k] = at(p_back + RB, o_back);
        if constexpr (SEG) o_back += jn >= 0 && jn < last - 1 ? (unsigned)RB * 32u : 0u;
        else p_back += jn >= 0 && jn < N - 1 ? 2 * RB : 0;
        ++jn;
    };
#pragma unroll
    for (int k = 0; k < RD; ++k) ld(k);
    if (low) {   // level 0: the fluxes stay as they are
        r0[0] = make_double2(1.0, 0.0);
        r1[0] = make_double2(0.0, Fd);
    }
    const bool bins = args().F_up_bin || args().F_dn_bin;
    double Fu_toa = 0.0;
    for (int k0 = 0; k0 <= LPT; k0 += kChunk) {
        opaque_args(ap);
#pragma unroll
        for (int k = 0; k < kChunk; ++k) {
            const int i = first + k0 + k;
            back_step(r0[k % RD].x, r0[k % RD].y, r1[k % RD].x, r1[k % RD].y, Fu, Fd);
            ld(k % RD);
            s_val[k * kSumStride + ln] = wgt * Fu;
            s_val2[k * kSumStride + ln] = wgt * Fd;
            if (i == N) Fu_toa = Fu;
            if (bins && act && i <= last) {
                if (args().F_up_bin) args().F_up_bin[i * LB + lane] = Fu;
                if (args().F_dn_bin) args().F_dn_bin[i * LB + lane] = Fd;
            }
        }
        auto level = [&](const Group &g, int q) {
            const int l = (g.s == S - 1 ? 0 : N - g.e1 + 1) + k0 + q;
            return l <= N - g.e ? l : -1;
        };
        sum_rows(s_val, 0, level);
        sum_rows(s_val2, 1, level);
    }
    opaque_args(ap);
    if (act && me.s == 0 && args().F_up_toa_bin) {
        if (NG == 1) args().F_up_toa_bin[lane] = Fu_toa;
        else if (!wide) s_top[me.kk * NB + b] = Fu_toa;
    }
    sync();
    if (!wide) {
        if (NG > 1 && args().F_up_toa_bin) {   // the spectrum: weighted sums over each bin's points
            for (int t = tid; t < K * sh.NBR; t += W) {
                const int k = small_div(t, sh.NBR), r = t - k * sh.NBR, cc = c0 + k;
                if (cc >= C) continue;
                const double *f = s_top + k * NB + r * NG;
                double s = 0.0;
                for (int g = 0; g < NG; ++g) s += args().wg[g] * f[g];
                args().F_up_toa_bin[(long long)cc * sh.NBR + r] = s;
            }
        }
        write_columns(ap, c0, K, s_flag, [&](int l, int v, int k) { return s_sum[(3 * l + v) * K + k]; });
    } else {
        // this slice's sums and flags in the place of its used records
        double *rec = reinterpret_cast<double *>(records());
        for (int t = tid; t < 3 * (N + 1); t += W) rec[t] = t % 3 == 2 && !wday ? 0.0 : s_sum[t];
        if (tid == 0) rec[3 * (N + 1)] = (double)s_flag[0];
        if (act && me.s == 0 && NG > 1) rec[(2 * N - 1) * RB * 2 + (b - lane0)] = Fu_toa;
    }
}

// Columns of more than 64 lanes, after k_solve_stream: a workgroup adds its column's
// slices, in order, each sum once and eight slices' loads at a time (added at each use, one
// load after the other, 10242 x 80 x 300 took 169 us here and 2562 x 40 x 600 lanes 44).
__device__ __forceinline__ void solve_columns(ArgsK ap, const int c)
{
    extern __shared__ double s_sums[];   // [3 (N + 1)]
    __shared__ uint32_t s_flag;
    auto args = [&]() -> const SolveArgs & { return *(const SolveArgs *)ap; };
    const int NG = args().NG, N = args().N, tid = threadIdx.x;
    const StreamShape sh = StreamShape::unpack(args().CH, args().L);
    const int NB = args().NB;
    auto slice = [&](int w) -> const double * {
        return reinterpret_cast<const double *>(record_block(args().scratch, N, NB, c, w * sh.NBs));
    };
    const int n = 3 * (N + 1);
    if (tid == 0) s_flag = 0u;
    __syncthreads();
    if (tid < sh.NBw) atomicOr(&s_flag, (uint32_t)slice(tid)[n]);
    for (int t = tid; t < n; t += blockDim.x) {
        double s = 0.0;
        for (int w = 0; w < sh.NBw; w += 8) {
            double v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = slice(min(w + k, sh.NBw - 1))[t];
#pragma unroll
            for (int k = 0; k < 8; ++k) s += w + k < sh.NBw ? v[k] : 0.0;
        }
        s_sums[t] = s;
    }
    __syncthreads();
    if (NG > 1 && args().F_up_toa_bin) {   // the spectrum: weighted sums over each bin's points
        for (int r = tid; r < sh.NBR; r += blockDim.x) {
            double s = 0.0;
            for (int g = 0; g < NG; ++g) {
                const int l = r * NG + g, w = small_div(l, sh.NBs), lanes = min(sh.NBs, NB - w * sh.NBs);
                s += args().wg[g] * slice(w)[(2 * N - 1) * lanes * 2 + l - w * sh.NBs];
            }
            args().F_up_toa_bin[(long long)c * sh.NBR + r] = s;
        }
    }
    write_columns(ap, c, 1, &s_flag, [&](int l, int v, int) { return s_sums[3 * l + v]; });
}

constexpr int kColumnThreads = 128;   // of k_stream_columns
constexpr int kColumnStaticLds = 1024;   // more than its static LDS
size_t columns_lds(int N) { return 3 * (size_t)(N + 1) * sizeof(double); }

// Workgroup g of a grid of 8 n takes tile (g % 8) n + g / 8, so each XCD's L2 sees a run of
// neighbouring columns (slices of a column share cache lines).
__device__ __forceinline__ int xcd_tile(int g, int n) { return (g % kXcds) * n + g / kXcds; }
int xcd_grid(int tiles) { return (tiles + kXcds - 1) / kXcds * kXcds; }

// Whether a request has that tile: a set of K columns, or a slice of a wide column.
__device__ __forceinline__ bool has_tile(const SolveArgs &a, int tile)
{
    const int nbw = StreamShape::unpack(0, a.L).NBw;
    return nbw > 1 ? tile < a.C * nbw : (long long)tile * a.K < a.C;
}

template <bool MIXED, bool IN32, bool SEG>
__global__ void __launch_bounds__(SEG ? kStreamThreads : 64, MIXED && !SEG ? 4 : 3) k_solve_stream(const SolveArgs a)
{
    const int tile = xcd_tile(blockIdx.x, gridDim.x / kXcds);
    if (has_tile(a, tile)) solve_tile_stream<MIXED, IN32, SEG>(kernel_args(a), tile);
}

__global__ void __launch_bounds__(kColumnThreads) k_stream_columns(const SolveArgs a)
{
    solve_columns(kernel_args(a), blockIdx.x);
}

template <bool MIXED, bool IN32, bool SEG>
__global__ void __launch_bounds__(SEG ? kStreamThreads : 64, MIXED && !SEG ? 4 : 3)
k_solve_stream_batch(const SolveArgs *__restrict__ reqs, const int *__restrict__ first, int n)
{
    const int r = batch_request(first, n, blockIdx.x);
    const int end = r + 1 < n ? first[r + 1] : (int)gridDim.x;
    const int tile = xcd_tile(blockIdx.x - first[r], (end - first[r]) / kXcds);
    if (has_tile(reqs[r], tile)) solve_tile_stream<MIXED, IN32, SEG>((ArgsK)(reqs + r), tile);
}

// first: of k_solve_stream_batch, whose launch has NBw workgroups or more per column (one
// handle's requests all have the same lanes per column): request r's columns start at
// workgroup ceil(first[r] / NBw), and the next one's start after all of them.
__global__ void __launch_bounds__(kColumnThreads)
k_stream_columns_batch(const SolveArgs *__restrict__ reqs, const int *__restrict__ first, int n, int NBw)
{
    const int r = batch_request(first, n, blockIdx.x * NBw), c = blockIdx.x - (first[r] + NBw - 1) / NBw;
    if (c < reqs[r].C) solve_columns((ArgsK)(reqs + r), c);
}

// f(kernel) for the variant of a launch
template <class F>
void with_kernel(int precision, int in_f32, bool seg, F f)
{
    using std::integral_constant;
    auto pick = [&](auto mixed, auto in32) {
        if (seg) f(mixed, in32, integral_constant<bool, true>{});
        else f(mixed, in32, integral_constant<bool, false>{});
    };
    if (precision != 1) pick(integral_constant<bool, false>{}, integral_constant<bool, false>{});
    else if (in_f32) pick(integral_constant<bool, true>{}, integral_constant<bool, true>{});
    else pick(integral_constant<bool, true>{}, integral_constant<bool, false>{});
}

}  // namespace

// S segments per column; direct: the first wavefront holds first segments only.
static Geometry stream_shape(int C, int N, int NB, int NG, int S, bool direct, bool mixed, const DeviceLimits &dev)
{
    Geometry g{};
    const LaneLayout ll = lane_layout(NB);
    // columns per workgroup: whole wavefronts of segments
    int K = 1;
    while (K * S % ll.gw) ++K;
    if (S > 1 && direct) K = ll.gw;
    const int waves = K * S / ll.gw;
    if (64 * waves > kStreamThreads || S > N || (S > 1 && N % S && (N + S - 1) / S < 2)) return g;
    // 32-bit byte offsets of a lane's record in a plane of lanes, of all records where segments differ
    if ((long long)C * NB >= (1ll << 28) || (S > 1 && (long long)C * NB * N >= (1ll << 27))) return g;
    const StreamShape sh = stream_sizes(N, NB, NG, S);
    g.lds = stream_lds(sh, N, NB, NG, K, ll.gw, waves, mixed).total;
    if (g.lds > dev.lds || (NB > 64 && columns_lds(N) > dev.lds - kColumnStaticLds)) return g;
    g.kernel = KERNEL_STREAM;
    g.K = K;
    g.PC = S;
    g.CH = sh.LPT;
    g.threads = 64 * waves;
    g.blocks = xcd_grid(NB > 64 ? C * ll.NBw : (C + K - 1) / K);
    g.lanes = sh.pack();   // (SolveArgs::L)
    g.scratch = (size_t)N * 4 * (size_t)C * NB * sizeof(double);
    return g;
}

// Estimated time of a launch, us.  A compute unit holds wg workgroups at once (12 wavefronts,
// three per SIMD at 168 registers; 16 unsegmented in mixed precision; fewer where the level sums
// fill its LDS), in rounds; c wavefronts per SIMD take layer + layer_c c for each layer of a
// segment and chunk + chunk_c c for each chunk of levels.  A full round of segments costs
// more than the last one, whose records the caches hold.  Coefficients: least squares of
// measured times, 1 to 1000 layers, 1 to 300 lanes, up to 30000 columns (8 percent rms in FP64, 9 in
// mixed precision, 10 in segments).
static double stream_time(const Geometry &g, int C, int N, int NB, bool mixed, const DeviceLimits &dev)
{
    struct Fit {
        double base, seg, half, wide, layer, layer_c, chunk, chunk_c, round;   // half: 33 to 64 lanes per column
    };
    static constexpr Fit fits[2][2] = {{{6.5, 0.0, 0.8, 4.0, 1.07, 0.45, 0.0, 2.4, 0.9}, {8.7, 0.25, 0.8, 3.5, 1.35, 0.46, 0.0, 3.4, 1.03}},
                                       {{7.0, 0.2, 3.0, 5.7, 0.98, 0.38, 0.17, 1.78, 1.0}, {9.3, 0.2, 3.0, 5.1, 1.25, 0.35, 0.05, 2.13, 1.17}}};
    const Fit &f = fits[mixed][g.PC > 1];
    const int n_cu = dev.n_cu > 0 ? dev.n_cu : 256, w = g.threads / 64;
    const int tiles = NB > 64 ? C * lane_layout(NB).NBw : (C + g.K - 1) / g.K, per_cu = (tiles + n_cu - 1) / n_cu;
    const int wg = std::max(1, std::min((mixed && g.PC == 1 ? 16 : 12) / w, (int)(dev.lds / g.lds)));
    const int full = (per_cu - 1) / wg, odd = g.CH & 1;
    const int chunks = 1 + std::max(0, g.CH - odd - (kChunk - 2 - 2 * odd) + kChunk - 1) / kChunk;
    auto round = [&](double c) {
        c = std::max(1.0, c);
        return g.CH * (f.layer + f.layer_c * c) + chunks * (f.chunk + f.chunk_c * c);
    };
    // (segments of a few lanes read and write pieces of cache lines)
    const double rounds = full * f.round * (g.PC > 1 && NB <= 16 ? 2.0 : 1.0);
    const double us = f.base + f.seg * g.PC + (NB > 64 ? f.wide : NB > 32 ? f.half : 0.0) + rounds * round(wg * w / 4.0) +
                      round(((per_cu - full * wg) * w + 3) / 4);
    // inputs and records, and the coefficients of all segments but the first, from memory (where
    // they are many times the caches; 3.8 TB/s)
    const double bytes = (double)C * N * NB * (88.0 + 64.0 * (g.PC - 1) / g.PC);
    return bytes > 3e9 ? std::max(us, bytes / 3.8e6) : us;
}

// Segments per column: the least estimated time, where the most segments whose wavefronts
// the registers hold count a tenth less (us, C x N x NB by S, FP64; the last column: mixed):
//   162 x 40 x 30     1: 83    2: 55    4: 36    8: 25   16: 27     1: 73    8: 22   16: 24
//   512 x 40 x 30     1: 82    2: 58    4: 39    8: 33   16: 54     1: 73    8: 28   16: 46
//   1500 x 40 x 30    1: 85    2: 74    3: 70    4: 60    8: 69     1: 77    4: 48    8: 57
//   1800 x 40 x 30    1: 85    2: 75    3: 71    4: 84              1: 77    3: 54    4: 75
//   2562 x 40 x 30    1: 111   2: 95    3: 106                      1: 88    2: 73    3: 94
//   3200 x 40 x 30    1: 112   2: 141                               1: 89    2: 124
//   100 x 60 x 300    1: 125   2: 106   3: 80    4: 67    5: 101    1: 120   4: 57    5: 90
//   300 x 100 x 16    1: 198   4: 73    8: 53   16: 41   20: 59     1: 168  16: 35   20: 51
//   162 x 20 x 100    4: 32    8: 47 (workgroups of eight wavefronts, one per CU: two rounds)
// (5 and 20 give workgroups of five wavefronts, which pack badly on four SIMDs.)  Short
// segments give less than their hand-over costs: 48 layers take 26 in 8 segments and 28
// in 16, 60 layers 34 and 30; 20 layers 23 in 4 and 21 in 8; 12 layers 19.7 in 4, 23 in 2; 5
// layers 17.6 in 2 and 16.8 in 1.
// Up to 4 segments, a workgroup takes as many columns as a wavefront holds groups,
// so that its first wavefront eliminates as it goes (2562 x 40 x 30: 100 to 95, mixed 85 to
// 73; 3000 x 60 x 16: 112 to 85); with 8 the larger workgroup costs more.
Geometry stream_geometry(int C, int N, int NB, int NG, bool mixed, const DeviceLimits &dev)
{
    static constexpr struct {
        int S, layers;
    } splits[] = {{16, 48}, {8, 20}, {4, 7}, {3, 9}, {2, 8}, {1, 1}};
    const LaneLayout ll = lane_layout(NB);
    const int n_cu = dev.n_cu > 0 ? dev.n_cu : 256;
    const long long waves = NB > 64 ? (long long)C * ll.NBw : (C + ll.gw - 1) / ll.gw;
    Geometry best{};
    bool fits = false;   // a split whose wavefronts the registers hold was met
    double least = 0.0;
    for (const auto &v : splits) {
        if (N < v.layers) continue;
        Geometry g = stream_shape(C, N, NB, NG, v.S, v.S > 1 && v.S <= 4, mixed, dev);
        if (g.threads == 0) continue;
        g.us = stream_time(g, C, N, NB, mixed, dev);
        const bool first = !fits && waves * v.S <= 12ll * n_cu;
        fits = fits || first;
        const double us = first ? g.us / 1.1 : g.us;
        if (best.threads == 0 || us < least) {
            best = g;
            least = us;
        }
    }
    return best;
}

hipError_t launch_stream(const SolveArgs &a, const Geometry &g, int precision, hipStream_t s)
{
    SolveArgs b = a;
    b.K = g.K;
    b.PC = g.PC;
    b.CH = g.CH;
    b.L = g.lanes;
    with_kernel(precision, a.in_f32, g.PC > 1, [&](auto mixed, auto in32, auto seg) {
        hipLaunchKernelGGL((k_solve_stream<decltype(mixed)::value, decltype(in32)::value, decltype(seg)::value>),
                           dim3(g.blocks), dim3(g.threads), g.lds, s, b);
    });
    if (a.NB > 64) hipLaunchKernelGGL(k_stream_columns, dim3(a.C), dim3(kColumnThreads), columns_lds(a.N), s, b);
    return hipGetLastError();
}

hipError_t launch_stream_batch(const SolveArgs *d_reqs, const int *d_first, int n, int total_blocks,
                               int layers, const Geometry &g, int NB, int precision, int in_f32, hipStream_t s)
{
    with_kernel(precision, in_f32, g.PC > 1, [&](auto mixed, auto in32, auto seg) {
        hipLaunchKernelGGL((k_solve_stream_batch<decltype(mixed)::value, decltype(in32)::value, decltype(seg)::value>),
                           dim3(total_blocks), dim3(g.threads), g.lds, s, d_reqs, d_first, n);
    });
    if (NB > 64) {
        const int NBw = lane_layout(NB).NBw;
        hipLaunchKernelGGL(k_stream_columns_batch, dim3((total_blocks + NBw - 1) / NBw), dim3(kColumnThreads),
                           columns_lds(layers), s, d_reqs, d_first, n, NBw);
    }
    return hipGetLastError();
}

hipError_t prepare_stream_kernels(const DeviceLimits &dev)
{
    hipError_t e = hipSuccess;
    for (int v = 0; v < 6; ++v)
        with_kernel(v > 1, v > 3, v & 1, [&](auto mixed, auto in32, auto seg) {
            constexpr bool M = decltype(mixed)::value, I = decltype(in32)::value, G = decltype(seg)::value;
            const void *fns[] = {reinterpret_cast<const void *>(&k_solve_stream<M, I, G>),
                                 reinterpret_cast<const void *>(&k_solve_stream_batch<M, I, G>)};
            for (const void *f : fns)
                if (e == hipSuccess)
                    e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dev.lds);
        });
    for (const void *f : {reinterpret_cast<const void *>(&k_stream_columns), reinterpret_cast<const void *>(&k_stream_columns_batch)})
        if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dev.lds - kColumnStaticLds);
    return e != hipSuccess ? e : upload_planck_table();
}

}  // namespace rtk
