#pragma once
// Square-lattice step as a column march of independent wavefronts (Sec. IV.B
// and V.A of Komeili, Mirzaei, Shabouei, arXiv 1602.02675; tau = 1, so a step
// is the migration of the equilibrium, eq. 10 / eq. 30).
//
// A packet's displacement is floor(v) + k + c' (corner k in {0,1}^2, lane c'
// = +-c along x or y).  The corner weights do not depend on the lane, so the
// migration factors into two stages, both linear:
//   A  interpolation: per speed c, every source puts the mass of one lane of
//      that speed onto its four corner nodes.  This gives the corner sums
//      U_c(x, y) = sum of m (1, v_x, v_y, K) over the sources and corners
//      that land on (x, y), K = |v|^2/2 + phi;
//   B  lanes: the new moments of a node are those of U_c at (x -+ c, y) for
//      the lanes +-c along x and (x, y -+ c) along y: mass M, momentum
//      V +- c M, energy E_c +- c V with E_c = sum m (K + c^2/2) (eq. 14, 21).
//      Speed 0 (c'_1 = 0: all four lanes; and the rest group) stays at U_0.
// Against rebuilding each of the 32 packets at its destination, stage A forms
// a packet's payload once for all four lanes of a speed, and stage B is a
// handful of additions.
//
// One wavefront owns a tile of kMCols destination columns (64 lanes less the
// halo of H = 5 on each side) by a strip of rows and marches down the strip,
// one source column per lane.  Columns exchange by wavefront shifts (DPP
// moves between neighbouring lanes), rows through FIFOs in registers or, for the
// largest instances of the general pass, in LDS of the wavefront's own
// (MarchStash): no barriers, and wavefronts never wait for each other.
//
// Sources of one row that share floor(v) and c'_1 form a class; a row's
// classes are taken one after another, the lanes of other classes with zero
// mass, so a node whose sources are all of one class gets the same bits
// whatever else is in its wavefront, and, since every pass and every cut of
// the rows adds a node's terms in the same order (source rows ascending),
// whichever pass or tile computes it.  Without that, wavefronts next to a
// transition would round an at-rest region differently from their
// neighbours, and the 1-ulp differences grow into momentum noise.
//
// The kernels and helpers below sit in an anonymous namespace: each
// translation unit that includes this header instantiates its own kernels.
#include "lb_wave.hpp"

namespace lbsd {

namespace {

constexpr int kMTPB = 256;               // threads per block: 4 independent wavefronts
constexpr int kMNW = kMTPB / 64;
constexpr int kMH = kHalo;               // largest displacement of a packet per axis
constexpr int kMCols = 64 - 2 * kMH;     // destination columns per tile
static_assert(kMCols == kMarchCols, "tile width shared with the host");

// (h, l) += x with the rounding error of h + x carried into l (TwoSum).
__device__ __forceinline__ void dd_add(double& h, double& l, double x)
{
#pragma clang fp contract(off)
    const double s = h + x;
    const double bp = s - h;
    const double e = (h - (s - bp)) + (x - bp);
    h = s;
    l = l + e;
}

// ---- sources ----------------------------------------------------------------
// One source node as the march uses it.
template <typename T, bool REST, bool SP>
struct MNode {
    T vx, vy, ry, K;      // v (lattice units), y fraction, |v|^2/2 + phi
    T m[2][2];            // lane mass of level l + 1 at x corner k: d (1 - r_x), d r_x
    T z[REST ? 2 : 1];    // rest-group mass at x corner k
    T chi;                // two gases: mass fraction of gas 1
    int fx, fy, c1;
};

// Per-node primitives (eq. 15, 24-26, 28-29) in FP64 whatever the storage
// type: in FP32 storage the energy bookkeeping (E -> e, A, the d_1 / d_2 split
// near a switch of c'_1) is where FP32 arithmetic would lose the most, and FP64
// costs the same VALU issue rate on this chip.  IEEE: any operands, bad states
// included (they get zero mass); otherwise the operands are tame.  NOVY: v_y is
// +-0.  SP: the node's gas is the mixture of the two by mass fraction (c_v
// weighted, one gas constant).
template <typename T, bool REST, bool SP, bool NOVY, bool IEEE>
__device__ __forceinline__ MNode<T, REST, SP> march_node(double m0, double m1, double m2, double m3, double m4,
                                                         const Consts& kc, bool bad)
{
#pragma clang fp contract(off)
    constexpr bool FAST = sizeof(T) < 8;
    MNode<T, REST, SP> s;
    if constexpr (IEEE) {  // a bad state emits nothing: a harmless node of zero mass stands for it
        m0 = bad ? 1.0 : m0;
        m1 = bad ? 0.0 : m1;
        m2 = bad ? 0.0 : m2;
        m3 = bad ? 0.0 : m3;
        m4 = bad ? 0.0 : m4;
    }
    const Quot<FAST, IEEE> by_rho(m0);
    double Dg1 = kc.Dg1, phi = kc.phi_coef;
    s.chi = (T)0;
    if constexpr (SP) {
        double chi = by_rho(m4);
        chi = chi < 0.0 ? 0.0 : (chi > 1.0 ? 1.0 : chi);
        const double gm1 = pdiv<FAST>(1.0, pdiv<FAST>(chi, kc.g1m1) + pdiv<FAST>(1.0 - chi, kc.g2m1));
        Dg1 = 2.0 * gm1;
        phi = 1.0 - 1.0 * gm1;
        s.chi = (T)chi;
    }
    const double vx = by_rho(m1), vy = NOVY ? 0.0 : by_rho(m2), E = by_rho(m3);
    double v2 = vx * vx;
    if constexpr (!NOVY) v2 += vy * vy;
    double e = E - 0.5 * v2;
    if (e < 0.0) e = 0.0;
    double d0 = 0.0, rest = m0;
    double A;
    if constexpr (REST) {
        d0 = kc.delta0 * m0;
        rest = m0 - d0;
        A = Quot<FAST, IEEE>(rest)(Dg1 * e * m0);
    } else {
        A = by_rho(Dg1 * e * m0);
    }
    if constexpr (IEEE) {
        if (!(A >= 0.0)) A = 0.0;
        if (A > (double)kMaxC1 * (double)kMaxC1) A = (double)kMaxC1 * (double)kMaxC1;
    }
    // c'_1 (eq. 26) and w = (A - c'_1^2) / (2 c'_1 + 1): exact comparisons
    // for the usual c'_1 <= 2, the integer root elsewhere
    double w;
    if (__any(A >= 9.0)) {
        s.c1 = isqrt_floor<double>(A);
        w = level_w(A, s.c1);
    } else {
        const bool g1 = A >= 1.0, g2 = A >= 4.0;
        s.c1 = (g1 ? 1 : 0) + (g2 ? 1 : 0);
        w = (A - (g2 ? 4.0 : (g1 ? 1.0 : 0.0))) * (g2 ? 1.0 / 5.0 : (g1 ? 1.0 / 3.0 : 1.0));
    }
    const double per = rest * kc.inv_b1;
    double d2 = per * w, d1 = per - d2;
    if constexpr (IEEE) {
        d2 = bad ? 0.0 : d2;
        d1 = bad ? 0.0 : d1;
        if constexpr (REST) d0 = bad ? 0.0 : d0;
    }
    const double fvx = floor(vx), rx = vx - fvx, ax = 1.0 - rx;
    s.fx = (int)fvx;
    s.vx = (T)vx;
    s.fy = 0;
    s.vy = s.ry = (T)0;
    if constexpr (!NOVY) {
        const double fvy = floor(vy);
        s.fy = (int)fvy;
        s.vy = (T)vy;
        s.ry = (T)(vy - fvy);
    }
    s.m[0][0] = (T)(d1 * ax);
    s.m[0][1] = (T)(d1 * rx);
    s.m[1][0] = (T)(d2 * ax);
    s.m[1][1] = (T)(d2 * rx);
    if constexpr (REST) {
        s.z[0] = (T)(d0 * ax);
        s.z[1] = (T)(d0 * rx);
    }
    s.K = (T)__builtin_fma(phi, e, 0.5 * v2);
    return s;
}

// ---- stage A ----------------------------------------------------------------
// Corner sums of one speed in this lane's column: m, m v_x, m v_y, m K (after
// march_lane_energy: m (K + c^2/2)), m chi.
template <typename T>
struct CSum {
    T m, v, w, e, x;
    CSum() = default;
    // (member by member: a copy of the whole struct would keep arrays of it in memory)
    __device__ __forceinline__ CSum(const CSum& o) : m(o.m), v(o.v), w(o.w), e(o.e), x(o.x) {}
    __device__ __forceinline__ CSum& operator=(const CSum& o)
    {
        m = o.m, v = o.v, w = o.w, e = o.e, x = o.x;
        return *this;
    }
    __device__ __forceinline__ void zero() { m = v = w = e = x = (T)0; }
};
template <bool VY, bool SP, typename T>
__device__ __forceinline__ void cadd(CSum<T>& a, const CSum<T>& b)
{
#pragma clang fp contract(off)
    a.m += b.m;
    a.v += b.v;
    a.e += b.e;
    if constexpr (VY) a.w += b.w;
    if constexpr (SP) a.x += b.x;
}
template <bool VY, bool SP, typename T>
__device__ __forceinline__ CSum<T> cshr(CSum<T> a)
{
    a.m = lshr(a.m);
    a.v = lshr(a.v);
    a.e = lshr(a.e);
    if constexpr (VY) a.w = lshr(a.w);
    if constexpr (SP) a.x = lshr(a.x);
    return a;
}
template <bool VY, bool SP, typename T>
__device__ __forceinline__ CSum<T> cshl(CSum<T> a)
{
    a.m = lshl(a.m);
    a.v = lshl(a.v);
    a.e = lshl(a.e);
    if constexpr (VY) a.w = lshl(a.w);
    if constexpr (SP) a.x = lshl(a.x);
    return a;
}

// Masses m0, m1 at the x corners 0, 1 of sources with floor(v_x) = F
// (wave-uniform), gathered into the columns they land on.
template <bool VY, bool SP, typename T, typename Node>
__device__ __forceinline__ CSum<T> corner_sum(T m0, T m1, const Node& s, int F)
{
#pragma clang fp contract(off)
    CSum<T> r;
    r.w = r.x = (T)0;
    if (F >= 0) {
        r.m = m0 + lshr(m1);
        r.v = fmaT(m0, s.vx, lshr(m1 * s.vx));
        r.e = fmaT(m0, s.K, lshr(m1 * s.K));
        if constexpr (VY) r.w = fmaT(m0, s.vy, lshr(m1 * s.vy));
        if constexpr (SP) r.x = fmaT(m0, s.chi, lshr(m1 * s.chi));
#pragma unroll 1
        for (int i = 0; i < F; ++i) r = cshr<VY, SP>(r);
    } else {
        r.m = m1 + lshl(m0);
        r.v = fmaT(m1, s.vx, lshl(m0 * s.vx));
        r.e = fmaT(m1, s.K, lshl(m0 * s.K));
        if constexpr (VY) r.w = fmaT(m1, s.vy, lshl(m0 * s.vy));
        if constexpr (SP) r.x = fmaT(m1, s.chi, lshl(m0 * s.chi));
#pragma unroll 1
        for (int i = F; i < -1; ++i) r = cshl<VY, SP>(r);
    }
    return r;
}

// ---- stage B ----------------------------------------------------------------
// What lands on one destination row in this column: rho, rho v_x, the m v_y
// part of rho v_y, rho E, rho chi.
template <typename T>
struct Dest {
    T m, p, w, e, x;
    Dest() = default;
    __device__ __forceinline__ Dest(const Dest& o) : m(o.m), p(o.p), w(o.w), e(o.e), x(o.x) {}
    __device__ __forceinline__ Dest& operator=(const Dest& o)
    {
        m = o.m, p = o.p, w = o.w, e = o.e, x = o.x;
        return *this;
    }
    __device__ __forceinline__ void zero() { m = p = w = e = x = (T)0; }
};

// The lanes +-c along x of the corner sums u (u.e = sum m (K + c^2/2)), added
// to t.  The pair's lane momentum enters as (m_+ - m_-) c, exactly zero for
// mirrored packets.
template <int C, bool VY, bool SP, typename T>
__device__ __forceinline__ void add_xlanes(Dest<T>& t, const CSum<T>& u)
{
#pragma clang fp contract(off)
    CSum<T> a = u, b = u;
#pragma unroll
    for (int i = 0; i < C; ++i) {
        a = cshr<VY, SP>(a);
        b = cshl<VY, SP>(b);
    }
    t.m += a.m + b.m;
    t.p += fmaT((T)C, a.m - b.m, a.v + b.v);
    t.e += fmaT((T)C, a.v - b.v, a.e + b.e);
    if constexpr (VY) t.w += a.w + b.w;
    if constexpr (SP) t.x += a.x + b.x;
}
// The lane +-c along y (sc = +-c) of the corner sums u, added to t.
template <bool VY, bool SP, typename T>
__device__ __forceinline__ void add_ylane(Dest<T>& t, const CSum<T>& u, T sc)
{
#pragma clang fp contract(off)
    t.m += u.m;
    t.p += u.v;
    if constexpr (VY) {
        t.w += u.w;
        t.e += fmaT(sc, u.w, u.e);
    } else {
        t.e += u.e;
    }
    if constexpr (SP) t.x += u.x;
}
template <bool VY, bool SP, typename T>
__device__ __forceinline__ void add_here(Dest<T>& t, const CSum<T>& u)
{
#pragma clang fp contract(off)
    t.m += u.m;
    t.p += u.v;
    t.e += u.e;
    if constexpr (VY) t.w += u.w;
    if constexpr (SP) t.x += u.x;
}

// Speeds of the corner sums kept in registers: 0, 1, 2 (c'_1 <= 1), and 3 with
// a rest level (whose A is larger by 1 / (1 - delta0), so c'_1 = 2 is common).
template <bool REST>
constexpr int kSpeeds = REST ? 4 : 3;

// The lane momentum of rho v_y at a row d, sum over c of c (M_c[d - c] -
// M_c[d + c]), in double-length arithmetic: a planar flow (equal rows) must
// keep v_y = 0 exactly.  hist[c][k] = M_c of the k-th row before the current
// one; the current row is d + LB.  Equal rows give exactly 0.
template <int LB, typename T>
struct LaneHist {
    T h[LB + 1][2 * LB + 1];
    __device__ __forceinline__ void zero()
    {
#pragma unroll
        for (int c = 1; c <= LB; ++c)
#pragma unroll
            for (int k = 0; k <= LB + c; ++k) h[c][k] = (T)0;
    }
    __device__ __forceinline__ double lane_py() const  // h[c][0] holds the current row
    {
        bool eq = true;
#pragma unroll
        for (int c = 1; c <= LB; ++c) eq = eq && h[c][LB + c] == h[c][LB - c];
        if (__all(eq)) return 0.0;
        double a = 0.0, l = 0.0;
#pragma unroll
        for (int c = LB; c >= 1; --c) dd_add(a, l, (double)c * (double)h[c][LB + c]);
#pragma unroll
        for (int c = 1; c <= LB; ++c) dd_add(a, l, -((double)c * (double)h[c][LB - c]));
        return eq ? 0.0 : a + l;
    }
    __device__ __forceinline__ void shift()
    {
#pragma unroll
        for (int c = 1; c <= LB; ++c)
#pragma unroll
            for (int k = LB + c; k > 0; --k) h[c][k] = h[c][k - 1];
    }
};

// LaneHist in LDS (the lane's own columns): a ring by row for each speed, LB + c
// values.
template <int LB>
struct LaneHistLds {
    static constexpr int N = LB * LB + LB * (LB + 1) / 2;  // sum over c = 1 .. LB of LB + c
    double* h;        // this lane's column, rows 64 apart
    int at[LB + 1];   // the current row's place (so far: the row LB + c before it)
    double now[LB + 1];
    static constexpr int off(int c) { return (c - 1) * LB + c * (c - 1) / 2; }
    __device__ __forceinline__ void init(double* column)
    {
        h = column;
        static_for<N>([&](auto i) { h[i * 64] = 0.0; });
        static_for<LB>([&](auto i) { at[i + 1] = 0; });
    }
    __device__ __forceinline__ void set(int c, double m) { now[c] = m; }
    __device__ __forceinline__ double lane_py() const
    {
        bool eq = true;
        double up[LB + 1], dn[LB + 1];
        static_for<LB>([&](auto i) {
            constexpr int c = i + 1;
            up[c] = h[(off(c) + at[c]) * 64];
            const int k = at[c] - (LB - c);
            dn[c] = c == LB ? now[c] : h[(off(c) + (k < 0 ? k + LB + c : k)) * 64];
            eq = eq && up[c] == dn[c];
        });
        if (__all(eq)) return 0.0;
        double a = 0.0, l = 0.0;
        static_for<LB>([&](auto i) { dd_add(a, l, (double)(LB - i) * up[LB - i]); });
        static_for<LB>([&](auto i) { dd_add(a, l, -((double)(i + 1) * dn[i + 1])); });
        return eq ? 0.0 : a + l;
    }
    __device__ __forceinline__ void shift()
    {
        static_for<LB>([&](auto i) {
            constexpr int c = i + 1;
            h[(off(c) + at[c]) * 64] = now[c];
            at[c] = at[c] + 1 == LB + c ? 0 : at[c] + 1;
        });
    }
};

// Fields of a pass over a tile: rho, rho v_x and rho E; rho v_y; rho chi.
constexpr int kMPE = 1, kVy = 2, kChi = 4, kAllFields = 7;
constexpr bool has_field(int fields, int c) { return fields >> (c == 2 ? 1 : (c == 4 ? 2 : 0)) & 1; }
constexpr int field_count(int fields)
{
    return (fields & kMPE ? 3 : 0) + (fields & kVy ? 1 : 0) + (fields & kChi ? 1 : 0);
}
// Place of field c of Dest (m, p, w, e, x) among them, -1 if it is none.
constexpr int field_place(int fields, int c)
{
    int n = 0;
    for (int i = 0; i < c; ++i) n += has_field(fields, i) ? 1 : 0;
    return has_field(fields, c) ? n : -1;
}

// The 2 H + 1 pending rows of a far march for the fields FIELDS (a ring by row):
// those of them that are kept in LDS (LDS) and, with rho v_y, the lane momentum that
// far-reaching classes bring, in double-length sums (in LDS with HL).  COLS: 64, or
// the destination columns and one more, where the halo lanes put what they form.
template <typename T_, int FIELDS_, int LDS, bool HL_, int COLS>
struct FarRows {
    using T = T_;
    static constexpr int NR = 2 * kMH + 1, FIELDS = FIELDS_, IN = FIELDS & LDS, OUT = FIELDS & ~LDS;
    static constexpr int NV = field_count(IN);
    static constexpr bool HL = HL_, L = (FIELDS & kVy) != 0;
    double hl[L && HL ? NR : 1][2][L && HL ? COLS : 1];
    T v[NV ? NR : 1][NV ? NV : 1][NV ? COLS : 1];
    // The rest of a lane's rows, in scratch memory (an array of its own: in one struct
    // with a pointer to the rows, that pointer would be in memory too, and the rows'
    // accesses would not know that they are LDS).
    struct Own {
        T v[NR][OUT ? field_count(OUT) : 1];
        double hl[L && !HL ? NR : 1][2];
    };
    static __device__ __forceinline__ int col(int lane)
    {
        return COLS == 64 ? lane : (int)min((unsigned)(lane - kMH), (unsigned)kMCols);
    }
};
template <typename R>
__device__ __forceinline__ Dest<typename R::T> far_get(const R& rows, const typename R::Own& own, int j, int col)
{
    typename R::T f[5] = {};
    static_for<5>([&](auto c) {
        constexpr int in = field_place(R::IN, c), out = field_place(R::OUT, c);
        if constexpr (in >= 0) f[c] = rows.v[j][in][col];
        if constexpr (out >= 0) f[c] = own.v[j][out];
    });
    Dest<typename R::T> d;
    d.m = f[0], d.p = f[1], d.w = f[2], d.e = f[3], d.x = f[4];
    return d;
}
template <typename R>
__device__ __forceinline__ void far_put(R& rows, typename R::Own& own, int j, int col, const Dest<typename R::T>& d)
{
    const typename R::T f[5] = {d.m, d.p, d.w, d.e, d.x};
    static_for<5>([&](auto c) {
        constexpr int in = field_place(R::IN, c), out = field_place(R::OUT, c);
        if constexpr (in >= 0) rows.v[j][in][col] = f[c];
        if constexpr (out >= 0) own.v[j][out] = f[c];
    });
}
// The lane momentum of row j: its two parts.
template <typename R>
__device__ __forceinline__ void far_get_lane(const R& rows, const typename R::Own& own, int j, int col, double& h, double& l)
{
    if constexpr (R::HL) h = rows.hl[j][0][col], l = rows.hl[j][1][col];
    else h = own.hl[j][0], l = own.hl[j][1];
}
template <typename R>
__device__ __forceinline__ void far_put_lane(R& rows, typename R::Own& own, int j, int col, double h, double l)
{
    if constexpr (R::HL) rows.hl[j][0][col] = h, rows.hl[j][1][col] = l;
    else own.hl[j][0] = h, own.hl[j][1] = l;
}
template <typename R>
__device__ __forceinline__ void far_zero(R& rows, typename R::Own& own, int j, int col)
{
    Dest<typename R::T> d;
    d.zero();
    far_put(rows, own, j, col, d);
    if constexpr (R::L) far_put_lane(rows, own, j, col, 0.0, 0.0);
}
template <typename R>
__device__ __forceinline__ void far_add(R& rows, typename R::Own& own, int j, int col, const Dest<typename R::T>& d)
{
#pragma clang fp contract(off)
    Dest<typename R::T> q = far_get(rows, own, j, col);
    q.m += d.m;
    q.p += d.p;
    q.w += d.w;
    q.e += d.e;
    q.x += d.x;
    far_put(rows, own, j, col, q);
}
// Lane momentum g to row j.
template <typename R>
__device__ __forceinline__ void far_add_lane(R& rows, typename R::Own& own, int j, int col, double g)
{
    if constexpr (R::L) {
        double h, l;
        far_get_lane(rows, own, j, col, h, l);
        dd_add(h, l, g);
        far_put_lane(rows, own, j, col, h, l);
    }
}

// What a wavefront of the general pass keeps in LDS: the rows of a far march or,
// with NEAR, the near form's destination FIFO and lane momentum history (they take
// 86 registers in FP64 with a rest level, 64 with two gases, and without them two
// wavefronts fit a SIMD: four states on 2048^2 nodes 309 and 310 us per step, with
// one wavefront and all of it in registers 407 and 382).
//
// A far march's 11 rows of four or five fields do not fit scratch memory's way to the
// L2 (flows with |v_y| around 1.5 waited for it 76 % of the time), nor does all of
// it fit a wavefront's 20 KB of LDS in FP64: what is read and written most is there,
// the lane momentum's two parts and rho chi in scratch memory.  us per step on 2048^2
// nodes, all in scratch memory / so: |v_y| around 1.5 804 / 370, two gases 1664 /
// 1043; four states after 200 steps, when a few nodes in some tiles are far, 548 /
// 510, two gases 683 / 549.  (Two marches, each with all it needs in LDS: 417, 769,
// 666 and 668.)  With a rest level, one march would spill 116 registers, and far tiles
// are marched twice, for some of the fields each (1090 / 531).  With a rest level and
// two gases one wavefront fits a SIMD, and the LDS holds all fields (1448 / 637).
// FP32 keeps its fields, half the size, in scratch memory: in LDS they would cost
// the pools' third block per CU (409 / 369; two gases 779 / 627).
template <typename T, bool REST, bool SP>
struct MarchStash {
    static constexpr bool FP64 = sizeof(T) == 8, NEAR = FP64 && REST != SP;
    static constexpr int LB = kSpeeds<REST> - 1, ND = SP ? 5 : 4;
    // fields of the far marches (F2 = 0: all in the first), those of them in LDS, and
    // whether the lane momentum is
    static constexpr int ALL = kMPE | kVy | (SP ? kChi : 0);
    static constexpr int F1 = FP64 && REST && !SP ? kMPE : ALL, F2 = ALL & ~F1;
    static constexpr int LDS = !FP64 ? 0 : SP && !REST ? kMPE | kVy : ALL;
    static constexpr bool HL = !FP64 || REST;
    static constexpr int COLS = FP64 && REST && SP ? 64 : kMCols + 1;
    struct Near {
        double hist[NEAR ? LaneHistLds<LB>::N : 1][NEAR ? 64 : 1], fifo[NEAR ? 2 * LB * ND : 1][NEAR ? 64 : 1];
    };
    union {
        Near near;
        FarRows<T, F1, LDS, HL, COLS> far1;
        FarRows<T, F2, LDS, HL, COLS> far2;
    };
    template <int FIELDS>
    __device__ __forceinline__ auto& far()
    {
        if constexpr (FIELDS != F1 && FIELDS == F2) return far2;
        else return far1;  // (unused by the near form)
    }
};

template <typename T, int NF>
struct MarchIO {  // a tile's source columns and destination columns of one lane
    const T* Y;
    T* Yn;
    int64_t nx, ny, nn;
    int bc_y;
    uint32_t sxb, gxb;  // byte offsets of the source / destination column in a row (nx <= 2^28)
    bool mir_x, dest;

    __device__ __forceinline__ void set(const T* Yi, T* Yo, const Grid& g, int64_t X0, int lane)
    {
        Y = Yi;
        Yn = Yo;
        nx = g.nx;
        ny = g.ny;
        nn = nx * ny;
        bc_y = g.bc_y;
        const int64_t gx = X0 - kMH + lane;
        const int64_t sx = source_idx(gx, nx, g.bc_x, &mir_x);
        sxb = (uint32_t)sx * (uint32_t)sizeof(T);
        gxb = (uint32_t)gx * (uint32_t)sizeof(T);
        dest = lane >= kMH && lane < 64 - kMH && gx < nx;
    }
    // Moments of this lane's source column in row gy (halo rows mapped by the
    // boundary); *mir_y: the row is a mirror image beyond a wall.  Mirror
    // images negate normal momentum when the row is used, not here, so that
    // loads issued a row ahead are not waited for.
    __device__ __forceinline__ void load(int64_t gy, T (&m)[NF], bool* mir_y) const
    {
        const int64_t yy = source_idx(gy, ny, bc_y, mir_y);
        const T* row = Y + yy * nx;
#pragma unroll
        for (int c = 0; c < NF; ++c) m[c] = *(const T*)((const char*)(row + (int64_t)c * nn) + sxb);
    }
    template <int FIELDS = kAllFields>
    __device__ __forceinline__ void store(int64_t row, T r, T p, T py, T e, T x) const
    {
        T* o = Yn + row * nx;
        const T v[5] = {r, p, py, e, x};
        static_for<NF>([&](auto c) {
            if constexpr (has_field(FIELDS, c)) *(T*)((char*)(o + c * nn) + gxb) = v[c];
        });
    }
};

// A tile's row of partials: field sums (rho chi at index 6), reach, error bits;
// of a march for some of the fields, theirs.
template <int NF, int FIELDS = kAllFields>
__device__ __forceinline__ void march_partials(double (&tot)[NF], int reach, bool bad, double* __restrict__ prow,
                                               int lane)
{
    static_for<NF>([&](auto c) {
        if constexpr (has_field(FIELDS, c)) tot[c] = wave_sum(tot[c]);
    });
    if (lane == 0) {
        static_for<NF>([&](auto c) {
            if constexpr (has_field(FIELDS, c)) prow[c < 4 ? c : 6] = tot[c];
        });
        if constexpr ((FIELDS & kMPE) != 0) {
            prow[4] = (double)reach;
            prow[5] = (double)((reach > kMH ? kErrReach : 0) | (bad ? kErrState : 0));
        }
    }
}

// The lean pass, one tile of rows [Y0, ylast): x-planar flows, every source
// staged with v_y = 0 exactly, c'_1 <= kSpeeds - 2 and a reach within H.  A
// packet then moves at most LB = kSpeeds - 1 rows, stage A needs no row FIFO
// (a source's corners lie in its own row) and no packet carries m v_y.  At
// the first row that breaks these conditions the wavefront gives the tile up
// (returns false) and the general pass computes it.
//
// Bound by HBM at large sizes: 4 loads and 4 stores per lane and row against
// about 200 VALU instructions (FP64), in four wavefronts per SIMD: 4096^2 nodes
// take 262 us (4.5 TB/s, a copy 5.1), where packets rebuilt from LDS rows
// took 352; in FP32 VALU issue bounds it, 158 us against 452.
template <typename T, bool REST, bool SP>
__device__ __forceinline__ bool march_tile_lean(const MarchIO<T, SP ? 5 : 4>& io, const Consts& k, int64_t Y0,
                                                int64_t ylast, double* __restrict__ prow)
{
#pragma clang fp contract(off)
    constexpr int NF = SP ? 5 : 4, NS = kSpeeds<REST>, LB = NS - 1;
    const int lane = threadIdx.x & 63;
    const int nrows = (int)(ylast - Y0) + 2 * LB;
    Dest<T> f[2 * LB + 1];  // slot j + LB: destination row (current row) + j
#pragma unroll
    for (int j = 0; j <= 2 * LB; ++j) f[j].zero();
    LaneHist<LB, T> hist;
    hist.zero();
    double tot[NF] = {};
    int reach = 0;
    T cur[NF];
    bool mir_y = false;
    io.load(Y0 - LB, cur, &mir_y);

#pragma unroll 1
    for (int r = 0; r < nrows; ++r) {
        const T r0 = cur[0], r1 = io.mir_x ? -cur[1] : cur[1], r3 = cur[3];
        const bool vy0 = cur[2] == (T)0;  // a mirrored row's sign does not matter
        bool ok = tame(r0, r1, (T)0, r3) && (!REST || k.delta0 <= kTameDelta0);
        if constexpr (SP) ok = ok && zero_or_normal(cur[NF - 1]);
        if (!__all(vy0)) return false;
        MNode<T, REST, SP> s;
        if (__all(ok)) {
            s = march_node<T, REST, SP, true, false>(r0, r1, 0.0, r3, cur[NF - 1], k, false);
        } else {
            bool bad = !((double)r0 > 0.0) || !isfinite(r0) || !isfinite(r1) || !isfinite(r3);
            if constexpr (SP) bad = bad || !isfinite(cur[NF - 1]);
            if (__any(bad)) return false;  // reported by the general pass
            s = march_node<T, REST, SP, true, true>(r0, r1, 0.0, r3, cur[NF - 1], k, false);
        }
        if (r + 1 < nrows) io.load(Y0 - LB + r + 1, cur, &mir_y);  // arrives while this row is gathered

        // stage A, class by class (floor(v_x), which its conversion saturates, clamped
        // far beyond any admissible reach)
        CSum<T> u[NS];
        int has = 0;  // speeds present in the row (bit c)
        const int key = min(max(s.fx, -16), 15) * 8 + min(s.c1, 7);
        const int key0 = __builtin_amdgcn_readfirstlane(key);
        if (__all(key == key0)) {
            const int F = key0 >> 3, C = key0 & 7;
            const int cr = class_reach(F, C);
            if (C > NS - 2 || cr > kMH) return false;
            reach = max(reach, cr);
            has = 3 << C;
#pragma unroll
            for (int c = 0; c < NS; ++c) u[c].zero();
#pragma unroll
            for (int c = 0; c + 1 < NS; ++c) {
                if (C != c) continue;
                T a0 = s.m[0][0], a1 = s.m[0][1];
                if (c == 0) {
                    a0 = (T)4 * a0;
                    a1 = (T)4 * a1;
                    if constexpr (REST) {
                        a0 += s.z[0];
                        a1 += s.z[1];
                    }
                }
                u[c] = corner_sum<false, SP, T>(a0, a1, s, F);
                u[c + 1] = corner_sum<false, SP, T>(s.m[1][0], s.m[1][1], s, F);
            }
            if constexpr (REST) {
                has |= 1;
                if (C > 0) u[0] = corner_sum<false, SP, T>(s.z[0], s.z[1], s, F);
            }
        } else {
#pragma unroll
            for (int c = 0; c < NS; ++c) u[c].zero();
            unsigned long long todo = __ballot(true);
#pragma unroll 1
            while (todo != 0) {
                const int kc = __builtin_amdgcn_readlane(key, __builtin_ctzll(todo));
                const bool in = key == kc;
                todo &= ~__ballot(in);
                const int F = kc >> 3, C = kc & 7;
                const int cr = class_reach(F, C);
                if (C > NS - 2 || cr > kMH) return false;
                reach = max(reach, cr);
                has |= 3 << C;
                const T b0 = in ? s.m[1][0] : (T)0, b1 = in ? s.m[1][1] : (T)0;
                const CSum<T> ub = corner_sum<false, SP, T>(b0, b1, s, F);
                T a0 = in ? s.m[0][0] : (T)0, a1 = in ? s.m[0][1] : (T)0;
                T z0 = (T)0, z1 = (T)0;
                if constexpr (REST) {
                    has |= 1;
                    z0 = in ? s.z[0] : (T)0;
                    z1 = in ? s.z[1] : (T)0;
                }
                if (C == 0) {
                    a0 = (T)4 * a0;
                    a1 = (T)4 * a1;
                    if constexpr (REST) {
                        a0 += z0;
                        a1 += z1;
                    }
                }
                const CSum<T> ua = corner_sum<false, SP, T>(a0, a1, s, F);
                static_for<NS - 1>([&](auto c) {
                    if (C != c) return;
                    cadd<false, SP>(u[c], ua);
                    cadd<false, SP>(u[c + 1], ub);
                    keep_apart<c>();
                });
                if constexpr (REST) {
                    if (C > 0) cadd<false, SP>(u[0], corner_sum<false, SP, T>(z0, z1, s, F));
                }
            }
        }

        // stage B
        Dest<T> t;
        t.zero();
        if (has & 1) add_here<false, SP>(t, u[0]);
#pragma unroll
        for (int c = 1; c < NS; ++c) {
            hist.h[c][0] = u[c].m;
            if (!(has >> c & 1)) continue;
            u[c].e = fmaT((T)(0.5 * c * c), u[c].m, u[c].e);
            if (c == 1) add_xlanes<1, false, SP>(t, u[c]);
            if (c == 2) add_xlanes<2, false, SP>(t, u[c]);
            if (c == 3) add_xlanes<3, false, SP>(t, u[c]);
            add_ylane<false, SP>(f[LB - c], u[c], (T)0);
            add_ylane<false, SP>(f[LB + c], u[c], (T)0);
        }
        f[LB].m += t.m;
        f[LB].p += t.p;
        f[LB].e += t.e;
        if constexpr (SP) f[LB].x += t.x;

        // row (current) - LB is complete
        if (r >= 2 * LB && io.dest) {
            const T py = (T)hist.lane_py();
            io.store(Y0 + r - 2 * LB, f[0].m, f[0].p, py, f[0].e, f[0].x);
            tot[0] += (double)f[0].m;
            tot[1] += (double)f[0].p;
            tot[2] += (double)py;
            tot[3] += (double)f[0].e;
            if constexpr (SP) tot[NF - 1] += (double)f[0].x;
        }
        hist.shift();
#pragma unroll
        for (int j = 0; j < 2 * LB; ++j) f[j] = f[j + 1];
        f[2 * LB].zero();
    }
    march_partials<NF>(tot, reach, false, prow, lane);
    return true;
}

// The general pass, rows [Y0, ylast) of one tile: any flow within the halo.
// Near classes (floor(v_y) in {-1, 0}, c'_1 <= kSpeeds - 2) go through the two
// stages: their corners reach the rows -1 .. 1 from the source, so the corner
// sums have a FIFO of three rows, and row (current) - 1 goes through stage B
// once the current row is in.  FAR = false marches these alone and returns
// false at the first source of another class within H rows of the
// destinations (the rows further out than the packets of near classes come
// from are looked at for that only).  FAR = true takes every class: the others
// add their packets, class by class and corner row by corner row, straight to
// the 2 H + 1 destination rows they can reach (FarRows), for the fields FIELDS (what
// the others alone need falls away; the first march, with rho, reports reach and
// errors).  A node that no far source reaches gets the same bits either way.
// Returns 1 when complete, 0 when a far class was met (FAR = false only).
// *unlean: some source within LB rows is beyond the lean pass.
template <typename T, bool REST, bool SP, bool FAR, int FIELDS>
__device__ __forceinline__ bool march_tile_general(const MarchIO<T, SP ? 5 : 4>& io, const Consts& k, int64_t Y0,
                                                   int64_t ylast, double* __restrict__ prow,
                                                   MarchStash<T, REST, SP>& st, bool* unlean)
{
#pragma clang fp contract(off)
    constexpr int NF = SP ? 5 : 4, NS = kSpeeds<REST>, LB = NS - 1;
    constexpr int NSL = 2 * LB + 1;         // destination FIFO: slot j + LB is row (current) - 1 + j
    constexpr int LD = FAR ? kMH : LB + 1;  // row (current) - LD is written out
    constexpr int EDGE = kMH - LB - 1;      // rows looked at only (FAR = false)
    constexpr bool VY = (FIELDS & kVy) != 0;
    using S = MarchStash<T, REST, SP>;
    auto& far = st.template far<FIELDS>();
    using Rows = std::remove_reference_t<decltype(far)>;
    typename Rows::Own own;
    const auto far_row = [](int r, int o) { return (r + o + 2 * (2 * kMH + 1)) % (2 * kMH + 1); };  // row (current) + o
    const int lane = threadIdx.x & 63, col = Rows::col(lane);
    const int nrows = (int)(ylast - Y0) + 2 * kMH;
    Dest<T> f[NSL];  // (with FIFO: in LDS)
    static_for<NSL>([&](auto j) { f[j].zero(); });
    CSum<T> u[3][NS];  // corner sums of rows (current) - 1, 0, + 1
    static_for<NS>([&](auto c) {
        u[0][c].zero();
        u[1][c].zero();
        u[2][c].zero();
    });
    int has0 = 0, has1 = 0, has2 = 0;  // speeds present in them
    constexpr bool FIFO = S::NEAR && !FAR;
    constexpr int ND = S::ND;
    std::conditional_t<FIFO, LaneHistLds<LB>, LaneHist<LB, T>> hist;
    if constexpr (FIFO) {
        hist.init(&st.near.hist[0][lane]);
        static_for<2 * LB * ND>([&](auto j) { st.near.fifo[j][lane] = 0.0; });
    } else {
        hist.zero();
    }
    if constexpr (FAR) {
#pragma unroll 1
        for (int j = 0; j <= 2 * kMH; ++j) far_zero(far, own, j, col);
    }
    double tot[NF] = {};
    int reach = 0;
    bool anybad = false, notlean = false;
    T cur[NF];
    bool mir_y = false, mir_next = false;
    io.load(Y0 - kMH, cur, &mir_y);

#pragma unroll 1
    for (int r = 0; r < nrows; ++r) {
        const T r0 = cur[0], r1 = io.mir_x ? -cur[1] : cur[1], r2 = mir_y ? -cur[2] : cur[2], r3 = cur[3];
        bool ok = tame(r0, r1, r2, r3) && (!REST || k.delta0 <= kTameDelta0);
        if constexpr (SP) ok = ok && zero_or_normal(cur[NF - 1]);
        MNode<T, REST, SP> s;
        bool badw = false;
        if (__all(ok)) {
            s = march_node<T, REST, SP, false, false>(r0, r1, r2, r3, cur[NF - 1], k, false);
        } else {
            bool bad = !((double)r0 > 0.0) || !isfinite(r0) || !isfinite(r1) || !isfinite(r2) || !isfinite(r3);
            if constexpr (SP) bad = bad || !isfinite(cur[NF - 1]);
            badw = __any(bad);
            s = march_node<T, REST, SP, false, true>(r0, r1, r2, r3, cur[NF - 1], k, bad);
        }
        anybad |= badw;
        if (r + 1 < nrows) io.load(Y0 - kMH + r + 1, cur, &mir_next);
        mir_y = mir_next;
        if (r >= kMH - LB && r < nrows - (kMH - LB))
            notlean |= badw || __any(s.vy != (T)0 || s.c1 > NS - 2);

        // stage A, class by class (floor(v) clamped far beyond any admissible reach)
        const int kfx = min(max(s.fx, -32), 31), kfy = min(max(s.fy, -32), 31), kc1 = min(s.c1, 31);
        const int key = (kfy + 32) << 11 | (kfx + 32) << 5 | kc1;
        const bool gather = FAR || (r >= EDGE && r < nrows - EDGE);
        unsigned long long todo = __ballot(true);
#pragma unroll 1
        while (todo != 0) {
            const int kc = __builtin_amdgcn_readlane(key, __builtin_ctzll(todo));
            const bool in = key == kc;
            todo &= ~__ballot(in);
            const int FY = (kc >> 11) - 32, F = (kc >> 5 & 63) - 32, C = kc & 31;
            const int cr = max(class_reach(F, C), class_reach(FY, C));
            reach = max(reach, cr);
            const bool near = (FY == 0 || FY == -1) && C <= NS - 2 && cr <= kMH;
            if (!near && !FAR) return false;
            if (!gather || cr > kMH) continue;  // too far a reach is reported, not gathered
#pragma unroll 1
            for (int ky = 0; ky < 2; ++ky) {
                const T w = ky ? s.ry : (T)1 - s.ry;
                const T wi = in ? w : (T)0;
                if (ky && !__any(wi != (T)0)) break;  // integral v_y: no mass at the second corner row
                T a0 = s.m[0][0] * wi, a1 = s.m[0][1] * wi;
                const T b0 = s.m[1][0] * wi, b1 = s.m[1][1] * wi;
                T z0 = (T)0, z1 = (T)0;
                if constexpr (REST) {
                    z0 = s.z[0] * wi;
                    z1 = s.z[1] * wi;
                }
                if (C == 0) {
                    a0 = (T)4 * a0;
                    a1 = (T)4 * a1;
                    if constexpr (REST) {
                        a0 += z0;
                        a1 += z1;
                    }
                }
                CSum<T> ua = corner_sum<true, SP, T>(a0, a1, s, F);
                CSum<T> ub = corner_sum<true, SP, T>(b0, b1, s, F);
                const int row = FY + ky;  // relative to the current row
                if (near) {
                    auto put = [&](CSum<T>(&uu)[NS], int& has, auto row_id) {
                        has |= 3 << C | (REST ? 1 : 0);
                        static_for<NS - 1>([&](auto c) {
                            if (C != c) return;
                            cadd<true, SP>(uu[c], ua);
                            cadd<true, SP>(uu[c + 1], ub);
                            keep_apart<c>();
                        });
                        if constexpr (REST) {
                            if (C > 0) cadd<true, SP>(uu[0], corner_sum<true, SP, T>(z0, z1, s, F));
                        }
                        keep_apart<row_id>();
                    };
                    if (row == -1) put(u[0], has0, std::integral_constant<int, 0>{});
                    if (row == 0) put(u[1], has1, std::integral_constant<int, 1>{});
                    if (row == 1) put(u[2], has2, std::integral_constant<int, 2>{});
                } else if constexpr (FAR) {
                    // add d to row (current) + o, and the lane momentum g
                    auto fadd = [&](int o, const Dest<T>& d) { far_add(far, own, far_row(r, o), col, d); };
                    auto gadd = [&](int o, T g) { far_add_lane(far, own, far_row(r, o), col, (double)g); };
                    Dest<T> t;
                    t.zero();
                    if (C == 0) add_here<true, SP>(t, ua);
                    if constexpr (REST) {
                        if (C > 0) add_here<true, SP>(t, corner_sum<true, SP, T>(z0, z1, s, F));
                    }
                    auto far_speed = [&](int c, CSum<T> q) {
                        const T cc = (T)c;
                        q.e = fmaT((T)0.5 * cc * cc, q.m, q.e);
                        CSum<T> a = q, b = q;
#pragma unroll 1
                        for (int i = 0; i < c; ++i) {
                            a = cshr<true, SP>(a);
                            b = cshl<true, SP>(b);
                        }
                        t.m += a.m + b.m;
                        t.p += fmaT(cc, a.m - b.m, a.v + b.v);
                        t.e += fmaT(cc, a.v - b.v, a.e + b.e);
                        t.w += a.w + b.w;
                        if constexpr (SP) t.x += a.x + b.x;
                        Dest<T> d;
                        d.zero();
                        add_ylane<true, SP>(d, q, cc);
                        fadd(row + c, d);
                        gadd(row + c, cc * q.m);
                        d.zero();
                        add_ylane<true, SP>(d, q, -cc);
                        fadd(row - c, d);
                        gadd(row - c, -(cc * q.m));
                    };
                    if (C > 0) far_speed(C, ua);
                    far_speed(C + 1, ub);
                    fadd(row, t);
                }
            }
        }

        // stage B of row (current) - 1, whose corner sums are complete
        if constexpr (FIFO) asm volatile("" ::: "memory");
        Dest<T> t;
        t.zero();
        if (has0 & 1) add_here<true, SP>(t, u[0][0]);
        static_for<LB>([&](auto cm) {
            constexpr int c = cm + 1;
            CSum<T>& q = u[0][c];
            if constexpr (FIFO) hist.set(c, q.m);
            else hist.h[c][0] = q.m;
            if (!(has0 >> c & 1)) return;
            q.e = fmaT((T)(0.5 * c * c), q.m, q.e);
            add_xlanes<c, true, SP>(t, q);
            if constexpr (!FIFO) {
                add_ylane<true, SP>(f[LB - c], q, (T)-c);
                add_ylane<true, SP>(f[LB + c], q, (T)c);
            }
        });
        Dest<T> o;
        const auto add_t = [&](Dest<T>& d) {
            d.m += t.m;
            d.p += t.p;
            d.w += t.w;
            d.e += t.e;
            if constexpr (SP) d.x += t.x;
        };
        if constexpr (FIFO) {  // row by row, each one place on
            static_for<NSL>([&](auto j) {
                constexpr int c = j < LB ? LB - j : j - LB;
                Dest<T> q;
                q.zero();
                if constexpr (j < 2 * LB) {
                    const double* const p = &st.near.fifo[j * ND][lane];
                    q.m = p[0], q.p = p[64], q.w = p[128], q.e = p[192];
                    if constexpr (SP) q.x = p[256];
                }
                if constexpr (c == 0) add_t(q);
                else if (has0 >> c & 1) add_ylane<true, SP>(q, u[0][c], (T)(j < LB ? -c : c));
                if constexpr (j == 0) {
                    o = q;
                } else {
                    double* const p = &st.near.fifo[(j - 1) * ND][lane];
                    p[0] = q.m, p[64] = q.p, p[128] = q.w, p[192] = q.e;
                    if constexpr (SP) p[256] = q.x;
                }
            });
        } else {
            add_t(f[LB]);
            o = f[0];
        }
        // row (current) - 1 - LB has all it gets from near classes
        if constexpr (VY) o.w = (T)((double)o.w + hist.lane_py());
        hist.shift();
        if constexpr (FIFO) asm volatile("" ::: "memory");
        static_for<NS>([&](auto c) {
            u[0][c] = u[1][c];
            u[1][c] = u[2][c];
            u[2][c].zero();
        });
        has0 = has1;
        has1 = has2;
        has2 = 0;

        // row (current) - LD is complete
        const int64_t d = Y0 - kMH + r - LD;
        if constexpr (FAR) {
            far_add(far, own, far_row(r, -1 - LB), col, o);
            const int j = far_row(r, -kMH);
            o = far_get(far, own, j, col);
            if constexpr (VY) {
                double h, l;
                far_get_lane(far, own, j, col, h, l);
                o.w = (T)((double)o.w + (h + l));
            }
            far_zero(far, own, j, col);
        }
        if (d >= Y0 && d < ylast && io.dest) {
            io.template store<FIELDS>(d, o.m, o.p, o.w, o.e, o.x);
            tot[0] += (double)o.m;
            tot[1] += (double)o.p;
            tot[2] += (double)o.w;
            tot[3] += (double)o.e;
            if constexpr (SP) tot[NF - 1] += (double)o.x;
        }
        if constexpr (!FIFO) {
            static_for<NSL - 1>([&](auto j) { f[j] = f[j + 1]; });
            f[NSL - 1].zero();
        }
    }
    march_partials<NF, FIELDS>(tot, reach, anybad, prow, lane);
    *unlean = notlean;
    return true;
}

// Either form of the general pass on rows [Y0, ylast) of a tile.
template <typename T, bool REST, bool SP>
__device__ __forceinline__ bool march_rows_general(const MarchIO<T, SP ? 5 : 4>& io, const Consts& k, int64_t Y0,
                                                   int64_t ylast, double* __restrict__ prow, MarchStash<T, REST, SP>& st)
{
    using S = MarchStash<T, REST, SP>;
    bool unlean = false;
    if (!march_tile_general<T, REST, SP, false, kAllFields>(io, k, Y0, ylast, prow, st, &unlean)) {
        march_tile_general<T, REST, SP, true, S::F1>(io, k, Y0, ylast, prow, st, &unlean);
        if constexpr (S::F2 != 0) march_tile_general<T, REST, SP, true, S::F2>(io, k, Y0, ylast, prow, st, &unlean);
    }
    return unlean;
}

// Whether the general pass must compute the tile of destination rows [Y0,
// ylast) whose row chunk Y0 / sy has flag index tbase + (Y0 / sy) tiles_x + tx,
// after a lean pass that staged LB rows on each side of its tiles and wrote
// flags (1: given up).  A source up to H rows away can reach the tile: the rows [Y0
// - H, Y0 - LB) and [ylast + LB, ylast + H), mapped by the y boundary, belong
// to other row chunks (or the same one).  A source there that reaches the
// tile is beyond the lean pass (its packets move more than LB rows), so the
// chunk owning its row was given up: a periodic or clamped halo row is the
// very source it stands for, and a mirror image beyond a wall reaches inside
// only with packets whose mirror images, from the node inside, reach as far
// out (zero-mass corners aside, which add nothing).
template <int LB>
__device__ __forceinline__ bool needs_general(const int* __restrict__ flags, int64_t tbase, int64_t tiles_x,
                                              int64_t tx, int64_t Y0, int64_t ylast, int sy, int64_t ny, int bc_y)
{
    if (flags[tbase + (Y0 / sy) * tiles_x + tx]) return true;
#pragma unroll 1
    for (int i = 0; i < 2 * (kMH - LB); ++i) {
        const int d = i % (kMH - LB);
        const int64_t row = i < kMH - LB ? Y0 - kMH + d : ylast + LB + d;
        bool mir = false;
        const int64_t src = source_idx(row, ny, bc_y, &mir);
        if (flags[tbase + (src / sy) * tiles_x + tx]) return true;
    }
    return false;
}

// Wavefronts per SIMD the kernels are compiled for: as many as leave the row loop
// (nearly) free of spills, since a reload from scratch memory waits for the
// moments prefetched before it.  Lean: FP64 four, whose FIFO, history and corner
// sums need about 110 registers; two gases three; with a rest level two (4096^2
// planar nodes 391 us per step, with three and 27 spilled registers 787; both 463,
// with three and 126 spilled 2650).  FP32 five; two gases or a rest level four,
// both three (226 and 288 us, with five 277 and 1157).  General: two, in FP64 with
// both a rest level and two gases one (391 registers; with two 139 of them are
// spilled, and 2048^2 four-state nodes take 718 us per step instead of 447).
template <typename T, bool REST, bool SP>
constexpr int kLeanWpe = sizeof(T) == 8 ? (REST ? 2 : (SP ? 3 : 4)) : (REST && SP ? 3 : (REST || SP ? 4 : 5));
template <typename T, bool REST, bool SP>
constexpr int kGeneralWpe = sizeof(T) == 8 && REST && SP ? 1 : 2;

// Counters of StepCtl::next / PoolView::next: tile claims of the two passes;
// pools: non-zero when the lean pass gave a tile up.
enum { kNextLean = 0, kNextGeneral = 1, kNextGiven = 2 };

// Index of block b among nb, with the blocks of one XCD (the hardware deals blocks
// out to the 8 XCDs in turn) on neighbouring tiles, whose halo columns and rows are
// then in that XCD's L2.
__device__ __forceinline__ int march_block(int b, int nb)
{
    return (nb & 7) == 0 ? (b & 7) * (nb >> 3) + (b >> 3) : b;
}
// This wavefront's index among those of the launch, or of its first nb blocks (the
// test for these in the lean pass's one cost it 1 % in FP32).
__device__ __forceinline__ int march_wave()
{
    return __builtin_amdgcn_readfirstlane(march_block(blockIdx.x, gridDim.x) * kMNW + (int)(threadIdx.x >> 6));
}
__device__ __forceinline__ int march_wave(int nb)
{
    const int b = blockIdx.x;
    return __builtin_amdgcn_readfirstlane((b < nb ? march_block(b, nb) : b) * kMNW + (int)(threadIdx.x >> 6));
}
// As many of the launch's blocks as njobs jobs need, over all XCDs (the jobs of a
// small grid would else all fall to the blocks of one or two: us per step without /
// with it, four states on 200^2 nodes FP64 81 / 75, rest level 83 / 73; pools of 6
// planar tubes of 300 x 200 64 / 43).
__device__ __forceinline__ int march_blocks(int64_t njobs)
{
    return (int)min((int64_t)gridDim.x, (njobs + 8 * kMNW - 1) / (8 * kMNW) * 8);
}
// The wavefront's next tile: its first is its own index, later ones come from
// the counter (a slow tile delays only the wavefront that holds it).
__device__ __forceinline__ int march_claim(int* counter)
{
    int t = 0;
    if ((threadIdx.x & 63) == 0) t = (int)(gridDim.x * kMNW) + atomicAdd(counter, 1);
    return __builtin_amdgcn_readfirstlane(t);
}

// The lean pass (first of a step): wavefronts take the tiles (tiles_x column
// strips x row chunks of sy rows, row chunk major).  flags[t] tells whether a
// tile was given up; keep[t] (nullptr: none) holds, from the previous step's
// general pass, that it will be: such a tile is given up at once.
template <typename T, bool REST, bool SP>
__global__ void __launch_bounds__(kMTPB)
    __attribute__((amdgpu_waves_per_eu(kLeanWpe<T, REST, SP>)))
march2d_lean_kernel(const T* __restrict__ Y, T* __restrict__ Yn, Grid g, Consts k, StepCtl* __restrict__ ctl,
                    double* __restrict__ partials, MarchWords w, long long step, int sy, int tiles_x, int ntiles)
{
    if (ctl->err_step < step) return;
    const int lane = threadIdx.x & 63;
    const int nwaves = gridDim.x * kMNW;
    for (int t = march_wave(); t < ntiles;) {
        bool done = false;
        if (!(w.keep && w.keep[t])) {
            const int64_t tx = t % tiles_x, ty = t / tiles_x;
            MarchIO<T, SP ? 5 : 4> io;
            io.set(Y, Yn, g, tx * kMCols, lane);
            const int64_t Y0 = ty * sy, ylast = min(Y0 + sy, g.ny);
            done = march_tile_lean<T, REST, SP>(io, k, Y0, ylast, partials + (int64_t)t * kPartialStride);
        }
        if (lane == 0) {
            w.flags[t] = done ? 0 : 1;
            w.nch[t] = 1;
            if (!done) {
                if (w.keep) w.keep[t] = 0;  // set again by the general pass if it still holds
                atomicAdd(&ctl->given_up[(t & (kGivenUp - 1)) * kGivenUpStride], 1);
            }
        }
        t = ntiles > nwaves ? march_claim(&ctl->next[kNextLean]) : ntiles;
    }
}

// The general pass: the tiles the lean pass gave up and their row-chunk
// neighbours (needs_general).  When few were given up, each is cut into row
// chunks (at most smax, of at least kChunkRows rows) so that every wavefront
// has about one: a tile's wavefront would otherwise hold the pass up for its
// whole march.  Chunk p of tile t writes the row p ntiles + t of partials.  A
// node's value does not depend on the cut.
constexpr int kChunkRows = 8;
template <typename T, bool REST, bool SP>
__global__ void __launch_bounds__(kMTPB) __attribute__((amdgpu_waves_per_eu(kGeneralWpe<T, REST, SP>)))
march2d_general_kernel(const T* __restrict__ Y, T* __restrict__ Yn, Grid g, Consts k, StepCtl* __restrict__ ctl,
                       double* __restrict__ partials, MarchWords w, long long step, int sy, int tiles_x, int ntiles)
{
    __shared__ MarchStash<T, REST, SP> stash[kMNW];
    if (ctl->err_step < step) return;
    const int lane = threadIdx.x & 63;
    // (in a scalar register, and with it every job's rows and columns: 2048^2 four-state
    // nodes 264 -> 237 us per step in FP64, 226 -> 185 in FP32)
    const int given = __builtin_amdgcn_readfirstlane(wave_sum(lane < kGivenUp ? ctl->given_up[lane * kGivenUpStride] : 0));
    if (given == 0) return;
    const int nwaves = gridDim.x * kMNW;
    const int want = max(1, min(w.smax, nwaves / given));
    const int h = max(kChunkRows, (sy + want - 1) / want);
    const int ns = (sy + h - 1) / h;
    const int64_t njobs = (int64_t)ntiles * ns;
    for (int64_t j = march_wave(march_blocks(njobs)); j < njobs;) {
        // (chunks of one tile on neighbouring wavefronts)
        const int t = (int)(j / ns), p = (int)(j % ns);
        const int64_t tx = t % tiles_x, ty = t / tiles_x;
        const int64_t Y0 = ty * sy, ylast = min(Y0 + sy, g.ny);
        const int64_t c0 = Y0 + (int64_t)p * h, c1 = min(c0 + h, ylast);
        if (c0 < ylast && needs_general<kSpeeds<REST> - 1>(w.flags, 0, tiles_x, tx, Y0, ylast, sy, g.ny, g.bc_y)) {
            MarchIO<T, SP ? 5 : 4> io;
            io.set(Y, Yn, g, tx * kMCols, lane);
            const bool unlean = march_rows_general<T, REST, SP>(
                io, k, c0, c1, partials + ((int64_t)p * ntiles + t) * kPartialStride, stash[threadIdx.x >> 6]);
            if (lane == 0) {
                if (unlean && w.keep) w.keep[t] = 1;
                if (p == 0) w.nch[t] = (int)((ylast - Y0 + h - 1) / h);
            }
        }
        if (ns > 1) j += nwaves;
        else j = njobs > nwaves ? march_claim(&ctl->next[kNextGeneral]) : njobs;
    }
}

// Pool form of the two passes: wavefronts take the tiles of the tile table
// (PoolTile); a slot's tiles are its row chunks, then column strips,
// from its t0, which is how needs_general finds a tile's neighbours.
template <typename T, bool REST, bool SP>
__global__ void __launch_bounds__(kMTPB)
    __attribute__((amdgpu_waves_per_eu(kLeanWpe<T, REST, SP>)))
pool2d_lean_kernel(PoolView v, Consts k)
{
    const int nt = *v.ntiles, lane = threadIdx.x & 63, nwaves = gridDim.x * kMNW;
    T* arena = (T*)v.arena;
    for (int t = march_wave(march_blocks(nt)); t < nt;) {
        const int ts = v.tstate[t];
        if (ts & kTileLive) {
            bool done = false;
            if (!v.flags[t]) {  // the general pass found it beyond this pass last step
                const PoolTile& tl = v.tiles[t];
                const int64_t o0 = tl.off[0], o1 = tl.off[1];
                const int64_t from = (ts & kTileSet) ? o1 : o0, to = (ts & kTileSet) ? o0 : o1;
                const Grid g{tl.nx, tl.ny, tl.bc_x, tl.bc_y};
                const int64_t Y0 = tl.y0, ylast = min(Y0 + (int64_t)tl.rows, g.ny);
                MarchIO<T, SP ? 5 : 4> io;
                io.set(arena + from, arena + to, g, tl.x0, lane);
                done = march_tile_lean<T, REST, SP>(io, k, Y0, ylast, v.partials + (int64_t)t * kPartialStride);
            }
            if (lane == 0) {
                v.flags_lean[t] = done ? 0 : 1;
                if (!done) {
                    v.flags[t] = 0;  // set again by the general pass if it still holds
                    if (v.next[kNextGiven] == 0) atomicAdd(&v.next[kNextGiven], 1);
                }
            }
        }
        t = nt > nwaves ? march_claim(&v.next[kNextLean]) : nt;
    }
}

template <typename T, bool REST, bool SP>
__global__ void __launch_bounds__(kMTPB) __attribute__((amdgpu_waves_per_eu(kGeneralWpe<T, REST, SP>)))
pool2d_general_kernel(PoolView v, Consts k)
{
    __shared__ MarchStash<T, REST, SP> stash[kMNW];
    if (v.next[kNextGiven] == 0) return;  // nothing left to it
    const int nt = *v.ntiles, lane = threadIdx.x & 63, nwaves = gridDim.x * kMNW;
    T* arena = (T*)v.arena;
    for (int t = march_wave(march_blocks(nt)); t < nt;) {
        const int ts = v.tstate[t];
        if (ts & kTileLive) {
            const PoolTile& tl = v.tiles[t];
            const int64_t tiles_x = (tl.nx + kMCols - 1) / kMCols;
            const int64_t tbase = v.probs[tl.prob].t0, tx = tl.x0 / kMCols;
            const int64_t ylast = min(tl.y0 + (int64_t)tl.rows, tl.ny);
            if (needs_general<kSpeeds<REST> - 1>(v.flags_lean, tbase, tiles_x, tx, tl.y0, ylast, tl.rows, tl.ny,
                                                 tl.bc_y)) {
                const int64_t o0 = tl.off[0], o1 = tl.off[1];
                const int64_t from = (ts & kTileSet) ? o1 : o0, to = (ts & kTileSet) ? o0 : o1;
                const Grid g{tl.nx, tl.ny, tl.bc_x, tl.bc_y};
                MarchIO<T, SP ? 5 : 4> io;
                io.set(arena + from, arena + to, g, tl.x0, lane);
                const bool unlean = march_rows_general<T, REST, SP>(
                    io, k, tl.y0, ylast, v.partials + (int64_t)t * kPartialStride, stash[threadIdx.x >> 6]);
                if (lane == 0 && unlean) v.flags[t] = 1;
            }
        }
        t = nt > nwaves ? march_claim(&v.next[kNextGeneral]) : nt;
    }
}

// The integer decisions of every node, as the passes take them: rows of 64 nodes
// without v_y by the lean pass's form, others by the general one (bad states: 0).
template <typename T, bool REST, bool SP>
__global__ void __launch_bounds__(kMTPB)
march_lanes_kernel(const T* __restrict__ Y, int64_t nn, Consts k, int32_t* __restrict__ fx, int32_t* __restrict__ fy,
                   int32_t* __restrict__ c1)
{
    const int64_t q = (int64_t)blockIdx.x * kMTPB + threadIdx.x, p = min(q, nn - 1);
    const T r0 = Y[p], r1 = Y[nn + p], r2 = Y[2 * nn + p], r3 = Y[3 * nn + p], r4 = SP ? Y[(SP ? 4 : 0) * nn + p] : (T)0;
    bool ok = tame(r0, r1, r2, r3) && (!REST || k.delta0 <= kTameDelta0);
    bool bad = !((double)r0 > 0.0) || !isfinite(r0) || !isfinite(r1) || !isfinite(r2) || !isfinite(r3);
    if constexpr (SP) {
        ok = ok && zero_or_normal(r4);
        bad = bad || !isfinite(r4);
    }
    const bool tame_all = __all(ok), lean = __all(r2 == (T)0 && !bad);
    MNode<T, REST, SP> s;
    if (lean) s = tame_all ? march_node<T, REST, SP, true, false>(r0, r1, 0.0, r3, r4, k, false)
                           : march_node<T, REST, SP, true, true>(r0, r1, 0.0, r3, r4, k, false);
    else s = tame_all ? march_node<T, REST, SP, false, false>(r0, r1, r2, r3, r4, k, false)
                      : march_node<T, REST, SP, false, true>(r0, r1, r2, r3, r4, k, bad);
    if (q >= nn) return;
    fx[q] = bad ? 0 : s.fx;
    fy[q] = bad ? 0 : s.fy;
    c1[q] = bad ? 0 : s.c1;
}
template <typename T, bool REST, bool SP>
hipError_t launch_lanes_w(const T* Y, const Grid& g, const Consts& k, int32_t* fx, int32_t* fy, int32_t* c1,
                          hipStream_t stream)
{
    const int64_t nn = g.nx * g.ny;
    march_lanes_kernel<T, REST, SP><<<(unsigned)((nn + kMTPB - 1) / kMTPB), kMTPB, 0, stream>>>(Y, nn, k, fx, fy, c1);
    return hipGetLastError();
}

// The two passes of one step.
template <typename T, bool REST, bool SP>
hipError_t launch_march2d_w(const T* Y, T* Yn, const Grid& g, const MarchGeom& m, const Consts& k,
                            StepCtl* ctl, double* partials, const MarchWords& w, long long step, hipStream_t stream)
{
    const int nt = (int)m.blocks();
    march2d_lean_kernel<T, REST, SP><<<m.nblocks_lean, kMTPB, 0, stream>>>(Y, Yn, g, k, ctl, partials, w, step, m.sy,
                                                                           (int)m.grid_x, nt);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    march2d_general_kernel<T, REST, SP><<<m.nblocks, kMTPB, 0, stream>>>(Y, Yn, g, k, ctl, partials, w, step, m.sy,
                                                                         (int)m.grid_x, nt);
    return hipGetLastError();
}

// Resident blocks per CU of one instance's lean or general pass.
template <typename T, bool REST, bool SP, bool POOL>
int march_resident(bool lean)
{
    int nb = 0;
    hipError_t e;
    if constexpr (POOL)
        e = lean ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, pool2d_lean_kernel<T, REST, SP>, kMTPB, 0)
                 : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, pool2d_general_kernel<T, REST, SP>, kMTPB, 0);
    else
        e = lean ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, march2d_lean_kernel<T, REST, SP>, kMTPB, 0)
                 : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, march2d_general_kernel<T, REST, SP>, kMTPB, 0);
    return e == hipSuccess && nb > 0 ? nb : 1;
}

// The two passes of one pool step.
template <typename T, bool REST, bool SP>
hipError_t launch_pool2d_w(const PoolView& v, const Consts& k, int nblocks_lean, int nblocks, hipStream_t stream)
{
    pool2d_lean_kernel<T, REST, SP><<<nblocks_lean, kMTPB, 0, stream>>>(v, k);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    pool2d_general_kernel<T, REST, SP><<<nblocks, kMTPB, 0, stream>>>(v, k);
    return hipGetLastError();
}

}  // namespace

// Two gases (lb_march2d_sp.hip, lb_pool2d_sp.hip): the instances with the
// species field.
template <typename T>
int march2d_blocks_per_cu_species(bool lean, bool rest);
template <typename T>
int pool2d_blocks_per_cu_species(bool lean, bool rest);
template <typename T>
hipError_t launch_march2d_species(const T* Y, T* Yn, const Grid& g, const MarchGeom& m, const Consts& k,
                                  StepCtl* ctl, double* partials, const MarchWords& w, long long step,
                                  hipStream_t stream);
template <typename T>
hipError_t launch_lanes_species(const T* Y, const Grid& g, const Consts& k, int32_t* fx, int32_t* fy, int32_t* c1,
                                hipStream_t stream);
template <typename T>
hipError_t launch_pool2d_species(const PoolView& v, const Consts& k, int nblocks_lean, int nblocks,
                                 hipStream_t stream);

}  // namespace lbsd
