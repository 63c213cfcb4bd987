#pragma once
// The 1-D step (triple-level set) on a wavefront's registers, several steps per
// launch (Sec. III-V of Komeili, Mirzaei, Shabouei, arXiv 1602.02675; tau = 1).
//
// As on the square lattice (lb_march2d.hpp) the migration (FP64) factors into the
// corner sums of each speed, U_c(x) = sum of m (1, v, K) over the sources and
// corners landing on x with one lane of speed c, and the lanes: the new moments
// of x are U_0(x) (rest level, and both lanes of c'_1 = 0) plus those of U_c
// at x -+ c for the lanes +-c, with momentum V +- c M and energy E +- c V + c^2/2 M.
//
// A lane holds J consecutive nodes in registers, a wavefront 64 J; a shift by one
// node is a change of register names and one lane shift.  No packet moves
// further than H = 5 nodes a step, so after every step ceil(5 / J) lanes more on
// each side have lost what they needed: a wavefront that starts with K times as
// many halo lanes on each side makes K steps before it touches memory again, and
// stores the nodes in the middle.  Long tubes take J = 5, where a step costs
// exactly one halo lane: one step per launch is bound by HBM (48 bytes per node
// and step in FP64), from K = 3 or so on by VALU issue.  Short tubes take J = 2,
// whose steps are the shortest: with most of the chip idle a launch lasts as
// long as one wavefront's K steps.
//
// Sources that share floor(v) and c'_1 form a class.  A wavefront of one class
// takes it without a test per node; otherwise the values of floor(v), and for
// each the speeds, are taken one after another, the nodes without them with zero
// mass, so that a node's value does not depend on the
// wavefront, the number of steps per launch or the halo it was computed with.
#include "lb_wave.hpp"

namespace lbsd {

namespace {

// Parts of a step that the scheduler must not interleave: with all J nodes' or
// all speeds' temporaries alive at once the kernel spills.
template <int J>
__device__ __forceinline__ void step_apart()
{
    if constexpr (J > 2) __builtin_amdgcn_sched_barrier(0);
}

// Constants of the primitives formed once per kernel.
struct TubeConsts {
    double cA;    // A / e: D (gamma - 1) / (1 - delta0) (two gases: 1 / (1 - delta0))
    double near;  // relative distance from a switch of c'_1 within which A is formed as eq. 26 prints it
};
__device__ __forceinline__ TubeConsts tube_consts(const Consts& k, bool sp)
{
    const double rest = 1.0 - k.b0 * k.delta0;
    return TubeConsts{(sp ? 1.0 : k.Dg1) / rest, 1e-14 + 1e-14 / rest};
}

// What a class's packets are formed from: v, A (eq. 26), K and the density of
// a lane's J nodes (0 for a bad state, which then emits nothing).
template <typename T, bool SP, int J>
struct TubeNodes {
    double v[J], A[J];
    T rho[J], K[J];
    T chi[SP ? J : 1];
};

// Per-node primitives (eq. 15, 26) in FP64 whatever the storage type, as on the
// square lattice (march_node).  IEEE: any operands, bad states included; otherwise
// the operands are tame.  A = e D (gamma - 1) / (1 - delta0) takes one product instead of the
// quotient by rho - d_0; the two differ by rounding alone, so they agree on c'_1
// except next to a switch, where (FP64, whose c'_1 matches the plain definition
// bit for bit) a node takes the quotient after all.
template <bool IEEE, typename T, bool SP, int J>
__device__ __forceinline__ void tube_node(TubeNodes<T, SP, J>& n, int j, T r0, double m1, double m2, double m3,
                                          const Consts& kc, const TubeConsts& tc, bool bad)
{
#pragma clang fp contract(off)
    constexpr bool FAST = sizeof(T) < 8;
    double m0 = r0;
    if constexpr (IEEE) {
        m0 = bad ? 1.0 : m0;
        m1 = bad ? 0.0 : m1;
        m2 = bad ? 0.0 : m2;
        m3 = bad ? 0.0 : m3;
        r0 = bad ? (T)0 : r0;
    }
    const Quot<FAST, IEEE> by_rho(m0);
    double Dg1 = kc.Dg1, phi = kc.phi_coef, cA = tc.cA;
    if constexpr (SP) {
        double chi = by_rho(m3);
        chi = chi < 0.0 ? 0.0 : (chi > 1.0 ? 1.0 : chi);
        const double gm1 = pdiv<FAST>(1.0, pdiv<FAST>(chi, kc.g1m1) + pdiv<FAST>(1.0 - chi, kc.g2m1));
        Dg1 = 1.0 * gm1;
        phi = 1.0 - 0.5 * gm1;
        cA = gm1 * tc.cA;
        n.chi[j] = (T)chi;
    }
    const double v = by_rho(m1), E = by_rho(m2), v2 = v * v;
    double e = E - 0.5 * v2;
    if (e < 0.0) e = 0.0;
    double A = e * cA;
    if constexpr (!FAST) {
        bool near = fabs(A - 1.0) < tc.near || fabs(A - 4.0) < 4.0 * tc.near || A > 8.0;
        if constexpr (IEEE) near = near || m0 < 1e-290;  // (rho - d_0 is short of bits there)
        if (__any(near)) A = near ? Dg1 * e * m0 / (m0 - kc.b0 * (kc.delta0 * m0)) : A;
    }
    if constexpr (IEEE) {
        if (!(A >= 0.0)) A = 0.0;
        if (A > (double)kMaxC1 * (double)kMaxC1) A = (double)kMaxC1 * (double)kMaxC1;
    }
    n.v[j] = v;
    n.A[j] = A;
    n.rho[j] = r0;
    n.K[j] = (T)__builtin_fma(phi, e, 0.5 * v2);
}

// c'_1 (eq. 26): exact comparisons for the usual values, the integer root elsewhere.
__device__ __forceinline__ int tube_c1(double A)
{
    if (__any(A >= 9.0)) return isqrt_floor<double>(A);
    return (A >= 1.0 ? 1 : 0) + (A >= 4.0 ? 1 : 0);
}
// Class of a node: floor(v) + 32 and c'_1, clamped far beyond any admissible reach.
__device__ __forceinline__ int tube_key(double v, double A)
{
    return (min(max((int)floor(v), -32), 31) + 32) << 5 | min(tube_c1(A), 31);
}

// Whether all of a lane's nodes are tame (see tame()).
template <bool SP, typename T, int J, int NF>
__device__ __forceinline__ bool tube_tame(const T (&y)[NF][J])
{
    bool ok = true;
    if constexpr (sizeof(T) == 8) {
        const auto hi = [](double v) { return (uint32_t)(__builtin_bit_cast(uint64_t, v) >> 32); };
        uint32_t lo = 0xffffffffu, up = 0;
        static_for<J>([&](auto j) {
            lo = min(lo, min(hi(y[0][j]), hi(y[2][j])));
            up = max(up, max(hi(y[0][j]), hi(y[2][j])));
            ok = ok && zero_or_normal(y[1][j]);
        });
        ok = ok && lo >= 0x30000000u && up < 0x50000000u;
    } else {
        static_for<J>([&](auto j) { ok = ok && tame(y[0][j], y[1][j], (T)0, y[2][j]); });
    }
    if constexpr (SP) static_for<J>([&](auto j) { ok = ok && zero_or_normal(y[NF - 1][j]); });
    return ok;
}

// rho <= 0 or a non-finite moment.
template <bool SP, typename T, int J, int NF>
__device__ __forceinline__ bool tube_bad(const T (&y)[NF][J], int j)
{
    bool bad = !((double)y[0][j] > 0.0) || !isfinite(y[0][j]) || !isfinite(y[1][j]) || !isfinite(y[2][j]);
    if constexpr (SP) bad = bad || !isfinite(y[NF - 1][j]);
    return bad;
}

// Shifts of a wavefront's 64 J values by N nodes up (node x gets node x - N's
// value) and down.
template <int N, typename T, int J>
__device__ __forceinline__ void node_up(const T (&a)[J], T (&o)[J])
{
    if constexpr (N > J) {
        T s[J];
        node_up<J>(a, s);
        node_up<N - J>(s, o);
    } else {
        static_for<J>([&](auto j) {
            if constexpr (j >= N) o[j] = a[j - N];
            else o[j] = lshr(a[J - N + j]);
        });
    }
}
template <int N, typename T, int J>
__device__ __forceinline__ void node_down(const T (&a)[J], T (&o)[J])
{
    if constexpr (N > J) {
        T s[J];
        node_down<J>(a, s);
        node_down<N - J>(s, o);
    } else {
        static_for<J>([&](auto j) {
            if constexpr (j + N < J) o[j] = a[j + N];
            else o[j] = lshl(a[j + N - J]);
        });
    }
}

// Masses w0, w1 at the corners 0, 1 of sources with floor(v) = F (wave-uniform)
// and a payload per unit mass q, summed onto the nodes they land on.
template <bool UNIT, typename T, int J>
__device__ __forceinline__ void tube_corners(const T (&w0)[J], const T (&w1)[J], const T (&q)[J], int F, T (&o)[J])
{
#pragma clang fp contract(off)
    T p[J], s[J];
    if (F >= 0) {
        static_for<J>([&](auto j) { p[j] = UNIT ? w1[j] : w1[j] * q[j]; });
        node_up<1>(p, s);
        static_for<J>([&](auto j) { o[j] = UNIT ? w0[j] + s[j] : fmaT(w0[j], q[j], s[j]); });
#pragma unroll 1
        for (int i = 0; i < F; ++i) {
            node_up<1>(o, s);
            static_for<J>([&](auto j) { o[j] = s[j]; });
        }
    } else {
        static_for<J>([&](auto j) { p[j] = UNIT ? w0[j] : w0[j] * q[j]; });
        node_down<1>(p, s);
        static_for<J>([&](auto j) { o[j] = UNIT ? w1[j] + s[j] : fmaT(w1[j], q[j], s[j]); });
#pragma unroll 1
        for (int i = F; i < -1; ++i) {
            node_down<1>(o, s);
            static_for<J>([&](auto j) { o[j] = s[j]; });
        }
    }
}

// One speed C of a class, masses d per lane of the speed (corner fractions
// 1 - r, r): its corner sums, moved along its lanes, added to the new moments t
// (rho, rho v, rho E, rho chi).  C = 0: d stands for all packets that stay where
// the corners put them.  SET: t starts here.
template <int C, bool SET, bool SP, typename T, int J, int NF>
__device__ __forceinline__ void tube_speed(const double (&d)[J], const double (&r)[J], const T (&v)[J],
                                           const TubeNodes<T, SP, J>& n, int F, T (&t)[NF][J])
{
#pragma clang fp contract(off)
    T w0[J], w1[J], M[J], V[J], E[J];
    static_for<J>([&](auto j) {
        w0[j] = (T)(d[j] * (1.0 - r[j]));
        w1[j] = (T)(d[j] * r[j]);
    });
    const auto put = [&](T& o, T x) { o = SET ? x : o + x; };
    tube_corners<true>(w0, w1, v, F, M);
    step_apart<J>();
    tube_corners<false>(w0, w1, v, F, V);
    step_apart<J>();
    tube_corners<false>(w0, w1, n.K, F, E);
    step_apart<J>();
    if constexpr (C == 0) {
        static_for<J>([&](auto j) {
            put(t[0][j], M[j]);
            put(t[1][j], V[j]);
            put(t[2][j], E[j]);
        });
    } else {
        T ms[J];
        T u[J], w[J], vu[J], vd[J];
        node_up<C>(M, u);
        node_down<C>(M, w);
        static_for<J>([&](auto j) {
            const T sm = u[j] + w[j];
            put(t[0][j], sm);
            u[j] -= w[j];
            ms[j] = sm;
        });
        step_apart<J>();
        node_up<C>(V, vu);
        node_down<C>(V, vd);
        static_for<J>([&](auto j) {
            put(t[1][j], fmaT((T)C, u[j], vu[j] + vd[j]));
            vu[j] -= vd[j];
        });
        step_apart<J>();
        node_up<C>(E, u);
        node_down<C>(E, w);
        static_for<J>([&](auto j) { put(t[2][j], fmaT((T)(0.5 * C * C), ms[j], fmaT((T)C, vu[j], u[j] + w[j]))); });
    }
    step_apart<J>();
    if constexpr (SP) {
        tube_corners<false>(w0, w1, n.chi, F, M);
        if constexpr (C == 0) {
            static_for<J>([&](auto j) { put(t[3][j], M[j]); });
        } else {
            T u[J], w[J];
            node_up<C>(M, u);
            node_down<C>(M, w);
            static_for<J>([&](auto j) { put(t[3][j], u[j] + w[j]); });
        }
    }
}

// The packets of a wavefront of one class (F, C).  r = v - F and g = A - C^2 of the
// nodes; the level weights (eq. 24-25 rewritten, see level_w) are formed here,
// where c'_1 is a constant.
template <int C, bool SP, typename T, int J, int NF>
__device__ __forceinline__ void tube_class(const TubeNodes<T, SP, J>& n, const double (&r)[J], const double (&g)[J],
                                           int F, const Consts& k, T (&t)[NF][J])
{
#pragma clang fp contract(off)
    constexpr double inv = C == 0 ? 1.0 : (C == 1 ? 1.0 / 3.0 : (C == 2 ? 1.0 / 5.0 : 1.0 / 7.0));
    double w[J], d[J];
    T v[J];
    static_for<J>([&](auto j) {
        w[j] = g[j] * inv;
        v[j] = (T)n.v[j];
    });
    // masses per lane of the levels: d_0 = delta0 rho, b_1 d_2 = (rho - b_0 d_0) w,
    // b_1 d_1 = (rho - b_0 d_0) (1 - w)
    const auto level = [&](int l, int j) {
        const double rho = (double)n.rho[j], d0 = k.delta0 * rho;
        if (l == 0 && C > 0) return d0;
        const double per = (rho - k.b0 * d0) * k.inv_b1, d2 = per * w[j];
        if (l == 2) return d2;
        if (l == 1) return per - d2;
        return __builtin_fma(2.0, per - d2, d0);  // both lanes of c'_1 = 0 stay too
    };
    static_for<J>([&](auto j) { d[j] = level(0, j); });
    tube_speed<0, true, SP>(d, r, v, n, F, t);
    if constexpr (C > 0) {
        static_for<J>([&](auto j) { d[j] = level(1, j); });
        tube_speed<C, false, SP>(d, r, v, n, F, t);
    }
    static_for<J>([&](auto j) { d[j] = level(2, j); });
    tube_speed<C + 1, false, SP>(d, r, v, n, F, t);
}

// The integer decisions of one node of each lane, as the step takes them (bad
// states: 0).
template <typename T, bool SP>
__device__ __forceinline__ void tube_decisions(const T (&y)[SP ? 4 : 3][1], const Consts& k, int* f, int* c1)
{
    constexpr int NF = SP ? 4 : 3;
    const TubeConsts tc = tube_consts(k, SP);
    TubeNodes<T, SP, 1> n;
    bool bad = false;
    if (__all(tube_tame<SP>(y) && k.delta0 <= kTameDelta0)) {
        tube_node<false>(n, 0, y[0][0], y[1][0], y[2][0], y[NF - 1][0], k, tc, false);
    } else {
        bad = tube_bad<SP>(y, 0);
        tube_node<true>(n, 0, y[0][0], y[1][0], y[2][0], y[NF - 1][0], k, tc, bad);
    }
    const int c = tube_c1(n.A[0]);
    *f = bad ? 0 : (int)floor(n.v[0]);
    *c1 = bad ? 0 : c;
}

// ---- FP32 ----
//
// FP32 fields are summed packet by packet in the order of the packet definition
// (corner 0, then 1; of each the rest level, +c'_1, -c'_1, +c'_2, -c'_2; of each
// the sources by ascending displacement).  Where the state is uniform every step
// rounds alike, so the rounding of a step's sums is a drift, not noise: behind a
// strong shock it moves the plateau by up to 1e-4 and the shock by some 1e-3 node
// in 400 steps.  Another order has another drift: with corner sums an FP32 tube
// differs at the front by up to 1.3e-3 from what packets in this order give.  30
// products and 30 sums a node: 256 tubes of 3.1 M nodes in all take 17.9 us per
// step with them, 16.5 with corner sums, and 45 where every step was a launch that
// rebuilt its packets from LDS.

// A lane's nodes as their packets are formed: rounded to FP32 from FP64
// primitives; key as tube_key.
template <bool SP, int J>
struct TubePackets {
    float rho[J], r[J], d2[J], K[J], chi[SP ? J : 1];
    int key[J];
};

template <int N, int J>
__device__ __forceinline__ void node_shift(const float (&a)[J], float (&o)[J])
{
    if constexpr (N > 0) node_up<N>(a, o);
    else if constexpr (N < 0) node_down<-N>(a, o);
    else static_for<J>([&](auto j) { o[j] = a[j]; });
}

// All sums F nodes on.
template <int J, int NF>
__device__ __forceinline__ void tube_shift(float (&o)[NF][J], int F)
{
#pragma unroll 1
    for (int i = 0; i < F; ++i)
        static_for<NF>([&](auto f) {
            float s[J];
            node_up<1>(o[f], s);
            static_for<J>([&](auto j) { o[f][j] = s[j]; });
        });
#pragma unroll 1
    for (int i = F; i < 0; ++i)
        static_for<NF>([&](auto f) {
            float s[J];
            node_down<1>(o[f], s);
            static_for<J>([&](auto j) { o[f][j] = s[j]; });
        });
}

// Sources of one class, floor(v) = F and c'_1 = C.
template <int C, bool SP, int J, int NF>
__device__ __forceinline__ void tube_packets(const TubePackets<SP, J>& n, int F, const Consts& k, float (&o)[NF][J])
{
#pragma clang fp contract(off)
    const float delta0 = (float)k.delta0, b0 = (float)k.b0, inv_b1 = (float)k.inv_b1;
    static_for<NF>([&](auto f) { static_for<J>([&](auto j) { o[f][j] = 0.0f; }); });
    static_for<2>([&](auto corner) {
        static_for<5>([&](auto l) {
            constexpr int lev = l == 0 ? 0 : (l <= 2 ? 1 : 2);
            constexpr int c = l == 0 ? 0 : ((l & 1) ? 1 : -1) * (C + lev - 1), N = corner + c;
            float m[J], p[J], s[J];
            static_for<J>([&](auto j) {
                const float d0 = delta0 * n.rho[j];
                const float d = lev == 0 ? d0 : (lev == 2 ? n.d2[j] : (n.rho[j] - b0 * d0) * inv_b1 - n.d2[j]);
                m[j] = (corner ? n.r[j] : 1.0f - n.r[j]) * d;
            });
            node_shift<N>(m, s);
            static_for<J>([&](auto j) {
                o[0][j] += s[j];
                p[j] = m[j] * (((float)F + n.r[j]) + (float)c);
            });
            node_shift<N>(p, s);
            static_for<J>([&](auto j) {
                o[1][j] += s[j];
                const float v = (float)F + n.r[j];
                p[j] = m[j] * (c == 0 ? n.K[j] : n.K[j] + (float)c * v + 0.5f * (float)c * (float)c);
            });
            node_shift<N>(p, s);
            static_for<J>([&](auto j) { o[2][j] += s[j]; });
            if constexpr (SP) {
                static_for<J>([&](auto j) { p[j] = m[j] * n.chi[j]; });
                node_shift<N>(p, s);
                static_for<J>([&](auto j) { o[3][j] += s[j]; });
            }
            step_apart<J>();
        });
    });
    tube_shift(o, F);
}

// Sources with floor(v) in {F, F + 1} and c'_1 in {C, C + 1}: per packet of the
// order above, the displacements in ascending order, the nodes of others with
// zero mass (what a node gets from sources of one class is what tube_packets
// gives it).
template <int C, bool SP, int J, int NF>
__device__ __forceinline__ void tube_packets_near(const TubePackets<SP, J>& n, int F, bool valid, const Consts& k,
                                                  float (&o)[NF][J])
{
#pragma clang fp contract(off)
    const float delta0 = (float)k.delta0, b0 = (float)k.b0, inv_b1 = (float)k.inv_b1;
    float v[J], a1[J];  // v; 1 if c'_1 = C + 1
    int sF[J], sC[J];
    static_for<J>([&](auto j) {
        // (a lane that does not count must not ask for a displacement beyond H)
        const int key = valid ? n.key[j] : (F + 32) << 5 | C, f = (key >> 5) - 32;
        v[j] = (float)f + n.r[j];
        sF[j] = f - F;
        sC[j] = (key & 31) - C;
        a1[j] = (float)sC[j];
    });
    static_for<NF>([&](auto f) { static_for<J>([&](auto j) { o[f][j] = 0.0f; }); });
    static_for<2>([&](auto corner) {
        static_for<5>([&](auto l) {
            constexpr int lev = l == 0 ? 0 : (l <= 2 ? 1 : 2), sg = l == 0 ? 0 : ((l & 1) ? 1 : -1);
            // displacement: base + e
            constexpr int base = corner + (sg > 0 ? C + lev - 1 : (sg < 0 ? -(C + lev) : 0));
            float m[J], xi[J], zeta[J];
            int e[J];
            static_for<J>([&](auto j) {
                const float d0 = delta0 * n.rho[j];
                const float d = lev == 0 ? d0 : (lev == 2 ? n.d2[j] : (n.rho[j] - b0 * d0) * inv_b1 - n.d2[j]);
                const float c = (float)sg * ((float)(C + lev - 1) + a1[j]);
                m[j] = (corner ? n.r[j] : 1.0f - n.r[j]) * d;
                xi[j] = sg == 0 ? v[j] : v[j] + c;
                zeta[j] = sg == 0 ? n.K[j] : n.K[j] + c * v[j] + 0.5f * c * c;
                e[j] = sF[j] + (sg > 0 ? sC[j] : (sg < 0 ? 1 - sC[j] : 0));
            });
            static_for<(sg == 0 ? 2 : 3)>([&](auto i) {
                constexpr int N = base + i;
                bool any = false;
                static_for<J>([&](auto j) { any = any || e[j] == i; });
                if (__any(any)) {
                    float w[J], p[J], s[J];
                    static_for<J>([&](auto j) { w[j] = e[j] == i ? m[j] : 0.0f; });
                    node_shift<N>(w, s);
                    static_for<J>([&](auto j) {
                        o[0][j] += s[j];
                        p[j] = w[j] * xi[j];
                    });
                    node_shift<N>(p, s);
                    static_for<J>([&](auto j) {
                        o[1][j] += s[j];
                        p[j] = w[j] * zeta[j];
                    });
                    node_shift<N>(p, s);
                    static_for<J>([&](auto j) { o[2][j] += s[j]; });
                    if constexpr (SP) {
                        static_for<J>([&](auto j) { p[j] = w[j] * n.chi[j]; });
                        node_shift<N>(p, s);
                        static_for<J>([&](auto j) { o[3][j] += s[j]; });
                    }
                }
            });
            step_apart<J>();
        });
    });
    tube_shift(o, F);
}

// Any classes within reach, likewise.
template <bool SP, int J, int NF>
__device__ __forceinline__ void tube_packets_mixed(const TubePackets<SP, J>& n, int Fmin, int Fmax, int Cmin, int Cmax,
                                                   const Consts& k, float (&o)[NF][J])
{
#pragma clang fp contract(off)
    const float delta0 = (float)k.delta0, b0 = (float)k.b0, inv_b1 = (float)k.inv_b1;
    static_for<NF>([&](auto f) { static_for<J>([&](auto j) { o[f][j] = 0.0f; }); });
#pragma unroll 1
    for (int i = 0; i < 10; ++i) {
        const int corner = i >= 5, l = i - 5 * corner, lev = (l + 1) >> 1, sg = l == 0 ? 0 : ((l & 1) ? 1 : -1);
        float q[NF][J];
        int D[J];
        static_for<J>([&](auto j) {
            const int c = sg * ((n.key[j] & 31) + lev - 1), F = (n.key[j] >> 5) - 32;
            const float cf = (float)c, v = (float)F + n.r[j], d0 = delta0 * n.rho[j];
            const float d = lev == 0 ? d0 : (lev == 2 ? n.d2[j] : (n.rho[j] - b0 * d0) * inv_b1 - n.d2[j]);
            const float m = (corner ? n.r[j] : 1.0f - n.r[j]) * d;
            D[j] = F + corner + c;
            q[0][j] = m;
            q[1][j] = m * (v + cf);
            q[2][j] = m * (n.K[j] + cf * v + 0.5f * cf * cf);
            if constexpr (SP) q[3][j] = m * n.chi[j];
        });
        const int clo = sg == 0 ? 0 : (sg > 0 ? Cmin + lev - 1 : -(Cmax + lev - 1));
        const int chi = sg == 0 ? 0 : (sg > 0 ? Cmax + lev - 1 : -(Cmin + lev - 1));
        const int last = min(Fmax + corner + chi, kHalo);
#pragma unroll 1
        for (int dl = max(Fmin + corner + clo, -kHalo); dl <= last; ++dl) {
            bool any = false;
            static_for<J>([&](auto j) { any = any || D[j] == dl; });
            if (!__any(any)) continue;
            float p[NF][J];
            static_for<J>([&](auto j) {
                const bool here = D[j] == dl;
                static_for<NF>([&](auto f) { p[f][j] = here ? q[f][j] : 0.0f; });
            });
            static_for<2 * kHalo + 1>([&](auto x) {
                constexpr int N = x - kHalo;
                if (dl == N) {
                    static_for<NF>([&](auto f) {
                        float s[J];
                        node_shift<N>(p[f], s);
                        static_for<J>([&](auto j) { o[f][j] += s[j]; });
                    });
                    keep_apart<N>();
                }
            });
        }
    }
}

// The packets of a wavefront's nodes.  Returns the largest reach; beyond H, or
// for bad states, t is not formed.
template <bool SP, int J, int NF>
__device__ __forceinline__ int tube_all_packets(const TubePackets<SP, J>& n, bool valid, bool bad, const Consts& k,
                                                float (&t)[NF][J])
{
    const int key0 = __builtin_amdgcn_readlane(n.key[0], __builtin_ctzll(__ballot(valid)));
    bool same = true;
    static_for<J>([&](auto j) { same = same && n.key[j] == key0; });
    if (__all(same || !valid)) {
        const int F = (key0 >> 5) - 32, C = key0 & 31, far = class_reach(F, C);
        if (far > kHalo || bad) return far;  // (such a reach admits c'_1 <= 3)
        if (C == 0) tube_packets<0, SP>(n, F, k, t);
        if (C == 1) tube_packets<1, SP>(n, F, k, t);
        if (C == 2) tube_packets<2, SP>(n, F, k, t);
        if (C == 3) tube_packets<3, SP>(n, F, k, t);
        return far;
    }
    int far = 0, Fmin = INT_MAX, Fmax = INT_MIN, Cmin = INT_MAX, Cmax = 0;
    static_for<J>([&](auto j) {
        const int F = (n.key[j] >> 5) - 32, C = n.key[j] & 31;
        far = max(far, class_reach(F, C));
        Fmin = min(Fmin, F);
        Fmax = max(Fmax, F);
        Cmin = min(Cmin, C);
        Cmax = max(Cmax, C);
    });
    far = -wave_min_dpp(valid ? -far : 0);
    if (far > kHalo || bad) return far;
    Fmin = wave_min_dpp(valid ? Fmin : INT_MAX);
    Fmax = -wave_min_dpp(valid ? -Fmax : INT_MAX);
    Cmin = wave_min_dpp(valid ? Cmin : INT_MAX);
    Cmax = -wave_min_dpp(valid ? -Cmax : INT_MAX);
    const bool near = Fmax - Fmin <= 1 && Cmax - Cmin <= 1;
    if (near && Cmin == 0) tube_packets_near<0, SP>(n, Fmin, valid, k, t);
    else if (near && Cmin == 1) tube_packets_near<1, SP>(n, Fmin, valid, k, t);
    else tube_packets_mixed<SP>(n, Fmin, Fmax, Cmin, Cmax, k, t);
    return far;
}

// One FP32 step (see tube_step).
template <bool SP, int J, int NF>
__device__ __forceinline__ int tube_step32(const float (&y)[NF][J], float (&t)[NF][J], const Consts& k,
                                           const TubeConsts& tc, bool valid, int* reach)
{
#pragma clang fp contract(off)
    TubePackets<SP, J> n;
    int err = 0;
    const bool plain = __all((tube_tame<SP>(y) && k.delta0 <= kTameDelta0) || !valid);
    bool anybad = false;
    const auto stage = [&](auto j, const TubeNodes<float, SP, 1>& q) {
        const double f = floor(q.v[0]), rho = q.rho[0];
        n.key[j] = tube_key(q.v[0], q.A[0]);
        const int C = n.key[j] & 31;
        const double inv = C == 0 ? 1.0 : (C == 1 ? 1.0 / 3.0 : (C == 2 ? 1.0 / 5.0 : 1.0 / 7.0));
        n.rho[j] = q.rho[0];
        n.r[j] = (float)(q.v[0] - f);
        n.d2[j] = (float)((rho - k.b0 * (k.delta0 * rho)) * k.inv_b1 * ((q.A[0] - (double)(C * C)) * inv));
        n.K[j] = q.K[0];
        if constexpr (SP) n.chi[j] = q.chi[0];
    };
    if (plain) {
        static_for<J>([&](auto j) {
            TubeNodes<float, SP, 1> q;
            tube_node<false>(q, 0, y[0][j], y[1][j], y[2][j], y[NF - 1][j], k, tc, false);
            stage(j, q);
            step_apart<J>();
        });
    } else {
        static_for<J>([&](auto j) {
            const bool bad = tube_bad<SP>(y, j);
            anybad = anybad || bad;
            TubeNodes<float, SP, 1> q;
            tube_node<true>(q, 0, y[0][j], y[1][j], y[2][j], y[NF - 1][j], k, tc, bad);
            stage(j, q);
        });
        if (__any(anybad && valid)) err |= kErrState;
    }
    *reach = tube_all_packets<SP>(n, valid, err != 0, k, t);
    if (*reach > kHalo) err |= kErrReach;
    return err;
}

// ---- FP64 ----

// LDS of one wavefront: the nodes and the new moments of a wavefront that mixes
// classes (each lane its own).  Five nodes per lane only: kept in registers
// across the loops below they would push the one-class path's values into
// scratch memory.
template <typename T, bool SP, int J>
struct TubeStash {
    static constexpr bool USED = J > 3 && sizeof(T) == 8;
    static constexpr int N = USED ? J : 1, L = USED ? 64 : 1;
    double v[N][L], A[N][L];
    T rho[N][L], K[N][L], t[SP ? 4 : 3][N][L];
    T chi[SP ? N : 1][SP ? L : 1];
};

// A wavefront that mixes classes: for each value of floor(v), ascending, and
// each speed, ascending, the packets of the nodes that have both (the others
// with zero mass: a node whose sources are all of one class gets the bits of the
// one-class form).  Zero mass times what a lane that does not count may hold (NaN)
// is no zero, so nothing is moved further than H: of each floor(v) only the speeds
// that an admissible source can have with it are taken.  Returns the largest
// reach; beyond H, or for bad states, t is not formed.
template <bool SP, typename T, int J, int NF>
__device__ __forceinline__ int tube_mixed(const TubeNodes<T, SP, J>& n, bool valid, bool bad, const Consts& k,
                                          TubeStash<T, SP, J>& st, int lane, T (&t)[NF][J])
{
#pragma clang fp contract(off)
    constexpr bool STASH = J > 3;
    int F[J], C[J], cmin = INT_MAX, cmax = 0, far = 0, next = INT_MAX;
    static_for<J>([&](auto j) {
        const int key = tube_key(n.v[j], n.A[j]);
        F[j] = (key >> 5) - 32;
        C[j] = key & 31;
        cmin = min(cmin, C[j]);
        cmax = max(cmax, C[j]);
        next = min(next, F[j]);
        far = max(far, class_reach(F[j], C[j]));
        if constexpr (STASH) {
            st.v[j][lane] = n.v[j];
            st.A[j][lane] = n.A[j];
            st.rho[j][lane] = n.rho[j];
            st.K[j][lane] = n.K[j];
            if constexpr (SP) st.chi[j][lane] = n.chi[j];
        }
    });
    far = -wave_min_dpp(valid ? -far : 0);
    if (far > kHalo || bad) return far;
    next = wave_min_dpp(valid ? next : INT_MAX);
    cmin = wave_min_dpp(valid ? cmin : INT_MAX);
    cmax = -wave_min_dpp(valid ? -cmax : 0);  // at most 3: the reach is within H
    static_for<NF>([&](auto f) {
        static_for<J>([&](auto j) {
            if constexpr (STASH) st.t[f][j][lane] = (T)0;
            else t[f][j] = (T)0;
        });
    });
#pragma unroll 1
    while (next != INT_MAX) {
        T o[NF][J];
        // level masses of the nodes with floor(v) = next, and what moves with them
        double r[J], d0[J], d1[J], d2[J];
        T v[J];
        TubeNodes<T, SP, J> m;
        const auto masses = [&]() {
            if constexpr (STASH) asm volatile("" ::: "memory");  // read back from LDS, not kept in registers
            static_for<J>([&](auto j) {
                const double vv = STASH ? st.v[STASH ? j : 0][STASH ? lane : 0] : n.v[j];
                const double A = STASH ? st.A[STASH ? j : 0][STASH ? lane : 0] : n.A[j];
                const double rho0 = STASH ? (double)st.rho[STASH ? j : 0][STASH ? lane : 0] : (double)n.rho[j];
                const double rho = F[j] == next ? rho0 : 0.0;
                d0[j] = k.delta0 * rho;
                const double per = (rho - k.b0 * d0[j]) * k.inv_b1;
                const double inv = C[j] == 0 ? 1.0 : (C[j] == 1 ? 1.0 / 3.0 : (C[j] == 2 ? 1.0 / 5.0 : 1.0 / 7.0));
                d2[j] = per * ((A - (double)(C[j] * C[j])) * inv);
                d1[j] = per - d2[j];
                if (C[j] == 0) d0[j] = __builtin_fma(2.0, d1[j], d0[j]);  // both lanes of c'_1 = 0 stay
                r[j] = vv - (double)next;
                v[j] = (T)vv;
                m.K[j] = STASH ? st.K[STASH ? j : 0][STASH ? lane : 0] : n.K[j];
                if constexpr (SP) m.chi[j] = STASH ? st.chi[STASH ? j : 0][STASH ? lane : 0] : n.chi[j];
            });
        };
        const auto of_speed = [&](int c, double (&d)[J]) {
            static_for<J>([&](auto j) { d[j] = C[j] == c ? d1[j] : (C[j] + 1 == c ? d2[j] : 0.0); });
        };
        double d[J];
        masses();
        tube_speed<0, true, SP>(d0, r, v, m, next, o);
        // the usual case in one piece (two or three nodes per lane, whose halo lanes hold H + 1 nodes: next + 3 at most)
        if (!STASH && cmax <= 1) {
            of_speed(1, d);
            tube_speed<1, false, SP>(d, r, v, m, next, o);
            of_speed(2, d);
            tube_speed<2, false, SP>(d, r, v, m, next, o);
        } else {
#pragma unroll 1
            for (int c = max(cmin, 1); c <= min(cmax + 1, kHalo + 1 - class_reach(next, 0)); ++c) {
                masses();
                of_speed(c, d);
                if (c == 1) tube_speed<1, false, SP>(d, r, v, m, next, o);
                if (c == 2) tube_speed<2, false, SP>(d, r, v, m, next, o);
                if (c == 3) tube_speed<3, false, SP>(d, r, v, m, next, o);
                if (c == 4) tube_speed<4, false, SP>(d, r, v, m, next, o);
            }
        }
        static_for<NF>([&](auto f) {
            static_for<J>([&](auto j) {
                if constexpr (STASH) st.t[f][j][lane] += o[f][j];
                else t[f][j] += o[f][j];
            });
        });
        int more = INT_MAX;
        static_for<J>([&](auto j) { more = min(more, F[j] > next ? F[j] : INT_MAX); });
        next = wave_min_dpp(valid ? more : INT_MAX);
    }
    if constexpr (STASH) static_for<NF>([&](auto f) { static_for<J>([&](auto j) { t[f][j] = st.t[f][j][lane]; }); });
    return far;
}

__device__ __forceinline__ double lane_value(double v, int lane)
{
    const Words w = __builtin_bit_cast(Words, v);
    return __builtin_bit_cast(double, Words{__builtin_amdgcn_readlane(w.lo, lane), __builtin_amdgcn_readlane(w.hi, lane)});
}

// One step of the lane's nodes, y -> t.  Lanes [lo, hi) hold real nodes (or
// halo images of them); the others' values do not matter.  Returns the error
// bits of those sources and *reach, their largest reach; on an error t is
// not used.
template <typename T, bool SP, int J, int NF>
__device__ __forceinline__ int tube_step(const T (&y)[NF][J], T (&t)[NF][J], const Consts& k, const TubeConsts& tc,
                                         TubeStash<T, SP, J>& st, int lo, int hi, int lane, int* reach)
{
#pragma clang fp contract(off)
    const bool valid = lane >= lo && lane < hi;
    if constexpr (sizeof(T) == 4) {
        return tube_step32<SP>(y, t, k, tc, valid, reach);
    } else {
        TubeNodes<T, SP, J> n;
        int err = 0;
        if (__all((tube_tame<SP>(y) && k.delta0 <= kTameDelta0) || !valid)) {
            static_for<J>([&](auto j) {
                tube_node<false>(n, j, y[0][j], y[1][j], y[2][j], y[NF - 1][j], k, tc, false);
                step_apart<J>();
            });
        } else {
            bool anybad = false;
            static_for<J>([&](auto j) {
                const bool bad = tube_bad<SP>(y, j);
                anybad = anybad || bad;
                tube_node<true>(n, j, y[0][j], y[1][j], y[2][j], y[NF - 1][j], k, tc, bad);
            });
            if (__any(anybad && valid)) err |= kErrState;
        }
        // the class of the first node; the others are of it if v - F lies in [0, 1)
        // and A - C^2 in [0, 2 C + 1), tested on the high words (the upper ends are
        // whole numbers)
        double r[J], g[J];
        const int key0 = __builtin_amdgcn_readfirstlane(tube_key(lane_value(n.v[0], lo), lane_value(n.A[0], lo)));
        const int F0 = (key0 >> 5) - 32, C0 = key0 & 31;
        const uint32_t gtop = C0 == 0 ? 0x3ff00000u : (C0 == 1 ? 0x40080000u : (C0 == 2 ? 0x40140000u : (C0 == 3 ? 0x401c0000u : 0u)));
        const double Fd = (double)F0, Cd = (double)(C0 * C0);
        bool same = true;
        static_for<J>([&](auto j) {
            const auto hw = [](double x) { return (uint32_t)(__builtin_bit_cast(uint64_t, x) >> 32); };
            r[j] = n.v[j] - Fd;
            g[j] = n.A[j] - Cd;
            same = same && hw(r[j]) < 0x3ff00000u && hw(g[j]) < gtop;
        });
        int far;
        if (__all(same || !valid)) {
            far = class_reach(F0, C0);
            if (far <= kHalo && !err) {  // (such a reach admits c'_1 <= 3)
                if (C0 == 0) tube_class<0, SP>(n, r, g, F0, k, t);
                if (C0 == 1) tube_class<1, SP>(n, r, g, F0, k, t);
                if (C0 == 2) tube_class<2, SP>(n, r, g, F0, k, t);
                if (C0 == 3) tube_class<3, SP>(n, r, g, F0, k, t);
            }
        } else {
            far = tube_mixed<SP>(n, valid, err != 0, k, st, lane, t);
        }
        *reach = far;
        if (far > kHalo) err |= kErrReach;
        return err;
    }
}

// The first and last H nodes of the domain, for the ghost nodes beyond its ends
// (transmissive: copies of the edge node; walls: mirror images).
template <typename T>
struct TubeEdges {
    T lo[4][kHalo], hi[4][kHalo];  // nodes i and nx - 1 - i
};

template <typename T, int J, int NF>
__device__ __forceinline__ void edges_put(TubeEdges<T>& e, const T (&y)[NF][J], int64_t xb, int64_t nx)
{
    static_for<J>([&](auto j) {
        const int64_t x = xb + j;
        if (x >= 0 && x < nx) {
            if (x < kHalo) static_for<NF>([&](auto f) { e.lo[f][x] = y[f][j]; });
            if (nx - 1 - x < kHalo) static_for<NF>([&](auto f) { e.hi[f][nx - 1 - x] = y[f][j]; });
        }
    });
}
// Ghost nodes within a lane or two of the ends (those further out than H reach
// no real node and need only be harmless).
template <typename T, int J, int NF>
__device__ __forceinline__ void edges_get(const TubeEdges<T>& e, T (&y)[NF][J], int64_t xb, int64_t nx, int bc)
{
    const bool wall = bc == kBcReflecting;
    static_for<J>([&](auto j) {
        const int64_t x = xb + j;
        if (x < 0 && x >= -2 * kHalo) {
            const int i = wall ? min((int)(-1 - x), kHalo - 1) : 0;
            static_for<NF>([&](auto f) { y[f][j] = e.lo[f][i]; });
            if (wall) y[1][j] = -y[1][j];
        }
        if (x >= nx && x < nx + 2 * kHalo) {
            const int i = wall ? min((int)(x - nx), kHalo - 1) : 0;
            static_for<NF>([&](auto f) { y[f][j] = e.hi[f][i]; });
            if (wall) y[1][j] = -y[1][j];
        }
    });
}
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename T, int J, int NF>
__device__ __forceinline__ void tube_load(const T* __restrict__ Y, T (&y)[NF][J], int64_t xb, int64_t nx, int bc,
                                          bool inside)
{
    if (inside) {  // the whole wavefront within the domain: a lane's nodes as one block
        static_for<NF>([&](auto f) { __builtin_memcpy(&y[f][0], Y + f * nx + xb, sizeof(T) * J); });
    } else {
        static_for<J>([&](auto j) {
            bool mir = false;
            const int64_t s = source_idx(xb + j, nx, bc, &mir);
            static_for<NF>([&](auto f) { y[f][j] = Y[f * nx + s]; });
            if (mir) y[1][j] = -y[1][j];
        });
    }
}
template <typename T, int J, int NF>
__device__ __forceinline__ void tube_store(T* __restrict__ Yn, const T (&y)[NF][J], int64_t xb, int64_t nx,
                                           bool own, double (&tot)[NF])
{
    if (!own || xb >= nx) return;
    if (xb + J <= nx) {
        static_for<NF>([&](auto f) { __builtin_memcpy(Yn + f * nx + xb, &y[f][0], sizeof(T) * J); });
    } else {
        static_for<J>([&](auto j) {
            if (xb + j < nx) static_for<NF>([&](auto f) { Yn[f * nx + xb + j] = y[f][j]; });
        });
    }
    static_for<J>([&](auto j) {
        if (xb + j < nx) static_for<NF>([&](auto f) { tot[f] += (double)y[f][j]; });
    });
}

// Outcome of a wavefront's steps: reach of the last (or the failing) step,
// error bits and the step that failed (1-based; 0: none).
struct TubeOut {
    int reach, err, errsub;
};

// `steps` <= K steps of the destination nodes [X0, X0 + tube_cols(J, K)), from Y
// to Yn, with the halo lanes of K steps; adds the new moments to tot.  Stops at
// the first step with a bad source or a reach beyond H (Yn is then not written).
// AGAIN: the last step is made for its outcome alone, and Yn gets the state before
// it (unless it is the first).
template <typename T, bool SP, int J, bool AGAIN = false>
__device__ __forceinline__ TubeOut tube_run(const T* __restrict__ Y, T* __restrict__ Yn, int64_t nx, int bc,
                                            int64_t X0, int K, int steps, const Consts& k, TubeEdges<T>& edges,
                                            TubeStash<T, SP, J>& st, double (&tot)[SP ? 4 : 3])
{
    constexpr int NF = SP ? 4 : 3, LOST = tube_lost(J);
    const int lane = threadIdx.x & 63, halo = K * LOST;
    const int64_t w0 = X0 - (int64_t)halo * J, xb = w0 + lane * J;
    // lanes that may hold real nodes or ghosts next to them
    const bool open = bc != kBcPeriodic;
    const int first = open && w0 < -kHalo ? (int)((-kHalo - w0) / J) : 0;
    const int top = open ? (int)min((nx + kHalo - w0 + J - 1) / J, (int64_t)64) : 64;
    const bool ends = open && (w0 < 0 || w0 + 64 * J > nx);
    T y[NF][J], t[NF][J];
    tube_load(Y, y, xb, nx, bc, w0 >= 0 && w0 + 64 * J <= nx);
    const TubeConsts tc = tube_consts(k, SP);
    TubeOut out{0, 0, 0};
#pragma unroll 1
    for (int i = 0; i < steps; ++i) {
        if (ends && i > 0) {  // the ghosts follow the edge nodes
            edges_put(edges, y, xb, nx);
            wave_sync();
            edges_get(edges, y, xb, nx, bc);
            wave_sync();
        }
        if constexpr (AGAIN) {
            if (i > 0 && i == steps - 1) tube_store(Yn, y, xb, nx, lane >= halo && lane < 64 - halo, tot);
        }
        out.err = tube_step<T, SP>(y, t, k, tc, st, max(i * LOST, first), min(64 - i * LOST, top), lane, &out.reach);
        if (out.err) {
            out.errsub = i + 1;
            return out;
        }
        static_for<NF>([&](auto f) { static_for<J>([&](auto j) { y[f][j] = t[f][j]; }); });
    }
    if constexpr (!AGAIN) tube_store(Yn, y, xb, nx, lane >= halo && lane < 64 - halo, tot);
    return out;
}

}  // namespace

}  // namespace lbsd
