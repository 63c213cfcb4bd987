// The tau = 1 step on the hexagonal lattice (Fig. 1 of Komeili, Mirzaei,
// Shabouei, arXiv 1602.02675; Sec. III.B with b_v = 6).
//
// Nodes sit at i e_1 + j e_2 (e_1 = (1, 0), e_2 = (1/2, sqrt(3)/2), unit
// spacing), stored SoA Y[f][j][i]; momenta are Cartesian.  A source node
// emits, per lane (rest group; six directions u_d at c'_1 and at c'_2), one
// packet to each vertex of the lattice triangle around the end point of its
// velocity, with the vertex's barycentric weight: mass alpha_k d_v (eq. 23),
// momentum m (v + c' u_d), energy m (K + c' u_d . v + c'^2 / 2) with K =
// |v|^2 / 2 + phi (eq. 14, 21), to x + f + k + c' u_d in axial steps.
//
// The migration factors into the vertex sums of each speed c, U_c(x) = the sum
// of m (1, v, K) over the sources and vertices that land on x with one lane of
// that speed, and the lanes: the new moments of x take U_c at x - c u_d for the
// six d.  (The rest group and both speeds' lanes at c = 0 stay where the
// vertices put them.)  That is 3 packets per speed and node where the lanes
// taken one by one make 18, each looked up in LDS: 4096^2 nodes in FP64 took
// 1697 us so.
//
// A block computes tiles of kHX x kHY destinations, one per thread.  A tile's
// sources, a halo of H = kHalo nodes included, are held by the threads in
// registers (up to kHSlots each); per speed they put m (1, v, K) in LDS (zero
// mass where the source lacks the speed), the threads gather U_c on the tile
// and a halo of c nodes, class of sources by class (floor of the axial
// velocity, triangle), and each adds its six lanes.  The order of every sum is
// that of the classes, whatever else a tile holds: results do not depend on the
// tiling.  Two blocks share a CU's LDS (80 KB each in FP64), so that one
// computes while the other waits at a barrier: 4096^2 nodes in FP64 take 632 us,
// half of it VALU issue (685 instructions per node, a third of them the
// primitives of 2.1 sources per destination), the rest barriers and LDS reads.
#include "lb_wave.hpp"

namespace lbsd {
namespace {

constexpr int kHX = 32, kHY = 16, kHH = kHalo;  // tile (axial i x j) and halo
constexpr int kHTPB = kHX * kHY;                // one destination per thread
constexpr int kSW = kHX + 2 * kHH, kSH = kHY + 2 * kHH, kSN = kSW * kSH;  // sources
constexpr int kHSlots = (kSN + kHTPB - 1) / kHTPB;
constexpr int kHNW = kHTPB / 64;
// Blocks of a launch: two per CU of a 256-CU device, which take tiles in turn.
constexpr int64_t kHexBlocks = 512;
constexpr int kHexTurn = 29;
// U_c on the tile and c nodes around it: four fields for c <= 2; the speeds 3
// and 4 (the largest within H) take two passes of two fields in the same LDS.
constexpr int u_nodes(int c) { return (kHX + 2 * c) * (kHY + 2 * c); }
constexpr int kU4 = u_nodes(2), kU2 = u_nodes(4), kUN = 4 * kU4;
static_assert(2 * kU2 <= kUN, "");
constexpr int kHMaxC = 4;

constexpr double kH3 = 0.8660254037844386;  // sqrt(3) / 2, correctly rounded

// Class of a source that can be within the halo: floors -4 .. 3 of both axial
// coordinates, triangle; kNoClass: any other, and bad sources.
constexpr int kNoClass = 255;
__device__ __forceinline__ int hex_class(int fa, int fb, int tri)
{
    const bool in = fa >= -4 && fa <= 3 && fb >= -4 && fb <= 3;
    return in ? (fa + 4) | (fb + 4) << 3 | tri << 6 : kNoClass;
}

template <typename T>
struct HexLds {
    int cls[kSN];
    T w1[kSN], w2[kSN];  // weights of the vertices (1, 0) and (0, 1); the third has the rest
    T s[4][kSN];         // m (1, v_x, v_y, K) of one speed's lanes
    T u[kUN];
    uint32_t present[2][4];  // classes of the tile's sources (one set per tile in turn)
    int clo[2], chi[2];
    double sum[kHNW][4];
    int ir[kHNW][2];
};

template <typename T>
struct SrcHex {   // one source node of the hexagonal lattice
    int fa, fb;   // floor of the axial coordinates (a, b) of v = a e_1 + b e_2
    int c1;
    int tri;      // triangle of the cell that holds the end point of v: 0 has
                  // the vertex (0, 0), 1 the vertex (1, 1) (both (1,0), (0,1))
    T ra, rb;     // (a, b) - (f_a, f_b)
    T vx, vy;     // Cartesian v (lattice units)
    T K;          // |v|^2 / 2 + phi
    T d0, d1, d2; // level weights (d0 = 0 without the rest group)
    bool bad;
};

constexpr double kSqrt3 = 1.7320508075688772;  // sqrt(3), correctly rounded

// A source as its thread holds it.
template <typename T>
struct HexSrc {
    T vx, vy, K, d0, d1, d2;
    int c1;
};

// Per-node primitives, level speeds and weights of a source (Fig. 1; eq. 15, 24-26
// with b_1 = b_2 = 6, Consts::inv_b1 = 1/6) in FP64 whatever the storage type, and
// the end point of v in axial coordinates, b = 2 v_y / sqrt(3), a = v_x - b / 2
// (e_1 = (1, 0), e_2 = (1/2, sqrt(3)/2)), whose cell (f_a, f_b) + [0, 1]^2 splits
// into the triangles below and above the diagonal r_a + r_b = 1.  REST: the set
// with a rest group, d_0 = delta0 rho.  IEEE: any operands of a good state;
// otherwise they are tame, and the quotients come from shared reciprocals.  Both
// forms give the same bits: which one a wavefront takes depends on its other nodes.
template <typename T, bool REST, bool IEEE>
__device__ __forceinline__ SrcHex<T> hex_node(double m0, double m1, double m2, double m3, const Consts& k)
{
#pragma clang fp contract(off)
    constexpr bool FAST = sizeof(T) < 8;
    SrcHex<T> s;
    s.bad = false;
    const Quot<FAST, IEEE> by_rho(m0);
    const double vx = by_rho(m1), vy = by_rho(m2), E = by_rho(m3);
    const double v2 = vx * vx + vy * vy;
    const Quot<FAST, IEEE> by_s3(kSqrt3);
    const double b = by_s3(2.0 * vy), a = vx - 0.5 * b;
    const double d0 = REST ? k.delta0 * m0 : 0.0, rest = m0 - k.b0 * d0;
    double e = E - 0.5 * v2;
    if (e < 0.0) e = 0.0;
    const double Ar = k.Dg1 * e * m0;
    double A;
    if constexpr (REST) {
        const Quot<FAST, IEEE> by_rest(rest);
        A = by_rest(Ar);
    } else {
        A = by_rho(Ar);
    }
    if constexpr (IEEE) {
        if (!(A >= 0.0)) A = 0.0;
    }
    if (__any(A >= 9.0)) {
        if (A > (double)kMaxC1 * (double)kMaxC1) A = (double)kMaxC1 * (double)kMaxC1;
        s.c1 = isqrt_floor<double>(A);
    } else {
        s.c1 = (A >= 1.0 ? 1 : 0) + (A >= 4.0 ? 1 : 0);
    }
    // floors clamped far beyond any admissible reach (the step reports those)
    const double fa = fmin(fmax(floor(a), -32.0), 31.0), fb = fmin(fmax(floor(b), -32.0), 31.0);
    s.fa = (int)fa;
    s.fb = (int)fb;
    const double ra = a - fa, rb = b - fb;
    s.tri = ra + rb > 1.0 ? 1 : 0;
    s.ra = (T)ra;
    s.rb = (T)rb;
    s.vx = (T)vx;
    s.vy = (T)vy;
    const double per = rest * k.inv_b1, d2 = per * level_w(A, s.c1);
    s.d2 = (T)d2;
    s.d1 = (T)(per - d2);
    s.d0 = (T)d0;
    s.K = (T)__builtin_fma(k.phi_coef, e, 0.5 * v2);
    return s;
}
template <typename T, bool REST>
__device__ __forceinline__ SrcHex<T> hex_source(T m0, T m1, T m2, T m3, const Consts& k)
{
    if (__all(tame(m0, m1, m2, m3) && (!REST || k.delta0 <= kTameDelta0)))
        return hex_node<T, REST, false>(m0, m1, m2, m3, k);
    const bool bad = !((double)m0 > 0.0) || !isfinite(m0) || !isfinite(m1) || !isfinite(m2) || !isfinite(m3);
    SrcHex<T> s = hex_node<T, REST, true>(bad ? (T)1 : m0, bad ? (T)0 : m1, bad ? (T)0 : m2, bad ? (T)0 : m3, k);
    s.bad = bad;
    return s;
}

// U_c (fields F0 .. F0 + NFLD) on the tile and c nodes around it.
template <typename T, int F0, int NFLD>
__device__ __forceinline__ void hex_vertices(HexLds<T>& st, int c, const uint32_t* present, int tid)
{
    constexpr int US = NFLD == 4 ? kU4 : kU2;
    const int w = kHX + 2 * c, n = w * (kHY + 2 * c);
    const uint32_t inv = (65536u + w - 1) / w;  // q / w for q < 960, w <= 40
    for (int q = tid; q < n; q += kHTPB) {
        const int uj = (int)(((uint32_t)q * inv) >> 16), ui = q - uj * w;
        const int x = (uj + kHH - c) * kSW + ui + kHH - c;
        T acc[NFLD];
        static_for<NFLD>([&](auto f) { acc[f] = (T)0; });
        for (int i = 0; i < 4; ++i) {
            uint32_t m = present[i];
            while (m) {
                const int cl = i * 32 + __builtin_ctz(m);
                m &= m - 1;
                const int fa = (cl & 7) - 4, fb = ((cl >> 3) & 7) - 4, tri = cl >> 6;
                // vertices (tri, tri), (1, 0), (0, 1); one whose lanes of this
                // speed would leave the halo has no admissible source
                const auto in = [&](int f) { return f + c <= kHH && c - f <= kHH; };
                const int x0 = x - (fb + tri) * kSW - (fa + tri), x1 = x - fb * kSW - (fa + 1),
                          x2 = x - (fb + 1) * kSW - fa;
                const int p0 = in(fa + tri) && in(fb + tri) ? st.cls[x0] : kNoClass;
                const int p1 = in(fa + 1) && in(fb) ? st.cls[x1] : kNoClass;
                const int p2 = in(fa) && in(fb + 1) ? st.cls[x2] : kNoClass;
                if (p0 == cl) {
                    const T wt = ((T)1 - st.w1[x0]) - st.w2[x0];
                    static_for<NFLD>([&](auto f) { acc[f] = fmaT(wt, st.s[F0 + f][x0], acc[f]); });
                }
                if (p1 == cl) {
                    const T wt = st.w1[x1];
                    static_for<NFLD>([&](auto f) { acc[f] = fmaT(wt, st.s[F0 + f][x1], acc[f]); });
                }
                if (p2 == cl) {
                    const T wt = st.w2[x2];
                    static_for<NFLD>([&](auto f) { acc[f] = fmaT(wt, st.s[F0 + f][x2], acc[f]); });
                }
            }
        }
        static_for<NFLD>([&](auto f) { st.u[f * US + q] = acc[f]; });
    }
}

// A destination's new moments, in FP64.
struct HexSum {
    double R, PX, PY, E;
};

// Adds the lanes of speed c that fields F0 .. F0 + NFLD of U_c (at x - c u_d,
// u_d the axial steps (1,0), (0,1), (-1,1), (-1,0), (0,-1), (1,-1)) give.
template <typename T, int F0, int NFLD>
__device__ __forceinline__ void hex_lanes(const HexLds<T>& st, int c, int li, int lj, HexSum& o)
{
#pragma clang fp contract(off)
    constexpr int US = NFLD == 4 ? kU4 : kU2;
    const int w = kHX + 2 * c, x = (lj + c) * w + li + c;
    if (c == 0) {
        const auto u = [&](int f) { return (double)st.u[f * US + x]; };
        if constexpr (F0 == 0) {
            o.R += u(0);
            o.PX += u(1);
        }
        if constexpr (F0 + NFLD == 4) {
            o.PY += u(2 - F0);
            o.E += u(3 - F0);
        }
        return;
    }
    const int at[6] = {x - c, x - c * w, x - c * w + c, x + c, x + c * w, x + c * w - c};
    const double cc = (double)c;
    // sum over the lanes; the lanes' x and y components
    const auto sum = [&](const double (&v)[6]) { return ((v[0] + v[3]) + (v[1] + v[4])) + (v[2] + v[5]); };
    const auto ux = [&](const double (&v)[6]) { return (v[0] - v[3]) + 0.5 * ((v[1] - v[4]) + (v[5] - v[2])); };
    const auto uy = [&](const double (&v)[6]) { return kH3 * ((v[1] - v[4]) + (v[2] - v[5])); };
    double v[6];
    const auto get = [&](int f) { static_for<6>([&](auto d) { v[d] = (double)st.u[f * US + at[d]]; }); };
    if constexpr (F0 == 0) {
        get(0);
        const double M = sum(v);
        o.R += M;
        o.E += 0.5 * cc * cc * M;
        double px = cc * ux(v);
        o.PY += cc * uy(v);
        get(1);
        o.PX += sum(v) + px;
        o.E += cc * ux(v);
    }
    if constexpr (F0 + NFLD == 4) {
        get(2 - F0);
        o.PY += sum(v);
        o.E += cc * uy(v);
        get(3 - F0);
        o.E += sum(v);
    }
}

template <typename T, bool REST>
__global__ void __launch_bounds__(kHTPB) __attribute__((amdgpu_waves_per_eu(4, 4)))
hex_step_kernel(const T* __restrict__ Y, T* __restrict__ Yn, Grid g, Consts k, StepCtl* __restrict__ ctl,
                double* __restrict__ partials, long long step, uint32_t tiles_x, uint32_t tiles_y)
{
    __shared__ HexLds<T> st;
    if (ctl->err_step < step) return;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int64_t nx = g.nx, ny = g.ny, nn = nx * ny;
    const uint32_t tiles = (uint32_t)tiles_x * tiles_y;
    const int li = tid % kHX, lj = tid / kHX;
    HexSum tot{0.0, 0.0, 0.0, 0.0};
    int reach = 0, bad = 0;
    if (tid < 8) st.present[tid >> 2][tid & 3] = 0;
    if (tid < 2) {
        st.clo[tid] = INT_MAX;
        st.chi[tid] = -1;
    }
    __syncthreads();
    // Tiles in rounds of one per block.  Consecutive tiles of a round, whose halos
    // overlap, go to the blocks of one XCD (which are eight apart), and the round
    // is turned a little further each time: a planar flow's slow tiles (sources of
    // several classes) stand in one column of tiles, which would else fall to the
    // same blocks every time.
    const uint32_t nb = gridDim.x, b = blockIdx.x, pos = nb % 8 ? b : (b % 8) * (nb / 8) + b / 8;
    int par = 0;
    for (uint32_t round = 0; round * nb < tiles; ++round) {
        const uint32_t tile = round * nb + (pos + round * kHexTurn) % nb;
        if (tile >= tiles) continue;
        const int64_t X0 = (int64_t)(tile % tiles_x) * kHX, Y0 = (int64_t)(tile / tiles_x) * kHY;  // i fastest
        // a tile whose halo lies within the domain reads it by 32-bit offsets
        const bool inner = X0 >= kHH && X0 + kHX + kHH <= nx && Y0 >= kHH && Y0 + kHY + kHH <= ny && nx < (1 << 24);
        const T* const Yt = Y + ((Y0 - kHH) * nx + (X0 - kHH));
        // the sources (boundaries map the halo), their classes and speeds
        HexSrc<T> src[kHSlots];
        uint64_t had0 = 0, had1 = 0;
        int lo = INT_MAX, hi = -1;
        static_for<kHSlots>([&](auto n) {
            const int q = n * kHTPB + tid;
            HexSrc<T>& h = src[n];
            h.c1 = -2;
            int cl = kNoClass;
            if (q < kSN) {
                const int sj = q / kSW, si = q - sj * kSW;
                const int64_t gi = X0 - kHH + si, gj = Y0 - kHH + sj;
                T m0, m1, m2, m3;
                if (inner) {
                    const uint32_t p = (uint32_t)sj * (uint32_t)nx + (uint32_t)si;
                    m0 = Yt[p];
                    m1 = (Yt + nn)[p];
                    m2 = (Yt + 2 * nn)[p];
                    m3 = (Yt + 3 * nn)[p];
                } else {
                    const int64_t i = g.bc_x == kBcPeriodic ? wrap_near(gi, nx) : clamp_idx(gi, nx);
                    const int64_t j = g.bc_y == kBcPeriodic ? wrap_near(gj, ny) : clamp_idx(gj, ny);
                    const int64_t p = j * nx + i;
                    m0 = Y[p];
                    m1 = Y[nn + p];
                    m2 = Y[2 * nn + p];
                    m3 = Y[3 * nn + p];
                }
                const SrcHex<T> s = hex_source<T, REST>(m0, m1, m2, m3, k);
                h.vx = s.vx;
                h.vy = s.vy;
                h.K = s.K;
                h.d0 = s.bad ? (T)0 : s.d0;
                h.d1 = s.d1;
                h.d2 = s.d2;
                h.c1 = s.bad ? -2 : s.c1;
                cl = s.bad ? kNoClass : hex_class(s.fa, s.fb, s.tri);
                st.cls[q] = cl;
                st.w1[q] = s.tri ? (T)1 - s.rb : s.ra;
                st.w2[q] = s.tri ? (T)1 - s.ra : s.rb;
                if (!s.bad) {
                    lo = min(lo, s.c1);
                    hi = max(hi, s.c1);
                }
                if (si >= kHH && si < kHH + kHX && sj >= kHH && sj < kHH + kHY && (inner || (gi < nx && gj < ny))) {
                    bad |= s.bad ? 1 : 0;
                    if (!s.bad) reach = max(reach, max(axis_reach(s.fa, s.c1), axis_reach(s.fb, s.c1)));
                }
            }
            for (uint64_t todo = __ballot(cl != kNoClass); todo;) {
                const int first = __builtin_amdgcn_readlane(cl, __builtin_ctzll(todo));
                (first & 64 ? had1 : had0) |= 1ull << (first & 63);
                todo &= ~__ballot(cl == first);
            }
        });
        lo = wave_min_dpp(lo);
        hi = -wave_min_dpp(-hi);
        if (lane < 4) {
            const uint64_t had = lane & 2 ? had1 : had0;
            atomicOr(&st.present[par][lane], (uint32_t)(lane & 1 ? had >> 32 : had));
        }
        if (lane == 0) {
            atomicMin(&st.clo[par], lo);
            atomicMax(&st.chi[par], hi);
        }
        __syncthreads();
        if (tid < 4) st.present[par ^ 1][tid] = 0;
        if (tid == 0) {
            st.clo[par ^ 1] = INT_MAX;
            st.chi[par ^ 1] = -1;
        }
        uint32_t present[4];
        for (int i = 0; i < 4; ++i) present[i] = __builtin_amdgcn_readfirstlane((int)st.present[par][i]);
        const int clo = __builtin_amdgcn_readfirstlane(st.clo[par]);
        const int chi = __builtin_amdgcn_readfirstlane(st.chi[par]);

        HexSum o{0.0, 0.0, 0.0, 0.0};
        for (int c = REST ? 0 : clo; c <= min(chi + 1, kHMaxC); ++c) {
            if (REST && c > 0 && c < clo) continue;
            // what the sources' lanes of this speed carry (c = 0: all that stay)
            static_for<kHSlots>([&](auto n) {
                const int q = n * kHTPB + tid;
                const HexSrc<T>& h = src[n];
                T m = h.c1 == c ? h.d1 : (h.c1 + 1 == c ? h.d2 : (T)0);
                if (c == 0) m = fmaT((T)6, m, REST && h.c1 >= 0 ? h.d0 : (T)0);
                if (q < kSN) {
                    st.s[0][q] = m;
                    st.s[1][q] = m * h.vx;
                    st.s[2][q] = m * h.vy;
                    st.s[3][q] = m * h.K;
                }
            });
            __syncthreads();
            if (c <= 2) {
                hex_vertices<T, 0, 4>(st, c, present, tid);
                __syncthreads();
                hex_lanes<T, 0, 4>(st, c, li, lj, o);
            } else {
                hex_vertices<T, 0, 2>(st, c, present, tid);
                __syncthreads();
                hex_lanes<T, 0, 2>(st, c, li, lj, o);
                __syncthreads();
                hex_vertices<T, 2, 2>(st, c, present, tid);
                __syncthreads();
                hex_lanes<T, 2, 2>(st, c, li, lj, o);
            }
        }
        // (no speed within the halo: the next tile's classes must wait here)
        if ((REST ? 0 : clo) > min(chi + 1, kHMaxC)) __syncthreads();
        const int64_t gi = X0 + li, gj = Y0 + lj;
        if (gi < nx && gj < ny) {
            const int64_t q = gj * nx + gi;
            const T r = (T)o.R, px = (T)o.PX, py = (T)o.PY, en = (T)o.E;
            Yn[q] = r;
            Yn[nn + q] = px;
            Yn[2 * nn + q] = py;
            Yn[3 * nn + q] = en;
            tot.R += (double)r;  // the totals are those of the stored fields
            tot.PX += (double)px;
            tot.PY += (double)py;
            tot.E += (double)en;
        }
        par ^= 1;
    }

    const double R = wave_sum(tot.R), PX = wave_sum(tot.PX), PY = wave_sum(tot.PY), E = wave_sum(tot.E);
    reach = wave_max(reach);
    bad = wave_max(bad);
    if (lane == 0) {
        st.sum[wid][0] = R; st.sum[wid][1] = PX; st.sum[wid][2] = PY; st.sum[wid][3] = E;
        st.ir[wid][0] = reach;
        st.ir[wid][1] = bad;
    }
    __syncthreads();
    if (tid == 0) {
        double* prow = partials + (int64_t)blockIdx.x * kPartialStride;
        int rr = 0, bb = 0;
        for (int f = 0; f < 4; ++f) {
            double t = st.sum[0][f];
            for (int w = 1; w < kHNW; ++w) t += st.sum[w][f];
            prow[f] = t;
        }
        for (int w = 0; w < kHNW; ++w) {
            rr = max(rr, st.ir[w][0]);
            bb |= st.ir[w][1];
        }
        prow[4] = (double)rr;
        prow[5] = (double)((rr > kHH ? kErrReach : 0) | (bb ? kErrState : 0));
        prow[6] = 0.0;
    }
}

// The integer decisions of every node, as the step takes them (bad states: 0).
template <typename T, bool REST>
__global__ void __launch_bounds__(256)
hex_lanes_kernel(const T* __restrict__ Y, int64_t nn, Consts k, int32_t* __restrict__ fa, int32_t* __restrict__ fb,
                 int32_t* __restrict__ c1)
{
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x, p = min(q, nn - 1);
    const SrcHex<T> s = hex_source<T, REST>(Y[p], Y[nn + p], Y[2 * nn + p], Y[3 * nn + p], k);
    if (q >= nn) return;
    fa[q] = s.bad ? 0 : s.fa;
    fb[q] = s.bad ? 0 : s.fb;
    c1[q] = s.bad ? 0 : s.c1;
}

}  // namespace

int64_t hex_blocks(const Grid& g)
{
    const int64_t tiles = ((g.nx + kHX - 1) / kHX) * ((g.ny + kHY - 1) / kHY);
    return tiles < kHexBlocks ? tiles : kHexBlocks;
}

template <typename T>
hipError_t launch_hex(const T* Y, T* Yn, const Grid& g, const Consts& k, StepCtl* ctl, double* partials,
                      long long step, hipStream_t stream)
{
    const unsigned grid = (unsigned)hex_blocks(g);
    const uint32_t tx = (uint32_t)((g.nx + kHX - 1) / kHX), ty = (uint32_t)((g.ny + kHY - 1) / kHY);
    if (k.b0 > 0.0)
        hex_step_kernel<T, true><<<grid, kHTPB, 0, stream>>>(Y, Yn, g, k, ctl, partials, step, tx, ty);
    else
        hex_step_kernel<T, false><<<grid, kHTPB, 0, stream>>>(Y, Yn, g, k, ctl, partials, step, tx, ty);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_lanes_hex(const T* Y, const Grid& g, const Consts& k, int32_t* fa, int32_t* fb, int32_t* c1,
                            hipStream_t stream)
{
    const int64_t nn = g.nx * g.ny;
    const unsigned nb = (unsigned)((nn + 255) / 256);
    if (k.b0 > 0.0) hex_lanes_kernel<T, true><<<nb, 256, 0, stream>>>(Y, nn, k, fa, fb, c1);
    else hex_lanes_kernel<T, false><<<nb, 256, 0, stream>>>(Y, nn, k, fa, fb, c1);
    return hipGetLastError();
}

template hipError_t launch_lanes_hex<double>(const double*, const Grid&, const Consts&, int32_t*, int32_t*, int32_t*,
                                             hipStream_t);
template hipError_t launch_lanes_hex<float>(const float*, const Grid&, const Consts&, int32_t*, int32_t*, int32_t*,
                                            hipStream_t);
template hipError_t launch_hex<double>(const double*, double*, const Grid&, const Consts&, StepCtl*, double*,
                                       long long, hipStream_t);
template hipError_t launch_hex<float>(const float*, float*, const Grid&, const Consts&, StepCtl*, double*,
                                      long long, hipStream_t);

}  // namespace lbsd
