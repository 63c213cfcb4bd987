// Device-side building blocks shared by the lattices' tau = 1 steps on gfx950
// (Komeili, Mirzaei, Shabouei, arXiv 1602.02675).
//
// One node's equilibrium (Sec. III.B) is reduced to a handful of numbers:
//   f      floor of the flow velocity per axis (corner 0 of eq. 28/29)
//   r      v - f per axis: the interpolation fraction (alpha_1 = r, alpha_0 = 1 - r)
//   c1     c'_1 of eq. 26 (c'_2 = c1 + 1)
//   d0..d2 level weights (eq. 24-25 and d_0 = delta0 rho)
//   K      |v|^2 / 2 + phi, so that a packet on lane c' carries
//          zeta = K + c'.v + |c'|^2 / 2 (eq. 14, 21)
// Each lattice forms them in a function of its own (tube_node, march_node,
// hex_node), from which its step and the dump of its integer decisions are made.
// In FP64 those decisions (f, c1) are those of the plain definition, bit for bit,
// with FMA contraction off.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lbsd {

constexpr int kMaxC1 = 1000;  // caps A (any real reach check fails far earlier)

// Boundary of a grid axis (the values of LB_BC_*).
constexpr int kBcTransmissive = 0;
constexpr int kBcPeriodic = 1;
constexpr int kBcReflecting = 2;

// Problem constants shared by every kernel (lattice units).
struct Consts {
    double Dg1;       // D (gamma - 1)
    double phi_coef;  // 1 - (D/2)(gamma - 1), eq. 15
    double delta0;    // d_0 / rho on the triple-level sets (0 on the square dual-level set)
    double b0;        // rest-lane multiplicity b_0 (1 with a rest level, else 0)
    double inv_b1;    // 1 / b_1
    double g1m1;      // two gases: gamma_1 - 1 (gas 1, the species field's gas)
    double g2m1;      // two gases: gamma_2 - 1
    int species;      // 1: two gases, a species moment rho chi after rho E
    int hex;          // 1: the hexagonal lattice (2-D)
    int rest;         // 1: the square lattice with a rest level
};

// Largest integer c <= kMaxC1 with c*c <= A, for A >= 0 (eq. 26: "int" of sqrt).
template <typename T>
__device__ __forceinline__ int isqrt_floor(T A)
{
#pragma clang fp contract(off)
    // a single-precision root (relative error < 1e-7), capped before it becomes a
    // whole number, is within one of the answer, and the exact comparisons settle it
    int c = (int)fminf(sqrtf((float)A), (float)kMaxC1);
    if (c > 0 && (T)c * (T)c > A) --c;
    if ((T)(c + 1) * (T)(c + 1) <= A) ++c;
    return c < kMaxC1 ? c : kMaxC1;
}

// a / b in the per-node primitives.  FAST = false (FP64 storage): the
// correctly rounded quotient, so that floor(v) and c'_1 match the plain
// definition bit for bit.  FAST = true (FP32 storage, whose results are
// rounded to FP32 and whose decisions the step does not need bit for bit):
// the hardware reciprocal refined by one Newton step, r (2 - b r), in two
// FMAs, then a product; relative error near 1e-16, far below FP32 rounding,
// for a few instructions instead of the IEEE division sequence.  b > 0, finite.
template <bool FAST>
__device__ __forceinline__ double pdiv(double a, double b)
{
    if constexpr (FAST) {
        double r = __builtin_amdgcn_rcp(b);
        r = __builtin_fma(r, __builtin_fma(-b, r, 1.0), r);
        return a * r;
    } else {
#pragma clang fp contract(off)
        return a / b;
    }
}

// w = (A - c'_1^2) / (2 c'_1 + 1) in [0, 1]: the share of level 2 (eq. 24-25
// rewritten; b_1 d_2 = (rho - b_0 d_0) w).  The divisor is a small odd
// integer: its reciprocal is a constant for the usual c'_1 <= 3.
__device__ __forceinline__ double level_w(double A, int c1)
{
    const double num = A - (double)(c1 * c1);
    double w;
    if (c1 <= 3)
        w = num * (c1 == 0 ? 1.0 : (c1 == 1 ? 1.0 / 3.0 : (c1 == 2 ? 1.0 / 5.0 : 1.0 / 7.0)));
    else
        w = num / (double)(2 * c1 + 1);
    return w < 0.0 ? 0.0 : (w > 1.0 ? 1.0 : w);
}

// Reach of a node: the largest |displacement| of any of its packets along one
// axis, max(f + 1 + c'_2, c'_2 - f).
__device__ __forceinline__ int axis_reach(int f, int c1)
{
    const int c2 = c1 + 1;
    const int a = f + 1 + c2, b = c2 - f;
    return a > b ? a : b;
}

// Wavefront (64-lane) reductions.
template <typename V>
__device__ __forceinline__ V wave_sum(V x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}
__device__ __forceinline__ int wave_max(int x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { int y = __shfl_xor(x, o, 64); x = y > x ? y : x; }
    return x;
}
__device__ __forceinline__ int64_t wrap_idx(int64_t i, int64_t n)
{
    int64_t r = i % n;
    return r < 0 ? r + n : r;
}
// Periodic index for i within a few periods of [0, n): the full modulo runs
// only for the (halo) indices that are out of range.
__device__ __forceinline__ int64_t wrap_near(int64_t i, int64_t n)
{
    if (i >= 0 && i < n) return i;
    if (i < 0 && i + n >= 0) return i + n;
    if (i >= n && i - n < n) return i - n;
    return wrap_idx(i, n);
}
__device__ __forceinline__ int64_t clamp_idx(int64_t i, int64_t n)
{
    return i < 0 ? 0 : (i >= n ? n - 1 : i);
}
// Reflecting walls stand on the outer faces of nodes 0 and n - 1: a node
// beyond a wall is the mirror image of node -1 - i (low end) or 2n - 1 - i
// (high end), with its normal momentum negated.  Sources within the halo of
// the domain (n >= halo) map exactly; indices further out, which only the
// spare columns of a last tile read and whose packets reach no destination,
// are clamped into range.
__device__ __forceinline__ int64_t mirror_idx(int64_t i, int64_t n)
{
    if (i < 0) { const int64_t m = -1 - i; return m < n ? m : n - 1; }
    if (i >= n) { const int64_t m = 2 * n - 1 - i; return m >= 0 ? m : 0; }
    return i;
}
// Source index of (possibly halo) index i along an axis of n nodes with
// boundary bc; *mirrored tells whether the normal momentum must be negated.
__device__ __forceinline__ int64_t source_idx(int64_t i, int64_t n, int bc, bool* mirrored)
{
    *mirrored = bc == kBcReflecting && (i < 0 || i >= n);
    if (bc == kBcPeriodic) return wrap_near(i, n);
    if (bc == kBcReflecting) return mirror_idx(i, n);
    return clamp_idx(i, n);
}

}  // namespace lbsd
