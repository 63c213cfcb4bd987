#pragma once
// Wavefront building blocks shared by the 1-D and the square-lattice step
// kernels, whose wavefronts hold one or a few neighbouring nodes per lane and
// exchange packets by lane shifts.  Everything sits in an anonymous namespace:
// each translation unit instantiates its own.
#include <climits>
#include <type_traits>

#include "lb_kernels.hpp"

namespace lbsd {

namespace {

// ---- lane shifts ----------------------------------------------------------
// lshr: lane i gets lane i - 1's value (data moves one column up); lshl: lane
// i gets lane i + 1's.  The end lanes get 0; a chain of at most H shifts
// leaves the destination lanes exact.
__device__ __forceinline__ int dpp_r(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xf, 0xf, true); }
__device__ __forceinline__ int dpp_l(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x130, 0xf, 0xf, true); }
__device__ __forceinline__ float lshr(float v) { return __builtin_bit_cast(float, dpp_r(__builtin_bit_cast(int, v))); }
__device__ __forceinline__ float lshl(float v) { return __builtin_bit_cast(float, dpp_l(__builtin_bit_cast(int, v))); }
struct Words {
    int lo, hi;
};
__device__ __forceinline__ double lshr(double v)
{
    const Words w = __builtin_bit_cast(Words, v);
    return __builtin_bit_cast(double, Words{dpp_r(w.lo), dpp_r(w.hi)});
}
__device__ __forceinline__ double lshl(double v)
{
    const Words w = __builtin_bit_cast(Words, v);
    return __builtin_bit_cast(double, Words{dpp_l(w.lo), dpp_l(w.hi)});
}

// Smallest of the wavefront's values, in every lane's scalar registers: six
// DPP minima (rows of 16, then rows to rows) instead of six trips through the
// LDS permute unit.
__device__ __forceinline__ int wave_min_dpp(int v)
{
#define LB_MIN_STEP(CTRL, ROWS) v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, CTRL, ROWS, 0xf, false))
    LB_MIN_STEP(0x111, 0xf);  // row_shr:1
    LB_MIN_STEP(0x112, 0xf);
    LB_MIN_STEP(0x114, 0xf);
    LB_MIN_STEP(0x118, 0xf);
    LB_MIN_STEP(0x142, 0xa);  // lane 15 of each row to the next row
    LB_MIN_STEP(0x143, 0xc);  // lane 31 to the upper half
#undef LB_MIN_STEP
    return __builtin_amdgcn_readlane(v, 63);
}

// f(0), f(1) .. f(N - 1) with the index as a compile-time constant (register
// arrays indexed by it stay in registers whatever the optimiser does before it
// unrolls loops).
template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<N, I + 1>(f);
    }
}

// At the end of alternatives that differ only in which element of a register
// array they change: an empty statement of its own for each, so that the
// optimiser does not merge them into one that picks the element's address
// (which would move the array to memory).
template <int I>
__device__ __forceinline__ void keep_apart()
{
    asm volatile("; alternative %0" ::"i"(I));
}

__device__ __forceinline__ float fmaT(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmaT(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Whether every moment is finite, rho > 0 and (FP64) every exponent is small
// enough for the quotients of march_node to need no scaling: zero or within
// [2^-511, 2^257), rho and rho E within [2^-255, 2^257).  Integer tests on
// the high words (the same number of instructions as the plain finiteness
// tests); states outside take the general form.
__device__ __forceinline__ bool tame(double m0, double m1, double m2, double m3)
{
    const auto hi = [](double v) { return (uint32_t)(__builtin_bit_cast(uint64_t, v) >> 32); };
    const auto win = [&](double v) { return hi(v) - 0x30000000u < 0x20000000u; };
    const auto zwin = [&](double v) { return (hi(v) & 0x7fffffffu) - 0x20000000u < 0x30000000u || v == 0.0; };
    return win(m0) && zwin(m1) && zwin(m2) && win(m3);
}
__device__ __forceinline__ bool tame(float m0, float m1, float m2, float m3)
{
    const auto b = [](float v) { return __builtin_bit_cast(uint32_t, v); };
    return b(m0) - 1u < 0x7f7fffffu && (b(m1) & 0x7fffffffu) < 0x7f800000u && (b(m2) & 0x7fffffffu) < 0x7f800000u &&
           (b(m3) & 0x7fffffffu) < 0x7f800000u;
}
__device__ __forceinline__ bool zero_or_normal(double v)
{
    const uint32_t h = (uint32_t)(__builtin_bit_cast(uint64_t, v) >> 32);
    return (h & 0x7fffffffu) - 0x20000000u < 0x30000000u || v == 0.0;
}
__device__ __forceinline__ bool zero_or_normal(float v)
{
    return (__builtin_bit_cast(uint32_t, v) & 0x7fffffffu) < 0x7f800000u;
}

// Quotients by one divisor.  FP64 storage: correctly rounded (floor(v) and
// c'_1 then match the plain definition bit for bit).  For tame operands the
// reciprocal (hardware estimate, two Newton steps) is shared between the
// quotients and each takes one correction, RN(q + (a - b q) y): the operations
// of the compiler's own division without its per-quotient scaling, so the
// same bits, at 3 instructions per quotient after 5 for the reciprocal
// against 11 each.  FP32 storage (whose decisions need not match bit for
// bit): one Newton step and a product.
template <bool FAST, bool IEEE>
struct Quot {
    double b, y;
    __device__ __forceinline__ explicit Quot(double d) : b(d), y(0.0)
    {
        if constexpr (!IEEE || FAST) {
            y = __builtin_amdgcn_rcp(d);
            y = __builtin_fma(y, __builtin_fma(-d, y, 1.0), y);
            if constexpr (!FAST) y = __builtin_fma(y, __builtin_fma(-d, y, 1.0), y);
        }
    }
    __device__ __forceinline__ double operator()(double a) const
    {
#pragma clang fp contract(off)
        if constexpr (FAST) {
            return a * y;
        } else if constexpr (IEEE) {
            return a / b;
        } else {
            const double q = a * y;
            return __builtin_fma(__builtin_fma(-b, q, a), y, q);
        }
    }
};

// The largest d_0 / rho for which rho - d_0 keeps enough bits to be a tame
// divisor; rest levels beyond it take the general form.
constexpr double kTameDelta0 = 0.999999;

// Largest displacement of a class along an axis: max(f + 1 + c'_2, c'_2 - f).
__device__ __forceinline__ int class_reach(int F, int C) { return C + 2 + (F < 0 ? -F - 1 : F); }

}  // namespace

}  // namespace lbsd
