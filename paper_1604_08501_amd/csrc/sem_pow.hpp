// FP64 x^gamma by tables in LDS, for kernels that can spare 2 KB of it.
//
// Tang's table-driven scheme ("Table-driven implementation of the logarithm /
// exponential function in IEEE floating-point arithmetic", ACM TOMS 1990 and
// 1989): x = 2^e m with m in [1/2, 1), i the six bits below m's leading one
// and c_i ~ 1/m from a table, r = m c_i - 1, |r| < 2^-7, so
//   log2 x = (e - log2 c_i) + log2(1 + r),
// the second term a short Taylor polynomial.  y = gamma log2 x is kept as the
// rounded product plus a correction (the roundings of the sum and the product
// recovered by a fast two-sum and an FMA), y = n/64 + f with n whole, and
//   2^y = 2^(n >> 6) 2^((n & 63) / 64) 2^f,
// the middle factor from a table together with its own rounding error.
// About 38 instructions, half of exp(gamma log x) with a polynomial log and
// the library's exp, and fewer registers.  Error against 80-bit powl, gamma =
// 1.4, 4e6 arguments each, in units of 2^-53 relative, largest and rms: 1.5
// and 0.48 on [0.6, 1.1] (an atmosphere's R Theta / p0; the other: 2.7, 0.55),
// 1.5 and 0.48 on [250, 350] (9.6, 3.6), 1.5 and 0.46 on [1e-30, 1e30] (66,
// 24).
#pragma once
#include "sem_device.hpp"

namespace semk {

#include "sem_pow_tables.inc"

constexpr int kPowTableValues = 256;   // doubles: {c, -log2 c} x 64, {2^(j/64), error} x 64

// Physical constants with the tables staged in LDS.
struct PowPhys : Phys {
    const double* tab;
};

// Place of the tables behind n values of LDS: two values are written at a time.
constexpr int pow_tables_at(int n)
{
    return (n + 1) & ~1;
}

// The tables to smem + AT (smem: 16-byte aligned), by NT lanes.
template <int NT, int AT>
__device__ __forceinline__ void stage_pow_tables(double* __restrict__ smem)
{
    static_assert(AT % 2 == 0, "the tables are written 16 bytes at a time");
    typedef double double2_t __attribute__((ext_vector_type(2)));
    double* __restrict__ tab = smem + AT;
    for (int x = threadIdx.x; x < kPowTableValues / 2; x += NT)
        reinterpret_cast<double2_t*>(tab)[x] =
            reinterpret_cast<const double2_t*>(kPowTables)[x];
}

// x^gamma for 0 < x < inf (any other x: see pow_special)
__device__ __forceinline__ double pow_table(double x, const PowPhys& ph)
{
    const double m = __builtin_amdgcn_frexp_mant(x);   // [1/2, 1), subnormals too
    const double e = (double)__builtin_amdgcn_frexp_exp(x);
    const int i = (int)(__builtin_bit_cast(unsigned long long, m) >> 46) & 63;
    const double c = ph.tab[2 * i], t = ph.tab[2 * i + 1];
    const double r = fma(m, c, -1.0);
    // log2(1 + r) / r by its Taylor series, 1 / (n ln 2) with alternating signs
    constexpr double k1 = 0x1.71547652b82fep+0, k3 = 0x1.ec709dc3a03fdp-2,
                     k5 = 0x1.2776c50ef9bfep-2, k7 = 0x1.a61762a7aded9p-3;
    const double r2 = r * r;
    const double p01 = fma(-0.5 * k1, r, k1), p23 = fma(-0.25 * k1, r, k3),
                 p45 = fma(-0.5 * k3, r, k5);
    const double p = fma(fma(fma(k7, r2, p45), r2, p23), r2, p01);
    const double s = e + t;
    const double lo2 = fma(p, r, t - (s - e));   // |e| >= |t| or e = 0: the sum's rounding
    const double yh = ph.gamma * s;
    const double yl = fma(ph.gamma, lo2, fma(ph.gamma, s, -yh));
    const double n = __builtin_rint((yh + yl) * 64.0);
    const double f = fma(n, -1.0 / 64.0, yh) + yl;
    const int ni = (int)n;
    const int j = ni & 63;
    const double E = ph.tab[128 + 2 * j], dE = ph.tab[129 + 2 * j];
    // 2^f = 1 + f (ln 2 + ...), to f^6
    constexpr double l1 = 0x1.62e42fefa39efp-1, l2 = 0x1.ebfbdff82c58fp-3,
                     l3 = 0x1.c6b08d704a0c0p-5, l4 = 0x1.3b2ab6fba4e77p-7,
                     l5 = 0x1.5d87fe78a6731p-10, l6 = 0x1.430912f86c787p-13;
    const double f2 = f * f;
    const double w = fma(fma(fma(l6, f, l5), f2, fma(l4, f, l3)), f2, fma(l2, f, l1));
    return __builtin_amdgcn_ldexp(fma(E, fma(w, f, dE), E), ni >> 6);
}

__device__ __forceinline__ bool pow_regular(double x)
{
    return __builtin_amdgcn_class(x, 0x180);   // positive, subnormal or normal
}

// exp(gamma log x) at 0, +inf, negative x and NaN
__device__ __forceinline__ double pow_special(double x, double gamma)
{
    const double l = x == 0.0 ? -__builtin_inf() : (x > 0.0 ? x : __builtin_nan(""));
    const double y = gamma * l;
    return y < 0.0 ? 0.0 : (y > 0.0 ? y : __builtin_nan(""));
}

// the flux pressure (the perturbation when there is a reference) and the full
// pressure, as Pressure<double>::eval_full
__device__ __forceinline__ void table_pressure(double Th, bool has_ref, double thr,
                                               const PowPhys& ph, double& pflux, double& pfull)
{
    const double a = ph.r_over_p0 * Th, b = ph.r_over_p0 * thr;
    double x = pow_table(a, ph);
    double xr = has_ref ? pow_table(b, ph) : 0.0;
    if (__builtin_expect(!(pow_regular(a) && (!has_ref || pow_regular(b))), 0)) {
        if (!pow_regular(a))
            x = pow_special(a, ph.gamma);
        if (has_ref && !pow_regular(b))
            xr = pow_special(b, ph.gamma);
    }
    pfull = ph.p0 * x;
    pflux = ph.p0 * (x - xr);
}

}  // namespace semk
