// The FP64 normal CDF of the integrands, from a table of cells.  No device
// built-ins: a host compiler takes this header as it is, with the qualifiers
// __host__, __device__ and __forceinline__ defined away.
#pragma once
#include <math.h>
#include <stdint.h>

namespace bmd {

// The FP64 integrands' Phi from a table in LDS: cell j holds
// (Phi(x_j) - 1/2, phi(x_j)) at x_j = j / 64, and with d = |x| - x_j, u = x_j d,
// v = d^2 (|d| <= 1/128) the Taylor series of the integral of phi from x_j,
//   Phi(|x|) - 1/2 = F_j + phi_j d sum_n (-1)^n He_n(x_j) d^n / (n + 1)!,
// is summed through n = 5 as a polynomial in u whose coefficients are
// polynomials in v; the first term left out is below 6e-18.  Beyond the last
// cell (x = 8.5, Phi = 1 to rounding) its density is taken as 0.  Absolute
// error 1.2e-16: enough where Phi, or an integral of it, is subtracted from 1,
// but not where Phi is a factor of the result (the derivatives: density_cdf).
// Why a table: the library's erfc costs 346 SIMD
// cycles a wavefront, this 22 operations of four to five and one 16-byte LDS
// read; without a division or an exponential there is nothing left to branch
// on.  A cell of 1/64 needs two polynomial terms fewer than 1/32 and keeps the
// table at 8.7 KB.  Infinite x gives 0 or 1; a NaN is clamped like a large
// value, so callers whose designs may have no critical value mask their sums.
struct alignas(16) CdfCell {
    double F, p;
};
constexpr int kCdfPerUnit = 64;
constexpr int kCdfCells = 8 * kCdfPerUnit + kCdfPerUnit / 2 + 1;   // x_j = 0 .. 8.5

__host__ __device__ __forceinline__ CdfCell cdf_cell(int j) {
    const double x = static_cast<double>(j) / kCdfPerUnit;
    return {0.5 * erf(x * 0.70710678118654752440),
            j < kCdfCells - 1 ? 0.39894228040143267794 * exp(-0.5 * x * x) : 0.0};
}

__host__ __device__ __forceinline__ double norm_cdf_table(double x, const CdfCell* t) {
    // adding 1.5 * 2^52 / 64 rounds to a multiple of 1/64 and leaves its index in the low word
    constexpr double kRound = 6755399441055744.0 / kCdfPerUnit;
    const double y = fmin(fabs(x), static_cast<double>(kCdfCells - 1) / kCdfPerUnit);
    const double s = y + kRound;
    const CdfCell c = t[static_cast<uint32_t>(__builtin_bit_cast(uint64_t, s))];
    const double xj = s - kRound;
    const double d = y - xj;
    const double u = xj * d, v = d * d;
    const double c0 = fma(v, fma(v, 1.0 / 40.0, -1.0 / 6.0), 1.0);
    const double c1 = fma(v, fma(v, -1.0 / 48.0, 1.0 / 8.0), -0.5);
    const double c2 = fma(v, -1.0 / 20.0, 1.0 / 6.0);
    const double c3 = fma(v, 1.0 / 72.0, -1.0 / 24.0);
    double q = fma(u, -1.0 / 720.0, 1.0 / 120.0);
    q = fma(u, q, c3);
    q = fma(u, q, c2);
    q = fma(u, q, c1);
    q = fma(u, q, c0);
    return 0.5 + copysign(fma(c.p * d, q, c.F), x);
}

}  // namespace bmd
