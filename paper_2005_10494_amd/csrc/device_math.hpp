// Device-side numerics for the design-objective kernels (gfx950).
//
// The FP64 normal CDF and quantile of the setup kernels come from the device
// math library (ocml: erfc, normcdfinv); the FP64 integrands take the CDF from
// a table in LDS (CdfTable) and 2^x from a polynomial (exp2_fast); the FP32
// normal CDF is a fitted tail form (see norm_cdf(float)); the bivariate normal CDF is evaluated from Plackett's identity
// d Phi_2 / d rho = phi_2 integrated over the angle theta = asin(rho)
// (Drezner & Wesolowsky 1990, as organised by Genz 2004, Stat. Comput. 14:251),
// with a Gauss-Legendre rule whose node count grows with the correlation.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cdf_table.hpp"
#include "exp2_fit.hpp"
#include "mills_fit.hpp"
#include "normal_cdf_fit.hpp"

namespace bmd {

// ---------------------------------------------------------------------------
// Counter-based random numbers: Philox4x32-10 (Salmon et al., SC 2011).
// Round: multiply words 0 and 2 by fixed constants, xor the high halves into
// words 1 and 3 with the key; the key advances by two Weyl constants.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint32_t lo0 = 0xD2511F53u * c.x, hi0 = __umulhi(0xD2511F53u, c.x);
        const uint32_t lo1 = 0xCD9E8D57u * c.z, hi1 = __umulhi(0xCD9E8D57u, c.z);
        c = make_uint4(hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0);
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

// (n + 1/2) * 2^-52 with n the 52-bit integer made of the top 26 bits of each
// word; exact in FP64, strictly inside (0, 1).
__device__ __forceinline__ double uniform52(uint32_t wa, uint32_t wb) {
#pragma clang fp contract(off)
    const uint64_t n = (static_cast<uint64_t>(wa >> 6) << 26) | static_cast<uint64_t>(wb >> 6);
    const double t = static_cast<double>(n) + 0.5;
    return t * 0x1p-52;
}

// Fill u[0..nu) for draw k: block b uses counter (k lo, k hi, scenario, b).
template <int NU>
__device__ __forceinline__ void draw_uniforms(uint64_t k, uint32_t scenario, uint32_t key0,
                                              uint32_t key1, int nu, double* u) {
    uint32_t w[2 * NU + 4];
#pragma unroll
    for (int b = 0; b < (2 * NU + 3) / 4; ++b) {
        if (4 * b < 2 * nu) {
            const uint4 o = philox4x32_10(
                make_uint4(static_cast<uint32_t>(k), static_cast<uint32_t>(k >> 32), scenario,
                           static_cast<uint32_t>(b)),
                key0, key1);
            w[4 * b + 0] = o.x;
            w[4 * b + 1] = o.y;
            w[4 * b + 2] = o.z;
            w[4 * b + 3] = o.w;
        }
    }
#pragma unroll
    for (int i = 0; i < NU; ++i)
        if (i < nu) u[i] = uniform52(w[2 * i], w[2 * i + 1]);
}

// Grid coordinate q_lo + ((q_hi - q_lo) * i) / (m - 1), each step rounded
// (no fused multiply-add: the value must be bit-identical to a plain IEEE
// evaluation in this order).
__device__ __forceinline__ double grid_coord(double q_lo, double q_hi, int64_t i, int m) {
#pragma clang fp contract(off)
    const double span = q_hi - q_lo;
    const double t = (span * static_cast<double>(i)) / static_cast<double>(m - 1);
    return q_lo + t;
}

// lo + (hi - lo) * u, each step rounded (no fused multiply-add).
__device__ __forceinline__ double affine_uniform(double lo, double hi, double u) {
#pragma clang fp contract(off)
    const double span = hi - lo;
    const double x = span * u;
    return lo + x;
}

// Sum over L consecutive lanes (the wavefront by default) by a butterfly; each
// returns the first lane's total.
template <int L = 64>
__device__ __forceinline__ double wave_total(double v) {
#pragma unroll
    for (int off = L / 2; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return __shfl(v, 0, L);
}

// ---------------------------------------------------------------------------
// Univariate normal
// ---------------------------------------------------------------------------
__device__ __forceinline__ double norm_cdf(double x) { return 0.5 * erfc(-x * 0.70710678118654752440); }
// Single precision, argument prescaled: for xs = x sqrt(log2(e)/2) and
// y = |xs|, Phi(-|x|) = r' 2^(P(r') - y^2) with r' = 1/(y + 2 sqrt(log2 e))
// (the hardware reciprocal, within one ulp) and P the degree-7 fit of
// normal_cdf_fit.hpp in r' itself (tail relative error within 3e-6 while the
// tail exceeds 1e-9, max abs error of Phi 5.6e-7, unbiased), signed as
// 1/2 + copysign(1/2 - Phi(-|x|), x).  One reciprocal, one exp2 and twelve
// full-rate operations.  Callers that can fold the factor into constants they
// already hold pass xs directly.  xs must be finite: beyond |x| = 14.8 the
// exponent underflows and Phi saturates to 0 or 1.
__device__ __forceinline__ float norm_cdf_scaled(float xs, float shift = kPhiShift) {
    const float r = __builtin_amdgcn_rcpf(fabsf(xs) + shift);
    float p = kPhiFit[kPhiFitDeg];
#pragma unroll
    for (int i = kPhiFitDeg - 1; i >= 0; --i) p = fmaf(p, r, kPhiFit[i]);
    const float t = fmaf(-r, __builtin_amdgcn_exp2f(fmaf(-xs, xs, p)), 0.5f);   // 1/2 - Phi(-|x|)
    return 0.5f + __builtin_copysignf(t, xs);
}
__device__ __forceinline__ float norm_cdf(float x) { return norm_cdf_scaled(x * kPhiScale); }
__device__ __forceinline__ double norm_pdf(double x) { return 0.39894228040143267794 * exp(-0.5 * x * x); }
__device__ __forceinline__ float norm_pdf(float x) {
    return 0.39894228040143267794f * __builtin_amdgcn_exp2f(-0.72134752044448170368f * x * x);
}

// 2^t in double precision for finite t (NaN stays NaN): t = n + f with n the
// nearest integer, the polynomial of exp2_fit.hpp in f (1.1e-16 relative), the
// power of two by the exponent (0 or infinity outside the range).  15
// operations at four to five SIMD cycles each, against 92 cycles of the
// library's exp, which also handles the special cases with selects.
__device__ __forceinline__ double exp2_fast(double t) {
    const double n = __builtin_rint(t);
    const double f = t - n;
    double p = kExp2Fit[kExp2Deg];
#pragma unroll
    for (int i = kExp2Deg - 1; i >= 0; --i) p = fma(p, f, kExp2Fit[i]);
    return __builtin_amdgcn_ldexp(p, static_cast<int>(n));
}

// 2^t for any t <= 0, -infinity included (NaN stays NaN): where t is a product, the
// compiler contracts it into exp2_fast's t - n, whose result then carries t's own
// rounding, past |t| = 1e44 enough to overflow the polynomial.
__device__ __forceinline__ double exp2_low(double t) { return exp2_fast(t < -2000.0 ? -2000.0 : t); }

// Mills' ratio M(y) = (1 - Phi(y))/phi(y), y >= 0, by the fit of mills_fit.hpp (4e-16
// relative); the reciprocal by two Newton steps.
__device__ __forceinline__ double mills(double y) {
    const double a = fmin(y, 1e9) + kMillsK;
    double r = __builtin_amdgcn_rcp(a);
    r = fma(r, fma(-a, r, 1.0), r);
    r = fma(r, fma(-a, r, 1.0), r);
    const double s = fma(-2.0 * kMillsK, r, 1.0);
    double p = kMillsFit[kMillsDeg];
#pragma unroll
    for (int i = kMillsDeg - 1; i >= 0; --i) p = fma(p, s, kMillsFit[i]);
    return r * p;
}

// A density times Phi(x) with every digit of the lower tail, joint being the
// density times phi(x): joint M(-x), or what is left of the density.  Phi from the
// table below (absolute error 1.2e-16) has few digits there, 4e-11 relative at -5
// and 2e-2 at -8, and the library's erfc costs 346 SIMD cycles a wavefront where this
// takes 35 operations (a gradient call of one biomarker, 4,096 points x 200,000 draws:
// 16.4 ms with erfc, 14.2 here).
__device__ __forceinline__ double density_cdf(double density, double joint, double x) {
    const double v = joint * mills(fabs(x));
    return x < 0.0 ? v : density - v;
}

// Fill a workgroup's table of cdf_table.hpp (every thread of the block calls it;
// the caller synchronises before the first use).
__device__ __forceinline__ void cdf_table_fill(CdfCell* t) {
    for (int j = threadIdx.x; j < kCdfCells; j += blockDim.x) t[j] = cdf_cell(j);
}

// Keep a wave-uniform FP32 value in a vector register: a multiply-add takes 2.5 SIMD
// cycles a wavefront from vector registers or a literal, 4.4 with a scalar
// register operand.  It also takes the value out of the compiler's sight, so only
// kernels that gain call it: the matrix-core sweep's sums from three biomarkers on
// (11^5 designs x 6,000 draws 2.30 -> 2.21 ms; with squares only these five, 2.33 ->
// 2.25, where six lose, 2.18 -> 2.39) and the kernels of three and four
// populations (97 x 97 levels x 100,000 draws 13.65 -> 13.51).  The
// one-design-per-thread sweeps took 14 to 30 registers more (logistic cutoffs, two to
// six biomarkers: 2.78, 9.3, 6.7, 8.9, 8.5 ms against 1.47, 7.0, 5.9, 6.9, 7.0).
__device__ __forceinline__ void pin_vector(float& v) { asm volatile("" : "+v"(v)); }

// Where an integrand's Phi comes from: the FP32 fit, the FP64 table in LDS, or
// (setup kernels) the library.
template <typename T>
struct NormCdf;
template <>
struct NormCdf<float> {
    float shift = kPhiShift;
    __device__ explicit NormCdf(const CdfCell*) {}
    __device__ __forceinline__ void pin() { pin_vector(shift); }
    __device__ __forceinline__ float operator()(float x) const { return norm_cdf(x); }
    __device__ __forceinline__ float scaled(float xs) const { return norm_cdf_scaled(xs, shift); }   // xs = x sqrt(log2(e)/2)
};
template <>
struct NormCdf<double> {
    const CdfCell* t;
    __device__ explicit NormCdf(const CdfCell* table) : t(table) {}
    __device__ __forceinline__ double operator()(double x) const { return norm_cdf_table(x, t); }
    __device__ __forceinline__ double scaled(double x) const { return norm_cdf_table(x, t); }   // FP64 is not prescaled
};
struct LibraryCdf {
    __device__ __forceinline__ double operator()(double x) const { return norm_cdf(x); }
    __device__ __forceinline__ double scaled(double x) const { return norm_cdf(x); }
};
// Cells of the table a kernel in T keeps in static LDS (one unused cell in FP32).
template <typename T>
constexpr int kCdfTableSize = sizeof(T) == 8 ? kCdfCells : 1;

// Phi^-1(p): the library quantile, then one Newton step on a residual that
// keeps relative accuracy (erf form near 1/2, where p - 1/2 is exact; erfc
// forms in the tails, where p or 1 - p is exact).
__device__ __forceinline__ double norm_quantile(double p) {
    const double x = p <= 0.5 ? normcdfinv(p) : -normcdfinv(1.0 - p);
    const double a = p - 0.5;
    double res;
    if (fabs(a) <= 0.25) res = 0.5 * erf(x * 0.70710678118654752440) - a;
    else if (a < 0.0) res = 0.5 * erfc(-x * 0.70710678118654752440) - p;
    else res = (1.0 - p) - 0.5 * erfc(x * 0.70710678118654752440);
    return x - res / norm_pdf(x);
}

// ---------------------------------------------------------------------------
// Bivariate normal CDF with per-design constants.
//
// Phi_2(h,k;rho) = Phi(h) Phi(k) + (1/2pi) int_0^{asin rho}
//                      exp(-(h^2 + k^2 - 2 h k sin t) / (2 cos^2 t)) dt.
// With Gauss-Legendre nodes x_i on [-1,1], s_i = sin(asin(rho)(1 + x_i)/2):
//   integrand_i = exp(b_i h k - a_i (h^2 + k^2)),  a_i = 1/(2 (1 - s_i^2)), b_i = 2 s_i a_i
// (evaluated as a power of two, log2(e) folded into a_i and b_i),
// and the integral is asin(rho)/(4 pi) sum_i w_i integrand_i.
// The per-design constants (a_i, b_i, scale) live in registers; the weights w_i
// belong to the n-point rule shared by the wavefront.
// ---------------------------------------------------------------------------

// Number of Gauss-Legendre nodes for a target accuracy at correlation rho:
// max abs error of the integral <= 1e-14 for FP64 (h, k in [-6, 4]) and
// <= 2e-8 for FP32 (h, k in [-8, 5]), up to rho = 0.975.
__device__ __forceinline__ int bvn_nodes_fp64(double rho) {
    return rho < 0.3 ? 6 : rho < 0.5 ? 8 : rho < 0.75 ? 12 : rho < 0.9 ? 16 : rho < 0.95 ? 20 : 24;
}
__device__ __forceinline__ int bvn_nodes_fp32(double rho) {
    return rho < 0.58 ? 4 : rho < 0.8 ? 6 : rho < 0.91 ? 8 : rho < 0.95 ? 10 : 12;
}

// Offsets of the n-point rules inside the packed Gauss-Legendre table
// (rules for n = 4, 6, 8, 10, 12, 16, 20, 24; x then w, n doubles each).
__device__ __forceinline__ int gl_offset(int n) {
    // 2 * (sum of smaller rule sizes)
    return n == 4 ? 0 : n == 6 ? 8 : n == 8 ? 20 : n == 10 ? 36 : n == 12 ? 56
         : n == 16 ? 80 : n == 20 ? 112 : 152;
}

// A Gauss-Legendre rule is symmetric: nodes p and n - 1 - p share a weight, so
// the constants are held pair by pair (entries 2 p and 2 p + 1) and a pair
// needs one weight.
template <typename T, int NMAX>
struct BvnConst {
    T a[NMAX], b[NMAX];
    T scale;  // asin(rho) / (4 pi)

    // gl: packed table; n: wave-uniform rule size (<= NMAX).  Both precisions
    // evaluate powers of two.  FP32 arguments come prescaled by sqrt(log2(e)/2)
    // (norm_cdf_scaled's), so its exponent coefficients become 1/(1 - s^2) and
    // 2 s/(1 - s^2); FP64 arguments are plain, so it folds log2(e) in.
    __device__ __forceinline__ void init(double rho, int n, const double* __restrict__ gl) {
        const double th = asin(rho);
        scale = static_cast<T>(th * 0.079577471545947667884);  // 1/(4 pi)
        const double* x = gl + gl_offset(n);
#pragma unroll
        for (int i = 0; i < NMAX; ++i) {
            if (i < n) {
                const int node = i % 2 == 0 ? i / 2 : n - 1 - i / 2;
                const double s = sin(0.5 * th * (1.0 + x[node]));
                const double ai = 1.0 / ((1.0 - s) * (1.0 + s));
                constexpr double l2e = 1.4426950408889634074;
                a[i] = static_cast<T>(sizeof(T) == 4 ? ai : 0.5 * l2e * ai);
                b[i] = static_cast<T>(sizeof(T) == 4 ? 2.0 * s * ai : l2e * s * ai);
            } else {
                a[i] = T(0);
                b[i] = T(0);
            }
        }
    }
};

// The same constants of one design kept in memory (wave-uniform addresses, so
// they arrive in scalar registers).
template <typename T>
struct BvnView {
    const T* a;
    const T* b;
    T scale;
};

// The pair weights of a wavefront's rule, read once per design into scalar
// registers.
template <typename T, int NMAX>
struct BvnWeights {
    T w[NMAX / 2];
    __device__ __forceinline__ void load(const T* __restrict__ src, int n) {
#pragma unroll
        for (int i = 0; i < NMAX / 2; ++i) {
            T v = 2 * i < n ? src[i] : T(0);
            if constexpr (sizeof(T) == 8)
                v = __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                                     __builtin_amdgcn_readfirstlane(__double2loint(v)));
            w[i] = v;
        }
    }
    // FP32: into vector registers (see pin_vector).
    __device__ __forceinline__ void pin() {
#pragma unroll
        for (int i = 0; i < NMAX / 2; ++i) pin_vector(w[i]);
    }
    __device__ __forceinline__ T operator[](int i) const { return w[i]; }
};

// Node sums  sum_{i<n} w_i 2^(b_i hk - a_i hs)  of R argument pairs at once.
// Every rule size is even and n is wave-uniform, so the nodes go in pairs
// behind a scalar exit test, unrolled by template recursion: only n nodes are
// evaluated and every coefficient index is a compile-time constant (registers,
// no indexed scratch).  (A guard per node in a loop is if-converted into
// evaluating all NMAX exponentials; a loop with an early exit is kept rolled
// for FP64, its coefficients then indexed in scratch.)  The R sums share the
// tests and give the scheduler independent chains.
__device__ __forceinline__ double node_exp(double x) { return exp2_fast(x); }
__device__ __forceinline__ float node_exp(float x) { return __builtin_amdgcn_exp2f(x); }

// c: BvnConst<T, NMAX>, or a BvnView of constants in memory; w: the pair weights.
template <int I, int NMAX, int R, typename T, typename C, typename W>
__device__ __forceinline__ void bvn_node_pairs(int n, const T (&hk)[R], const T (&hs)[R], const C& c, const W& w,
                                               T (&acc)[R]) {
    // smallest rule: 4 nodes (FP32 table) or 6 (FP64 table); those need no test
    constexpr int kMinRule = sizeof(T) == 4 ? 4 : 6;
    if constexpr (I < NMAX) {
        if (I >= kMinRule && I >= n) return;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const T e0 = node_exp(fma(c.b[I], hk[r], -(c.a[I] * hs[r])));
            const T e1 = node_exp(fma(c.b[I + 1], hk[r], -(c.a[I + 1] * hs[r])));
            acc[r] = I == 0 ? w[0] * (e0 + e1) : fma(w[I / 2], e0 + e1, acc[r]);
        }
        bvn_node_pairs<I + 2, NMAX, R>(n, hk, hs, c, w, acc);
    }
}

// 1 - Phi_2(h_r, k_r; rho) = (1 - scale S_r) - Phi(h_r) Phi(k_r), r < R, S_r the
// node sums: two fused multiply-adds.  FP32 arguments are prescaled
// (norm_cdf_scaled's); cdf: NormCdf<T>, or LibraryCdf in the setup kernels.
template <int NMAX, int R, typename T, typename W, typename Cdf>
__device__ __forceinline__ void bvn_sf_many(const T (&h)[R], const T (&k)[R], const BvnConst<T, NMAX>& c, const W& w,
                                            int n, const Cdf& cdf, T (&sf)[R]) {
    T hk[R], hs[R], acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        hk[r] = h[r] * k[r];
        hs[r] = fma(h[r], h[r], k[r] * k[r]);
        acc[r] = T(0);
    }
    bvn_node_pairs<0, NMAX, R>(n, hk, hs, c, w, acc);
#pragma unroll
    for (int r = 0; r < R; ++r)
        sf[r] = fma(-cdf.scaled(h[r]), cdf.scaled(k[r]), fma(-c.scale, acc[r], T(1)));
}

// Phi_2(h, k; rho), arguments as above.
template <int NMAX, typename T, typename C, typename W, typename Cdf>
__device__ __forceinline__ T bvn_cdf_scaled(T h, T k, const C& c, const W& w, int n, const Cdf& cdf) {
    const T hk[1] = {h * k}, hs[1] = {fma(h, h, k * k)};
    T acc[1] = {T(0)};
    bvn_node_pairs<0, NMAX, 1>(n, hk, hs, c, w, acc);
    return fma(cdf.scaled(h), cdf.scaled(k), c.scale * acc[0]);
}
// Plain arguments in both precisions.
template <int NMAX, typename T, typename C, typename W, typename Cdf>
__device__ __forceinline__ T bvn_cdf(T h, T k, const C& c, const W& w, int n, const Cdf& cdf) {
    if constexpr (sizeof(T) == 4)
        return bvn_cdf_scaled<NMAX>(h * kPhiScale, k * kPhiScale, c, w, n, cdf);
    else
        return bvn_cdf_scaled<NMAX>(h, k, c, w, n, cdf);
}

// Row of the 16x16 result held in accumulator element v of a lane in quarter
// kq = lane / 16 (the column is lane % 16).  Operands: lane l supplies A[l%16][l/16]
// and B[l/16][l%16].  The FP32 16x16x4 instruction gives each quarter four
// consecutive rows; the FP64 one interleaves them with stride 4.
template <typename T>
__device__ __forceinline__ int mfma16_row(int kq, int v) {
    return sizeof(T) == 8 ? kq + 4 * v : 4 * kq + v;
}

}  // namespace bmd
