// Objective and gradient at continuous design points (the differentiation
// form): d obj / d q_j and d obj / d (mu_b0, mu_b1), averaged over the prior
// draws, which the draw kernel writes to HBM in passes.
//
// Per (point, draw) the summand is f = 1 - Phi_2(h, k; rho) with
//   h = z1 - sqrt(I) (b0 + b1 P(R)),  k = z2 - sqrt(r I) (b0 + b1 O / r),  rho = sqrt(r),
// and its adjoint is propagated through
//   dPhi_2/dh = phi(h) Phi((k - rho h)/s),  dPhi_2/dk = phi(k) Phi((h - rho k)/s),
//   dPhi_2/drho = phi_2(h, k; rho),  s = sqrt(1 - rho^2)   (Plackett),
// the overlap O (logistic or exact cutoff indicator, leave-one-out products
// over the Gauss-Hermite nodes), the subgroup fraction r(q) and the equal-FWER
// critical value z*(r) (implicit derivative of Formula 2).
#include <algorithm>
#include <cstdlib>

#include "bmd_internal.hpp"
#include "device_math.hpp"

namespace bmd {
namespace {

constexpr int kGradThreads = 256;   // four wavefronts, over points and draws

// What the gradient kernel reads of a point.  FP64: validity, cutoffs, rule
// size.  T: the constants below, then the bivariate rule's a[NMAX], b[NMAX].
constexpr int kInfoFields = 9;      // 0 valid, 1..6 q_j, 7 Gauss-Legendre nodes, 8 rho
enum { kZ1, kZ2, kSrI, kInvR, kRho, kISig, kVV, kScale, kDA, kDZ = kDA + kMaxDim, kUU = kDZ + kMaxDim,
       kWW = kUU + kMaxDim, kRecHead = kWW + kMaxDim };
template <typename T>
constexpr int kGradNmax = sizeof(T) == 8 ? 24 : 12;
template <typename T>
constexpr int kGradNodeBlock = 2;   // nodes loaded ahead together
template <typename T>
constexpr int kRecSize = kRecHead + 2 * kGradNmax<T>;

// Common critical value with family-wise error alpha0 at null correlation rho
// (Formula 2 for two tests), as the design precompute: F(z) = 2 Phi(-z) -
// Phi_2(-z, -z; rho) - alpha0 falls in z; safeguarded Newton inside [z(alpha0),
// z(alpha0 / 2)].  Phi_2 by the largest rule, its 24 nodes on the point's L
// lanes (node constants formed once); every value the same on all of them.
template <int L>
__device__ double zstar_lanes(double rho, double alpha0, const double* __restrict__ gl, int lane) {
    constexpr int n = 24, N = (n + L - 1) / L;
    const double* x = gl + gl_offset(n);
    const double th = asin(rho);
    double e[N], w[N];   // the lane's nodes: w exp(e z^2), e = -1 / (1 + s)
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int at = lane + i * L;
        e[i] = w[i] = 0.0;
        if (at < n) {
            e[i] = -1.0 / (1.0 + sin(0.5 * th * (1.0 + x[at])));
            w[i] = x[n + at] * (th * 0.079577471545947667884);
        }
    }
    double lo = -norm_quantile(alpha0), hi = -norm_quantile(0.5 * alpha0);
    double z = 0.5 * (lo + hi);
    const double c = sqrt((1.0 - rho) / (1.0 + rho));
    for (int it = 0; it < 60; ++it) {
        const double t = norm_cdf(-z);
        double nodes = 0.0;
#pragma unroll
        for (int i = 0; i < N; ++i) nodes += w[i] * exp(e[i] * (z * z));
        const double F = 2.0 * t - (t * t + wave_total<L>(nodes)) - alpha0;
        if (F > 0.0) lo = z; else hi = z;
        const double dF = -2.0 * norm_pdf(z) * norm_cdf(z * c);
        double zn = z - F / dF;
        if (!(zn > lo && zn < hi)) zn = 0.5 * (lo + hi);
        const double step = fabs(zn - z);
        z = zn;
        if (step <= 4e-16 * z || hi - lo <= 4e-16 * z) break;
    }
    return z;
}

// Node i's constants of the n-point bivariate rule at correlation rho, in
// BvnConst's pair order (0 past the rule's end).
template <typename T>
__device__ __forceinline__ void rule_constants(double rho, int n, int i, const double* __restrict__ gl, T* a, T* b) {
    *a = *b = T(0);
    if (i >= n) return;
    const int node = i % 2 == 0 ? i / 2 : n - 1 - i / 2;
    const double s = sin(0.5 * asin(rho) * (1.0 + gl[gl_offset(n) + node]));
    const double ai = 1.0 / ((1.0 - s) * (1.0 + s));
    constexpr double l2e = 1.4426950408889634074;
    *a = static_cast<T>(sizeof(T) == 4 ? ai : 0.5 * l2e * ai);
    *b = static_cast<T>(sizeof(T) == 4 ? 2.0 * s * ai : l2e * s * ai);
}

// FP32 only, one thread per point and node (blockIdx.y): `share` consecutive
// points (a power of two up to a wavefront) take the largest of their node
// counts.  A count at the upper end of its range of rho is 1e-8 off, which the
// FP32 values show; a neighbour's larger count takes that away (7e-10 of the
// objective over 512 points).
__global__ __launch_bounds__(256) void k_grad_rule(int64_t b0, int64_t B, int share, const double* __restrict__ gl,
                                                   double* __restrict__ info, float* __restrict__ rec) {
    const int64_t bw = b0 + static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int64_t b = bw < B ? bw : B - 1;
    const int i = blockIdx.y;
    const double rho = info[b * kInfoFields + 8];
    int n = bvn_nodes_fp32(rho);
    for (int off = share / 2; off > 0; off >>= 1) n = max(n, __shfl_xor(n, off));
    if (bw >= B) return;
    if (i == 0) info[b * kInfoFields + 7] = n;
    float* f = rec + b * kRecSize<float> + kRecHead + i;
    rule_constants<float>(rho, n, i, gl, f, f + kGradNmax<float>);
}

// L lanes per point: subgroup fraction r and its q-derivatives (the lanes
// share the Gauss-Hermite nodes), critical values (the lanes share the bivariate
// rule), the constants of the gradient kernel, and the node table
// AD[b][m][j] = (A_jm, d A_jm / d q_j), A_jm = Phi(a_jm), a_jm = (sqrt(rho_b)
// x_m - c_j)/sqrt(1 - rho_b), weights folded into j = 0.  (One thread per
// point walked 128 nodes of up to six CDFs seven times over and the node
// tables in turn: 1.7 ms however few the points; a wavefront each takes 50 us
// for 8, 104 for 2,048.)  L = 64 keeps the latency of few points low as long as
// its workgroups of four points have a compute unit each; beyond that 16 lanes waste
// less on the values that all of them form alike.  A call of 100 draws, 64 / 16 lanes,
// FP64, one and five biomarkers: 1,024 points 94 / 100 and 148 / 171 us, 1,536 points
// 109 / 100 and 172 / 167, 4,096 points 157 / 104 and 275 / 218.
template <typename T, int L>
__global__ __launch_bounds__(256) void k_grad_points(DevProblem P, const double* __restrict__ q_in, int64_t b0, int64_t B,
                                                     const double* __restrict__ ghp, int Kp,
                                                     const double* __restrict__ gh, int K,
                                                     const double* __restrict__ gl, double* __restrict__ info,
                                                     T* __restrict__ rec, T* __restrict__ AD) {
    const int64_t bw = b0 + (static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x) / L;
    const bool inside = bw < B;
    const int64_t b = inside ? bw : B - 1;   // lanes past the end shadow the last point (and store nothing)
    const int lane = threadIdx.x & (L - 1);
    const int d = P.d;
    double q[kMaxDim], c[kMaxDim], dens[kMaxDim];
    bool valid = true;
#pragma unroll
    for (int j = 0; j < kMaxDim; ++j) {
        q[j] = j < d ? q_in[b * d + j] : 0.5;
        // grid endpoints may round a few ulp past q_lo / q_hi
        valid = valid && (j >= d || (q[j] >= P.q_lo - 1e-12 && q[j] <= P.q_hi + 1e-12));
        if (!valid) q[j] = P.q_lo;
    }
    double mine = q[0];
#pragma unroll
    for (int j = 1; j < kMaxDim; ++j) mine = lane == j ? q[j] : mine;
    const double cl = norm_quantile(mine), dl = norm_pdf(cl);   // lane j: axis j
#pragma unroll
    for (int j = 0; j < kMaxDim; ++j) {
        c[j] = __shfl(cl, j, L);
        dens[j] = __shfl(dl, j, L);
    }
    double r = 0.0, dr[kMaxDim];
#pragma unroll
    for (int j = 0; j < kMaxDim; ++j) dr[j] = 0.0;
    if (d == 1) {
        r = 1.0 - q[0];
        dr[0] = -1.0;
    } else {
        for (int m = lane; m < Kp; m += L) {
            const double t = P.sr * ghp[m];
            double cd[kMaxDim], pd[kMaxDim], pre[kMaxDim + 1];
            pre[0] = ghp[Kp + m];
#pragma unroll
            for (int j = 0; j < kMaxDim; ++j) {
                const double a = (t - c[j]) / P.sq;
                cd[j] = j < d ? norm_cdf(a) : 1.0;
                pd[j] = j < d ? norm_pdf(a) : 0.0;
                pre[j + 1] = pre[j] * cd[j];
            }
            r += pre[kMaxDim];
            double suf = 1.0;
#pragma unroll
            for (int j = kMaxDim - 1; j >= 0; --j) {
                dr[j] += pd[j] * (pre[j] * suf);
                suf *= cd[j];
            }
        }
        r = wave_total<L>(r);
#pragma unroll
        for (int j = 0; j < kMaxDim; ++j)
            if (j < d) dr[j] = -wave_total<L>(dr[j]) / P.sq / dens[j];
    }
    const double rho = sqrt(r);
    double z1, z2, dzdrho = 0.0;
    if (P.alpha_rule == BMD_ALPHA_FWER_EQUAL) {
        z1 = z2 = zstar_lanes<L>(rho, P.alpha0, gl, lane);
        // Formula 2 held fixed: dz*/drho = -phi_2(z,z;rho) / (2 phi(z) Phi(z sqrt((1-rho)/(1+rho))))
        const double om = (1.0 - rho) * (1.0 + rho);
        const double pd2 = exp(-z1 * z1 / (1.0 + rho)) / (2.0 * M_PI * sqrt(om));
        dzdrho = -pd2 / (2.0 * norm_pdf(z1) * norm_cdf(z1 * sqrt((1.0 - rho) / (1.0 + rho))));
    } else {
        z1 = P.zf1;
        z2 = P.zf2;
    }
    const int n = bvn_nodes_fp64(rho);
    T* f = rec + b * kRecSize<T>;
    if (lane == 0 && inside) {
        double* in = info + b * kInfoFields;
        in[0] = valid ? 1.0 : 0.0;
        if constexpr (sizeof(T) == 8) in[7] = n;
        in[8] = rho;
        f[kZ1] = static_cast<T>(z1);
        f[kZ2] = static_cast<T>(z2);
        f[kSrI] = static_cast<T>(sqrt(r * P.info));
        f[kInvR] = static_cast<T>(1.0 / r);
        f[kRho] = static_cast<T>(rho);
        f[kISig] = static_cast<T>(1.0 / sqrt((1.0 - rho) * (1.0 + rho)));
        f[kVV] = static_cast<T>(P.sqrtI / rho);
        f[kScale] = static_cast<T>(asin(rho) * 0.079577471545947667884);   // BvnConst's 1/(4 pi)
#pragma unroll
        for (int j = 0; j < kMaxDim; ++j) {
            const double drho = dr[j] / (2.0 * rho);
            in[1 + j] = q[j];
            f[kDA + j] = static_cast<T>(drho);
            f[kDZ + j] = static_cast<T>(dzdrho * drho);
            f[kUU + j] = static_cast<T>(P.sqrtI * dr[j] / (2.0 * rho));
            f[kWW + j] = static_cast<T>(P.sqrtI * dr[j] / (2.0 * r * rho));
        }
    }
    if constexpr (sizeof(T) == 8)   // FP32: k_grad_rule
        for (int i = lane; i < kGradNmax<T>; i += L) {
            T ca, cb;
            rule_constants<T>(rho, n, i, gl, &ca, &cb);
            if (inside) {
                f[kRecHead + i] = ca;
                f[kRecHead + kGradNmax<T> + i] = cb;
            }
        }
    if (d >= 2) {
        for (int e0 = 0; e0 < d * K; e0 += L) {   // every lane stays for the shuffles
            const int e = e0 + lane, m = min(e / d, K - 1), j = e % d;
            const double cj = __shfl(cl, j, L), dj = __shfl(dl, j, L);
            if (e >= d * K || !inside) continue;
            const double a = (P.sr * gh[m] - cj) / P.sq;
            const double wf = j == 0 ? gh[K + m] : 1.0;
            T* o = AD + (b * K * d + e) * 2;
            o[0] = static_cast<T>(wf * norm_cdf(a));
            o[1] = static_cast<T>(-wf * norm_pdf(a) / P.sq / dj);
        }
    }
}

// Logistic 1/(1 + e^-x); FP32 with the hardware exp2 and reciprocal.
__device__ __forceinline__ double lgst(double x) { return 1.0 / (1.0 + exp2_fast(-1.4426950408889634074 * x)); }
__device__ __forceinline__ float lgst(float x) {
    return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634074f * x));
}
// e^x, x <= 0; FP32 with the hardware exp2.
__device__ __forceinline__ double expT(double x) { return exp2_low(1.4426950408889634074 * x); }
__device__ __forceinline__ float expT(float x) { return __builtin_amdgcn_exp2f(1.4426950408889634074f * x); }
__device__ __forceinline__ double norm_pdf_fast(double x) {
    return 0.39894228040143267794 * exp2_low(x * x * -0.72134752044448170368);
}
__device__ __forceinline__ float norm_pdf_fast(float x) { return norm_pdf(x); }

template <typename T>
struct GradArgs {
    DevProblem P;
    int64_t B;
    int64_t M;
    int K;
    int64_t slice_len;
    int64_t slice0;        // first draw slice of this launch (a pass over draws)
    int64_t slices;        // slices of this launch
    int64_t group0, groups;   // workgroup rows of points (pw * PP points each) of this launch
    int pw;                // wavefronts of a workgroup along the points (1, 2 or 4); the others along the draws
    bool by_xcd;           // workgroup numbering: see k_grad
    int64_t draw_k0;       // first draw held by the draw arrays of this pass
    double* partials;      // [n_slices][d+3][B]
};

// One draw per lane, PP points at a time: the lanes of a wavefront hold 64
// consecutive draws, whose node tables (draw index fastest) load coalesced,
// and a point's constants and node table are wave-uniform scalar loads.  Per
// (node m, point), with mix_j = b_j + s_j (a_j - b_j) and L_j the product of the
// other axes' mixes,
//   O += prod_j mix_j,  U_j += (a_j - b_j) L_j,  V_j += a'_j L_j,
// and d O / d q_j = s'_j U_j + s_j V_j after the nodes: 6 D operations a node.
// FP32 adds (s'_j (a_j - b_j) + s_j a'_j) L_j node by node, 7 D operations: the
// rounding of V_j is the same for every draw whose other axes have s = 1, so it
// does not average out over the draws (4e-9 of the gradient).
// A workgroup takes one slice of draws and one row of points: its wavefronts
// hold different points and the same draws, so that the node tables come from
// the L1 for all but the first (from the L2 for every pair of points they
// limited the kernel at 9.4 TB/s); with fewer points than that the
// wavefronts split the draws.  A wavefront's sums go through its lanes by a
// butterfly, draw wavefronts are added in order through LDS.
// Workgroups reach the XCDs round-robin; with `by_xcd` the rows of one slice
// get consecutive numbers on one XCD, so that its L2 reads the slice's node
// tables once.
// Bound: vector issue (scalar operands of FP32 operations cost 4.4 cycles in
// place of 2.5, on 2 of the 6).  With one point per lane and the draws staged
// through LDS, as before, every (node, axis) cost an LDS broadcast a draw and
// two table loads a pass, and few points left the staging exposed.
// Measured, d = 5: 2,048 points x 500,000 draws FP32 a call of 35.1 -> 27.4 ms; 8 points x
// 200,000 draws FP64 1,056 -> 260 us.
// FP64 is held to 168 registers, three wavefronts per SIMD (a refinement call 2.00 ->
// 1.90 ms against two); six biomarkers, which would spill 276 bytes a thread,
// take two (256 points x 50,000 draws: 2.50 -> 1.62 ms).  FP32 with six takes three in
// place of two, 143 registers (1,024 points x 1e6 draws 60.8 -> 48.3 ms; four spill, 52.3).
template <typename T, int D, int PP>
__global__ __launch_bounds__(kGradThreads, sizeof(T) == 8 ? (D == 6 ? 2 : 3) : D == 6 ? 3 : 1) void k_grad(GradArgs<T> a, const double* __restrict__ info,
                                                       const T* __restrict__ rec, const T* __restrict__ AD,
                                                       const T* __restrict__ glw, DrawArrays<T> Dr) {
    constexpr int NMAX = kGradNmax<T>;
    constexpr int NS = D + 3;   // sums per point: objective, d q_j, d mu_b0, d mu_b1
    constexpr bool kSplit = sizeof(T) == 8;
    __shared__ CdfCell cells[kCdfTableSize<T>];
    __shared__ double red[kGradThreads / 64][PP * NS];
    int64_t slice, group;
    if (a.by_xcd) {
        const uint32_t i = blockIdx.x >> 3, gr = static_cast<uint32_t>(a.groups);
        slice = static_cast<int64_t>(i / gr) * 8 + (blockIdx.x & 7);
        group = i % gr;
        if (slice >= a.slices) return;   // the whole workgroup
    } else {
        slice = blockIdx.y;
        group = blockIdx.x;
    }
    group += a.group0;
    if constexpr (sizeof(T) == 8) {
        cdf_table_fill(cells);
        __syncthreads();
    }
    NormCdf<T> cdf(cells);
    if constexpr (sizeof(T) == 4) cdf.pin();
    const DevProblem& P = a.P;
    const int K = a.K;
    const T sI = static_cast<T>(P.sqrtI);
    const bool logistic = P.width > 0.0;
    const double iw64 = logistic ? 1.0 / P.width : 0.0;
    const T iw = static_cast<T>(iw64);
    const double sw64 = fmin(iw64, 1e30);   // as sharp, and finite through exp2_fast (see exp2_low)
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int dw = kGradThreads / 64 / a.pw;
    const int64_t first = (group * a.pw + wave % a.pw) * PP;   // this wavefront's points
    int64_t b[PP];
#pragma unroll
    for (int p = 0; p < PP; ++p) b[p] = min(first + p, a.B - 1);   // past the end: the last point again

    double sum[PP][NS];
#pragma unroll
    for (int p = 0; p < PP; ++p)
#pragma unroll
        for (int i = 0; i < NS; ++i) sum[p][i] = 0.0;

    const int64_t kb = (a.slice0 + slice) * a.slice_len;
    const int64_t ke = min(a.M, kb + a.slice_len);
    for (int64_t k = kb + 64 * (wave / a.pw) + lane; k < ke; k += 64 * dw) {
        const int64_t kk = k - a.draw_k0;
        T O[PP], U[PP][D], V[PP][D], s[PP][D];   // kSplit: the sums; else U is d O / d q_j, V is s'_j
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const double tau = Dr.tau[j * Dr.M + kk];
#pragma unroll
            for (int p = 0; p < PP; ++p) {
                const double dq = info[b[p] * kInfoFields + 1 + j] - tau;
                s[p][j] = logistic ? lgst(static_cast<T>(dq * sw64)) : dq > 0.0 ? T(1) : T(0);
                U[p][j] = T(0);
                V[p][j] = kSplit || !logistic ? T(0) : s[p][j] * (T(1) - s[p][j]) * iw;
            }
        }
#pragma unroll
        for (int p = 0; p < PP; ++p) O[p] = T(0);
        if constexpr (D == 1) {
            const double tau64 = Dr.tau[kk];
            const T tau = static_cast<T>(tau64);
#pragma unroll
            for (int p = 0; p < PP; ++p) {   // O and its derivative in closed form
                const double q64 = info[b[p] * kInfoFields + 1];
                const T q0 = static_cast<T>(q64);
                O[p] = logistic ? T(1) - fma(s[p][0], q0, (T(1) - s[p][0]) * tau) : s[p][0] > T(0) ? T(1) - q0 : T(1) - tau;
                const T du = -static_cast<T>(q64 - tau64);
                U[p][0] = kSplit ? du : fma(V[p][0], du, -s[p][0]);
                if constexpr (kSplit) V[p][0] = T(-1);
            }
        } else {
            // node rows by a uniform base and the lane's byte offset (grad_plan_of keeps it
            // below 2^32); the next block of nodes is in flight while one is used
            constexpr int NB = kGradNodeBlock<T>;
            const uint32_t off = static_cast<uint32_t>(kk) * static_cast<uint32_t>(sizeof(T));
            const auto load = [&](int m0, T (&to)[NB][D]) {
#pragma unroll
                for (int i = 0; i < NB; ++i)
#pragma unroll
                    for (int j = 0; j < D; ++j)
                        to[i][j] = *reinterpret_cast<const T*>(
                            reinterpret_cast<const char*>(Dr.B + (static_cast<int64_t>(m0 + i) * D + j) * Dr.M) + off);
            };
            T cur[NB][D], nxt[NB][D];
            load(0, nxt);
            for (int m0 = 0; m0 < K; m0 += NB) {   // K is a multiple of 4
#pragma unroll
                for (int i = 0; i < NB; ++i)
#pragma unroll
                    for (int j = 0; j < D; ++j) cur[i][j] = nxt[i][j];
                load(min(m0 + NB, K - NB), nxt);
#pragma unroll
                for (int i = 0; i < NB; ++i)
#pragma unroll
                    for (int p = 0; p < PP; ++p) {
                        const T* ad = AD + (b[p] * K + m0 + i) * (2 * D);
                        T dif[D], mix[D], pre[D];
#pragma unroll
                        for (int j = 0; j < D; ++j) {
                            dif[j] = ad[2 * j] - cur[i][j];
                            mix[j] = fma(s[p][j], dif[j], cur[i][j]);
                        }
                        pre[0] = T(1);
#pragma unroll
                        for (int j = 1; j < D; ++j) pre[j] = j == 1 ? mix[0] : pre[j - 1] * mix[j - 1];
                        O[p] = fma(pre[D - 1], mix[D - 1], O[p]);
                        T suf = T(1);
#pragma unroll
                        for (int j = D - 1; j >= 0; --j) {
                            const T L = j == D - 1 ? pre[j] : j == 0 ? suf : pre[j] * suf;
                            if constexpr (kSplit) {
                                U[p][j] = fma(dif[j], L, U[p][j]);
                                V[p][j] = fma(ad[2 * j + 1], L, V[p][j]);
                            } else {
                                U[p][j] = fma(fma(V[p][j], dif[j], s[p][j] * ad[2 * j + 1]), L, U[p][j]);
                            }
                            suf = j == D - 1 ? mix[j] : suf * mix[j];
                        }
                    }
            }
        }
        const T b0 = Dr.b0[kk], b1 = Dr.b1[kk], PR = Dr.PR[kk], mu1 = Dr.mu1[kk];
#pragma unroll
        for (int p = 0; p < PP; ++p) {
            const T* f = rec + b[p] * kRecSize<T>;
            const int n = __builtin_amdgcn_readfirstlane(static_cast<int>(info[b[p] * kInfoFields + 7]));
            const T* w = glw + gl_offset(n) + n;
            const T srI = f[kSrI], invr = f[kInvR], rhoT = f[kRho], isig = f[kISig], vv = f[kVV];
            const T mu2 = srI * (b0 + b1 * O[p] * invr);
            const T h = f[kZ1] - mu1, kq = f[kZ2] - mu2;
            T pc, ph, pk, pr;
            if (P.zinf == 0) {
                const BvnView<T> bc{f + kRecHead, f + kRecHead + NMAX, f[kScale]};
                pc = bvn_cdf<NMAX>(h, kq, bc, w, n, cdf);
                const T u = (kq - rhoT * h) * isig, v = (h - rhoT * kq) * isig;
                ph = norm_pdf_fast(h);
                pk = norm_pdf_fast(kq);
                if constexpr (sizeof(T) == 8) {
                    // phi(h) phi(u) = phi(k) phi(v): also the joint density without 1/sqrt(1 - rho^2)
                    const T joint = T(0.15915494309189533577) * expT(-T(0.5) * fma(h, h, u * u));
                    ph = density_cdf(ph, joint, u);
                    pk = density_cdf(pk, joint, v);
                    pr = joint * isig;
                } else {
                    ph *= cdf(u);
                    pk *= cdf(v);
                    const T e = (h * h - T(2) * rhoT * h * kq + kq * kq) * isig * isig;
                    pr = expT(-T(0.5) * e) * isig * T(0.15915494309189533577);
                }
            } else if (P.zinf == 2) {
                pc = cdf(h); ph = norm_pdf_fast(h); pk = T(0); pr = T(0);
            } else if (P.zinf == 1) {
                pc = cdf(kq); ph = T(0); pk = norm_pdf_fast(kq); pr = T(0);
            } else {
                pc = T(1); ph = T(0); pk = T(0); pr = T(0);
            }
            sum[p][0] += static_cast<double>(T(1) - pc);
#pragma unroll
            for (int j = 0; j < D; ++j) {
                T dO = U[p][j];
                if constexpr (kSplit) {
                    const T sp = logistic ? s[p][j] * (T(1) - s[p][j]) * iw : T(0);
                    dO = fma(sp, U[p][j], s[p][j] * V[p][j]);
                }
                const T dmu2 = b0 * f[kUU + j] + b1 * (vv * dO - O[p] * f[kWW + j]);
                const T dp = (ph + pk) * f[kDZ + j] - pk * dmu2 + pr * f[kDA + j];
                sum[p][1 + j] -= static_cast<double>(dp);
            }
            sum[p][1 + D] += static_cast<double>(ph * sI + pk * srI);
            sum[p][2 + D] += static_cast<double>(ph * sI * PR + pk * srI * O[p] * invr);
        }
    }
#pragma unroll
    for (int p = 0; p < PP; ++p)
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            double v = sum[p][i];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
            if (lane == 0) red[wave][p * NS + i] = v;
        }
    __syncthreads();
    if (threadIdx.x < a.pw * PP * NS) {   // the draw wavefronts' sums in order
        const int w0 = threadIdx.x / (PP * NS), c = threadIdx.x % (PP * NS), p = c / NS, i = c % NS;
        const int64_t bp = (group * a.pw + w0) * PP + p;
        double v = red[w0][c];
        for (int w = w0 + a.pw; w < kGradThreads / 64; w += a.pw) v += red[w][c];
        if (bp < a.B) a.partials[((a.slice0 + slice) * NS + i) * a.B + bp] = v;
    }
}

__global__ void k_grad_finalize(int d, int64_t B, int64_t M, int n_slices, const double* __restrict__ part,
                                const double* __restrict__ info, double* __restrict__ obj,
                                double* __restrict__ gq, double* __restrict__ gmu) {
    const int64_t b = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (b >= B) return;
    const bool valid = info[b * kInfoFields] != 0.0;
    const double Md = static_cast<double>(M);
    for (int c = 0; c < d + 3; ++c) {
        double s = 0.0;
        for (int sl = 0; sl < n_slices; ++sl) s += part[(static_cast<int64_t>(sl) * (d + 3) + c) * B + b];
        const double v = valid ? s / Md : NAN;
        if (c == 0) obj[b] = v;
        else if (c <= d) { if (gq) gq[b * d + (c - 1)] = v; }
        else if (gmu) gmu[b * 2 + (c - 1 - d)] = v;
    }
}

// The same reduction with one workgroup per (point, component): for few points
// and many slices, where one thread per point would walk thousands of slices.
// Thread t adds slices t, t + 256, ... in order, then a fixed-order tree.
__global__ __launch_bounds__(256) void k_grad_finalize_wide(int d, int64_t B, int64_t M, int n_slices,
                                                            const double* __restrict__ part,
                                                            const double* __restrict__ info, double* __restrict__ obj,
                                                            double* __restrict__ gq, double* __restrict__ gmu) {
    __shared__ double red[256];
    const int64_t b = blockIdx.x / (d + 3);
    const int c = static_cast<int>(blockIdx.x % (d + 3));
    double s = 0.0;
    for (int sl = threadIdx.x; sl < n_slices; sl += 256) s += part[(static_cast<int64_t>(sl) * (d + 3) + c) * B + b];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (static_cast<int>(threadIdx.x) < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    const bool valid = info[b * kInfoFields] != 0.0;
    const double v = valid ? red[0] / static_cast<double>(M) : NAN;
    if (c == 0) obj[b] = v;
    else if (c <= d) { if (gq) gq[b * d + (c - 1)] = v; }
    else if (gmu) gmu[b * 2 + (c - 1 - d)] = v;
}

template <typename T, int PP>
const void* grad_kernel(int d) {
    switch (d) {
        case 1: return reinterpret_cast<const void*>(k_grad<T, 1, PP>);
        case 2: return reinterpret_cast<const void*>(k_grad<T, 2, PP>);
        case 3: return reinterpret_cast<const void*>(k_grad<T, 3, PP>);
        case 4: return reinterpret_cast<const void*>(k_grad<T, 4, PP>);
        case 5: return reinterpret_cast<const void*>(k_grad<T, 5, PP>);
        default: return reinterpret_cast<const void*>(k_grad<T, 6, PP>);
    }
}

constexpr int kGradPoints = 2;   // points per wavefront

// Wavefronts of a workgroup along the points (as many as they fill), and the
// rows of points that gives.
int grad_point_waves(int64_t B) { return B > 2 * kGradPoints ? 4 : B > kGradPoints ? 2 : 1; }
int64_t grad_groups(int64_t B) {
    const int64_t per = static_cast<int64_t>(grad_point_waves(B)) * kGradPoints;
    return (B + per - 1) / per;
}

// Node-table bytes of a slice, at most: the rows of points that read a slice drift
// apart along it, and past the XCD's 4 MB L2 each fetches it for itself.  4,096
// points x 1e6 draws, five biomarkers, FP32 (slices of 30 MB by the rounds alone): 144.7 ms
// without a bound, 106.6 / 105.9 / 105.9 / 104.9 / 103.7 at 16 / 8 / 4 / 2 / 1 MB; FP64, 1,024 points
// x 200,000 draws, six: 33.6 at 16 MB, 24.4 at 2, 25.5 at 1.
constexpr int64_t kGradWindow = int64_t(2) << 20;
// Partial sums that more slices than the rounds need may take.
constexpr size_t kGradPartials = size_t(1) << 30;

// Points go in launches of at most kGradGrid groups or wavefronts (the grid's
// thread count stays below 2^32).
constexpr int64_t kGradGrid = 1 << 22;

template <typename T>
hipError_t launch_grad_typed(GradArgs<T> ga, const double* info, const T* rec, const T* AD, const T* glw,
                             const DrawArrays<T>& Dr, int d, hipStream_t s) {
    const int64_t rounds = (ga.slices + 7) / 8, groups = grad_groups(ga.B);
    ga.pw = grad_point_waves(ga.B);
    for (ga.group0 = 0; ga.group0 < groups; ga.group0 += kGradGrid) {
        ga.groups = std::min(groups - ga.group0, kGradGrid);
        // the XCD numbering needs a slice for every XCD, and a workgroup count within the first dimension
        ga.by_xcd = ga.slices >= 8 && ga.groups * rounds <= (int64_t(1) << 20);
        const dim3 grid = ga.by_xcd ? dim3(static_cast<unsigned>(8 * rounds * ga.groups))
                                    : dim3(static_cast<unsigned>(ga.groups), static_cast<unsigned>(ga.slices));
        void* args[] = {&ga, &info, &rec, &AD, &glw, const_cast<DrawArrays<T>*>(&Dr)};
        const hipError_t e = hipLaunchKernel(grad_kernel<T, kGradPoints>(d), grid, dim3(kGradThreads), args, 0, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <typename T>
hipError_t run_grad(const bmd_problem* p, int prec, const double* d_q, int64_t B, int64_t M, char* ws, const GradPlan& g,
                    bool draws_ready, double* info, double* part, T* rec, T* AD, hipStream_t s) {
    const int d = p->P.d, K = p->tab[prec].K;
    const int per = B > 4 * static_cast<int64_t>(p->n_cu) ? 16 : 4;   // points per workgroup of 256: 16 or 64 lanes each
    for (int64_t b0 = 0; b0 < B; b0 += per * kGradGrid) {
        const dim3 grid(static_cast<unsigned>(std::min((B - b0 + per - 1) / per, kGradGrid)));
        if (per == 16)
            hipLaunchKernelGGL((k_grad_points<T, 16>), grid, dim3(256), 0, s, p->P, d_q, b0, B, p->d_ghp, kPrecomputeGH,
                               p->tab[prec].gh, K, p->d_gl, info, rec, AD);
        else
            hipLaunchKernelGGL((k_grad_points<T, 64>), grid, dim3(256), 0, s, p->P, d_q, b0, B, p->d_ghp, kPrecomputeGH,
                               p->tab[prec].gh, K, p->d_gl, info, rec, AD);
    }
    if constexpr (sizeof(T) == 4) {
        int share = 64;   // few points: fewer of them, as few as one for one or two
        while (share > 1 && B * (64 / share) < 128) share /= 2;
        for (int64_t b0 = 0; b0 < B; b0 += 256 * kGradGrid)
            hipLaunchKernelGGL(k_grad_rule, dim3(static_cast<unsigned>(std::min((B - b0 + 255) / 256, kGradGrid)), kGradNmax<T>),
                               dim3(256), 0, s, b0, B, share, p->d_gl, info, rec);
    }
    hipError_t e = hipGetLastError();
    // Passes over the draws: generate a pass into HBM, then the slices it holds.
    for (int64_t k0 = 0; k0 < M && e == hipSuccess; k0 += g.pass) {
        const int64_t np = std::min<int64_t>(g.pass, M - k0);
        if (!draws_ready) e = launch_grad_draws(p, prec, static_cast<uint64_t>(k0), np, ws, s);
        if (e != hipSuccess) return e;
        GradArgs<T> ga{p->P, B, M, K, g.slice_len, k0 / g.slice_len, (np + g.slice_len - 1) / g.slice_len,
                       0, 0, 1, false, k0, part};
        DrawArrays<T> D;
        if constexpr (sizeof(T) == 8) D = draws_fp64_at(p, np, ws);
        else D = draws_fp32_at(p, np, ws);
        e = launch_grad_typed<T>(ga, info, rec, AD, static_cast<const T*>(p->tab[prec].glw), D, d, s);
    }
    return e;
}

}  // namespace

static size_t al256(size_t x) { return (x + 255) / 256 * 256; }
static size_t rec_bytes(int prec, int64_t B) {
    return prec == BMD_FP64 ? sizeof(double) * kRecSize<double> * B : sizeof(float) * kRecSize<float> * B;
}

// Layout: the draws of a pass first (so that a later call on the same draws
// finds them whatever its point count), then the points' records and tables,
// then the partial sums.
size_t grad_workspace_bytes(const bmd_problem* p, int prec, int64_t B, const GradPlan& g) {
    const size_t T = prec == BMD_FP64 ? 8 : 4;
    const int d = p->P.d, K = p->tab[prec].K;
    return al256(draw_workspace_bytes(p, prec, g.pass)) +
           al256(sizeof(double) * kInfoFields * B) + al256(rec_bytes(prec, B)) + al256(2 * T * d * K * B) +
           al256(sizeof(double) * (d + 3) * B * g.n_slices);
}

// Draw slices of a call: about kSweepRounds rounds of resident workgroups over
// the point groups, whole workgroups of draws.  Draws held in HBM per pass: whole
// slices, at most kGradDrawBudget bytes (BMD_GRAD_BUDGET, in bytes, overrides it;
// small values force many passes).
GradPlan grad_plan(const bmd_problem* p, int prec, int64_t B, int64_t M) {
    const void* f = prec == BMD_FP64 ? grad_kernel<double, kGradPoints>(p->P.d) : grad_kernel<float, kGradPoints>(p->P.d);
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, kGradThreads, 0) != hipSuccess || nb < 1) {
        (void)hipGetLastError();
        nb = 1;
    }
    size_t budget = kGradDrawBudget;
    if (const char* env = std::getenv("BMD_GRAD_BUDGET")) {
        const long long v = std::atoll(env);
        if (v > 0) budget = static_cast<size_t>(v);
    }
    const double per = static_cast<double>(draw_workspace_bytes(p, prec, 1 << 20)) / (1 << 20);
    const int d = p->P.d;
    const int64_t row = static_cast<int64_t>(prec == BMD_FP64 ? 8 : 4) * d * p->tab[prec].K;
    return grad_plan_of(grad_groups(B), kGradThreads / grad_point_waves(B), static_cast<int64_t>(p->n_cu) * nb,
                        kSweepRounds, M, per, budget, d >= 2 ? kGradWindow / row : 0,
                        static_cast<int64_t>(kGradPartials / (sizeof(double) * (d + 3) * B)));
}

hipError_t launch_grad(const bmd_problem* p, int prec, const double* d_q, int64_t B, int64_t M, void* ws,
                       const GradPlan& g, bool draws_ready, double* obj, double* gq, double* gmu, hipStream_t s) {
    const size_t T = prec == BMD_FP64 ? 8 : 4;
    const int d = p->P.d, K = p->tab[prec].K;
    char* base = static_cast<char*>(ws);
    const int n_slices = static_cast<int>(g.n_slices);
    char* c = base + al256(draw_workspace_bytes(p, prec, g.pass));
    auto take = [&](size_t bytes) {
        char* at = c;
        c += al256(bytes);
        return at;
    };
    double* info = reinterpret_cast<double*>(take(sizeof(double) * kInfoFields * B));
    char* rec = take(rec_bytes(prec, B));
    char* AD = take(2 * T * d * K * B);
    double* part = reinterpret_cast<double*>(take(sizeof(double) * (d + 3) * B * n_slices));
    hipError_t e;
    if (prec == BMD_FP64)
        e = run_grad<double>(p, prec, d_q, B, M, base, g, draws_ready, info, part,
                             reinterpret_cast<double*>(rec), reinterpret_cast<double*>(AD), s);
    else
        e = run_grad<float>(p, prec, d_q, B, M, base, g, draws_ready, info, part,
                            reinterpret_cast<float*>(rec), reinterpret_cast<float*>(AD), s);
    if (e != hipSuccess) return e;
    // one thread per point walking the slices is a serial chain of loads: few
    // points with more than a handful of slices take a workgroup per component
    if (n_slices > 16 && B * (d + 3) <= (int64_t(1) << (n_slices > 256 ? 20 : 14)))
        hipLaunchKernelGGL(k_grad_finalize_wide, dim3(static_cast<unsigned>(B * (d + 3))), dim3(256), 0, s, d, B, M,
                           n_slices, part, info, obj, gq, gmu);
    else
        hipLaunchKernelGGL(k_grad_finalize, dim3(static_cast<unsigned>((B + 127) / 128)), dim3(128), 0, s, d, B, M,
                           n_slices, part, info, obj, gq, gmu);
    return hipGetLastError();
}

}  // namespace bmd
