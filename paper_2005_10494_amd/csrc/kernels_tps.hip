// Thin-plate spline smoothing of a grid surface (Sec. 2.3: the Monte Carlo
// estimates are fitted by a thin-plate spline, whose maximum is then refined).
// The spline of order 2 in d = 1..3 dimensions,
//   f(u) = sum_i c_i phi(|u - u_i|) + a_0 + a^T u,
//   phi(r) = r^3 (d = 1), r^2 log r (d = 2), -r (d = 3),
// on the designs with a value, their coordinates in the grid's unit box
// (u_j = i_j / (m_j - 1)), with the coefficients of the smoothing system
//   (Phi + lam I) c + P a = y,   P^T c = 0,   P = [1, u].
// The polynomial block is eliminated with the QR factors of P: d + 1
// Householder reflectors give Q^T P = [R; 0]; with c = Q [0; w] the reduced
// matrix M22 of M = Q^T (Phi + lam I) Q is positive definite when the designs
// determine a plane, so w solves M22 w = z2 (z = Q^T y) by a blocked Cholesky
// factorisation, and R a = z1 - M12 w.  FP64 throughout.
#include <cmath>

#include "bmd_internal.hpp"

namespace bmd {

struct TpsFit {
    int64_t n = 0;              // centres
    int d = 0;
    double* mem = nullptr;      // device: U [n d], c [n], a [d + 1]
};

namespace {

constexpr int kMaxTpsDim = 3;
constexpr int kNB = 64;          // Cholesky and triangular-solve block, and the update's output tile
constexpr int kLS = kNB + 2;     // LDS row stride of a tile: a 16 x 4 operand read touches every bank twice
constexpr int kHalf = kNB / 2;   // columns staged at a time
constexpr int kHS = kHalf + 2;   // their LDS row stride (as kLS)
constexpr int kIS = 18;          // LDS row stride of a 16 x 16 inverse

// The radial function for D dimensions, fixed at compile time: with the
// dimension chosen at run time inside one function, the gfx950 code of an
// earlier build skipped the -r branch for D = 3 and stored the unnegated
// square root (NaN at r = 0), so every kernel that evaluates phi is a
// template on D.
template <int D>
__device__ __forceinline__ double tps_phi(double r2) {   // of the squared distance
    if constexpr (D == 1) return r2 * sqrt(r2);
    else if constexpr (D == 2) return r2 > 0.0 ? 0.5 * r2 * log(r2) : 0.0;
    else return -sqrt(r2);
}

// Unit-box coordinates of grid design g.
__device__ __forceinline__ void unit_coords(const DevProblem& P, int64_t g, double* u) {
    int64_t rem = g;
    for (int j = 0; j < P.d; ++j) {
        const int64_t i = rem / P.stride[j];
        rem -= i * P.stride[j];
        u[j] = static_cast<double>(i) / static_cast<double>(P.m[j] - 1);
    }
}

// Lane src's value of v on every lane (src wave-uniform): two reads into
// scalar registers, no round trip through LDS as a shuffle takes.
__device__ __forceinline__ double lane_value(double v, int src) {
    const unsigned long long u = static_cast<unsigned long long>(__double_as_longlong(v));
    const unsigned lo = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(u & 0xffffffffu), src));
    const unsigned hi = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(u >> 32), src));
    return __longlong_as_double(static_cast<long long>((static_cast<unsigned long long>(hi) << 32) | lo));
}

__device__ double block_sum(double v, double* red) {
    const int t = threadIdx.x, nt = blockDim.x;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    __syncthreads();
    if ((t & 63) == 0) red[t >> 6] = v;
    __syncthreads();
    double s = 0.0;
    for (int w = 0; w < nt / 64; ++w) s += red[w];   // same order on every thread
    return s;
}

// Designs with a value, in index order (one workgroup of 1024: a scan per
// tile); their count goes to *n_out.
__global__ __launch_bounds__(1024) void k_tps_compact(int64_t G, const double* __restrict__ f,
                                                      int64_t* __restrict__ idx, int64_t* __restrict__ n_out) {
    __shared__ int scan[1024];
    const int t = threadIdx.x;
    int64_t base = 0;
    for (int64_t g0 = 0; g0 < G; g0 += 1024) {
        const int64_t g = g0 + t;
        const int ok = g < G && f[g] == f[g];
        scan[t] = ok;
        __syncthreads();
        for (int off = 1; off < 1024; off <<= 1) {
            const int v = t >= off ? scan[t - off] : 0;
            __syncthreads();
            scan[t] += v;
            __syncthreads();
        }
        if (ok) idx[base + scan[t] - 1] = g;
        base += scan[1023];
        __syncthreads();
    }
    if (t == 0) *n_out = base;
}

// Centres U [n d], values y [n] and the polynomial block P [n][d + 1].
__global__ void k_tps_points(DevProblem P, int64_t n, const int64_t* __restrict__ idx, const double* __restrict__ f,
                             double* __restrict__ U, double* __restrict__ y, double* __restrict__ Pm) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double u[kMaxDim];
    unit_coords(P, idx[i], u);
    const int d = P.d;
    Pm[i * (d + 1)] = 1.0;
    for (int j = 0; j < d; ++j) {
        U[i * d + j] = u[j];
        Pm[i * (d + 1) + 1 + j] = u[j];
    }
    y[i] = f[idx[i]];
}

// Householder QR of P [n][d + 1] (one workgroup): reflector k is
// I - tau_k v_k v_k^T with v_k zero above row k; R [(d+1)^2] upper
// triangular.  A column whose remaining norm is below 1e-12 of its first
// norm raises *bad (the designs do not determine a plane).
__global__ __launch_bounds__(1024) void k_tps_qr(int64_t n, int d, double* __restrict__ Pm, double* __restrict__ V,
                                                 double* __restrict__ tau, double* __restrict__ R,
                                                 int* __restrict__ bad) {
    __shared__ double red[16];
    const int t = threadIdx.x;
    const int np = d + 1;
    for (int k = 0; k < np; ++k) {
        double s = 0.0, s0 = 0.0;
        for (int64_t i = t; i < n; i += blockDim.x) {
            const double x = Pm[i * np + k];
            s0 = fma(x, x, s0);
            if (i >= k) s = fma(x, x, s);
        }
        const double sigma2 = block_sum(s, red);
        const double full2 = block_sum(s0, red);
        const double xk = Pm[k * np + k];
        const double sigma = sqrt(sigma2);
        const double alpha = xk >= 0.0 ? -sigma : sigma;
        if (!(sigma > 1e-12 * sqrt(full2)) && t == 0) *bad = 1;
        const double vk = xk - alpha;
        const double vnorm2 = sigma2 - xk * xk + vk * vk;
        const double tk = vnorm2 > 0.0 ? 2.0 / vnorm2 : 0.0;
        for (int64_t i = t; i < n; i += blockDim.x) V[i * np + k] = i < k ? 0.0 : i == k ? vk : Pm[i * np + k];
        if (t == 0) {
            tau[k] = tk;
            R[k * np + k] = alpha;
        }
        __syncthreads();
        for (int j = k + 1; j < np; ++j) {
            double dj = 0.0;
            for (int64_t i = t + k; i < n; i += blockDim.x) dj = fma(V[i * np + k], Pm[i * np + j], dj);
            const double sj = block_sum(dj, red) * tk;
            for (int64_t i = t + k; i < n; i += blockDim.x) Pm[i * np + j] -= sj * V[i * np + k];
            __syncthreads();
            if (t == 0) R[k * np + j] = Pm[k * np + j];
        }
        if (t < k && t < np) R[k * np + t] = 0.0;
        __syncthreads();
    }
}

// Row blockIdx.x of A = Phi + lam I (n x n, row stride ld) and of Y = A V, one
// workgroup: the reflectors' products with the row while it is formed.
template <int D>
__global__ __launch_bounds__(256) void k_tps_matrix(int64_t n, int64_t ld, const double* __restrict__ U, double lam,
                                                    const double* __restrict__ V, double* __restrict__ A,
                                                    double* __restrict__ Y) {
    constexpr int NP = D + 1;
    __shared__ double red[4];
    const int64_t i = blockIdx.x;
    double u[D], s[NP] = {};
#pragma unroll
    for (int j = 0; j < D; ++j) u[j] = U[i * D + j];
    for (int64_t k = threadIdx.x; k < n; k += 256) {
        double r2 = 0.0;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const double t = u[j] - U[k * D + j];
            r2 = fma(t, t, r2);
        }
        const double a = tps_phi<D>(r2) + (i == k ? lam : 0.0);
        A[i * ld + k] = a;
#pragma unroll
        for (int q = 0; q < NP; ++q) s[q] = fma(a, V[k * NP + q], s[q]);
    }
#pragma unroll
    for (int q = 0; q < NP; ++q) {
        const double v = block_sum(s[q], red);
        if (threadIdx.x == 0) Y[i * NP + q] = v;
    }
}

// The reflectors together, Q = H_0 ... H_d = I - V T V^T with T upper triangular
// (T_kk = tau_k, column k above it -tau_k T V^T v_k), give
//   Q^T A Q = A - Z V^T - V Z^T,  Z = Y T - V T^T (V^T Y) T / 2.
// One workgroup forms T (to Tm) and B = T^T (V^T Y) T / 2 (to Tm + np^2).
__global__ __launch_bounds__(1024) void k_tps_wy(int64_t n, int np, const double* __restrict__ V, const double* __restrict__ Y,
                                                 const double* __restrict__ tau, double* __restrict__ Tm) {
    constexpr int NP = kMaxTpsDim + 1;
    __shared__ double red[16], VV[NP][NP], VY[NP][NP];
    double sv[NP][NP] = {}, sy[NP][NP] = {};
    for (int64_t i = threadIdx.x; i < n; i += 1024) {
        double v[NP], y[NP];
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            v[q] = q < np ? V[i * np + q] : 0.0;
            y[q] = q < np ? Y[i * np + q] : 0.0;
        }
#pragma unroll
        for (int a = 0; a < NP; ++a)
#pragma unroll
            for (int b = 0; b < NP; ++b) {
                if (a < b) sv[a][b] = fma(v[a], v[b], sv[a][b]);
                sy[a][b] = fma(v[a], y[b], sy[a][b]);
            }
    }
#pragma unroll
    for (int a = 0; a < NP; ++a)
#pragma unroll
        for (int b = 0; b < NP; ++b) {
            if (a >= np || b >= np) continue;   // uniform
            const double x = a < b ? block_sum(sv[a][b], red) : 0.0;
            const double y = block_sum(sy[a][b], red);
            if (threadIdx.x == 0) {
                VV[a][b] = x;
                VY[a][b] = y;
            }
        }
    if (threadIdx.x != 0) return;
    double T[NP][NP] = {}, X[NP][NP];
    for (int k = 0; k < np; ++k) {
        T[k][k] = tau[k];
        for (int a = 0; a < k; ++a) {
            double x = 0.0;
            for (int b = a; b < k; ++b) x = fma(T[a][b], VV[b][k], x);
            T[a][k] = -tau[k] * x;
        }
    }
    for (int a = 0; a < np; ++a)
        for (int b = 0; b < np; ++b) {
            double x = 0.0;
            for (int k = 0; k <= b; ++k) x = fma(VY[a][k], T[k][b], x);
            X[a][b] = x;
        }
    for (int a = 0; a < np; ++a)
        for (int b = 0; b < np; ++b) {
            double x = 0.0;
            for (int k = 0; k <= a; ++k) x = fma(T[k][a], X[k][b], x);
            Tm[a * np + b] = T[a][b];
            Tm[np * np + a * np + b] = 0.5 * x;
        }
}

// Z, one thread per row.
__global__ void k_tps_z(int64_t n, int np, const double* __restrict__ V, const double* __restrict__ Y,
                        const double* __restrict__ Tm, double* __restrict__ Z) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    for (int k = 0; k < np; ++k) {
        double z = 0.0;
        for (int j = 0; j < np; ++j) z += Y[i * np + j] * Tm[j * np + k] - V[i * np + j] * Tm[np * np + j * np + k];
        Z[i * np + k] = z;
    }
}

// A <- A - Z V^T - V Z^T where it is read afterwards: the first np rows and the
// lower triangle.  (One reflector after another, both sides each, read the
// whole matrix twice and wrote it once for every reflector: 414 us for 5,754
// centres and three of them, against 106 with T, B and Z.)
template <int NP>
__global__ __launch_bounds__(256) void k_tps_reduce(int64_t n, int64_t ld, const double* __restrict__ V,
                                                    const double* __restrict__ Z, double* __restrict__ A) {
    const int64_t i = blockIdx.y, j = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (j >= n || (j > i && i >= NP)) return;
    double x = A[i * ld + j];
#pragma unroll
    for (int k = 0; k < NP; ++k) x -= V[i * NP + k] * Z[j * NP + k] + Z[i * NP + k] * V[j * NP + k];
    A[i * ld + j] = x;
}

// FP64 16x16x4 matrix instruction: lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16]; element v of its result is row l / 16 + 4 v, column
// l % 16.  So a result's element v is also the B operand of the v-th slice of
// four of a following product's 16 inner indices.
typedef double tps_d4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ tps_d4 mfma64(double a, double b, tps_d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Orders a wavefront's LDS writes before its other lanes' reads.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// 1/sqrt(x) and 1/x: the hardware's estimates (2^-24) and one third-order step.
__device__ __forceinline__ double rsqrt64(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-(x * y), y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}
__device__ __forceinline__ double rcp64(double x) {
    const double y = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, y, 1.0);
    return fma(y, fma(e, e, e), y);
}

// The kHalf columns [c0, c0 + kHalf) of rows [r0, r0 + kNB) of the reduced system
// (rows from `rows` on: 0), consecutive lanes on consecutive columns, and
// their place in LDS.
constexpr int kTileIt = kNB * kHalf / 256, kTileStep = 256 / kHalf;
__device__ __forceinline__ void load_tile(const double* __restrict__ M, int64_t ld, int64_t r0, int64_t rows, int64_t c0,
                                          double (&v)[kTileIt]) {
    const int c = threadIdx.x % kHalf, r = threadIdx.x / kHalf, left = static_cast<int>(min<int64_t>(rows - r0, kNB));
    const uint32_t off = static_cast<uint32_t>(r * static_cast<int>(ld) + c);
    if (left == kNB) {   // whole tiles without a branch per load
#pragma unroll
        for (int q = 0; q < kTileIt; ++q) v[q] = (M + (r0 + kTileStep * q) * ld + c0)[off];
    } else {
#pragma unroll
        for (int q = 0; q < kTileIt; ++q) v[q] = r + kTileStep * q < left ? (M + (r0 + kTileStep * q) * ld + c0)[off] : 0.0;
    }
}
__device__ __forceinline__ void store_tile(const double (&v)[kTileIt], double (*X)[kHS]) {
    const int c = threadIdx.x % kHalf, r = threadIdx.x / kHalf;
#pragma unroll
    for (int q = 0; q < kTileIt; ++q) X[r + kTileStep * q][c] = v[q];
}

// Cholesky factor L of the kNB x kNB block in the lower triangle of S by four
// wavefronts, in blocks of 16: block (j, i) of S, i > j, receives -L's block (i, j),
// Iv[j] the inverse of diagonal block j.  Each wavefront eliminates the diagonal
// block by itself in registers, its rows in lanes 0..15 and the rows of the
// unit matrix in lanes 16..31 (the same steps turn those into the inverse's
// transpose; a column's elements go to all lanes as scalars).  Columns are
// scaled by 1/sqrt(pivot) afterwards, and the next pivot is formed beside the
// row updates, so a column's chain is a reciprocal and two operations.  All
// wavefronts form the same inverse, so each goes on without waiting for the
// others; a panel block is formed transposed, which is the operand of its
// product either way.  True if a pivot was not positive.
__device__ __forceinline__ bool factor_block(double (*S)[kLS], double (*Iv)[16][kIS], double (*T)[kIS]) {
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63, r16 = lane & 15, kq = lane >> 4;
    bool neg = false;
#pragma unroll 1
    for (int j = 0; j < kNB / 16; ++j) {
        const int j0 = 16 * j;
        double row[16];
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            const double v = S[j0 + r16][j0 + c];
            row[c] = lane < 16 ? (c <= r16 ? v : 0.0) : lane < 32 && c == r16 ? 1.0 : 0.0;
        }
        double pv = lane_value(row[0], 0), mine = 1.0;   // mine: pivot r16
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            const bool ok = pv > 0.0;
            neg |= !ok;
            pv = ok ? pv : 1.0;
            mine = r16 == c ? pv : mine;
            const double inv = rcp64(pv);
            if (c < 15) {
                const double a = lane_value(row[c], c + 1);
                pv = fma(-(a * inv), a, lane_value(row[c + 1], c + 1));
            }
            const double u = row[c] * inv;
#pragma unroll
            for (int e = c + 1; e < 16; ++e) row[e] = fma(-u, lane_value(row[c], e), row[e]);
        }
        if (kq == 1) {
#pragma unroll
            for (int c = 0; c < 16; ++c) T[c][r16] = row[c];
        }
        wave_sync();
        const double rs = rsqrt64(mine);
        double inv[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            inv[k] = T[r16][4 * k + kq] * rs;
            Iv[j][r16][4 * k + kq] = inv[k];
        }
        const auto panel = [&](int b) {   // element (4 v + kq, r16) of block (b, j)'s transpose
            tps_d4 x{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int k = 0; k < 4; ++k) x = mfma64(inv[k], S[16 * b + r16][j0 + 4 * k + kq], x);
            return x;
        };
#pragma unroll 1
        for (int b = wave, bi = j + 1, bk = j + 1;; ++bk) {   // blocks (bi, bk), j < bk <= bi, every fourth
            if (bk > bi) bk = j + 1, ++bi;
            if (bi == kNB / 16) break;
            if (b-- != 0) continue;
            b = 3;
            const tps_d4 y = panel(bk);
            tps_d4 z = y;
            if (bi != bk) z = panel(bi);
            else {
#pragma unroll
                for (int v = 0; v < 4; ++v) S[j0 + r16][16 * bk + 4 * v + kq] = -y[v];
            }
            tps_d4 x{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int k = 0; k < 4; ++k) x = mfma64(z[k], y[k], x);
#pragma unroll
            for (int v = 0; v < 4; ++v) S[16 * bi + kq + 4 * v][16 * bk + r16] -= x[v];
        }
        __syncthreads();
    }
    return neg;
}

// Step kb of the blocked Cholesky M22 = L L^T, one launch: the update by the
// previous `depth` block columns (A -= L21 L21^T) and, in the same launch, block
// column kb's factor.  M is the reduced system, lower triangle, its row n2 the
// right-hand side z2, which the steps turn into the forward solve L^-1 z2.
//   Workgroups 0 .. panels: the block column.  Each updates the diagonal block
//     for itself (it is only read: no workgroup sees another's results within
//     a launch), factors it, then updates its own kNB rows below it and solves
//     them, X L11^T = A21, sixteen rows a wavefront: held transposed, each
//     16 x 16 block's result is the next product's operand as it stands.
//     Workgroup 0 solves the unit matrix instead and stores Ld = L11^-T for
//     the backward solve.
//   The others: one tile of the trailing update each, four wavefronts of 32 x 32.
// The trailing matrix is updated at every second step, by two block columns at
// once (the steps between update their own block column only): 113 us at 5,700
// rows, where two updates by one take 88 each.  It costs as much in matrix
// instructions (59 us) as in reading and writing that matrix (57 us), and the
// two overlap little.  A step without it is the factor's serial chain (14 of
// 25 us).  5,754 centres: a launch for the factor (22 us) and one for the
// update (26 us) per 32 columns, and two (9 us) for the solves, took 12.0 ms;
// a launch per 64 columns (a square root and a division in each column's chain)
// and one (5.5 us) for the backward solve 4.5 ms; this 4.1 ms.  Half a block
// column staged at a time lets three workgroups share a compute unit (two: 118
// us); giving each XCD a compact part of the tiles changes nothing.
// A pivot <= 0 raises *bad.
__global__ __launch_bounds__(256, 3) void k_chol_step(int64_t ld, int64_t kb, int bs, int64_t n2, int panels, int depth,
                                                      double* __restrict__ M, double* __restrict__ Ld,
                                                      int* __restrict__ bad) {
    // the staged halves of the previous block columns, then the block being factored
    constexpr int kTile = 2 * kNB * kHS;
    static_assert(kTile >= kNB * kLS, "the block fits the staged tiles' place");
    __shared__ double tiles[kTile];
    double (*Xi)[kHS] = reinterpret_cast<double (*)[kHS]>(tiles);
    double (*Xk)[kHS] = reinterpret_cast<double (*)[kHS]>(tiles + kNB * kHS);
    double (*S)[kLS] = reinterpret_cast<double (*)[kLS]>(tiles);
    __shared__ double Iv[kNB / 16][16][kIS], T[16][kIS];
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63, r16 = lane & 15, kq = lane >> 4;
    const int64_t rows = n2 + 1;
    double vi[kTileIt], vk[kTileIt];   // the next half's tiles, in flight during a product
    const int64_t done = kb - depth * kNB;   // first column of the update
    if (static_cast<int>(blockIdx.x) > panels) {
        // workgroup b -> lower-triangle tile (ti, tk), tk <= ti, b = ti (ti + 1) / 2 + tk
        const int64_t b = static_cast<int64_t>(blockIdx.x) - panels - 1;
        int ti = __builtin_amdgcn_readfirstlane(static_cast<int>((sqrt(8.0 * static_cast<double>(b) + 1.0) - 1.0) * 0.5));
        while (ti * (ti + 1) / 2 > b) --ti;
        while ((ti + 1) * (ti + 2) / 2 <= b) ++ti;
        const int64_t i0 = kb + kNB + ti * kNB, k0 = kb + kNB + (b - ti * (ti + 1) / 2) * kNB;
        const int rb = (wave >> 1) * 32, cb = (wave & 1) * 32;
        // element v of block (p, q) of the wavefront's quarter: row 16 p + 4 v + rb + kq, column 16 q + cb + r16
        double* tile = M + i0 * ld + k0;
        const uint32_t off = static_cast<uint32_t>((rb + kq) * static_cast<int>(ld) + cb + r16);
        const auto inside = [&](int p, int q, int v) {
            const int i = rb + kq + 16 * p + 4 * v, k = cb + r16 + 16 * q;
            return i0 + i < rows && k0 + k < n2 && k0 + k <= i0 + i;
        };
        load_tile(M, ld, i0, rows, done, vi);
        load_tile(M, ld, k0, rows, done, vk);
        const bool whole = i0 + kNB <= rows && k0 + kNB <= n2 && k0 < i0;
        double old[2][2][4];
        const auto load_old = [&](auto in) {
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int v = 0; v < 4; ++v) old[p][q][v] = in(p, q, v) ? (tile + (16 * p + 4 * v) * ld + 16 * q)[off] : 0.0;
        };
        const auto all = [](int, int, int) { return true; };
        if (whole) load_old(all);
        else load_old(inside);
        tps_d4 acc[2][2];
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int q = 0; q < 2; ++q) acc[p][q] = tps_d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
        for (int64_t from = done; from < kb; from += kHalf) {
            if (from > done) __syncthreads();
            store_tile(vi, Xi);
            store_tile(vk, Xk);
            __syncthreads();
            if (from + kHalf < kb) {
                load_tile(M, ld, i0, rows, from + kHalf, vi);
                load_tile(M, ld, k0, rows, from + kHalf, vk);
            }
#pragma unroll
            for (int c0 = 0; c0 < kHalf; c0 += 4) {
                const double x0 = Xi[rb + r16][c0 + kq], x1 = Xi[rb + 16 + r16][c0 + kq];
                const double y0 = Xk[cb + r16][c0 + kq], y1 = Xk[cb + 16 + r16][c0 + kq];
                acc[0][0] = mfma64(x0, y0, acc[0][0]);
                acc[0][1] = mfma64(x0, y1, acc[0][1]);
                acc[1][0] = mfma64(x1, y0, acc[1][0]);
                acc[1][1] = mfma64(x1, y1, acc[1][1]);
            }
        }
        const auto store = [&](auto in) {
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (in(p, q, v)) (tile + (16 * p + 4 * v) * ld + 16 * q)[off] = old[p][q][v] - acc[p][q][v];
        };
        if (whole) store(all);
        else store(inside);
        return;
    }
    const bool unit = blockIdx.x == 0;
    const int64_t r0 = kb + bs + (static_cast<int64_t>(blockIdx.x) - 1) * kNB;   // this workgroup's rows
    // diag[q]: block 4 q + wave of the ten lower 16 x 16 blocks of the diagonal block (past the
    // block column's end: the unit matrix); x[q]: columns 16 q .. of rows 16 wave .., transposed
    tps_d4 diag[3], x[4];
    int bi[3], bk[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int b = min(4 * q + wave, 9);
        bi[q] = b < 1 ? 0 : b < 3 ? 1 : b < 6 ? 2 : 3;
        bk[q] = b - bi[q] * (bi[q] + 1) / 2;
    }
    double own[16];
    const auto load_block = [&](auto in, auto below) {
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = 16 * bi[q] + kq + 4 * v, k = 16 * bk[q] + r16;
                diag[q][v] = in(i, k) ? M[(kb + i) * ld + kb + k] : i == k ? 1.0 : 0.0;
            }
#pragma unroll
        for (int r = 0; r < 16; ++r) {   // the wavefront's rows, a row at a time
            const int i = 16 * wave + r;
            own[r] = below(i, lane) ? M[(r0 + i) * ld + kb + lane] : unit && i == lane ? 1.0 : 0.0;
        }
    };
    const bool whole = bs == kNB && r0 + kNB <= rows && !unit;
    const auto all = [](int, int) { return true; };
    if (whole)   // with the diagonal blocks' upper elements, which factor_block leaves out
        load_block(all, all);
    else
        load_block([&](int i, int k) { return i < bs && k < bs; },
                   [&](int i, int k) { return !unit && r0 + i < rows && k < bs; });
    if (depth > 0) {
        if (!unit) load_tile(M, ld, r0, rows, done, vi);
        load_tile(M, ld, kb, kb + bs, done, vk);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) S[16 * wave + r][lane] = own[r];
    wave_sync();
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) x[q][v] = S[16 * wave + r16][16 * q + kq + 4 * v];
    __syncthreads();
#pragma unroll 1
    for (int64_t from = done; from < kb; from += kHalf) {
        if (!unit) store_tile(vi, Xi);
        store_tile(vk, Xk);
        __syncthreads();
        if (from + kHalf < kb) {
            if (!unit) load_tile(M, ld, r0, rows, from + kHalf, vi);
            load_tile(M, ld, kb, kb + bs, from + kHalf, vk);
        }
#pragma unroll 4
        for (int c0 = 0; c0 < kHalf; c0 += 4)
#pragma unroll
            for (int q = 0; q < 3; ++q) diag[q] = mfma64(-Xk[16 * bi[q] + r16][c0 + kq], Xk[16 * bk[q] + r16][c0 + kq], diag[q]);
        if (!unit) {
#pragma unroll 4
            for (int c0 = 0; c0 < kHalf; c0 += 4) {
                const double y = Xi[16 * wave + r16][c0 + kq];
#pragma unroll
                for (int q = 0; q < 4; ++q) x[q] = mfma64(-Xk[16 * q + r16][c0 + kq], y, x[q]);
            }
        }
        __syncthreads();   // the tiles' place takes the next half, at the end the diagonal block
    }
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v)   // the tenth block comes from waves 1..3 alike
            S[16 * bi[q] + kq + 4 * v][16 * bk[q] + r16] = diag[q][v];
    __syncthreads();
    const bool neg = factor_block(S, Iv, T);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int e = 0; e < q; ++e)
#pragma unroll
            for (int k = 0; k < 4; ++k) x[q] = mfma64(S[16 * e + r16][16 * q + 4 * k + kq], x[e][k], x[q]);
        tps_d4 y{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < 4; ++k) y = mfma64(Iv[q][r16][4 * k + kq], x[q][k], y);
        x[q] = y;
    }
    __syncthreads();   // S is read by all until here
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) S[16 * wave + r16][16 * q + kq + 4 * v] = x[q][v];
    wave_sync();
    double* to = unit ? Ld + kb * kNB + lane : M + r0 * ld + kb + lane;
    const int64_t stride = unit ? kNB : ld;
    const int left = unit || whole ? kNB : static_cast<int>(min<int64_t>(rows - r0, kNB));
#pragma unroll
    for (int r = 0; r < 16; ++r)
        if (16 * wave + r < left && (unit || lane < bs)) to[(16 * wave + r) * stride] = S[16 * wave + r][lane];
    if (unit && t == 0 && neg) *bad = 1;
}

// z = Q^T y = H_d ... H_0 y (one workgroup).
__global__ __launch_bounds__(1024) void k_tps_qty(int64_t n, int np, const double* __restrict__ V,
                                                  const double* __restrict__ tau, const double* __restrict__ y,
                                                  double* __restrict__ z) {
    __shared__ double red[16];
    for (int64_t i = threadIdx.x; i < n; i += blockDim.x) z[i] = y[i];
    __syncthreads();
    for (int k = 0; k < np; ++k) {
        double s = 0.0;
        for (int64_t i = threadIdx.x + k; i < n; i += blockDim.x) s = fma(V[i * np + k], z[i], s);
        s = block_sum(s, red) * tau[k];
        for (int64_t i = threadIdx.x + k; i < n; i += blockDim.x) z[i] -= s * V[i * np + k];
        __syncthreads();
    }
}

// One block of kNB rows of the backward solve L^T w = t: every workgroup forms
// the block's w = L11^-T t from Ld (four threads a row), workgroup 0 stores
// it, and each subtracts L[kb ..][r]^T w from kNB of the rows r above (sixteen
// block rows a wavefront, loaded before w is formed).  The block's own
// elements of t are only read.
__global__ __launch_bounds__(256) void k_back_step(int64_t ld, int64_t kb, int bs, const double* __restrict__ M,
                                                   const double* __restrict__ Ld, double* __restrict__ tv,
                                                   double* __restrict__ w) {
    __shared__ double wb[kNB];
    __shared__ double part[4][kNB];
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
    const int64_t r = static_cast<int64_t>(blockIdx.x) * kNB + lane;
    double l[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) l[c] = r < kb && 16 * wave + c < bs ? M[(kb + 16 * wave + c) * ld + r] : 0.0;
    const int row = t >> 2, q = t & 3;
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < 16; ++j) {   // columns 4 j + q: the four threads of a row read one segment
        const int c = 4 * j + q;
        if (c < bs) s = fma(Ld[(kb + row) * kNB + c], tv[kb + c], s);
    }
    s += __shfl_xor(s, 1);
    s += __shfl_xor(s, 2);
    if (q == 0) {
        wb[row] = s;
        if (blockIdx.x == 0 && row < bs) w[kb + row] = s;
    }
    __syncthreads();
    double a = 0.0;
#pragma unroll
    for (int c = 0; c < 16; ++c) a = fma(l[c], wb[16 * wave + c], a);
    part[wave][lane] = a;
    __syncthreads();
    if (wave == 0 && r < kb) tv[r] -= (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
}

// c = Q [0; w] = H_0 ... H_d [0; w] and R a = z1 - M12 w; writes c and a into
// the fit (one workgroup).
__global__ __launch_bounds__(1024) void k_tps_coeffs(int64_t n, int64_t ld, int np, const double* __restrict__ A,
                                                     const double* __restrict__ V, const double* __restrict__ tau,
                                                     const double* __restrict__ R, const double* __restrict__ z,
                                                     const double* __restrict__ w, double* __restrict__ c,
                                                     double* __restrict__ a) {
    __shared__ double red[16];
    __shared__ double rhs[kMaxDim + 1];
    const int t = threadIdx.x;
    for (int k = 0; k < np; ++k) {   // z1_k - sum_j M[k][np + j] w_j
        double s = 0.0;
        for (int64_t j = np + t; j < n; j += blockDim.x) s = fma(A[k * ld + j], w[j - np], s);
        s = block_sum(s, red);
        if (t == 0) rhs[k] = z[k] - s;
    }
    for (int64_t i = t; i < n; i += blockDim.x) c[i] = i < np ? 0.0 : w[i - np];
    __syncthreads();
    for (int k = np - 1; k >= 0; --k) {
        double s = 0.0;
        for (int64_t i = t + k; i < n; i += blockDim.x) s = fma(V[i * np + k], c[i], s);
        s = block_sum(s, red) * tau[k];
        for (int64_t i = t + k; i < n; i += blockDim.x) c[i] -= s * V[i * np + k];
        __syncthreads();
    }
    if (t == 0) {
        for (int k = np - 1; k >= 0; --k) {
            double s = rhs[k];
            for (int j = k + 1; j < np; ++j) s -= R[k * np + j] * a[j];
            a[k] = s / R[k * np + k];
        }
    }
}

// The fitted surface at every grid design (NaN where f has no value), one
// wavefront per design: the lanes take every 64th centre, a butterfly sums.
template <int D>
__global__ __launch_bounds__(256) void k_tps_eval_grid(DevProblem P, int64_t n, const double* __restrict__ U,
                                                       const double* __restrict__ c, const double* __restrict__ a,
                                                       const double* __restrict__ f, double* __restrict__ out) {
    const int64_t g = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (g >= P.G) return;   // wave-uniform
    if (f[g] != f[g]) {
        if (lane == 0) out[g] = f[g];
        return;
    }
    double u[kMaxDim];
    unit_coords(P, g, u);
    double v = 0.0;
    for (int64_t i = lane; i < n; i += 64) {
        double r2 = 0.0;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const double s = u[j] - U[i * D + j];
            r2 = fma(s, s, r2);
        }
        v = fma(c[i], tps_phi<D>(r2), v);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if (lane == 0) {
        double poly = a[0];
#pragma unroll
        for (int j = 0; j < D; ++j) poly = fma(a[1 + j], u[j], poly);
        out[g] = poly + v;
    }
}

// Value, gradient and Hessian in unit coordinates at u (one workgroup):
// out = [value, grad (d), Hessian rows j <= l (d (d + 1) / 2)].  At a centre
// its own term adds no derivative (r^2 log r's Hessian diverges there, -r has
// a kink).
template <int D>
__global__ __launch_bounds__(1024) void k_tps_at(int64_t n, const double* __restrict__ U, const double* __restrict__ c,
                                                 const double* __restrict__ a, double u0, double u1, double u2,
                                                 double* __restrict__ out) {
    constexpr int NA = 1 + D + D * (D + 1) / 2;
    __shared__ double red[16];
    const double u[3] = {u0, u1, u2};
    double acc[NA] = {};
    for (int64_t i = threadIdx.x; i < n; i += blockDim.x) {
        double s[D], r2 = 0.0;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            s[j] = u[j] - U[i * D + j];
            r2 = fma(s[j], s[j], r2);
        }
        const double r = sqrt(r2);
        acc[0] = fma(c[i], tps_phi<D>(r2), acc[0]);
        if (r == 0.0) continue;
        double p1, p2;   // phi'(r), phi''(r)
        if constexpr (D == 1) {
            p1 = 3.0 * r * r;
            p2 = 6.0 * r;
        } else if constexpr (D == 2) {
            p1 = r * (2.0 * log(r) + 1.0);
            p2 = 2.0 * log(r) + 3.0;
        } else {
            p1 = -1.0;
            p2 = 0.0;
        }
        const double g1 = c[i] * p1 / r, g2 = c[i] * (p2 - p1 / r) / r2;
        int k = 1 + D;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            acc[1 + j] = fma(g1, s[j], acc[1 + j]);
#pragma unroll
            for (int l = j; l < D; ++l, ++k) acc[k] += g2 * s[j] * s[l] + (j == l ? g1 : 0.0);
        }
    }
    double poly = a[0];
#pragma unroll
    for (int j = 0; j < D; ++j) poly = fma(a[1 + j], u[j], poly);
#pragma unroll
    for (int q = 0; q < NA; ++q) {
        const double v = block_sum(acc[q], red);
        if (threadIdx.x == 0) out[q] = v + (q == 0 ? poly : q <= D ? a[q] : 0.0);
        __syncthreads();
    }
}

}  // namespace

void tps_release(bmd_problem* p) {
    if (!p || !p->tps) return;
    if (p->tps->mem) (void)hipFree(p->tps->mem);
    delete p->tps;
    p->tps = nullptr;
}

#define TPS_TRY(expr)                \
    do {                             \
        res.err = (expr);            \
        if (res.err != hipSuccess) { \
            res.code = kTpsHip;      \
            goto done;               \
        }                            \
    } while (0)

TpsFitResult tps_fit_grid(bmd_problem* p, const double* d_in, double lam, double* d_out, hipStream_t s) {
    const DevProblem& P = p->P;
    const int d = P.d, np = d + 1;
    const int64_t G = P.G;
    TpsFitResult res{kTpsOk, 0, hipSuccess};
    int64_t n = 0, n2 = 0, ld = 0;
    int bad = 0;
    char* small = nullptr;   // idx [G], n, bad flag; tau, R, T and B
    double* big = nullptr;   // A [n ld], z [n] as its row n, V, P, Y and Z [n (d + 1)], y, w [n], Ld
    double* fitmem = nullptr;
    int64_t* d_idx = nullptr;
    int64_t* d_n = nullptr;
    int* d_bad = nullptr;
    double *d_tau = nullptr, *d_R = nullptr, *d_T = nullptr;
    double *A = nullptr, *V = nullptr, *Pm = nullptr, *y = nullptr, *z = nullptr, *Y = nullptr, *Z = nullptr, *M = nullptr;
    double *Ld = nullptr, *w = nullptr;   // inverses of the factor's diagonal blocks; the reduced system's solution
    double *U = nullptr, *c = nullptr, *a = nullptr;
    const size_t small_bytes = sizeof(int64_t) * (G + 2) + 64 + sizeof(double) * (2 * np + 3 * np * np + 8);
    if (hipMalloc(&small, small_bytes) != hipSuccess) {
        (void)hipGetLastError();
        res.code = kTpsNoMem;
        return res;
    }
    d_idx = reinterpret_cast<int64_t*>(small);
    d_n = d_idx + G;
    d_bad = reinterpret_cast<int*>(d_n + 1);
    d_tau = reinterpret_cast<double*>(small + sizeof(int64_t) * (G + 2) + 64);
    d_R = d_tau + np;
    d_T = d_R + np * np;
    TPS_TRY(hipMemsetAsync(d_bad, 0, sizeof(int), s));
    hipLaunchKernelGGL(k_tps_compact, dim3(1), dim3(1024), 0, s, G, d_in, d_idx, d_n);
    TPS_TRY(hipGetLastError());
    TPS_TRY(hipMemcpyAsync(&n, d_n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    TPS_TRY(hipStreamSynchronize(s));
    res.n = n;
    if (n < d + 2 || n > kTpsMaxPoints) {
        res.code = kTpsCount;
        goto done;
    }
    {
        const size_t nn = static_cast<size_t>(n);
        // the reduced system's rows begin on a cache line: row stride and first column in 16 doubles
        ld = (n + 15) / 16 * 16;
        const size_t lead = 16 - np, full = static_cast<size_t>(ld);
        const size_t big_count = lead + (nn + 1) * full + 4 * nn * np + 2 * nn + kNB * (nn + kNB);
        if (hipMalloc(&big, sizeof(double) * big_count) != hipSuccess ||
            hipMalloc(&fitmem, sizeof(double) * (nn * d + nn + np)) != hipSuccess) {
            (void)hipGetLastError();
            res.code = kTpsNoMem;
            goto done;
        }
        A = big + lead;
        z = A + nn * full;
        V = z + full;
        Pm = V + nn * np;
        Y = Pm + nn * np;
        Z = Y + nn * np;
        y = Z + nn * np;
        w = y + nn;
        Ld = w + nn;
        U = fitmem;
        c = U + nn * d;
        a = c + nn;
    }
    hipLaunchKernelGGL(k_tps_points, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, s, P, n, d_idx, d_in,
                       U, y, Pm);
    TPS_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_tps_qr, dim3(1), dim3(1024), 0, s, n, d, Pm, V, d_tau, d_R, d_bad);
    TPS_TRY(hipGetLastError());
    {
        const dim3 grid(static_cast<unsigned>(n)), part(static_cast<unsigned>((n + 255) / 256), static_cast<unsigned>(n));
        if (d == 1) hipLaunchKernelGGL(k_tps_matrix<1>, grid, dim3(256), 0, s, n, ld, U, lam, V, A, Y);
        else if (d == 2) hipLaunchKernelGGL(k_tps_matrix<2>, grid, dim3(256), 0, s, n, ld, U, lam, V, A, Y);
        else hipLaunchKernelGGL(k_tps_matrix<3>, grid, dim3(256), 0, s, n, ld, U, lam, V, A, Y);
        TPS_TRY(hipGetLastError());
        hipLaunchKernelGGL(k_tps_wy, dim3(1), dim3(1024), 0, s, n, np, V, Y, d_tau, d_T);   // M = Q^T A Q
        hipLaunchKernelGGL(k_tps_z, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, s, n, np, V, Y, d_T, Z);
        if (d == 1) hipLaunchKernelGGL(k_tps_reduce<2>, part, dim3(256), 0, s, n, ld, V, Z, A);
        else if (d == 2) hipLaunchKernelGGL(k_tps_reduce<3>, part, dim3(256), 0, s, n, ld, V, Z, A);
        else hipLaunchKernelGGL(k_tps_reduce<4>, part, dim3(256), 0, s, n, ld, V, Z, A);
        TPS_TRY(hipGetLastError());
    }
    hipLaunchKernelGGL(k_tps_qty, dim3(1), dim3(1024), 0, s, n, np, V, d_tau, y, z);
    TPS_TRY(hipGetLastError());
    n2 = n - np;
    M = A + np * ld + np;   // the reduced system; its row n2 is z2
    for (int64_t kb = 0; kb < n2; kb += kNB) {   // M22 = L L^T, L t = z2
        const int bs = static_cast<int>(std::min<int64_t>(kNB, n2 - kb));
        const int64_t panels = (n2 + 1 - kb - bs + kNB - 1) / kNB;
        const int64_t step = kb / kNB;
        const int depth = step == 0 ? 0 : step % 2 == 0 ? 2 : 1;
        const int64_t tiles = depth == 2 && kb + kNB < n2 ? (n2 + 1 - kb - kNB + kNB - 1) / kNB : 0;
        hipLaunchKernelGGL(k_chol_step, dim3(static_cast<unsigned>(1 + panels + tiles * (tiles + 1) / 2)), dim3(256), 0,
                           s, ld, kb, bs, n2, static_cast<int>(panels), depth, M, Ld, d_bad);
        TPS_TRY(hipGetLastError());
    }
    for (int64_t kb = ((n2 - 1) / kNB) * kNB; kb >= 0; kb -= kNB) {   // L^T w = t
        const int bs = static_cast<int>(std::min<int64_t>(kNB, n2 - kb));
        hipLaunchKernelGGL(k_back_step, dim3(static_cast<unsigned>(std::max<int64_t>(1, kb / kNB))), dim3(256), 0, s, ld,
                           kb, bs, M, Ld, z + np, w);
    }
    hipLaunchKernelGGL(k_tps_coeffs, dim3(1), dim3(1024), 0, s, n, ld, np, A, V, d_tau, d_R, z, w, c, a);
    TPS_TRY(hipGetLastError());
    TPS_TRY(hipMemcpyAsync(&bad, d_bad, sizeof(int), hipMemcpyDeviceToHost, s));
    TPS_TRY(hipStreamSynchronize(s));
    if (bad) {
        res.code = kTpsSingular;
        goto done;
    }
    if (d_out) {
        const dim3 grid(static_cast<unsigned>((G + 3) / 4));
        if (d == 1) hipLaunchKernelGGL(k_tps_eval_grid<1>, grid, dim3(256), 0, s, P, n, U, c, a, d_in, d_out);
        else if (d == 2) hipLaunchKernelGGL(k_tps_eval_grid<2>, grid, dim3(256), 0, s, P, n, U, c, a, d_in, d_out);
        else hipLaunchKernelGGL(k_tps_eval_grid<3>, grid, dim3(256), 0, s, P, n, U, c, a, d_in, d_out);
        TPS_TRY(hipGetLastError());
    }
    TPS_TRY(hipStreamSynchronize(s));
    tps_release(p);
    p->tps = new TpsFit;
    p->tps->n = n;
    p->tps->d = d;
    p->tps->mem = fitmem;
    fitmem = nullptr;
done:
    (void)hipStreamSynchronize(s);
    if (fitmem) (void)hipFree(fitmem);
    if (big) (void)hipFree(big);
    (void)hipFree(small);
    return res;
}

hipError_t tps_at_unit(const bmd_problem* p, const double* u, double* h_out, hipStream_t s) {
    const TpsFit& F = *p->tps;
    const int d = F.d;
    const double* U = F.mem;
    const double* c = U + F.n * d;
    const double* a = c + F.n;
    const double u1 = d > 1 ? u[1] : 0.0, u2 = d > 2 ? u[2] : 0.0;
    if (d == 1) hipLaunchKernelGGL(k_tps_at<1>, dim3(1), dim3(1024), 0, s, F.n, U, c, a, u[0], u1, u2, h_out);
    else if (d == 2) hipLaunchKernelGGL(k_tps_at<2>, dim3(1), dim3(1024), 0, s, F.n, U, c, a, u[0], u1, u2, h_out);
    else hipLaunchKernelGGL(k_tps_at<3>, dim3(1), dim3(1024), 0, s, F.n, U, c, a, u[0], u1, u2, h_out);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    return e;
}

int tps_dims(const bmd_problem* p) { return p->tps ? p->tps->d : 0; }

}  // namespace bmd
