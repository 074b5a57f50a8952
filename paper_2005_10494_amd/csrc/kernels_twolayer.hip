// The paper's two-layer sampling estimator of the expected power (Formula 7,
// with the inner layer of Formula 6): N1 outer draws Delta^(k) from the prior,
// N2 inner draws x^(l) of the null statistics (Formula 1), and
//   P = 1 - (1 / (N1 N2)) sum_k sum_l [x^(l)_j <= z_j - sqrt(r_j I) Delta^(k)_j for all j],
// the same inner draws serving every outer draw.  The comparisons are counted in
// A x B blocks (outer-draw groups x inner-draw groups), from which the
// finalize forms the estimate and an unbiased estimate of its variance.
//
// Inner draws: n standard normals e'_1..e'_n per l from the Philox stream whose
// fourth counter word has its top bit set, chained into the nested null
// correlations of Appendix A.1: x_1 = e'_1,
// x_{i+1} = sqrt(r_{i+1}/r_i) x_i + sqrt(1 - r_{i+1}/r_i) e'_{i+1}.
#include <algorithm>
#include <cstdint>

#include "bmd_internal.hpp"
#include "device_math.hpp"

namespace bmd {
namespace {

constexpr int kTwoBlock = 256;   // threads per workgroup (and outer draws per LDS chunk)
constexpr int kTwoR = 4;         // inner draws per lane
constexpr uint32_t kInnerStream = 0x80000000u;

// Uniform i (< 4) of inner draw l: Philox counter (l lo, l hi, scenario, top bit | block).
__device__ __forceinline__ double inner_uniform(uint64_t l, const DevProblem& P, int i) {
    const uint4 o = philox4x32_10(make_uint4(static_cast<uint32_t>(l), static_cast<uint32_t>(l >> 32), P.scenario,
                                             kInnerStream | static_cast<uint32_t>(i / 2)),
                                  P.key0, P.key1);
    return (i & 1) ? uniform52(o.z, o.w) : uniform52(o.x, o.y);
}

// e[j * N2 + l] = Phi^-1(u_j(l)), j < n.
__global__ void k_inner_draws(DevProblem P, int n, int64_t N2, double* __restrict__ e) {
    const int64_t l = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (l >= N2) return;
    for (int j = 0; j < n; ++j) e[j * N2 + l] = norm_quantile(inner_uniform(static_cast<uint64_t>(l), P, j));
}

__global__ void k_zero_u32(uint32_t* __restrict__ p, int64_t n) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

struct TwoLayerArgs {
    DevProblem P;
    int n;                      // nested populations
    const double* r;            // [G] second fraction (cutoff and two-population alpha designs)
    const double* z[4];         // [G] critical values
    const double* e[4];         // outer draws' normals, FP64 [N1]
    const double* ei;           // inner draws' normals [n][N2]
    int64_t N1, N2;
    int A, B;                   // outer and inner groups
    uint32_t* blocks;           // [G][A][B]
};

// Fractions r_1..r_n of design g (r_1 = 1).
__device__ __forceinline__ void design_fractions(const TwoLayerArgs& a, int64_t g, double* r) {
    r[0] = 1.0;
    r[1] = a.n == 2 ? a.r[g] : a.P.r_lo;
    r[2] = a.P.r_hi;
    r[3] = a.P.r_4;
}

// Constants of a design's fractions r_1..r_N: the outer means mu_i = sqrt(r_i I)
// (theta_i + sigma_i Y_i) of Formula 10, Y the chain of the outer normals, as
// mu_i = m0_i + sum_{j<=i} mc[i][j] e_j, and the chain's own steps.
template <int N>
struct ChainConst {
    double m0[N], mc[N][N], f[N], g[N];
    __device__ void init(const TwoLayerArgs& a, const double* r) {
        double ch[N][N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const double th = -log1p(-(a.P.paper_a - a.P.paper_b * r[i]));
            const double sc = sqrt(r[i] * a.P.info) / sqrt(a.P.paper_events * r[i] / 4.0);
            m0[i] = sqrt(r[i] * a.P.info) * th;
            f[i] = i == 0 ? 0.0 : sqrt(r[i] / r[i > 0 ? i - 1 : 0]);
            g[i] = i == 0 ? 1.0 : sqrt(1.0 - r[i] / r[i > 0 ? i - 1 : 0]);
#pragma unroll
            for (int j = 0; j < N; ++j) ch[i][j] = j < i ? f[i] * ch[i > 0 ? i - 1 : 0][j] : 0.0;
            ch[i][i] = g[i];
#pragma unroll
            for (int j = 0; j < N; ++j) mc[i][j] = sc * ch[i][j];
        }
    }
    // The outer draw's means and the inner draw's statistics.
    __device__ __forceinline__ void means(const double* e, double* mu) const {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            mu[i] = m0[i];
#pragma unroll
            for (int j = 0; j <= i; ++j) mu[i] += mc[i][j] * e[j];
        }
    }
    __device__ __forceinline__ double statistic(int i, double before, double e) const {
        return i == 0 ? e : f[i] * before + g[i] * e;
    }
};

// One workgroup: design blockIdx.x and 1,024 inner draws; wavefront w's lane
// holds the four draws blockIdx.y * 1024 + w * 256 + 64 i + lane (i < 4), so
// a wavefront's draws are contiguous and lie in one inner group.  The outer
// draws' thresholds b_kj = z_j - mu_j^(k) go through LDS in chunks of 256 (one
// per thread) and each read serves the lane's four inner draws (one read per
// comparison would exceed the LDS bandwidth).  Each lane counts, over the
// outer draws of the current group, how often its inner draws stay below the
// thresholds in every coordinate, and at the end of each outer group the
// wavefront's counts go to the design's block (outer group, inner group of the
// wavefront) by one atomic add.  T is the comparison type (FP64, or FP32 with
// both sides rounded).
template <typename T, int N>
__global__ __launch_bounds__(kTwoBlock) void k_two_layer(TwoLayerArgs a) {
    // thresholds of a chunk, each draw's padded to 2 or 4 values so that one
    // vector LDS read fetches them
    constexpr int NP = N == 2 ? 2 : 4;
    __shared__ __align__(16) T sb[kTwoBlock * NP];
    const int64_t g = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    double r[4], z[N];
    design_fractions(a, g, r);
    bool skip = false;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        z[j] = a.z[j][g];
        skip = skip || z[j] != z[j];   // no valid level split: the finalize writes NaN
    }
    if (skip) return;
    ChainConst<N> cc;
    cc.init(a, r);
    // this lane's inner draws, the same chain of their own normals
    const int64_t l0 = static_cast<int64_t>(blockIdx.y) * (kTwoBlock * kTwoR) + (tid >> 6) * (64 * kTwoR) + lane;
    T x[kTwoR][N];
#pragma unroll
    for (int q = 0; q < kTwoR; ++q) {
        double xd[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            xd[i] = cc.statistic(i, i == 0 ? 0.0 : xd[i > 0 ? i - 1 : 0], a.ei[i * a.N2 + l0 + 64 * q]);
            x[q][i] = static_cast<T>(xd[i]);
        }
    }
    const int64_t SA = a.N1 / a.A;
    const int bgrp = static_cast<int>(l0 / (a.N2 / a.B));
    uint32_t* blk = a.blocks + (g * a.A) * a.B + bgrp;
    uint32_t cnt = 0;
    for (int64_t k0 = 0; k0 < a.N1; k0 += kTwoBlock) {
        const int nk = static_cast<int>(min<int64_t>(kTwoBlock, a.N1 - k0));
        __syncthreads();   // the previous chunk's thresholds are no longer read
        if (tid < nk) {
            double e[N];
#pragma unroll
            for (int j = 0; j < N; ++j) e[j] = a.e[j][k0 + tid];
            double mu[N];
            cc.means(e, mu);
#pragma unroll
            for (int i = 0; i < N; ++i) sb[tid * NP + i] = static_cast<T>(z[i] - mu[i]);
        }
        __syncthreads();
        int kk = 0;
        while (kk < nk) {
            // the outer draws of this chunk up to the end of the current group
            const int64_t k = k0 + kk;
            const int end = static_cast<int>(min<int64_t>(nk, (k / SA + 1) * SA - k0));
            // every coordinate compared, the results combined without branches;
            // two outer draws at a time so that their LDS reads are in flight together
            for (; kk + 2 <= end; kk += 2) {
                T bk[2][NP];
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int j = 0; j < NP; ++j) bk[u][j] = sb[(kk + u) * NP + j];
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int q = 0; q < kTwoR; ++q) {
                        uint32_t in = 1u;
#pragma unroll
                        for (int j = 0; j < N; ++j) in &= static_cast<uint32_t>(x[q][j] <= bk[u][j]);
                        cnt += in;
                    }
            }
            for (; kk < end; ++kk) {
#pragma unroll
                for (int q = 0; q < kTwoR; ++q) {
                    uint32_t in = 1u;
#pragma unroll
                    for (int j = 0; j < N; ++j) in &= static_cast<uint32_t>(x[q][j] <= sb[kk * NP + j]);
                    cnt += in;
                }
            }
            if ((k0 + kk) % SA == 0) {   // group done: add the wavefront's counts to its block
                uint32_t s = cnt;
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
                if (lane == 0) atomicAdd(blk + ((k0 + kk) / SA - 1) * a.B, s);
                cnt = 0;
            }
        }
    }
}

// The same counts from ranks and bit sets.  One workgroup: kBitDraws inner
// draws (blockIdx.x) and up to kBitDesigns consecutive designs of the launch
// order with the same fractions (group blockIdx.y), hence the same inner
// statistics.  Per coordinate the draws are sorted once and row q of a table
// holds the set of the q smallest as bits.  A threshold's rank q_j = #{x_j <=
// b_j} is a search in the sorted values (a balanced tree in LDS, root first:
// nine compare-and-descend steps, conflict-free in its upper levels), and the
// draws inside all thresholds are the common bits of rows q_1 .. q_N: 16 words,
// N - 1 ands and a bit count each, for 512 comparisons.  The counts are whole
// numbers, so they equal the comparing kernel's above.
// Split: one outer draw per lane, 64 consecutive ones per wavefront pass; its
// means are formed once and serve every design of the group, and a coordinate
// whose critical value the previous design shares (levels of one grid row) is
// not searched again.  Rows of 64 bytes start on 4 banks of the 64 only, so
// the four 16-byte pieces of row q are stored in the order piece ^ (q / 4) % 4.
// Bound: LDS (12 16-byte row reads and up to 27 search reads a pass at N = 3)
// and vector issue, about level; the tables take 98 KB at N = 3, so one
// workgroup of 16 wavefronts per compute unit.
// Measured at N1 = 10,240, N2 = 20,480, three populations, 49 x 49 levels,
// FP32: 36.9 ms comparing, 4.3 ms here (8.3e12 and 7.3e13 comparisons/s).
constexpr int kBitDraws = 512;
constexpr int kBitWords = kBitDraws / 32;
constexpr int kBitThreads = 1024;
constexpr int kBitDesigns = 16;

// Sum over the wavefront, returned in every lane.
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
    return __builtin_amdgcn_readlane(v, 63);
}

template <typename T, int N>
__global__ __launch_bounds__(kBitThreads) void k_two_layer_bits(TwoLayerArgs a, const int32_t* __restrict__ order,
                                                                int64_t shared_designs, int64_t groups_per_share,
                                                                int per_group) {
    __shared__ __align__(16) uint32_t rows[N][kBitDraws + 1][kBitWords];
    __shared__ T tree[N][kBitDraws];           // sorted values; then nodes 1..511 (root first) and, at 0, the largest
    __shared__ uint16_t ids[N][kBitDraws];     // draw of each rank
    __shared__ uint32_t cnt[kBitDesigns][64][2];   // per design: outer group, half of the chunk
    __shared__ double zs[kBitDesigns][N];
    __shared__ int32_t gs[kBitDesigns];        // designs of the group (-1: no valid level split)
    __shared__ int same[kBitDesigns];          // bit j: critical value j equals the previous design's

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // designs [i0, i1) of the launch order, within one run of shared fractions
    const int64_t run = static_cast<int64_t>(blockIdx.y) / groups_per_share;
    const int64_t i0 = run * shared_designs + (static_cast<int64_t>(blockIdx.y) % groups_per_share) * per_group;
    const int64_t i1 = min(min(i0 + per_group, (run + 1) * shared_designs), a.P.G);
    const int nd = static_cast<int>(i1 - i0);
    if (nd <= 0) return;
    if (tid < nd) {
        const int64_t g = order ? order[i0 + tid] : i0 + tid;
        bool skip = false;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            zs[tid][j] = a.z[j][g];
            skip = skip || zs[tid][j] != zs[tid][j];
        }
        gs[tid] = skip ? -1 : static_cast<int32_t>(g);
    }
    __syncthreads();
    bool any = false;
    for (int d = 0; d < nd; ++d) any = any || gs[d] >= 0;
    if (!any) return;   // uniform: the finalize writes NaN
    if (tid < nd) {
        int m = 0;
#pragma unroll
        for (int j = 0; j < N; ++j)
            if (tid > 0 && gs[tid - 1] >= 0 && zs[tid][j] == zs[tid - 1][j]) m |= 1 << j;
        same[tid] = m;
    }
    for (int i = tid; i < kBitDesigns * 64 * 2; i += kBitThreads) (&cnt[0][0][0])[i] = 0u;

    double r[4];
    design_fractions(a, order ? order[i0] : i0, r);
    ChainConst<N> cc;
    cc.init(a, r);

    // the chunk's inner statistics, then per coordinate a bitonic sort of (value, draw)
    const int64_t l0 = static_cast<int64_t>(blockIdx.x) * kBitDraws;
    if (tid < kBitDraws) {
        double x = 0.0;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            x = cc.statistic(i, x, a.ei[i * a.N2 + l0 + tid]);
            tree[i][tid] = static_cast<T>(x);
            ids[i][tid] = static_cast<uint16_t>(tid);
        }
    }
    const int sj = tid >> 8, sp = tid & 255;   // coordinate and pair (or table part) of this thread
    for (int size = 2; size <= kBitDraws; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            __syncthreads();
            if (sj < N) {
                const int lo = 2 * sp - (sp & (stride - 1)), hi = lo + stride;
                const T u = tree[sj][lo], v = tree[sj][hi];
                if ((u > v) == ((lo & size) == 0)) {   // ascending where bit `size` of the index is clear
                    const uint16_t iu = ids[sj][lo], iv = ids[sj][hi];
                    tree[sj][lo] = v;
                    tree[sj][hi] = u;
                    ids[sj][lo] = iv;
                    ids[sj][hi] = iu;
                }
            }
        }
    }
    __syncthreads();
    // sorted values to tree order
    T node[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int i = sp + 256 * h;
        if (sj < N) {
            int at = kBitDraws - 1;   // node 0: the largest value
            if (i > 0) {
                const int level = 31 - __clz(i);
                at = (2 * (i - (1 << level)) + 1) * (kBitDraws >> (level + 1)) - 1;
            }
            node[h] = tree[sj][at];
        }
    }
    __syncthreads();
    if (sj < N) {
#pragma unroll
        for (int h = 0; h < 2; ++h) tree[sj][sp + 256 * h] = node[h];
        // rows: thread = (coordinate, word w, segment of 32 ranks); the segment's own bits, the
        // bits of the segments before it (a scan over 16 lanes), then its 32 rows
        const int w = sp >> 4, seg = sp & 15;
        uint32_t mine = 0u;
        for (int i = 0; i < 32; ++i) {
            const uint32_t id = ids[sj][seg * 32 + i];
            if (static_cast<int>(id >> 5) == w) mine |= 1u << (id & 31);
        }
        uint32_t upto = mine;
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) {
            const uint32_t t = __shfl_up(upto, off, 16);
            if (seg >= off) upto |= t;
        }
        uint32_t cur = upto & ~mine;   // every draw has one rank, so the segments' bits are disjoint
        for (int i = 0; i < 32; ++i) {
            const int q = seg * 32 + i;
            rows[sj][q][(((w >> 2) ^ (q >> 2)) & 3) * 4 + (w & 3)] = cur;
            const uint32_t id = ids[sj][q];
            if (static_cast<int>(id >> 5) == w) cur |= 1u << (id & 31);
        }
        if (seg == 15) rows[sj][kBitDraws][(((w >> 2) ^ (kBitDraws >> 2)) & 3) * 4 + (w & 3)] = cur;
    }
    __syncthreads();

    const uint32_t SA = static_cast<uint32_t>(a.N1 / a.A);
    for (int64_t kb = static_cast<int64_t>(wave) * 64; kb < a.N1; kb += kBitThreads) {
        const int64_t k = kb + lane;
        const bool in_range = k < a.N1;
        double e[N], mu[N];
#pragma unroll
        for (int j = 0; j < N; ++j) e[j] = a.e[j][in_range ? k : a.N1 - 1];
        cc.means(e, mu);
        const int grp = static_cast<int>(static_cast<uint32_t>(in_range ? k : a.N1 - 1) / SA);
        const int g_first = __builtin_amdgcn_readlane(grp, 0), g_last = __builtin_amdgcn_readlane(grp, 63);
        int q[N];
#pragma unroll
        for (int j = 0; j < N; ++j) q[j] = 0;
        for (int d = 0; d < nd; ++d) {
            if (gs[d] < 0) continue;   // uniform
            const int keep = __builtin_amdgcn_readfirstlane(same[d]);
#pragma unroll
            for (int j = 0; j < N; ++j) {
                if (keep & (1 << j)) continue;
                const T b = static_cast<T>(zs[d][j] - mu[j]);
                int i = 1;
#pragma unroll
                for (int step = 0; step < 9; ++step) i = 2 * i + (tree[j][i] <= b ? 1 : 0);
                q[j] = i - kBitDraws + (tree[j][0] <= b ? 1 : 0);
            }
            uint32_t half[2] = {0u, 0u};
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                uint4 m = make_uint4(~0u, ~0u, ~0u, ~0u);
#pragma unroll
                for (int j = 0; j < N; ++j) {
                    const uint4 v = *reinterpret_cast<const uint4*>(&rows[j][q[j]][((t ^ (q[j] >> 2)) & 3) * 4]);
                    m = make_uint4(m.x & v.x, m.y & v.y, m.z & v.z, m.w & v.w);
                }
                half[t >> 1] += __popc(m.x) + __popc(m.y) + __popc(m.z) + __popc(m.w);
            }
            uint32_t both = in_range ? half[0] | (half[1] << 16) : 0u;   // at most 256 each a lane, 16,384 a wavefront
            if (g_first == g_last) {
                both = wave_sum_u32(both);
                if (lane < 2) atomicAdd(&cnt[d][g_first][lane], lane ? both >> 16 : both & 0xffffu);
            } else if (both) {
                atomicAdd(&cnt[d][grp][0], both & 0xffffu);
                atomicAdd(&cnt[d][grp][1], both >> 16);
            }
        }
    }
    __syncthreads();
    // the two halves of the chunk lie in one inner group each (256 divides the group size)
    const int64_t per_inner = a.N2 / a.B;
    for (int i = tid; i < nd * a.A * 2; i += kBitThreads) {
        const int h = i & 1, grp = (i >> 1) % a.A, d = (i >> 1) / a.A;
        const uint32_t c = cnt[d][grp][h];
        if (gs[d] >= 0 && c)
            atomicAdd(a.blocks + (static_cast<int64_t>(gs[d]) * a.A + grp) * a.B + (l0 + 256 * h) / per_inner, c);
    }
}

// One workgroup of 64 threads per design: estimate 1 - T / (N1 N2) from the
// block counts and, with block means m_ab, row and column means R_a, C_b and
// grand mean M, the two-way crossed random-effects estimate of its variance
//   (MS_A + MS_B - MS_E) / (A B),
//   MS_A = B sum_a (R_a - M)^2 / (A - 1),  MS_B = A sum_b (C_b - M)^2 / (B - 1),
//   MS_E = sum_ab (m_ab - R_a - C_b + M)^2 / ((A - 1)(B - 1)),
// unbiased for the estimate's variance (the Hoeffding parts of the indicator
// are uncorrelated, so the block means follow that model).  Designs without a
// valid level split get NaN.
__global__ __launch_bounds__(64) void k_two_layer_final(TwoLayerArgs a, double* __restrict__ mean,
                                                        double* __restrict__ var) {
    __shared__ double sR[64], sC[64], sE[64];
    const int64_t g = blockIdx.x;
    const int t = threadIdx.x;
    bool skip = false;
    for (int j = 0; j < a.n; ++j) skip = skip || a.z[j][g] != a.z[j][g];
    if (skip) {
        if (t == 0) {
            mean[g] = NAN;
            if (var) var[g] = NAN;
        }
        return;
    }
    const int A = a.A, B = a.B;
    const uint32_t* n = a.blocks + g * A * B;
    const double cell = static_cast<double>(a.N1 / A) * static_cast<double>(a.N2 / B);
    if (t < A) {
        double s = 0.0;
        for (int b = 0; b < B; ++b) s += n[t * B + b] / cell;
        sR[t] = s / B;
    }
    if (t < B) {
        double s = 0.0;
        for (int i = 0; i < A; ++i) s += n[i * B + t] / cell;
        sC[t] = s / A;
    }
    __syncthreads();
    double M = 0.0;
    uint64_t T = 0;
    for (int i = 0; i < A; ++i) {
        M += sR[i];
        for (int b = 0; b < B; ++b) T += n[i * B + b];
    }
    M /= A;
    if (t < A) {
        double s = 0.0;
        for (int b = 0; b < B; ++b) {
            const double d = n[t * B + b] / cell - sR[t] - sC[b] + M;
            s += d * d;
        }
        sE[t] = s;
    }
    __syncthreads();
    if (t == 0) {
        mean[g] = 1.0 - static_cast<double>(T) / (static_cast<double>(a.N1) * static_cast<double>(a.N2));
        if (var) {
            double sa = 0.0, sc = 0.0, se = 0.0;
            for (int i = 0; i < A; ++i) sa += (sR[i] - M) * (sR[i] - M);
            for (int b = 0; b < B; ++b) sc += (sC[b] - M) * (sC[b] - M);
            for (int i = 0; i < A; ++i) se += sE[i];
            const double msa = B * sa / (A - 1), msb = A * sc / (B - 1), mse = se / ((A - 1) * (B - 1));
            var[g] = (msa + msb - mse) / (static_cast<double>(A) * B);
        }
    }
}

template <typename T, int N>
void launch_bits(const TwoLayerArgs& a, const int32_t* order, int64_t shared, int per_group, hipStream_t s) {
    const int64_t runs = (a.P.G + shared - 1) / shared, gps = (shared + per_group - 1) / per_group;
    const dim3 grid(static_cast<unsigned>(a.N2 / kBitDraws), static_cast<unsigned>(runs * gps));
    hipLaunchKernelGGL((k_two_layer_bits<T, N>), grid, dim3(kBitThreads), 0, s, a, order, shared, gps, per_group);
}

// Designs that share their fractions and hence their inner statistics (runs of
// the launch order), at most kBitDesigns to a workgroup and as few as keep
// every compute unit busy four times over.  The tables cost a workgroup about
// 20 us; with fewer than kBitMinOuter (outer draw, design) pairs to use them on
// the comparing kernel runs (also beyond the grid's second dimension).
// Measured, comparing / bit sets, over 45 to 2,401 designs of two to four populations,
// 64 to 8,192 outer and 1,024 to 16,384 inner draws, both precisions: at 4,096 pairs 1.14 to
// 5.2 (median 2.6), at 2,048 0.77 to 3.2, at 1,024 0.52 to 2.0, at 512 0.30 to 1.4.
constexpr int64_t kBitMinOuter = 4096;

template <typename T>
hipError_t launch_counts(const TwoLayerArgs& a, int64_t G, int64_t shared, const int32_t* order, int n_cu,
                         hipStream_t s) {
    const int64_t wanted = 4 * static_cast<int64_t>(n_cu), chunks = a.N2 / kBitDraws;
    const int64_t per_group = std::max<int64_t>(
        1, std::min<int64_t>({shared, static_cast<int64_t>(kBitDesigns), G * chunks / wanted}));
    const int64_t groups = (G + shared - 1) / shared * ((shared + per_group - 1) / per_group);
    if (a.N1 * per_group >= kBitMinOuter && groups <= 65535) {
        switch (a.n) {
            case 2: launch_bits<T, 2>(a, order, shared, static_cast<int>(per_group), s); break;
            case 3: launch_bits<T, 3>(a, order, shared, static_cast<int>(per_group), s); break;
            default: launch_bits<T, 4>(a, order, shared, static_cast<int>(per_group), s); break;
        }
        return hipGetLastError();
    }
    const dim3 grid(static_cast<unsigned>(G), static_cast<unsigned>(a.N2 / (kTwoBlock * kTwoR)));
    switch (a.n) {
        case 2: hipLaunchKernelGGL((k_two_layer<T, 2>), grid, dim3(kTwoBlock), 0, s, a); break;
        case 3: hipLaunchKernelGGL((k_two_layer<T, 3>), grid, dim3(kTwoBlock), 0, s, a); break;
        default: hipLaunchKernelGGL((k_two_layer<T, 4>), grid, dim3(kTwoBlock), 0, s, a); break;
    }
    return hipGetLastError();
}

}  // namespace

size_t two_layer_inner_bytes(int n, int64_t N2) { return sizeof(double) * static_cast<size_t>(n) * N2; }

hipError_t launch_two_layer(const bmd_problem* p, int prec, int n, int64_t N1, int64_t N2, int A, int B,
                            const DrawArrays<double>& outer, double* inner, uint32_t* blocks, double* mean,
                            double* var, hipStream_t s) {
    const int64_t G = p->P.G;
    hipLaunchKernelGGL(k_inner_draws, dim3(static_cast<unsigned>((N2 + 255) / 256)), dim3(256), 0, s, p->P, n, N2,
                       inner);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t nb = G * A * B;
    hipLaunchKernelGGL(k_zero_u32, dim3(static_cast<unsigned>((nb + 255) / 256)), dim3(256), 0, s, blocks, nb);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    TwoLayerArgs a{};
    a.P = p->P;
    a.n = n;
    a.r = p->d_r;
    a.z[0] = p->d_z1;
    a.z[1] = p->d_z2;
    a.z[2] = p->d_z3 ? p->d_z3 : p->d_z2;
    a.z[3] = p->d_z4 ? p->d_z4 : p->d_z2;
    a.e[0] = outer.e1;
    a.e[1] = outer.e2;
    a.e[2] = outer.e3;
    a.e[3] = outer.e4;
    a.ei = inner;
    a.N1 = N1;
    a.N2 = N2;
    a.A = A;
    a.B = B;
    a.blocks = blocks;
    // designs with the same fractions: all of them where the fractions are fixed, a grid row of
    // the (r_2, alpha_1) grid, else each design alone; three and four populations go in the
    // problem's order, whose designs with a last level come first
    const int space = p->P.design_space;
    const bool nested = space == BMD_DESIGN_ALPHA3 || space == BMD_DESIGN_ALPHA4;
    const int64_t shared = nested || (space == BMD_DESIGN_ALPHA && p->P.d == 1) ? G
                           : space == BMD_DESIGN_ALPHA                          ? p->P.stride[0]
                                                                                : 1;
    const int32_t* order = nested ? p->d_order : nullptr;
    e = prec == BMD_FP64 ? launch_counts<double>(a, G, shared, order, p->n_cu, s)
                         : launch_counts<float>(a, G, shared, order, p->n_cu, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_two_layer_final, dim3(static_cast<unsigned>(G)), dim3(64), 0, s, a, mean, var);
    return hipGetLastError();
}

}  // namespace bmd
