// Kernels of the three-dimensional problem (k3.h): the steps of Alg. 1 on the
// 7-point grid around an ellipsoid.
//   k_jumps3    eight lanes per control point: surface derivatives of the
//               density from its fit neighbours (a fixed weighted sum), then
//               the Cartesian jumps from the local frame and shape operator
//               (for the caller; the solves use k_surface3).
//   k_surface3  the jumps along the crossing's own axis and the far-side terms
//               of its interpolation, from the same neighbours.
//   k_fill3     the base right-hand side in the interior layout.
//   k_correct3  one thread per irregular node: the Taylor-corrected jumps of
//               its arms (Alg. 2), added to the right-hand side.
//   k_rows3     one wavefront per (z-mode, y-mode) row: the tridiagonal
//               solve along x (chunked recurrences, as in two dimensions).
//   k_interp3   the ten-node quadratic interpolation (Alg. 3) as fixed
//               weights, plus the jump terms of far-side nodes.
//   k_slab3, k_zgather3  the fast solve of an apply, from the corrections to
//               the stencils' nodes (N <= kSlabMax).
// The sine transforms along z and y are the column transforms of dst.hip,
// applied to the planes of the grid.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device.h"
#include "gmres.h"
#include "graph.h"
#include "k3.h"
#include "plan3.h"

namespace kfbi {

namespace {

constexpr int kFitLanes = 8;       // lanes sharing one control point's neighbour sum in k_jumps3
constexpr int kSurfaceLanes = 16;  // and in k_surface3

__global__ __launch_bounds__(256) void k_jumps3(DevPlan3 p, const double* __restrict__ phi,
                                                const double* __restrict__ fgam, double* __restrict__ J) {
    const int gid = blockIdx.x * blockDim.x + threadIdx.x;
    const int m = gid / kFitLanes, sub = gid % kFitLanes;
    const int M = p.M;
    const bool valid = m < M;
    const double ph = valid ? phi[m] : 0.0;
    // the surface derivatives: each of the point's kFitLanes lanes takes every
    // kFitLanes-th neighbour, then the lanes' sums are combined (fixed order)
    double d0 = 0.0, d1 = 0.0, d2 = 0.0, d3 = 0.0, d4 = 0.0;
    if (valid) {
        for (int e = p.fit_off[m] + sub, e1 = p.fit_off[m + 1]; e < e1; e += kFitLanes) {
            const double dv = phi[p.fit_idx[e]] - ph;
            const double* w = p.fit_w + 5 * (size_t)e;
            d0 = fma(w[0], dv, d0);
            d1 = fma(w[1], dv, d1);
            d2 = fma(w[2], dv, d2);
            d3 = fma(w[3], dv, d3);
            d4 = fma(w[4], dv, d4);
        }
    }
#pragma unroll
    for (int off = kFitLanes / 2; off >= 1; off >>= 1) {
        d0 += __shfl_xor(d0, off, 64);
        d1 += __shfl_xor(d1, off, 64);
        d2 += __shfl_xor(d2, off, 64);
        d3 += __shfl_xor(d3, off, 64);
        d4 += __shfl_xor(d4, off, 64);
    }
    if (!valid || sub != 0) return;
    const double* g = p.geo + 12 * (size_t)m;
    const double nx = g[0], ny = g[1], nz = g[2];
    const double ax = g[3], ay = g[4], az = g[5];     // t1
    const double bx = g[6], by = g[7], bz = g[8];     // t2
    const double s11 = g[9], s12 = g[10], s22 = g[11];
    // tangential block, mixed (tangent, normal) entries, normal-normal entry
    const double h11 = d2, h12 = d3, h22 = d4;
    const double h1n = -(s11 * d0 + s12 * d1);
    const double h2n = -(s12 * d0 + s22 * d1);
    const double F = fgam ? fgam[m] : 0.0;
    const double hnn = F + p.kappa * ph - h11 - h22;
    auto H = [&](double ui, double uj, double vi, double vj, double ni, double nj) {
        return h11 * ui * uj + h22 * vi * vj + h12 * (ui * vj + vi * uj) + h1n * (ui * nj + ni * uj) +
               h2n * (vi * nj + ni * vj) + hnn * ni * nj;
    };
    J[m] = ph;
    J[(size_t)1 * M + m] = d0 * ax + d1 * bx;
    J[(size_t)2 * M + m] = d0 * ay + d1 * by;
    J[(size_t)3 * M + m] = d0 * az + d1 * bz;
    J[(size_t)4 * M + m] = H(ax, ax, bx, bx, nx, nx);
    J[(size_t)5 * M + m] = H(ay, ay, by, by, ny, ny);
    J[(size_t)6 * M + m] = H(az, az, bz, bz, nz, nz);
    J[(size_t)7 * M + m] = H(ax, ay, bx, by, nx, ny);
    J[(size_t)8 * M + m] = H(ax, az, bx, bz, nx, nz);
    J[(size_t)9 * M + m] = H(ay, az, by, bz, ny, nz);
}

// What an apply needs of the surface derivatives: three sums over the fit neighbours
// with weights made once (Apply3Host) in place of five, and three numbers a point in
// place of ten.  What bounds it: the weights' intake (28 bytes a neighbour, 21 MB at
// 128^3 with 25514 points) behind three dependent loads, so sixteen lanes a point with
// two neighbours in flight each: 8.3 us against 12.8 for the ten jumps by eight lanes.
__global__ __launch_bounds__(256) void k_surface3(DevPlan3 p, const double* __restrict__ phi,
                                                  const double* __restrict__ fgam, double2* __restrict__ S,
                                                  double* __restrict__ far, const int* __restrict__ skip,
                                                  DensityCheck check) {
    if (skip && *skip) return;
    const int gid = blockIdx.x * blockDim.x + threadIdx.x;
    const int m = gid / kSurfaceLanes, sub = gid % kSurfaceLanes;
    const int M = p.M;
    const bool valid = m < M;
    const int at = valid ? m : M - 1;
    const double ph = phi[at];
    const int e0 = p.fit_off[at], e1 = p.fit_off[at + 1];
    double g = 0.0, h = 0.0, f = 0.0;
    // (at least kFitMin neighbours; the second of a lane's pair may be past the last)
    for (int e = e0 + sub; e < e1; e += 2 * kSurfaceLanes) {
        const int q = min(e + kSurfaceLanes, e1 - 1);
        const double in = e + kSurfaceLanes < e1 ? 1.0 : 0.0;
        const double va = phi[p.fit_idx[e]] - ph, vb = in * (phi[p.fit_idx[q]] - ph);
        g = fma(p.fit[q], vb, fma(p.fit[e], va, g));
        h = fma(p.fit[(size_t)p.E + q], vb, fma(p.fit[(size_t)p.E + e], va, h));
        f = fma(p.fit[(size_t)2 * p.E + q], vb, fma(p.fit[(size_t)2 * p.E + e], va, f));
    }
#pragma unroll
    for (int off = kSurfaceLanes / 2; off >= 1; off >>= 1) {
        g += __shfl_xor(g, off, 64);
        h += __shfl_xor(h, off, 64);
        f += __shfl_xor(f, off, 64);
    }
    if (check.flag && gid == 0) *check.flag_next = 0;
    if (!valid || sub != 0) return;
    if (check.flag && !isfinite(ph)) {
        *check.flag = 1;
        __hip_atomic_store(check.bad, check.number, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    const double nn = fma(p.kappa, ph, fgam ? fgam[m] : 0.0);
    S[m] = make_double2(g, fma(p.point[m], nn, h));
    far[m] = fma(p.point[(size_t)2 * M + m], ph, fma(p.point[(size_t)M + m], nn, f));
}

__global__ __launch_bounds__(256) void k_fill3(DevPlan3 p, const double* __restrict__ f, double* __restrict__ G,
                                               const int* __restrict__ skip) {
    if (skip && *skip) return;
    const int N = p.N;
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (size_t)N * N * N) return;
    const int i = (int)(idx % N) + 1, j = (int)((idx / N) % N) + 1, k = (int)(idx / ((size_t)N * N)) + 1;
    double v = 0.0;
    if (f && i < N && j < N && k < N) {
        const size_t g = ((size_t)k * (N + 1) + j) * (N + 1) + i;
        if (p.inside[g]) v = f[g];
    }
    G[idx] = v;
}

__global__ __launch_bounds__(256) void k_correct3(DevPlan3 p, const double* __restrict__ phi,
                                                  const double2* __restrict__ S, double* __restrict__ G,
                                                  double* __restrict__ corr, const int* __restrict__ skip) {
    if (skip && *skip) return;
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= p.I) return;
    const double s = p.irr_sign[r];
    double acc = 0.0;
    for (int a = p.arm_off[r], a1 = p.arm_off[r + 1]; a < a1; ++a) {
        const int q = p.arm_q[a];
        const double d = p.arm_d[a];
        const double2 g = S[q];
        const double jv = phi[q] + d * g.x + 0.5 * d * d * g.y;
        acc -= s * jv / p.h2;
    }
    if (G) G[p.irr_node[r]] += acc;
    else corr[p.irr_pos[r]] = acc;
}

template <int C>
__global__ __launch_bounds__(256) void k_rows3(DevPlan3 p, double* __restrict__ G, const int* __restrict__ skip) {
    if (skip && *skip) return;
    const int lane = threadIdx.x & 63;
    const int n = p.N - 1;
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= n * n) return;
    const int kk = r / n, jj = r % n;
    double* row = G + ((size_t)kk * p.N + jj) * p.N;
    double e[C];
#pragma unroll
    for (int c = 0; c < C; ++c) e[c] = row[lane * C + c] * p.h2;
    mode_solve<C>(e, p.modes[r], lane, p.N);
#pragma unroll
    for (int c = 0; c < C; ++c) row[lane * C + c] = e[c];
}

// The fast solve between corrections and stencils: nothing of the grid is read or
// written but the half planes W.  One workgroup per z-mode l and parity of the y-modes:
// the folded rows y' = 1..H (H = N / 2) of the corrections' sine sums along z, u(y) +
// u(N - y) for the odd y-modes and u(y) - u(N - y) for the even ones; their H x H sine
// transform along y by the FP64 matrix cores; the tridiagonal solves along x of its H
// modes; the transform back, whose rows are the symmetric (odd modes) or antisymmetric
// part of the solution in y.  The half plane (64 KiB at N = 128) stays in LDS, and twice
// N - 1 workgroups fill the chip.
// What bounds it: the corrections' intake (a compute unit takes in 64 bytes a clock) and
// a table lookup a piece, the matrix cores (3.4 us a product at N = 128 if every row has
// nodes), and seven barriers of one workgroup a compute unit.  At 128^3 with 29360 nodes
// it takes 18 us (sums 4.5, product 3.6, solves 1.5, product back and store 4); the
// launches it replaces took 68: fill 7.7, corrections added 5.8, transforms 14 + 14, row
// solves 12, transform back 14.
typedef double f64x4 __attribute__((ext_vector_type(4)));
// The sines sin(pi k / N), k = 0..2N-1, in LDS, entry k at tslot(k): reads at a power
// of two times the lane's index then land on distinct banks.
__device__ __forceinline__ int tslot(int k) { return k + (k >> 5); }
template <int C>
constexpr int table_len() {
    return 128 * C + 4 * C;
}
template <int C>
constexpr int slab_stride() {
    return 64 * C + 16;         // N and the lanes' gaps; a matrix-core operand's four rows 32 banks apart
}
// weighted scan over each row of 16 lanes with multiplier m a lane, up (kDppRowShr1) or
// down (kDppRowShl1); the sum over each row, the same in its lanes
template <int SHIFT>
__device__ __forceinline__ double row16_scan(double v, double m) {
    const double m2 = m * m, m4 = m2 * m2;
    v = fma(m, dpp_f64<SHIFT>(v), v);
    v = fma(m2, dpp_f64<SHIFT + 1>(v), v);
    v = fma(m4, dpp_f64<SHIFT + 3>(v), v);
    return fma(m4 * m4, dpp_f64<SHIFT + 7>(v), v);
}
__device__ __forceinline__ double row16_sum(double v) {
    v += dpp_f64<kDppQuadSwap1>(v);
    v += dpp_f64<kDppQuadSwap2>(v);
    v += dpp_f64<kDppRowHalfMirror>(v);
    return v + dpp_f64<kDppRowMirror>(v);
}
template <int C>
constexpr int slab_threads() {
    return 512 * C;
}
template <int C>
constexpr size_t slab_lds() {
    return sizeof(double) * (table_len<C>() + 32 * C * slab_stride<C>());
}
// sin(pi k / N), k = 0..2N-1, by the whole workgroup
template <int C>
__device__ __forceinline__ void sine_table(const double* __restrict__ sinq, double* tab) {
    constexpr int N = 64 * C;
    for (int k = threadIdx.x; k < 2 * N; k += blockDim.x) {
        const int q = k & (N - 1);
        const double s = sinq[min(q, N - q)];
        tab[tslot(k)] = k < N ? s : -s;
    }
}
constexpr int kSlabBatch = 4;                                // pieces whose loads a lane issues together
template <int C>
__global__ __launch_bounds__(slab_threads<C>()) void k_slab3(DevPlan3 p, const double* __restrict__ corr,
                                                           double* __restrict__ W, const int* __restrict__ skip) {
    constexpr int N = 64 * C, H = N / 2, XS = slab_stride<C>(), NW = 8 * C, RT = H / 16, KS = H / 4, K = N / 16;
    auto place = [](int x) { return x + x / K; };            // of column x: see the solves
    extern __shared__ double smem[];
    double* tab = smem;
    double* X = smem + table_len<C>();
    if (skip && *skip) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l = 1 + (int)(blockIdx.x >> 1), even = blockIdx.x & 1;
    sine_table<C>(p.sinq, tab);
    for (int k = tid; k < H * XS; k += slab_threads<C>()) X[k] = 0.0;
    __syncthreads();
    // the sums along z, a piece a lane: its four nodes share the sine up to sign.  All of
    // a batch's loads first
    const double sz = l & 1 ? 1.0 : -1.0, sy = even ? -1.0 : 1.0;
    const int r1 = p.sp_wave[wave + 1];
    for (int r = p.sp_wave[wave]; r < r1; r += kSlabBatch) {
        double2 c[kSlabBatch][2];
        int at[kSlabBatch];
#pragma unroll
        for (int u = 0; u < kSlabBatch; ++u) {
            const size_t piece = (size_t)min(r + u, r1 - 1) * 64 + lane;
            at[u] = p.sp_piece[piece];
            c[u][0] = reinterpret_cast<const double2*>(corr)[2 * piece];
            c[u][1] = reinterpret_cast<const double2*>(corr)[2 * piece + 1];
        }
#pragma unroll
        for (int u = 0; u < kSlabBatch; ++u) {
            if (r + u >= r1 || at[u] < 0) continue;
            const double v = fma(sz, c[u][0].y, c[u][0].x) + sy * fma(sz, c[u][1].y, c[u][1].x);
            X[(at[u] >> 8 & 255) * XS + place(at[u] & 255)] += v * tab[tslot(((at[u] >> 16) * l) & (2 * N - 1))];
        }
    }
    // the constants of the lane's row (below), requested before the product
    const int own = wave * 4 + (lane >> 4), sub = lane & 15;
    const ModeConst& mode = p.modes[(size_t)(l - 1) * (N - 1) + min(2 * own + 1 + even, N - 1) - 1];
    const double mr = mode.r, msmc = mode.smc, mrN1 = mode.rN1;
    __syncthreads();
    // Y[i][x] = sum_y sin(pi m y / N) X[y][x] with m = 2 i + 1 (+ 1 for the even modes:
    // the last, m = N, is zero), and the same transposed: element (i, y) is
    // entry m y mod 2N of the table either way
    const int rt = wave % RT, ct = wave / RT, ar = lane & 15, ak = lane >> 4;
    f64x4 acc[C];
    auto product = [&](auto transposed) {
        constexpr bool back = decltype(transposed)::value;
        const int row = rt * 16 + ar;
#pragma unroll
        for (int t = 0; t < C; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
        // forward, the rows below the first with a node are zero
#pragma unroll 4
        for (int ks = back ? 0 : p.y_first / 4; ks < KS; ++ks) {
            const int k = 4 * ks + ak;
            const int m = 2 * (back ? k : row) + 1 + even, y = (back ? row : k) + 1;
            const double a = tab[tslot((m * y) & (2 * N - 1))];
#pragma unroll
            for (int t = 0; t < C; ++t)
                acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, X[k * XS + place((ct + 4 * t) * 16 + ar)], acc[t], 0, 0, 0);
        }
    };
    product(std::false_type{});
    __syncthreads();
#pragma unroll
    for (int t = 0; t < C; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) X[(rt * 16 + 4 * r + ak) * XS + place((ct + 4 * t) * 16 + ar)] = acc[t][r];
    __syncthreads();
    // The solves along x, and both transforms' factors 2 / N: sixteen lanes a row, K nodes
    // each (a gap after each lane's share spreads them over the banks).  The recurrences
    // of the sparse fast solve in two dimensions (device.h): the forward one from w0, which
    // carries the rank-one fix, and the backward one, each run once for the carry and once
    // from it.  The even modes' last row, m = N, is zero and stays so
    static_assert(H == 4 * NW, "four rows a wavefront");
    {
        double* row = X + own * XS + sub * (K + 1);
        const double r = mr, r2 = r * r, r4 = r2 * r2;
        const double rK = K == 4 ? r4 : r4 * r4, rsub = pow_u<4>(rK, sub);
        double e[K], w = 0.0, g = 0.0;
#pragma unroll
        for (int c = 0; c < K; ++c) {
            e[c] = row[c] * (p.h2 * r);
            w = fma(r, w, -e[c]);
        }
#pragma unroll
        for (int c = K - 1; c >= 0; --c) g = fma(r, g, e[c]);
        const double up = row16_scan<kDppRowShr1>(w, rK);
        const double total = row16_sum(fma(g, rsub, sub == 15 ? mrN1 * up : 0.0));
        w = fma(rsub, -msmc * total, dpp_f64<kDppRowShr1>(up));
#pragma unroll
        for (int c = 0; c < K; ++c) {
            w = fma(r, w, -e[c]);
            e[c] = w;
        }
        if (sub == 15) e[K - 1] = 0.0;                       // node N
        double y = 0.0;
#pragma unroll
        for (int c = K - 1; c >= 0; --c) y = fma(r, y, e[c]);
        y = dpp_f64<kDppRowShl1>(row16_scan<kDppRowShl1>(y, rK));
        const double scale = 4.0 / ((double)N * N);
#pragma unroll
        for (int c = K - 1; c >= 0; --c) {
            y = fma(r, y, e[c]);
            row[c] = y * scale;
        }
    }
    __syncthreads();
    if (rt * 16 + 15 < p.y_first) return;                    // no node there
    product(std::true_type{});
    double* out = W + (size_t)(2 * (l - 1) + even) * H * N;
#pragma unroll
    for (int t = 0; t < C; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) out[(size_t)(rt * 16 + 4 * r + ak) * N + (ct + 4 * t) * 16 + ar] = acc[t][r];
}

// The inverse transform along z at the stencils' nodes alone: one workgroup per tile of
// 32 folded columns, whose N - 1 modes (both parts' sum and difference: the columns y
// and N - y) it holds in LDS.  Four lanes share an entry's sums, the odd modes' in two and
// the even modes' in two: their sum and difference are the nodes z and N - z.
// What bounds it: the half planes' intake, then LDS reads (a mode and two sines for two
// multiply-adds).  8 us at 128^3, where the transform of the whole grid took 14.
constexpr int kZCols = 32, kZStride = kZCols + 1, kZThreads = 1024;
template <int C>
constexpr size_t zgather_lds() {
    return sizeof(double) * (table_len<C>() + 2 * (64 * C - 1) * kZStride);
}
template <int C>
__global__ __launch_bounds__(kZThreads) void k_zgather3(DevPlan3 p, const double* __restrict__ W,
                                                        double* __restrict__ val, const int* __restrict__ skip) {
    constexpr int N = 64 * C, H = N / 2;
    extern __shared__ double smem[];
    double* tab = smem;
    double* part = smem + table_len<C>();                    // sums, then differences
    constexpr int PD = (N - 1) * kZStride;
    const int q0 = p.zg_off[blockIdx.x], q1 = p.zg_off[blockIdx.x + 1];
    if (q0 == q1 || (skip && *skip)) return;
    const int tid = threadIdx.x, row = blockIdx.x / (N / kZCols), x0 = blockIdx.x % (N / kZCols) * kZCols;
    sine_table<C>(p.sinq, tab);
    constexpr int LB = (N * kZCols + kZThreads - 1) / kZThreads;
    double a[LB], b[LB];
#pragma unroll
    for (int u = 0; u < LB; ++u) {
        const int k = min(u * kZThreads + tid, (N - 1) * kZCols - 1), l = k / kZCols, x = x0 + k % kZCols;
        a[u] = W[((size_t)(2 * l) * H + row) * N + x];
        b[u] = W[((size_t)(2 * l + 1) * H + row) * N + x];
    }
#pragma unroll
    for (int u = 0; u < LB; ++u) {
        const int k = min(u * kZThreads + tid, (N - 1) * kZCols - 1), at = k / kZCols * kZStride + k % kZCols;
        part[at] = a[u] + b[u];
        part[PD + at] = a[u] - b[u];
    }
    __syncthreads();
    const int sub = tid & 3;
    for (int base = q0; base < q1; base += kZThreads / 4) {
        const int q = base + (tid >> 2), code = p.zg_code[min(q, q1 - 1)];
        const int z1 = code & 255, z2 = code >> 8 & 255;
        const double* v = part + (code >> 24) * PD + (code >> 16 & 31);
        double s1 = 0.0, s2 = 0.0;
#pragma unroll 8
        for (int i = 0; i < N / 4; ++i) {
            const int l = 1 + sub + 4 * i;
            if (l < N) {
                const double x = v[(l - 1) * kZStride];
                s1 = fma(x, tab[tslot((z1 * l) & (2 * N - 1))], s1);
                s2 = fma(x, tab[tslot((z2 * l) & (2 * N - 1))], s2);
            }
        }
        s1 += __shfl_xor(s1, 2, 64);
        s2 += __shfl_xor(s2, 2, 64);
        const double t1 = __shfl_xor(s1, 1, 64), t2 = __shfl_xor(s2, 1, 64);
        // sub 0 has the odd modes' sums and sub 1 the even ones'
        if (sub == 0 && q < q1) {
            reinterpret_cast<double2*>(val)[2 * (size_t)q] = make_double2(s1 + t1, s1 - t1);
            reinterpret_cast<double2*>(val)[2 * (size_t)q + 1] = make_double2(s2 + t2, s2 - t2);
        }
    }
}

__global__ __launch_bounds__(256) void k_interp3(DevPlan3 p, const double* __restrict__ v, const int* __restrict__ node,
                                                 const double* __restrict__ far, double* __restrict__ out,
                                                 const int* __restrict__ skip) {
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= p.M || (skip && *skip)) return;
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < kStencil3; ++k) {
        const int at = node[(size_t)k * p.M + m];
        s = fma(p.st_w[(size_t)k * p.M + m], at >= 0 ? v[at] : 0.0, s);
    }
    out[m] = s + far[m];
}

// inside GMRES: v+ at 64 NC control points (a wavefront for each of the ten nodes,
// one for the far-side terms), then the reduce part of the step; the last workgroup
// commits the previous column
template <int NC>
__global__ __launch_bounds__(1024) void k_interp3_gm(DevPlan3 p, const double* __restrict__ v,
                                                     const int* __restrict__ node, const double* __restrict__ far,
                                                     GmresBufs b) {
    __shared__ double red[kStencil3 + 1][64 * NC];
    if ((int)blockIdx.x == b.gc64) {
        gm_commit(b, p.M);
        return;
    }
    if (b.st->converged) return;
    const GmPre<NC> pre = gm_reduce_prefetch<NC>(b, p.M, blockIdx.x);
    const GmPh ph{b.st->ph, b.st->j, b.st->second, b.st->reorth};
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m0 = blockIdx.x * 64 * NC + lane;
    if (wave <= kStencil3) {
        int at[NC];
        double w[NC];
#pragma unroll
        for (int h = 0; h < NC; ++h) {
            const int m = min(m0 + 64 * h, p.M - 1);
            at[h] = wave < kStencil3 ? node[(size_t)wave * p.M + m] : m;
            w[h] = wave < kStencil3 ? p.st_w[(size_t)wave * p.M + m] : 1.0;
        }
        const double* from = wave < kStencil3 ? v : far;
#pragma unroll
        for (int h = 0; h < NC; ++h) red[wave][64 * h + lane] = at[h] >= 0 ? w[h] * from[at[h]] : 0.0;
    }
    __syncthreads();
    if (wave < NC) {
        double s = 0.0;
#pragma unroll
        for (int k = 0; k <= kStencil3; ++k) s += red[k][64 * wave + lane];
        red[0][64 * wave + lane] = m0 + 64 * wave < p.M ? s : 0.0;
    }
    __syncthreads();
    gm_reduce64<NC>(b, p.M, blockIdx.x, red[0], pre, ph);
}

__global__ __launch_bounds__(256) void k_grid_out3(DevPlan3 p, const double* __restrict__ G, int mask,
                                                   double* __restrict__ u) {
    const int N = p.N, W = N + 1;
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (size_t)W * W * W) return;
    const int i = (int)(idx % W), j = (int)((idx / W) % W), k = (int)(idx / ((size_t)W * W));
    double v = 0.0;
    if (i >= 1 && j >= 1 && k >= 1 && i < N && j < N && k < N) v = G[((size_t)(k - 1) * N + (j - 1)) * N + (i - 1)];
    if (mask && !p.inside[idx]) v = 0.0;
    u[idx] = v;
}

}  // namespace

hipError_t launch_jumps3(const DevPlan3& p, const double* phi, const double* fgam, double* J, hipStream_t s) {
    const size_t threads = (size_t)p.M * kFitLanes;
    return klaunch(&k_jumps3, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, p, phi, fgam, J);
}

hipError_t launch_surface3(const DevPlan3& p, const double* phi, const double* fgam, double2* S, double* far,
                           const int* skip, const DensityCheck* check, hipStream_t s) {
    const size_t threads = (size_t)p.M * kSurfaceLanes;
    return klaunch(&k_surface3, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, p, phi, fgam, S, far, skip,
                   check ? *check : DensityCheck{});
}

hipError_t launch_fill3(const DevPlan3& p, const double* f, double* G, const int* skip, hipStream_t s) {
    const size_t tot = (size_t)p.N * p.N * p.N;
    if (hipError_t e = klaunch(&k_fill3, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, p, f, G, skip))
        return e;
    return hipGetLastError();
}

hipError_t launch_correct3(const DevPlan3& p, const double* phi, const double2* S, double* G, double* corr,
                           const int* skip, hipStream_t s) {
    if (p.I == 0) return hipSuccess;
    return klaunch(&k_correct3, dim3((p.I + 255) / 256), dim3(256), 0, s, p, phi, S, G, corr, skip);
}

namespace {
template <int C>
hipError_t solve3_sparse(const DevPlan3& p, const double* corr, double* W, double* val, const int* skip, hipStream_t s) {
    constexpr int N = 64 * C;
    if (hipError_t e = hipFuncSetAttribute((const void*)k_slab3<C>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)slab_lds<C>()))
        return e;
    if (hipError_t e = hipFuncSetAttribute((const void*)k_zgather3<C>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)zgather_lds<C>()))
        return e;
    if (hipError_t e = klaunch(&k_slab3<C>, dim3(2 * (N - 1)), dim3(slab_threads<C>()), slab_lds<C>(), s, p, corr, W, skip))
        return e;
    return klaunch(&k_zgather3<C>, dim3(N / 2 * (N / kZCols)), dim3(kZThreads), zgather_lds<C>(), s, p, (const double*)W,
                   val, skip);
}
}  // namespace

hipError_t launch_solve3_sparse(const DevPlan3& p, const double* corr, double* W, double* val, const int* skip,
                                hipStream_t s) {
    switch (p.N) {
        case 64: return solve3_sparse<1>(p, corr, W, val, skip, s);
        case 128: return solve3_sparse<2>(p, corr, W, val, skip, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_solve3(const DevPlan3& p, double* G, int B, const int* skip, hipStream_t s) {
    const int N = p.N;
    const size_t plane = (size_t)N * N;
    const double inv = 2.0 / N;
    // along z: N^2 columns of N rows, rows N^2 apart
    if (hipError_t e = launch_dst_lines(N, p.log2N, p.sinq, G, 1.0, B, N * N, 1, 0, skip, s)) return e;
    // along y: each of the N-1 interior planes, rows N apart
    if (hipError_t e = launch_dst_lines(N, p.log2N, p.sinq, G, 1.0, B, N, N - 1, plane, skip, s)) return e;
    const int rows = (N - 1) * (N - 1);
    const dim3 g((rows + 3) / 4), t(256);
    hipError_t e = hipSuccess;
    switch (N) {
        case 64: e = klaunch(&k_rows3<1>, g, t, 0, s, p, G, skip); break;
        case 128: e = klaunch(&k_rows3<2>, g, t, 0, s, p, G, skip); break;
        case 256: e = klaunch(&k_rows3<4>, g, t, 0, s, p, G, skip); break;
        default: return hipErrorInvalidValue;
    }
    if (e) return e;
    if (hipError_t e2 = launch_dst_lines(N, p.log2N, p.sinq, G, inv, B, N, N - 1, plane, skip, s)) return e2;
    return launch_dst_lines(N, p.log2N, p.sinq, G, inv, B, N * N, 1, 0, skip, s);
}

hipError_t launch_interp3(const DevPlan3& p, const double* v, const int* node, const double* far, double* out,
                          const int* skip, const GmresBufs* gm, hipStream_t s) {
    if (gm && reduce3_chunks(p.M) == 4)
        return klaunch(&k_interp3_gm<4>, dim3(gm->gc64 + 1), dim3(1024), 0, s, p, v, node, far, *gm);
    if (gm) return klaunch(&k_interp3_gm<1>, dim3(gm->gc64 + 1), dim3(1024), 0, s, p, v, node, far, *gm);
    return klaunch(&k_interp3, dim3((p.M + 255) / 256), dim3(256), 0, s, p, v, node, far, out, skip);
}

hipError_t launch_grid_out3(const DevPlan3& p, const double* G, bool mask, double* u, hipStream_t s) {
    const size_t tot = (size_t)(p.N + 1) * (p.N + 1) * (p.N + 1);
    if (hipError_t e = klaunch(&k_grid_out3, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, p, G,
                               mask ? 1 : 0, u))
        return e;
    return hipGetLastError();
}

}  // namespace kfbi
