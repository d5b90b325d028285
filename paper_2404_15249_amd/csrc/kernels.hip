// HIP kernels of the KFBI hot path for gfx950 (MI355X), FP64.
//
// One K_D apply (Sec. 3, Alg. 1 steps 4-6) is three launches:
//   k_density  the density's check and spline and, one thread per irregular
//              node, the jumps at the crossings on its arms (Alg. 2 line 4) and
//              the correction of its right-hand side (Alg. 2 line 5).  For the
//              double-layer apply F = 0, so the right-hand side of the corrected
//              system is nonzero only here.  Inside GMRES the step launch of
//              gmres.h makes them for the next input.
//   k_modes    the fast solver (Alg. 4) restricted to what the interpolation
//              reads, R sine modes per workgroup.  Along y the right-hand side
//              is expanded in sines; for a sparse right-hand side each
//              coefficient is a short sum over the irregular nodes of one grid
//              column.  Along x each sine mode is a constant-coefficient
//              tridiagonal system, solved by one wavefront as two first-order
//              recurrences (chunked, with wave-wide carry scans) plus a rank-one
//              boundary fix.  The inverse sine sum along y is evaluated only at
//              the six stencil nodes of each boundary sample, already weighted
//              by the interpolation weights, and written as the workgroup's row
//              of partial sums.
//   k_reduce_interp  64 samples per workgroup of sixteen wavefronts: the partials
//              summed in a fixed order plus the jump terms of the stencil nodes
//              outside Omega (Alg. 3); inside GMRES k_reduce_gm, with the dots.
// k_correct and k_spline are launches of their own where only one of them is
// wanted (given jumps, the FP32 interface solves, timed applies).
// The dense solve (volume potential, final solution) stands between two column
// sine transforms (dst.hip): k_modes_dense, which adds the corrections' sums and
// makes the samples' partials, or the rows' tridiagonal solves alone
// (k_rows_solve; in the FP32 mode on FP32 rows).
#include <hip/hip_runtime.h>

#include "device.h"
#include "gmres.h"
#include "graph.h"
#include "kernels.h"

namespace kfbi {

namespace {

// ---------------------------------------------------------------- correction (Alg. 2)

__global__ __launch_bounds__(256) void k_correct(DevPlan p, JumpSrc js, double* __restrict__ corr,
                                                 double* __restrict__ corr_il, double* __restrict__ dense,
                                                 const int* __restrict__ skip) {
    if (skip && *skip) return;
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= p.I) return;
    const double acc = correction_at(p, js, r);
    if (corr) corr[r] = acc;
    if (corr_il) corr_il[p.il_pos[r]] = acc;
    if (dense) dense[(size_t)(p.irr_j[r] - 1) * p.N + (p.irr_i[r] - 1)] += acc;
}

// ---------------------------------------------------------------- sparse fast solve + weighted gather

template <int C, int R>
__global__ __launch_bounds__(kModeWaves * 64) void k_modes(DevPlan p, const double* __restrict__ corr,
                                                          double* __restrict__ partial, const int* __restrict__ skip) {
    extern __shared__ double smem[];
    const ModesLds L = modes_lds<C>(smem);
    double* row = partial + (size_t)blockIdx.x * p.M;
    modes_round<C, R, true, false>(p, corr, blockIdx.x, L, [&](int, int cp, double v) { row[cp] = v; }, skip);
}

// The same with the whole grid's transformed right-hand side (see ModesDense): the
// row solves of an interface solve, its corrections and its samples in one launch.
// What bounds it is what bounds k_modes, then the grid's rows (read once, written
// once): 15 us at 2048^2 where only the samples are wanted and 19 with the rows
// stored, against 13.4 (the row solves alone) + 5.7 (corrections on the grid) + 4.5
// (interpolation), and an inverse transform of 23 where only the samples are wanted;
// at 1024^2 7 and 9, at 4096^2 108 (of which the corrections' sums make half).
template <int C, int R>
__global__ __launch_bounds__(kModeWaves * 64) void k_modes_dense(DevPlan p, const double* __restrict__ corr,
                                                                ModesDense dn, double* __restrict__ partial,
                                                                double* __restrict__ partial2) {
    extern __shared__ double smem[];
    const ModesLds L = modes_lds<C>(smem);
    const size_t at = (size_t)blockIdx.x * p.M;
    modes_round<C, R, true, true>(
        p, corr, blockIdx.x, L, [&](int set, int cp, double v) { (set ? partial2 : partial)[at + cp] = v; }, nullptr, dn);
}

// ---------------------------------------------------------------- spline of a density

__global__ __launch_bounds__(256) void k_spline(DevPlan p, const double* __restrict__ y, double* __restrict__ s2,
                                                const int* __restrict__ skip) {
    if (skip && *skip) return;
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m < p.M) s2[m] = spline_s2(y, p.M, p.taps, m);
}

// ---------------------------------------------------------------- interpolation (Alg. 3)

// 64 samples per workgroup of 16 wavefronts (reduce_samples64).
__global__ __launch_bounds__(1024) void k_reduce_interp(DevPlan p, JumpSrc js, const double* __restrict__ partial,
                                                        int G, double* __restrict__ out, const int* __restrict__ skip,
                                                        const double* __restrict__ from) {
    __shared__ double red[16 * 64];
    reduce_samples64(p, js, partial, G, blockIdx.x * 64, out, red, skip, from);
}

// Interpolation from a full grid solution (dense path): V in the padded interior
// layout, or (user) the caller's grid.
__global__ __launch_bounds__(256) void k_interp_grid(DevPlan p, JumpSrc js, const double* __restrict__ V, int user,
                                                     double* __restrict__ out) {
    const int cp = blockIdx.x * blockDim.x + threadIdx.x;
    if (cp >= p.M) return;
    int ni[6], nj[6];
    stencil_nodes(p, cp, ni, nj);
    const double* w = p.cp_w + cp;
    double s = 0.0;
    for (int k = 0; k < 6; ++k) s += w[(size_t)k * p.M] * (user ? V[(size_t)nj[k] * (p.N + 1) + ni[k]] : V[(size_t)(nj[k] - 1) * p.N + (ni[k] - 1)]);
    out[cp] = s + outside_terms(p, js, cp, ni, nj, w, p.M);
}

// ---------------------------------------------------------------- dense path

// R (N x N, interior node (i, j) at (j-1) N + (i-1), row/column N-1 zero pad)
// from a grid array; `mask` keeps only nodes in Omega (the zero extension f~).
__global__ __launch_bounds__(256) void k_fill_rhs(DevPlan p, const double* __restrict__ f, int mask,
                                                  double* __restrict__ R) {
    const int N = p.N;
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (size_t)N * N) return;
    const int i = (int)(idx % N) + 1, j = (int)(idx / N) + 1;
    double v = 0.0;
    if (i < N && j < N) {
        const size_t g = (size_t)j * (N + 1) + i;
        v = f ? f[g] : 0.0;
        if (mask && !p.inside[g]) v = 0.0;
    }
    R[idx] = v;
}

// One wavefront per sine mode l (row l-1 of A): the tridiagonal solve along x,
// in FP64 whatever the storage type T.  The solve wants each lane's C
// consecutive values in registers; the row goes through LDS so that the global
// loads and stores stay coalesced (lane-consecutive), one skipped slot per C
// values keeping the lanes' chunk reads on distinct banks.  Rows per
// workgroup: 4 up to C = 16, 2 at C = 32, 1 at C = 64 (33.8 KB of LDS).
template <int C>
constexpr int rows_per_group() { return C <= 16 ? 4 : C == 32 ? 2 : 1; }

template <int C, class T>
__global__ __launch_bounds__(64 * rows_per_group<C>()) void k_rows_solve(DevPlan p, T* __restrict__ A) {
    constexpr int RPW = rows_per_group<C>(), W = 64 * C, WP = W + 64;
    __shared__ double rs[RPW][WP];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int l = blockIdx.x * RPW + w + 1;
    const bool live = l <= p.n;                          // the barriers below are the workgroup's
    T* row = A + (size_t)(l - 1) * p.N;
    double* r = rs[w];
    auto pad = [](int e) { return e + e / C; };
    if (live) {
#pragma unroll 8
        for (int c = 0; c < C; ++c) r[pad(c * 64 + lane)] = (double)row[c * 64 + lane] * p.h2;
    }
    __syncthreads();
    double e[C];
    if (live) {
#pragma unroll
        for (int c = 0; c < C; ++c) e[c] = r[pad(lane * C + c)];
        mode_solve<C>(e, p.modes[l], lane, p.N);
#pragma unroll
        for (int c = 0; c < C; ++c) r[pad(lane * C + c)] = e[c];
    }
    __syncthreads();
    if (live) {
#pragma unroll 8
        for (int c = 0; c < C; ++c) row[c * 64 + lane] = (T)r[pad(c * 64 + lane)];
    }
}

__global__ __launch_bounds__(256) void k_grid_out(DevPlan p, const double* __restrict__ R, int mask,
                                                  double* __restrict__ u) {
    const int W1 = p.N + 1;
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (size_t)W1 * W1) return;
    const int i = (int)(idx % W1), j = (int)(idx / W1);
    double v = 0.0;
    if (i >= 1 && j >= 1 && i <= p.n && j <= p.n) v = R[(size_t)(j - 1) * p.N + (i - 1)];
    if (mask && !p.inside[idx]) v = 0.0;
    u[idx] = v;
}

__global__ __launch_bounds__(256) void k_axpby(int n, double a, const double* __restrict__ x, double b,
                                               const double* __restrict__ y, double* __restrict__ z) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) z[i] = a * x[i] + (y ? b * y[i] : 0.0);
}

__global__ __launch_bounds__(256) void k_fill(size_t n, double v, double* __restrict__ x) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = v;
}

// flag <- 1 if any of x[0..n) is NaN or Inf, else 0: one workgroup, which
// writes the flag whatever it finds (nothing to clear beforehand)
__global__ __launch_bounds__(256) void k_nonfinite(int n, const double* __restrict__ x, int* __restrict__ flag) {
    __shared__ int any;
    if (threadIdx.x == 0) any = 0;
    __syncthreads();
    int bad = 0;
    for (int i = threadIdx.x; i < n; i += 256) bad |= !isfinite(x[i]);
    if (bad) any = 1;                                    // benign race: every writer stores 1
    __syncthreads();
    if (threadIdx.x == 0) *flag = any;
}

// ---------------------------------------------------------------- GMRES step (Alg. 5)

// the apply's last launch inside GMRES: its output at 64 samples, then the reduce
// part of the step; the last workgroup commits the previous column
__global__ __launch_bounds__(1024) void k_reduce_gm(DevPlan p, JumpSrc js, const double* __restrict__ partial, int G,
                                                    GmresBufs b) {
    __shared__ double red[16 * 64];
    if ((int)blockIdx.x == b.gc64) {
        gm_commit(b, p.M);
        return;
    }
    const GmPre<1> pre = gm_reduce_prefetch(b, p.M, blockIdx.x);
    const GmPh ph{load_flag_late(&b.st->ph), load_flag_late(&b.st->j), load_flag_late(&b.st->second),
                  load_real_late(&b.st->reorth)};       // waited for where used
    if (!reduce_samples64(p, js, partial, G, blockIdx.x * 64, nullptr, red, &b.st->converged)) return;
    gm_reduce64(b, p.M, blockIdx.x, red, pre, ph);
}
__global__ __launch_bounds__(kGmChunk) void k_gm_begin(DevPlan p, int has_p, const double* taps, GmresBufs b, int M,
                                                       const double* rhs, const double* phi_in, double tol,
                                                       int max_iter, double reorth, double* xout, double* corr_il,
                                                       unsigned epoch) {
    gm_begin(has_p ? &p : nullptr, taps, b, M, rhs, phi_in, tol, max_iter, reorth, xout, corr_il, epoch);
}
__global__ __launch_bounds__(kGmChunk) void k_gm_step(const double* taps, GmresBufs b, int M) {
    gm_step(taps, b, M, blockIdx.x);
}
// the step launch with the next apply's corrections: workgroups 0 .. gc-1 make the
// vector's chunks, the rest one correction chunk each
__global__ __launch_bounds__(kGmChunk) void k_gm_step_corr(DevPlan p, GmresBufs b, double* __restrict__ corr_il) {
    if ((int)blockIdx.x < b.gc) {
        gm_step(p.taps, b, p.M, blockIdx.x);
    } else {
        gm_step_corrections(p, b, (int)blockIdx.x - b.gc, corr_il);
    }
}

__global__ __launch_bounds__(kGmChunk) void k_density(DevPlan p, const double* __restrict__ y, double* __restrict__ s2,
                                                      double* __restrict__ corr_il, int gc, const int* __restrict__ skip,
                                                      int* flag, int* flag_next, unsigned* bad, unsigned number) {
    if (skip && *skip) return;
    gm_density(p, y, s2, corr_il, gc, flag, flag_next, bad, number);
}

// The same for an interface solve: the density y and f on Gamma (either null: zero).
__global__ __launch_bounds__(kGmChunk) void k_density_f(DevPlan p, const double* __restrict__ y,
                                                        const double* __restrict__ f, double* __restrict__ s2,
                                                        double* __restrict__ f2, double* __restrict__ corr_il, int gc) {
    gm_density_f(p, y, f, s2, f2, corr_il, gc);
}

// One launch of the sparse fast solve: the apply's (dn null) or an interface solve's.
struct ModesArgs {
    const double* corr;
    double *partial, *partial2;
    const int* skip;
    const ModesDense* dn;
};

template <int C, int R>
hipError_t modes_launch(const DevPlan& p, const ModesArgs& a, hipStream_t s) {
    constexpr size_t lds = sizeof(double) * modes_lds_len<C, R>();
    if constexpr (lds > 160 * 1024) {
        return hipErrorInvalidValue;                  // never fits the local data share
    } else {
        const void* f = a.dn ? (const void*)k_modes_dense<C, R> : (const void*)k_modes<C, R>;
        if (hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)) return e;
        const dim3 groups((p.n + R - 1) / R), t(kModeWaves * 64);
        if (a.dn) return klaunch(&k_modes_dense<C, R>, groups, t, lds, s, p, a.corr, *a.dn, a.partial, a.partial2);
        return klaunch(&k_modes<C, R>, groups, t, lds, s, p, a.corr, a.partial, a.skip);
    }
}

template <int C>
hipError_t modes_dispatch_r(const DevPlan& p, int R, const ModesArgs& a, hipStream_t s) {
    switch (R) {
        case 1: return modes_launch<C, 1>(p, a, s);
        case 2: return modes_launch<C, 2>(p, a, s);
        case 4: return modes_launch<C, 4>(p, a, s);
        case 8: return modes_launch<C, 8>(p, a, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t modes_dispatch(const DevPlan& p, int R, const ModesArgs& a, hipStream_t s) {
    switch (p.N) {
        case 64: return modes_dispatch_r<1>(p, R, a, s);
        case 128: return modes_dispatch_r<2>(p, R, a, s);
        case 256: return modes_dispatch_r<4>(p, R, a, s);
        case 512: return modes_dispatch_r<8>(p, R, a, s);
        case 1024: return modes_dispatch_r<16>(p, R, a, s);
        case 2048: return modes_dispatch_r<32>(p, R, a, s);
        case 4096: return modes_dispatch_r<64>(p, R, a, s);
        default: return hipErrorInvalidValue;
    }
}

template <int C, class T>
hipError_t rows_dispatch(const DevPlan& p, T* A, hipStream_t s) {
    constexpr int RPW = rows_per_group<C>();
    if (hipError_t e_ = klaunch(&k_rows_solve<C, T>, dim3((p.n + RPW - 1) / RPW), dim3(64 * RPW), 0, s, p, A))
        return e_;
    return hipGetLastError();
}

template <class T>
hipError_t rows_solve_any(const DevPlan& p, T* A, hipStream_t s) {
    switch (p.N) {
        case 64: return rows_dispatch<1>(p, A, s);
        case 128: return rows_dispatch<2>(p, A, s);
        case 256: return rows_dispatch<4>(p, A, s);
        case 512: return rows_dispatch<8>(p, A, s);
        case 1024: return rows_dispatch<16>(p, A, s);
        case 2048: return rows_dispatch<32>(p, A, s);
        case 4096: return rows_dispatch<64>(p, A, s);
        default: return hipErrorInvalidValue;
    }
}

template <int C>
size_t modes_lds_bytes_r(int R) {
    return sizeof(double) * (R <= 1 ? modes_lds_len<C, 1>() : R == 2 ? modes_lds_len<C, 2>() : R == 4 ? modes_lds_len<C, 4>()
                                                                                            : modes_lds_len<C, 8>());
}

}  // namespace

size_t modes_lds_bytes(int N, int R) {
    switch (N) {
        case 64: return modes_lds_bytes_r<1>(R);
        case 128: return modes_lds_bytes_r<2>(R);
        case 256: return modes_lds_bytes_r<4>(R);
        case 512: return modes_lds_bytes_r<8>(R);
        case 1024: return modes_lds_bytes_r<16>(R);
        case 2048: return modes_lds_bytes_r<32>(R);
        default: return modes_lds_bytes_r<64>(R);
    }
}

hipError_t launch_correct(const DevPlan& p, JumpSrc js, double* corr, double* corr_il, double* dense,
                          const int* skip, hipStream_t s) {
    if (p.I == 0) return hipSuccess;
    if (hipError_t e_ = klaunch(&k_correct, dim3((p.I + 255) / 256), dim3(256), 0, s, p, js, corr, corr_il, dense, skip)) return e_;
    return hipGetLastError();
}

hipError_t launch_modes(const DevPlan& p, const double* corr, double* partial, int R, const int* skip,
                        hipStream_t s) {
    return modes_dispatch(p, R, ModesArgs{corr, partial, nullptr, skip, nullptr}, s);
}

hipError_t launch_modes_dense(const DevPlan& p, const double* corr, double* rows, bool load, bool store, int R,
                              double* partial, const double* w2, double* partial2, hipStream_t s) {
    const ModesDense dn{rows, load, store, partial != nullptr, w2};
    return modes_dispatch(p, R, ModesArgs{corr, partial, partial2, nullptr, &dn}, s);
}

hipError_t launch_spline(const DevPlan& p, const double* y, double* s2, const int* skip, hipStream_t s) {
    if (hipError_t e_ = klaunch(&k_spline, dim3((p.M + 255) / 256), dim3(256), 0, s, p, y, s2, skip)) return e_;
    return hipGetLastError();
}

hipError_t launch_density(const DevPlan& p, const double* y, double* s2, double* corr_il, const int* skip,
                          const DensityCheck* check, hipStream_t s) {
    const int gc = gm_chunks(p.M, true);
    const DensityCheck k = check ? *check : DensityCheck{};
    return klaunch(&k_density, dim3(gc + p.n_cc), dim3(kGmChunk), 0, s, p, y, s2, corr_il, gc, skip, k.flag, k.flag_next,
                   k.bad, k.number);
}

hipError_t launch_density_f(const DevPlan& p, const double* y, const double* f, double* s2, double* f2, double* corr_il,
                            hipStream_t s) {
    const int gc = gm_chunks(p.M, true);
    return klaunch(&k_density_f, dim3(gc + p.n_cc), dim3(kGmChunk), 0, s, p, y, f, s2, f2, corr_il, gc);
}

hipError_t launch_reduce_interp(const DevPlan& p, JumpSrc js, const double* partial, int G, double* out,
                                const int* skip, const GmresBufs* gm, hipStream_t s, const double* from) {
    if (gm) return klaunch(&k_reduce_gm, dim3(gm->gc64 + 1), dim3(1024), 0, s, p, js, partial, G, *gm);
    if (hipError_t e_ = klaunch(&k_reduce_interp, dim3((p.M + 63) / 64), dim3(1024), 0, s, p, js, partial, G, out, skip, from)) return e_;
    return hipGetLastError();
}

hipError_t launch_interp_grid(const DevPlan& p, JumpSrc js, const double* V, bool user, double* out, hipStream_t s) {
    if (hipError_t e_ = klaunch(&k_interp_grid, dim3((p.M + 255) / 256), dim3(256), 0, s, p, js, V, user ? 1 : 0, out)) return e_;
    return hipGetLastError();
}

hipError_t launch_fill_rhs(const DevPlan& p, const double* f, bool mask, double* R, hipStream_t s) {
    const size_t tot = (size_t)p.N * p.N;
    if (hipError_t e_ = klaunch(&k_fill_rhs, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, p, f, mask ? 1 : 0, R)) return e_;
    return hipGetLastError();
}

hipError_t launch_rows_solve(const DevPlan& p, double* A, hipStream_t s) { return rows_solve_any(p, A, s); }

hipError_t launch_rows_solve_f32(const DevPlan& p, float* A, hipStream_t s) { return rows_solve_any(p, A, s); }

hipError_t launch_grid_out(const DevPlan& p, const double* R, bool mask, double* u, hipStream_t s) {
    const size_t tot = (size_t)(p.N + 1) * (p.N + 1);
    if (hipError_t e_ = klaunch(&k_grid_out, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, p, R, mask ? 1 : 0, u)) return e_;
    return hipGetLastError();
}

hipError_t launch_axpby(int n, double a, const double* x, double b, const double* y, double* z, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    if (hipError_t e_ = klaunch(&k_axpby, dim3((n + 255) / 256), dim3(256), 0, s, n, a, x, b, y, z)) return e_;
    return hipGetLastError();
}

hipError_t launch_fill(size_t n, double v, double* x, hipStream_t s) {
    if (n == 0) return hipSuccess;
    if (hipError_t e_ = klaunch(&k_fill, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, v, x)) return e_;
    return hipGetLastError();
}

hipError_t launch_nonfinite(int n, const double* x, int* flag, hipStream_t s) {
    if (hipError_t e_ = klaunch(&k_nonfinite, dim3(1), dim3(256), 0, s, n, x, flag)) return e_;
    return hipGetLastError();
}

hipError_t launch_gmres_step_corr(const DevPlan& p, GmresBufs b, double* corr_il, hipStream_t s) {
    return klaunch(&k_gm_step_corr, dim3(b.gc + p.n_cc), dim3(kGmChunk), 0, s, p, b, corr_il);
}

hipError_t launch_gmres_start(const DevPlan* p, const double* taps, int M, GmresBufs b, const double* rhs,
                              const double* phi_in, double tol, int max_iter, double reorth, double* xout,
                              double* corr_il, unsigned epoch, hipStream_t s) {
    const bool corr = p && corr_il;
    const DevPlan pv = corr ? *p : DevPlan{};
    const int groups = b.gc + (corr ? p->n_cc : 0);
    return klaunch(&k_gm_begin, dim3(groups), dim3(kGmChunk), 0, s, pv, corr ? 1 : 0, taps, b, M, rhs, phi_in, tol,
                   max_iter, reorth, xout, corr ? corr_il : nullptr, epoch);
}

hipError_t launch_gmres_step(const double* taps, int M, GmresBufs b, hipStream_t s) {
    return klaunch(&k_gm_step, dim3(b.gc), dim3(kGmChunk), 0, s, taps, b, M);
}

}  // namespace kfbi
