// Device functions shared by the single-problem and the batched kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.h"

namespace kfbi {

// A flag or state word another launch wrote, read through the vector memory
// path: such loads are waited for only where the value is used, where a scalar
// load here is waited for at once, before the loads issued after it.
__device__ __forceinline__ int load_flag(const int* f) {
    // a global (not flat) load: a flat load also counts as a scalar-memory
    // access, so the next wait for the kernel's arguments would wait for it too
    using global_int = __attribute__((address_space(1))) int;
    return __hip_atomic_load((global_int*)f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// load_flag for a value used only late in the kernel: the address is offset by
// a zero the compiler cannot see through, so the value stays per lane and is
// not moved to a scalar register (which waits for it) right after the load.
__device__ __forceinline__ int load_flag_late(const int* f) {
    int zero;
    asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
    return load_flag(f + zero);
}
__device__ __forceinline__ double load_real_late(const double* f) {
    using global_real = __attribute__((address_space(1))) double;
    int zero;
    asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
    return __hip_atomic_load((global_real*)(f + zero), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A flag that is never set, read in place of a null one (a load from one of two
// addresses, with no branch that would wait for it).
static __device__ const int kFlagZero = 0;
__device__ __forceinline__ int load_flag_or_zero(const int* f) { return load_flag(f ? f : &kFlagZero); }


// sin(pi m / N), 0 <= m < 2N, from the quarter-period table sq[0..N/2].
__device__ __forceinline__ double sinpi_n(const double* __restrict__ sq, int m, int N) {
    const double sgn = (m & N) ? -1.0 : 1.0;
    m &= N - 1;
    m = min(m, N - m);
    return sgn * sq[m];
}

// Second derivative of the periodic spline through y at sample m: the inverse
// of the (1, 4, 1) circulant decays like (2 - sqrt 3)^|k|, so a filter of
// 2K+3 taps reproduces it to double precision.  Computed once per density by
// k_spline; the kernels below read the result.
__device__ inline double spline_s2(const double* __restrict__ y, int M, const double* __restrict__ taps, int m) {
    constexpr int K = kSplineK;
    double s = 0.0;
    if (M > K + 1 && m >= K + 1 && m + K + 1 < M) {
#pragma unroll
        for (int q = -K - 1; q <= K + 1; ++q) s = fma(taps[q + K + 1], y[m + q], s);
    } else {
#pragma unroll
        for (int q = -K - 1; q <= K + 1; ++q) {
            int idx = (m + q) % M;
            if (idx < 0) idx += M;
            s = fma(taps[q + K + 1], y[idx], s);
        }
    }
    return s;
}

// Value and first two parameter derivatives of the spline on segment seg at u.
__device__ __forceinline__ void spline_at(const double* __restrict__ y, const double* __restrict__ s2,
                                          const DevPlan& p, int seg, double u, double& v, double& d1, double& d2) {
    const int k1 = seg + 1 == p.M ? 0 : seg + 1;
    const double s0 = s2[seg], s1 = s2[k1];
    const double y0 = y[seg], y1 = y[k1], w = 1.0 - u;
    const double sixth = 1.0 / 6.0;
    v = w * y0 + u * y1 + (w * w * w - w) * s0 * sixth + (u * u * u - u) * s1 * sixth;
    d1 = (y1 - y0) - (3.0 * w * w - 1.0) * s0 * sixth + (3.0 * u * u - 1.0) * s1 * sixth;
    d2 = w * s0 + u * s1;
}

struct J6 {
    double v, gx, gy, hxx, hxy, hyy;
};

// Cartesian jumps of the interface problem at one point of Gamma.  With n the
// outward normal, c the curvature and the density D along arc length:
//   [v] = D, [d_n v] = 0 (Sec. 2.2):  [v_tau] = D_s, [v_tautau] = D_ss, [v_taun] = -c D_s;
//   [v] = 0, [d_n v] = D (Neumann):   [v_n] = D, [v_tautau] = c D, [v_taun] = D_s;
// and the equation gives [v_nn] = [F] + kappa [v] - [v_tautau].
// P, P1, P2: the density's spline value and parameter derivatives at the
// point; F: the jump of f there.
__device__ inline J6 jumps_from(const DevPlan& p, const PointGeom& g, double P, double P1, double P2, double F) {
    const double Ps = P1 * g.a1;
    J6 J;
    if (p.normal_jump) {
        const double vtt = g.curv * P, vtn = Ps, vnn = F - vtt;
        J.v = 0.0;
        J.gx = P * g.nx;
        J.gy = P * g.ny;
        J.hxx = vtt * g.tx * g.tx + 2.0 * vtn * g.tx * g.nx + vnn * g.nx * g.nx;
        J.hxy = vtt * g.tx * g.ty + vtn * (g.tx * g.ny + g.nx * g.ty) + vnn * g.nx * g.ny;
        J.hyy = vtt * g.ty * g.ty + 2.0 * vtn * g.ty * g.ny + vnn * g.ny * g.ny;
        return J;
    }
    const double Pss = P2 * g.a2 - P1 * g.a3;
    const double vtt = Pss, vtn = -g.curv * Ps, vnn = F + p.kappa * P - vtt;
    J.v = P;
    J.gx = Ps * g.tx;
    J.gy = Ps * g.ty;
    J.hxx = vtt * g.tx * g.tx + 2.0 * vtn * g.tx * g.nx + vnn * g.nx * g.nx;
    J.hxy = vtt * g.tx * g.ty + vtn * (g.tx * g.ny + g.nx * g.ty) + vnn * g.nx * g.ny;
    J.hyy = vtt * g.ty * g.ty + 2.0 * vtn * g.ty * g.ny + vnn * g.ny * g.ny;
    return J;
}

// The same at the point of segment g.seg, offset g.u, from the densities' splines.
__device__ inline J6 jumps_at(const DevPlan& p, const PointGeom& g, const JumpSrc& js) {
    double P = 0.0, P1 = 0.0, P2 = 0.0, F = 0.0, t1, t2;
    if (js.phi) spline_at(js.phi, js.phi_s2, p, g.seg, g.u, P, P1, P2);
    if (js.fgam) spline_at(js.fgam, js.fgam_s2, p, g.seg, g.u, F, t1, t2);
    return jumps_from(p, g, P, P1, P2, F);
}

// ---------------------------------------------------------------- tridiagonal mode solve (Alg. 4)
//
// Solve x[i-1] - beta x[i] + x[i+1] = e[i], i = 1..N-1, x[0] = x[N] = 0, with
// tridiag(1, -beta, 1) = -(1/r)(I - r S)(I - r S^T) - r e1 e1^T (S the down
// shift): the forward recurrence w[i] = r (w[i-1] - e[i]), the backward one
// y[i] = w[i] + r y[i+1], and x = y + y[1] zeta with
// zeta[i] = -r (r^i - r^(2N-i)) / (1 - r^(2N)) from the rank-one term.
// Lane L of the wavefront owns i = L C + 1 .. L C + C (i = N is a zero pad);
// each recurrence runs locally per lane and the lanes are joined by a scan of
// the carries with multiplier r^C.
// ---------------------------------------------------------------- wavefront scans with DPP
//
// A lane's FP64 value moved by a DPP control (row shifts stay inside rows of
// 16 lanes, wave shifts cross them); lanes without a source get 0.
constexpr int kDppRowShl1 = 0x101, kDppRowShr1 = 0x111, kDppWaveShl1 = 0x130, kDppWaveShr1 = 0x138;

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double readlane_f64(double v, int l) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
    return __hiloint2double(hi, lo);
}

// The sum over the wavefront, the same in every lane: the partner lane of each
// step differs in one more bit of the lane index (DPP quad swaps for bits 0
// and 1, the half-row and row mirrors, lane ^ 7 and lane ^ 15, for bits 2 and
// 3), so every lane holds its row's sum after four steps; the four row sums
// are then read as scalars.  Each step adds the same two values in either
// partner, so all lanes agree to the bit.
constexpr int kDppQuadSwap1 = 0xB1, kDppQuadSwap2 = 0x4E, kDppRowMirror = 0x140, kDppRowHalfMirror = 0x141;
__device__ __forceinline__ double wave_allsum(double v) {
    v += dpp_f64<kDppQuadSwap1>(v);
    v += dpp_f64<kDppQuadSwap2>(v);
    v += dpp_f64<kDppRowHalfMirror>(v);
    v += dpp_f64<kDppRowMirror>(v);
    return (readlane_f64(v, 0) + readlane_f64(v, 16)) + (readlane_f64(v, 32) + readlane_f64(v, 48));
}

// base^k for 0 <= k < 2^BITS by repeated squaring (BITS fixed steps)
template <int BITS>
__device__ __forceinline__ double pow_u(double base, int k) {
    double res = 1.0;
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        if ((k >> b) & 1) res *= base;
        base *= base;
    }
    return res;
}
__device__ __forceinline__ double pow_u8(double base, int k) { return pow_u<8>(base, k); }

// Weighted inclusive scans over the wavefront, v_L <- sum_k m^|L-k| v_k over
// k <= L (up) or k >= L (down): inside each row of 16 lanes by four DPP row
// shifts, then across the rows from the row ends read as scalars.
// pl: m^((lane & 15) + 1) (up), m^(16 - (lane & 15)) (down).
__device__ __forceinline__ double wave_scan_up(double v, double m, double pl, int lane) {
    const double m2 = m * m, m4 = m2 * m2, m8 = m4 * m4, m16 = m8 * m8;
    v = fma(m, dpp_f64<kDppRowShr1>(v), v);
    v = fma(m2, dpp_f64<kDppRowShr1 + 1>(v), v);
    v = fma(m4, dpp_f64<kDppRowShr1 + 3>(v), v);
    v = fma(m8, dpp_f64<kDppRowShr1 + 7>(v), v);
    const double p0 = readlane_f64(v, 15);
    const double p1 = fma(m16, p0, readlane_f64(v, 31));
    const double p2 = fma(m16, p1, readlane_f64(v, 47));
    const int row = lane >> 4;
    const double before = row == 0 ? 0.0 : row == 1 ? p0 : row == 2 ? p1 : p2;
    return fma(pl, before, v);
}

__device__ __forceinline__ double wave_scan_down(double v, double m, double pl, int lane) {
    const double m2 = m * m, m4 = m2 * m2, m8 = m4 * m4, m16 = m8 * m8;
    v = fma(m, dpp_f64<kDppRowShl1>(v), v);
    v = fma(m2, dpp_f64<kDppRowShl1 + 1>(v), v);
    v = fma(m4, dpp_f64<kDppRowShl1 + 3>(v), v);
    v = fma(m8, dpp_f64<kDppRowShl1 + 7>(v), v);
    const double q3 = readlane_f64(v, 48);
    const double q2 = fma(m16, q3, readlane_f64(v, 32));
    const double q1 = fma(m16, q2, readlane_f64(v, 16));
    const int row = lane >> 4;
    const double after = row == 3 ? 0.0 : row == 2 ? q3 : row == 1 ? q2 : q1;
    return fma(pl, after, v);
}

template <int C>
__device__ __forceinline__ void mode_solve(double (&e)[C], const ModeConst& mc, int lane, int N) {
    const double r = mc.r, rinv = mc.rinv;
    // forward recurrence w = r (w - e): one dependent fma per step
    double w = 0.0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const double re = r * e[c];
        w = fma(r, w, -re);
        e[c] = w;
    }
    // the lanes' carries: the weighted prefix of the chunk ends, from lane L-1
    double carry = dpp_f64<kDppWaveShr1>(wave_scan_up(w, mc.rC, pow_u8(mc.rC, (lane & 15) + 1), lane));
    // e[c] += r^(c+1) carry; the powers in four interleaved chains
    const double r2 = r * r, r4 = r2 * r2;
    double pw[4] = {r, r2, r2 * r, r4};
#pragma unroll
    for (int c = 0; c < C; ++c) {
        e[c] = fma(pw[c & 3], carry, e[c]);
        pw[c & 3] *= r4;
    }
    if (lane == 63) e[C - 1] = 0.0;
    double y = 0.0;
#pragma unroll
    for (int c = C - 1; c >= 0; --c) {
        y = fma(r, y, e[c]);
        e[c] = y;
    }
    carry = dpp_f64<kDppWaveShl1>(wave_scan_down(y, mc.rC, pow_u8(mc.rC, 16 - (lane & 15)), lane));
    // e[c] += r^(C-c) carry
    pw[0] = r;
    pw[1] = r2;
    pw[2] = r2 * r;
    pw[3] = r4;
#pragma unroll
    for (int c = C - 1; c >= 0; --c) {
        const int k = (C - 1 - c) & 3;
        e[c] = fma(pw[k], carry, e[c]);
        pw[k] *= r4;
    }
    // rank-one fix: e[c] += y1 smc (r^i - r^(2N-i)) at i = lane C + 1 + c, with
    // r^(lane C + 1) = r (r^C)^lane and r^(2N - lane C - 1) = (r^C)^(128 - lane) / r
    // (2N = 128 C); the powers along c again in four chains
    const double y1 = readlane_f64(e[0], 0);
    const double coef = y1 * mc.smc;
    const double p1 = r * pow_u8(mc.rC, lane);
    const double p2 = rinv * pow_u8(mc.rC, 128 - lane);
    const double ri2 = rinv * rinv, ri4 = ri2 * ri2;
    double pa[4] = {p1, p1 * r, p1 * r2, p1 * r2 * r};
    double pb[4] = {p2, p2 * rinv, p2 * ri2, p2 * ri2 * rinv};
#pragma unroll
    for (int c = 0; c < C; ++c) {
        e[c] = fma(coef, pa[c & 3] - pb[c & 3], e[c]);
        pa[c & 3] *= r4;
        pb[c & 3] *= ri4;
    }
    if (lane == 63) e[C - 1] = 0.0;
}

// Jump terms of the stencil nodes outside Omega: the far-side value is moved to
// the Omega side with the Taylor expansion of the jumps at the sample.  Every
// load is issued before any is used: sample cp is the knot that starts spline
// segment cp (u = 0, as the plan builds it), so the density's values there do
// not wait for the sample's geometry.
__device__ inline double outside_terms(const DevPlan& p, const JumpSrc& js, int cp, const int (&ni)[6], const int (&nj)[6],
                                const double* __restrict__ w, int ldw) {
    const unsigned char* o6 = p.cp_out + 6 * (size_t)cp;
    unsigned char o[6];
    double wk[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        o[k] = o6[k];
        wk[k] = w[(size_t)k * ldw];
    }
    const PointGeom g = p.z_geo[cp];
    const double zx = p.zx[cp], zy = p.zy[cp];
    J6 J;
    if (js.jz) {
        const double* q = js.jz + 6 * (size_t)cp;
        J = {q[0], q[1], q[2], q[3], q[4], q[5]};
    } else {
        double P = 0.0, P1 = 0.0, P2 = 0.0, F = 0.0, t1, t2;
        if (js.phi) spline_at(js.phi, js.phi_s2, p, cp, 0.0, P, P1, P2);
        if (js.fgam) spline_at(js.fgam, js.fgam_s2, p, cp, 0.0, F, t1, t2);
        J = jumps_from(p, g, P, P1, P2, F);
    }
    if (!(o[0] | o[1] | o[2] | o[3] | o[4] | o[5])) return 0.0;
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        if (!o[k]) continue;
        const double dx = p.lo + ni[k] * p.h - zx, dy = p.lo + nj[k] * p.h - zy;
        s += wk[k] * (J.v + dx * J.gx + dy * J.gy + 0.5 * (dx * dx * J.hxx + 2.0 * dx * dy * J.hxy + dy * dy * J.hyy));
    }
    return s;
}

__device__ __forceinline__ void stencil_nodes(const DevPlan& p, int cp, int (&ni)[6], int (&nj)[6]) {
    const int i0 = p.cp_i0[cp], j0 = p.cp_j0[cp], sxy = p.cp_sxy[cp];
    const int sx = (sxy & 1) ? 1 : -1, sy = (sxy & 2) ? 1 : -1;
    ni[0] = i0; nj[0] = j0;
    ni[1] = i0 + 1; nj[1] = j0;
    ni[2] = i0 - 1; nj[2] = j0;
    ni[3] = i0; nj[3] = j0 + 1;
    ni[4] = i0; nj[4] = j0 - 1;
    ni[5] = i0 + sx; nj[5] = j0 + sy;
}

__device__ inline double block_sum(double v, double* red) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    v = wave_allsum(v);
    __syncthreads();
    if (lane == 0) red[wave] = v;
    __syncthreads();
    double s = 0.0;
    for (int k = 0; k < nw; ++k) s += red[k];
    return s;
}

// ---------------------------------------------------------------- correction (Alg. 2)

// Correction of the right-hand side at irregular node r: for each arm to a
// neighbour across Gamma, the jump continued from the crossing along the arm by
// its second-order Taylor expansion, times -s_r / h^2.
__device__ inline double correction_at(const DevPlan& p, const JumpSrc& js, int r) {
    const double s = p.irr_s[r];
    double acc = 0.0;
    for (int a = 0; a < 4; ++a) {
        const int k = p.arm_q[4 * r + a];
        if (k < 0) break;
        const double d = p.arm_d[4 * r + a];
        const int ax = p.q_axis[k];
        double v, g, hh;
        if (js.jq) {
            const double* J = js.jq + 6 * (size_t)k;
            v = J[0];
            g = ax ? J[2] : J[1];
            hh = ax ? J[5] : J[3];
        } else {
            const J6 J = jumps_at(p, p.q_geo[k], js);
            v = J.v;
            g = ax ? J.gy : J.gx;
            hh = ax ? J.hyy : J.hxx;
        }
        acc -= s * (v + d * g + 0.5 * d * d * hh);
    }
    return acc * p.inv_h2;
}

// Samples cp0 .. cp0 + 63 (one per lane) by a workgroup of 16 wavefronts: the
// workgroup partials of the weighted sine sums (row g of `partial` holds
// workgroup g's sums for all M samples) are split over wavefronts 0..14, added
// in a fixed order; wavefront 15 makes the jump terms of the stencil nodes
// outside Omega, and wavefront 0 adds them and writes out[cp] (unless out is null;
// also to red[lane], for the caller); with `from`, out[cp] = from[cp] - that.
// red: 16 x 64 doubles of LDS.  Returns false, having written nothing, while
// *skip is nonzero (skip may be null); the flag's latency overlaps the loads.
__device__ inline bool reduce_samples64(const DevPlan& p, const JumpSrc& js, const double* __restrict__ partial,
                                        int G, int cp0, double* __restrict__ out, double* red,
                                        const int* __restrict__ skip = nullptr,
                                        const double* __restrict__ from = nullptr) {
    __shared__ double outside[64];
    constexpr int kOutsideWave = 15;                    // makes the jump terms only
    constexpr int kRowWaves = 15, kRows = 18;           // rows wave + 15 k, k < 18, requested at once
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int cp = cp0 + lane, M = p.M;
    const int skipped = load_flag_or_zero(skip);
    double s = 0.0;
    if (cp < M) {
        if (wave == kOutsideWave) {
            int ni[6], nj[6];
            stencil_nodes(p, cp, ni, nj);
            outside[lane] = outside_terms(p, js, cp, ni, nj, p.cp_w + cp, M);
        } else {
            // every row is loaded from a row that exists (then selected), so no
            // load waits under its own condition before the next is requested
            double r[kRows];
#pragma unroll
            for (int k = 0; k < kRows; ++k) {
                const int g = wave + kRowWaves * k;
                const double v = partial[(size_t)(g < G ? g : G - 1) * M + cp];
                r[k] = g < G ? v : 0.0;
            }
#pragma unroll
            for (int k = 0; k < kRows; ++k) s += r[k];
            for (int g = wave + kRowWaves * kRows; g < G; g += kRowWaves) s += partial[(size_t)g * M + cp];
        }
    }
    if (skipped) return false;                          // the same for the whole workgroup
    red[wave * 64 + lane] = s;
    __syncthreads();
    if (wave == 0 && cp < M) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < 16; ++w) t += red[w * 64 + lane];
        const double v = t * (2.0 / p.N) + outside[lane];
        if (out) out[cp] = from ? from[cp] - v : v;
        red[lane] = v;                                  // left in LDS for the caller
    }
    __syncthreads();
    return true;
}

// ---------------------------------------------------------------- sparse fast solve, R modes per workgroup
//
// LDS of the sparse fast solve: the block's row sines (two per row up to N/2) and
// the rows' 2 cos(pi j / N); at N = 4096, where they would not fit beside the
// solutions, the quarter-period table sin(pi m / N), m <= N/2, they are looked up
// in, and the carries between a mode's wavefronts.  Then the
// padded mode solutions (node i at i + (i - 1) / CH with CH nodes a lane, so the
// lanes' chunk-strided accesses fall in different banks).
struct ModesLds {
    double* sq;   // modes_table_len
    double* xs;   // modes_pairs<R> x modes_pair_len<C>
};

template <int C>
constexpr bool kRowSines = C <= 32;
template <int C>
constexpr int modes_table_len() { return kRowSines<C> ? 96 * C + 4 : 32 * C + 2 + 3 * kModeWaves; }
// the rows' cosines in the table, after the 32 C + 1 pairs of sines
template <int C>
constexpr int modes_cos_at() { return 64 * C + 2; }
// doubles of one padded solution: CH = modes_chunk(N) nodes a lane
template <int C>
constexpr int modes_stride() { return modes_stride_of(64 * C); }
// a pair of mirrored modes: the sums over even rows, those over odd rows (then the
// two solutions) and the sums of the extra pieces of long column halves
template <int C>
constexpr int modes_pair_len() { return 2 * modes_stride<C>() + kMaxExtra; }
template <int R>
constexpr int modes_pairs() { return R >= 2 ? R / 2 : 1; }
template <int C, int R>
constexpr size_t modes_lds_len() {
    return (size_t)modes_table_len<C>() + (size_t)modes_pairs<R>() * modes_pair_len<C>();
}

template <int C>
__device__ __forceinline__ ModesLds modes_lds(double* smem) {
    ModesLds L;
    L.sq = smem;
    L.xs = smem + modes_table_len<C>();
    return L;
}

// v with its sign flipped where bit 31 of `sign` is set
__device__ __forceinline__ double flip_sign(double v, unsigned sign) {
    return __hiloint2double(__double2hiint(v) ^ (int)sign, __double2loint(v));
}

// (sin(l0 t), sin((l0 + 1) t)), t = pi j / N, 0 <= j <= N/2, N = 64 C, at16 = 16
// modes_row_place(j): from the block's row sines in LDS, at N = 4096 by two lookups in the
// quarter-period table.
template <int C>
__device__ __forceinline__ double2 row_sines(const double* sq, int at16, int l0) {
    constexpr int N = 64 * C;
    if constexpr (kRowSines<C>) return *reinterpret_cast<const double2*>(reinterpret_cast<const char*>(sq) + at16);
    const int j = at16 >> 4;
    const int m0 = (int)(__umul24((unsigned)j, (unsigned)l0) & (2 * N - 1));
    return make_double2(sinpi_n(sq, m0, N), sinpi_n(sq, (m0 + j) & (2 * N - 1), N));
}

// 2 cos(pi j / N) of the row at the same place.
template <int C>
__device__ __forceinline__ double row_c2(const double* sq, int at16) {
    if constexpr (kRowSines<C>)
        return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(sq + modes_cos_at<C>()) + (at16 >> 1));
    return 2.0 * sq[32 * C - (at16 >> 4)];
}

// The block's row sines into LDS (every node's and every sample's sines are then
// one 16-byte read at its row, nearly free of bank conflicts because the lanes'
// rows follow the curve; a table indexed by j l mod 2N, which scatters them, took
// three reads of three passes each and bounded the sums), or at N = 4096 the
// quarter-period table.
template <int C>
__device__ __forceinline__ void modes_load_table(double* sq, const double* __restrict__ sinq, int l0, int tid) {
    constexpr int N = 64 * C;
    if constexpr (kRowSines<C>) {
        if (tid == 0) {
            reinterpret_cast<double2*>(sq)[0] = make_double2(0.0, 0.0);
            sq[modes_cos_at<C>()] = 2.0;
        }
        for (int j = 1 + tid; j <= N / 2; j += kModeWaves * 64) {
            const int m0 = (int)(__umul24((unsigned)j, (unsigned)l0) & (2 * N - 1));
            sq[modes_cos_at<C>() + modes_row_place(j, N)] = 2.0 * sinq[N / 2 - j];
            reinterpret_cast<double2*>(sq)[modes_row_place(j, N)] =
                make_double2(sinpi(m0 * (1.0 / N)), sinpi(((m0 + j) & (2 * N - 1)) * (1.0 / N)));
        }
    } else {
        for (int k = tid; k <= N / 2; k += kModeWaves * 64) sq[k] = sinq[k];
    }
}

// The sine modes of block g by a workgroup of kModeWaves wavefronts: the H = R/2
// mirrored pairs (l, N - l) for l = g H + 1 .. g H + H (N/2 is its own mirror),
// or with R = 1 the one mode l = g + 1.
//  1. Sparse sine sums of the corrected right-hand side along y: wavefront w
//     walks sub-table w of the interleaved node table: steps of 64 column halves
//     (the nodes of one column and one parity of j) of about equal length, one a
//     lane, so all lanes end and store their H sums together.  Per node the sines
//     of the H modes l are two values of its row (modes_load_table) and the
//     recurrence sin((l+1)t) = 2 cos t sin(lt) - sin((l-1)t).  With E and O the sums over even
//     and odd j, mode l has E + O and mode N - l, whose sine at row j is
//     (-1)^(j+1) that of mode l, has O - E: a pair costs the sines and the
//     multiply-adds of one mode.
//  2. The tridiagonal solve along x of each mode (mode_solve's steps) by S = C / CH
//     wavefronts: a lane holds CH <= 32 nodes in registers, and the S wavefronts'
//     carries are joined through LDS (a row of 4096 nodes would not fit one
//     wavefront's registers beside sixteen wavefronts' worth of the rest).
//  3. The weighted six-point gather at every sample: the row sines by the same
//     recurrence, again one set per pair (the rows j0 and j0 +- 1 have opposite
//     signs in the mirrored mode).  emit(0, cp, s) gets the sum s over the block's
//     modes, for cp = tid, tid + 64 kModeWaves, ...
// What bounds it: a compute unit's intake of the node and sample tables from L2
// (64 bytes a clock, 12 bytes a node) until the sums are done, then LDS and issue;
// the R padded solutions fill the LDS, so it holds one workgroup, and sixteen
// wavefronts hide more latency than eight.  At 2048^2 with 7656 nodes (256
// workgroups) one launch went from 16.7 us (eight wavefronts, every mode summed
// by itself with three lookups a node, powers recomputed in the solve) to 12.3 us,
// at 1024^2 from 10.6 to 7.6 us.
// Must be called by the whole workgroup; N = 64 C.  The round does nothing while *skip is nonzero (skip may be null);
// the flag is checked after the first requests and the clear, so its latency
// overlaps theirs.
// EARLY: the wavefront's mode constants and the thread's first stencil are
// requested ahead of their phases (off where the registers are short: the
// batched kernel holds every grid size's code).
// dense (DENSE): the rows of the modes' transformed right-hand side on the whole
// grid, added to the sums (null: none); with `store` the solutions are written back
// there; emit(1, cp, s) gets the sums with the weights w2 (null: not wanted), and
// with gather = false phase 3 is left out.
struct ModesDense {
    double* rows;
    bool load, store, gather;
    const double* w2;
};
template <int C, int R, bool EARLY, bool DENSE, class Emit>
__device__ __forceinline__ void modes_round(const DevPlan& p, const double* __restrict__ corr, int g,
                                            const ModesLds& L, Emit emit, const int* __restrict__ skip = nullptr,
                                            const ModesDense& dn = ModesDense{}) {
    constexpr int N = 64 * C, XS = modes_stride<C>(), PS = modes_pair_len<C>();
    constexpr int CH = modes_chunk(N), S = C / CH;
    static_assert(R * S <= kModeWaves, "S wavefronts for each mode");
    static_assert(S == 1 || !kRowSines<C>, "the carries' place");
    double* carry_up = L.sq + 32 * C + 2;               // S > 1: one value a wavefront each, after the table
    double* carry_dn = carry_up + kModeWaves;
    double* carry_g = carry_dn + kModeWaves;
    constexpr int NT = kModeWaves * 64;
    constexpr int H = modes_pairs<R>();
    const int M = p.M;
    int tid = threadIdx.x;
    // in the batched kernel's item loop the thread's addresses for every grid size
    // would otherwise be kept in registers across the loop
    if (!EARLY) asm volatile("" : "+v"(tid));
    // the wavefront's index as a scalar: its branches are then uniform
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const double* sq = L.sq;
    const int l0 = g * H + 1;
    const int skipped = load_flag_or_zero(skip);
    // the first rows of this wavefront's node table are requested before
    // anything waits, so their latency overlaps the table load and the clear;
    // the sub-table's bounds come with the plan's fields, not from memory
    int t_beg, t_end;                                  // multiples of kSlots
    if constexpr (EARLY) {
        t_beg = p.sub_offv[0];
        t_end = p.sub_offv[1];
#pragma unroll
        for (int w = 1; w < kModeWaves; ++w)           // constant indices: loaded with the other fields
            if (wave == w) {
                t_beg = p.sub_offv[w];
                t_end = p.sub_offv[w + 1];
            }
    } else {                                           // the plan is in memory: no gain, and seventeen registers
        t_beg = p.sub_off[wave];
        t_end = p.sub_off[wave + 1];
    }
    struct Rows {                                       // kSlots rows of the node table
        int pk[kSlots];
        double cv[kSlots];
    };
    auto load_rows = [&](Rows& n, int t0) {
#pragma unroll
        for (int q = 0; q < kSlots; ++q) {
            n.pk[q] = p.il_ij[(unsigned)(t0 + q) * 64u + (unsigned)lane];
            n.cv[q] = corr[(unsigned)(t0 + q) * 64u + (unsigned)lane];
        }
    };
    Rows ra, rb;
    if (t_beg < t_end) load_rows(ra, t_beg);
    if (EARLY && t_beg + kSlots < t_end) load_rows(rb, t_beg + kSlots);
    // also requested now: this wavefront's mode constants (phase 2)
    const int mode = wave / S, sub = wave % S;          // mode of the block (pairs' l first, then their mirrors)
    const bool mirror = R >= 2 && mode >= H, solves = mode < R;
    const int lw = mirror ? N - (l0 + mode - H) : l0 + mode;
    ModeConst mcw{};
    if (EARLY && solves) mcw = p.modes[lw];
    // ... and the thread's entry of the split list (the end of phase 1)
    int sp_at = 0, sp_e0 = 0, sp_ne = 0;
    if (tid < p.n_split * H) {
        const int* e = p.split + 3 * (tid / H);
        sp_at = e[0];
        sp_e0 = e[1];
        sp_ne = e[2];
    }
    modes_load_table<C>(L.sq, p.sinq, l0, tid);
    double2* xs2 = reinterpret_cast<double2*>(L.xs);
    for (int k = tid; k < H * PS / 2; k += NT) xs2[k] = make_double2(0.0, 0.0);
    if (skipped) return;                                // the same for the whole workgroup
    __syncthreads();
    {
        double acc[H];
#pragma unroll
        for (int r = 0; r < H; ++r) acc[r] = 0.0;
        // a row beyond N/2 is looked up at its mirror N - j: sin(l t) changes sign there for even l
        const unsigned flip0 = (l0 & 1) ? 0u : 0x80000000u, flip1 = flip0 ^ 0x80000000u;
        auto sum_rows = [&](const Rows& n) {
            // the group's row sines are read before any of its sums is stored, so
            // their latencies overlap
            double2 s01[kSlots];
            double c2[kSlots];
#pragma unroll
            for (int q = 0; q < kSlots; ++q) {
                s01[q] = row_sines<C>(sq, n.pk[q] & kIlRow, l0);
                c2[q] = H > 2 ? row_c2<C>(sq, n.pk[q] & kIlRow) : 0.0;
            }
#pragma unroll
            for (int q = 0; q < kSlots; ++q) {
                double sp = flip_sign(s01[q].x, (unsigned)n.pk[q] & flip0), sc = flip_sign(s01[q].y, (unsigned)n.pk[q] & flip1);
                const double c = flip_sign(c2[q], (unsigned)n.pk[q] & 0x80000000u);
                acc[0] = fma(n.cv[q], sp, acc[0]);
                if (H > 1) acc[1] = fma(n.cv[q], sc, acc[1]);
#pragma unroll
                for (int r = 2; r < H; ++r) {
                    const double sn = fma(c, sc, -sp);
                    acc[r] = fma(n.cv[q], sn, acc[r]);
                    sp = sc;
                    sc = sn;
                }
                if (__builtin_amdgcn_readfirstlane(n.pk[q]) & kIlLast) {   // the step's last row, for every lane
                    double* to = L.xs + (((unsigned)n.pk[q] >> 16) & 0x7fff);
#pragma unroll
                    for (int r = 0; r < H; ++r) to[r * PS] = acc[r];
#pragma unroll
                    for (int r = 0; r < H; ++r) acc[r] = 0.0;
                }
            }
        };
        // two groups in turn: each one's next rows are requested when its sums are done
        for (int t0 = t_beg; t0 < t_end; t0 += 2 * kSlots) {
            if (!EARLY && t0 + kSlots < t_end) load_rows(rb, t0 + kSlots);
            sum_rows(ra);
            if (t0 + kSlots >= t_end) break;
            if (t0 + 2 * kSlots < t_end) load_rows(ra, t0 + 2 * kSlots);
            sum_rows(rb);
            if (EARLY && t0 + 3 * kSlots < t_end) load_rows(rb, t0 + 3 * kSlots);
        }
    }
    // the stencil data of the thread's first sample (phase 3), requested once the
    // nodes' loads are through: a compute unit takes in 64 bytes a clock, and at
    // the start these would hold up the nodes
    int pre_pk = 0;
    double pre_w[6] = {};
    if (EARLY && !DENSE && tid < M) {
        pre_pk = p.cp_pack[tid];
        for (int k = 0; k < 6; ++k) pre_w[k] = p.cp_w[(size_t)k * M + tid];
    }
    __syncthreads();
    // long column halves: add their extra pieces in a fixed order (at most
    // kMaxExtra of them, and H <= 4: one a thread)
    static_assert(kMaxExtra * H <= NT, "a thread for each split column half and pair");
    if (tid < p.n_split * H) {
        double* x = L.xs + (tid % H) * PS;
        double v = x[sp_at];
        for (int e = 0; e < sp_ne; ++e) v += x[2 * XS + sp_e0 + e];
        x[sp_at] = v;
    }
    __syncthreads();
    // row l of the dense arrays: element (l - 1) N + i - 1, node i at i + (i - 1) / CH here
    auto place = [](int i) { return i + (i - 1) / CH; };
    auto row_of = [&](int l) { return dn.rows + (size_t)(l - 1) * N; };
    if constexpr (DENSE) {
        // the sums become the two modes' right-hand sides in place, with the dense rows
#pragma unroll
        for (int r = 0; r < H; ++r) {
            const int l = l0 + r;
            const bool self = R < 2 || l == N / 2;
            const double* da = row_of(l);
            const double* db = row_of(self ? l : N - l);
            double* xe = L.xs + r * PS;
            for (int i = 1 + tid; i < N; i += NT) {
                const double ga = dn.load ? da[i - 1] : 0.0, gb = dn.load ? db[i - 1] : 0.0;
                const int at = place(i);
                const double e = xe[at], o = xe[XS + at];
                xe[at] = e + o + ga;
                xe[XS + at] = self ? 0.0 : o - e + gb;
            }
        }
        __syncthreads();
    }
    {
        // the mode's right-hand side from the pair's sums over even and odd rows
        // (N/2 is its own mirror: solved once, its mirror is zero)
        const int gl = sub * 64 + lane, at = gl * (CH + 1) + 1;   // lane of the mode, place of its first node
        double e[CH];
        if (!EARLY && solves) mcw = p.modes[lw];
        if (solves) {
            const double* xe = L.xs + (mirror ? mode - H : mode) * PS + at;
            const double* xo = xe + XS;
            if constexpr (DENSE) {
                const double* x = mirror ? xo : xe;
#pragma unroll
                for (int c = 0; c < CH; ++c) e[c] = p.h2 * x[c];
            } else {
                const double so = mirror && lw == N / 2 ? 0.0 : p.h2, se = mirror ? -so : so;
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    e[c] = fma(so, xo[c], se * xe[c]);
                    if (CH > 16 && c % 8 == 7) __builtin_amdgcn_sched_barrier(0);   // not all 2 CH reads in registers at once
                }
            }
        }
        if (!DENSE) __syncthreads();                    // both of a pair have read its sums
        // The steps of mode_solve, with the rank-one fix taken into the forward
        // recurrence: y[1] zeta is what an initial value
        //   w[0] = r / (1 - r^(2N)) sum_k e[k] (r^k - r^(2N-k))
        // adds (the forward recurrence turns w[0] into r^i w[0], the backward one
        // that into w[0] (r^i - r^(2N-i)) / (1 - r^2)), and both sums come with
        // the carries: the first by a Horner sum per lane, the second is
        // -r^(N-1) w[N].  Each recurrence then runs twice per lane, once for the
        // carry it passes on and once from the carry it gets: six operations a
        // node where adding the carries' powers and the fix took eleven.
        const double r = mcw.r, rH = mcw.rH;
        const double rl = pow_u<4>(rH, lane & 15), r16 = pow_u<5>(rH, 16);
        const double rlane = rl * pow_u<2>(r16, lane >> 4);      // rH^lane
        const double r64 = (r16 * r16) * (r16 * r16);            // from one wavefront of a mode to the next
        double w = 0.0, g1 = 0.0, up = 0.0;
        if (solves) {
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                e[c] *= r;
                w = fma(r, w, -e[c]);
            }
#pragma unroll
            for (int c = CH - 1; c >= 0; --c) g1 = fma(r, g1, e[c]);
            up = wave_scan_up(w, rH, rl * rH, lane);
            g1 = wave_allsum(g1 * rlane);
            if (S > 1 && lane == 63) {
                carry_up[wave] = up;
                carry_g[wave] = g1;
            }
        }
        double in = 0.0, wN = readlane_f64(up, 63);
        if constexpr (S > 1) {
            __syncthreads();
            if (solves) {
                wN = g1 = 0.0;
#pragma unroll
                for (int q = S - 1; q >= 0; --q) g1 = fma(r64, g1, carry_g[wave - sub + q]);
#pragma unroll
                for (int q = 0; q < S; ++q) {
                    if (q == sub) in = wN;
                    wN = fma(r64, wN, carry_up[wave - sub + q]);
                }
            }
        }
        double y = 0.0, dn = 0.0;
        if (solves) {
            const double w0 = -mcw.smc * fma(mcw.rN1, wN, g1);
            // the value at the node before the lane's first: the lanes below and w[0]
            double rg = 1.0;
#pragma unroll
            for (int q = 1; q < S; ++q) rg *= sub >= q ? r64 : 1.0;
            w = dpp_f64<kDppWaveShr1>(up) + rlane * fma(rg, w0, in);
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                w = fma(r, w, -e[c]);
                e[c] = w;
            }
            if (gl == 64 * S - 1) e[CH - 1] = 0.0;      // node N
#pragma unroll
            for (int c = CH - 1; c >= 0; --c) y = fma(r, y, e[c]);
            dn = wave_scan_down(y, rH, pow_u<4>(rH, 15 - (lane & 15)) * rH, lane);
            if (S > 1 && lane == 0) carry_dn[wave] = dn;
        }
        in = 0.0;
        if constexpr (S > 1) {
            __syncthreads();
            if (solves) {
#pragma unroll
                for (int q = S - 1; q > 0; --q)
                    if (q > sub) in = fma(r64, in, carry_dn[wave - sub + q]);
                in *= pow_u<6>(rH, 63 - lane);
            }
        }
        if (solves) {
            y = dpp_f64<kDppWaveShl1>(dn) + in;
            double* x = L.xs + (mirror ? (mode - H) * PS + XS : mode * PS) + at;
#pragma unroll
            for (int c = CH - 1; c >= 0; --c) {
                y = fma(r, y, e[c]);
                if (c < CH - 1 || gl < 64 * S - 1) x[c] = y;
            }
        }
    }
    __syncthreads();
    if constexpr (DENSE) {
        if (dn.store) {
#pragma unroll
            for (int r = 0; r < H; ++r) {
                const int l = l0 + r;
                const bool self = R < 2 || l == N / 2;
                double* da = row_of(l);
                double* db = row_of(N - l);
                const double* xe = L.xs + r * PS;
                for (int i = 1 + tid; i <= N; i += NT) {   // i = N: the pad
                    const int at = place(i);
                    da[i - 1] = i < N ? xe[at] : 0.0;
                    if (!self) db[i - 1] = i < N ? xe[XS + at] : 0.0;
                }
            }
        }
        if (!dn.gather) return;
    }
    auto gather = [&](int set, int cp, int pk1, const double (&w6)[6]) {
        const int i0 = pk1 & 0x1fff, j0 = (pk1 >> 13) & 0x1fff;
        const bool sxp = (pk1 & (1 << 26)) != 0, syp = (pk1 & (1 << 27)) != 0;
        const double w0 = w6[0], wE = w6[1], wW = w6[2], wN = w6[3], wS = w6[4];
        const double wDp = syp ? w6[5] : 0.0, wDm = syp ? 0.0 : w6[5];   // the diagonal node's row
        // places of the stencil columns in the padded layout (node 0 lies on
        // the box: zero); the sine arguments advance by j per mode
        const int pc = i0 + (i0 - 1) / CH, pe = i0 + i0 / CH + 1, pw = i0 > 1 ? i0 - 1 + (i0 - 2) / CH : -1;
        const double odd = (j0 & 1) ? 1.0 : -1.0;           // sign of the mirrored mode's sine at row j0
        // sines of the rows j0, j0 + 1, j0 - 1 for the modes l0 + q: two values
        // each, then the three-term recurrence in q
        const unsigned flip0 = (l0 & 1) ? 0u : 0x80000000u, flip1 = flip0 ^ 0x80000000u;
        struct Row {
            double s0, s1, c2;
        };
        auto at_row = [&](int j) {
            const bool mir = j > N / 2;
            const int at16 = 16 * modes_row_place(mir ? N - j : j, N);
            const double2 v = row_sines<C>(sq, at16, l0);
            return Row{flip_sign(v.x, mir ? flip0 : 0u), flip_sign(v.y, mir ? flip1 : 0u),
                       H > 2 ? flip_sign(row_c2<C>(sq, at16), mir ? 0x80000000u : 0u) : 0.0};
        };
        const Row r0 = at_row(j0), rp = at_row(j0 + 1), rm = at_row(j0 - 1);
        double s0p = r0.s0, spp = rp.s0, smp = rm.s0, s0c = r0.s1, spc = rp.s1, smc = rm.s1;
        const double c0 = r0.c2, cpl = rp.c2, cmi = rm.c2;
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < H; ++q) {
            const double* xq = L.xs + q * PS;
            double s0, sp, sm;
            if (q == 0) {
                s0 = s0p;
                sp = spp;
                sm = smp;
            } else if (q == 1) {
                s0 = s0c;
                sp = spc;
                sm = smc;
            } else {
                s0 = fma(c0, s0c, -s0p);
                sp = fma(cpl, spc, -spp);
                sm = fma(cmi, smc, -smp);
                s0p = s0c;
                spp = spc;
                smp = smc;
                s0c = s0;
                spc = sp;
                smc = sm;
            }
            // the pair's values with the mirrored mode's signs: sums at row j0,
            // differences at the rows next to it
            double xc = xq[pc], xe = xq[pe], xw = pw >= 0 ? xq[pw] : 0.0;
            double xcd = xc, xdd = sxp ? xe : xw;
            if constexpr (R >= 2) {
                const double* xm = xq + XS;
                const double yc = xm[pc], ye = xm[pe], yw = pw >= 0 ? xm[pw] : 0.0;
                xcd = fma(-odd, yc, xcd);
                xdd = fma(-odd, sxp ? ye : yw, xdd);
                xc = fma(odd, yc, xc);
                xe = fma(odd, ye, xe);
                xw = fma(odd, yw, xw);
            }
            s += s0 * (w0 * xc + wE * xe + wW * xw) + sp * (wN * xcd + wDp * xdd) + sm * (wS * xcd + wDm * xdd);
        }
        emit(set, cp, s);
    };
    if (EARLY && !DENSE && tid < M) gather(0, tid, pre_pk, pre_w);
    for (int cp = EARLY && !DENSE ? tid + NT : tid; cp < M; cp += NT) {
        double w6[6];
        for (int k = 0; k < 6; ++k) w6[k] = p.cp_w[(size_t)k * M + cp];
        gather(0, cp, p.cp_pack[cp], w6);
        if (DENSE && dn.w2) {
            for (int k = 0; k < 6; ++k) w6[k] = dn.w2[(size_t)k * M + cp];
            gather(1, cp, p.cp_pack[cp], w6);
        }
    }
    __syncthreads();
}

}  // namespace kfbi
