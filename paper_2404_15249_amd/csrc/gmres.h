// Restarted GMRES (Alg. 5) on the boundary density, resident on the device.
//
// One step slot is a K apply and, with its last launch, two roles of GMRES work:
//   reduce  (the apply's last launch, per 64 samples) finishes what the step launch
//           before it left: with |z| from that launch's norm partials it scales the
//           apply's output, w = K z / |z|, stores the basis vector V_j = z / |z| and
//           makes the partial dots V_i . w, i <= j.  One more workgroup of the same
//           launch commits column j - 1 meanwhile (gm_commit): the Hessenberg
//           column, the Givens rotations, the residual estimate, and whether the
//           cycle ends (then the triangular solve).
//   step    (gm_step, per chunk of the vector) acts on that: the next K input
//           z = w - sum h_i V_i with its norm partials (not yet scaled: the operator
//           is linear, so |z| is only needed after the apply), or the updated
//           iterate x = phi + sum y_i V_i at the end of a cycle, or the residual
//           as the first vector of a new cycle, or the end of the run; in extra
//           workgroups the next apply's corrections, from the same values.
// So a step needs no launch that waits for the norm, and no count of finished
// workgroups; what it pays is one slot more per cycle (its end is found in that), with
// an apply that is not used, and is left out where that is known beforehand (skip).
// Classical Gram-Schmidt keeps the new vector orthogonal to the basis to about
// eps |w| / |z|; only when |z| < reorth |w| (1e-3 by default) does the reduce launch
// put the dots V_i . z in place of the apply's, and the step launch makes a second
// pass; the next slot's apply is of its result.  For these second-kind operators the
// cancellation stays far above that bound.
// Partial sums are added in a fixed order, so results do not depend on timing.
// The state's two halves alternate: the step launch writes what the apply's
// launches read (ph, converged, r0), the reduce launch what the step launch reads
// (act); no launch reads what it writes, but for the commit's own counters.  So the
// end of a run, which makes the other launches return, is written by the step launch
// alone, also when the commit meets a NaN: a workgroup whose wavefronts read the flag
// before and after the commit's write would part at the next barrier.
#pragma once

#include "device.h"

namespace kfbi {

constexpr int kGmChunk = 256;            // threads of a step workgroup: one vector place each
constexpr int kGmHalo = kSplineK + 1;    // reach of the spline filter on each side
constexpr int kGmOwnSpline = kGmChunk - 2 * kGmHalo;   // places a step workgroup owns beside its halos

enum GmPhase { kGmResidualPh = 0, kGmArnoldi = 1, kGmOver = 2 };
enum GmAct { kGmNextVector = 0, kGmSecondPass = 1, kGmCycleEnd = 2, kGmResidual = 3, kGmDone = 4, kGmFailed = 5 };

// GmresState::converged when a norm of the iteration came out NaN or Inf
constexpr int kGmNonfinite = -2;

// places a step workgroup owns: fewer with a spline, whose filter reads neighbours
__host__ __device__ constexpr int gm_own(bool spline) { return spline ? kGmOwnSpline : kGmChunk; }
__host__ __device__ inline int gm_chunks(int M, bool spline) { return (M + gm_own(spline) - 1) / gm_own(spline); }
__host__ __device__ inline int gm_chunks64(int M) { return (M + 63) / 64; }
// doubles of partial sums a problem needs: dots (m+1) x gc64, norms of the new
// vector and of the apply's output (gc each) and of the residual (gc64)
__host__ __device__ inline size_t gm_part_size(int m, int gc, int gc64) {
    return (size_t)(m + 1) * gc64 + 2 * gc + gc64;
}

struct GmPart {
    double* d1;     // [i * gc64 + c64]
    double* nrm;    // [c]: |z|^2 of the chunk
    double* nrmw;   // [c]: |w|^2 of the chunk
    double* nrm0;   // [c64]
};
__device__ __forceinline__ GmPart gm_part(const GmresBufs& b) {
    GmPart q;
    q.d1 = b.part;
    q.nrm = q.d1 + (size_t)(b.m + 1) * b.gc64;
    q.nrmw = q.nrm + b.gc;
    q.nrm0 = q.nrmw + b.gc;
    return q;
}

// The end of the run, told to the host (GmresPub) by the thread that just wrote the
// state: the state, then (ordered after it) the run's number.
__device__ inline void gm_publish_end(const GmresBufs& b) {
    if (!b.pub) return;
    b.pub->st = *b.st;
    __hip_atomic_store(&b.pub->done, b.st->epoch, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}
// A slot's commit, told to the host; `last`: the next slot's residual is expected to
// end the run.
__device__ __forceinline__ void gm_publish_slot(const GmresBufs& b, bool last) {
    const unsigned slot = (b.st->slot += 1) & (kGmLastSlot - 1);
    if (!b.pub) return;
    __hip_atomic_store(&b.pub->prog, (unsigned long long)b.st->epoch << 32 | (last ? kGmLastSlot : 0u) | slot,
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ double wave_sum(double v) { return wave_allsum(v); }

__device__ inline double gm_block_sum(double v, double* red) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    v = wave_allsum(v);
    __syncthreads();
    if (lane == 0) red[wave] = v;
    __syncthreads();
    return red[0] + red[1] + red[2] + red[3];
}

// This lane's share of n partial sums (every 64th); a wave_sum of it is the same
// in every wavefront that forms it.
__device__ __forceinline__ double gm_lane_share(const double* part, int n) {
    const int lane = threadIdx.x & 63;
    double s = lane < n ? part[lane] : 0.0;
    for (int k = lane + 64; k < n; k += 64) s += part[k];
    return s;
}

// Whether |z|^2 (after the first pass over w) calls for a second pass: with reorth = 1
// always, so that it is known before the norm.
__device__ __forceinline__ bool gm_cancelled(double zz, double ww, double reorth) {
    return reorth >= 1.0 || zz < reorth * reorth * ww;
}

// ---------------------------------------------------------------- reduce launch

// What the reduce launch reads besides the apply's partials, requested before the
// reduction so that the latencies overlap: V_i at the lane's sample for
// i = wave, wave + 16, ... (kMaxRestart <= 64; every row that can be in use, none
// waits for the state), the apply's input, ghat, and the lane's share of the norm
// partials.  NC chunks of 64 samples a workgroup.
template <int NC>
struct GmPre {
    double v[NC][4];
    double xc[NC], gh[NC], zz, ww;
};
template <int NC = 1>
__device__ __forceinline__ GmPre<NC> gm_reduce_prefetch(const GmresBufs& b, int M, int c64) {
    static_assert(kMaxRestart <= 64, "four basis values per lane");
    GmPre<NC> pre;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const GmPart q = gm_part(b);
#pragma unroll
    for (int h = 0; h < NC; ++h) {
        const int cp = (c64 * NC + h) * 64 + lane;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = wave + 16 * k;
            pre.v[h][k] = (i < b.m && cp < M) ? b.V[(size_t)i * M + cp] : 0.0;
        }
        pre.xc[h] = cp < M ? b.xcur[cp] : 0.0;
        pre.gh[h] = wave == 0 && cp < M ? b.ghat[cp] : 0.0;
    }
    pre.zz = gm_lane_share(q.nrm, b.gc);
    pre.ww = gm_lane_share(q.nrmw, b.gc);
    return pre;
}

// The state the reduce launch works from.
struct GmPh {
    int phase, j, second;
    double reorth;
};

// Samples 64 NC c64 .. + 64 NC - 1 by a workgroup of 16 wavefronts right after the
// apply's output there (wv[64 h + lane] in LDS).
template <int NC>
__device__ inline void gm_reduce64(const GmresBufs& b, int M, int c64, const double* wv, const GmPre<NC>& pre, GmPh ph) {
    if (ph.phase == kGmOver) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int cp0 = c64 * NC * 64 + lane;
    const GmPart q = gm_part(b);
    if (ph.phase == kGmResidualPh) {                       // the apply was given the iterate
        if (wave != 0) return;
        double s = 0.0;
#pragma unroll
        for (int h = 0; h < NC; ++h) {
            const int cp = cp0 + 64 * h;
            if (cp >= M) continue;
            b.phi[cp] = pre.xc[h];
            const double r = pre.gh[h] - wv[64 * h + lane];
            b.z[cp] = r;
            s = fma(r, r, s);
        }
        s = wave_sum(s);
        if (lane == 0) q.nrm0[c64] = s;
        return;
    }
    const double zz = wave_sum(pre.zz), ww = wave_sum(pre.ww);
    const bool second = ph.j > 0 && !ph.second && gm_cancelled(zz, ww, ph.reorth);
    const double hn = sqrt(zz), sc = hn > 0.0 ? 1.0 / hn : 0.0;
    double vj[NC], x[NC];                                  // the new basis vector, its product
#pragma unroll
    for (int h = 0; h < NC; ++h) {
        const int cp = cp0 + 64 * h;
        vj[h] = pre.xc[h] * sc;
        x[h] = second ? pre.xc[h] : cp < M ? wv[64 * h + lane] * sc : 0.0;
        if (wave == 0 && cp < M) {
            b.w[cp] = x[h];
            if (!second) b.V[(size_t)ph.j * M + cp] = vj[h];
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int i = wave + 16 * k;
        if (i < ph.j) {
            double s = pre.v[0][k] * x[0];
#pragma unroll
            for (int h = 1; h < NC; ++h) s = fma(pre.v[h][k], x[h], s);
            s = wave_sum(s);
            if (lane == 0) q.d1[(size_t)i * b.gc64 + c64] = s;
        }
    }
    if (!second && wave == (ph.j & 15)) {
        double s = vj[0] * x[0];
#pragma unroll
        for (int h = 1; h < NC; ++h) s = fma(vj[h], x[h], s);
        s = wave_sum(s);
        if (lane == 0) q.d1[(size_t)ph.j * b.gc64 + c64] = s;
    }
}

// The commit, by one more workgroup of the reduce launch: the column the last step
// launch made (its coefficients in b.h, |z| from its norm partials), and what the
// next step launch has to do (st->act).
__device__ inline void gm_commit(const GmresBufs& b, int M) {
    __shared__ double col[kMaxRestart + 2];
    __shared__ double rot[kMaxRestart];
    __shared__ double cs[kMaxRestart], sn[kMaxRestart];
    __shared__ double Hs[kMaxRestart * (kMaxRestart + 1)];
    __shared__ int s_end;
    GmresState* st = b.st;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, m = b.m;
    const GmPart q = gm_part(b);
    // requested together: the norms and what the column needs whatever j is
    const double zzl = gm_lane_share(q.nrm, b.gc), wwl = gm_lane_share(q.nrmw, b.gc);
    double hv = 0.0, cv = 0.0, sv = 0.0;
    if (tid < m) {
        hv = b.h[tid];
        cv = b.cs[tid];
        sv = b.sn[tid];
    }
    const GmPh ph{st->ph, st->j, st->second, st->reorth};
    if (st->converged || ph.phase == kGmOver) {
        if (tid == 0) st->act = kGmDone;
        return;
    }
    if (ph.phase == kGmResidualPh) {
        if (tid == 0) {
            st->act = kGmResidual;
            gm_publish_slot(b, false);
        }
        return;
    }
    const double zz = wave_sum(zzl), ww = wave_sum(wwl), hn = sqrt(zz);
    if (ph.j == 0) {                                       // a new cycle's first vector
        if (tid <= m) b.g[tid] = tid == 0 ? hn : 0.0;
        if (tid == 0) {
            st->first = 0;                                 // read by the residual's step launch only
            st->act = kGmNextVector;
            st->act_j = 0;
            gm_publish_slot(b, false);
        }
        return;
    }
    const int j = ph.j - 1, jn = ph.j;                     // the column committed; columns made
    if (!ph.second && gm_cancelled(zz, ww, ph.reorth)) {
        if (tid == 0) {
            st->act = kGmSecondPass;
            st->act_j = j;
            gm_publish_slot(b, false);
        }
        return;
    }
    if (tid <= j) col[tid] = hv;
    if (tid < j) {
        cs[tid] = cv;
        sn[tid] = sv;
    }
    __syncthreads();
    if (tid == 0) {
        // previous rotations down the column, eight at a time: their operands
        // are read together; the rotated entries go to rot[]
        double a = col[0];
        for (int i0 = 0; i0 < j; i0 += 8) {
            double cn[8], c8[8], s8[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const bool in = i0 + u < j;
                cn[u] = in ? col[i0 + u + 1] : 0.0;
                c8[u] = in ? cs[i0 + u] : 1.0;
                s8[u] = in ? sn[i0 + u] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (i0 + u < j) {
                    rot[i0 + u] = c8[u] * a + s8[u] * cn[u];
                    a = -s8[u] * a + c8[u] * cn[u];
                }
            }
        }
        for (int i = 0; i < j; ++i) col[i] = rot[i];
        const double den = hypot(a, hn), gj = b.g[j];
        if (!isfinite(den) || !isfinite(gj)) {             // NaN or Inf in the data: stop here
            st->act = kGmFailed;
            s_end = -1;
        } else {
            const double c = den > 0.0 ? a / den : 1.0;
            const double s = den > 0.0 ? hn / den : 0.0;
            col[j] = den;
            col[j + 1] = 0.0;
            b.cs[j] = c;
            b.sn[j] = s;
            b.g[j + 1] = -s * gj;
            b.g[j] = c * gj;
            const int itn = st->it + 1;
            const double est = fabs(s * gj) / st->r0;
            st->relres = est;
            st->it = itn;
            const bool end = est < st->tol || jn == m || itn >= st->max_iter || hn == 0.0;
            s_end = end ? 1 : 0;
            st->jn = jn;
            st->act = end ? kGmCycleEnd : kGmNextVector;
            st->act_j = jn;
            gm_publish_slot(b, est < st->tol || itn >= st->max_iter || hn == 0.0);
        }
    }
    __syncthreads();
    if (s_end < 0) return;
    double* Hj = b.H + (size_t)j * (m + 1);
    if (tid <= j + 1) Hj[tid] = col[tid];
    if (!s_end) return;
    // end of the cycle: H[0:jn, 0:jn] y = g[0:jn], one wavefront, column by column
    for (int t = tid; t < jn * (m + 1); t += blockDim.x) {
        const int kc = t / (m + 1), i = t % (m + 1);
        Hs[t] = kc == j ? (i <= jn ? col[i] : 0.0) : b.H[t];
    }
    __syncthreads();
    if (wave == 0) {
        double gk = lane < jn ? b.g[lane] : 0.0;
        double yk = 0.0;
        for (int i = jn - 1; i >= 0; --i) {
            const double yi = readlane_f64(gk, i) / Hs[i * (m + 1) + i];   // i is the same in every lane
            if (lane == i) yk = yi;
            if (lane < i) gk -= Hs[i * (m + 1) + lane] * yi;
        }
        if (lane < jn) b.y[lane] = yk;
    }
}

// ---------------------------------------------------------------- step launch

// Chunk counts up to which one thread adds a row of dot partials itself; above
// them (the surface problem's long vectors) the workgroup's threads split the work,
// so the chain of dependent loads stays short.
constexpr int kGmSerialSums = 32;

// h_i = the sum of row i of the nco chunk partials, i < m, for many chunks:
// kGmChunk / m threads per row, each adding every (kGmChunk / m)-th chunk in
// order, then the parts added in order.  Returns h_tid for tid < m; the same
// order in every workgroup, so they all agree.  Called by the whole workgroup.
__device__ inline double gm_dots_spread(const double* d1, int m, int nco) {
    __shared__ double part[kGmChunk];
    const int tid = threadIdx.x, P = kGmChunk / m;
    double s = 0.0;
    if (tid < m * P) {
        const int i = tid / P, r = tid - i * P;
        const double* row = d1 + (size_t)i * nco;
        for (int c0 = r; c0 < nco; c0 += 16 * P) {
            double v[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) v[u] = c0 + u * P < nco ? row[c0 + u * P] : 0.0;   // issued together
#pragma unroll
            for (int u = 0; u < 16; ++u) s += v[u];
        }
    }
    part[tid] = s;
    __syncthreads();
    double h = 0.0;
    if (tid < m)
        for (int r = 0; r < P; ++r) h += part[tid * P + r];
    return h;
}

// What a step workgroup reads, requested before the state is known: at the
// thread's vector element every basis row that can be in use (rows past the current
// column are not used), the apply's output, the iterate and the residual; per
// thread i < m the sum of row i's dot partials and y_i; the lane's share of the
// residual's norm.
struct GmStepIn {
    double v[4][16];
    double w, phi, z;
    double h, y, rr;
};
__device__ __forceinline__ GmStepIn gm_step_loads(const GmresBufs& b, int M, int e, bool in) {
    const int tid = threadIdx.x, m = b.m, nco = b.gc64;
    const GmPart q = gm_part(b);
    GmStepIn u;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int i = 16 * g + k;
            u.v[g][k] = (in && i < m) ? b.V[(size_t)i * M + e] : 0.0;
        }
    }
    u.w = in ? b.w[e] : 0.0;
    u.phi = in ? b.phi[e] : 0.0;
    u.z = in ? b.z[e] : 0.0;
    u.h = u.y = 0.0;
    if (tid < m) u.y = b.y[tid];
    u.rr = gm_lane_share(q.nrm0, nco);
    if (nco <= kGmSerialSums) {
        if (tid < m) {
            double sum = 0.0;
#pragma unroll 16
            for (int cc = 0; cc < nco; ++cc) sum += q.d1[(size_t)tid * nco + cc];   // loads issued together
            u.h = sum;
        }
    } else {
        u.h = gm_dots_spread(q.d1, m, nco);
    }
    return u;
}

// What a step does, the same in every workgroup of the launch.
struct GmTodo {
    int act, j;              // act_j
    bool done;               // the run has ended (with kGmResidual or kGmFailed), or had (kGmDone)
    int converged;           // then
    int it, max_iter;        // the state's
    double reorth;
    double rel, r0;
};
__device__ __forceinline__ GmTodo gm_todo(const GmresBufs& b, const GmStepIn& u) {
    const GmresState* st = b.st;
    GmTodo t{st->act, st->act_j, false, 0, st->it, st->max_iter, st->reorth, 0.0, 0.0};
    if (t.act == kGmDone) t.done = true;
    if (t.act == kGmFailed) {
        t.done = true;
        t.converged = kGmNonfinite;
    }
    if (t.act != kGmResidual) return t;
    const double beta = sqrt(wave_sum(u.rr));
    if (!isfinite(beta)) {                                 // NaN or Inf in the data: stop here
        t.done = true;
        t.converged = kGmNonfinite;
        return t;
    }
    t.r0 = st->first ? beta : st->r0;
    t.rel = t.r0 > 0.0 ? beta / t.r0 : 0.0;
    const bool small = t.r0 == 0.0 || beta == 0.0 || t.rel < st->tol;
    if (small || t.it >= t.max_iter) {
        t.done = true;
        t.converged = small ? 1 : -1;
    }
    return t;
}

// The coefficients of the basis vectors (into coef, kMaxRestart doubles of LDS) and
// the next input at the thread's element: the new vector w - sum h_i V_i (the
// second pass the same with its own dots), the updated iterate phi + sum y_i V_i,
// or the residual.
__device__ __forceinline__ double gm_next_value(const GmTodo& t, const GmStepIn& u, double* coef) {
    const int tid = threadIdx.x;
    const bool cycle_end = t.act == kGmCycleEnd;
    const int n = t.act == kGmResidual ? 0 : cycle_end ? t.j : t.j + 1;   // basis vectors used
    double cy = u.y, ch = -u.h;
    asm volatile("" : "+v"(cy), "+v"(ch));
    if (tid < kMaxRestart) coef[tid] = tid < n ? (cycle_end ? cy : ch) : 0.0;
    __syncthreads();
    // values, not addresses, to choose from (the struct has to stay in registers)
    double aw = u.w, ap = u.phi, az = u.z;
    asm volatile("" : "+v"(aw), "+v"(ap), "+v"(az));
    double a = t.act == kGmResidual ? az : cycle_end ? ap : aw;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        if (16 * g < n) {
#pragma unroll
            for (int k = 0; k < 16; ++k)
                if (16 * g + k < n) a = fma(coef[16 * g + k], u.v[g][k], a);
        }
    }
    return a;
}

// Spline second derivative at window place w (the filter reads kGmHalo places
// on each side).
__device__ __forceinline__ double gm_spline_s2(const double* __restrict__ taps, const double* win, int w) {
    constexpr int K = kSplineK;
    double s = 0.0;
#pragma unroll
    for (int q = -K - 1; q <= K + 1; ++q) s = fma(taps[q + K + 1], win[w + q], s);
    return s;
}

// The state for the next slot, by thread 0 of the step launch's first workgroup.  The
// next apply is not used (skip) when its input ends the cycle, by the restart length or
// the iteration cap, or is to have a second pass first; the reduce launch only commits
// it then.  At 4096^2 twelve steps in cycles of one went from 3.25 to 2.63 ms so, and
// with reorth = 1 in one cycle from 2.58 to 1.93.
__device__ __forceinline__ void gm_advance(const GmresBufs& b, const GmTodo& t) {
    GmresState* st = b.st;
    if (t.act == kGmNextVector || t.act == kGmSecondPass) {
        st->ph = kGmArnoldi;
        st->j = t.j + 1;
        st->second = t.act == kGmSecondPass;
        st->skip = t.j + 1 == b.m || t.it + 1 >= t.max_iter || (t.act == kGmNextVector && t.reorth >= 1.0);
    } else if (t.act == kGmCycleEnd) {
        st->ph = kGmResidualPh;
        st->skip = 0;
    } else if (t.act == kGmFailed) {
        st->converged = t.converged;
        st->skip = 1;
        st->ph = kGmOver;
        gm_publish_end(b);
    } else if (t.act == kGmResidual) {
        if (t.converged != kGmNonfinite) {
            st->res_applies += 1;
            st->r0 = t.r0;
            st->relres = t.rel;
        }
        if (t.done) {
            st->converged = t.converged;
            st->skip = 1;
            st->ph = kGmOver;
            gm_publish_end(b);
        } else {
            st->cycles += 1;
            st->ph = kGmArnoldi;
            st->j = 0;
            st->second = 0;
            if (b.pub) b.pub->again += 1;
        }
    }
}

// The place of window index tid of chunk c: the element, whether it exists and
// whether the chunk owns it (with a spline the window wraps around Gamma and has
// kGmHalo places on each side).
struct GmPlaceOf {
    int e;
    bool in, own;
};
__device__ __forceinline__ GmPlaceOf gm_place(const GmresBufs& b, int M, int c, bool spline) {
    const int tid = threadIdx.x;
    if (!spline) {
        const int e = c * kGmChunk + tid;
        return {e, e < M, e < M};
    }
    const int at = c * kGmOwnSpline - kGmHalo + tid;
    int e = at % M;
    if (e < 0) e += M;
    return {e, true, tid >= kGmHalo && tid < kGmHalo + kGmOwnSpline && at < M};
}

// Chunk c of the step launch (see the head of this file); taps: the spline filter
// of a curve's density, null where the density has no spline (the surface problem).
__device__ inline void gm_step(const double* __restrict__ taps, const GmresBufs& b, int M, int c) {
    __shared__ double win[kGmChunk];
    __shared__ double coef[kMaxRestart];
    __shared__ double red[kGmChunk / 64];
    const int tid = threadIdx.x;
    const GmPlaceOf pl = gm_place(b, M, c, taps != nullptr);
    const GmStepIn u = gm_step_loads(b, M, pl.e, pl.in);
    const GmTodo t = gm_todo(b, u);
    if (t.act == kGmDone) return;
    if (t.done) {                                          // the run has ended: the iterate goes out
        double* xo = b.st->xout;
        if (xo && t.converged != kGmNonfinite && pl.own) xo[pl.e] = u.phi;
        if (c == 0 && tid == 0) gm_advance(b, t);
        return;
    }
    const double x = gm_next_value(t, u, coef);
    if (pl.own) b.xcur[pl.e] = x;
    if (taps) {
        win[tid] = x;
        __syncthreads();
        if (pl.own) b.s2cur[pl.e] = gm_spline_s2(taps, win, tid);
    }
    if (t.act != kGmCycleEnd) {
        const GmPart q = gm_part(b);
        const double sz = gm_block_sum(pl.own ? x * x : 0.0, red);
        const double sw = gm_block_sum(pl.own ? u.w * u.w : 0.0, red);
        if (tid == 0) {
            q.nrm[c] = sz;
            q.nrmw[c] = sw;
        }
    }
    if (c == 0) {
        if (tid <= t.j && t.act == kGmNextVector) b.h[tid] = u.h;
        if (tid <= t.j && t.act == kGmSecondPass) b.h[tid] += u.h;
        if (tid == 0) gm_advance(b, t);
    }
}

// The corrections (Alg. 2) of correction chunk cc from the density's values and
// second derivatives over the chunk's window (xw, sw), requested plan data in hand.
struct GmCorr {
    int4 arm, ch;
    double4 dd;
    double sg;
    int slot;
    PointGeom gs[4];
    int axs[4];
};
__device__ __forceinline__ GmCorr gm_corr_loads(const DevPlan& p, int cc) {
    static_assert(kCorrWindow <= kGmChunk && kCorrChunk <= kGmChunk, "one window place and one node place per thread");
    const int tid = threadIdx.x;
    // the node's plan data (place tid of the chunk's kCorrChunk) is requested
    // with the chunk itself: neither waits for the other
    GmCorr k;
    k.arm = make_int4(-1, -1, -1, -1);
    k.dd = make_double4(0.0, 0.0, 0.0, 0.0);
    k.sg = 0.0;
    k.slot = 0;
    if (tid < kCorrChunk) {
        const size_t at = (size_t)cc * kCorrChunk + tid;
        k.arm = p.cc_arm[at];
        k.dd = p.cc_d[at];
        k.sg = p.cc_s[at];
        k.slot = p.cc_pos[at];
    }
    k.ch = p.cc_chunk[cc];                                 // first, end, first knot, width
    return k;
}
__device__ __forceinline__ void gm_corr_geometry(const DevPlan& p, GmCorr& k) {
    const int ks[4] = {k.arm.x, k.arm.y, k.arm.z, k.arm.w};
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        if (ks[a] >= 0) {
            k.gs[a] = p.q_geo[ks[a]];
            k.axs[a] = p.q_axis[ks[a]];
        } else {
            k.gs[a] = PointGeom{};
            k.axs[a] = 0;
        }
    }
}
// xw: the window's values (place tid written by thread tid before a barrier here);
// fw (null: [F] = 0), f2w: the same of f on Gamma
__device__ inline void gm_corr_finish(const DevPlan& p, const GmCorr& k, const double* xw, double* sw,
                                      double* __restrict__ corr_il, const double* fw = nullptr, double* f2w = nullptr) {
    const int M = p.M, tid = threadIdx.x;
    const int4 ch = k.ch;
    __syncthreads();
    if (tid >= kGmHalo && tid < ch.w - kGmHalo) {
        sw[tid] = gm_spline_s2(p.taps, xw, tid);
        if (fw) f2w[tid] = gm_spline_s2(p.taps, fw, tid);
    }
    __syncthreads();
    if (tid >= ch.y - ch.x) return;
    const int ks[4] = {k.arm.x, k.arm.y, k.arm.z, k.arm.w};
    const double ds[4] = {k.dd.x, k.dd.y, k.dd.z, k.dd.w};
    const double sg = k.sg;
    double acc = 0.0;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        if (ks[a] < 0) continue;
        const double d = ds[a];
        const PointGeom& g = k.gs[a];
        // the segment's first knot in the window: the first copy past the filter's reach
        // of its start (a window longer than M holds knots several times, and those
        // inside the reach of its ends have no second derivative)
        const int l = kGmHalo + ((g.seg - ch.z - kGmHalo) % M + M) % M;
        // the spline on the segment, as spline_at computes it
        const double s0 = sw[l], s1 = sw[l + 1];
        const double y0 = xw[l], y1 = xw[l + 1], u = g.u, w = 1.0 - u;
        const double sixth = 1.0 / 6.0;
        const double P = w * y0 + u * y1 + (w * w * w - w) * s0 * sixth + (u * u * u - u) * s1 * sixth;
        const double P1 = (y1 - y0) - (3.0 * w * w - 1.0) * s0 * sixth + (3.0 * u * u - 1.0) * s1 * sixth;
        const double P2 = w * s0 + u * s1;
        const double F = fw ? w * fw[l] + u * fw[l + 1] + (w * w * w - w) * f2w[l] * sixth + (u * u * u - u) * f2w[l + 1] * sixth
                            : 0.0;
        // the jumps, as jumps_at computes them
        const double Ps = P1 * g.a1;
        double jv, gv, hh;
        if (p.normal_jump) {
            const double vtt = g.curv * P, vtn = Ps, vnn = F - vtt;
            jv = 0.0;
            if (k.axs[a]) {
                gv = P * g.ny;
                hh = vtt * g.ty * g.ty + 2.0 * vtn * g.ty * g.ny + vnn * g.ny * g.ny;
            } else {
                gv = P * g.nx;
                hh = vtt * g.tx * g.tx + 2.0 * vtn * g.tx * g.nx + vnn * g.nx * g.nx;
            }
        } else {
            const double Pss = P2 * g.a2 - P1 * g.a3;
            const double vtt = Pss, vtn = -g.curv * Ps, vnn = F + p.kappa * P - vtt;
            jv = P;
            if (k.axs[a]) {
                gv = Ps * g.ty;
                hh = vtt * g.ty * g.ty + 2.0 * vtn * g.ty * g.ny + vnn * g.ny * g.ny;
            } else {
                gv = Ps * g.tx;
                hh = vtt * g.tx * g.tx + 2.0 * vtn * g.tx * g.nx + vnn * g.nx * g.nx;
            }
        }
        acc -= sg * (jv + d * gv + 0.5 * d * d * hh);
    }
    corr_il[k.slot] = acc * p.inv_h2;
}

// Correction chunk cc in the step launch: the chunk's window of the next input is
// formed here from the same values, in the same order, as gm_step forms it, so the
// next apply starts at its sparse sums.  corr_il in the sparse-sum layout.
__device__ inline void gm_step_corrections(const DevPlan& p, const GmresBufs& b, int cc, double* __restrict__ corr_il) {
    __shared__ double xw[kCorrWindow];
    __shared__ double sw[kCorrWindow];
    __shared__ double coef[kMaxRestart];
    const int tid = threadIdx.x;
    GmCorr k = gm_corr_loads(p, cc);
    const GmStepIn u = gm_step_loads(b, p.M, (k.ch.z + tid) % p.M, tid < k.ch.w);
    gm_corr_geometry(p, k);
    const GmTodo t = gm_todo(b, u);
    if (t.done) return;
    const double x = gm_next_value(t, u, coef);
    if (tid < k.ch.w) xw[tid] = x;
    gm_corr_finish(p, k, xw, sw, corr_il);
}

// ---------------------------------------------------------------- a caller's density

// What an apply needs of a caller's density y before its sparse solve, in one launch
// of kGmChunk-thread workgroups: gc chunks make the spline second derivatives
// (s2), the rest one correction chunk each from their own windows of y, as the step
// launch does (three launches before: the check, the spline, the corrections, 13 us
// together against 5).  With flag, the chunks also look for a NaN or Inf: flag is
// set (it is 0 before: the launch of the call before cleared it, as this one clears
// flag_next), and the call's number goes to *bad for the host.
__device__ inline void gm_density(const DevPlan& p, const double* __restrict__ y, double* __restrict__ s2,
                                  double* __restrict__ corr_il, int gc, int* flag, int* flag_next, unsigned* bad,
                                  unsigned number) {
    __shared__ double win[kGmChunk];
    __shared__ double sw[kGmChunk];
    const int tid = threadIdx.x, c = blockIdx.x, M = p.M;
    if (c >= gc) {
        GmCorr k = gm_corr_loads(p, c - gc);
        if (tid < k.ch.w) win[tid] = y[(k.ch.z + tid) % M];
        gm_corr_geometry(p, k);
        gm_corr_finish(p, k, win, sw, corr_il);
        return;
    }
    const int at = c * kGmOwnSpline - kGmHalo + tid;
    int e = at % M;
    if (e < 0) e += M;
    const double x = y[e];
    win[tid] = x;
    if (flag) {
        if (!isfinite(x)) {                                // benign races: every writer stores the same
            *flag = 1;
            __hip_atomic_store(bad, number, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        if (c == 0 && tid == 0) *flag_next = 0;
    }
    __syncthreads();
    if (tid >= kGmHalo && tid < kGmHalo + kGmOwnSpline && at < M) s2[e] = gm_spline_s2(p.taps, win, tid);
}

// gm_density for an interface solve: the density y and f on Gamma (either null: zero).
__device__ inline void gm_density_f(const DevPlan& p, const double* __restrict__ y, const double* __restrict__ f,
                                    double* __restrict__ s2, double* __restrict__ f2, double* __restrict__ corr_il, int gc) {
    __shared__ double win[kGmChunk], sw[kGmChunk], fw[kGmChunk], f2w[kGmChunk];
    const int tid = threadIdx.x, c = blockIdx.x, M = p.M;
    if (c >= gc) {
        GmCorr k = gm_corr_loads(p, c - gc);
        if (tid < k.ch.w) {
            const int e = (k.ch.z + tid) % M;
            win[tid] = y ? y[e] : 0.0;
            fw[tid] = f ? f[e] : 0.0;
        }
        gm_corr_geometry(p, k);
        gm_corr_finish(p, k, win, sw, corr_il, fw, f2w);
        return;
    }
    const int at = c * kGmOwnSpline - kGmHalo + tid;
    int e = at % M;
    if (e < 0) e += M;
    win[tid] = y ? y[e] : 0.0;
    fw[tid] = f ? f[e] : 0.0;
    __syncthreads();
    if (tid >= kGmHalo && tid < kGmHalo + kGmOwnSpline && at < M) {
        if (y) s2[e] = gm_spline_s2(p.taps, win, tid);
        if (f) f2[e] = gm_spline_s2(p.taps, fw, tid);
    }
}

// ---------------------------------------------------------------- start of a run

// The start of a GMRES run, one launch of kGmChunk-thread workgroups: the gc
// step chunks, then (with p) one per correction chunk.  Every workgroup first
// tests the initial guess phi_in (null: zero) for nonzero values and sums |ghat|^2
// (ghat <- rhs when rhs is given, else already in place) in one fixed order, so all
// of them hold the same beta and know what the run does:
//  - a zero guess has the residual ghat itself (K 0 = 0; Alg. 5 with x_0 = 0),
//    so its first cycle starts here: ghat is the first K input;
//  - any other guess makes phi_in the first K input, and the first slot is a
//    residual slot;
//  - beta = 0 (x = 0 solves it) or a NaN or Inf ends the run at once.
// Workgroup 0 writes the whole state (nothing is uploaded from the host); the step
// chunks copy phi_in and rhs into phi and ghat and write the
// first input with its spline second derivatives; the correction workgroups make
// its corrections.  xout (may be null) is where the step launch that ends the run
// copies the iterate.
__device__ inline void gm_begin(const DevPlan* p, const double* __restrict__ taps, const GmresBufs& b, int M,
                                const double* __restrict__ rhs, const double* __restrict__ phi_in, double tol,
                                int max_iter, double reorth, double* xout, double* __restrict__ corr_il,
                                unsigned epoch) {
    __shared__ double red[kGmChunk / 64];
    __shared__ double win[kGmChunk];
    __shared__ double sw[kGmChunk];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c = blockIdx.x;
    const double* gsrc = rhs ? rhs : b.ghat;
    double ss = 0.0;
    int nz = 0;
    for (int e = tid; e < M; e += kGmChunk) {
        const double gh = gsrc[e];
        if (phi_in) nz |= phi_in[e] != 0.0;                // a NaN counts as nonzero
        ss = fma(gh, gh, ss);
    }
    ss = wave_sum(ss);
    if (lane == 0) red[wave] = ss;
    const bool nonzero = __syncthreads_or(nz) != 0;
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kGmChunk / 64; ++w) t += red[w];   // fixed order
    const double beta = sqrt(t);
    const bool bad = !nonzero && !isfinite(beta), zero = !nonzero && beta == 0.0, over = bad || zero;
    const double* xsrc = nonzero ? phi_in : gsrc;
    if (c == 0) {
        const GmPart q = gm_part(b);
        for (int k = tid; k < b.gc; k += kGmChunk) {       // the first vector's norm, for the reduce launch
            q.nrm[k] = k == 0 ? t : 0.0;
            q.nrmw[k] = 0.0;
        }
        if (tid == 0) {
            GmresState* st = b.st;
            st->j = 0;
            st->second = 0;
            st->it = 0;
            st->res_applies = 0;
            st->tol = tol;
            st->max_iter = max_iter;
            st->reorth = reorth;
            st->jn = 0;
            st->xout = xout;
            st->converged = bad ? kGmNonfinite : zero ? 1 : 0;
            st->skip = over ? 1 : 0;
            st->first = nonzero ? 1 : 0;
            st->r0 = nonzero ? 0.0 : beta;
            st->relres = zero ? 0.0 : 1.0;
            st->cycles = nonzero || over ? 0 : 1;
            st->ph = over ? kGmOver : nonzero ? kGmResidualPh : kGmArnoldi;
            st->act = kGmDone;
            st->act_j = 0;
            st->epoch = epoch;
            st->slot = 0;
            if (over) gm_publish_end(b);
        }
    }
    if (c < b.gc) {
        const GmPlaceOf pl = gm_place(b, M, c, taps != nullptr);
        if (pl.own) {
            b.phi[pl.e] = phi_in ? phi_in[pl.e] : 0.0;
            if (rhs) b.ghat[pl.e] = rhs[pl.e];
            if (zero && xout) xout[pl.e] = 0.0;
        }
        if (over) return;
        const double x = pl.in ? xsrc[pl.e] : 0.0;
        if (pl.own) b.xcur[pl.e] = x;
        if (!taps) return;
        win[tid] = x;
        __syncthreads();
        if (pl.own) b.s2cur[pl.e] = gm_spline_s2(taps, win, tid);
    } else {
        if (over) return;
        GmCorr k = gm_corr_loads(*p, c - b.gc);
        if (tid < k.ch.w) win[tid] = xsrc[(k.ch.z + tid) % M];
        gm_corr_geometry(*p, k);
        gm_corr_finish(*p, k, win, sw, corr_il);
    }
}

}  // namespace kfbi
