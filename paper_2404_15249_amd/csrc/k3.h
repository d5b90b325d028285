// Device side of the three-dimensional problem (ellipsoid, 7-point stencil).
//
// Grid layout: the interior nodes 1..N-1 of each axis in an N x N x N FP64
// array, node (i, j, k) at ((k-1) N + (j-1)) N + (i-1); index N-1 of any axis is
// a zero pad.  Jumps at the control points are stored by component:
// J[c M + m] for c = [v], [v_x], [v_y], [v_z], [v_xx], [v_yy], [v_zz], [v_xy],
// [v_xz], [v_yz].
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.h"

namespace kfbi {

// Chunks of 64 samples a workgroup of a GMRES step's reduce launch takes: four where one
// would make more workgroups than compute units.  At 128^3 one leaves 399 partial sums a
// dot for every workgroup of the step launch to add (11.9 us, five rounds of loads) and
// four 100 (7.4 us), and the reduce launch takes as long (9.4 and 9.3); at 64^3 (100
// chunks) four in 25 workgroups make the reduce launch 8.8 us, one in 100 5.6.
inline int reduce3_chunks(int M) { return (M + 63) / 64 > 256 ? 4 : 1; }

struct DevPlan3 {
    int N, log2N, M, I;
    double h, h2, kappa;
    const double* sinq;         // N/2 + 1: sin(pi k / N)
    const ModeConst* modes;     // (N-1)^2: row (k, j) of the x-solve at (k-1)(N-1) + (j-1)
    const double* geo;          // 12 M: normal, t1, t2, S11, S12, S22
    const int* fit_off;         // M + 1
    const int* fit_idx;
    const double* fit_w;        // 5 per neighbour
    const int* irr_node;        // I
    const double* irr_sign;     // I
    // the apply's tables (Apply3Host)
    int E;                      // fit neighbours in all
    const double* fit;          // 3 E
    const double* point;        // 3 M
    const int* sp_wave;         // N <= kSlabMax, as all below
    const int* sp_piece;
    int y_first;
    const int* irr_pos;         // I
    const int* zg_off;
    const int* zg_code;
    const int* st_pos;          // 10 M
    const int* arm_off;         // I + 1
    const int* arm_q;
    const double* arm_d;
    const int* st_node;         // 10 M (-1: a node on the box), node s of point m at s M + m
    const double* st_w;         // 10 M, the same order
    const unsigned char* inside;   // (N+1)^3
};

// J <- Cartesian jumps at every control point for [v] = phi, [F] = fgam (null:
// zero), [d_n v] = 0.
hipError_t launch_jumps3(const DevPlan3& p, const double* phi, const double* fgam, double* J, hipStream_t s);
// The jumps an apply uses: S[m] <- ([v_a], [v_aa]) along the crossing's own axis a and
// far[m] <- the jump terms of its interpolation, for [v] = phi, [F] = fgam (null: zero);
// with check (may be null) also the density's check.
hipError_t launch_surface3(const DevPlan3& p, const double* phi, const double* fgam, double2* S, double* far,
                           const int* skip, const DensityCheck* check, hipStream_t s);
// G <- f masked to Omega (f on the (N+1)^3 grid; null: zero), in the interior layout
hipError_t launch_fill3(const DevPlan3& p, const double* f, double* G, const int* skip, hipStream_t s);
// The correction at every irregular node (Alg. 2 along the three axes): added to G, or
// (G null) put in its place in corr.
hipError_t launch_correct3(const DevPlan3& p, const double* phi, const double2* S, double* G, double* corr,
                           const int* skip, hipStream_t s);
// G <- (L_h - kappa)^-1 G: sine transforms along z and y, tridiagonal solves
// along x, inverse transforms (Alg. 4 in three dimensions); B: transform tile
hipError_t launch_solve3(const DevPlan3& p, double* G, int B, const int* skip, hipStream_t s);
// The same for a right-hand side of corrections alone, in their places in corr, and the
// stencils' nodes alone, into val (N <= kSlabMax; W: scratch, (N-1) N^2).
hipError_t launch_solve3_sparse(const DevPlan3& p, const double* corr, double* W, double* val, const int* skip,
                                hipStream_t s);
// out[m] <- v+ at control point m (Alg. 3, ten-node stencil) from the nodes' values v at
// node (st_node or st_pos); with gm non-null (a GMRES step) the reduce part of the step
// follows instead
hipError_t launch_interp3(const DevPlan3& p, const double* v, const int* node, const double* far, double* out,
                          const int* skip, const GmresBufs* gm, hipStream_t s);
// u <- the grid solution on the (N+1)^3 grid, zero outside Omega when mask
hipError_t launch_grid_out3(const DevPlan3& p, const double* G, bool mask, double* u, hipStream_t s);

}  // namespace kfbi
