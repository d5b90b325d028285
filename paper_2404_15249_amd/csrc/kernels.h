// Device data layouts and kernel launchers of the KFBI library (gfx950).
#pragma once

#include <hip/hip_runtime.h>

#include "plan.h"

namespace kfbi {

// Per y-mode constants of the tridiagonal solve along x (Alg. 4).  For mode l
// the system is x[i-1] - beta x[i] + x[i+1] = e[i], beta = 2 + h^2 (kappa - lambda_l),
// lambda_l = -(4/h^2) sin^2(pi l / 2N); r is the root of r^2 - beta r + 1 = 0 in (0, 1).
struct ModeConst {
    double r;      // decay root
    double rinv;   // 1 / r
    double logr;   // log r
    double rC;     // r^C (C = N / 64, the chunk one lane owns)
    double smc;    // -r / (1 - r^(2N)): scale of the rank-one boundary fix
    double rH;     // r^modes_chunk(N): the chunk of a lane of the sparse fast solve
    double rN1;    // r^(N-1)
    double pad;
};

// nodes of a row one lane of the sparse fast solve owns: N / 64 up to 32 (a row of
// 4096 takes two wavefronts)
__host__ __device__ constexpr int modes_chunk(int N) { return N / 64 < 32 ? N / 64 : 32; }

// doubles of one padded solution of the sparse fast solve
__host__ __device__ constexpr int modes_stride_of(int N) { return N + N / modes_chunk(N); }

// place of row j (0 <= j <= N/2) among a block's row sines: even rows, then odd
// ones, so that neighbouring columns' nodes of one parity read neighbouring
// places (at N = 4096 j itself: the sines are looked up)
__host__ __device__ constexpr int modes_row_place(int j, int N) { return N <= 2048 ? (j >> 1) + (j & 1) * (N / 4 + 1) : j; }

constexpr int kModeWaves = 16;     // wavefronts of a sparse-fast-solve workgroup (= node sub-tables)

// Everything a kernel needs to read one problem's plan on the device.
struct DevPlan {
    int n, N, M, Q, I;
    int log2N;
    int normal_jump;          // 0: the density is [v] ([d_n v] = 0); 1: it is [d_n v] ([v] = 0)
    double lo, h, inv_h2, h2, kappa;
    const PointGeom* q_geo;   // Q
    const int* q_axis;        // Q
    const PointGeom* z_geo;   // M
    const double* zx;         // M sample positions
    const double* zy;         // M
    const int* irr_i;         // I
    const int* irr_j;         // I
    const double* irr_s;      // I
    const int* arm_q;         // 4 I
    const double* arm_d;      // 4 I
    const int* col_ptr;       // N + 1 entries used (i = 0..N)
    const int* sub_off;       // kModeWaves + 1: rows [sub_off[w], sub_off[w+1]) of the interleaved
                              // table are sub-table w (multiples of kSlots)
    int sub_offv[kModeWaves + 1];   // the same offsets by value, so that a kernel given the plan by
                                    // value reads them with its arguments
    const int* split;         // 3 n_split: (dest, first extra piece, extra pieces) of each
                              // column half whose nodes are cut into several pieces (see il_ij)
    int n_split;
    const int* il_ij;         // T x 64, slot t*64 + L of lane L of the sub-table owning row t: kIl* below.
                              // A column's nodes with even j and those with odd j form
                              // one piece each, or several when there are many; a step is 64 pieces of
                              // about equal length, one a lane, padded to the longest (pads: zero
                              // corrections).  In the step's last row dest is the place of the lane's
                              // sums in a pair's block: for a first piece xpos = i + (i - 1) /
                              // modes_chunk(N), column i's place in the padded solution, plus
                              // modes_stride_of(N) for odd j; for an extra piece 2 modes_stride_of(N) +
                              // its index; 0 (a place nothing reads) for a lane with no piece
    const int* il_pos;        // I: slot of irregular node r in the interleaved layout
    int T;                    // slots per lane, a multiple of kSlots
    const int* cp_pack;       // M: i0 | j0 << 13 | (sx > 0) << 26 | (sy > 0) << 27
    const int* cp_i0;         // M
    const int* cp_j0;         // M
    const int* cp_sxy;        // M: bit 0 sx>0, bit 1 sy>0
    const double* cp_w;       // 6 x M (row k: node k of every sample): weights of the six stencil values in the extracted quantity (v+, or
                              // d_n v+ for a plan that extracts the normal derivative)
    const unsigned char* cp_out;   // 6 M
    const unsigned char* inside;   // (n+1)^2
    const unsigned char* mask8;    // (n+1) n / 8: the same for interior nodes as bits, byte j (n/8) + (i-1)/8, bit (i-1)%8
    const double* sinq;       // N/2 + 1: sin(pi k / N)
    const ModeConst* modes;   // N (index l = 1..N-1 used)
    const double* taps;       // 2 K + 3 spline filter taps
    int K;                    // must equal kSplineK
    // the irregular nodes in the order of their first crossing along Gamma, cut
    // into chunks of at most kCorrChunk nodes whose crossings' spline segments
    // span at most a window of kCorrWindow knots (with the filter's reach):
    // chunk c = (first, end, first window knot, window length) of that order.
    // Per node, at place c kCorrChunk + (its place in the order - first): its
    // arms (crossing index, -1 unused; the distance d), its side and its slot in
    // the sparse-sum layout; the places past a chunk's end are pads with no arms.
    const int4* cc_arm;       // n_cc kCorrChunk
    const double4* cc_d;      // n_cc kCorrChunk
    const double* cc_s;       // n_cc kCorrChunk
    const int* cc_pos;        // n_cc kCorrChunk
    const int4* cc_chunk;     // n_cc
    int n_cc;
};

constexpr int kSplineK = 30;
constexpr int kCorrChunk = 256;    // irregular nodes per correction chunk (one workgroup)
constexpr int kCorrWindow = 256;   // knots of a chunk's density window
constexpr int kSlots = 4;          // table rows loaded together by the sparse sine sums
constexpr int kMaxModesPerGroup = 8;
constexpr int kMaxExtra = 126;      // extra pieces of long column halves (per pair of modes): what the LDS has room for at 2048
// a node table entry: bit 31 j > N/2; 16-30 dest; 4-15 modes_row_place(min(j, N - j)); 1 last row of a step
constexpr int kIlRow = 0xfff0, kIlLast = 2;
constexpr int kMaxRestart = 64;    // GMRES restart length cap (LDS-resident Hessenberg)
constexpr int kMaxSamples = 12288; // boundary samples per problem (the one-workgroup steps of krylov.hip: twelve a thread)

// Source of the interface jumps: either computed from densities on the
// spline (phi, fgam may be null) or given directly (jq / jz, 6 per point).
struct JumpSrc {
    const double* phi;
    const double* phi_s2;    // spline second derivatives of phi (required with phi)
    const double* fgam;
    const double* fgam_s2;   // spline second derivatives of fgam (required with fgam)
    const double* jq;
    const double* jz;
};

struct GmresState {
    int ph;          // what the next apply is of (GmPhase in gmres.h): the iterate, or basis vector j
    int j;           // the basis vector the apply makes (its input is that vector, not yet scaled)
    int second;      // 1: the input has had its second Gram-Schmidt pass
    int act;         // what the next step launch does (GmAct in gmres.h), and the column it is about
    int act_j;
    int it;          // K_D applications made by the Arnoldi process
    int first;       // 1 until r0 is known
    int converged;   // 1 converged, -1 iteration cap, -2 a NaN or Inf met (kGmNonfinite), 0 running
    int skip;        // 1: the next apply is not used (the run is over, or see gm_advance in gmres.h)
    int cycles;
    double r0;
    double relres;
    double tol;      // stop when the relative residual drops below tol (<= 0: never)
    int max_iter;    // cap on Arnoldi steps
    int jn;          // columns of the cycle just finished
    int res_applies; // K applications made for residuals (cycle starts and the final check)
    double reorth;   // second Gram-Schmidt pass when |z| < reorth |w| (0: never, 1: always)
    double* xout;    // where the step launch that ends the run copies the iterate (null: nowhere)
    unsigned epoch;  // the run's number, for the host (GmresPub)
    unsigned slot;   // slots whose commit has run
};

constexpr int kIterNonfinite = -2;

// State of a Richardson or BiCGSTAB run (krylov.hip), in device memory.
struct IterState {
    int it;          // Richardson: updates made; BiCGSTAB: iterations begun
    int done;        // 0 running, 1 converged, -1 iteration cap or breakdown, -2 (kIterNonfinite)
                     // a NaN or Inf met (launches skip while nonzero)
    int max_iter;
    int started;     // 1 once r0 is known
    int half;        // BiCGSTAB: 1 if it stopped half way through an iteration (one apply short)
    unsigned slot;   // slots whose step has run: Richardson's updates, BiCGSTAB's half iterations
    double tol, r0, relres;
    double rho, alpha, omega;
    double gamma;    // Richardson relaxation
    unsigned epoch;  // the run's number, for the host (GmresPub)
};

// What a run tells the host while it goes on (pinned, coherent host memory the
// device writes; the host reads it without waiting for the stream).  prog: epoch in
// the upper half; then kGmLastSlot when the commit found that the run ends at the
// next slot's residual if that confirms it; slots committed in the 31 bits below (modulo).
struct GmresPub {
    GmresState st;             // the final state, written before `done`
    unsigned long long prog;
    unsigned done;             // the run's epoch once it is over
    unsigned again;            // residuals that did not end a run (any run's)
    unsigned bad;              // number of the last apply whose density held a NaN or Inf
    IterState iter;            // a Richardson or BiCGSTAB run's final state, likewise
};
constexpr unsigned kGmLastSlot = 0x80000000u;

struct GmresBufs {
    double* V;       // (m+1) M
    double* H;       // (m+1) m, column j at H + j (m+1)
    double* h;       // m: the column's coefficients, as the step launch made them
    double* cs;      // m
    double* sn;      // m
    double* g;       // m + 1
    double* ghat;    // M
    double* phi;     // M
    double* xcur;    // M: input of the next K_D apply
    double* s2cur;   // M: spline second derivatives of xcur
    double* w;       // M: K of the last basis vector
    double* z;       // M: the residual
    double* part;    // gm_part_size(m, gc, gc64): per-chunk partial dots and norms
    double* y;       // m + 1: solution of the cycle's triangular system
    GmresState* st;  // state machine; also holds tol and max_iter so launches are call independent
    GmresPub* pub;   // what the host sees of the run (may be null)
    int m;
    int gc;          // chunks of the step launch (gm_chunks)
    int gc64;        // workgroups of the reduce launch: chunks of 64 samples (3D: of 64 reduce3_chunks(M))
};


// Vectors of a Richardson or BiCGSTAB run (M doubles each).  The apply reads q
// (BiCGSTAB) or x (Richardson) and writes w.
struct IterBufs {
    double *b, *x, *r, *rhat, *p, *v, *s, *q, *w, *s2;
    IterState* st;
    GmresPub* pub;
    int M;
};

constexpr int kIterRich = 0, kIterBicgInit = 1, kIterBicgHalf = 2, kIterBicgFull = 3, kIterTrueRes = 4;

// The start of a run: b <- rhs, x <- the initial guess, the state.
hipError_t launch_iter_start(const IterBufs& B, const double* rhs, const double* x, const IterState& st, hipStream_t s);
// One single-workgroup step of the iterations (krylov.hip): which = kIter*.
hipError_t launch_iter_step(int which, const IterBufs& B, hipStream_t s);

// launchers (return hipError_t of the launch)
hipError_t launch_correct(const DevPlan& p, JumpSrc js, double* corr, double* corr_il, double* dense,
                          const int* skip, hipStream_t s);
// R modes per workgroup (a power of two <= kMaxModesPerGroup whose LDS fits);
// ceil((N-1) / R) workgroups, each writing one row of M partial sums
hipError_t launch_modes(const DevPlan& p, const double* corr, double* partial, int R,
                        const int* skip, hipStream_t s);
// A check of a density for NaN or Inf: flag (0 before the launch) is set and number
// stored to *bad (host memory the device can write) when there is one; flag_next, the
// flag of the next call, is cleared.
struct DensityCheck {
    int* flag;
    int* flag_next;
    unsigned* bad;
    unsigned number;
};
// What an apply needs of a density y before the sparse solve (gm_density in
// gmres.h): its spline second derivatives and its corrections in the sparse-sum
// layout; with check (may be null) also the check.
hipError_t launch_density(const DevPlan& p, const double* y, double* s2, double* corr_il, const int* skip,
                          const DensityCheck* check, hipStream_t s);
// The same for an interface solve (no check): the density y and f on Gamma (either
// null: zero), their spline second derivatives into s2 and f2.
hipError_t launch_density_f(const DevPlan& p, const double* y, const double* f, double* s2, double* f2, double* corr_il,
                            hipStream_t s);
// The row solves of an interface solve (k_modes_dense): rows, the transformed
// right-hand side on the whole grid (added to the corrections' sums when `load`),
// becomes the transformed solution when `store`; with partial (may be null) the
// samples' partial sums as launch_modes, with w2 also those with the weights w2.
hipError_t launch_modes_dense(const DevPlan& p, const double* corr, double* rows, bool load, bool store, int R,
                              double* partial, const double* w2, double* partial2, hipStream_t s);
hipError_t launch_spline(const DevPlan& p, const double* y, double* s2, const int* skip, hipStream_t s);
// with gm non-null (a GMRES step) the output goes to gm->w, the launch is skipped
// once GMRES is done, and it also makes its part of the GMRES step (gmres.h); with
// `from` (gm null) out = from - the result
hipError_t launch_reduce_interp(const DevPlan& p, JumpSrc js, const double* partial, int G, double* out,
                                const int* skip, const GmresBufs* gm, hipStream_t s, const double* from = nullptr);
// v+ (or d_n v+) at the samples from a grid solution V in the padded layout, or (user)
// on the caller's grid
hipError_t launch_interp_grid(const DevPlan& p, JumpSrc js, const double* V, bool user, double* out, hipStream_t s);
hipError_t launch_fill_rhs(const DevPlan& p, const double* f, bool mask, double* R, hipStream_t s);
// column sine transforms (dst.hip)
// B: columns per workgroup (4, 8 or 16; 32 or 64 with FP64 pairs; see dst_tile_ok)
// FP64 (alpha = 1) reading the user's grid f, zero outside Omega with mask, into the
// padded layout; and from there writing the user's grid u (the box's rows and columns
// zero), zero outside Omega with mask.
hipError_t launch_dst_from_grid(const DevPlan& p, const double* f, bool mask, double* out, int B, hipStream_t s);
hipError_t launch_dst_to_grid(const DevPlan& p, const double* in, double* u, double alpha, bool mask, int B,
                              hipStream_t s);
// whether the two above read B (up to 512 rows they do not)
bool dst_grid_tiled(int N);
// FP32 arithmetic reading an FP64 grid into FP32 storage, or FP32 storage into an FP64
// grid (written, or added to add, padded as well)
hipError_t launch_dst_cols_f32(const DevPlan& p, const double* in, float* out, double alpha, int B, hipStream_t s);
hipError_t launch_dst_cols_f32_to64(const DevPlan& p, const float* in, double* out, double alpha, const double* add,
                                    int B, hipStream_t s);
// The FP32 transform of the FP64 residual r - (L_h - kappa) v, r in the padded layout or
// (user) the user's grid.
hipError_t launch_dst_residual_f32(const DevPlan& p, const double* r, bool user, const double* v, float* out, int B,
                                   hipStream_t s);
// The FP32 transforms reading the user's grid f, and writing the user's grid u.
hipError_t launch_dst_from_grid_f32(const DevPlan& p, const double* f, float* out, int B, hipStream_t s);
hipError_t launch_dst_f32_to_grid(const DevPlan& p, const float* in, double* u, double alpha, const double* add, int B,
                                  hipStream_t s);
// In-place FP64 transforms of `slices` N-row arrays (rows ld elements apart,
// ld columns, arrays `slice` elements apart): the column transforms of the
// planes of a 3D grid.  Skipped while *skip is nonzero (skip may be null).
hipError_t launch_dst_lines(int N, int log2N, const double* sinq, double* a, double alpha, int B, int ld, int slices,
                            size_t slice, const int* skip, hipStream_t s);
// LDS of a column-transform workgroup with B columns whose complex pairs take
// cpx_bytes each; whether B is a valid tile for N within lds_max.
size_t dst_lds_bytes(int N, int B, size_t cpx_bytes);
bool dst_tile_ok(int N, int B, size_t cpx_bytes, size_t lds_max);
// The default tile: the widest valid one that splits `lines` columns into at
// least min_groups workgroups, else the narrowest valid one (0 if none).
int dst_default_tile(int N, size_t cpx_bytes, size_t lds_max, long lines, int min_groups);
// tridiagonal solves along x of every sine mode (FP64 arithmetic; FP64 or FP32 storage)
hipError_t launch_rows_solve(const DevPlan& p, double* A, hipStream_t s);
hipError_t launch_rows_solve_f32(const DevPlan& p, float* A, hipStream_t s);
hipError_t launch_grid_out(const DevPlan& p, const double* V, bool mask, double* u, hipStream_t s);
hipError_t launch_axpby(int n, double a, const double* x, double b, const double* y, double* z,
                        hipStream_t s);
// x[0..n) <- v (a kernel, so it may sit in a graph where a memset node may not)
hipError_t launch_fill(size_t n, double v, double* x, hipStream_t s);
// *flag = 1 if x[0..n) holds a NaN or Inf, else 0 (one workgroup; n up to a few 10^4)
hipError_t launch_nonfinite(int n, const double* x, int* flag, hipStream_t s);
// The start of a GMRES run (gm_begin in gmres.h), one launch: the state and
// the first K input (its spline second derivatives with taps; with p and
// corr_il also its corrections, in the sparse-sum layout).  rhs may be null
// (ghat already in place); phi_in may be null (a zero guess); xout (may be
// null) receives the iterate from the step launch that ends the run; epoch: the run's
// number (not 0, another for each run).
hipError_t launch_gmres_start(const DevPlan* p, const double* taps, int M, GmresBufs b, const double* rhs,
                              const double* phi_in, double tol, int max_iter, double reorth, double* xout,
                              double* corr_il, unsigned epoch, hipStream_t s);
// The step launch (gmres.h).  taps: the spline filter of the density (null: no
// spline, the surface problem)
hipError_t launch_gmres_step(const double* taps, int M, GmresBufs b, hipStream_t s);
// default of GmresState::reorth (see gmres.h)
constexpr double kGmReorthDefault = 1e-3;
// the same with the next apply's corrections made in the launch
// (into corr_il, the sparse-sum layout)
hipError_t launch_gmres_step_corr(const DevPlan& p, GmresBufs b, double* corr_il, hipStream_t s);

size_t modes_lds_bytes(int N, int R);

}  // namespace kfbi
