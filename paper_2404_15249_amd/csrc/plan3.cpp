// Host-side plan of the three-dimensional problem (see plan3.h for the readings).
#include "plan3.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <unordered_map>

namespace kfbi {

namespace {

[[noreturn]] void fail3(const char* msg) { throw GeometryError{msg}; }

// Solves the dense n x n system A X = B (B: n x r, row-major, overwritten by X)
// by Gaussian elimination with partial pivoting.  A is overwritten.
void solve_dense(std::vector<double>& A, std::vector<double>& B, int n, int r) {
    for (int c = 0; c < n; ++c) {
        int piv = c;
        for (int i = c + 1; i < n; ++i)
            if (std::fabs(A[i * n + c]) > std::fabs(A[piv * n + c])) piv = i;
        if (A[piv * n + c] == 0.0) fail3("singular local fit (degenerate control points)");
        if (piv != c) {
            for (int k = 0; k < n; ++k) std::swap(A[c * n + k], A[piv * n + k]);
            for (int k = 0; k < r; ++k) std::swap(B[c * r + k], B[piv * r + k]);
        }
        for (int i = c + 1; i < n; ++i) {
            const double f = A[i * n + c] / A[c * n + c];
            if (f == 0.0) continue;
            for (int k = c; k < n; ++k) A[i * n + k] -= f * A[c * n + k];
            for (int k = 0; k < r; ++k) B[i * r + k] -= f * B[c * r + k];
        }
    }
    for (int c = n - 1; c >= 0; --c) {
        for (int k = 0; k < r; ++k) {
            double s = B[c * r + k];
            for (int j = c + 1; j < n; ++j) s -= A[c * n + j] * B[j * r + k];
            B[c * r + k] = s / A[c * n + c];
        }
    }
}

}  // namespace

Plan3Host build_plan3(int N, double lo, double hi, const double axes_in[3]) {
    if (N < 64 || (N & (N - 1)) != 0) fail3("3D grids need a power of two >= 64 intervals per axis");
    Plan3Host P;
    P.N = N;
    P.lo = lo;
    P.hi = hi;
    P.h = (hi - lo) / N;
    for (int a = 0; a < 3; ++a) {
        if (!(axes_in[a] > 0.0)) fail3("ellipsoid semi-axes must be positive");
        P.axes[a] = axes_in[a];
    }
    const double h = P.h;
    const double a2 = P.axes[0] * P.axes[0], b2 = P.axes[1] * P.axes[1], c2 = P.axes[2] * P.axes[2];
    const int S = N + 1;
    std::vector<double> c(S);
    for (int k = 0; k < S; ++k) c[k] = lo + (double)k * h;
    auto lin = [S](int i, int j, int k) { return ((size_t)k * S + j) * S + i; };
    P.inside.assign((size_t)S * S * S, 0);
    // each coordinate's term once (three divisions a node took a tenth of the plan)
    std::vector<double> tx(S), ty(S), tz(S);
    for (int k = 0; k < S; ++k) {
        tx[k] = c[k] * c[k] / a2;
        ty[k] = c[k] * c[k] / b2;
        tz[k] = c[k] * c[k] / c2;
    }
    for (int k = 0; k < S; ++k)
        for (int j = 0; j < S; ++j)
            for (int i = 0; i < S; ++i) P.inside[lin(i, j, k)] = tx[i] + ty[j] + tz[k] - 1.0 < 0.0 ? 1 : 0;
    // whether a grid line along axis a has a node inside: line[a][t_hi * S + t_lo] (below)
    std::vector<unsigned char> line[3];
    for (auto& l : line) l.assign((size_t)S * S, 0);
    for (int k = 0; k < S; ++k)
        for (int j = 0; j < S; ++j) {
            unsigned char any = 0;
            for (int i = 0; i < S; ++i) {
                const unsigned char in = P.inside[lin(i, j, k)];
                any |= in;
                line[1][(size_t)k * S + i] |= in;
                line[2][(size_t)j * S + i] |= in;
            }
            line[0][(size_t)k * S + j] = any;
        }
    for (int k = 0; k < S; ++k)
        for (int j = 0; j < S; ++j)
            for (int i = 0; line[0][(size_t)k * S + j] && i < S; ++i)
                if (P.inside[lin(i, j, k)] && (i < 2 || j < 2 || k < 2 || i > N - 2 || j > N - 2 || k > N - 2))
                    fail3("the ellipsoid must keep two grid cells away from the box");

    // crossings
    std::unordered_map<long long, int> q_of_edge;   // (axis, lower node) -> crossing
    auto edge_key = [&](int ax, size_t node) { return (long long)node * 3 + ax; };
    for (int ax = 0; ax < 3; ++ax) {
        const int o0 = ax == 0 ? 1 : 0, o1 = ax == 2 ? 1 : 2;
        const double A = P.axes[ax];
        for (int t_hi = 0; t_hi < S; ++t_hi)
            for (int t_lo = 0; t_lo < S; ++t_lo)
                for (int s = 0; line[ax][(size_t)t_hi * S + t_lo] && s < N; ++s) {
                    int ia[3], ib[3];
                    ia[ax] = s;
                    ia[o0] = t_lo;
                    ia[o1] = t_hi;
                    ib[0] = ia[0];
                    ib[1] = ia[1];
                    ib[2] = ia[2];
                    ib[ax] = s + 1;
                    const size_t na = lin(ia[0], ia[1], ia[2]), nb = lin(ib[0], ib[1], ib[2]);
                    if (P.inside[na] == P.inside[nb]) continue;
                    const double p0 = c[t_lo] / P.axes[o0];
                    const double p1 = c[t_hi] / P.axes[o1];
                    const double rest = 1.0 - p0 * p0 - p1 * p1;
                    const double root = A * std::sqrt(std::max(rest, 0.0));
                    const double sa = c[s], sb = c[s + 1];
                    double xi = sa + sb > 0.0 ? root : -root;
                    xi = std::min(std::max(xi, sa), sb);
                    double pos[3];
                    pos[ax] = xi;
                    pos[o0] = c[t_lo];
                    pos[o1] = c[t_hi];
                    q_of_edge[edge_key(ax, na)] = P.M();
                    P.pos.insert(P.pos.end(), pos, pos + 3);
                    P.axis.push_back(ax);
                }
    }
    const int M = P.M();
    if (M < kFitMin + 1) fail3("too few crossings for the surface fits");

    // local frames: outward normal, tangent basis, second fundamental form
    P.geo.resize((size_t)12 * M);
    const double hess[3] = {2.0 / a2, 2.0 / b2, 2.0 / c2};
    for (int m = 0; m < M; ++m) {
        const double* p = &P.pos[3 * m];
        const double g[3] = {2.0 * p[0] / a2, 2.0 * p[1] / b2, 2.0 * p[2] / c2};
        const double gn = std::sqrt(g[0] * g[0] + g[1] * g[1] + g[2] * g[2]);
        const double n[3] = {g[0] / gn, g[1] / gn, g[2] / gn};
        int amin = 0;
        for (int a = 1; a < 3; ++a)
            if (std::fabs(n[a]) < std::fabs(n[amin])) amin = a;
        double e[3] = {0, 0, 0};
        e[amin] = 1.0;
        double t1[3] = {e[1] * n[2] - e[2] * n[1], e[2] * n[0] - e[0] * n[2], e[0] * n[1] - e[1] * n[0]};
        const double t1n = std::sqrt(t1[0] * t1[0] + t1[1] * t1[1] + t1[2] * t1[2]);
        for (double& v : t1) v /= t1n;
        const double t2[3] = {n[1] * t1[2] - n[2] * t1[1], n[2] * t1[0] - n[0] * t1[2], n[0] * t1[1] - n[1] * t1[0]};
        double s11 = 0, s12 = 0, s22 = 0;
        for (int a = 0; a < 3; ++a) {
            s11 += t1[a] * hess[a] * t1[a];
            s12 += t1[a] * hess[a] * t2[a];
            s22 += t2[a] * hess[a] * t2[a];
        }
        double* G = &P.geo[(size_t)12 * m];
        for (int a = 0; a < 3; ++a) {
            G[a] = n[a];
            G[3 + a] = t1[a];
            G[6 + a] = t2[a];
        }
        G[9] = s11 / gn;
        G[10] = s12 / gn;
        G[11] = s22 / gn;
    }

    // weighted least-squares surface fits; neighbours found through cells of
    // size 2.5 h (a point's neighbours lie in its cell and the 26 around it)
    const double rad = 0.5 * kFitRadiusNum * h;
    const int nc = (int)std::ceil((hi - lo) / rad) + 1;
    auto cell_of = [&](const double* p, int a) { return (int)std::floor((p[a] - lo) / rad); };
    auto cell_key = [&](int x, int y, int z) { return ((size_t)z * nc + y) * nc + x; };
    auto cell_at = [&](int m) {
        return cell_key(cell_of(&P.pos[3 * m], 0), cell_of(&P.pos[3 * m], 1), cell_of(&P.pos[3 * m], 2));
    };
    // cell c's points, in order: cells[cell_first[c]] up to cells[cell_first[c + 1]]
    // (counted into place: a hash map's 27 look-ups a point took a twelfth of the plan)
    std::vector<int> cell_first((size_t)nc * nc * nc + 2, 0), cells(M);
    for (int m = 0; m < M; ++m) cell_first[cell_at(m) + 2] += 1;
    for (size_t k = 2; k < cell_first.size(); ++k) cell_first[k] += cell_first[k - 1];
    for (int m = 0; m < M; ++m) cells[cell_first[cell_at(m) + 1]++] = m;
    P.fit_off.assign(1, 0);
    std::vector<int> near;
    std::vector<double> A, wts, B;
    for (int m = 0; m < M; ++m) {
        const double* pm = &P.pos[3 * m];
        auto dist_to = [&](int k) {
            const double dx = P.pos[3 * k] - pm[0], dy = P.pos[3 * k + 1] - pm[1], dz = P.pos[3 * k + 2] - pm[2];
            return std::sqrt(dx * dx + dy * dy + dz * dz);
        };
        near.clear();
        const int cx = cell_of(pm, 0), cy = cell_of(pm, 1), cz = cell_of(pm, 2);
        for (int z = cz - 1; z <= cz + 1; ++z)
            for (int y = cy - 1; y <= cy + 1; ++y)
                for (int x = cx - 1; x <= cx + 1; ++x) {
                    if (std::min({x, y, z}) < 0 || std::max({x, y, z}) >= nc) continue;
                    const size_t cell = cell_key(x, y, z);
                    for (int at = cell_first[cell]; at < cell_first[cell + 1]; ++at)
                        if (cells[at] != m && dist_to(cells[at]) <= rad) near.push_back(cells[at]);
                }
        if ((int)near.size() < kFitMin) {           // the nearest kFitMin, ties by index
            std::vector<int> all;
            for (int k = 0; k < M; ++k)
                if (k != m) all.push_back(k);
            std::stable_sort(all.begin(), all.end(), [&](int a, int b) { return dist_to(a) < dist_to(b); });
            near.assign(all.begin(), all.begin() + kFitMin);
        }
        std::sort(near.begin(), near.end());
        const int K = (int)near.size();
        const double* G = &P.geo[(size_t)12 * m];
        A.resize((size_t)K * 5);
        wts.resize(K);
        B.resize((size_t)5 * K);
        for (int e = 0; e < K; ++e) {
            const int k = near[e];
            const double rel[3] = {P.pos[3 * k] - pm[0], P.pos[3 * k + 1] - pm[1], P.pos[3 * k + 2] - pm[2]};
            const double u = (rel[0] * G[3] + rel[1] * G[4] + rel[2] * G[5]) / h;
            const double v = (rel[0] * G[6] + rel[1] * G[7] + rel[2] * G[8]) / h;
            const double row[5] = {u, v, 0.5 * u * u, u * v, 0.5 * v * v};
            for (int q = 0; q < 5; ++q) A[(size_t)e * 5 + q] = row[q];
            const double d = dist_to(k) / h;
            wts[e] = 1.0 / (1.0 + d * d);
        }
        std::vector<double> Gm(25, 0.0);
        for (int a = 0; a < 5; ++a) {
            for (int b = 0; b < 5; ++b) {
                double s = 0.0;
                for (int e = 0; e < K; ++e) s += A[(size_t)e * 5 + a] * wts[e] * A[(size_t)e * 5 + b];
                Gm[a * 5 + b] = s;
            }
            for (int e = 0; e < K; ++e) B[(size_t)a * K + e] = A[(size_t)e * 5 + a] * wts[e];
        }
        solve_dense(Gm, B, 5, K);
        const double scale[5] = {1.0 / h, 1.0 / h, 1.0 / (h * h), 1.0 / (h * h), 1.0 / (h * h)};
        for (int e = 0; e < K; ++e) {
            P.fit_idx.push_back(near[e]);
            for (int a = 0; a < 5; ++a) P.fit_w.push_back(B[(size_t)a * K + e] * scale[a]);
        }
        P.fit_off.push_back((int)P.fit_idx.size());
    }

    // irregular nodes and their arms, in (k, j, i) order
    P.arm_off.assign(1, 0);
    for (int k = 1; k < N; ++k)
        for (int j = 1; j < N; ++j)
            for (int i = 1; i < N; ++i) {
                const unsigned char* at = &P.inside[lin(i, j, k)];
                const unsigned char here = *at;
                const size_t sy = S, sz = (size_t)S * S;
                if (*(at - 1) + at[1] + *(at - sy) + at[sy] + *(at - sz) + at[sz] == 6 * here) continue;   // no arm
                const int before = (int)P.arm_q.size();
                for (int ax = 0; ax < 3; ++ax)
                    for (int step = -1; step <= 1; step += 2) {
                        int nb[3] = {i, j, k};
                        nb[ax] += step;
                        if (P.inside[lin(nb[0], nb[1], nb[2])] == here) continue;
                        const int* low = step > 0 ? nullptr : nb;
                        const int ijk[3] = {i, j, k};
                        if (!low) low = ijk;
                        const auto it = q_of_edge.find(edge_key(ax, lin(low[0], low[1], low[2])));
                        if (it == q_of_edge.end()) fail3("internal: an arm without its crossing");
                        P.arm_q.push_back(it->second);
                        P.arm_d.push_back(c[nb[ax]] - P.pos[3 * it->second + ax]);
                    }
                if ((int)P.arm_q.size() > before) {
                    P.irr_node.push_back((k - 1) * N * N + (j - 1) * N + (i - 1));
                    P.irr_sign.push_back(here ? 1.0 : -1.0);
                    P.arm_off.push_back((int)P.arm_q.size());
                }
            }

    // interpolation stencils, weights and far-side jump coefficients
    static const int offs[kStencil3][3] = {{0, 0, 0}, {1, 0, 0}, {-1, 0, 0}, {0, 1, 0}, {0, -1, 0},
                                           {0, 0, 1}, {0, 0, -1}, {1, 1, 0}, {1, 0, 1}, {0, 1, 1}};
    P.st_node.resize((size_t)kStencil3 * M);
    P.st_w.resize((size_t)kStencil3 * M);
    P.st_t.assign((size_t)kStencil3 * M, 0.0);
    for (int m = 0; m < M; ++m) {
        const double* z = &P.pos[3 * m];
        int i0[3], sg[3];
        for (int a = 0; a < 3; ++a) {
            i0[a] = (int)std::floor((z[a] - lo) / h + 0.5);
            sg[a] = z[a] >= lo + i0[a] * h ? 1 : -1;
        }
        std::vector<double> A(kStencil3 * kStencil3), e0(kStencil3, 0.0);
        double D[kStencil3][3];
        bool out[kStencil3];
        for (int s = 0; s < kStencil3; ++s) {
            int ijk[3];
            for (int a = 0; a < 3; ++a) {
                const int o = s < 7 ? offs[s][a] : offs[s][a] * sg[a];
                ijk[a] = i0[a] + o;
                if (ijk[a] < 0 || ijk[a] > N) fail3("an interpolation stencil leaves the grid");
            }
            const bool box = ijk[0] == 0 || ijk[1] == 0 || ijk[2] == 0 || ijk[0] == N || ijk[1] == N || ijk[2] == N;
            P.st_node[(size_t)kStencil3 * m + s] =
                box ? -1 : (ijk[2] - 1) * N * N + (ijk[1] - 1) * N + (ijk[0] - 1);
            out[s] = !P.inside[lin(ijk[0], ijk[1], ijk[2])];
            for (int a = 0; a < 3; ++a) D[s][a] = lo + ijk[a] * h - z[a];
            const double x = D[s][0] / h, y = D[s][1] / h, w = D[s][2] / h;
            const double row[kStencil3] = {1.0, x, y, w, x * x, y * y, w * w, x * y, x * w, y * w};
            // A^T: column s holds the basis at node s
            for (int q = 0; q < kStencil3; ++q) A[q * kStencil3 + s] = row[q];
        }
        e0[0] = 1.0;
        solve_dense(A, e0, kStencil3, 1);
        for (int s = 0; s < kStencil3; ++s) {
            const double wt = e0[s];
            P.st_w[(size_t)kStencil3 * m + s] = wt;
            if (!out[s]) continue;
            const double dx = D[s][0], dy = D[s][1], dz = D[s][2];
            const double t[kJump3] = {1.0, dx, dy, dz, 0.5 * dx * dx, 0.5 * dy * dy, 0.5 * dz * dz,
                                      dx * dy, dx * dz, dy * dz};
            for (int q = 0; q < kJump3; ++q) P.st_t[(size_t)kJump3 * m + q] += wt * t[q];
        }
    }
    return P;
}

Apply3Host build_apply3(const Plan3Host& P) {
    Apply3Host A;
    const int M = P.M(), N = P.N, H = N / 2;
    const size_t E = P.fit_idx.size();
    A.fit.resize(3 * E);
    A.point.resize(3 * (size_t)M);
    A.st_node.resize((size_t)kStencil3 * M);
    A.st_w.resize((size_t)kStencil3 * M);
    for (int m = 0; m < M; ++m) {
        const double *g = &P.geo[12 * (size_t)m], *n = g, *t1 = g + 3, *t2 = g + 6;
        const double s11 = g[9], s12 = g[10], s22 = g[11];
        const double* t = &P.st_t[(size_t)kJump3 * m];
        // the jump [v_ij] in the tangent derivatives d0..d4 of the fit and in
        // [v_nn] + d2 + d4 (which is [F] + kappa [v])
        struct Lin {
            double d[5], nn;
        };
        auto hess = [&](int i, int j) {
            const double a = t1[i] * n[j] + n[i] * t1[j], b = t2[i] * n[j] + n[i] * t2[j];
            return Lin{{-(s11 * a + s12 * b), -(s12 * a + s22 * b), t1[i] * t1[j] - n[i] * n[j],
                        t1[i] * t2[j] + t2[i] * t1[j], t2[i] * t2[j] - n[i] * n[j]},
                       n[i] * n[j]};
        };
        const int ax = P.axis[m];
        const Lin grad{{t1[ax], t2[ax], 0.0, 0.0, 0.0}, 0.0}, second = hess(ax, ax);
        Lin far{{0.0, 0.0, 0.0, 0.0, 0.0}, 0.0};
        for (int c = 0; c < 3; ++c) {
            far.d[0] += t[1 + c] * t1[c];
            far.d[1] += t[1 + c] * t2[c];
        }
        static const int ij[6][2] = {{0, 0}, {1, 1}, {2, 2}, {0, 1}, {0, 2}, {1, 2}};
        for (int c = 0; c < 6; ++c) {
            const Lin h = hess(ij[c][0], ij[c][1]);
            for (int q = 0; q < 5; ++q) far.d[q] += t[4 + c] * h.d[q];
            far.nn += t[4 + c] * h.nn;
        }
        A.point[m] = second.nn;
        A.point[(size_t)M + m] = far.nn;
        A.point[(size_t)2 * M + m] = t[0];
        for (int e = P.fit_off[m]; e < P.fit_off[m + 1]; ++e) {
            const double* w = &P.fit_w[5 * (size_t)e];
            const Lin* of[3] = {&grad, &second, &far};
            for (int k = 0; k < 3; ++k) {
                double v = 0.0;
                for (int q = 0; q < 5; ++q) v += of[k]->d[q] * w[q];
                A.fit[k * E + e] = v;
            }
        }
        for (int s = 0; s < kStencil3; ++s) {
            A.st_node[(size_t)s * M + m] = P.st_node[(size_t)kStencil3 * m + s];
            A.st_w[(size_t)s * M + m] = P.st_w[(size_t)kStencil3 * m + s];
        }
    }
    if (N > kSlabMax) return A;
    // a node's folded column (y' - 1) N + x - 1, its z and its side
    struct Fold {
        int col, z, side;
    };
    auto fold = [&](int node) {
        const int x = node % N, y = node / N % N + 1, z = node / (N * N) + 1, side = y > H;
        return Fold{((side ? N - y : y) - 1) * N + x, z, side};
    };
    // the pieces' heights of every folded column
    std::vector<std::vector<int>> column((size_t)H * N);
    for (int node : P.irr_node) {
        const Fold f = fold(node);
        column[f.col].push_back(std::min(f.z, N - f.z));
    }
    std::vector<int> order;
    for (int c = 0; c < H * N; ++c) {
        auto& z = column[c];
        std::sort(z.begin(), z.end());
        z.erase(std::unique(z.begin(), z.end()), z.end());
        if (!z.empty()) order.push_back(c);
    }
    A.y_first = order.empty() ? 0 : order[0] / N;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return column[a].size() > column[b].size(); });
    // groups of 64 columns, longest first, each to the wavefront with the fewest rows yet
    const int waves = N / 8;
    std::vector<std::vector<size_t>> of(waves);
    std::vector<size_t> rows(waves, 0);
    for (size_t g = 0; g < order.size(); g += 64) {
        const size_t w = std::min_element(rows.begin(), rows.end()) - rows.begin();
        of[w].push_back(g);
        rows[w] += column[order[g]].size();
    }
    std::vector<size_t> first((size_t)H * N, 0);             // a column's first piece
    A.sp_wave.assign(1, 0);
    for (int w = 0; w < waves; ++w) {
        for (size_t g : of[w]) {
            const size_t at = A.sp_piece.size();
            A.sp_piece.resize(at + 64 * column[order[g]].size(), -1);
            for (size_t lane = 0; lane < 64 && g + lane < order.size(); ++lane) {
                const int c = order[g + lane];
                first[c] = at + lane;
                for (size_t t = 0; t < column[c].size(); ++t)
                    A.sp_piece[at + 64 * t + lane] = c % N | (c / N) << 8 | column[c][t] << 16;
            }
        }
        A.sp_wave.push_back((int)(A.sp_piece.size() / 64));
    }
    A.irr_pos.resize(P.I());
    for (int r = 0; r < P.I(); ++r) {
        const Fold f = fold(P.irr_node[r]);
        const auto& z = column[f.col];
        const size_t t = std::lower_bound(z.begin(), z.end(), std::min(f.z, N - f.z)) - z.begin();
        A.irr_pos[r] = (int)(4 * (first[f.col] + 64 * t)) + 2 * f.side + (f.z > H);
    }
    // the stencils' nodes by tile: place[column, side, z'] is first a mark, then the place
    // of the node at z' in the entries
    const size_t per = H + 1;
    std::vector<int> place((size_t)H * N * 2 * per, -1);
    auto at = [&](const Fold& f) { return ((size_t)f.col * 2 + f.side) * per + std::min(f.z, N - f.z); };
    for (int node : A.st_node)
        if (node >= 0) {
            const Fold f = fold(node);
            place[at(f)] = 0;
            A.y_first = std::min(A.y_first, f.col / N);
        }
    A.zg_off.assign(1, 0);
    for (int t = 0; t < H * (N / 32); ++t) {
        for (int x = 0; x < 32; ++x)
            for (int side = 0; side < 2; ++side) {
                const int col = t / (N / 32) * N + t % (N / 32) * 32 + x;
                int* p = &place[((size_t)col * 2 + side) * per];
                int waiting = 0;                             // a height without a second one yet
                for (int z = 1; z <= H; ++z) {
                    if (p[z] < 0) continue;
                    if (waiting) {
                        A.zg_code.back() = waiting | z << 8 | x << 16 | side << 24;
                        p[z] = 4 * (int)A.zg_code.size() - 2;
                        waiting = 0;
                    } else {
                        A.zg_code.push_back(z | z << 8 | x << 16 | side << 24);
                        p[z] = 4 * (int)A.zg_code.size() - 4;
                        waiting = z;
                    }
                }
            }
        A.zg_off.push_back((int)A.zg_code.size());
    }
    A.st_pos.resize(A.st_node.size());
    for (size_t k = 0; k < A.st_node.size(); ++k) {
        A.st_pos[k] = -1;
        if (A.st_node[k] < 0) continue;
        const Fold f = fold(A.st_node[k]);
        A.st_pos[k] = place[at(f)] + (f.z > H);
    }
    return A;
}

}  // namespace kfbi
