// Affine fields in 2D: the host's map of a whole step, the foot's split, the
// gather from staged nodes, and the update, shared by the single step and by
// the several-steps-a-launch kernel.
#pragma once

#include <type_traits>

#include "hermite.h"

namespace gals {

template <typename T>
struct AffineMap {
    double Mc[9], kc[3];  // foot in cell units: s_a = kc_a + sum_b Mc[a][b] idx_b
    double Md[9];         // Mc - I: the displacement in cells s_a - idx_a = kc_a + sum_b Md[a][b] idx_b
    T J[9];               // Jacobian of the foot map (J form), uniform
    T An[9], Af[9];       // Heun: grad v at the node (t + dt) and at the foot (t)
};

template <typename T>
inline AffineMap<T> make_affine_map(const gals_ctx *ctx, double dt, double c1, double c2,
                                    double c3)
{
    const int D = ctx->dim;
    const Vel<double> &p = ctx->vd;
    double A[9] = {0}, b[3] = {0}, xc[3] = {0};
    for (int i = 0; i < D; i++) {
        b[i] = p.b[i];
        xc[i] = p.c[i];
        for (int j = 0; j < D; j++) A[i * 3 + j] = p.A[i * 3 + j];
    }
    auto mm = [&](const double *X, const double *Y, double *Z) {  // Z = X Y (3x3)
        double t[9];
        for (int i = 0; i < 3; i++)
            for (int j = 0; j < 3; j++) {
                double acc = 0.0;
                for (int k = 0; k < 3; k++) acc += X[i * 3 + k] * Y[k * 3 + j];
                t[i * 3 + j] = acc;
            }
        for (int k = 0; k < 9; k++) Z[k] = t[k];
    };
    auto mv = [&](const double *X, const double *y, double *z) {
        double t[3];
        for (int i = 0; i < 3; i++) t[i] = X[i * 3] * y[0] + X[i * 3 + 1] * y[1] + X[i * 3 + 2] * y[2];
        for (int i = 0; i < 3; i++) z[i] = t[i];
    };
    double V0[9], V1[9], V2[9], P[9], w0[3], w1[3], w2[3], q[3];
    for (int k = 0; k < 9; k++) V0[k] = c1 * A[k];
    for (int i = 0; i < 3; i++) w0[i] = c1 * b[i];
    for (int k = 0; k < 9; k++) P[k] = double(k % 4 == 0) - dt * V0[k];  // I - dt V0
    mm(A, P, V1);
    for (int k = 0; k < 9; k++) V1[k] *= c2;
    mv(A, w0, q);
    for (int i = 0; i < 3; i++) w1[i] = c2 * (b[i] - dt * q[i]);
    for (int k = 0; k < 9; k++) P[k] = double(k % 4 == 0) - dt * 0.25 * (V0[k] + V1[k]);
    mm(A, P, V2);
    for (int k = 0; k < 9; k++) V2[k] *= c3;
    double s01[3];
    for (int i = 0; i < 3; i++) s01[i] = w0[i] + w1[i];
    mv(A, s01, q);
    for (int i = 0; i < 3; i++) w2[i] = c3 * (b[i] - dt * 0.25 * q[i]);
    double M[9], m[3];
    for (int k = 0; k < 9; k++)
        M[k] = double(k % 4 == 0) - dt * (V0[k] * (1.0 / 6.0) + V1[k] * (1.0 / 6.0) + V2[k] * (2.0 / 3.0));
    for (int i = 0; i < 3; i++)
        m[i] = -dt * (w0[i] * (1.0 / 6.0) + w1[i] * (1.0 / 6.0) + w2[i] * (2.0 / 3.0));
    // cell units: s_a = (foot_a - lo_a) / h_a with node x_b = lo_b + idx_b h_b
    AffineMap<T> am;
    for (int a = 0; a < 3; a++) {
        am.kc[a] = 0.0;
        for (int j = 0; j < 3; j++) am.Mc[a * 3 + j] = 0.0;
    }
    const Geom &g = ctx->g;
    for (int a = 0; a < D; a++) {
        double k = (xc[a] - g.lo[a]) + m[a];
        for (int j = 0; j < D; j++) {
            am.Mc[a * 3 + j] = M[a * 3 + j] * g.h[j] / g.h[a];
            k += M[a * 3 + j] * (g.lo[j] - xc[j]);
        }
        am.kc[a] = k / g.h[a];
    }
    for (int k = 0; k < 9; k++) am.Md[k] = am.Mc[k] - double(k % 4 == 0);
    for (int i = 0; i < D; i++)
        for (int j = 0; j < D; j++) {
            am.J[i * D + j] = T(M[i * 3 + j]);
            am.An[i * D + j] = T(c1 * A[i * 3 + j]);
            am.Af[i * D + j] = T(c2 * A[i * 3 + j]);
        }
    return am;
}

template <typename T>
__device__ __forceinline__ void split_cell_axis(const Geom &g, int a, double s, int &cell, T &xi,
                                                bool &outb)
{
    const bool below = s < g.lowc[a], above = s > g.outc[a];
    const double fl = fmin(fmax(floor(s), 0.0), g.lastc[a]);
    cell = int(fl);
    T x = T(s - fl);
    x = below ? T(0) : x;
    xi = above ? T(1) : x;
    outb = below || above;
}

// Boundary treatment and split of a foot given in cell units: outside only
// beyond kFootTol cells (then projected: local coordinate 0 or 1 and the
// normal derivative dropped), cell index clamped to [0, nc - 1], local
// coordinate unclamped otherwise (the same rules as project_foot + split).
template <typename T, int D>
__device__ __forceinline__ void split_cells(const Geom &g, const double *s, int *cell, T *xi,
                                            bool *outb)
{
#pragma unroll
    for (int a = 0; a < D; a++) split_cell_axis(g, a, s[a], cell[a], xi[a], outb[a]);
}

// The same for an FP32 state from the displacement in cells e = s - idx
// (FP64, rounded to FP32 here: one rounding, u |e|): with c = floor(e), a
// foot whose cell idx + c lies in [0, nc-1] (not outside, not clamped)
// splits into cell idx + c and local coordinate e - c, both exact in FP32.
// Only the other lanes take the FP64 treatment of split_cells (from
// s = idx + e), and a wave without such lanes skips it; each lane's result
// is the same either way.
template <typename T, int D>
__device__ __forceinline__ void split_disp(const Geom &g, const int *idx, const double *e64,
                                           int *cell, T *xi, bool *outb)
{
    static_assert(sizeof(T) == 4, "FP32 states only");
    float e[D], c[D];
    int cu[D];
    bool in = true;
#pragma unroll
    for (int a = 0; a < D; a++) {
        e[a] = float(e64[a]);
        c[a] = floor(e[a]);
        cu[a] = idx[a] + int(c[a]);
        in = in && unsigned(cu[a]) <= unsigned(g.nc[a] - 1);
    }
    if (__builtin_expect(__all(in), 1)) {
#pragma unroll
        for (int a = 0; a < D; a++) {
            cell[a] = cu[a];
            xi[a] = e[a] - c[a];
            outb[a] = false;
        }
        return;
    }
#pragma unroll
    for (int a = 0; a < D; a++) {
        const float fr = e[a] - c[a];
        if (unsigned(cu[a]) <= unsigned(g.nc[a] - 1)) {
            cell[a] = cu[a];
            xi[a] = fr;
            outb[a] = false;
        } else if (cu[a] == g.nc[a] && double(fr) <= g.outc[a] - g.ncd[a]) {
            // at most kFootTol past the last node: the last cell at local
            // coordinate 1 + fr (split_cells' rule, evaluated in FP32)
            cell[a] = g.nc[a] - 1;
            xi[a] = 1.0f + fr;
            outb[a] = false;
        } else {
            split_cell_axis(g, a, double(idx[a]) + e64[a], cell[a], xi[a], outb[a]);
        }
    }
}

// Cell data from staged nodes (node-interleaved: a node's phi, psi_x, psi_y
// side by side) with t0 and t1 at the node before the cell's lower-left and
// upper-left one (LDS offsets are not negative): every neighbour sits at a fixed
// offset from one of the two. The central
// cross derivative reads one column beyond each side of the cell; at the
// first and last cell of a row that column lies outside the grid, and the
// one-sided differences used there do not read it (same values as gather2d).
template <typename T, int MIX>
__device__ __forceinline__ void gather2d_lds(const Geom &g, const T *t0, const T *t1, int cx,
                                             T d[4][4])
{
    auto lo_ = [&](int k, int f) { return t0[3 * (k + 1) + f]; };
    auto up_ = [&](int k, int f) { return t1[3 * (k + 1) + f]; };
    d[0][0] = lo_(0, 0); d[1][0] = lo_(1, 0); d[2][0] = up_(0, 0); d[3][0] = up_(1, 0);
    d[0][1] = lo_(0, 1); d[1][1] = lo_(1, 1); d[2][1] = up_(0, 1); d[3][1] = up_(1, 1);
    if constexpr (MIX == GALS_MIXED_CENTRAL) {
        const T u0[4] = {lo_(-1, 2), lo_(0, 2), lo_(1, 2), lo_(2, 2)};
        const T u1[4] = {up_(-1, 2), up_(0, 2), up_(1, 2), up_(2, 2)};
        d[0][2] = u0[1]; d[1][2] = u0[2];
        d[2][2] = u1[1]; d[3][2] = u1[2];
        const T inv2h = geo_i2h<T>(g, 0);
        const bool lo = cx == 0, hi = cx + 1 == g.nc[0];
        diff_pair<T, sizeof(T) == 4>(u0, lo, hi, inv2h, d[0][3], d[1][3]);
        diff_pair<T, sizeof(T) == 4>(u1, lo, hi, inv2h, d[2][3], d[3][3]);
    } else {
        d[0][2] = lo_(0, 2); d[1][2] = lo_(1, 2); d[2][2] = up_(0, 2); d[3][2] = up_(1, 2);
        if constexpr (MIX == GALS_MIXED_CELL) {
            T ga[4], gb[4], out[4];
#pragma unroll
            for (int v = 0; v < 4; v++) {
                ga[v] = d[v][1];
                gb[v] = d[v][2];
            }
            cell_cross(ga, gb, geo_ih<T>(g, 0), geo_ih<T>(g, 1), out);
#pragma unroll
            for (int v = 0; v < 4; v++) d[v][3] = out[v];
        } else {
            d[0][3] = d[1][3] = d[2][3] = d[3][3] = T(0);
        }
    }
}

// Value and gradient of the bicubic of cell c from staged nodes (FOLD as in
// bicubic).
template <typename T, int MIX, bool FOLD>
__device__ __forceinline__ void bicubic_lds(const Geom &g, const T *t0, const T *t1, const int *c,
                                            const T *xi, T &H, T &Hx, T &Hy)
{
    if constexpr (FOLD) {
        const int xm = c[0] == 0 ? 3 : 0;  // the window starts at node 0 at the first cell
        bicubic_central<T>(
            g, c[0], xi,
            [&](int r) {
                const T *t = r ? t1 : t0;
                Row2d<T> q;
#pragma unroll
                for (int k = 0; k < 4; k++) q.gy[k] = t[3 * k + 2 + xm];
#pragma unroll
                for (int k = 0; k < 2; k++) {
                    q.phi[k] = t[3 * (k + 1)];
                    q.gx[k] = t[3 * (k + 1) + 1];
                }
                return q;
            },
            [&](int vx, int vy) { return (vy ? t1 : t0)[3 * (vx + 1)]; }, H, Hx, Hy);
    } else {
        T d[4][4];
        gather2d_lds<T, MIX>(g, t0, t1, c[0], d);
        Basis<T> bx, by;
        basis<T, false>(xi[0], geo_h<T>(g, 0), geo_ih<T>(g, 0), bx);
        basis<T, false>(xi[1], geo_h<T>(g, 1), geo_ih<T>(g, 1), by);
        hermite2d(d, bx, by, H, Hx, Hy);
    }
}

// The 2D part of an AffineMap (rows of two).
template <typename T>
struct AffineMap2 {
    double Mc[4], kc[2], Md[4];
    T J[4], An[4], Af[4];
};

template <typename T>
inline AffineMap2<T> affine_map2(const AffineMap<T> &m)
{
    AffineMap2<T> q;
    for (int a = 0; a < 2; a++) {
        q.kc[a] = m.kc[a];
        for (int b = 0; b < 2; b++) {
            q.Mc[2 * a + b] = m.Mc[3 * a + b];
            q.Md[2 * a + b] = m.Md[3 * a + b];
        }
    }
    for (int k = 0; k < 4; k++) {
        q.J[k] = m.J[k];
        q.An[k] = m.An[k];
        q.Af[k] = m.Af[k];
    }
    return q;
}

// The foot of node (i, j), split.
template <typename T>
__device__ __forceinline__ void affine_foot(const Geom &g, const AffineMap2<T> &am, int i, int j,
                                            int *cell, T *xi, bool *outb)
{
    double s[2];
    if constexpr (sizeof(T) == 4) {
        const int idx[2] = {i, j};
#pragma unroll
        for (int a = 0; a < 2; a++)
            s[a] = am.kc[a] + am.Md[2 * a] * double(i) + am.Md[2 * a + 1] * double(j);
        split_disp<T, 2>(g, idx, s, cell, xi, outb);
    } else {
#pragma unroll
        for (int a = 0; a < 2; a++)
            s[a] = am.kc[a] + am.Mc[2 * a] * double(i) + am.Mc[2 * a + 1] * double(j);
        split_cells<T, 2>(g, s, cell, xi, outb);
    }
}

// The boundary treatment of the bicubic's gradient and the gradient update: phi,
// psi_x, psi_y.
template <typename T, int PSI>
__device__ __forceinline__ void affine_values(const AffineMap2<T> &am, double dt, const bool *outb,
                                              T H, T Hx, T Hy, T *out)
{
    if (outb[0]) Hx = T(0);
    if (outb[1]) Hy = T(0);
    out[0] = H;
    if constexpr (PSI == GALS_PSI_HEUN) {
        const T gH[2] = {Hx, Hy};
        heun_gradient<T, 2>(am.Af, am.An, T(dt), gH, out + 1);
    } else {
        out[1] = am.J[0] * Hx + am.J[2] * Hy;
        out[2] = am.J[1] * Hx + am.J[3] * Hy;
    }
}

// Run f with the cross-derivative mode and the gradient update as
// compile-time constants.
template <class F>
inline hipError_t with_modes(int mixed, int psi, F &&f)
{
    auto on_psi = [&](auto mix) -> hipError_t {
        if (psi == GALS_PSI_HEUN) return f(mix, std::integral_constant<int, GALS_PSI_HEUN>{});
        return f(mix, std::integral_constant<int, GALS_PSI_SUPERCONSISTENT>{});
    };
    if (mixed == GALS_MIXED_ZERO) return on_psi(std::integral_constant<int, GALS_MIXED_ZERO>{});
    if (mixed == GALS_MIXED_CELL) return on_psi(std::integral_constant<int, GALS_MIXED_CELL>{});
    return on_psi(std::integral_constant<int, GALS_MIXED_CENTRAL>{});
}

}  // namespace gals
