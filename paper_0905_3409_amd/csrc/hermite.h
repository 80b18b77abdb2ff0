// Device building blocks of one GA-CIR step: the superconsistent Shu-Osher
// trace, the FP64 cell split, the cell gather with on-the-fly central cross
// derivatives, and the bi-/tri-cubic Hermite evaluation.
#pragma once

#include "velocity.h"

namespace gals {

// ---------------------------------------------------------------------------
// Superconsistent Shu-Osher trace (sec. 5.1, Ex. ex:superconsistent_ShuOsher).
// Positions are FP64; velocities and the Jacobian chain are in T. J is the
// Jacobian of the foot map in J form, J[i*D+j] = dX_i/dx_j, so the gradient
// update of eq. (superconsistency) is psi_new = J^T grad H.
// ---------------------------------------------------------------------------
template <typename T, int D>
__device__ __forceinline__ void matmul_acc(const T *A, const T *B, T *C)
{
#pragma unroll
    for (int i = 0; i < D; i++)
#pragma unroll
        for (int j = 0; j < D; j++) {
            T s = A[i * D] * B[j];
#pragma unroll
            for (int k = 1; k < D; k++) s += A[i * D + k] * B[k * D + j];
            C[i * D + j] = s;
        }
}

// Superconsistent Jacobian of the Shu-Osher foot map from the velocity
// Jacobians A0, A1, A2 at the three stage points (J form):
// J1 = I - dt A0; J2 = I - dt (A0/4 + A1 J1 / 4);
// J = I - dt (A0/6 + A1 J1 / 6 + 2 A2 J2 / 3).
template <typename T, int D>
__device__ __forceinline__ void jacobian_chain(const T *A0, const T *A1, const T *A2, T dtT, T *J)
{
    T J1[D * D], B1[D * D], J2[D * D], B2[D * D];
#pragma unroll
    for (int k = 0; k < D * D; k++) J1[k] = T((k % (D + 1)) == 0) - dtT * A0[k];
    matmul_acc<T, D>(A1, J1, B1);
#pragma unroll
    for (int k = 0; k < D * D; k++)
        J2[k] = T((k % (D + 1)) == 0) - dtT * (T(0.25) * A0[k] + T(0.25) * B1[k]);
    matmul_acc<T, D>(A2, J2, B2);
#pragma unroll
    for (int k = 0; k < D * D; k++)
        J[k] = T((k % (D + 1)) == 0) -
               dtT * (A0[k] * T(1.0 / 6.0) + B1[k] * T(1.0 / 6.0) + B2[k] * T(2.0 / 3.0));
}

// The same chain from the stage Jacobians without their time factors,
// R_k = A_k / c_k, with dt c_k folded into the weights of Stage:
// J1 = I - e1 R0; J2 = I - q1 R0 - q2 R1 J1; J = I - f1 R0 - f2 R1 J1 - f3 R2 J2.
template <typename T, int D>
__device__ __forceinline__ void jacobian_chain_w(const T *R0, const T *R1, const T *R2,
                                                 const Stage<T> &st, T *J)
{
    T J1[D * D], P1[D * D], J2[D * D], P2[D * D];
#pragma unroll
    for (int k = 0; k < D * D; k++) J1[k] = T((k % (D + 1)) == 0) - st.e1 * R0[k];
    matmul_acc<T, D>(R1, J1, P1);
#pragma unroll
    for (int k = 0; k < D * D; k++) J2[k] = T((k % (D + 1)) == 0) - st.q1 * R0[k] - st.q2 * P1[k];
    matmul_acc<T, D>(R2, J2, P2);
#pragma unroll
    for (int k = 0; k < D * D; k++)
        J[k] = T((k % (D + 1)) == 0) - st.f1 * R0[k] - st.f2 * P1[k] - st.f3 * P2[k];
}

// CHAIN = false (Heun's gradient update) skips the Jacobian chain; J then
// receives A0, the velocity Jacobian at the node at time t + dt.
template <typename T, int D, int KIND, bool CHAIN = true>
__device__ __forceinline__ void trace(const Vel<T> &p, const Stage<T> &st, double dt,
                                      const double *x, double *X, T *J)
{
    T v0[D], A0[D * D], v1[D], A1[D * D], v2[D], A2[D * D];
    double x1[D], x2[D];
    const T dtT = T(dt);
    // stage 1: v(x, t+dt)
    velocity<T, D, KIND>(p, x, st.c1, v0, A0);
#pragma unroll
    for (int i = 0; i < D; i++) x1[i] = x[i] - dt * double(v0[i]);
    // stage 2: v(x1, t)
    velocity<T, D, KIND>(p, x1, st.c2, v1, A1);
#pragma unroll
    for (int i = 0; i < D; i++) x2[i] = x[i] - dt * (0.25 * double(v0[i]) + 0.25 * double(v1[i]));
    // stage 3: v(x2, t+dt/2)
    velocity<T, D, KIND>(p, x2, st.c3, v2, A2);
#pragma unroll
    for (int i = 0; i < D; i++)
        X[i] = x[i] - dt * (double(v0[i]) * (1.0 / 6.0) + double(v1[i]) * (1.0 / 6.0) +
                            double(v2[i]) * (2.0 / 3.0));
    if constexpr (CHAIN) {
        jacobian_chain<T, D>(A0, A1, A2, dtT, J);
    } else {
#pragma unroll
        for (int k = 0; k < D * D; k++) J[k] = A0[k];
    }
}

// The chain with the weighted terms summed before they leave the identity: one
// rounding at the size of 1 in place of three, as in jacobian_chain.
template <typename T, int D>
__device__ __forceinline__ void jacobian_chain_s(const T *R0, const T *R1, const T *R2,
                                                 const Stage<T> &st, T *J)
{
    T J1[D * D], P1[D * D], J2[D * D], P2[D * D];
#pragma unroll
    for (int k = 0; k < D * D; k++) J1[k] = T((k % (D + 1)) == 0) - st.e1 * R0[k];
    matmul_acc<T, D>(R1, J1, P1);
#pragma unroll
    for (int k = 0; k < D * D; k++)
        J2[k] = T((k % (D + 1)) == 0) - (st.q1 * R0[k] + st.q2 * P1[k]);
    matmul_acc<T, D>(R2, J2, P2);
#pragma unroll
    for (int k = 0; k < D * D; k++)
        J[k] = T((k % (D + 1)) == 0) - (st.f1 * R0[k] + st.f2 * P1[k] + st.f3 * P2[k]);
}

// The same trace for a trig field (kTrigField) in FP64: sin and cos of twice the
// node's angles once, from the per-axis table (tab, entries ti[a]) or, without
// one, from sincospi, and at the two off-node stages by angle addition while every
// offset is in the series' range, sincospi beyond. An FP64 sincospi costs about 45
// instructions, a shifted pair 22: 101^3 FP64 deformation field 40.5 -> 37 us per
// step, 513^2 FP64 vortex 8.7 -> 7.4. The node's rounded sine enters all three
// stages alike, so with sin and cos of the angles themselves the Jacobian's largest
// error would be up to 1.4 times trace's at 3 cells a step on coarse grids; with
// twice the angles foot and Jacobian are no further off than trace's. An FP32 state
// keeps trace: angles added in FP32 raise the foot's largest error from 5.5e-7 to
// 8.0e-7 cells and the Jacobian's from 7e-8 to 1.8e-7 at 3 cells a step on 151^3
// nodes (57 us per step against 65).
// w_k, R_k are the stage fields without the time factor (see Stage).
template <typename T, int D, int KIND, bool CHAIN = true>
__device__ __forceinline__ void trace_trig(const Stage<T> &st, const T *__restrict__ tab,
                                           const int64_t *ti, const double *x, double *X, T *J)
{
    static_assert(sizeof(T) == 8, "FP64 states only");
    T s0[D], c0[D];
#pragma unroll
    for (int a = 0; a < D; a++) {
        if (tab) {
            s0[a] = tab[2 * ti[a]];
            c0[a] = tab[2 * ti[a] + 1];
        } else {
            sincospi(2.0 * x[a], &s0[a], &c0[a]);  // as the table is built
        }
    }
    auto stage = [&](const T *d, T *w, T *R) {
        T s[D], c[D];
        bool near = true;
#pragma unroll
        for (int a = 0; a < D; a++) near = near && fabs(d[a]) <= kShift2Max / (2.0 * kPi);
        if (near) {
#pragma unroll
            for (int a = 0; a < D; a++) shifted_sincos2(s0[a], c0[a], d[a], s[a], c[a]);
        } else {
#pragma unroll
            for (int a = 0; a < D; a++) sincospi(2.0 * (x[a] + d[a]), &s[a], &c[a]);
        }
        trig_field2<T, KIND, D>(s, c, T(1), w, R);
    };
    T w0[D], R0[D * D], w1[D], R1[D * D], w2[D], R2[D * D], d[D];
    trig_field2<T, KIND, D>(s0, c0, T(1), w0, R0);  // at x, t + dt
#pragma unroll
    for (int a = 0; a < D; a++) d[a] = -st.e1 * w0[a];
    stage(d, w1, R1);  // at x + d, t
#pragma unroll
    for (int a = 0; a < D; a++) d[a] = -(st.q1 * w0[a] + st.q2 * w1[a]);
    stage(d, w2, R2);  // at x + d, t + dt/2
#pragma unroll
    for (int a = 0; a < D; a++) X[a] = x[a] - (st.f1 * w0[a] + st.f2 * w1[a] + st.f3 * w2[a]);
    if constexpr (CHAIN) {
        jacobian_chain_s<T, D>(R0, R1, R2, st, J);
    } else {
#pragma unroll
        for (int k = 0; k < D * D; k++) J[k] = st.c1 * R0[k];
    }
}

// The trace of a grid node: tab and ti as in trace_trig.
template <typename T, int D, int KIND, bool CHAIN>
__device__ __forceinline__ void trace_node(const Vel<T> &p, const Stage<T> &st, double dt,
                                           const T *__restrict__ tab, const int64_t *ti,
                                           const double *x, double *X, T *J)
{
    if constexpr (kTrigField<KIND> && sizeof(T) == 8)
        trace_trig<T, D, KIND, CHAIN>(st, tab, ti, x, X, J);
    else
        trace<T, D, KIND, CHAIN>(p, st, dt, x, X, J);
}

// Heun's method for d psi/d tau = -grad v . psi (eq. cir_evolution_psi)
// from the foot (time t, velocity Jacobian Af) to the node (time t + dt,
// An), J form (A[i][j] = dv_i/dx_j, so grad v . psi = A^T psi):
// k1 = -Af^T g, k2 = -An^T (g + dt k1), psi = g + dt (k1 + k2) / 2.
template <typename T, int D>
__device__ __forceinline__ void heun_gradient(const T *Af, const T *An, T dtT, const T *g, T *psi)
{
    T k1[D], pp[D];
#pragma unroll
    for (int i = 0; i < D; i++) {
        T s = Af[i] * g[0];
#pragma unroll
        for (int j = 1; j < D; j++) s += Af[j * D + i] * g[j];
        k1[i] = -s;
    }
#pragma unroll
    for (int i = 0; i < D; i++) pp[i] = g[i] + dtT * k1[i];
#pragma unroll
    for (int i = 0; i < D; i++) {
        T s = An[i] * pp[0];
#pragma unroll
        for (int j = 1; j < D; j++) s += An[j * D + i] * pp[j];
        psi[i] = g[i] + T(0.5) * dtT * (k1[i] - s);
    }
}

// Keep values computed here: the compiler would sink the Jacobian chain past the
// interpolation's branches to its use after them, and hold the stage Jacobians
// across the gather instead of their product.
template <typename T>
__device__ __forceinline__ void pin4(T *v)
{
    asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));
}

// ---------------------------------------------------------------------------
// Homogeneous Neumann treatment of a foot outside the domain: project it onto
// the domain and remember the axes whose normal derivative must vanish. A
// foot counts as outside only when it lies more than kFootTol cells beyond
// the boundary; closer, it stays where it is (the boundary cell's cubic is
// evaluated there), so that a foot within rounding of the boundary, e.g. of a
// node on a face the flow runs along, is not decided by that rounding.
// ---------------------------------------------------------------------------

template <int D>
__device__ __forceinline__ unsigned project_foot(const Geom &g, double *X)
{
    unsigned out = 0;
    if (g.bc == GALS_BC_NEUMANN) {
#pragma unroll
        for (int a = 0; a < D; a++) {
            const double tol = kFootTol * g.h[a];
            if (X[a] < g.lo[a] - tol) {
                X[a] = g.lo[a];
                out |= 1u << a;
            } else if (X[a] > g.top[a] + tol) {
                X[a] = g.top[a];
                out |= 1u << a;
            }
        }
    }
    return out;
}

// ---------------------------------------------------------------------------
// Cell split in FP64: clamped cell index, unclamped local coordinate (a foot
// outside the grid evaluates the boundary cell's polynomial). Not-a-number
// feet land in cell 0 and propagate.
// ---------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ void split(const Geom &g, const double *X, int *cell, double *xi)
{
#pragma unroll
    for (int a = 0; a < D; a++) {
        const double s = (X[a] - g.lo[a]) * g.inv_h[a];
        const double fl = floor(s);
        const double top = double(g.nc[a] - 1);
        int c;
        if (fl >= 0.0 && fl <= top) c = int(fl);
        else if (fl > top) c = g.nc[a] - 1;
        else c = 0;
        cell[a] = c;
        xi[a] = s - double(c);
    }
}

// ---------------------------------------------------------------------------
// Raw buffer loads: one descriptor per plane (base, bytes of the plane, or, for
// wide loads, which may hang over its last node, up to that node: g.span), 32-bit
// element offsets; what lies beyond is not accessed and reads as 0, word by word.
// The host keeps every plane below 2 GiB, so its size in bytes and every byte
// offset into it fit a signed 32-bit integer.
// ---------------------------------------------------------------------------
typedef __amdgpu_buffer_rsrc_t Rsrc;

template <typename T>
__device__ __forceinline__ Rsrc plane_rsrc(const T *base, int64_t elems)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(base), 0, int(elems * int64_t(sizeof(T))),
                                             0x00020000);
}

__device__ __forceinline__ float bload(Rsrc r, unsigned elem, float)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, elem * 4u, 0, 0));
}

__device__ __forceinline__ double bload(Rsrc r, unsigned elem, double)
{
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, elem * 8u, 0, 0));
}

// Two (four) consecutive elements from `elem` on, as one or two wide loads.
template <typename T, int N>
using Vec = T __attribute__((ext_vector_type(N)));

__device__ __forceinline__ void bload2(Rsrc r, unsigned elem, float *u)
{
    const auto v =
        __builtin_bit_cast(Vec<float, 2>, __builtin_amdgcn_raw_buffer_load_b64(r, elem * 4u, 0, 0));
    u[0] = v.x;
    u[1] = v.y;
}

__device__ __forceinline__ void bload2(Rsrc r, unsigned elem, double *u)
{
    const auto v =
        __builtin_bit_cast(Vec<double, 2>, __builtin_amdgcn_raw_buffer_load_b128(r, elem * 8u, 0, 0));
    u[0] = v.x;
    u[1] = v.y;
}

__device__ __forceinline__ void bload4(Rsrc r, unsigned elem, float *u)
{
    const auto v =
        __builtin_bit_cast(Vec<float, 4>, __builtin_amdgcn_raw_buffer_load_b128(r, elem * 4u, 0, 0));
    u[0] = v.x;
    u[1] = v.y;
    u[2] = v.z;
    u[3] = v.w;
}

__device__ __forceinline__ void bload4(Rsrc r, unsigned elem, double *u)
{
    bload2(r, elem, u);
    bload2(r, elem + 2u, u + 2);
}

// Store element `elem` of a plane through a 32-bit byte offset (every plane
// is below 2 GiB), so the address is the plane's scalar base plus one vector
// offset.
template <typename T>
__device__ __forceinline__ void pstore(T *base, unsigned elem, T v)
{
    *reinterpret_cast<T *>(reinterpret_cast<char *>(base) + elem * unsigned(sizeof(T))) = v;
}

// ---------------------------------------------------------------------------
// Cross derivatives (sec. 2.3, approach (A)) at the two corners c, c+1 of a
// cell from samples u[0..3] at nodes c-1..c+2 (clamped into [0, N]): central
// differences inside, one-sided 3-point differences at node 0 and node N.
// ---------------------------------------------------------------------------
// WAVE: the one-sided forms are evaluated only by waves that hold an edge
// cell (a uniform branch; FP32 2D only: elsewhere the branch costs registers).
template <typename T, bool WAVE = false>
__device__ __forceinline__ void diff_pair(const T *u, bool lo_edge, bool hi_edge, T inv2h,
                                          T &d0, T &d1)
{
    T a = u[2] - u[0], b = u[3] - u[1];
    if (!WAVE || __builtin_amdgcn_ballot_w64(lo_edge || hi_edge)) {
        a = lo_edge ? T(4) * u[2] - T(3) * u[1] - u[3] : a;
        b = hi_edge ? T(3) * u[2] - T(4) * u[1] + u[0] : b;
    }
    d0 = a * inv2h;
    d1 = b * inv2h;
}

// Cross derivative by the cell-based approach (B) (sec. 2.3) on one cell
// facet spanned by axes a, b: ga = phi_a, gb = phi_b at the facet's vertices
// (index bit 0 along a, bit 1 along b). Differences along the four edges
// give the cross derivative at the edge centres; a vertex takes 3/4 of its
// two edges and -1/4 of the two opposite ones (bilinear extrapolation).
template <typename T>
__device__ __forceinline__ void cell_cross(const T *ga, const T *gb, T inv_ha, T inv_hb, T *out)
{
    const T ea0 = (ga[2] - ga[0]) * inv_hb, ea1 = (ga[3] - ga[1]) * inv_hb;  // edges along b
    const T eb0 = (gb[1] - gb[0]) * inv_ha, eb1 = (gb[3] - gb[2]) * inv_ha;  // edges along a
    out[0] = T(0.75) * (ea0 + eb0) - T(0.25) * (ea1 + eb1);
    out[1] = T(0.75) * (ea1 + eb0) - T(0.25) * (ea0 + eb1);
    out[2] = T(0.75) * (ea0 + eb1) - T(0.25) * (ea1 + eb0);
    out[3] = T(0.75) * (ea1 + eb1) - T(0.25) * (ea0 + eb0);
}

// Cell data d[v][alpha]: v = vertex bits (x = bit 0), alpha = derivative bits.
// 2D alpha: 0 phi, 1 psi_x, 2 psi_y, 3 phi_xy.
template <typename T, int MIX>
__device__ __forceinline__ void gather2d(const Geom &g, Rsrc rphi, Rsrc rgx, Rsrc rgy, int cx,
                                         int cy, T d[4][4])
{
    const unsigned r0 = unsigned(cy) * unsigned(g.pitch), r1 = r0 + unsigned(g.pitch);
    const unsigned i0 = unsigned(cx), i1 = unsigned(cx) + 1u;
    d[0][0] = bload(rphi, r0 + i0, T()); d[1][0] = bload(rphi, r0 + i1, T());
    d[2][0] = bload(rphi, r1 + i0, T()); d[3][0] = bload(rphi, r1 + i1, T());
    d[0][1] = bload(rgx, r0 + i0, T()); d[1][1] = bload(rgx, r0 + i1, T());
    d[2][1] = bload(rgx, r1 + i0, T()); d[3][1] = bload(rgx, r1 + i1, T());
    if constexpr (MIX == GALS_MIXED_CELL) {
        d[0][2] = bload(rgy, r0 + i0, T()); d[1][2] = bload(rgy, r0 + i1, T());
        d[2][2] = bload(rgy, r1 + i0, T()); d[3][2] = bload(rgy, r1 + i1, T());
        T ga[4], gb[4], out[4];
#pragma unroll
        for (int v = 0; v < 4; v++) {
            ga[v] = d[v][1];
            gb[v] = d[v][2];
        }
        cell_cross(ga, gb, geo_ih<T>(g, 0), geo_ih<T>(g, 1), out);
#pragma unroll
        for (int v = 0; v < 4; v++) d[v][3] = out[v];
    } else if constexpr (MIX == GALS_MIXED_CENTRAL) {
        const unsigned im = unsigned(cx > 0 ? cx - 1 : 0);
        const unsigned i2 = unsigned(cx + 2 <= g.nc[0] ? cx + 2 : g.nc[0]);
        const T u0[4] = {bload(rgy, r0 + im, T()), bload(rgy, r0 + i0, T()),
                         bload(rgy, r0 + i1, T()), bload(rgy, r0 + i2, T())};
        const T u1[4] = {bload(rgy, r1 + im, T()), bload(rgy, r1 + i0, T()),
                         bload(rgy, r1 + i1, T()), bload(rgy, r1 + i2, T())};
        d[0][2] = u0[1]; d[1][2] = u0[2];
        d[2][2] = u1[1]; d[3][2] = u1[2];
        const T inv2h = geo_i2h<T>(g, 0);
        const bool lo = cx == 0, hi = cx + 1 == g.nc[0];
        diff_pair<T, sizeof(T) == 4>(u0, lo, hi, inv2h, d[0][3], d[1][3]);
        diff_pair<T, sizeof(T) == 4>(u1, lo, hi, inv2h, d[2][3], d[3][3]);
    } else {
        d[0][2] = bload(rgy, r0 + i0, T()); d[1][2] = bload(rgy, r0 + i1, T());
        d[2][2] = bload(rgy, r1 + i0, T()); d[3][2] = bload(rgy, r1 + i1, T());
        d[0][3] = d[1][3] = d[2][3] = d[3][3] = T(0);
    }
}

// 3D alpha: 0 phi, 1 psi_x, 2 psi_y, 3 phi_xy, 4 psi_z, 5 phi_xz, 6 phi_yz,
// 7 phi_xyz, for the rules whose cross derivatives come from the cell's own
// vertices: cell-based (B), or all zero. (tricubic_central evaluates central
// differencing, (A), without forming them.)
template <typename T, int MIX>
__device__ __forceinline__ void gather3d(const Geom &g, Rsrc rphi, Rsrc rgx, Rsrc rgy, Rsrc rgz,
                                         int c0, int c1, int c2, T d[8][8])
{
    static_assert(MIX != GALS_MIXED_CENTRAL, "see tricubic_central");
    const unsigned P = unsigned(g.pitch), S = unsigned(g.pitch) * unsigned(g.n[1]);
#pragma unroll
    for (int v = 0; v < 8; v++) {
        const unsigned o = unsigned(c2 + (v >> 2)) * S + unsigned(c1 + ((v >> 1) & 1)) * P +
                           unsigned(c0 + (v & 1));
        d[v][0] = bload(rphi, o, T());
        d[v][1] = bload(rgx, o, T());
        d[v][2] = bload(rgy, o, T());
        d[v][4] = bload(rgz, o, T());
        d[v][3] = d[v][5] = d[v][6] = d[v][7] = T(0);
    }
    if constexpr (MIX == GALS_MIXED_CELL) {
        // cross derivatives per facet
        const T ih[3] = {geo_ih<T>(g, 0), geo_ih<T>(g, 1), geo_ih<T>(g, 2)};
        // (a, b) = (x, y), (x, z), (y, z) into alpha 3, 5, 6; facet level along
        // the third axis c
        constexpr int pa[3] = {0, 0, 1}, pb[3] = {1, 2, 2}, pc[3] = {2, 1, 0};
        constexpr int slot[3] = {3, 5, 6};
#pragma unroll
        for (int q = 0; q < 3; q++)
#pragma unroll
            for (int lc = 0; lc < 2; lc++) {
                T ga[4], gb[4], out[4];
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const int v = ((k & 1) << pa[q]) | (((k >> 1) & 1) << pb[q]) | (lc << pc[q]);
                    ga[k] = d[v][1 << pa[q]];
                    gb[k] = d[v][1 << pb[q]];
                }
                cell_cross(ga, gb, ih[pa[q]], ih[pb[q]], out);
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const int v = ((k & 1) << pa[q]) | (((k >> 1) & 1) << pb[q]) | (lc << pc[q]);
                    d[v][slot[q]] = out[k];
                }
            }
        // phi_xyz, first order, from psi_z on the xy facet of each z level
#pragma unroll
        for (int lz = 0; lz < 2; lz++) {
            const int b = 4 * lz;
            const T xyz = (d[b + 3][4] - d[b + 2][4] - d[b + 1][4] + d[b][4]) * (ih[0] * ih[1]);
#pragma unroll
            for (int k = 0; k < 4; k++) d[b + k][7] = xyz;
        }
    }
}

// ---------------------------------------------------------------------------
// 1D Hermite factors (sec. 2.3, eq. 1-cubic_basis_functions), with the h^alpha
// scaling of eq. (p-cubic_interpolant) folded in. Index k = v + 2 alpha:
//   k=0 f(t), k=1 f(1-t), k=2 h g(t), k=3 -h g(1-t),
// f = 1 - 3t^2 + 2t^3, g = t (1-t)^2; dw = d/dx, ddw = d2/dx2.
// ---------------------------------------------------------------------------
template <typename T>
struct Basis {
    T w[4], dw[4], ddw[4];
};

template <typename T, bool SECOND>
__device__ __forceinline__ void basis(T t, T h, T inv_h, Basis<T> &b)
{
    const T s = T(1) - t;
    const T t2 = t * t;
    const T f1 = t2 * (T(3) - T(2) * t);  // f(1-t) = 1 - f(t)
    b.w[0] = T(1) - f1;
    b.w[1] = f1;
    b.w[2] = h * t * s * s;
    b.w[3] = -h * s * t2;
    const T df = T(6) * t * s * inv_h;  // d/dx f(1-t)
    b.dw[0] = -df;
    b.dw[1] = df;
    b.dw[2] = s * (T(1) - T(3) * t);
    b.dw[3] = t * (T(3) * t - T(2));
    if constexpr (SECOND) {
        const T ddf = (T(12) * t - T(6)) * inv_h * inv_h;
        b.ddw[0] = ddf;
        b.ddw[1] = -ddf;
        b.ddw[2] = (T(6) * t - T(4)) * inv_h;
        b.ddw[3] = (T(6) * t - T(2)) * inv_h;
    }
}

// Value and gradient of the bicubic (contract y, then x).
template <typename T>
__device__ __forceinline__ void hermite2d(const T d[4][4], const Basis<T> &bx, const Basis<T> &by,
                                          T &H, T &Hx, T &Hy)
{
    H = Hx = Hy = T(0);
#pragma unroll
    for (int vx = 0; vx < 2; vx++)
#pragma unroll
        for (int ax = 0; ax < 2; ax++) {
            T s = T(0), sy = T(0);
#pragma unroll
            for (int vy = 0; vy < 2; vy++)
#pragma unroll
                for (int ay = 0; ay < 2; ay++) {
                    const T dd = d[vx + 2 * vy][ax + 2 * ay];
                    s += dd * by.w[vy + 2 * ay];
                    sy += dd * by.dw[vy + 2 * ay];
                }
            const int k = vx + 2 * ax;
            H += s * bx.w[k];
            Hx += s * bx.dw[k];
            Hy += sy * bx.w[k];
        }
}

// Value, gradient and Hessian of the bicubic.
template <typename T>
__device__ __forceinline__ void hermite2d_full(const T d[4][4], const Basis<T> &bx,
                                               const Basis<T> &by, T &H, T *G, T *Hs)
{
    T h = 0, hx = 0, hy = 0, hxx = 0, hxy = 0, hyy = 0;
#pragma unroll
    for (int vx = 0; vx < 2; vx++)
#pragma unroll
        for (int ax = 0; ax < 2; ax++) {
            T s0 = 0, s1 = 0, s2 = 0;
#pragma unroll
            for (int vy = 0; vy < 2; vy++)
#pragma unroll
                for (int ay = 0; ay < 2; ay++) {
                    const T dd = d[vx + 2 * vy][ax + 2 * ay];
                    s0 += dd * by.w[vy + 2 * ay];
                    s1 += dd * by.dw[vy + 2 * ay];
                    s2 += dd * by.ddw[vy + 2 * ay];
                }
            const int k = vx + 2 * ax;
            h += s0 * bx.w[k];
            hx += s0 * bx.dw[k];
            hxx += s0 * bx.ddw[k];
            hy += s1 * bx.w[k];
            hxy += s1 * bx.dw[k];
            hyy += s2 * bx.w[k];
        }
    H = h;
    G[0] = hx; G[1] = hy;
    Hs[0] = hxx; Hs[1] = hxy; Hs[2] = hxy; Hs[3] = hyy;
}

// Value and gradient of the tricubic (contract z, then y, then x).
template <typename T>
__device__ __forceinline__ void hermite3d(const T d[8][8], const Basis<T> &bx, const Basis<T> &by,
                                          const Basis<T> &bz, T &H, T &Hx, T &Hy, T &Hz)
{
    H = Hx = Hy = Hz = T(0);
#pragma unroll
    for (int vx = 0; vx < 2; vx++)
#pragma unroll
        for (int ax = 0; ax < 2; ax++) {
            T a0 = 0, ay_ = 0, az_ = 0;
#pragma unroll
            for (int vy = 0; vy < 2; vy++)
#pragma unroll
                for (int ay = 0; ay < 2; ay++) {
                    T z0 = 0, z1 = 0;
#pragma unroll
                    for (int vz = 0; vz < 2; vz++)
#pragma unroll
                        for (int az = 0; az < 2; az++) {
                            const T dd = d[vx + 2 * vy + 4 * vz][ax + 2 * ay + 4 * az];
                            z0 += dd * bz.w[vz + 2 * az];
                            z1 += dd * bz.dw[vz + 2 * az];
                        }
                    const int ky = vy + 2 * ay;
                    a0 += z0 * by.w[ky];
                    ay_ += z0 * by.dw[ky];
                    az_ += z1 * by.w[ky];
                }
            const int k = vx + 2 * ax;
            H += a0 * bx.w[k];
            Hx += a0 * bx.dw[k];
            Hy += ay_ * bx.w[k];
            Hz += az_ * bx.w[k];
        }
}

// Value, gradient and Hessian (row-major 3x3) of the tricubic.
template <typename T>
__device__ __forceinline__ void hermite3d_full(const T d[8][8], const Basis<T> &bx,
                                               const Basis<T> &by, const Basis<T> &bz, T &H,
                                               T *G, T *Hs)
{
    T h = 0, hx = 0, hy = 0, hz = 0, hxx = 0, hyy = 0, hzz = 0, hxy = 0, hxz = 0, hyz = 0;
#pragma unroll
    for (int vx = 0; vx < 2; vx++)
#pragma unroll
        for (int ax = 0; ax < 2; ax++) {
            T a00 = 0, a10 = 0, a20 = 0, a01 = 0, a11 = 0, a02 = 0;
#pragma unroll
            for (int vy = 0; vy < 2; vy++)
#pragma unroll
                for (int ay = 0; ay < 2; ay++) {
                    T z0 = 0, z1 = 0, z2 = 0;
#pragma unroll
                    for (int vz = 0; vz < 2; vz++)
#pragma unroll
                        for (int az = 0; az < 2; az++) {
                            const T dd = d[vx + 2 * vy + 4 * vz][ax + 2 * ay + 4 * az];
                            z0 += dd * bz.w[vz + 2 * az];
                            z1 += dd * bz.dw[vz + 2 * az];
                            z2 += dd * bz.ddw[vz + 2 * az];
                        }
                    const int ky = vy + 2 * ay;
                    a00 += z0 * by.w[ky];
                    a10 += z0 * by.dw[ky];
                    a20 += z0 * by.ddw[ky];
                    a01 += z1 * by.w[ky];
                    a11 += z1 * by.dw[ky];
                    a02 += z2 * by.w[ky];
                }
            const int k = vx + 2 * ax;
            h += a00 * bx.w[k];
            hx += a00 * bx.dw[k];
            hxx += a00 * bx.ddw[k];
            hy += a10 * bx.w[k];
            hxy += a10 * bx.dw[k];
            hyy += a20 * bx.w[k];
            hz += a01 * bx.w[k];
            hxz += a01 * bx.dw[k];
            hyz += a11 * bx.w[k];
            hzz += a02 * bx.w[k];
        }
    H = h;
    G[0] = hx; G[1] = hy; G[2] = hz;
    Hs[0] = hxx; Hs[1] = hxy; Hs[2] = hxz;
    Hs[3] = hxy; Hs[4] = hyy; Hs[5] = hyz;
    Hs[6] = hxz; Hs[7] = hyz; Hs[8] = hzz;
}

// ---------------------------------------------------------------------------
// The tricubic with central cross derivatives (A), without forming them. The
// phi_xy, phi_xz, phi_yz and phi_xyz data are differences of psi_y and psi_z
// along x and y, and the interpolant is linear in them, so along such an axis
// the Hermite weights of a sample and of its difference combine into four
// weights on the nodes c - 1 .. c + 2 (with u the samples and D their
// difference: w0 u_c + w1 u_c+1 + w2 D_c + w3 D_c+1). psi_z is then a 4 x 4
// stencil times the two z data weights, psi_y a 4 x 2 stencil, and the
// one-sided differences of the grid's first and last cell change the weights
// of one axis instead of 20 difference pairs per node. Contracted x, y, z:
// 192 multiply-adds, the differences with their one-sided forms and selects
// (240 instructions a node) gone. phi enters as its differences from the
// cell's first vertex: its derivatives are divided differences, and rounding
// then acts on values of the size of h |grad phi| instead of |phi|. With the
// Hessian (SECOND) the whole linear part at that vertex is taken out of the data
// and added back: second differences of the gradient would leave u |grad phi| / h
// (error of the FP32 curvature on 257^3 nodes 1.5e-5 with neither, 8e-6 with the
// first, 2.9e-6 with both).
//
// Bound: vector issue (FP64 and the vector potential), the L1's rate for a node's
// scattered rows (20 loads in FP32, 32 in FP64) where the trace is cheap. Measured
// against forming the cross derivatives, both with one load per value, us per step
// on one card: 257^3 FP32 vector potential 610 -> 540, 101^3 FP64 deformation field
// 53 -> 43, 141 x 131 x 121 FP64 vector potential 250 -> 185, 385^3 FP32 rotation
// 980 -> 935; 10^6 points in FP32 363 -> 334 (with their transposed copy). A row's
// nodes by wide loads: 101^3 FP64 deformation field 45 -> 42, FP64 rotation 92 ->
// 62. Loads grouped by x node instead of by row cost the rotation 15 % and the
// points 75 % (a row's loads no longer meet in the L1); two or three groups in
// flight measured no faster than one and took the FP64 kernels from three waves per
// SIMD to two.
// ---------------------------------------------------------------------------
template <typename T>
struct StencilWeights {
    T w[4], dw[4], ddw[4];
};

// Weights over the nodes c - 1 .. c + 2 from the Hermite weights a (w0, w1,
// w2, w3) of one derivative order; i2h = 1 / (2 h). At the first (last) cell
// the node c - 1 (c + 2) does not exist and gets weight 0.
template <typename T>
__device__ __forceinline__ void stencil_weights(const T *a, T i2h, bool lo, bool hi, T *w)
{
    const T p = a[2] * i2h, q = a[3] * i2h;
    w[0] = -p;
    w[1] = a[0] - q;
    w[2] = a[1] + p;
    w[3] = q;
    if (__builtin_expect(lo, 0)) {  // D_c one-sided: (4 u_c+1 - 3 u_c - u_c+2) / 2h
        w[0] = T(0);
        w[1] = a[0] - (T(3) * p + q);
        w[2] = a[1] + T(4) * p;
        w[3] = q - p;
    }
    if (__builtin_expect(hi, 0)) {  // D_c+1 one-sided: (3 u_c+1 - 4 u_c + u_c-1) / 2h
        w[0] = q - p;
        w[1] = a[0] - T(4) * q;
        w[2] = a[1] + (p + T(3) * q);
        w[3] = T(0);
    }
}

// Value, gradient G and (SECOND) Hessian Hs (row-major 3 x 3).
template <typename T, bool SECOND>
__device__ __forceinline__ void tricubic_central(const Geom &g, Rsrc rphi, Rsrc rgx, Rsrc rgy,
                                                 Rsrc rgz, const int *c, const T *xi, T &H, T *G,
                                                 T *Hs)
{
    Basis<T> bx, by, bz;
    StencilWeights<T> sx, sy;  // x and y weights of psi_y and psi_z
    basis<T, SECOND>(xi[0], geo_h<T>(g, 0), geo_ih<T>(g, 0), bx);
    basis<T, SECOND>(xi[1], geo_h<T>(g, 1), geo_ih<T>(g, 1), by);
    basis<T, SECOND>(xi[2], geo_h<T>(g, 2), geo_ih<T>(g, 2), bz);
    const bool xlo = c[0] == 0, xhi = c[0] + 1 == g.nc[0];
    const bool ylo = c[1] == 0, yhi = c[1] + 1 == g.nc[1];
    const T i2hx = geo_i2h<T>(g, 0), i2hy = geo_i2h<T>(g, 1);
    stencil_weights(bx.w, i2hx, xlo, xhi, sx.w);
    stencil_weights(bx.dw, i2hx, xlo, xhi, sx.dw);
    stencil_weights(by.w, i2hy, ylo, yhi, sy.w);
    stencil_weights(by.dw, i2hy, ylo, yhi, sy.dw);
    if constexpr (SECOND) {
        stencil_weights(bx.ddw, i2hx, xlo, xhi, sx.ddw);
        stencil_weights(by.ddw, i2hy, ylo, yhi, sy.ddw);
    }
    const unsigned P = unsigned(g.pitch), S = unsigned(g.pitch) * unsigned(g.n[1]);
    const unsigned o0 = unsigned(c[2]) * S + unsigned(c[1]) * P + unsigned(c[0]);
    // A row's four x nodes are one window of wide loads: c - 1 .. c + 2, or
    // 0 .. 3 at the first cell, whose weights move down by one. The window's
    // last value belongs to no stencil at the first cell and lies past the row
    // at the last one (in the row's padding, the next row, or past the plane's
    // last node, where a buffer load gives 0): it is replaced by 0 there,
    // whatever it holds.
    // Rows past the grid repeat their neighbour with weight 0.
    const unsigned xm = xlo ? 0u : 1u;
    const bool xedge = xlo || xhi;
    if (xlo) {
#pragma unroll
        for (int k = 0; k < 3; k++) {
            sx.w[k] = sx.w[k + 1];
            sx.dw[k] = sx.dw[k + 1];
            if constexpr (SECOND) sx.ddw[k] = sx.ddw[k + 1];
        }
    }
    const unsigned ym = ylo ? 0u : P, yp = yhi ? 0u : P;
    const unsigned row[4] = {o0 - ym, o0, o0 + P, o0 + P + yp};

    // Eight groups of eight samples, four per plane c2 + vz: psi_z on rows
    // c1 - 1 and c1, on rows c1 + 1 and c1 + 2, then psi_y, phi and psi_x on
    // row c1 and on row c1 + 1. Whole rows at a time keep a row's loads in the
    // cache lines they share.
    auto load = [&](int q, T *u) {
        const unsigned zo = q < 4 ? 0u : S;
        const int part = q & 3;
        if (part < 2) {
#pragma unroll
            for (int r = 0; r < 2; r++) bload4(rgz, row[2 * part + r] + zo - xm, u + 4 * r);
        } else {
            const unsigned o = row[part - 1] + zo;
            bload4(rgy, o - xm, u);
            bload2(rphi, o, u + 4);
            bload2(rgx, o, u + 6);
        }
    };
    // a[dx dy]: sums over x and y of one plane's samples, derivative orders dx
    // and dy, those with phi-like z weights (0) and psi_z (1)
    struct Acc {
        T a00, a10, a01, a20, a11, a02;
    };
    Acc A[2] = {};
    T ref = T(0), p0 = T(0), p1 = T(0), p2 = T(0);  // phi and its gradient at the first vertex
    // a foot on the far vertex along an axis (a node of the grid's last row or
    // plane) takes that vertex's phi as the reference: an exact shift stays exact
    T far_phi = T(0);
    const bool far_side = !SECOND && (xi[0] == T(1) || xi[1] == T(1) || xi[2] == T(1));
    if (__builtin_expect(far_side, 0))
        far_phi = bload(rphi, o0 + (xi[0] == T(1) ? 1u : 0u) + (xi[1] == T(1) ? P : 0u) +
                                  (xi[2] == T(1) ? S : 0u), T());
    const T gh[3] = {geo_h<T>(g, 0), geo_h<T>(g, 1), geo_h<T>(g, 2)};
    auto dot = [](const T *u, const T *w) { return u[0] * w[0] + u[1] * w[1] + u[2] * w[2] + u[3] * w[3]; };
    auto sums = [&](Acc &a, bool first, T x0, T x1, T x2, T wy, T dwy, T ddwy) {
        a.a00 = first ? x0 * wy : a.a00 + x0 * wy;
        a.a01 = first ? x0 * dwy : a.a01 + x0 * dwy;
        a.a10 = first ? x1 * wy : a.a10 + x1 * wy;
        if constexpr (SECOND) {
            a.a02 = first ? x0 * ddwy : a.a02 + x0 * ddwy;
            a.a11 = first ? x1 * dwy : a.a11 + x1 * dwy;
            a.a20 = first ? x2 * wy : a.a20 + x2 * wy;
        }
    };
    auto add = [&](Acc &a, bool first, const T *w, T base, T wy, T dwy, T ddwy) {
        const T u[4] = {w[0] - base, w[1] - base, w[2] - base, xedge ? T(0) : w[3] - base};
        sums(a, first, dot(u, sx.w), dot(u, sx.dw), SECOND ? dot(u, sx.ddw) : T(0), wy, dwy, ddwy);
    };
    auto sum = [&](int q, const T *u) {
        const int part = q & 3, vz = q >> 2;
        if (part < 2) {
            if (SECOND && q == 0) p2 = xlo ? u[4] : u[5];
#pragma unroll
            for (int r = 0; r < 2; r++) {
                const int jy = 2 * part + r;
                add(A[1], jy == 0, u + 4 * r, p2, sy.w[jy], sy.dw[jy], SECOND ? sy.ddw[jy] : T(0));
            }
        } else {
            const int vy = part - 2;
            if (q == 2) {
                ref = far_side ? far_phi : u[4];
                if constexpr (SECOND) {
                    p0 = u[6];
                    p1 = xlo ? u[0] : u[1];
                }
            }
            T du = u[5] - u[4], r = u[4] - ref;  // phi along x, and above ref
            T g0 = u[6], g1 = u[7];
            if constexpr (SECOND) {
                du -= p0 * gh[0];
                if (vy) r -= p1 * gh[1];
                if (vz) r -= p2 * gh[2];
                g0 -= p0;
                g1 -= p0;
            }
            const T x0 = r + du * bx.w[1] + g0 * bx.w[2] + g1 * bx.w[3];
            const T x1 = du * bx.dw[1] + g0 * bx.dw[2] + g1 * bx.dw[3];
            T x2 = T(0);
            if constexpr (SECOND) x2 = du * bx.ddw[1] + g0 * bx.ddw[2] + g1 * bx.ddw[3];
            sums(A[0], vy == 0, x0, x1, x2, by.w[vy], by.dw[vy], SECOND ? by.ddw[vy] : T(0));
            add(A[0], false, u, p1, by.w[2 + vy], by.dw[2 + vy], SECOND ? by.ddw[2 + vy] : T(0));
        }
    };
    T h = 0, hx = 0, hy = 0, hz = 0;
    T hxx = 0, hyy = 0, hzz = 0, hxy = 0, hxz = 0, hyz = 0;
    auto reduce = [&](const Acc &a, int kz) {
        h += a.a00 * bz.w[kz];
        hx += a.a10 * bz.w[kz];
        hy += a.a01 * bz.w[kz];
        hz += a.a00 * bz.dw[kz];
        if constexpr (SECOND) {
            hxx += a.a20 * bz.w[kz];
            hxy += a.a11 * bz.w[kz];
            hyy += a.a02 * bz.w[kz];
            hxz += a.a10 * bz.dw[kz];
            hyz += a.a01 * bz.dw[kz];
            hzz += a.a00 * bz.ddw[kz];
        }
    };
    // A group's loads are issued before the previous group's sums, and the sums
    // are pinned there: left to itself the compiler issues every load first
    // and holds their values (the FP32 vector potential then spills).
    T u[2][8];
    load(0, u[0]);
#pragma unroll
    for (int q = 0; q < 8; q++) {
        if (q < 7) load(q + 1, u[(q + 1) & 1]);
        sum(q, u[q & 1]);
        asm volatile("" : "+v"(A[0].a00), "+v"(A[0].a10), "+v"(A[0].a01), "+v"(A[1].a00),
                     "+v"(A[1].a10), "+v"(A[1].a01));
        if constexpr (SECOND)
            asm volatile("" : "+v"(A[0].a20), "+v"(A[0].a11), "+v"(A[0].a02), "+v"(A[1].a20),
                         "+v"(A[1].a11), "+v"(A[1].a02));
        if ((q & 3) == 3) {
            reduce(A[0], q >> 2);
            reduce(A[1], 2 + (q >> 2));
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (SECOND) {
        h += p0 * (xi[0] * gh[0]) + p1 * (xi[1] * gh[1]) + p2 * (xi[2] * gh[2]);
        hx += p0;
        hy += p1;
        hz += p2;
        Hs[0] = hxx; Hs[1] = hxy; Hs[2] = hxz;
        Hs[3] = hxy; Hs[4] = hyy; Hs[5] = hyz;
        Hs[6] = hxz; Hs[7] = hyz; Hs[8] = hzz;
    }
    H = ref + h;
    G[0] = hx; G[1] = hy; G[2] = hz;
    if constexpr (SECOND) {
        // a point on a vertex takes its data as they are, also on one of the grid's
        // last nodes, which are far vertices of their cells (on the first vertex the
        // sums above are exact); data of the cell that are not finite show as they
        // do at its other points, as 0 times them
        bool on = true;
#pragma unroll
        for (int a = 0; a < 3; a++) on = on && (xi[a] == T(0) || xi[a] == T(1));
        if (__builtin_expect(on, 0)) {
            const unsigned o = o0 + (xi[0] == T(1) ? 1u : 0u) + (xi[1] == T(1) ? P : 0u) +
                               (xi[2] == T(1) ? S : 0u);
            H = bload(rphi, o, T()) + T(0) * H;
            G[0] = bload(rgx, o, T()) + T(0) * G[0];
            G[1] = bload(rgy, o, T()) + T(0) * G[1];
            G[2] = bload(rgz, o, T()) + T(0) * G[2];
        }
    }
}

// ---------------------------------------------------------------------------
// The bicubic with central cross derivatives in the same form, for FP64 states:
// psi_y a 4 x 2 stencil, phi as differences from one vertex, a row's samples by
// wide loads. FP32 states keep gather2d and hermite2d (another rounding of phi
// shows in psi as u |phi| / h), and so does the affine step, whose gather is in
// LDS: 19 more registers cost its FP64 kernel two waves per SIMD (513^2 186 -> 190
// us per 32 steps). 1729^2 FP64 stream function: 64 us per step with
// gather2d and hermite2d, 60 with this (VALU instructions per wave 539 ->
// 507, the address unit busy 73 % -> 64 % of the launch).
// ---------------------------------------------------------------------------
template <typename T, int MIX>
constexpr bool kFold2d = sizeof(T) == 8 && MIX == GALS_MIXED_CENTRAL;

// Where a 2D gather's descriptors end: its wide loads may hang over the last node,
// the others only read nodes.
template <typename T, int MIX>
__device__ __forceinline__ int64_t gather_end(const Geom &g)
{
    return kFold2d<T, MIX> ? g.span : g.plane;
}

// One row of the cell: phi and psi_x at c and c + 1, psi_y at the four nodes of the
// window (c - 1 .. c + 2, or 0 .. 3 at the first cell).
template <typename T>
struct Row2d {
    T phi[2], gx[2], gy[4];
};

// row(r) gives row r = 0, 1, phi(vx, vy) a vertex's phi.
template <typename T, class Row, class Phi>
__device__ __forceinline__ void bicubic_central(const Geom &g, int cx, const T *xi, Row row, Phi phi,
                                                T &H, T &Hx, T &Hy)
{
    Basis<T> bx, by;
    basis<T, false>(xi[0], geo_h<T>(g, 0), geo_ih<T>(g, 0), bx);
    basis<T, false>(xi[1], geo_h<T>(g, 1), geo_ih<T>(g, 1), by);
    const bool lo = cx == 0, hi = cx + 1 == g.nc[0], edge = lo || hi;
    const T i2h = geo_i2h<T>(g, 0);
    T w[4], dw[4];
    stencil_weights(bx.w, i2h, lo, hi, w);
    stencil_weights(bx.dw, i2h, lo, hi, dw);
    if (__builtin_expect(lo, 0)) {
#pragma unroll
        for (int k = 0; k < 3; k++) {
            w[k] = w[k + 1];
            dw[k] = dw[k + 1];
        }
    }
    // the vertex the foot is on, if it is on a far one (see tricubic_central)
    T ref = phi(0, 0);
    if (__builtin_expect(xi[0] == T(1) || xi[1] == T(1), 0))
        ref = phi(xi[0] == T(1) ? 1 : 0, xi[1] == T(1) ? 1 : 0);
    T h = 0, hx = 0, hy = 0;
#pragma unroll
    for (int r = 0; r < 2; r++) {
        const Row2d<T> q = row(r);
        const T u[4] = {q.gy[0], q.gy[1], q.gy[2], edge ? T(0) : q.gy[3]};
        const T y0 = u[0] * w[0] + u[1] * w[1] + u[2] * w[2] + u[3] * w[3];
        const T y1 = u[0] * dw[0] + u[1] * dw[1] + u[2] * dw[2] + u[3] * dw[3];
        const T du = q.phi[1] - q.phi[0], p = q.phi[0] - ref;
        const T x0 = p + du * bx.w[1] + q.gx[0] * bx.w[2] + q.gx[1] * bx.w[3];
        const T x1 = du * bx.dw[1] + q.gx[0] * bx.dw[2] + q.gx[1] * bx.dw[3];
        h += x0 * by.w[r];
        h += y0 * by.w[2 + r];
        hx += x1 * by.w[r];
        hx += y1 * by.w[2 + r];
        hy += x0 * by.dw[r];
        hy += y0 * by.dw[2 + r];
    }
    H = ref + h;
    Hx = hx;
    Hy = hy;
}

// Value and gradient of the bicubic of cell c at local coordinates xi, for any
// precision and cross-derivative rule, from the planes. FOLD as kFold2d, or false
// for the form with explicit cross derivatives.
template <typename T, int MIX, bool FOLD = kFold2d<T, MIX>>
__device__ __forceinline__ void bicubic(const Geom &g, Rsrc rphi, Rsrc rgx, Rsrc rgy, const int *c,
                                        const T *xi, T &H, T &Hx, T &Hy)
{
    if constexpr (FOLD) {
        const unsigned o = unsigned(c[1]) * unsigned(g.pitch) + unsigned(c[0]);
        const unsigned xm = c[0] == 0 ? 0u : 1u;
        Row2d<T> q[2];
#pragma unroll
        for (int r = 0; r < 2; r++) {
            const unsigned ro = o + (r ? unsigned(g.pitch) : 0u);
            bload4(rgy, ro - xm, q[r].gy);
            bload2(rphi, ro, q[r].phi);
            bload2(rgx, ro, q[r].gx);
        }
        bicubic_central<T>(
            g, c[0], xi, [&](int r) { return q[r]; },
            [&](int vx, int vy) {
                const T a = vx ? q[0].phi[1] : q[0].phi[0], b = vx ? q[1].phi[1] : q[1].phi[0];
                return vy ? b : a;
            },
            H, Hx, Hy);
    } else {
        T d[4][4];
        gather2d<T, MIX>(g, rphi, rgx, rgy, c[0], c[1], d);
        Basis<T> bx, by;
        basis<T, false>(xi[0], geo_h<T>(g, 0), geo_ih<T>(g, 0), bx);
        basis<T, false>(xi[1], geo_h<T>(g, 1), geo_ih<T>(g, 1), by);
        hermite2d(d, bx, by, H, Hx, Hy);
    }
}

// Value and gradient of the tricubic of cell c at local coordinates xi, for
// any cross-derivative rule.
template <typename T, int MIX>
__device__ __forceinline__ void tricubic(const Geom &g, Rsrc rphi, Rsrc rgx, Rsrc rgy, Rsrc rgz,
                                         const int *c, const T *xi, T &H, T *G)
{
    if constexpr (MIX == GALS_MIXED_CENTRAL) {
        tricubic_central<T, false>(g, rphi, rgx, rgy, rgz, c, xi, H, G, nullptr);
    } else {
        T d[8][8];
        gather3d<T, MIX>(g, rphi, rgx, rgy, rgz, c[0], c[1], c[2], d);
        Basis<T> b[3];
#pragma unroll
        for (int a = 0; a < 3; a++) basis<T, false>(xi[a], geo_h<T>(g, a), geo_ih<T>(g, a), b[a]);
        hermite3d(d, b[0], b[1], b[2], H, G[0], G[1], G[2]);
    }
}

}  // namespace gals
