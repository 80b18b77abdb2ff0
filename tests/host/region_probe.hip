// Host build of the several-steps kernel's plan and regions: every node that a
// block updates is traced on the CPU and the stencil of its foot's cell looked up
// in the region that the block stages for that step.
#include <hip/hip_runtime.h>
#include <math.h>
#include <string.h>

#undef __device__
#define __device__ __attribute__((host)) __attribute__((device))
__attribute__((host)) static inline int __all(int p) { return p; }
__attribute__((host)) static inline void sincospi(double x, double *s, double *c)
{
    *s = sin(3.14159265358979323846 * x);
    *c = cos(3.14159265358979323846 * x);
}
__attribute__((host)) static inline void sincospif(float x, float *s, float *c)
{
    *s = sinf(3.14159265f * x);
    *c = cosf(3.14159265f * x);
}
// no kernel is launched, so none has to be registered
#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(...) (void)0
#include "multi2d.hip"

using namespace gals;

// cells outside the staged region, over all tiles and steps of a launch
template <typename T, class F, class Foot>
static long outside(const Geom &g, const F &f, int k, Foot foot)
{
    long bad = 0;
    const dim3 grid = multi_grid(g);
    for (unsigned by = 0; by < grid.y; by++)
        for (unsigned bx = 0; bx < grid.x; bx++) {
            Region reg[kMultiMax + 1], r;
            r.x0 = int(bx) * kTileX;
            r.y0 = int(by) * kTileY;
            r.x1 = r.x0 + kTileX < g.n[0] ? r.x0 + kTileX - 1 : g.n[0] - 1;
            r.y1 = r.y0 + kTileY < g.n[1] ? r.y0 + kTileY - 1 : g.n[1] - 1;
            for (int s = k - 1; s >= 0; s--) {
                reg[s + 1] = r;
                r = f.source(g, s, r);
            }
            reg[0] = r;
            for (int s = 0; s < k; s++) {
                const Region &R = reg[s], &Q = reg[s + 1];
                for (int j = Q.y0; j <= Q.y1; j++)
                    for (int i = Q.x0; i <= Q.x1; i++) {
                        int c[2];
                        foot(s, i, j, c);
                        const int x0 = c[0] > 0 ? c[0] - 1 : 0;
                        const int x1 = c[0] + 2 < g.n[0] ? c[0] + 2 : g.n[0] - 1;
                        bad += x0 < R.x0 || x1 > R.x1 || c[1] < R.y0 || c[1] + 1 > R.y1;
                    }
            }
        }
    return bad;
}

template <typename T>
static long run(const gals_ctx &ctx, const Vel<T> &p, double t0, double dt, int *k)
{
    const int most = *k = multi_steps(&ctx, dt);
    if (most == 1) return 0;
    double c[kMultiMax][3];
    for (int q = 0; q < most; q++) {
        const double t = t0 + q * dt, w = ctx.period > 0.0 ? kPi / ctx.period : 0.0;
        c[q][0] = cos(w * (t + dt));
        c[q][1] = cos(w * t);
        c[q][2] = cos(w * (t + 0.5 * dt));
    }
    const Geom &g = ctx.g;
    int cap, updates, passes;
    size_t bytes;
    if (ctx.vel_kind == GALS_VEL_AFFINE) {
        AffineSteps<T> f;
        fill_steps(&ctx, p, most, c, dt, f);
        while (*k > 1 && !multi_plan<T>(g, f, *k, cap, bytes, updates, passes)) --*k;
        if (*k == 1) return 0;
        return outside<T>(g, f, *k, [&](int s, int i, int j, int *cell) {
            T xi[2];
            bool out[2];
            affine_foot(g, f.m[s], i, j, cell, xi, out);
        });
    }
    StreamSteps<T> f;
    fill_steps(&ctx, p, most, c, dt, f);
    while (*k > 1 && !multi_plan<T>(g, f, *k, cap, bytes, updates, passes)) --*k;
    if (*k == 1) return 0;
    return outside<T>(g, f, *k, [&](int s, int i, int j, int *cell) {
        T U[kJet] = {}, Y[kJet] = {};
        for (int n = 0; n < 4; n++) {
            const double y = node_coord(g.lo[1], j, g.h[1]), x = node_coord(g.lo[0], i, g.h[0]);
            for (int a = 0; a < 5; a++) {
                double u = 0.0;
                for (int m = 0; m < 4; m++)
                    u += ctx.vd.S[m][n] * pow((m + 1) * kPi, a) * sin((m + 1) * kPi * x + a * kPi / 2);
                U[4 * a + n] = T(u);
                Y[4 * a + n] = T(pow((n + 1) * kPi, a) * sin((n + 1) * kPi * y + a * kPi / 2));
            }
        }
        double sn, cs;
        sincospi(node_coord(g.lo[0], i, g.h[0]), &sn, &cs);
        U[kJetTaylor] = T(sn), U[kJetTaylor + 1] = T(cs);
        sincospi(node_coord(g.lo[1], j, g.h[1]), &sn, &cs);
        Y[kJetTaylor] = T(sn), Y[kJetTaylor + 1] = T(cs);
        StreamFoot<T> ft;
        stream_trace<T, sizeof(T) == 4, true>(g, f, f.st[s], dt, U, Y, i, j, ft);
        cell[0] = ft.cell[0];
        cell[1] = ft.cell[1];
    });
}

// par: affine b[2], c[2], A[4]; stream function S[16]. Returns the nodes whose
// cells lie outside their region; *k: the steps of the launch (1: none).
extern "C" long probe(int f32, int affine, int bc, const long *ncell, const double *lo,
                      const double *hi, const double *par, double period, double t0, double dt,
                      int *k)
{
    static gals_ctx ctx;
    memset(&ctx, 0, sizeof ctx);
    Geom &g = ctx.g;
    g.dim = ctx.dim = 2;
    g.bc = bc;
    g.nodes = 1;
    for (int a = 0; a < 3; a++) {
        g.nc[a] = a < 2 ? int(ncell[a]) : 0;
        g.n[a] = g.nc[a] + 1;
        g.lo[a] = a < 2 ? lo[a] : 0.0;
        g.h[a] = a < 2 ? (hi[a] - lo[a]) / double(ncell[a]) : 1.0;
        g.inv_h[a] = 1.0 / g.h[a];
        g.top[a] = node_coord(g.lo[a], g.nc[a], g.h[a]);
        g.nodes *= g.n[a];
    }
    geom_finish(g);
    ctx.prec = f32 ? GALS_F32 : GALS_F64;
    ctx.period = period;
    ctx.vel_kind = affine ? GALS_VEL_AFFINE : GALS_VEL_STREAM_SIN;
    if (affine) {
        for (int i = 0; i < 2; i++) {
            ctx.vd.b[i] = par[i];
            ctx.vd.c[i] = ctx.vf.c[i] = par[2 + i];
            ctx.vf.b[i] = float(par[i]);
            for (int j = 0; j < 2; j++) {
                ctx.vd.A[3 * i + j] = par[4 + 2 * i + j];
                ctx.vf.A[3 * i + j] = float(par[4 + 2 * i + j]);
            }
        }
    } else {
        int mx = 0, nx = 0;
        for (int q = 0; q < 16; q++) {
            ctx.vd.S[q / 4][q % 4] = par[q];
            ctx.vf.S[q / 4][q % 4] = float(par[q]);
            if (par[q] != 0.0) {
                mx = q / 4 + 1 > mx ? q / 4 + 1 : mx;
                nx = q % 4 + 1 > nx ? q % 4 + 1 : nx;
            }
        }
        ctx.vd.kx = kPi * mx, ctx.vd.ky = kPi * nx;
        ctx.vf.kx = float(kPi * mx), ctx.vf.ky = float(kPi * nx);
    }
    return f32 ? run<float>(ctx, ctx.vf, t0, dt, k) : run<double>(ctx, ctx.vd, t0, dt, k);
}
