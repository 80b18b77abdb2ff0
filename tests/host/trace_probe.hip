// Host build of the step kernels' characteristic trace: the device functions of
// the headers are compiled for the CPU, so their rounding can be measured there.
#include <hip/hip_runtime.h>
#include <math.h>

#undef __device__
#define __device__ __attribute__((host)) __attribute__((device))
__attribute__((host)) static inline void sincospi(double x, double *s, double *c)
{
    const long double pi = 3.14159265358979323846264338327950288L;
    *s = double(sinl(pi * x));
    *c = double(cosl(pi * x));
}
__attribute__((host)) static inline void sincospif(float x, float *s, float *c)
{
    double ds, dc;
    sincospi(double(x), &ds, &dc);
    *s = float(ds);
    *c = float(dc);
}
#include "hermite.h"

using namespace gals;

// plain: the general trace; otherwise the one the step kernels take. x, X: n x D,
// J: n x D x D.
template <typename T, int D, int KIND>
static void run(int plain, int n, const double *x, double dt, const double *c, double *X, double *J)
{
    static Vel<T> p;
    const Stage<T> st = make_stage<T>(dt, c[0], c[1], c[2]);
    for (int k = 0; k < n; k++) {
        T Jk[D * D];
        const int64_t ti[3] = {0, 0, 0};
        if (plain) trace<T, D, KIND, true>(p, st, dt, x + D * k, X + D * k, Jk);
        else trace_node<T, D, KIND, true>(p, st, dt, nullptr, ti, x + D * k, X + D * k, Jk);
        for (int q = 0; q < D * D; q++) J[D * D * k + q] = double(Jk[q]);
    }
}

extern "C" void probe(int f32, int dim, int plain, int n, const double *x, double dt,
                      const double *c, double *X, double *J)
{
    if (dim == 3) {
        if (f32) run<float, 3, GALS_VEL_LEVEQUE3D>(plain, n, x, dt, c, X, J);
        else run<double, 3, GALS_VEL_LEVEQUE3D>(plain, n, x, dt, c, X, J);
    } else {
        if (f32) run<float, 2, GALS_VEL_VORTEX>(plain, n, x, dt, c, X, J);
        else run<double, 2, GALS_VEL_VORTEX>(plain, n, x, dt, c, X, J);
    }
}
