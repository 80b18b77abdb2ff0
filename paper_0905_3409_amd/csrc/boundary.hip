// Inflow boundary conditions (boundary.h) as launches of their own after a step,
// one thread per boundary node (each node counted once), a few thousand threads
// against the step's millions of nodes.
#include "boundary.h"

namespace gals {

// ---------------------------------------------------------------------------
// Boundary enumeration: faces in the order (axis 0 low, axis 0 high, axis 1
// low, ...); face (a, side) holds nodes / n[a] nodes, the other axes in
// increasing order, fastest first. A node that also lies on a face of a lower
// axis belongs to that face and is skipped here.
// ---------------------------------------------------------------------------
int64_t boundary_count(const Geom &g)
{
    int64_t c = 0;
    for (int a = 0; a < g.dim; a++) c += 2 * (g.nodes / g.n[a]);
    return c;
}

template <int D>
__device__ __forceinline__ bool boundary_node(const Geom &g, int64_t id, int *ijk)
{
#pragma unroll
    for (int a = 0; a < D; a++) {
        const int64_t cnt = g.nodes / g.n[a];
        if (id < 2 * cnt) {
            const bool high = id >= cnt;
            int64_t r = high ? id - cnt : id;
#pragma unroll
            for (int b = 0; b < D; b++) {
                if (b == a) {
                    ijk[b] = high ? g.nc[a] : 0;
                } else {
                    ijk[b] = int(r % g.n[b]);
                    r /= g.n[b];
                }
            }
#pragma unroll
            for (int b = 0; b < a; b++)
                if (ijk[b] == 0 || ijk[b] == g.nc[b]) return false;
            return true;
        }
        id -= 2 * cnt;
    }
    return false;
}

template <typename T, int D, int KIND>
__global__ __launch_bounds__(kBlock) void k_inflow(Geom g, Vel<T> p, T c, double dt,
                                                   int64_t count, InflowData<T> b, T *phi,
                                                   T *grad)
{
    // phi and grad may hold the data themselves
    const int64_t id = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    int ijk[3] = {0, 0, 0};
    if (id >= count || !boundary_node<D>(g, id, ijk)) return;
    inflow_node<T, D, KIND>(g, p, c, dt, ijk, b, phi, grad);
}

template <typename T, int D, int KIND, int MIX>
__global__ __launch_bounds__(kBlock) void k_face(Geom g, Vel<T> p, Stage<T> st, double dt,
                                                 int64_t count, const T *__restrict__ sphi,
                                                 const T *__restrict__ sgrad,
                                                 T *__restrict__ dphi, T *__restrict__ dgrad)
{
    const int64_t id = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    int ijk[3] = {0, 0, 0};
    if (id >= count || !boundary_node<D>(g, id, ijk)) return;
    face_node<T, D, KIND, MIX>(g, p, st, dt, ijk, sphi, sgrad, dphi, dgrad);
}

// ---------------------------------------------------------------------------
// Launchers.
// ---------------------------------------------------------------------------
// The vortex and the 1D-like field come here only with data that lie in the
// state the step writes: their step kernel (k_step2d) treats its boundary nodes
// itself otherwise.
#define GALS_INFLOW_KINDS(X)                                                                      \
    GALS_BOUNDARY_KINDS(X)                                                                        \
    X(2, GALS_VEL_VORTEX)                                                                         \
    X(2, GALS_VEL_PSEUDO1D)
#define GALS_BOUNDARY_KINDS(X)                                                                    \
    X(2, GALS_VEL_AFFINE)                                                                         \
    X(2, GALS_VEL_STREAM_SIN)                                                                     \
    X(3, GALS_VEL_AFFINE)                                                                         \
    X(3, GALS_VEL_VECPOT_SIN)                                                                     \
    X(3, GALS_VEL_LEVEQUE3D)

template <typename T>
static hipError_t inflow_typed(const gals_ctx *ctx, const Vel<T> &p, void *phi, void *grad,
                               double c, double dt, hipStream_t s)
{
    const int64_t count = boundary_count(ctx->g);
    const dim3 grid(unsigned((count + kBlock - 1) / kBlock)), block(kBlock);
    const T cc = T(c);
    T *ph = (T *)phi, *gr = (T *)grad;
    const InflowData<T> b = inflow_data<T>(ctx);
#define GALS_INFLOW(D, K)                                                                         \
    case D * 16 + K:                                                                              \
        hipLaunchKernelGGL((k_inflow<T, D, K>), grid, block, 0, s, ctx->g, p, cc, dt, count, b,   \
                           ph, gr);                                                               \
        break;
    switch (ctx->dim * 16 + ctx->vel_kind) {
        GALS_INFLOW_KINDS(GALS_INFLOW)
    default:
        return hipErrorInvalidValue;
    }
#undef GALS_INFLOW
    return hipGetLastError();
}

hipError_t launch_inflow(const gals_ctx *ctx, void *phi, void *grad, double c, double dt,
                         hipStream_t s)
{
    return ctx->prec == GALS_F32 ? inflow_typed<float>(ctx, ctx->vf, phi, grad, c, dt, s)
                                 : inflow_typed<double>(ctx, ctx->vd, phi, grad, c, dt, s);
}

template <typename T, int MIX>
static hipError_t face_typed(const gals_ctx *ctx, const Vel<T> &p, const void *sphi,
                             const void *sgrad, void *dphi, void *dgrad, double dt, double c1,
                             double c2, double c3, hipStream_t s)
{
    const int64_t count = boundary_count(ctx->g);
    const dim3 grid(unsigned((count + kBlock - 1) / kBlock)), block(kBlock);
    const Stage<T> st = make_stage<T>(dt, c1, c2, c3);
    const T *sp = (const T *)sphi, *sg = (const T *)sgrad;
    T *dp = (T *)dphi, *dg = (T *)dgrad;
#define GALS_FACE(D, K)                                                                           \
    case D * 16 + K:                                                                              \
        hipLaunchKernelGGL((k_face<T, D, K, MIX>), grid, block, 0, s, ctx->g, p, st, dt, count,   \
                           sp, sg, dp, dg);                                                       \
        break;
    switch (ctx->dim * 16 + ctx->vel_kind) {
        GALS_BOUNDARY_KINDS(GALS_FACE)
    default:
        return hipErrorInvalidValue;
    }
#undef GALS_FACE
    return hipGetLastError();
}

template <typename T>
static hipError_t face_mix(const gals_ctx *ctx, const Vel<T> &p, const void *sphi,
                           const void *sgrad, void *dphi, void *dgrad, double dt, double c1,
                           double c2, double c3, hipStream_t s)
{
    if (ctx->mixed == GALS_MIXED_CELL)
        return face_typed<T, GALS_MIXED_CELL>(ctx, p, sphi, sgrad, dphi, dgrad, dt, c1, c2, c3, s);
    if (ctx->mixed == GALS_MIXED_ZERO)
        return face_typed<T, GALS_MIXED_ZERO>(ctx, p, sphi, sgrad, dphi, dgrad, dt, c1, c2, c3, s);
    return face_typed<T, GALS_MIXED_CENTRAL>(ctx, p, sphi, sgrad, dphi, dgrad, dt, c1, c2, c3, s);
}

hipError_t launch_face(const gals_ctx *ctx, const void *sphi, const void *sgrad, void *dphi,
                       void *dgrad, double dt, double c1, double c2, double c3, hipStream_t s)
{
    return ctx->prec == GALS_F32
               ? face_mix<float>(ctx, ctx->vf, sphi, sgrad, dphi, dgrad, dt, c1, c2, c3, s)
               : face_mix<double>(ctx, ctx->vd, sphi, sgrad, dphi, dgrad, dt, c1, c2, c3, s);
}

}  // namespace gals
