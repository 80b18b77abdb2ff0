// Point evaluation (value, normal, curvature) and deterministic FP64
// reductions (error norms, shape error, volume, max speed) for gfx950.
#include "hermite.h"
#include "reduce.h"

namespace gals {

constexpr int64_t kEvalMaxBlocks = int64_t(1) << 20;

// ---------------------------------------------------------------------------
// Point evaluation (sec. 3.2): n = grad H / |grad H|, and the curvature
// kappa = div n = (|g|^2 tr(Hess) - g^T Hess g) / |g|^3, which is eq.
// (curvature) in 2D and the sum of the principal curvatures in 3D.
// ---------------------------------------------------------------------------
template <typename T, int D, int MIX>
__device__ __forceinline__ void eval_point(const Geom &g, const T *__restrict__ phi,
                                           const T *__restrict__ grad,
                                           const double *__restrict__ pts, int64_t npts,
                                           int64_t id, T *__restrict__ val,
                                           T *__restrict__ normal, T *__restrict__ curv)
{
    double X[D];
#pragma unroll
    for (int a = 0; a < D; a++) X[a] = pts[a * npts + id];
    int cell[D];
    double xi[D];
    split<D>(g, X, cell, xi);
    T H, G[D], Hs[D * D];
    T x[D];
#pragma unroll
    for (int a = 0; a < D; a++) x[a] = T(xi[a]);
    if constexpr (D == 3 && MIX == GALS_MIXED_CENTRAL) {
        tricubic_central<T, true>(g, plane_rsrc(phi, g.span), plane_rsrc(grad, g.span),
                                  plane_rsrc(grad + g.plane, g.span),
                                  plane_rsrc(grad + 2 * g.plane, g.span), cell, x, H, G, Hs);
    } else {
        Basis<T> b[D];
#pragma unroll
        for (int a = 0; a < D; a++) basis<T, true>(x[a], geo_h<T>(g, a), geo_ih<T>(g, a), b[a]);
        if constexpr (D == 2) {
            T d[4][4];
            gather2d<T, MIX>(g, plane_rsrc(phi, g.plane), plane_rsrc(grad, g.plane),
                             plane_rsrc(grad + g.plane, g.plane), cell[0], cell[1], d);
            hermite2d_full(d, b[0], b[1], H, G, Hs);
        } else {
            T d[8][8];
            gather3d<T, MIX>(g, plane_rsrc(phi, g.plane), plane_rsrc(grad, g.plane),
                             plane_rsrc(grad + g.plane, g.plane),
                             plane_rsrc(grad + 2 * g.plane, g.plane), cell[0], cell[1], cell[2], d);
            hermite3d_full(d, b[0], b[1], b[2], H, G, Hs);
        }
    }
    T g2 = T(0), tr = T(0), gHg = T(0);
#pragma unroll
    for (int a = 0; a < D; a++) {
        g2 += G[a] * G[a];
        tr += Hs[a * D + a];
#pragma unroll
        for (int c = 0; c < D; c++) gHg += G[a] * Hs[a * D + c] * G[c];
    }
    const bool ok = g2 > T(0);
    const T nrm = sqrt(g2);
    if (val) val[id] = H;
    if (normal) {
#pragma unroll
        for (int a = 0; a < D; a++) normal[a * npts + id] = ok ? G[a] / nrm : T(0);
    }
    if (curv) curv[id] = ok ? (g2 * tr - gHg) / (g2 * nrm) : T(0);
}

template <typename T, int D, int MIX>
__global__ __launch_bounds__(kBlock) void k_eval(Geom g, const T *__restrict__ phi,
                                                 const T *__restrict__ grad,
                                                 const double *__restrict__ pts, int64_t npts,
                                                 T *__restrict__ val, T *__restrict__ normal,
                                                 T *__restrict__ curv)
{
    // grid-stride over the points: the launch caps its grid (eval_typed), so
    // any count the entry point accepts fits the launch's work-item count
    for (int64_t id = int64_t(blockIdx.x) * kBlock + threadIdx.x; id < npts;
         id += int64_t(gridDim.x) * kBlock)
        eval_point<T, D, MIX>(g, phi, grad, pts, npts, id, val, normal, curv);
}

template <typename T, int MIX>
static hipError_t eval_typed(const gals_ctx *ctx, const void *phi, const void *grad,
                             const double *pts, int64_t npts, void *val, void *normal, void *curv,
                             hipStream_t s)
{
    // at most 2^20 blocks of 256 (2^28 work items); larger counts loop
    const int64_t want = (npts + kBlock - 1) / kBlock;
    const unsigned blocks = unsigned(want < kEvalMaxBlocks ? want : kEvalMaxBlocks);
    if (ctx->dim == 2)
        hipLaunchKernelGGL((k_eval<T, 2, MIX>), dim3(blocks), dim3(kBlock), 0, s, ctx->g,
                           (const T *)phi, (const T *)grad, pts, npts, (T *)val, (T *)normal,
                           (T *)curv);
    else
        hipLaunchKernelGGL((k_eval<T, 3, MIX>), dim3(blocks), dim3(kBlock), 0, s, ctx->g,
                           (const T *)phi, (const T *)grad, pts, npts, (T *)val, (T *)normal,
                           (T *)curv);
    return hipGetLastError();
}

hipError_t launch_eval(const gals_ctx *ctx, const void *phi, const void *grad, const double *pts,
                       int64_t npts, void *val, void *normal, void *curv, hipStream_t s)
{
    if (npts == 0) return hipSuccess;
#define GALS_EVAL(T, M) eval_typed<T, M>(ctx, phi, grad, pts, npts, val, normal, curv, s)
    if (ctx->prec == GALS_F32)
        return ctx->mixed == GALS_MIXED_ZERO   ? GALS_EVAL(float, GALS_MIXED_ZERO)
               : ctx->mixed == GALS_MIXED_CELL ? GALS_EVAL(float, GALS_MIXED_CELL)
                                               : GALS_EVAL(float, GALS_MIXED_CENTRAL);
    return ctx->mixed == GALS_MIXED_ZERO   ? GALS_EVAL(double, GALS_MIXED_ZERO)
           : ctx->mixed == GALS_MIXED_CELL ? GALS_EVAL(double, GALS_MIXED_CELL)
                                           : GALS_EVAL(double, GALS_MIXED_CENTRAL);
#undef GALS_EVAL
}

// Offset of node id in a plane: 32-bit, by the row length's magic number (the
// host keeps nodes below 2^31 and planes below 2 GiB; rows of 3D planes are
// contiguous in (j, k)).
__device__ __forceinline__ unsigned node_offset(const Geom &g, unsigned id)
{
    unsigned i;
    const unsigned r = udiv_magic(id, unsigned(g.n[0]), g.n_magic[0], i);
    return r * unsigned(g.pitch) + i;
}

// slots: 0 max|dphi| 1 max|dpsi| 2 sum|dH| 3 max band 4 sum H(-phi)
//        5 sum H(-phi_ref) 6 nonfinite count 7 max|phi_ref|
constexpr unsigned kNormsMax = (1u << 0) | (1u << 1) | (1u << 3) | (1u << 7);

// Two nodes a pass, their loads issued together; per thread the nodes are summed
// in the order of their ids. Bound: the two states' bytes. 2049^2 FP32 (100 MB):
// 32 us with 64-bit divisions and one node a pass, 23 with this.
template <typename T, int D>
__global__ __launch_bounds__(kBlock) void k_norms(Geom g, const T *__restrict__ phi,
                                                  const T *__restrict__ grad,
                                                  const T *__restrict__ phr,
                                                  const T *__restrict__ grr, double eps,
                                                  double band, double *__restrict__ partials)
{
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    const unsigned stride = gridDim.x * unsigned(kBlock), nodes = unsigned(g.nodes);
    auto add = [&](const T *u, const T *w) {
        const double p = double(u[0]), r = double(w[0]);
        const double e = fabs(p - r);
        acc[0] = fmax(acc[0], e);
        double nf = isfinite(p) ? 0.0 : 1.0;
#pragma unroll
        for (int a = 0; a < D; a++) {
            const double q = double(u[1 + a]);
            acc[1] = fmax(acc[1], fabs(q - double(w[1 + a])));
            nf += isfinite(q) ? 0.0 : 1.0;
        }
        acc[2] += fabs(heaviside_eps(p, eps) - heaviside_eps(r, eps));
        if (fabs(r) <= band) acc[3] = fmax(acc[3], e);
        acc[4] += heaviside_eps(-p, eps);
        acc[5] += heaviside_eps(-r, eps);
        acc[6] += nf;
        acc[7] = fmax(acc[7], fabs(r));
    };
    auto load = [&](unsigned id, T *u, T *w) {
        const unsigned o = node_offset(g, id);
        u[0] = phi[o];
        w[0] = phr[o];
#pragma unroll
        for (int a = 0; a < D; a++) {
            u[1 + a] = grad[a * g.plane + o];
            w[1 + a] = grr[a * g.plane + o];
        }
    };
    // nodes and stride are below 2^31 and 2^19: id + 2 stride does not wrap
    for (unsigned id = blockIdx.x * unsigned(kBlock) + threadIdx.x; id < nodes; id += 2 * stride) {
        T u[2][1 + D], w[2][1 + D];
        load(id, u[0], w[0]);
        if (id + stride < nodes) {
            load(id + stride, u[1], w[1]);
            add(u[0], w[0]);
            add(u[1], w[1]);
        } else {
            add(u[0], w[0]);
        }
    }
    block_reduce<8>(acc, kNormsMax, partials + int64_t(blockIdx.x) * kRedSlots);
}

hipError_t launch_norms(const gals_ctx *ctx, const void *phi, const void *grad,
                        const void *phi_ref, const void *grad_ref, double eps, double band,
                        double *partials, double *out, hipStream_t s)
{
#define GALS_NORMS(T, D)                                                                           \
    hipLaunchKernelGGL((k_norms<T, D>), dim3(kRedBlocks), dim3(kBlock), 0, s, ctx->g,              \
                       (const T *)phi, (const T *)grad, (const T *)phi_ref, (const T *)grad_ref,   \
                       eps, band, partials)
    if (ctx->prec == GALS_F32) {
        if (ctx->dim == 2) GALS_NORMS(float, 2);
        else GALS_NORMS(float, 3);
    } else {
        if (ctx->dim == 2) GALS_NORMS(double, 2);
        else GALS_NORMS(double, 3);
    }
#undef GALS_NORMS
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_fold<8>, dim3(1), dim3(kBlock), 0, s, partials, kRedBlocks, kNormsMax,
                       out);
    return hipGetLastError();
}

// max over nodes of |v(x_node, t)|, c = c(t). The square root is monotone, so
// it is taken once, of the largest square.
template <typename T, int D>
__device__ __forceinline__ double speed2(const T *v)
{
    double s = 0.0;
#pragma unroll
    for (int a = 0; a < D; a++) s += double(v[a]) * double(v[a]);
    return s;
}

template <typename T, int D, int KIND>
__global__ __launch_bounds__(kBlock) void k_max_speed(Geom g, Vel<T> p, T c,
                                                      double *__restrict__ partials)
{
    double acc[1] = {0.0};
    const unsigned stride = gridDim.x * unsigned(kBlock), nodes = unsigned(g.nodes);
    for (unsigned id = blockIdx.x * unsigned(kBlock) + threadIdx.x; id < nodes; id += stride) {
        unsigned idx[3], r = udiv_magic(id, unsigned(g.n[0]), g.n_magic[0], idx[0]);
        if constexpr (D == 3) idx[2] = udiv_magic(r, unsigned(g.n[1]), g.n_magic[1], idx[1]);
        else idx[1] = r;
        double x[D];
#pragma unroll
        for (int a = 0; a < D; a++) x[a] = node_coord(g.lo[a], idx[a], g.h[a]);
        T v[D], J[D * D];
        velocity<T, D, KIND>(p, x, c, v, J);
        acc[0] = fmax(acc[0], speed2<T, D>(v));
    }
    acc[0] = sqrt(acc[0]);
    block_reduce<1>(acc, 1u, partials + int64_t(blockIdx.x) * kRedSlots);
}

// The same for a sine stream function, in tiles of kBlock columns x kSpeedRows
// rows: a thread keeps its column's sines and cosines, the block the tile's row
// sums P_m = sum_n S sin(n pi y), Q_m = sum_n S (n pi) cos(n pi y) in LDS, and a
// node is eight multiply-adds, those of stream_modes in its order. 2049^2 FP32:
// 26 us with both sines and the row sums at every node, 7 with this. On grids of a
// few columns most of a tile's threads have none: from kSpeedColumns on (us per
// call, node by node / in tiles, FP64: 3 x 2000001 52 / 146, 8 x 1000001 62 / 84, 32 x
// 400001 104 / 47; FP32: 40 / 130, 45 / 75, 80 / 43).
constexpr int kSpeedRows = 32, kSpeedColumns = 12;

template <typename T>
__global__ __launch_bounds__(kBlock) void k_max_speed_stream(Geom g, Vel<T> p, T c,
                                                             double *__restrict__ partials)
{
    __shared__ T rows[kSpeedRows][8];  // P_m, Q_m
    double acc[1] = {0.0};
    const unsigned tx = (unsigned(g.n[0]) + kBlock - 1) / kBlock;
    const unsigned ty = (unsigned(g.n[1]) + kSpeedRows - 1) / kSpeedRows;
    for (uint64_t t = blockIdx.x; t < uint64_t(tx) * ty; t += gridDim.x) {
        const int i = int(t % tx) * kBlock + int(threadIdx.x), j0 = int(t / tx) * kSpeedRows;
        const int nrows = g.n[1] - j0 < kSpeedRows ? g.n[1] - j0 : kSpeedRows;
        __syncthreads();  // the previous tile's rows are read
        if (int(threadIdx.x) < nrows) {
            T sy[4], cy[4], qy[4];
            sincos_multiples(T(node_coord(g.lo[1], j0 + int(threadIdx.x), g.h[1])), sy, cy);
#pragma unroll
            for (int n = 0; n < 4; n++) qy[n] = T((n + 1) * kPi) * cy[n];
#pragma unroll
            for (int m = 0; m < 4; m++) {
                T P = 0, Q = 0;
#pragma unroll
                for (int n = 0; n < 4; n++) {
                    P += p.S[m][n] * sy[n];
                    Q += p.S[m][n] * qy[n];
                }
                rows[threadIdx.x][m] = P;
                rows[threadIdx.x][4 + m] = Q;
            }
        }
        __syncthreads();
        if (i < g.n[0]) {
            T sx[4], cx[4], kc[4];
            sincos_multiples(T(node_coord(g.lo[0], i, g.h[0])), sx, cx);
#pragma unroll
            for (int m = 0; m < 4; m++) kc[m] = T((m + 1) * kPi) * cx[m];
            for (int r = 0; r < nrows; r++) {
                T fx = 0, fy = 0;
#pragma unroll
                for (int m = 0; m < 4; m++) {
                    fx += kc[m] * rows[r][m];
                    fy += sx[m] * rows[r][4 + m];
                }
                const T v[2] = {-c * fy, c * fx};
                acc[0] = fmax(acc[0], speed2<T, 2>(v));
            }
        }
    }
    acc[0] = sqrt(acc[0]);
    block_reduce<1>(acc, 1u, partials + int64_t(blockIdx.x) * kRedSlots);
}

template <typename T>
static hipError_t max_speed_typed(const gals_ctx *ctx, const Vel<T> &p, double c,
                                  double *partials, hipStream_t s)
{
    const dim3 grid(kRedBlocks), block(kBlock);
    const T cc = T(c);
    switch (ctx->dim * 16 + ctx->vel_kind) {
    case 2 * 16 + GALS_VEL_AFFINE:
        hipLaunchKernelGGL((k_max_speed<T, 2, GALS_VEL_AFFINE>), grid, block, 0, s, ctx->g, p, cc, partials);
        break;
    case 2 * 16 + GALS_VEL_STREAM_SIN:
        if (ctx->g.n[0] < kSpeedColumns)
            hipLaunchKernelGGL((k_max_speed<T, 2, GALS_VEL_STREAM_SIN>), grid, block, 0, s, ctx->g, p, cc, partials);
        else
            hipLaunchKernelGGL((k_max_speed_stream<T>), grid, block, 0, s, ctx->g, p, cc, partials);
        break;
    case 2 * 16 + GALS_VEL_VORTEX:
        hipLaunchKernelGGL((k_max_speed<T, 2, GALS_VEL_VORTEX>), grid, block, 0, s, ctx->g, p, cc, partials);
        break;
    case 2 * 16 + GALS_VEL_PSEUDO1D:
        hipLaunchKernelGGL((k_max_speed<T, 2, GALS_VEL_PSEUDO1D>), grid, block, 0, s, ctx->g, p, cc, partials);
        break;
    case 3 * 16 + GALS_VEL_AFFINE:
        hipLaunchKernelGGL((k_max_speed<T, 3, GALS_VEL_AFFINE>), grid, block, 0, s, ctx->g, p, cc, partials);
        break;
    case 3 * 16 + GALS_VEL_VECPOT_SIN:
        hipLaunchKernelGGL((k_max_speed<T, 3, GALS_VEL_VECPOT_SIN>), grid, block, 0, s, ctx->g, p, cc, partials);
        break;
    case 3 * 16 + GALS_VEL_LEVEQUE3D:
        hipLaunchKernelGGL((k_max_speed<T, 3, GALS_VEL_LEVEQUE3D>), grid, block, 0, s, ctx->g, p, cc, partials);
        break;
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_max_speed(const gals_ctx *ctx, double c, double *partials, double *out,
                            hipStream_t s)
{
    hipError_t e = ctx->prec == GALS_F32 ? max_speed_typed<float>(ctx, ctx->vf, c, partials, s)
                                         : max_speed_typed<double>(ctx, ctx->vd, c, partials, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_fold<1>, dim3(1), dim3(kBlock), 0, s, partials, kRedBlocks, 1u, out);
    return hipGetLastError();
}

}  // namespace gals
