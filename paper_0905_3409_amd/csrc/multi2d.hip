// Several GA-CIR steps of a small 2D grid in one launch, for the fields whose
// feet can be bounded before the launch (affine fields, sine stream functions).
//
// A step of a small grid is a launch of 4 to 6 us whatever its arithmetic:
// wave start, cold kernel arguments, one chain of dependent loads, the flush at
// its end. A block here owns a tile of output nodes and carries k steps through
// LDS: it stages the region of the old state that the tile's value after k steps
// depends on, and recomputes the shrinking regions in between, redundantly with
// its neighbours and without any exchange with them. The regions are known
// before the data: a foot lies in the image of the node under the affine map,
// or within the field's largest displacement of it, and the stencil of its
// cell adds one column below and two above, no row below and one above.
//
// The recomputed nodes (up to 6.6 times the tile's) cost a chip with little else to do
// nothing. With eight grids at work, each on a stream of its own, a launch of several
// steps still gains or is even (us for 64 steps of all eight, one step a launch ->
// this: FP64 rotation 101^2 1490 -> 517, 181^2 1346 -> 606, 257^2 1381 -> 1052; stream
// function 101^2 FP64 1449 -> 1159, 181^2 FP32 1446 -> 830).
//
// The node arithmetic is the single step's (split_disp, split_cells,
// affine_values; stream_trace, stream_values; the same LDS or global gather
// values), so results agree bit for bit with steps launched one by one.
#include "affine2d.h"
#include "stream2d.h"

namespace gals {

// Tiles of 8 x 8 output nodes and four steps a launch. us per call, one step a
// launch -> this: 65^2 FP64 rotation (2.2 cells a step at the corners), 128
// steps 633 -> 271 (two steps a launch 363, six 277, eight 310; 16 x 8 tiles
// 302, 16 x 16 365); 101 x 94 FP32 stream function, 32 steps 173 -> 109.
constexpr int kTileX = 8, kTileY = 8;
constexpr int kMultiMax = kMultiSteps;
// Threads per block: 512 while the blocks are few (a CU each, or two), else 256
// (257^2 FP32 rotation, 64 steps: 234 us with 512, 195 with 256).
constexpr int kMultiThreads = 512;
constexpr unsigned kFewBlocks = 512;
// What a launch costs, and so how many steps it should take. A block updates
// its regions in passes of one node per thread; a launch takes about 3.5 us and
// 1.25 us per pass for an affine field, 1.9 us for a stream function in FP32,
// 3 us in FP64, while one step a launch takes 5 us. Affine fields: at most 1700
// node updates a block. Stream functions: at most 2 k - 2 passes for k steps in
// FP32, (3 k - 2) / 2 in FP64 (141 x 134 FP32 at 1.7 cells a step, 32 steps: 172
// us one step a launch, 133 three in 4 passes, 141 four in 8; 238 x 160 at 3.1,
// 28 steps: 128 one, 187 two in 4 passes; 38 x 32 FP64 at 3.1, 12 steps: 71 one,
// 79 two in 3 passes), and two steps a launch only up to a block per CU (187 x
// 147 FP32 at 3.1, 35 steps: 159 one, 183 two).
constexpr int kMaxUpdates = 1700;
// Largest grids taken. Beyond them the chip is full and the recomputed nodes
// cost more than the launches: affine FP32 351^2 152 -> 137 us per 32 steps,
// 513^2 174 -> 227; FP64 257^2 292 -> 228 per 64, 513^2 197 -> 300 per 32; stream
// function FP32 181^2 162 -> 126 per 32, 257^2 165 -> 163; FP64 157 x 81 184 ->
// 146 per 38, 138 x 163 143 -> 194 per 28 (more blocks than CUs).
constexpr int64_t kMaxNodesAffine32 = 1 << 17, kMaxNodesAffine64 = 80000;
constexpr int64_t kMaxNodesStream32 = 40000, kMaxNodesStream64 = 1 << 14;
constexpr size_t kMultiLds = 60 << 10;  // dynamic LDS a block may take
constexpr int kMaxWidth = 127;          // nodes of a staged region, per row and in all
constexpr int kMaxNodes = 8191;
constexpr int kPad = 4;                 // LDS elements before and after a buffer

// Inclusive node ranges.
struct Region {
    int x0, x1, y0, y1;
};

// The nodes that the stencils of feet in [ax, bx] x [ay, by] (cell units) read:
// cells clamped into the grid, as the feet's are. kSlack covers the rounding
// between this estimate and a node's own foot: an FP32 displacement of up to
// kMaxCells32 cells is off by at most 4.9e-4 (fill_steps refuses longer axes, and
// numbers for which a foot may be NaN).
constexpr int kMaxCells32 = 8192;
__host__ __device__ inline Region stencil_region(const Geom &g, double ax, double bx, double ay,
                                                 double by)
{
    constexpr double kSlack = 1e-3;
    auto cell = [&](int a, double s) { return int(fmin(fmax(floor(s), 0.0), g.lastc[a])); };
    const int c0 = cell(0, ax - kSlack), c1 = cell(0, bx + kSlack);
    const int r0 = cell(1, ay - kSlack), r1 = cell(1, by + kSlack);
    return Region{c0 > 0 ? c0 - 1 : 0, c1 + 2 < g.n[0] ? c1 + 2 : g.n[0] - 1, r0, r1 + 1};
}

// The nodes that a step of each field reads to compute region r.
template <typename T>
struct AffineSteps {
    AffineMap2<T> m[kMultiMax];
    __host__ __device__ Region source(const Geom &g, int s, const Region &r) const
    {
        const AffineMap2<T> &q = m[s];
        double lo[2], hi[2];
        for (int a = 0; a < 2; a++) {
            const double u = q.Mc[2 * a], v = q.Mc[2 * a + 1];
            lo[a] = q.kc[a] + u * double(u >= 0.0 ? r.x0 : r.x1) + v * double(v >= 0.0 ? r.y0 : r.y1);
            hi[a] = q.kc[a] + u * double(u >= 0.0 ? r.x1 : r.x0) + v * double(v >= 0.0 ? r.y1 : r.y0);
        }
        return stencil_region(g, lo[0], hi[0], lo[1], hi[1]);
    }
    // Nodes along each axis that a w x h region can need, wherever it lies.
    void grow(int s, int &w, int &h) const
    {
        const AffineMap2<T> &q = m[s];
        const double ex = fabs(q.Mc[0]) * (w - 1) + fabs(q.Mc[1]) * (h - 1);
        const double ey = fabs(q.Mc[2]) * (w - 1) + fabs(q.Mc[3]) * (h - 1);
        // a far-flung map needs the whole grid (multi_plan clips to it)
        w = ex < 1e6 ? int(ex + 0.01) + 5 : 1 << 20;
        h = ey < 1e6 ? int(ey + 0.01) + 3 : 1 << 20;
    }
};

template <typename T>
struct StreamSteps {
    Stage<T> st[kMultiMax];
    T S[4][4];
    T kx, ky;
    double bound[kMultiMax][2];  // largest displacement of a foot, in cells
    const T *coltab, *rowtab;
    __host__ __device__ Region source(const Geom &g, int s, const Region &r) const
    {
        return stencil_region(g, double(r.x0) - bound[s][0], double(r.x1) + bound[s][0],
                              double(r.y0) - bound[s][1], double(r.y1) + bound[s][1]);
    }
    void grow(int s, int &w, int &h) const
    {
        w = bound[s][0] < 1e6 ? w - 1 + int(2.0 * bound[s][0] + 0.01) + 5 : 1 << 20;
        h = bound[s][1] < 1e6 ? h - 1 + int(2.0 * bound[s][1] + 0.01) + 3 : 1 << 20;
    }
};

// One node of one step from the staged region R (node-interleaved, rows of w
// nodes): phi and the gradient into out.
template <typename T, int MIX, int PSI>
__device__ __forceinline__ void multi_node(const Geom &g, const AffineSteps<T> &f, int s, double dt,
                                           const T *buf, const Region &R, int w, int i, int j,
                                           T *out)
{
    const AffineMap2<T> &am = f.m[s];
    int cell[2];
    T xi[2];
    bool outb[2];
    affine_foot(g, am, i, j, cell, xi, outb);
    T H, Hx, Hy;
    const T *t = buf + 3 * ((cell[1] - R.y0) * w + (cell[0] - 1 - R.x0));
    bicubic_lds<T, MIX, false>(g, t, t + 3 * w, cell, xi, H, Hx, Hy);
    affine_values<T, PSI>(am, dt, outb, H, Hx, Hy, out);
}

template <typename T, int MIX, int PSI>
__device__ __forceinline__ void multi_node(const Geom &g, const StreamSteps<T> &f, int s, double dt,
                                           const T *buf, const Region &R, int w, int i, int j,
                                           T *out)
{
    const Stage<T> &st = f.st[s];
    const T *U = f.coltab + i * kJet, *Y = f.rowtab + j * kJet;
    StreamFoot<T> ft;
    stream_trace<T, sizeof(T) == 4, PSI == GALS_PSI_SUPERCONSISTENT>(g, f, st, dt, U, Y, i, j, ft);
    if constexpr (kFold2d<T, MIX> && PSI == GALS_PSI_SUPERCONSISTENT) pin4(ft.J);
    T H, Hx, Hy;
    const T *t = buf + 3 * ((ft.cell[1] - R.y0) * w + (ft.cell[0] - 1 - R.x0));
    bicubic_lds<T, MIX, kFold2d<T, MIX>>(g, t, t + 3 * w, ft.cell, ft.xi, H, Hx, Hy);
    stream_values<T, sizeof(T) == 4, PSI>(g, f, st, dt, U, Y, ft, H, Hx, Hy, i, j,
                                          [&](int q, T v) { out[q] = v; });
}

template <typename T, class F, int MIX, int PSI>
__global__ __launch_bounds__(kMultiThreads) void k_multi2d(Geom g, F f, int k, int cap, double dt,
                                                           const T *__restrict__ phi,
                                                           const T *__restrict__ grad,
                                                           T *__restrict__ phi_o,
                                                           T *__restrict__ grad_o)
{
    extern __shared__ double lds[];
    __shared__ Region reg[kMultiMax + 1];
    // kPad elements around each buffer: a gather at the grid's first and last
    // column reads one node beyond the region and drops the value
    T *const buf[2] = {reinterpret_cast<T *>(lds) + kPad, reinterpret_cast<T *>(lds) + cap + kPad};
    const int tid = int(threadIdx.x);
    Region r;
    r.x0 = int(blockIdx.x) * kTileX;
    r.y0 = int(blockIdx.y) * kTileY;
    r.x1 = r.x0 + kTileX < g.n[0] ? r.x0 + kTileX - 1 : g.n[0] - 1;
    r.y1 = r.y0 + kTileY < g.n[1] ? r.y0 + kTileY - 1 : g.n[1] - 1;
    for (int s = k - 1; s >= 0; s--) {
        if (tid == 0) reg[s + 1] = r;
        r = f.source(g, s, r);
    }
    if (tid == 0) reg[0] = r;
    // node (row, col) of entry e of a region w nodes wide: e / w by a multiply,
    // exact while e w < 2^20 (kMaxWidth, kMaxNodes)
    auto split_entry = [](int e, int w, int inv, int &row, int &col) {
        row = int((unsigned(e) * unsigned(inv)) >> 20);
        col = e - row * w;
    };
    {
        const int w = r.x1 - r.x0 + 1, n = w * (r.y1 - r.y0 + 1);
        const int inv = (1 << 20) / w + 1;
        for (int e = tid; e < n; e += int(blockDim.x)) {
            int row, col;
            split_entry(e, w, inv, row, col);
            const unsigned o = unsigned(r.y0 + row) * unsigned(g.pitch) + unsigned(r.x0 + col);
            buf[0][3 * e] = phi[o];
            buf[0][3 * e + 1] = grad[o];
            buf[0][3 * e + 2] = grad[g.plane + o];
        }
    }
    __syncthreads();
    for (int s = 0; s < k; s++) {
        const Region R = reg[s], Q = reg[s + 1];
        const int w = R.x1 - R.x0 + 1, wq = Q.x1 - Q.x0 + 1, n = wq * (Q.y1 - Q.y0 + 1);
        const int inv = (1 << 20) / wq + 1;
        const T *src = buf[s & 1];
        T *dst = buf[(s + 1) & 1];
        for (int e = tid; e < n; e += int(blockDim.x)) {
            int row, col;
            split_entry(e, wq, inv, row, col);
            T v[3];
            multi_node<T, MIX, PSI>(g, f, s, dt, src, R, w, Q.x0 + col, Q.y0 + row, v);
            if (s == k - 1) {
                const unsigned o = unsigned(Q.y0 + row) * unsigned(g.pitch) + unsigned(Q.x0 + col);
                pstore(phi_o, o, v[0]);
                pstore(grad_o, o, v[1]);
                pstore(grad_o + g.plane, o, v[2]);
            } else {
                dst[3 * e] = v[0];
                dst[3 * e + 1] = v[1];
                dst[3 * e + 2] = v[2];
            }
        }
        __syncthreads();
    }
}

static dim3 multi_grid(const Geom &g)
{
    return dim3(unsigned((g.n[0] + kTileX - 1) / kTileX), unsigned((g.n[1] + kTileY - 1) / kTileY));
}

static int multi_threads(const Geom &g)
{
    const dim3 grid = multi_grid(g);
    return uint64_t(grid.x) * grid.y <= kFewBlocks ? kMultiThreads : kMultiThreads / 2;
}

// LDS bytes of the first k steps of f, the first buffer's elements in cap, and
// the node updates of a block and its passes; false if they do not fit.
template <typename T, class F>
static bool multi_plan(const Geom &g, const F &f, int k, int &cap, size_t &bytes, int &updates,
                       int &passes)
{
    const int threads = multi_threads(g);
    size_t size[2] = {0, 0};
    int w = kTileX < g.n[0] ? kTileX : g.n[0], h = kTileY < g.n[1] ? kTileY : g.n[1];
    updates = passes = 0;
    for (int s = k - 1; s >= 0; s--) {
        updates += w * h;
        passes += (w * h + threads - 1) / threads;
        f.grow(s, w, h);
        w = w < g.n[0] ? w : g.n[0];
        h = h < g.n[1] ? h : g.n[1];
        if (w > kMaxWidth || int64_t(w) * h > kMaxNodes) return false;
        const size_t n = 3 * size_t(w) * size_t(h);
        if (n > size[s & 1]) size[s & 1] = n;
    }
    cap = int(size[0]) + 2 * kPad;
    bytes = (size[0] + size[1] + 4 * kPad) * sizeof(T);
    return bytes <= kMultiLds;
}

void stream_reach(const gals_ctx *ctx, double dt, double c1, double c2, double c3, double reach[2])
{
    double sx = 0.0, sy = 0.0;  // bounds of |s_x| and |s_y|, everywhere
    for (int m = 0; m < 4; m++)
        for (int n = 0; n < 4; n++) {
            sx += fabs(ctx->vd.S[m][n]) * (m + 1) * kPi;
            sy += fabs(ctx->vd.S[m][n]) * (n + 1) * kPi;
        }
    // the stage weights' sum, and room for the rounding of a displacement
    const double w = 1.001 * dt * (fabs(c1) / 6.0 + fabs(c2) / 6.0 + fabs(c3) * 2.0 / 3.0);
    reach[0] = w * sy * ctx->g.inv_h[0];
    reach[1] = w * sx * ctx->g.inv_h[1];
}

// Fill f; false if its regions would not hold: numbers so large that a foot may be
// NaN (its cell is then not where the region is), or FP32 displacements that round
// by more than the regions' slack.
template <typename T>
static bool fill_steps(const gals_ctx *ctx, const Vel<T> &, int k, const double (*c)[3], double dt,
                       AffineSteps<T> &f)
{
    bool sound = sizeof(T) == 8 || (ctx->g.nc[0] <= kMaxCells32 && ctx->g.nc[1] <= kMaxCells32);
    for (int q = 0; q < k; q++) {
        f.m[q] = affine_map2(make_affine_map<T>(ctx, dt, c[q][0], c[q][1], c[q][2]));
        for (int a = 0; a < 2; a++)
            for (double v : {f.m[q].kc[a], f.m[q].Mc[2 * a], f.m[q].Mc[2 * a + 1]})
                sound = sound && fabs(v) <= __DBL_MAX__;
    }
    return sound;
}

template <typename T>
static bool fill_steps(const gals_ctx *ctx, const Vel<T> &p, int k, const double (*c)[3], double dt,
                       StreamSteps<T> &f)
{
    // the field's derivatives, up to the fourth, and dt stay numbers in T
    constexpr double kLargest = sizeof(T) == 4 ? 1e30 : 1e290;
    bool sound = dt <= kLargest;
    for (int m = 0; m < 4; m++)
        for (int n = 0; n < 4; n++) {
            f.S[m][n] = p.S[m][n];
            sound = sound && fabs(ctx->vd.S[m][n]) <= kLargest;
        }
    f.kx = p.kx;
    f.ky = p.ky;
    for (int q = 0; q < k; q++) {
        f.st[q] = make_stage<T>(dt, c[q][0], c[q][1], c[q][2]);
        stream_reach(ctx, dt, c[q][0], c[q][1], c[q][2], f.bound[q]);
    }
    return sound;
}

// Steps per launch for time factors of 1 (the largest displacements).
template <typename T, class F>
static int choose_steps(const gals_ctx *ctx, const Vel<T> &p, double dt)
{
    F f;
    double c[kMultiMax][3];
    for (int q = 0; q < kMultiMax; q++) c[q][0] = c[q][1] = c[q][2] = 1.0;
    if (!fill_steps(ctx, p, kMultiMax, c, dt, f)) return 1;
    for (int k = kMultiMax; k > 1; k--) {
        int cap, updates, passes;
        size_t bytes;
        if (!multi_plan<T>(ctx->g, f, k, cap, bytes, updates, passes)) continue;
        if (ctx->vel_kind == GALS_VEL_AFFINE) {
            if (updates <= kMaxUpdates) return k;
        } else if (passes <= (sizeof(T) == 4 ? 2 * k - 2 : (3 * k - 2) / 2) &&
                   (k > 2 || ctx->g.nodes <= kMaxNodesStream64)) {
            return k;
        }
    }
    return 1;
}

int multi_steps(const gals_ctx *ctx, double dt)
{
    if (ctx->dim != 2 || ctx->inflow || ctx->face) return 1;
    const bool f32 = ctx->prec == GALS_F32;
    if (ctx->vel_kind == GALS_VEL_AFFINE) {
        if (ctx->g.nodes > (f32 ? kMaxNodesAffine32 : kMaxNodesAffine64)) return 1;
        return f32 ? choose_steps<float, AffineSteps<float>>(ctx, ctx->vf, dt)
                   : choose_steps<double, AffineSteps<double>>(ctx, ctx->vd, dt);
    }
    if (ctx->vel_kind != GALS_VEL_STREAM_SIN || ctx->g.nodes > (f32 ? kMaxNodesStream32 : kMaxNodesStream64))
        return 1;
    return f32 ? choose_steps<float, StreamSteps<float>>(ctx, ctx->vf, dt)
               : choose_steps<double, StreamSteps<double>>(ctx, ctx->vd, dt);
}

template <typename T, class F>
static hipError_t launch_multi(const gals_ctx *ctx, const F &f, int k, const void *phi,
                               const void *grad, void *phi_o, void *grad_o, double dt,
                               hipStream_t s, int *took)
{
    int cap = 0, updates, passes;
    size_t bytes = 0;
    while (k > 1 && !multi_plan<T>(ctx->g, f, k, cap, bytes, updates, passes)) k--;
    if (k < 2) return hipSuccess;
    *took = k;
    return with_modes(ctx->mixed, ctx->psi, [&](auto mix, auto psi) -> hipError_t {
        hipLaunchKernelGGL((k_multi2d<T, F, decltype(mix)::value, decltype(psi)::value>),
                           multi_grid(ctx->g), dim3(unsigned(multi_threads(ctx->g))), bytes, s,
                           ctx->g, f, k, cap, dt, (const T *)phi, (const T *)grad,
                           (T *)phi_o, (T *)grad_o);
        return hipGetLastError();
    });
}

template <typename T>
static hipError_t multi_typed(const gals_ctx *ctx, const Vel<T> &p, int k, const double (*c)[3],
                              const void *phi, const void *grad, void *phi_o, void *grad_o,
                              double dt, const void *coltab, const void *rowtab, hipStream_t s,
                              int *took)
{
    *took = 0;
    if (ctx->vel_kind == GALS_VEL_AFFINE) {
        AffineSteps<T> f;
        if (!fill_steps(ctx, p, k, c, dt, f)) return hipSuccess;
        return launch_multi<T>(ctx, f, k, phi, grad, phi_o, grad_o, dt, s, took);
    }
    StreamSteps<T> f;
    if (!fill_steps(ctx, p, k, c, dt, f)) return hipSuccess;
    f.coltab = (const T *)coltab;
    f.rowtab = (const T *)rowtab;
    return launch_multi<T>(ctx, f, k, phi, grad, phi_o, grad_o, dt, s, took);
}

hipError_t launch_multi_step(const gals_ctx *ctx, int k, const double (*c)[3], const void *phi,
                             const void *grad, void *phi_o, void *grad_o, double dt,
                             const void *coltab, const void *rowtab, hipStream_t s, int *took)
{
    return ctx->prec == GALS_F32 ? multi_typed<float>(ctx, ctx->vf, k, c, phi, grad, phi_o, grad_o,
                                                      dt, coltab, rowtab, s, took)
                                 : multi_typed<double>(ctx, ctx->vd, k, c, phi, grad, phi_o,
                                                       grad_o, dt, coltab, rowtab, s, took);
}

}  // namespace gals
