// GA-CIR step kernels for gfx950: one thread per grid node, wave64, fused
// trace + split + gather + Hermite + gradient update (superconsistent, or
// Heun's method along the characteristic).
//
// Each node reads only the old state (never updated in place) and writes its
// new phi, psi with coalesced SoA stores. The affine 2D step stages its
// tile of the old state through LDS and gathers on-tile feet from there; the
// other steps gather departure cells through the cache hierarchy. Feet any
// number of cells away are gathered from global memory, so every CFL number
// is handled.
#include "affine2d.h"
#include "boundary.h"
#include "stream2d.h"

namespace gals {

// Inflow conditions that a step kernel applies itself, to its boundary nodes
// after their step: the dependent launch for a few hundred nodes took 3.5 us
// beside 4 to 5 for the step of a small grid (258 x 182 FP64 1D-like field,
// Dirichlet, 5 steps: 44 us with k_inflow, 29.5 with this; 806 x 1006 FP32
// vortex, Neumann, 3 steps: 62 and 53). The general 2D kernel only: the other
// fields' step kernels are at their register limits, and the conditions are
// theirs through boundary.hip.
enum { kBcNone = 0, kBcInflow = 1, kBcFace = 2 };

// Node index -> (i, j[, k]) with 32-bit arithmetic (the host caps the node
// count below 2^31).
template <typename T, int KIND, int MIX, int PSI, int BC>
__global__ __launch_bounds__(kBlock) void k_step2d(Geom g, Vel<T> p, Stage<T> st, double dt,
                                                   InflowData<T> b, const T *__restrict__ tab,
                                                   const T *__restrict__ phi,
                                                   const T *__restrict__ grad,
                                                   T *__restrict__ phi_o, T *__restrict__ grad_o)
{
    unsigned blk;
    if (!xcd_block(unsigned((g.nodes + kBlock - 1) / kBlock), blk)) return;
    const unsigned id = blk * kBlock + threadIdx.x;
    if (id >= unsigned(g.nodes)) return;
    unsigned ri;
    const int j = int(udiv_magic(id, unsigned(g.n[0]), g.n_magic[0], ri));
    const int i = int(ri);
    const T *gx = grad, *gy = grad + g.plane;

    const double x[2] = {node_coord(g.lo[0], i, g.h[0]), node_coord(g.lo[1], j, g.h[1])};
    double X[2];
    T J[4];  // superconsistent Jacobian, or (Heun) grad v at the node
    const int64_t ti[2] = {i, int64_t(g.n[0]) + j};
    trace_node<T, 2, KIND, PSI == GALS_PSI_SUPERCONSISTENT>(p, st, dt, tab, ti, x, X, J);
    const unsigned out = project_foot<2>(g, X);

    int cell[2];
    double xid[2];
    split<2>(g, X, cell, xid);
    const T xi[2] = {T(xid[0]), T(xid[1])};
    if constexpr (kFold2d<T, MIX>) pin4(J);
    T H, Hx, Hy;
    const int64_t end = gather_end<T, MIX>(g);
    bicubic<T, MIX>(g, plane_rsrc(phi, end), plane_rsrc(gx, end), plane_rsrc(gy, end), cell, xi, H,
                    Hx, Hy);
    if (out & 1u) Hx = T(0);
    if (out & 2u) Hy = T(0);

    const unsigned o = unsigned(j) * unsigned(g.pitch) + unsigned(i);
    pstore(phi_o, o, H);
    if constexpr (PSI == GALS_PSI_HEUN) {
        T vf[2], Af[4], ps[2];
        const T gH[2] = {Hx, Hy};
        velocity<T, 2, KIND>(p, X, st.c2, vf, Af);
        heun_gradient<T, 2>(Af, J, T(dt), gH, ps);
        pstore(grad_o, o, ps[0]);
        pstore(grad_o + g.plane, o, ps[1]);
    } else {
        pstore(grad_o, o, J[0] * Hx + J[2] * Hy);
        pstore(grad_o + g.plane, o, J[1] * Hx + J[3] * Hy);
    }
    if constexpr (BC != kBcNone) {
        if (i != 0 && i != g.nc[0] && j != 0 && j != g.nc[1]) return;
        const int ij[2] = {i, j};
        if constexpr (BC == kBcInflow)
            inflow_node<T, 2, KIND>(g, p, st.c1, dt, ij, b, phi_o, grad_o);
        else
            face_node<T, 2, KIND, MIX>(g, p, st, dt, ij, phi, grad, phi_o, grad_o);
    }
}

// ---------------------------------------------------------------------------
// LDS staging of the old state (used by the affine 2D step below). A block
// owns a tile of 64 x TY nodes (four waves, each a row of 64 nodes, TY / 4
// row groups) and stages phi, psi_x, psi_y of the tile and a halo of kHaloX
// columns and kHaloY rows around it: the scheme's stencil is one cell, so a
// foot less than a cell from its node (CFL < 1) reads only the node's
// neighbours, and the cross derivative (A) one column more on each side. The
// staging loads are coalesced and do not depend on the trace, so they are
// issued first and their latency hides behind it. A foot whose stencil leaves
// the staged region (CFL > 1 somewhere) gathers from global memory instead,
// lane by lane, so any CFL number is still handled.
// ---------------------------------------------------------------------------
constexpr int kHaloX = 2, kHaloY = 1;

template <int TY>
struct StageTile {
    static constexpr int W = 64 + 2 * kHaloX;  // staged columns
    static constexpr int H = TY + 2 * kHaloY;  // staged rows
    static constexpr int N = W * H;
    static constexpr int PER = (N + kBlock - 1) / kBlock;  // staged values per thread
};

// The staging of one block's tile: coalesced loads of phi, psi_x, psi_y over
// the tile and its halo into registers (issued before the foot is computed),
// then into LDS. Thread t stages the flattened tile's entries t, t + 256, ...
// Positions outside the grid load nothing (their offset is past the plane:
// the buffer load returns 0) and are never read. (Staging whole rows per
// wave, with one address add per load, cut the vector instructions by 3 % but
// cost FP64 one wave per SIMD and measured no faster in FP32.)
template <typename T, int TY>
struct TileStager {
    using S = StageTile<TY>;
    T sv[3][S::PER];

    __device__ __forceinline__ void load(const Geom &g, const T *phi, const T *gx, const T *gy,
                                         int cx0, int ry0)
    {
        const Rsrc r0 = plane_rsrc(phi, g.plane), r1 = plane_rsrc(gx, g.plane),
                   r2 = plane_rsrc(gy, g.plane);
        const unsigned past = unsigned(g.plane);
        const int tid = int(threadIdx.y) * 64 + int(threadIdx.x);
#pragma unroll
        for (int k = 0; k < S::PER; k++) {
            const int f = tid + k * kBlock;
            const int row = ry0 + f / S::W, col = cx0 + f % S::W;
            const bool in = f < S::N && row >= 0 && row < g.n[1] && col >= 0 && col < g.n[0];
            const unsigned off = in ? unsigned(row) * unsigned(g.pitch) + unsigned(col) : past;
            sv[0][k] = bload(r0, off, T());
            sv[1][k] = bload(r1, off, T());
            sv[2][k] = bload(r2, off, T());
        }
    }

    // Node f's three values sit together at tile[3 f .. 3 f + 2], so that a
    // cell's whole stencil lies within 216 elements of its first value and
    // every read of the gather is an immediate offset from one address.
    __device__ __forceinline__ void store(T *tile) const
    {
        const int tid = int(threadIdx.y) * 64 + int(threadIdx.x);
#pragma unroll
        for (int k = 0; k < S::PER; k++) {
            const int f = tid + k * kBlock;
            if (f < S::N) {
                tile[3 * f] = sv[0][k];
                tile[3 * f + 1] = sv[1][k];
                tile[3 * f + 2] = sv[2][k];
            }
        }
    }
};

// Tiles of 64 x TY nodes, dealt to the XCDs in contiguous bands (as
// xcd_tile does for 64 x 4 tiles of the stream-function step).
struct TileGrid {
    unsigned tiles_x, tiles, magic;  // tiles per row group, in all, floor(2^32 / tiles_x)
};

// Tiles of 64 x rows nodes over the grid.
static TileGrid tile_grid(const Geom &g, int rows)
{
    TileGrid tg;
    tg.tiles_x = unsigned((g.n[0] + 63) / 64);
    tg.tiles = tg.tiles_x * unsigned((g.n[1] + rows - 1) / rows);
    tg.magic = tg.tiles_x > 1 ? unsigned((uint64_t(1) << 32) / tg.tiles_x) : 0xFFFFFFFFu;
    return tg;
}

__device__ __forceinline__ bool xcd_tile_n(const TileGrid &tg, unsigned &tx, unsigned &ty)
{
    const unsigned per = (tg.tiles + 7u) / 8u;
    const unsigned t = (blockIdx.x % 8u) * per + blockIdx.x / 8u;
    unsigned r;
    ty = udiv_magic(t, tg.tiles_x, tg.magic, r);
    tx = r;
    return t < tg.tiles;
}

// Row groups of four per affine tile: 64 x 8 nodes (a 64 x 4 tile stages 1.6
// values per node and field, 64 x 8 1.3; 64 x 16 measured no faster).
constexpr int kAffineRows = 2;

// Non-temporal store of a result the next step reads only after the whole
// launch, from a grid far larger than the caches: the line is not kept in
// them, which leaves the L2 to the tile halos the neighbouring blocks re-read.
template <typename T>
__device__ __forceinline__ void pstore_nt(T *base, unsigned elem, T v)
{
    __builtin_nontemporal_store(v, reinterpret_cast<T *>(reinterpret_cast<char *>(base) +
                                                         elem * unsigned(sizeof(T))));
}

// 2D step for an affine field: the foot from the host's map, the old state
// staged in a 64 x 4R node tile with its halo, the gather
// from the tile at fixed offsets, or from global memory for a stencil off
// the tile.
template <typename T, int MIX, int PSI, int R>
__global__ __launch_bounds__(kBlock) void k_step2d_affine(Geom g, TileGrid tg, AffineMap2<T> am,
                                                          double dt, const T *__restrict__ phi,
                                                          const T *__restrict__ grad,
                                                          T *__restrict__ phi_o,
                                                          T *__restrict__ grad_o)
{
    using S = StageTile<4 * R>;
    __shared__ T tile[3 * S::N];
    unsigned tx, ty;
    if (!xcd_tile_n(tg, tx, ty)) return;  // whole blocks only: before the barrier
    const int cx0 = int(tx) * 64 - kHaloX, ry0 = int(ty) * (4 * R) - kHaloY;
    const T *gx = grad, *gy = grad + g.plane;
    TileStager<T, 4 * R> stager;
    stager.load(g, phi, gx, gy, cx0, ry0);
    const int i = int(tx) * 64 + int(threadIdx.x);
    int cell[R][2];
    T xi[R][2];
    bool outb[R][2];
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int j = __builtin_amdgcn_readfirstlane(ry0 + kHaloY + int(threadIdx.y) + 4 * r);
        affine_foot(g, am, i, j, cell[r], xi[r], outb[r]);
    }
    stager.store(tile);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int j = __builtin_amdgcn_readfirstlane(ry0 + kHaloY + int(threadIdx.y) + 4 * r);
        const int cx = cell[r][0], cy = cell[r][1];
        const bool on = cx - 1 >= cx0 && cx + 2 < cx0 + S::W && cy >= ry0 && cy + 1 < ry0 + S::H;
        const bool store = i < g.n[0] && j < g.n[1];
        // the Hermite evaluation and the update from the cell data of either
        // source; each source finishes on its own (merging the two sources'
        // cell data before one evaluation cost register moves on every lane)
        auto finish = [&](T H, T Hx, T Hy) {
            T v[3];
            affine_values<T, PSI>(am, dt, outb[r], H, Hx, Hy, v);
            if (!store) return;
            const unsigned o = unsigned(j) * unsigned(g.pitch) + unsigned(i);
            pstore_nt(phi_o, o, v[0]);
            pstore_nt(grad_o, o, v[1]);
            pstore_nt(grad_o + g.plane, o, v[2]);
        };
        if (__builtin_expect(on, 1)) {
            T H, Hx, Hy;
            const T *t = tile + 3 * ((cy - ry0) * S::W + (cx - 1 - cx0));
            bicubic_lds<T, MIX, false>(g, t, t + 3 * S::W, cell[r], xi[r], H, Hx, Hy);
            finish(H, Hx, Hy);
        } else {
            T H, Hx, Hy;
            bicubic<T, MIX, false>(g, plane_rsrc(phi, g.plane), plane_rsrc(gx, g.plane),
                                   plane_rsrc(gy, g.plane), cell[r], xi[r], H, Hx, Hy);
            finish(H, Hx, Hy);
        }
    }
}

// Node of this thread in a 3D step. Blocks are dealt to the 8 XCDs
// round-robin by id, and each XCD has its own L2: XCD x takes the nodes of
// every z-plane whose in-plane index (j n0 + i) lies in the x-th eighth of
// the plane, plane after plane in blocks of kBlock. A node gathers from rows
// j - 1 .. j + 2 of planes k and k + 1, so an XCD's gathers stay within its
// eighth of a few planes and the next eighth's first rows, which its L2
// holds (contiguous bands of the flat node order kept a few whole planes of
// every field in each L2, more than it holds in 3D). Returns false past the
// band's last node.
__device__ __forceinline__ bool band_node3d(const Geom &g, int &i, int &j, int &k)
{
    const unsigned x = blockIdx.x & 7u, b = blockIdx.x >> 3;
    const unsigned P = unsigned(g.n[0]) * unsigned(g.n[1]);  // nodes per plane
    const unsigned s0 = unsigned((uint64_t(x) * P) >> 3);
    const unsigned len = unsigned((uint64_t(x + 1u) * P) >> 3) - s0;  // this XCD's nodes per plane
    const unsigned id = b * unsigned(kBlock) + threadIdx.x;
    if (len == 0u || id >= len * unsigned(g.n[2])) return false;
    // plane from an FP32 estimate of id / len, corrected once: a state plane
    // under 2 GiB keeps id < 2^27 and the quotient (a plane index) < 2^21.5,
    // and the estimate's relative error (conversion, reciprocal, product) is
    // under 2^-22, so it is off by less than one
    int kk = int(float(id) * __builtin_amdgcn_rcpf(float(len)));
    int q = int(id) - kk * int(len);
    if (q < 0) { kk--; q += int(len); }
    else if (q >= int(len)) { kk++; q -= int(len); }
    unsigned ri;
    j = int(udiv_magic(s0 + unsigned(q), unsigned(g.n[0]), g.n_magic[0], ri));
    i = int(ri);
    k = kk;
    return true;
}

// Blocks of a 3D step's launch: 8 x the blocks of the largest XCD band.
inline unsigned band_blocks3d(const Geom &g)
{
    const uint64_t P = uint64_t(g.n[0]) * uint64_t(g.n[1]);
    const uint64_t band = (P + 7u) / 8u * uint64_t(g.n[2]);
    return unsigned(8u * ((band + kBlock - 1) / kBlock));
}

// 3D step for an affine field: the foot from the host's map, one thread per
// node, the gather through the caches.
template <typename T, int MIX, int PSI>
__global__ __launch_bounds__(kBlock) void k_step3d_affine(Geom g, AffineMap<T> am, double dt,
                                                          const T *__restrict__ phi,
                                                          const T *__restrict__ grad,
                                                          T *__restrict__ phi_o,
                                                          T *__restrict__ grad_o)
{
    int i, j, k;
    if (!band_node3d(g, i, j, k)) return;
    double sc[3];
#pragma unroll
    for (int a = 0; a < 3; a++)
        sc[a] = am.kc[a] + am.Mc[a * 3] * double(i) + am.Mc[a * 3 + 1] * double(j) +
                am.Mc[a * 3 + 2] * double(k);
    int cell[3];
    T xi[3];
    bool outb[3];
    split_cells<T, 3>(g, sc, cell, xi, outb);
    const T *gx = grad, *gy = grad + g.plane, *gz = grad + 2 * g.plane;
    T H, G[3];
    tricubic<T, MIX>(g, plane_rsrc(phi, g.span), plane_rsrc(gx, g.span), plane_rsrc(gy, g.span),
                     plane_rsrc(gz, g.span), cell, xi, H, G);
    T Hx = G[0], Hy = G[1], Hz = G[2];
    if (outb[0]) Hx = T(0);
    if (outb[1]) Hy = T(0);
    if (outb[2]) Hz = T(0);
    const unsigned o = (unsigned(k) * unsigned(g.n[1]) + unsigned(j)) * unsigned(g.pitch) +
                       unsigned(i);
    pstore(phi_o, o, H);
    if constexpr (PSI == GALS_PSI_HEUN) {
        T ps[3];
        const T gH[3] = {Hx, Hy, Hz};
        heun_gradient<T, 3>(am.Af, am.An, T(dt), gH, ps);
        pstore(grad_o, o, ps[0]);
        pstore(grad_o + g.plane, o, ps[1]);
        pstore(grad_o + 2 * g.plane, o, ps[2]);
    } else {
        const T *J = am.J;
        pstore(grad_o, o, J[0] * Hx + J[3] * Hy + J[6] * Hz);
        pstore(grad_o + g.plane, o, J[1] * Hx + J[4] * Hy + J[7] * Hz);
        pstore(grad_o + 2 * g.plane, o, J[2] * Hx + J[5] * Hy + J[8] * Hz);
    }
}

// The part of a 3D step after the trace: boundary treatment of the foot,
// split, gather, tricubic value and gradient, gradient update.
template <typename T, int KIND, int MIX, int PSI>
__device__ __forceinline__ void finish3d(const Geom &g, const Vel<T> &p, const Stage<T> &st,
                                         double dt, int i, int j, int k, double *X, const T *J,
                                         const T *__restrict__ phi, const T *__restrict__ grad,
                                         T *__restrict__ phi_o, T *__restrict__ grad_o)
{
    const T *gx = grad, *gy = grad + g.plane, *gz = grad + 2 * g.plane;
    const unsigned out = project_foot<3>(g, X);

    int cell[3];
    double xid[3];
    split<3>(g, X, cell, xid);
    const T xi[3] = {T(xid[0]), T(xid[1]), T(xid[2])};
    T H, gradH[3];
    tricubic<T, MIX>(g, plane_rsrc(phi, g.span), plane_rsrc(gx, g.span), plane_rsrc(gy, g.span),
                     plane_rsrc(gz, g.span), cell, xi, H, gradH);
    T Hx = gradH[0], Hy = gradH[1], Hz = gradH[2];
    if (out & 1u) Hx = T(0);
    if (out & 2u) Hy = T(0);
    if (out & 4u) Hz = T(0);

    const unsigned o = (unsigned(k) * unsigned(g.n[1]) + unsigned(j)) * unsigned(g.pitch) +
                       unsigned(i);
    pstore(phi_o, o, H);
    if constexpr (PSI == GALS_PSI_HEUN) {
        T vf[3], Af[9], ps[3];
        const T gH[3] = {Hx, Hy, Hz};
        velocity<T, 3, KIND>(p, X, st.c2, vf, Af);
        heun_gradient<T, 3>(Af, J, T(dt), gH, ps);
        pstore(grad_o, o, ps[0]);
        pstore(grad_o + g.plane, o, ps[1]);
        pstore(grad_o + 2 * g.plane, o, ps[2]);
    } else {
        pstore(grad_o, o, J[0] * Hx + J[3] * Hy + J[6] * Hz);
        pstore(grad_o + g.plane, o, J[1] * Hx + J[4] * Hy + J[7] * Hz);
        pstore(grad_o + 2 * g.plane, o, J[2] * Hx + J[5] * Hy + J[8] * Hz);
    }
}

// Waves per SIMD of the superconsistent 3D kernels. FP32: six for the vector
// potential (77 VGPRs; five with 81 by the compiler's choice, 555 against 539 us
// per 257^3 step), five with cell-based cross derivatives (six spill 14 VGPRs) and
// for the deformation field (six spill 4, 151 x 152 x 141 nodes 67.3 against 64.8
// us per step). FP64: three (vector potential 150 VGPRs; at the compiler's choice
// of 170 two waves, 480 against 375 us for two steps of 141 x 131 x 121 nodes), also
// with cell-based cross derivatives, where they spill 10 VGPRs (246 against 293
// with two waves and no spill; deformation field the same at two and three). The
// Heun kernels need more registers and keep the compiler's choice.
template <typename T, int KIND, int MIX, int PSI>
constexpr int kWaves3d = PSI != GALS_PSI_SUPERCONSISTENT                            ? 1
                         : sizeof(T) != 4                                           ? 3
                         : MIX == GALS_MIXED_CELL || KIND == GALS_VEL_LEVEQUE3D     ? 5
                                                                                    : 6;

template <typename T, int KIND, int MIX, int PSI>
__global__ __launch_bounds__(kBlock)
    __attribute__((amdgpu_waves_per_eu(kWaves3d<T, KIND, MIX, PSI>))) void k_step3d(
        Geom g, Vel<T> p, Stage<T> st, double dt, const T *__restrict__ tab,
        const T *__restrict__ phi, const T *__restrict__ grad, T *__restrict__ phi_o,
        T *__restrict__ grad_o)
{
    int i, j, k;
    if (!band_node3d(g, i, j, k)) return;

    const double x[3] = {node_coord(g.lo[0], i, g.h[0]), node_coord(g.lo[1], j, g.h[1]),
                         node_coord(g.lo[2], k, g.h[2])};
    double X[3];
    T J[9];
    const int64_t ti[3] = {i, int64_t(g.n[0]) + j, int64_t(g.n[0]) + g.n[1] + k};
    trace_node<T, 3, KIND, PSI == GALS_PSI_SUPERCONSISTENT>(p, st, dt, tab, ti, x, X, J);
    finish3d<T, KIND, MIX, PSI>(g, p, st, dt, i, j, k, X, J, phi, grad, phi_o, grad_o);
}

// ---------------------------------------------------------------------------
// Sine vector potentials in 3D: sin(pi x) and cos(pi x) of every node
// coordinate come from per-axis tables (FP64-built, one pair per node along
// each axis); the three stages take the multiples of the node's angles, and
// (SHIFT) the two off-node stages shift them by angle addition whenever
// every offset is small enough for the series of the precision, instead of
// evaluating sin and cos at the stage points. The mode sums are those of
// vel_vecpot.
// ---------------------------------------------------------------------------
// Velocity at one stage point from the multiples of each axis: through LDS
// (LDS, the FP32 kernel) or by per-lane selects.
template <typename T, bool LDS>
__device__ __forceinline__ void modes_at(const Vel<T> &p, T (*tab)[kBlock], const T *sx,
                                         const T *cx, const T *sy, const T *cy, const T *sz,
                                         const T *cz, T cf, T *v, T *A)
{
    if constexpr (LDS) {
        const int tid = int(threadIdx.x);
#pragma unroll
        for (int r = 0; r < 4; r++) {
            tab[r][tid] = sx[r];
            tab[4 + r][tid] = cx[r];
            tab[8 + r][tid] = sy[r];
            tab[12 + r][tid] = cy[r];
            tab[16 + r][tid] = sz[r];
            tab[20 + r][tid] = cz[r];
        }
        vecpot_modes_lds(p, tab, tid, cf, v, A);  // each thread reads only its own column
    } else {
        vecpot_modes(p, sx, cx, sy, cy, sz, cz, cf, v, A);
    }
}

template <typename T, bool SHIFT, bool LDS>
__device__ __forceinline__ void stage_vecpot(const Vel<T> &p, T (*tab)[kBlock], const T *s1,
                                             const T *c1, const double *x, const T *d, T *w,
                                             T *R)
{
    T sx[4], cx[4], sy[4], cy[4], sz[4], cz[4];
    // FP32: the short series up to |pi d| = kShiftMax; FP64: the long one
    constexpr double kMax = sizeof(T) == 4 ? kShiftMax : kShiftMaxLong<T>;
    bool near = SHIFT;
#pragma unroll
    for (int a = 0; a < 3; a++) near = near && fabs(d[a]) <= T(kMax / kPi);
    if (near) {
        T s[3], c[3];
#pragma unroll
        for (int a = 0; a < 3; a++) {
            if constexpr (sizeof(T) == 4)
                shifted_sincos(s1[a], c1[a], d[a], s[a], c[a]);
            else
                shifted_sincos_long(s1[a], c1[a], d[a], s[a], c[a]);
        }
        multiples_from(s[0], c[0], sx, cx);
        multiples_from(s[1], c[1], sy, cy);
        multiples_from(s[2], c[2], sz, cz);
    } else {
        sincos_multiples(T(x[0] + double(d[0])), sx, cx);
        sincos_multiples(T(x[1] + double(d[1])), sy, cy);
        sincos_multiples(T(x[2] + double(d[2])), sz, cz);
    }
    modes_at<T, LDS>(p, tab, sx, cx, sy, cy, sz, cz, T(1), w, R);
}

template <typename T, int MIX, bool SHIFT, int PSI>
__global__ __launch_bounds__(kBlock)
    __attribute__((amdgpu_waves_per_eu(
        kWaves3d<T, GALS_VEL_VECPOT_SIN, MIX, PSI>))) void k_step3d_vecpot(
        Geom g, Vel<T> p, Stage<T> st, double dt, const T *__restrict__ tab,
        const T *__restrict__ phi, const T *__restrict__ grad, T *__restrict__ phi_o,
        T *__restrict__ grad_o)
{
    constexpr bool LDS = sizeof(T) == 4;
    __shared__ T tab_s[LDS ? 24 : 1][kBlock];
    int i, j, k;
    if (!band_node3d(g, i, j, k)) return;

    const double x[3] = {node_coord(g.lo[0], i, g.h[0]), node_coord(g.lo[1], j, g.h[1]),
                         node_coord(g.lo[2], k, g.h[2])};
    const int64_t ti[3] = {i, int64_t(g.n[0]) + j, int64_t(g.n[0]) + g.n[1] + k};
    T s1[3], c1[3];
#pragma unroll
    for (int a = 0; a < 3; a++) {
        s1[a] = tab[2 * ti[a]];
        c1[a] = tab[2 * ti[a] + 1];
    }
    // w_k, R_k: velocity and velocity Jacobian at stage k without the time
    // factor c_k (Stage carries dt c_k in its weights, as in the 2D stream
    // step); the stage offsets and the foot's displacement are summed in T,
    // the foot itself in FP64
    T w0[3], R0[9], w1[3], R1[9], w2[3], R2[9];
    {
        T sx[4], cx[4], sy[4], cy[4], sz[4], cz[4];
        multiples_from(s1[0], c1[0], sx, cx);
        multiples_from(s1[1], c1[1], sy, cy);
        multiples_from(s1[2], c1[2], sz, cz);
        modes_at<T, LDS>(p, tab_s, sx, cx, sy, cy, sz, cz, T(1), w0, R0);  // at x, t + dt
    }
    T d1[3], d2[3];
#pragma unroll
    for (int a = 0; a < 3; a++) d1[a] = -st.e1 * w0[a];
    stage_vecpot<T, SHIFT, LDS>(p, tab_s, s1, c1, x, d1, w1, R1);  // at x1 = x + d1, t
#pragma unroll
    for (int a = 0; a < 3; a++) d2[a] = -(st.q1 * w0[a] + st.q2 * w1[a]);
    stage_vecpot<T, SHIFT, LDS>(p, tab_s, s1, c1, x, d2, w2, R2);  // at x2 = x + d2, t + dt/2
    double X[3];
#pragma unroll
    for (int a = 0; a < 3; a++)
        X[a] = x[a] - double(st.f1 * w0[a] + st.f2 * w1[a] + st.f3 * w2[a]);
    T J[9];
    if constexpr (PSI == GALS_PSI_SUPERCONSISTENT) {
        jacobian_chain_w<T, 3>(R0, R1, R2, st, J);
    } else {
#pragma unroll
        for (int q = 0; q < 9; q++) J[q] = st.c1 * R0[q];
    }
    finish3d<T, GALS_VEL_VECPOT_SIN, MIX, PSI>(g, p, st, dt, i, j, k, X, J, phi, grad, phi_o,
                                              grad_o);
}

// ---------------------------------------------------------------------------
// What an advance needs before its first step, in one launch: the field's tables
// (TAB), and, when an odd number of launches follows, the state's copy in the
// workspace that the first of them reads, so that the last one ends in the
// caller's buffers. The first `tab_blocks` blocks build entries, the others copy
// the nodes of every row, without the padding, 16 bytes a thread at a time where
// the caller's planes allow. (A table launch before and one pitched copy per
// plane after the last step: 24 us per one-step call on 501 x 380 FP32 nodes, 81
// on 2049^2, 303 on 4097 x 4096; 17, 62 and 244 with this. Rows of three nodes
// with their padding are 21 times the bytes: a step of 3 x 401 x 401 FP64 nodes 194
// us with whole planes, 68 with this.)
// ---------------------------------------------------------------------------
enum { kTabNone = 0, kTabStream = 1, kTabAxis = 2 };

// How the copy's work items cut a row: `per` items of `width` elements, the last
// of them with what is left of the row; magic = floor(2^32 / per).
struct RowCut {
    unsigned per, width, magic;
};

template <typename T>
__device__ __forceinline__ void copy_rows(const Geom &g, const RowCut &cut,
                                          const T *__restrict__ phi, const T *__restrict__ grad,
                                          T *__restrict__ copy, unsigned id, unsigned stride)
{
    // at most 2^31 items (a plane is under 2 GiB), stride at most 2^21: no index wraps
    const unsigned rows = unsigned(g.n[1]) * unsigned(g.n[2]);
    const unsigned items = cut.per * rows * unsigned(1 + g.dim);
    for (; id < items; id += stride) {
        unsigned v, r = udiv_magic(id, cut.per, cut.magic, v), a = 0;
        while (r >= rows) {
            r -= rows;
            a++;
        }
        const int64_t o = int64_t(r) * g.pitch + int64_t(v) * cut.width;
        const T *s = a == 0 ? phi + o : grad + int64_t(a - 1) * g.plane + o;
        T *d = copy + int64_t(a) * g.plane + o;
        const unsigned left = unsigned(g.n[0]) - v * cut.width;
        if (cut.width > 1u && left >= cut.width) {
            *reinterpret_cast<uint4 *>(d) = *reinterpret_cast<const uint4 *>(s);
            continue;
        }
        // the rest of a row, its loads issued together; one element where not wide
        const unsigned n = left < cut.width ? left : cut.width;
        T t[3];
#pragma unroll
        for (unsigned k = 0; k < 3u; k++)
            if (k < n) t[k] = s[k];
#pragma unroll
        for (unsigned k = 0; k < 3u; k++)
            if (k < n) d[k] = t[k];
    }
}

template <typename T, int TAB>
__global__ __launch_bounds__(kBlock) void k_prepare(Geom g, Vel<double> p, unsigned tab_blocks,
                                                    T *__restrict__ tab0, T *__restrict__ tab1,
                                                    const T *__restrict__ phi,
                                                    const T *__restrict__ grad,
                                                    T *__restrict__ copy, RowCut cut)
{
    if (blockIdx.x < tab_blocks) {
        const int id = int(blockIdx.x) * kBlock + int(threadIdx.x);
        if constexpr (TAB == kTabStream) {
            stream_table_entry(g, p.S, id, tab0, tab1);
        } else if constexpr (TAB == kTabAxis) {
            int r = id, a = 0;
            while (a < 3 && r >= g.n[a]) r -= g.n[a++];
            if (a >= 3) return;
            // the vector potential's angles, twice the trig fields' (trace_trig)
            const double turns = p.kind == GALS_VEL_VECPOT_SIN ? 1.0 : 2.0;
            double s, c;
            sincospi(turns * node_coord(g.lo[a], r, g.h[a]), &s, &c);
            tab0[2 * id] = T(s);
            tab0[2 * id + 1] = T(c);
        }
        return;
    }
    copy_rows(g, cut, phi, grad, copy, (blockIdx.x - tab_blocks) * unsigned(kBlock) + threadIdx.x,
              (gridDim.x - tab_blocks) * unsigned(kBlock));
}

template <typename T>
static hipError_t prepare_typed(const gals_ctx *ctx, int tab, void *tab0, void *tab1,
                                const void *phi, const void *grad, void *copy, hipStream_t s)
{
    const Geom &g = ctx->g;
    const int64_t entries = tab == kTabStream ? stream_table_threads(g)
                            : tab == kTabAxis ? int64_t(g.n[0]) + g.n[1] + g.n[2] : 0;
    const unsigned tb = unsigned((entries + kBlock - 1) / kBlock);
    // rows start at multiples of 64 elements, and the copy at a multiple of 256 bytes
    const bool wide = (uintptr_t(phi) | uintptr_t(grad)) % 16 == 0;
    RowCut cut;
    cut.width = wide ? unsigned(16 / sizeof(T)) : 1u;
    cut.per = (unsigned(g.n[0]) + cut.width - 1u) / cut.width;
    cut.magic = cut.per > 1u ? unsigned((uint64_t(1) << 32) / cut.per) : 0xFFFFFFFFu;
    int64_t cb = 0;
    if (copy) {
        const int64_t items = int64_t(cut.per) * g.n[1] * g.n[2] * (1 + g.dim);
        cb = (items + kBlock - 1) / kBlock;
        if (cb > 8192) cb = 8192;
    }
    if (tb + cb == 0) return hipSuccess;
    auto kern = tab == kTabStream ? k_prepare<T, kTabStream>
                : tab == kTabAxis ? k_prepare<T, kTabAxis> : k_prepare<T, kTabNone>;
    hipLaunchKernelGGL(kern, dim3(tb + unsigned(cb)), dim3(kBlock), 0, s, g, ctx->vd, tb, (T *)tab0,
                       (T *)tab1, (const T *)phi, (const T *)grad, (T *)copy, cut);
    return hipGetLastError();
}

hipError_t launch_prepare(const gals_ctx *ctx, void *coltab, void *rowtab, const void *phi,
                          const void *grad, void *copy, hipStream_t s)
{
    const int tab = !coltab ? kTabNone : ctx->vel_kind == GALS_VEL_STREAM_SIN ? kTabStream : kTabAxis;
    return ctx->prec == GALS_F32
               ? prepare_typed<float>(ctx, tab, coltab, rowtab, phi, grad, copy, s)
               : prepare_typed<double>(ctx, tab, coltab, rowtab, phi, grad, copy, s);
}

// ---------------------------------------------------------------------------
// Sine stream-function fields (see stream2d.h).
// ---------------------------------------------------------------------------
// GA-CIR step for the sine stream-function field. Launch: blocks of 64 x 4
// threads over 64 x 4 node tiles; each wave owns 64 consecutive nodes of one
// row, so the row table is read once per wave through scalar loads. The cell
// data are gathered through the caches after the trace: the kernel is bound
// by its vector ALU, and staging the tile through LDS (as the affine step
// does) measured slower in both precisions (FP32 34.0 -> 39.9 us, FP64 87.2
// -> 102.4 us per 2049^2 step: more instructions, and in FP64 one wave per
// SIMD fewer).
template <typename T, int MIX, bool TAYLOR, int PSI>
__global__ __launch_bounds__(kBlock) void k_step2d_stream(
    Geom g, Vel<T> p, Stage<T> st, double dt, const T *__restrict__ coltab,
    const T *__restrict__ rowtab, const T *__restrict__ phi, const T *__restrict__ grad,
    T *__restrict__ phi_o, T *__restrict__ grad_o)
{
    unsigned tx, ty;
    if (!xcd_tile(g, tx, ty)) return;
    const int i = int(tx) * 64 + int(threadIdx.x);
    const int j = __builtin_amdgcn_readfirstlane(int(ty) * 4 + int(threadIdx.y));
    if (j >= g.n[1] || i >= g.n[0]) return;
    stream_node<T, MIX, TAYLOR, PSI>(g, p, st, dt, coltab + int64_t(i) * kJet,
                                     rowtab + int64_t(j) * kJet, phi, grad, grad + g.plane,
                                     phi_o, grad_o, grad_o + g.plane, i, j);
}

template <typename T, int MIX, int PSI>
static hipError_t launch_stream(const gals_ctx *ctx, const Vel<T> &p, const void *phi,
                                const void *grad, void *phi_o, void *grad_o, double dt,
                                double c1, double c2, double c3, const void *coltab,
                                const void *rowtab, hipStream_t s)
{
    const Stage<T> st = make_stage<T>(dt, c1, c2, c3);
    const unsigned tiles = ctx->g.tiles;
    const dim3 grid((tiles + 7u) / 8u * 8u);
    hipLaunchKernelGGL((k_step2d_stream<T, MIX, sizeof(T) == 4, PSI>), grid, dim3(64, 4), 0, s,
                       ctx->g, p, st, dt, (const T *)coltab, (const T *)rowtab, (const T *)phi,
                       (const T *)grad, (T *)phi_o, (T *)grad_o);
    return hipGetLastError();
}

template <typename T, int MIX, int PSI>
static hipError_t launch_vecpot(const gals_ctx *ctx, const Vel<T> &p, const void *phi,
                                const void *grad, void *phi_o, void *grad_o, double dt,
                                double c1, double c2, double c3, const void *tab, hipStream_t s)
{
    const Stage<T> st = make_stage<T>(dt, c1, c2, c3);
    const unsigned blocks = band_blocks3d(ctx->g);
    hipLaunchKernelGGL((k_step3d_vecpot<T, MIX, true, PSI>), dim3(blocks),
                       dim3(kBlock), 0, s, ctx->g, p, st, dt, (const T *)tab, (const T *)phi,
                       (const T *)grad, (T *)phi_o, (T *)grad_o);
    return hipGetLastError();
}

template <typename T, int KIND, int MIX, int PSI>
static hipError_t launch_typed(const gals_ctx *ctx, const Vel<T> &p, const void *phi,
                               const void *grad, void *phi_o, void *grad_o, double dt, double c1,
                               double c2, double c3, const void *tab, hipStream_t s)
{
    const Stage<T> st = make_stage<T>(dt, c1, c2, c3);
    // rounded up to a multiple of 8 for the XCD band mapping (xcd_block)
    const unsigned blocks = unsigned((ctx->g.nodes + kBlock - 1) / kBlock + 7) / 8u * 8u;
    if constexpr (KIND == GALS_VEL_AFFINE) {
        const AffineMap<T> am = make_affine_map<T>(ctx, dt, c1, c2, c3);
        if (ctx->dim == 2) {
            const TileGrid tg = tile_grid(ctx->g, 4 * kAffineRows);
            const AffineMap2<T> am2 = affine_map2(am);
            hipLaunchKernelGGL((k_step2d_affine<T, MIX, PSI, kAffineRows>),
                               dim3((tg.tiles + 7u) / 8u * 8u),
                               dim3(64, 4), 0, s, ctx->g, tg, am2, dt, (const T *)phi,
                               (const T *)grad, (T *)phi_o, (T *)grad_o);
        } else {
            hipLaunchKernelGGL((k_step3d_affine<T, MIX, PSI>), dim3(band_blocks3d(ctx->g)),
                               dim3(kBlock), 0, s,
                               ctx->g, am, dt, (const T *)phi, (const T *)grad, (T *)phi_o,
                               (T *)grad_o);
        }
        return hipGetLastError();
    }
    if (ctx->dim == 2) {
        if constexpr (KIND == GALS_VEL_VORTEX || KIND == GALS_VEL_PSEUDO1D) {
            const bool in_step = ctx->inflow && !inflow_data_in(ctx, phi_o, grad_o);
            auto kern = in_step     ? k_step2d<T, KIND, MIX, PSI, kBcInflow>
                        : ctx->face ? k_step2d<T, KIND, MIX, PSI, kBcFace>
                                    : k_step2d<T, KIND, MIX, PSI, kBcNone>;
            hipLaunchKernelGGL(kern, dim3(blocks), dim3(kBlock), 0, s, ctx->g, p, st, dt,
                               inflow_data<T>(ctx), (const T *)tab, (const T *)phi,
                               (const T *)grad, (T *)phi_o, (T *)grad_o);
            return hipGetLastError();
        }
    } else {
        if constexpr (KIND == GALS_VEL_LEVEQUE3D) {
            hipLaunchKernelGGL((k_step3d<T, KIND, MIX, PSI>), dim3(band_blocks3d(ctx->g)),
                               dim3(kBlock), 0, s,
                               ctx->g, p, st, dt, (const T *)tab, (const T *)phi, (const T *)grad, (T *)phi_o,
                               (T *)grad_o);
            return hipGetLastError();
        }
    }
    return hipErrorInvalidValue;
}

template <typename T, int MIX, int PSI>
static hipError_t launch_kind(const gals_ctx *ctx, const Vel<T> &p, const void *phi,
                              const void *grad, void *phi_o, void *grad_o, double dt, double c1,
                              double c2, double c3, const void *tab, hipStream_t s)
{
#define GALS_KIND_CASE(K)                                                                         \
    case K:                                                                                       \
        return launch_typed<T, K, MIX, PSI>(ctx, p, phi, grad, phi_o, grad_o, dt, c1, c2, c3, tab, \
                                            s);
    switch (ctx->vel_kind) {
        GALS_KIND_CASE(GALS_VEL_AFFINE)
        GALS_KIND_CASE(GALS_VEL_VORTEX)
        GALS_KIND_CASE(GALS_VEL_PSEUDO1D)
        GALS_KIND_CASE(GALS_VEL_LEVEQUE3D)
    default:
        return hipErrorInvalidValue;
    }
#undef GALS_KIND_CASE
}

hipError_t launch_step(const gals_ctx *ctx, const void *phi, const void *grad, void *phi_o,
                       void *grad_o, double dt, double c1, double c2, double c3,
                       const void *coltab, const void *rowtab, hipStream_t s)
{
    const bool stream = ctx->vel_kind == GALS_VEL_STREAM_SIN && coltab && rowtab;
    const bool vecpot = ctx->dim == 3 && ctx->vel_kind == GALS_VEL_VECPOT_SIN && coltab;
    hipError_t e = with_modes(ctx->mixed, ctx->psi, [&](auto mix, auto psi) -> hipError_t {
        constexpr int MIX = decltype(mix)::value, PSI = decltype(psi)::value;
        if (vecpot)
            return ctx->prec == GALS_F32
                       ? launch_vecpot<float, MIX, PSI>(ctx, ctx->vf, phi, grad, phi_o, grad_o,
                                                        dt, c1, c2, c3, coltab, s)
                       : launch_vecpot<double, MIX, PSI>(ctx, ctx->vd, phi, grad, phi_o, grad_o,
                                                         dt, c1, c2, c3, coltab, s);
        if (stream)
            return ctx->prec == GALS_F32
                       ? launch_stream<float, MIX, PSI>(ctx, ctx->vf, phi, grad, phi_o, grad_o,
                                                        dt, c1, c2, c3, coltab, rowtab, s)
                       : launch_stream<double, MIX, PSI>(ctx, ctx->vd, phi, grad, phi_o, grad_o,
                                                         dt, c1, c2, c3, coltab, rowtab, s);
        return ctx->prec == GALS_F32
                   ? launch_kind<float, MIX, PSI>(ctx, ctx->vf, phi, grad, phi_o, grad_o, dt, c1,
                                                  c2, c3, coltab, s)
                   : launch_kind<double, MIX, PSI>(ctx, ctx->vd, phi, grad, phi_o, grad_o, dt, c1,
                                                   c2, c3, coltab, s);
    });
    // k_step2d has treated its boundary nodes, except with data in its own output
    if ((ctx->vel_kind == GALS_VEL_VORTEX || ctx->vel_kind == GALS_VEL_PSEUDO1D) &&
        !inflow_data_in(ctx, phi_o, grad_o))
        return e;
    if (e == hipSuccess && ctx->inflow) e = launch_inflow(ctx, phi_o, grad_o, c1, dt, s);
    if (e == hipSuccess && ctx->face)
        e = launch_face(ctx, phi, grad, phi_o, grad_o, dt, c1, c2, c3, s);
    return e;
}

}  // namespace gals
