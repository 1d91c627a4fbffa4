// vlct.hip -- one VL+CT step of 3D ideal MHD on gfx950 (Caddy & Schneider,
// "Cholla-MHD", Sec. 2.2) behind the C ABI of include/vlct.h.
//
// Step structure (all kernels on the caller's stream, state resident in HBM):
//   U^n       : the whole predictor (Steps 2-5) in one kernel, writing U^{n+1/2}
//               and its primitives; their ghost layers
//   U^{n+1/2} : x, y, z: reconstruction + HLLD, the hydro fluxes taken off the
//               cells, the face EMFs stored -> CT edge EMFs + faces, with the
//               per-block CFL maxima of the new state -> final next-dt
//               reduction (an in-place step reduces the CFL condition in a
//               kernel of its own)
// Boundary conditions enter through index mapping (wrap / clamp): in the
// predictor's loads, in the ghost layers of the half-step primitives, and when
// the stored normal field is read.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <unordered_map>
#include <vector>

#include "batch_tune.hpp"
#include "vlct_common.hpp"
#include "mhd_physics.hpp"

namespace vlct {

// ---------------------------------------------------------------------------
// logical block counts of the kernels (host launches and batch offsets)
// ---------------------------------------------------------------------------
constexpr int kRowCells = kBlock - 2;  // cells a block of the x kernel updates

// tile variants a batched step can give each instance (its plan byte: CT tile
// in the low nibble, march segment in the high nibble); variant 0 is the
// size-dependent choice for the instance's share of the chip, the others fix
// the block's columns (ring included) at 32 x 16 and 16 x 32, the segment at 32
// and 8 cells
constexpr int kCtVariants = 3;
constexpr int kMarchVariants = 3;  // march segments: automatic, 32 and 8 cells
constexpr int kCtThreads = 512;

__host__ __device__ __forceinline__ idx_t nblk_prims(const Geom &g)
{
    return ((idx_t)g.p[0] * g.p[1] * g.p[2] + kBlock - 1) / kBlock;
}
__host__ __device__ __forceinline__ idx_t nblk_row(const Geom &g)
{
    const idx_t items = (idx_t)(g.n[0] + 2) * (g.n[1] + 2) * (g.n[2] + 2);
    return (items - 1 + kRowCells - 1) / kRowCells;
}
__host__ __device__ __forceinline__ idx_t nblk_march(const Geom &g, int d)
{
    const int t = d == 1 ? 2 : 1;
    const idx_t cols = (idx_t)(g.n[0] + 2) * (g.n[t] + 2);
    return ((cols + kBlock - 1) / kBlock) * ((g.n[d] + g.march[d] - 1) / g.march[d]);
}
__host__ __device__ __forceinline__ idx_t nblk_ct(const Geom &g)
{
    return ct_tiles(g) * ((g.n[2] + g.ct_planes - 1) / g.ct_planes);
}
__host__ __device__ __forceinline__ idx_t nblk_dt(const Geom &g)
{
    return ((idx_t)g.n[0] * g.n[1] * g.n[2] + kBlock - 1) / kBlock;
}

// ---------------------------------------------------------------------------
// primitive variables on the ghost-padded grid (Sec. 2.1; B_cc = face average,
// Step 1); the boundary conditions are applied here by index mapping
// ---------------------------------------------------------------------------
// primitives of one cell from its conserved variables u and cell-centred
// field, floored (the conserved state is never changed); returns the floor
// status bits
__device__ __forceinline__ uint32_t prims_of(const Geom &g, const double u[5], double bcx,
                                             double bcy, double bcz, double w[8])
{
    double d = u[0];
    uint32_t st = 0;
    if (!(d >= kFloorRho)) { d = kFloorRho; st |= kStatusDensityFloor; }
    const double id = mrcp(d);
    const double vx = u[1] * id, vy = u[2] * id, vz = u[3] * id;
    const double ke = 0.5 * d * (vx * vx + vy * vy + vz * vz);
    const double me = 0.5 * (bcx * bcx + bcy * bcy + bcz * bcz);
    double pr = (g.gamma - 1.0) * (u[4] - ke - me);
    if (!(pr >= kFloorP)) { pr = kFloorP; st |= kStatusPressureFloor; }
    w[0] = d;
    w[1] = vx;
    w[2] = vy;
    w[3] = vz;
    w[4] = pr;
    w[5] = bcx;
    w[6] = bcy;
    w[7] = bcz;
    return st;
}

// primitives of padded cell (i, j, k), i, j, k in [-G, n + G - 1], with the
// boundary conditions applied by index mapping
__device__ __forceinline__ uint32_t prims_cell(const Geom &g, const StateP &s, const Prims &P,
                                               int i, int j, int k)
{
    const int mi = map_cell(i, g.n[0], g.bc[0]);
    const int mj = map_cell(j, g.n[1], g.bc[1]);
    const int mk = map_cell(k, g.n[2], g.bc[2]);
    const idx_t c = cell_store(g, mi, mj, mk);
    const double bx0 = s.b[0][face_store(g, 0, map_face(i, g.n[0], g.bc[0]), mj, mk)];
    const double bx1 = s.b[0][face_store(g, 0, map_face(i + 1, g.n[0], g.bc[0]), mj, mk)];
    const double by0 = s.b[1][face_store(g, 1, mi, map_face(j, g.n[1], g.bc[1]), mk)];
    const double by1 = s.b[1][face_store(g, 1, mi, map_face(j + 1, g.n[1], g.bc[1]), mk)];
    const double bz0 = s.b[2][face_store(g, 2, mi, mj, map_face(k, g.n[2], g.bc[2]))];
    const double bz1 = s.b[2][face_store(g, 2, mi, mj, map_face(k + 1, g.n[2], g.bc[2]))];
    const double u[5] = {s.u[0][c], s.u[1][c], s.u[2][c], s.u[3][c], s.u[4][c]};
    double w[8];
    const uint32_t st = prims_of(g, u, 0.5 * (bx0 + bx1), 0.5 * (by0 + by1), 0.5 * (bz0 + bz1), w);
    const idx_t o = pidx(g, i, j, k);
#pragma unroll
    for (int q = 0; q < 8; ++q) P.w[q][o] = w[q];
    return st;
}

__device__ __forceinline__ void prims_body(const Geom &g, const StateP &s, const Prims &P,
                                           uint32_t *status, u32 b)
{
    const u32 px = g.p[0], py = g.p[1];
    const u32 t = b * (u32)kBlock + threadIdx.x;
    if (t >= px * py * (u32)g.p[2]) return;
    const u32 r = t / px, k = r / py;
    const int pi = (int)(t - r * px), pj = (int)(r - k * py), pk = (int)k;
    const uint32_t st = prims_cell(g, s, P, pi - kGhost, pj - kGhost, pk - kGhost);
    if (st && status) atomicOr(status, st);
}

// ghost layers only: the padded cells outside the grid, enumerated as the
// z-ghost planes, then the y-ghost rows of interior planes, then the x-ghost
// cells of interior rows
__host__ __device__ __forceinline__ idx_t ghost_cells(const Geom &g)
{
    return (idx_t)g.p[0] * g.p[1] * g.p[2] - (idx_t)g.n[0] * g.n[1] * g.n[2];
}

// A ghost cell across periodic boundaries alone is a copy of its image; one
// beyond an outflow boundary has its own cell-centred field (the boundary
// face's) and is derived again.  Bound by memory, 16 doubles per cell, and by
// the index arithmetic, hence 32-bit (fewer than 2^32 padded cells fit the
// card): 256^3 94 -> 72 us, 128^3 25 -> 21, 64 runs of 16..96 193 -> 160.
__device__ __forceinline__ void prims_ghost_body(const Geom &g, const StateP &s, const Prims &P,
                                                 uint32_t *status, u32 b)
{
    const u32 t = b * (u32)kBlock + threadIdx.x;
    if (t >= (u32)ghost_cells(g)) return;
    const u32 px = g.p[0], py = g.p[1], G2 = 2 * kGhost;
    const u32 n1 = G2 * px * py, n2 = (u32)g.n[2] * G2 * px;
    int i, j, k;
    if (t < n1) {
        const u32 row = t / px, q = row / py;
        k = (int)q < kGhost ? (int)q - kGhost : g.n[2] + (int)q - kGhost;
        j = (int)(row - q * py) - kGhost;
        i = (int)(t - row * px) - kGhost;
    } else if (t < n1 + n2) {
        const u32 r = t - n1, row = r / px;
        const int q = (int)(row % G2);
        k = (int)(row / G2);
        j = q < kGhost ? q - kGhost : g.n[1] + q - kGhost;
        i = (int)(r - row * px) - kGhost;
    } else {
        const u32 r = t - n1 - n2, row = r / G2;
        const int q = (int)(r - row * G2);
        k = (int)(row / (u32)g.n[1]);
        j = (int)(row - (u32)k * (u32)g.n[1]);
        i = q < kGhost ? q - kGhost : g.n[0] + q - kGhost;
    }
    const int mi = map_cell(i, g.n[0], g.bc[0]), mj = map_cell(j, g.n[1], g.bc[1]),
              mk = map_cell(k, g.n[2], g.bc[2]);
    if ((mi == i || g.bc[0] == VLCT_BC_PERIODIC) && (mj == j || g.bc[1] == VLCT_BC_PERIODIC) &&
        (mk == k || g.bc[2] == VLCT_BC_PERIODIC)) {
        const idx_t o = pidx(g, i, j, k), m = pidx(g, mi, mj, mk);
        double w[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) w[q] = P.w[q][m];
#pragma unroll
        for (int q = 0; q < 8; ++q) P.w[q][o] = w[q];
        return;
    }
    const uint32_t st = prims_cell(g, s, P, i, j, k);
    if (st && status) atomicOr(status, st);
}

// some value, without an instruction to set it: for registers that lanes
// without a part in a step leave unused
__device__ __forceinline__ double any_value() { return __builtin_nondeterministic_value(0.0); }

// position of a block's thread in a box of rows of X items (x fastest) and Y
// rows per plane: block-uniform first plane k0, then the thread's column,
// row and plane past k0
struct BoxPos {
    u32 k0, c, j, dk;
};
__device__ __forceinline__ BoxPos box_pos(u32 q0, u32 X, u32 Y)
{
    const u32 row0 = q0 / X, e = q0 - row0 * X + threadIdx.x, dr = row_div(e, X);
    BoxPos p;
    p.k0 = row0 / Y;
    const u32 r = row0 - p.k0 * Y + dr;
    p.dk = row_div(r, Y);
    p.j = r - p.dk * Y;
    p.c = e - dr * X;
    return p;
}

// ---------------------------------------------------------------------------
// corrector (Steps 6, 7 and the cells of Step 9).  Every cell is reconstructed
// once per axis and its two interface states feed the faces on either side;
// the hydro fluxes of a face end in the flux differences of its two cells on
// chip, so the x, y and z kernels hand the partly updated cells on (out.u =
// base - x, then - y, then - z) and store only the faces' EMFs and upwind
// indicators for the CT update.  Per cell that is 5 doubles read and written
// per axis and 2 stored per face, where storing the fluxes took 7 written and
// 5 read back per face and the cells again (795 -> about 700 bytes per cell
// for the whole corrector, and the CT update keeps none of the hydro work).
// The linear reconstructions run near the copy rate of the card (256^3 PLMC
// 0.68-0.73 ms per axis, 3.9 of 4.7 TB/s; 0.58-0.60 ms when the fluxes were
// stored, with the CT update at 1.42 instead of 0.76 ms), the parabolic ones
// at FP64 issue with two waves per SIMD (PPMC 1.07-1.22 ms).
// ---------------------------------------------------------------------------
template <int RECON>
struct Recon {
    static constexpr bool kChar = RECON == VLCT_RECON_PLMC || RECON == VLCT_RECON_PPMC;
    static constexpr int R = RECON == VLCT_RECON_PCM ? 0  // stencil radius
                             : RECON == VLCT_RECON_PLMC || RECON == VLCT_RECON_PLMP ? 1 : 2;
    // waves per SIMD the marches are held to (512 / waves registers)
    static constexpr int kWaves = R == 0 ? 3 : 2;
    // interface states of the middle cell of the window, floored
    static __device__ __forceinline__ uint32_t states(const W7 *win, double bn, double gam, W7 &fm,
                                                      W7 &fp)
    {
        if constexpr (R == 0) {
            fm = fp = win[0];
            return 0;  // floored already
        } else {
            if constexpr (R == 1)
                plmc<kChar>(win[0], win[1], win[2], bn, gam, fm, fp);
            else
                ppmc<kChar>(win[0], win[1], win[2], win[3], win[4], bn, gam, fm, fp);
            const uint32_t st = floor_state(fm);
            return st | floor_state(fp);
        }
    }
};

// x axis: items = (row, cell) with cells -1..nx of every row (j in [-1, ny],
// k in [-1, nz]) in one flat sequence; a block reconstructs 256 consecutive
// items, solves the face between each item and its left neighbour in the same
// row (the high-face states go to the right through LDS) and updates the 254
// cells whose two faces it has (the fluxes go to the left through LDS);
// consecutive blocks overlap by two items
template <int RECON>
__device__ __forceinline__ void recon_x_body(const Geom &g, const StateP &s, const Prims &P,
                                             const Flux &F, const StateP &base, const StateW &out,
                                             const double *dt_dev, uint32_t *status, u32 b)
{
    constexpr int R = Recon<RECON>::R;
    __shared__ double lds[7][kBlock];
    const u32 nx = g.n[0], ny = g.n[1], nz = g.n[2];
    const u32 per_row = nx + 2, Y = ny + 2;
    const int t = threadIdx.x;
    const BoxPos p = box_pos(b * kRowCells, per_row, Y);
    const u32 k1 = p.k0 + p.dk;  // k + 1
    const bool have = k1 < nz + 2;
    const bool mine = t >= 1 && t <= kRowCells;  // the item this block answers for
    const bool cell = have && mine && p.c >= 1 && p.c <= nx && p.j >= 1 && p.j <= ny && k1 >= 1 &&
                      k1 <= nz;
    const u32 kb = p.k0 >= 1 ? p.k0 - 1 : 0;  // first interior plane of the block
    const idx_t ub = (idx_t)kb * ny * nx;
    const u32 uo = 8u * (((k1 - 1 - kb) * ny + p.j - 1) * nx + p.c - 1);
    double u[5];
    if (cell) {
#pragma unroll
        for (int q = 0; q < 5; ++q) u[q] = ld8(base.u[q] + ub, uo);
    }
    W7 fm{}, fp{};
    uint32_t st = 0;
    if (have) {
        const idx_t pb = (idx_t)(p.k0 + kGhost - 1) * g.p[1] * g.p[0];
        const u32 o = 8u * ((p.dk * g.p[1] + p.j + kGhost - 1) * g.p[0] + p.c + kGhost - 1);
        W7 win[2 * R + 1];
#pragma unroll
        for (int q = 0; q <= 2 * R; ++q) {
            auto w = [&](int f) { return ld8(P.w[f] + pb, o + 8 * (q - R)); };
            win[q] = W7{w(0), w(1), w(2), w(3), w(4), w(6), w(7)};
        }
        st = Recon<RECON>::states(win, ld8(P.w[5] + pb, o), g.gamma, fm, fp);
    }
    lds[0][t] = fp.d; lds[1][t] = fp.u; lds[2][t] = fp.v; lds[3][t] = fp.w;
    lds[4][t] = fp.p; lds[5][t] = fp.by; lds[6][t] = fp.bz;
    __syncthreads();
    const bool face = t >= 1 && have && p.c >= 1;
    double f[7];
    if (face) {
        const W7 wl{lds[0][t - 1], lds[1][t - 1], lds[2][t - 1], lds[3][t - 1],
                    lds[4][t - 1], lds[5][t - 1], lds[6][t - 1]};
        const int mj = map_cell((int)p.j - 1, g.n[1], g.bc[1]);
        const int mk = map_cell((int)k1 - 1, g.n[2], g.bc[2]);
        // the stored face n of a periodic axis holds face 0's value
        const double bn = ld8(s.b[0] + face_store(g, 0, (int)p.c - 1, mj, mk), 0);
        int8_t upw;
        hlld(wl, fm, bn, g.gamma, g.gm1i, f, upw);
        if (mine) {
            const u32 X = nx + 1;
            const idx_t fb = (idx_t)p.k0 * Y * X;
            const u32 fo = (p.dk * Y + p.j) * X + p.c - 1;
            st8(F.e[0][0] + fb, 8u * fo, -f[5]);
            st8(F.e[0][1] + fb, 8u * fo, f[6]);
            st1(F.sg[0] + fb, fo, upw);
        }
    }
    __syncthreads();
    if (face) {
#pragma unroll
        for (int q = 0; q < 5; ++q) lds[q][t] = f[q];
    }
    __syncthreads();
    if (cell) {
        const double cx = dt_dev[0] / g.dl[0];
#pragma unroll
        for (int q = 0; q < 5; ++q) st8(out.u[q] + ub, uo, u[q] - cx * (lds[q][t + 1] - f[q]));
    }
    if (st && status) atomicOr(status, st);
}

// y and z axes: one thread per transverse column (columns flattened with x
// fastest, so loads and stores are coalesced); each thread marches along the
// axis through a segment of Geom::march cells, keeping the stencil, the
// previous cell's high-face state and the previous face's hydro flux in
// registers (two extra reconstructions and one extra face per segment).  A
// step along the column moves three byte offsets and one pointer by strides.
template <int D, int RECON>
__device__ __forceinline__ void march_body(const Geom &g, const StateP &s, const Prims &P,
                                           const Flux &F, const StateW &out, const double *dt_dev,
                                           uint32_t *status, u32 b)
{
    constexpr int T = D == 1 ? 2 : 1;  // the transverse axis other than x
    constexpr int T1 = (D + 1) % 3, T2 = (D + 2) % 3;
    constexpr int R = Recon<RECON>::R;
    const int nD = g.n[D];
    // columns (i, it), i in [-1, nx], it in [-1, n_T], flattened with i fastest
    const u32 X2 = g.n[0] + 2;
    const u32 ncb = (X2 * (g.n[T] + 2) + kBlock - 1) / kBlock;
    const u32 nseg = (nD + g.march[D] - 1) / g.march[D];
    const u32 seg = b / ncb, cb = b - seg * ncb;
    if (seg >= nseg) return;
    const u32 it0 = cb * kBlock / X2;  // first row of columns of the block
    const u32 e = cb * kBlock - it0 * X2 + threadIdx.x, dr = row_div(e, X2);
    const u32 i1 = e - dr * X2;  // i + 1
    const int i = (int)i1 - 1, it = (int)(it0 + dr) - 1;
    if (it > g.n[T]) return;
    const int s0 = seg * g.march[D];
    const int s1 = min(s0 + g.march[D], nD);  // cells [s0, s1), faces [s0, s1]
    const bool interior = i >= 0 && i < g.n[0] && it >= 0 && it < g.n[T];
    // primitives: cell s0 - 1 - R of the column
    const u32 px = g.p[0], py = g.p[1];
    const idx_t pb = D == 1 ? ((idx_t)(it0 + kGhost - 1) * py + (s0 - 1 - R + kGhost)) * px
                            : ((idx_t)(s0 - 1 - R + kGhost) * py + (it0 + kGhost - 1)) * px;
    u32 po = 8u * ((D == 1 ? dr * px * py : dr * px) + i1 + kGhost - 1);
    const u32 pstep = 8u * (D == 1 ? px : px * py);
    auto cell = [&](u32 at) {
        auto w = [&](int q) { return ld8(P.w[q] + pb, at); };
        return W7{w(0), w(1 + D), w(1 + T1), w(1 + T2), w(4), w(5 + T1), w(5 + T2)};
    };
    // EMFs: face s0
    const u32 fx = X2, fy = g.n[1] + (D == 1 ? 1 : 2);
    const idx_t fb = D == 1 ? ((idx_t)it0 * fy + s0) * fx : ((idx_t)s0 * fy + it0) * fx;
    u32 fo = (D == 1 ? dr * fx * fy : dr * fx) + i1;
    const u32 fstep = D == 1 ? fx : fx * fy;
    // cells: cell s0
    const u32 tb = it0 >= 1 ? it0 - 1 : 0;  // first interior row of columns of the block
    const idx_t ub = D == 1 ? ((idx_t)tb * g.n[1] + s0) * g.n[0] : ((idx_t)s0 * g.n[1] + tb) * g.n[0];
    u32 uo = 8u * ((D == 1 ? (it - (int)tb) * g.n[1] * g.n[0] : (it - (int)tb) * g.n[0]) + i);
    const u32 ustep = 8u * (D == 1 ? g.n[0] : g.n[0] * g.n[1]);
    // stored normal field: face s0 (the face n of a periodic axis holds face 0's value)
    const int mt = map_cell(it, g.n[T], g.bc[T]), mi = map_cell(i, g.n[0], g.bc[0]);
    const double *nb = s.b[D] + (D == 1 ? face_store(g, 1, mi, s0, mt) : face_store(g, 2, mi, mt, s0));
    const idx_t nstep = D == 1 ? (idx_t)g.n[0] : (idx_t)g.n[0] * g.n[1];
    const double cd = uniform(dt_dev[0] / g.dl[D]);
    // stencil window of cells c-R .. c+R for c = s0 - 1
    W7 win[2 * R + 1];
#pragma unroll
    for (int q = 0; q < 2 * R + 1; ++q) {
        win[q] = cell(po);
        po += pstep;
    }
    double bnc = ld8(P.w[5 + D] + pb, po - (R + 1) * pstep);  // the middle cell's B_n
    uint32_t st = 0;
    bool bad = false;
    // the previous cell's high-face state and the previous face's hydro flux
    // wait in LDS (thread-private): 24 registers that the parabolic window
    // would otherwise spill
    __shared__ double park[12][kBlock];
    auto dopark = [&](const W7 &w) {
        double x[7];
        to_arr(w, x);
#pragma unroll
        for (int q = 0; q < 7; ++q) park[q][threadIdx.x] = x[q];
    };
    auto unpark = [&](int o) {
        const int t = threadIdx.x;
        return W7{park[o][t], park[o + 1][t], park[o + 2][t], park[o + 3][t],
                  park[o + 4][t], park[o + 5][t], park[o + 6][t]};
    };
    double bn = ld8(nb, 0);
    for (int c = s0 - 1; c <= s1; ++c) {
        W7 fm, fp;
        st |= Recon<RECON>::states(win, bnc, g.gamma, fm, fp);
        // the next cell of the window, the cell to update and the next face's
        // field, behind the Riemann solve and ahead of its stores (loads
        // return in order with the stores issued before them)
        double u[5], bn_next = any_value();
        const bool upd = interior && c > s0;  // cell c - 1
        if (upd) {
#pragma unroll
            for (int q = 0; q < 5; ++q) u[q] = ld8(out.u[q] + ub, uo);
        }
        if (c < s1) {
#pragma unroll
            for (int q = 0; q < 2 * R; ++q) win[q] = win[q + 1];
            win[2 * R] = cell(po);
            po += pstep;
            bnc = ld8(P.w[5 + D] + pb, po - (R + 1) * pstep);
            if (c >= s0) {
                nb += nstep;
                bn_next = ld8(nb, 0);
            }
        }
        if (c >= s0) {
            double f[7];
            int8_t upw;
            hlld(unpark(0), fm, bn, g.gamma, g.gm1i, f, upw);
            bn = bn_next;
            if (c < s1 || c == nD) {  // the face s1 belongs to the next segment
                st8(F.e[D][0] + fb, 8u * fo, -f[5]);
                st8(F.e[D][1] + fb, 8u * fo, f[6]);
                st1(F.sg[D] + fb, fo, upw);
            }
            fo += fstep;
            if (upd) {
                constexpr int comp[5] = {0, 1 + D, 1 + T1, 1 + T2, 4};
#pragma unroll
                for (int q = 0; q < 5; ++q) {
                    const double v = u[comp[q]] - cd * (f[q] - park[7 + q][threadIdx.x]);
                    st8(out.u[comp[q]] + ub, uo, v);
                    if (D == 2) bad |= !isfinite(v);
                }
                uo += ustep;
            }
#pragma unroll
            for (int q = 0; q < 5; ++q) park[7 + q][threadIdx.x] = f[q];
        }
        dopark(fp);
    }
    if (bad) st |= kStatusNonfinite;
    if (st && status) atomicOr(status, st);
}

// ---------------------------------------------------------------------------
// CFL condition of one cell (Step 1, Eq. dt): max_l (|v_l| + c_f,l) / d_l from
// its conserved variables and cell-centred field (face averages); floored
// rho / P as in the primitive recovery, the floors reported in `st`
// ---------------------------------------------------------------------------
__device__ __forceinline__ double cell_cfl(const Geom &g, double d, double mx, double my,
                                           double mz, double e, const double b[3], uint32_t &st)
{
    if (!(d >= kFloorRho)) { d = kFloorRho; st |= kStatusDensityFloor; }
    const double id = mrcp(d);
    const double v[3] = {mx * id, my * id, mz * id};
    const double sq[3] = {b[0] * b[0], b[1] * b[1], b[2] * b[2]};
    const double b2 = sq[0] + sq[1] + sq[2];
    const double ke = 0.5 * d * (v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
    double p = (g.gamma - 1.0) * (e - ke - 0.5 * b2);
    if (!(p >= kFloorP)) { p = kFloorP; st |= kStatusPressureFloor; }
    // c_f,l^2 = (gP + B^2 + disc_l) / (2 rho), the terms without l once
    const double gp = g.gamma * p, t2 = (gp - b2) * (gp - b2), hid = 0.5 * id;
    double m = 0.0;
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        const double disc = msqrt(t2 + 4.0 * gp * (sq[(l + 1) % 3] + sq[(l + 2) % 3]));
        const double s = fabs(v[l]) + msqrt((gp + b2 + disc) * hid);
        const double q = s * g.idl[l];
        m = fmax(m, fma(fma(-g.dl[l], q, s), g.idl[l], q));  // s / d_l
    }
    return m;
}

__device__ __forceinline__ double wave_max(double v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
    return v;
}

// ---------------------------------------------------------------------------
// CT edge EMFs (Step 4 / Step 8; Eqs. emf-edge, emf-upwind-slope, emf-slope)
// ---------------------------------------------------------------------------
__device__ __forceinline__ double upwind(int s, double lo, double hi)
{
    return s > 0 ? lo : (s < 0 ? hi : 0.5 * (lo + hi));
}

// the edge field from the EMFs and upwind indicators of its four faces and the
// reference fields of its four cells: B-faces at x0 and x0 - e_C, C-faces at
// x0 and x0 - e_B
__device__ __forceinline__ double edge_combine(double eb_c, double eb_cm, double ec_b,
                                               double ec_bm, int sb_c, int sb_cm, int sc_b,
                                               int sc_bm, double r00, double r10, double r01,
                                               double r11)
{
    const double avg = 0.25 * (eb_c + eb_cm + ec_b + ec_bm);
    const double t1 = upwind(sb_c, ec_bm - r10, ec_b - r00);
    const double t2 = upwind(sb_cm, ec_bm - r11, ec_b - r01);
    const double t3 = upwind(sc_b, eb_cm - r01, eb_c - r00);
    const double t4 = upwind(sc_bm, eb_cm - r11, eb_c - r10);
    return avg + 0.25 * (t1 + t2 + t3 + t4);
}

// ---------------------------------------------------------------------------
// CT update (Steps 8-9: edge fields and faces).  A block marches along z
// through Geom::ct_planes planes of a column tile; a thread owns one column of
// the tile or of its one-cell ring, and per new plane m
//   (A) shares the reference field -(v x B) of its cell and the EMFs and
//       upwind indicators of its low faces that the neighbours need (LDS);
//   (C) forms the three edge fields at its cell's low edges, E_z of plane m,
//       E_x and E_y of the half plane m - 1/2, from its own registers and one
//       neighbour each way, and shares them;
//   (D) finishes the faces of plane m - 1 and starts those of plane m.
// Two barriers per plane; the next plane's loads fly during (D) and, with two
// blocks per CU (126 registers, 67 KB of LDS), behind the other block's work.
// Bound by load latency: 187 bytes per cell at 256^3 in 0.76 ms (4.1 TB/s),
// 1.42 ms for the form with the hydro update and the edges dealt out by
// division from global memory; 32^3 37 -> 21 us.
// DT: the CFL condition of the updated cells is reduced on the way, one
// maximum per block into partial[b]: the ring's columns finish the high faces
// of the tile too (in the arithmetic of the blocks that own them), plane m - 1
// shares its finished faces, and its cells are evaluated after the next
// barrier.  An in-place step runs without it (the high faces' base values may
// have been overwritten by their owners) and reduces the CFL condition apart.
// ---------------------------------------------------------------------------
template <bool DT>
__device__ __forceinline__ void ct_body(const Geom &g, const Prims &P, const Flux &F,
                                        const StateP &base, const StateW &out,
                                        const double *dt_dev, uint32_t *status, u32 b,
                                        double *partial)
{
    constexpr int N = kCtThreads;
    __shared__ double s_rx[2][N], s_ry[2][N], s_rz[N];  // -(v x B): x, y of planes m - 1, m (slot m & 1), z
    __shared__ double s_xz[N], s_yz[N], s_zy[N], s_zx[N];  // EMFs: E_z of x- and y-faces, E_y and E_x of z-faces
    __shared__ int8_t s_sx[N], s_sy[N], s_sz[N];
    __shared__ double s_ez[N], s_ex[2][N], s_ey[2][N];  // edge fields (half planes: slot m & 1)
    __shared__ double s_bx[DT ? N : 1], s_by[DT ? N : 1];  // finished low x-, y-faces of plane m - 1
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    // positions owned by threads: cells/faces i in [0, ex), j in [0, ey)
    const int ex = nx + (g.bc[0] == VLCT_BC_OUTFLOW), ey = ny + (g.bc[1] == VLCT_BC_OUTFLOW);
    const int TX = g.ct_tx, TY = g.ct_ty, CX = TX + 2;
    const u32 ntx = (ex + TX - 1) / TX, nty = (ey + TY - 1) / TY;
    const u32 zb = b / (ntx * nty), tile = b - zb * (ntx * nty);
    const int k0 = __builtin_amdgcn_readfirstlane(zb * g.ct_planes);
    if (k0 >= nz) return;
    const int k1 = min(k0 + g.ct_planes, nz);
    const int i0 = (tile % ntx) * TX, j0 = (tile / ntx) * TY;
    const int t = threadIdx.x, c = t / CX, a = t - c * CX;
    const int ii = i0 - 1 + a, jj = j0 - 1 + c;
    const bool live = c < TY + 2 && ii <= nx && jj <= ny;
    const bool edge = live && a >= 1 && c >= 1;
    const bool own = edge && a <= TX && c <= TY && ii < ex && jj < ey;
    const bool interior = own && ii < nx && jj < ny;
    // low faces this thread finishes (and stores where it owns the position)
    const bool xface = edge && c <= TY && jj < ny && (DT || own);
    const bool yface = edge && a <= TX && ii < nx && (DT || own);
    const int lx = t - 1, ly = t - CX;
    const double dt = dt_dev[0];
    const double cx = uniform(dt / g.dl[0]), cy = uniform(dt / g.dl[1]), cz = uniform(dt / g.dl[2]);
    // byte offsets of the column in a plane of each array
    u32 op = 8u * (u32)((jj + kGhost) * g.p[0] + ii + kGhost);
    u32 oc = 8u * (u32)(jj * nx + ii);
    u32 ox = 8u * (u32)(jj * (nx + 1) + map_face(ii, nx, g.bc[0]));
    u32 oy = 8u * (u32)(map_face(jj, ny, g.bc[1]) * nx + ii);
    // (the ring's first columns have no low x- or y-face: those of the next are read)
    u32 fxo = (u32)((jj + 1) * (nx + 1) + max(ii, 0)), fyo = (u32)(max(jj, 0) * (nx + 2) + ii + 1);
    u32 fzo = (u32)((jj + 1) * (nx + 2) + ii + 1);
    const idx_t sp = (idx_t)g.p[0] * g.p[1], sc = (idx_t)nx * ny;
    const idx_t sbx = (idx_t)(nx + 1) * ny, sby = (idx_t)nx * (ny + 1);
    const idx_t sfx = (idx_t)(nx + 1) * (ny + 2), sfy = (idx_t)(nx + 2) * (ny + 1);
    const idx_t sfz = (idx_t)(nx + 2) * (ny + 2);
    const idx_t pstep = P.w[1] - P.w[0];  // the primitive arrays are equally spaced

    // plane m: velocity and field, EMFs and indicators of the low faces, base faces
    double w[6], em[6], bf[3];
    int sg[3] = {0, 0, 0};
    auto load_plane = [&](int m) {
        if (live) {
            const idx_t o = (idx_t)(m + kGhost) * sp;
#pragma unroll
            for (int q = 0; q < 6; ++q) w[q] = ld8(P.w[0] + ((q < 3 ? 1 + q : 2 + q) * pstep + o), op);
            const idx_t px = (idx_t)(m + 1) * sfx, py = (idx_t)(m + 1) * sfy, pz = (idx_t)m * sfz;
            em[0] = ld8(F.e[0][0] + px, 8u * fxo);
            em[1] = ld8(F.e[0][1] + px, 8u * fxo);
            em[2] = ld8(F.e[1][0] + py, 8u * fyo);
            em[3] = ld8(F.e[1][1] + py, 8u * fyo);
            sg[0] = ld1(F.sg[0] + px, fxo);
            sg[1] = ld1(F.sg[1] + py, fyo);
            if (m >= k0) {
                em[4] = ld8(F.e[2][0] + pz, 8u * fzo);
                em[5] = ld8(F.e[2][1] + pz, 8u * fzo);
                sg[2] = ld1(F.sg[2] + pz, fzo);
            }
        }
        if (m >= k0) {
            if (xface && m < k1) bf[0] = ld8(base.b[0] + m * sbx, ox);
            if (yface && m < k1) bf[1] = ld8(base.b[1] + m * sby, oy);
            if (interior && (DT || m < k1 || g.bc[2] == VLCT_BC_OUTFLOW))
                bf[2] = ld8(base.b[2] + map_face(m, nz, g.bc[2]) * sc, oc);
        }
    };
#pragma unroll
    for (int q = 0; q < 6; ++q) w[q] = em[q] = any_value();
#pragma unroll
    for (int q = 0; q < 3; ++q) bf[q] = any_value();
    load_plane(k0 - 1);
    // of plane m - 1: own EMFs and indicators, the low x- and y-face short of
    // their E_y and E_x terms and the finished low z-face
    double xy_p = any_value(), yx_p = any_value(), bxp = any_value(), byp = any_value();
    double bzp = any_value();
    // of the plane whose CFL condition is due: the cells and B_cc,z
    double u[5], bcz = any_value();
#pragma unroll
    for (int q = 0; q < 5; ++q) u[q] = any_value();
    int sx_p = 0, sy_p = 0;
    bool bad = false;
    double mcfl = 0.0;
    uint32_t stcfl = 0;
    auto cfl = [&]() {
        const double bcc[3] = {0.5 * (s_bx[t] + s_bx[t + 1]), 0.5 * (s_by[t] + s_by[t + CX]), bcz};
        mcfl = fmax(mcfl, cell_cfl(g, u[0], u[1], u[2], u[3], u[4], bcc, stcfl));
    };
    for (int m = k0 - 1; m <= k1; ++m) {
        const int hi = m & 1, lo = hi ^ 1;
        pin(op), pin(oc), pin(ox), pin(oy), pin(fxo), pin(fyo), pin(fzo);
        // (A)
        const double xz = em[0], xy = em[1], yx = em[2], yz = em[3], zy = em[4], zx = em[5];
        const int sx = sg[0], sy = sg[1], sz = sg[2];
        const double bx0 = bf[0], by0 = bf[1], bz0 = bf[2];
        if (live) {
            s_rx[hi][t] = -(w[1] * w[5] - w[2] * w[4]);
            s_ry[hi][t] = -(w[2] * w[3] - w[0] * w[5]);
            s_rz[t] = -(w[0] * w[4] - w[1] * w[3]);
            s_xz[t] = xz;
            s_yz[t] = yz;
            s_zy[t] = zy;
            s_zx[t] = zx;
            s_sx[t] = (int8_t)sx;
            s_sy[t] = (int8_t)sy;
            s_sz[t] = (int8_t)sz;
        }
        __syncthreads();
        // (C)
        if (DT && interior && m > k0 + 1) cfl();
        if (edge) {
            // E_z at (ii - 1/2, jj - 1/2, m): x-faces here and at jj - 1, y-faces here and at ii - 1
            s_ez[t] = edge_combine(xz, s_xz[ly], yz, s_yz[lx], sx, s_sx[ly], sy, s_sy[lx], s_rz[t],
                                   s_rz[lx], s_rz[ly], s_rz[ly - 1]);
            // E_x at (ii, jj - 1/2, m - 1/2): y-faces of planes m, m - 1, z-faces here and at jj - 1
            s_ex[hi][t] = edge_combine(yx, yx_p, zx, s_zx[ly], sy, sy_p, sz, s_sz[ly], s_rx[hi][t],
                                       s_rx[hi][ly], s_rx[lo][t], s_rx[lo][ly]);
            // E_y at (ii - 1/2, jj, m - 1/2): z-faces here and at ii - 1, x-faces of planes m, m - 1
            s_ey[hi][t] = edge_combine(zy, s_zy[lx], xy, xy_p, sz, s_sz[lx], sx, sx_p, s_ry[hi][t],
                                       s_ry[lo][t], s_ry[hi][lx], s_ry[lo][lx]);
        }
        xy_p = xy;
        yx_p = yx;
        sx_p = sx;
        sy_p = sy;
        // the next plane, behind the updates (and not above the edge work, whose
        // registers it would take)
        __builtin_amdgcn_sched_barrier(0);
        if (m < k1) load_plane(m + 1);
        __syncthreads();
        // (D)
        const idx_t k = m - 1;
        if (DT && interior && m > k0) {
#pragma unroll
            for (int q = 0; q < 5; ++q) u[q] = ld8(out.u[q] + k * sc, oc);
        }
        double bzn = any_value();
        if (interior) {
            bzn = bz0 - cx * (s_ey[hi][t + 1] - s_ey[hi][t]) + cy * (s_ex[hi][t + CX] - s_ex[hi][t]);
            if (m >= k0 && (m < k1 || (m == nz && g.bc[2] == VLCT_BC_OUTFLOW))) {
                st8(out.b[2] + m * sc, oc, bzn);
                if (g.bc[2] == VLCT_BC_PERIODIC && m == 0) st8(out.b[2] + nz * sc, oc, bzn);
                bad |= !isfinite(bzn);
            }
            bcz = 0.5 * (bzp + bzn);
        }
        if (m > k0) {
            if (xface) {  // face x (ii - 1/2, jj, k)
                const double v = bxp + cz * (s_ey[hi][t] - s_ey[lo][t]);
                if (DT) s_bx[t] = v;
                if (own) {
                    st8(out.b[0] + k * sbx, ox, v);
                    if (g.bc[0] == VLCT_BC_PERIODIC && ii == 0) st8(out.b[0] + k * sbx, ox + 8u * (u32)nx, v);
                    bad |= !isfinite(v);
                }
            }
            if (yface) {  // face y (ii, jj - 1/2, k)
                const double v = byp - cz * (s_ex[hi][t] - s_ex[lo][t]);
                if (DT) s_by[t] = v;
                if (own) {
                    st8(out.b[1] + k * sby, oy, v);
                    if (g.bc[1] == VLCT_BC_PERIODIC && jj == 0)
                        st8(out.b[1] + k * sby, oy + 8u * (u32)(nx * ny), v);
                    bad |= !isfinite(v);
                }
            }
        }
        // start plane m
        if (xface) bxp = bx0 - cy * (s_ez[t + CX] - s_ez[t]);
        if (yface) byp = by0 + cx * (s_ez[t + 1] - s_ez[t]);
        bzp = bzn;
    }
    if (DT) {
        __syncthreads();
        if (interior) cfl();
    }
    if (bad && status) atomicOr(status, kStatusNonfinite);
    if (DT) {
        if (stcfl && status) atomicOr(status, stcfl);
        __shared__ double red[N / 64];
        const double mx = wave_max(mcfl);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
        __syncthreads();
        if (threadIdx.x == 0) {
            double r = red[0];
            for (int q = 1; q < N / 64; ++q) r = fmax(r, red[q]);
            partial[b] = r;
        }
    }
}

// ---------------------------------------------------------------------------
// fused predictor (Steps 2-5 in one kernel): a block marches along z through
// the planes [k0, k1) of a column tile (Geom::pr_tx x pr_ty columns and
// pred_slab planes); neighbouring tiles of a slab are neighbouring blocks, so
// that they share their ring columns in L2.  A thread owns one column of the
// tile or of its one-cell ring, and per new plane m
//   (A) derives the primitives (Sec. 2.1, B_cc = face average, floors) and
//       the reference field -(v x B) of its cell into LDS;
//   (B) solves PCM HLLD on its cell's low x- and y-faces and on the z-face
//       m - 1/2 (Steps 2-3); hydro fluxes and what the neighbours need of the
//       face EMFs and upwind indicators go to LDS;
//   (C) forms the three edge fields at its cell's low edges: E_z of plane m,
//       E_x and E_y of the half plane m - 1/2 (Step 4, Eqs. emf-edge,
//       emf-upwind-slope, emf-slope), and takes the x and y flux differences
//       off its cell of plane m;
//   (D) finishes the cell and the faces of plane m - 1 (Step 5), derives the
//       half-step primitives of that cell for the corrector, and starts the
//       faces of plane m.
// What a thread alone uses of a plane stays in its registers until the next
// (its own EMFs, references, partial updates), so U^n is read once, each
// plane's three barriers separate LDS writes from reads and none closes the
// plane, and the next plane's U^n is loaded before (C), its latency behind the
// edge and update work.  The block also evaluates the faces of the planes
// k0 - 1 and k1 (the edges of its first and last half planes need them).
// Arithmetic per quantity is that of k_prims and k_ct_update, whatever the
// tiles.
//
// One block per CU (133 KB of LDS, 256 registers: two waves per SIMD), bound
// by FP64 issue and by the latency of three dependent Riemann solves between
// barriers.  Against the form that kept every EMF and reference of two planes
// in LDS, dealt the edges out by division and loaded U^n twice per plane
// (2321 vector instructions, 116 LDS accesses; now 1801 and 81): 256^3 2.04 ->
// 1.54 ms, 128^3 0.284 -> 0.225 ms, 32^3 52 -> 45 us (19 with tiles of 256
// threads and one plane).
// ---------------------------------------------------------------------------
constexpr int kPredThreads = 512;

// side0..2 (optional): the upwind side of every interior face, tape layout;
// a run-time choice of one kernel, so a taped step runs the very code of a
// plain one.  P: the half-step primitives of the interior cells are written
// there as k_prims would derive them from U^{n+1/2}; its ghost layers are left
// to k_prims_ghost.
// Block b is the run of tile b mod ntiles through z slab b / ntiles.
__device__ __forceinline__ void pred_body(const Geom &g, const StateP &s, const StateW &out,
                                          const Prims &P, const double *dt_dev, uint32_t *status,
                                          u32 b, uint8_t *side0, uint8_t *side1, uint8_t *side2)
{
    const int TX = g.pr_tx, TY = g.pr_ty, CX = TX + 2;  // columns along x with the ring
    constexpr int N = kPredThreads;
    __shared__ double s_pr[8][N];             // primitives of plane m
    __shared__ double s_rx[2][N], s_ry[2][N], s_rz[N];  // -(v x B): x, y of planes m - 1, m (slot m & 1), z
    __shared__ double s_fx[5][N], s_fy[5][N]; // hydro fluxes of the low x-, y-faces
    __shared__ double s_xz[N], s_yz[N];       // E_z EMFs of the x-faces (-F[B_y]), y-faces (F[B_x])
    __shared__ double s_zy[N], s_zx[N];       // E_y (-F[B_x]), E_x (F[B_y]) EMFs of the z-faces
    __shared__ int8_t s_sx[N], s_sy[N], s_sz[N];        // upwind indicators
    __shared__ double s_ez[N], s_ex[2][N], s_ey[2][N];  // edge fields (half planes: slot m & 1)

    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    const int ex = nx + (g.bc[0] == VLCT_BC_OUTFLOW), ey = ny + (g.bc[1] == VLCT_BC_OUTFLOW);
    const u32 ntx = (ex + TX - 1) / TX, nty = (ey + TY - 1) / TY, ntiles = ntx * nty;
    const u32 slab = b / ntiles, tile = b - slab * ntiles;
    const int k0 = __builtin_amdgcn_readfirstlane(slab * g.pred_slab);
    if (k0 >= nz) return;
    const int k1 = min(k0 + g.pred_slab, nz);
    const double dt = 0.5 * dt_dev[0];
    const double cx = uniform(dt / g.dl[0]), cy = uniform(dt / g.dl[1]), cz = uniform(dt / g.dl[2]);

    // this thread's column: (a, c) in the tile with its ring
    const int t = threadIdx.x;
    const int c = t / CX, a = t - c * CX;
    uint32_t st = 0;
    const int i0 = (int)(tile % ntx) * TX, j0 = (int)(tile / ntx) * TY;
    // cell (ii, jj) of the column
    const int ii = i0 - 1 + a, jj = j0 - 1 + c;
    const bool live = c < TY + 2 && ii <= nx && jj <= ny;
    // columns to the left and below (the ring's first ones take themselves:
    // what they solve there is not used)
    const int lx = a >= 1 ? t - 1 : t, ly = c >= 1 ? t - CX : t;
    const bool edge = live && a >= 1 && c >= 1;
    // owned positions: cells / faces of the tile proper
    const bool own = edge && a <= TX && c <= TY && ii < ex && jj < ey;
    const bool interior = own && ii < nx && jj < ny;
    // byte offsets of the column in a plane of each array
    const int mi = map_cell(ii, nx, g.bc[0]), mj = map_cell(jj, ny, g.bc[1]);
    const int fi0 = map_face(ii, nx, g.bc[0]), fi1 = map_face(ii + 1, nx, g.bc[0]);
    const int fj0 = map_face(jj, ny, g.bc[1]), fj1 = map_face(jj + 1, ny, g.bc[1]);
    u32 oc = 8u * (u32)(mj * nx + mi);
    u32 ox0 = 8u * (u32)(mj * (nx + 1) + fi0), ox1 = 8u * (u32)(mj * (nx + 1) + fi1);
    u32 oy0 = 8u * (u32)(fj0 * nx + mi), oy1 = 8u * (u32)(fj1 * nx + mi);
    u32 op = 8u * (u32)((jj + kGhost) * g.p[0] + ii + kGhost);
    const idx_t sc = (idx_t)nx * ny, sbx = (idx_t)(nx + 1) * ny, sby = (idx_t)nx * (ny + 1);
    const idx_t sp = (idx_t)g.p[0] * g.p[1];
    // the primitives' and the output cells' arrays are equally spaced in
    // their workspace: two pointers each in scalar registers
    const idx_t pstep = P.w[1] - P.w[0], ostep = out.u[1] - out.u[0];

    // U^n of this thread's cell in a plane: 5 conserved values, the six faces
    double pf[11];
    auto load_plane = [&](int m) {
        const idx_t mk = map_cell(m, nz, g.bc[2]);
#pragma unroll
        for (int q = 0; q < 5; ++q) pf[q] = ld8(s.u[q] + mk * sc, oc);
        pf[5] = ld8(s.b[0] + mk * sbx, ox0);
        pf[6] = ld8(s.b[0] + mk * sbx, ox1);
        pf[7] = ld8(s.b[1] + mk * sby, oy0);
        pf[8] = ld8(s.b[1] + mk * sby, oy1);
        pf[9] = ld8(s.b[2] + map_face(m, nz, g.bc[2]) * sc, oc);
        pf[10] = ld8(s.b[2] + map_face(m + 1, nz, g.bc[2]) * sc, oc);
    };

    // of plane m - 1: the cell's update short of the z fluxes, the hydro flux
    // of its low z-face, its faces short of the E_x and E_y terms (low and
    // high x, y) and its finished low z-face
    double up[5], hz_lo[5], bxp = any_value(), bxhp = any_value(), byp = any_value();
    double byhp = any_value(), bzp = any_value();
#pragma unroll
    for (int q = 0; q < 5; ++q) up[q] = hz_lo[q] = any_value();
    // own EMFs and indicators of plane m - 1 for the half-plane edges
    double xy_p = any_value(), yx_p = any_value();
    int sx_p = 0, sy_p = 0;
    if (live) load_plane(k0 - 1);
    for (int m = k0 - 1; m <= k1; ++m) {
        const int hi = m & 1, lo = hi ^ 1;  // slots of the half planes m -+ 1/2
        pin(oc), pin(ox0), pin(ox1), pin(oy0), pin(oy1), pin(op);
        // (A)
        double u0[5], bx0 = any_value(), bx1 = any_value(), by0 = any_value(), by1 = any_value();
        double bz0 = any_value();
#pragma unroll
        for (int q = 0; q < 5; ++q) u0[q] = any_value();
        W7 wz_prev{any_value(), any_value(), any_value(), any_value(),
                   any_value(), any_value(), any_value()};  // own cell of plane m - 1, z sweep frame
        if (live) {
            wz_prev = W7{s_pr[0][t], s_pr[3][t], s_pr[1][t], s_pr[2][t],
                         s_pr[4][t], s_pr[5][t], s_pr[6][t]};
#pragma unroll
            for (int q = 0; q < 5; ++q) u0[q] = pf[q];
            bx0 = pf[5];
            bx1 = pf[6];
            by0 = pf[7];
            by1 = pf[8];
            bz0 = pf[9];
            double w[8];
            st |= prims_of(g, u0, 0.5 * (bx0 + bx1), 0.5 * (by0 + by1), 0.5 * (bz0 + pf[10]), w);
#pragma unroll
            for (int q = 0; q < 8; ++q) s_pr[q][t] = w[q];
            s_rx[hi][t] = -(w[2] * w[7] - w[3] * w[6]);
            s_ry[hi][t] = -(w[3] * w[5] - w[1] * w[7]);
            s_rz[t] = -(w[1] * w[6] - w[2] * w[5]);
        }
        __syncthreads();
        // (B)
        double hzn[5], xz = any_value(), xy = any_value(), yx = any_value(), yz = any_value();
        double zx = any_value(), zy = any_value();
#pragma unroll
        for (int q = 0; q < 5; ++q) hzn[q] = any_value();
        int8_t sx = 0, sy = 0, sz = 0;
        if (live) {
            double f[7];
            if (m >= k0) {
                const W7 wr{s_pr[0][t], s_pr[3][t], s_pr[1][t], s_pr[2][t],
                            s_pr[4][t], s_pr[5][t], s_pr[6][t]};
                hlld(wz_prev, wr, bz0, g.gamma, g.gm1i, f, sz);
#pragma unroll
                for (int q = 0; q < 5; ++q) hzn[q] = f[q];
                zy = -f[5];
                zx = f[6];
                s_zy[t] = zy;
                s_zx[t] = zx;
                s_sz[t] = sz;
            }
            {
                const W7 wl{s_pr[0][lx], s_pr[1][lx], s_pr[2][lx], s_pr[3][lx],
                            s_pr[4][lx], s_pr[6][lx], s_pr[7][lx]};
                const W7 wr{s_pr[0][t], s_pr[1][t], s_pr[2][t], s_pr[3][t],
                            s_pr[4][t], s_pr[6][t], s_pr[7][t]};
                hlld(wl, wr, bx0, g.gamma, g.gm1i, f, sx);
#pragma unroll
                for (int q = 0; q < 5; ++q) s_fx[q][t] = f[q];
                xz = -f[5];
                xy = f[6];
                s_xz[t] = xz;
                s_sx[t] = sx;
            }
            {
                const W7 wl{s_pr[0][ly], s_pr[2][ly], s_pr[3][ly], s_pr[1][ly],
                            s_pr[4][ly], s_pr[7][ly], s_pr[5][ly]};
                const W7 wr{s_pr[0][t], s_pr[2][t], s_pr[3][t], s_pr[1][t],
                            s_pr[4][t], s_pr[7][t], s_pr[5][t]};
                hlld(wl, wr, by0, g.gamma, g.gm1i, f, sy);
#pragma unroll
                for (int q = 0; q < 5; ++q) s_fy[q][t] = f[q];
                yx = -f[5];
                yz = f[6];
                s_yz[t] = yz;
                s_sy[t] = sy;
            }
        }
        __syncthreads();
        // (C)
        if (live && m < k1) load_plane(m + 1);
        double upn[5];
#pragma unroll
        for (int q = 0; q < 5; ++q) upn[q] = any_value();
        if (edge) {
            // E_z at (ii - 1/2, jj - 1/2, m): x-faces here and at jj - 1, y-faces here and at ii - 1
            s_ez[t] = edge_combine(xz, s_xz[ly], yz, s_yz[lx], sx, s_sx[ly], sy, s_sy[lx], s_rz[t],
                                   s_rz[lx], s_rz[ly], s_rz[ly - 1]);
            // E_x at (ii, jj - 1/2, m - 1/2): y-faces of planes m, m - 1, z-faces here and at jj - 1
            s_ex[hi][t] = edge_combine(yx, yx_p, zx, s_zx[ly], sy, sy_p, sz, s_sz[ly], s_rx[hi][t],
                                       s_rx[hi][ly], s_rx[lo][t], s_rx[lo][ly]);
            // E_y at (ii - 1/2, jj, m - 1/2): z-faces here and at ii - 1, x-faces of planes m, m - 1
            s_ey[hi][t] = edge_combine(zy, s_zy[lx], xy, xy_p, sz, s_sz[lx], sx, sx_p, s_ry[hi][t],
                                       s_ry[lo][t], s_ry[hi][lx], s_ry[lo][lx]);
        }
        xy_p = xy;
        yx_p = yx;
        sx_p = sx;
        sy_p = sy;
        if (interior) {
            auto dx = [&](int q) { return s_fx[q][t + 1] - s_fx[q][t]; };
            auto dy = [&](int q) { return s_fy[q][t + CX] - s_fy[q][t]; };
            upn[0] = u0[0] - cx * dx(0) - cy * dy(0);
            upn[1] = u0[1] - cx * dx(1) - cy * dy(3);
            upn[2] = u0[2] - cx * dx(2) - cy * dy(1);
            upn[3] = u0[3] - cx * dx(3) - cy * dy(2);
            upn[4] = u0[4] - cx * dx(4) - cy * dy(4);
            // the tape: upwind sides of the cell's low faces
            if (side0 && m >= k0 && m < k1) {
                const idx_t cc = (idx_t)m * sc + (oc >> 3);
                side0[cc] = side_code(sx);
                side1[cc] = side_code(sy);
                side2[cc] = side_code(sz);
            }
        }
        __syncthreads();
        // (D)
        double bzn = any_value();
        if (own) {
            const idx_t k = m - 1;
            // the low z-face of plane m: the high one of the cell of plane m - 1
            bzn = bz0 - cx * (s_ey[hi][t + 1] - s_ey[hi][t]) + cy * (s_ex[hi][t + CX] - s_ex[hi][t]);
            if (interior && m >= k0 && (m < k1 || (m == nz && g.bc[2] == VLCT_BC_OUTFLOW))) {
                st8(out.b[2] + m * sc, oc, bzn);
                if (g.bc[2] == VLCT_BC_PERIODIC && m == 0) st8(out.b[2] + nz * sc, oc, bzn);
            }
            if (m > k0) {
                double bxl = any_value(), byl = any_value();
                if (jj < ny) {  // face x (ii - 1/2, jj, k)
                    bxl = bxp + cz * (s_ey[hi][t] - s_ey[lo][t]);
                    st8(out.b[0] + k * sbx, ox0, bxl);
                    if (g.bc[0] == VLCT_BC_PERIODIC && ii == 0)
                        st8(out.b[0] + k * sbx, ox0 + 8u * (u32)nx, bxl);
                }
                if (ii < nx) {  // face y (ii, jj - 1/2, k)
                    byl = byp - cz * (s_ex[hi][t] - s_ex[lo][t]);
                    st8(out.b[1] + k * sby, oy0, byl);
                    if (g.bc[1] == VLCT_BC_PERIODIC && jj == 0)
                        st8(out.b[1] + k * sby, oy0 + 8u * (u32)(nx * ny), byl);
                }
                if (interior) {
                    double u[5];
                    u[0] = up[0] - cz * (hzn[0] - hz_lo[0]);
                    u[1] = up[1] - cz * (hzn[2] - hz_lo[2]);
                    u[2] = up[2] - cz * (hzn[3] - hz_lo[3]);
                    u[3] = up[3] - cz * (hzn[1] - hz_lo[1]);
                    u[4] = up[4] - cz * (hzn[4] - hz_lo[4]);
#pragma unroll
                    for (int q = 0; q < 5; ++q) st8(out.u[0] + (q * ostep + k * sc), oc, u[q]);
                    // half-step primitives; the high faces in the arithmetic of the
                    // threads or blocks that own them
                    const double bxu = bxhp + cz * (s_ey[hi][t + 1] - s_ey[lo][t + 1]);
                    const double byu = byhp - cz * (s_ex[hi][t + CX] - s_ex[lo][t + CX]);
                    double w[8];
                    st |= prims_of(g, u, 0.5 * (bxl + bxu), 0.5 * (byl + byu),
                                   0.5 * (bzp + bzn), w);
#pragma unroll
                    for (int q = 0; q < 8; ++q) st8(P.w[0] + (q * pstep + (k + kGhost) * sp), op, w[q]);
                }
            }
            // start plane m
            const double dz0 = s_ez[t + CX] - s_ez[t], dz1 = s_ez[t + CX + 1] - s_ez[t + 1];
            const double dx0 = s_ez[t + 1] - s_ez[t], dx1 = s_ez[t + CX + 1] - s_ez[t + CX];
            bxp = bx0 - cy * dz0;
            bxhp = bx1 - cy * dz1;
            byp = by0 + cx * dx0;
            byhp = by1 + cx * dx1;
        }
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            up[q] = upn[q];
            hz_lo[q] = hzn[q];
        }
        bzp = bzn;
    }
    if (st && status) atomicOr(status, st);
}

// ---------------------------------------------------------------------------
// CFL reduction (Step 1, Eq. dt): per-block maxima of max_l (|v_l| + c_f,l)/d_l,
// then one block reduces the partials and writes dt = cfl / max.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void dt_partial_body(const Geom &g, const StateP &s, double *partial,
                                                uint32_t *status, idx_t b)
{
    __shared__ double red[kBlock / 64];
    const idx_t N = (idx_t)g.n[0] * g.n[1] * g.n[2];
    const idx_t t = b * kBlock + threadIdx.x;
    double m = 0.0;
    if (t < N) {
        const int i = (int)(t % g.n[0]);
        const idx_t r = t / g.n[0];
        const int j = (int)(r % g.n[1]);
        const int k = (int)(r / g.n[1]);
        // high faces through the face map: a periodic duplicate face is not read
        const int ip = map_face(i + 1, g.n[0], g.bc[0]);
        const int jp = map_face(j + 1, g.n[1], g.bc[1]);
        const int kp = map_face(k + 1, g.n[2], g.bc[2]);
        const double b[3] = {
            0.5 * (s.b[0][face_store(g, 0, i, j, k)] + s.b[0][face_store(g, 0, ip, j, k)]),
            0.5 * (s.b[1][face_store(g, 1, i, j, k)] + s.b[1][face_store(g, 1, i, jp, k)]),
            0.5 * (s.b[2][face_store(g, 2, i, j, k)] + s.b[2][face_store(g, 2, i, j, kp)])};
        uint32_t st = 0;
        m = cell_cfl(g, s.u[0][t], s.u[1][t], s.u[2][t], s.u[3][t], s.u[4][t], b, st);
        if (st && status) atomicOr(status, st);
    }
    m = wave_max(m);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) red[wv] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        double red_max = red[0];
        for (int q = 1; q < kBlock / 64; ++q) red_max = fmax(red_max, red[q]);
        partial[b] = red_max;
    }
}

__global__ void __launch_bounds__(1024) k_dt_final(const double *partial, int n, double cfl,
                                                   double *dt_out)
{
    __shared__ double red[1024 / 64];
    double m = 0.0;
    for (int q = threadIdx.x; q < n; q += blockDim.x) m = fmax(m, partial[q]);
    m = wave_max(m);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) red[wv] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        double b = red[0];
        for (int q = 1; q < (int)(blockDim.x / 64); ++q) b = fmax(b, red[q]);
        dt_out[0] = cfl / b;
    }
}

// ---------------------------------------------------------------------------
// single-instance kernels: the logical block comes from the XCD remap
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kBlock) k_prims(Geom g, StateP s, Prims P, uint32_t *status)
{
    prims_body(g, s, P, status, xcd_block(nblk_prims(g)));
}

template <int RECON>
__global__ void __launch_bounds__(kBlock) k_flux_recon_x(Geom g, StateP s, Prims P, Flux F,
                                                          StateP base, StateW out,
                                                          const double *dt_dev, uint32_t *status)
{
    recon_x_body<RECON>(g, s, P, F, base, out, dt_dev, status, xcd_block(nblk_row(g)));
}

template <int D, int RECON>
__global__ void __launch_bounds__(kBlock, Recon<RECON>::kWaves) k_flux_recon_march(Geom g, StateP s, Prims P, Flux F,
                                                              StateW out, const double *dt_dev,
                                                              uint32_t *status)
{
    march_body<D, RECON>(g, s, P, F, out, dt_dev, status, xcd_block(nblk_march(g, D)));
}

template <bool DT>
__global__ void __launch_bounds__(kCtThreads, 4) k_ct_update(Geom g, Prims P, Flux F, StateP base,
                                                             StateW out, const double *dt_dev,
                                                             uint32_t *status, double *partial)
{
    ct_body<DT>(g, P, F, base, out, dt_dev, status, xcd_block(nblk_ct(g)), partial);
}

static_assert(kPredThreads * kPredBlocksPerCU <= 1024,
              "the resident predictor blocks of a CU hold at most two waves per SIMD");

// blocks of the fused predictor: one per (slab, tile)
__host__ __device__ __forceinline__ idx_t nblk_pred(const Geom &g)
{
    return pred_tiles(g) * ((g.n[2] + g.pred_slab - 1) / g.pred_slab);
}

__global__ void __launch_bounds__(kPredThreads, kPredWavesPerSimd) k_pred(Geom g, StateP s, StateW out, Prims P,
                                                        const double *dt_dev, uint32_t *status,
                                                        uint8_t *side0, uint8_t *side1,
                                                        uint8_t *side2)
{
    pred_body(g, s, out, P, dt_dev, status, xcd_block(nblk_pred(g)), side0, side1, side2);
}

__global__ void __launch_bounds__(kBlock) k_prims_ghost(Geom g, StateP s, Prims P,
                                                        uint32_t *status)
{
    prims_ghost_body(g, s, P, status, xcd_block((ghost_cells(g) + kBlock - 1) / kBlock));
}

__global__ void __launch_bounds__(kBlock) k_dt_partial(Geom g, StateP s, double *partial,
                                                       uint32_t *status)
{
    dt_partial_body(g, s, partial, status, blockIdx.x);
}

// ---------------------------------------------------------------------------
// batched step: independent instances (own sizes, gamma, dt, boundaries,
// workspace) advanced by one launch per kernel for all of them.  Each launch
// flattens the logical blocks of every instance; a block finds its instance
// by binary search over the first block of each instance and runs the same
// body as the single-instance kernel, so an instance's result equals its
// single-instance step bit for bit.
// ---------------------------------------------------------------------------
// launches of a batched step
enum Slot { kSlotPred, kSlotGhost, kSlotRow, kSlotMarch1, kSlotMarch2, kSlotCt, kSlotDt, kSlots };

struct Inst {
    Geom g;
    StateP in;       // U^n
    StateW out;      // U^{n+1}
    StateW half;     // U^{n+1/2} (workspace)
    Prims P;         // primitives of the current stage (workspace)
    Flux F;          // face fluxes of the current stage (workspace)
    double *partial; // CFL partials (workspace)
    const double *dt;
    double *next_dt;
    uint32_t *status;
    // per-instance end times (vlct_step_batch_until; NULL otherwise): the
    // instance steps only while *active, by *dt = min(caller dt, t_end - t),
    // and its time *t advances at the end of the step
    const int *active;
    double *t;
    idx_t start[kSlots];  // first flattened block of this instance in each launch
};

__device__ __forceinline__ bool retired(const Inst &I) { return I.active && !I.active[0]; }

constexpr int kPackChunk = 6;  // records per pack launch (4 KiB of kernel arguments)
struct PackArgs {
    Inst rec[kPackChunk];
    Inst *tab;
    int first, n;
};

static_assert(sizeof(PackArgs) <= 4096, "kernel arguments");

// writes instance records into the device table (records travel as kernel
// arguments, so a step needs no host-to-device copy and can be captured)
__global__ void k_pack(PackArgs a)
{
    const int t = threadIdx.x;
    if (t < a.n) a.tab[a.first + t] = a.rec[t];
}

__device__ __forceinline__ const Inst &find_inst(const Inst *tab, int count, int slot, idx_t gb,
                                                 idx_t &lb)
{
    int lo = 0, hi = count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (tab[mid].start[slot] <= gb) lo = mid; else hi = mid - 1;
    }
    lb = gb - tab[lo].start[slot];
    return tab[lo];
}

__device__ __forceinline__ StateP const_view(const StateW &w)
{
    StateP p;
    for (int f = 0; f < 5; ++f) p.u[f] = w.u[f];
    for (int d = 0; d < 3; ++d) p.b[d] = w.b[d];
    return p;
}

// the fused predictor of every instance: U^n -> U^{n+1/2}
__global__ void __launch_bounds__(kPredThreads, kPredWavesPerSimd) kb_pred(const Inst *tab, int count, idx_t total)
{
    const idx_t gb = xcd_block(total);
    if (gb >= total) return;
    idx_t lb;
    const Inst &I = find_inst(tab, count, kSlotPred, gb, lb);
    if (retired(I)) return;
    const Geom g = I.g;
    const StateP in = I.in;
    const StateW half = I.half;
    const Prims P = I.P;
    pred_body(g, in, half, P, I.dt, I.status, lb, nullptr, nullptr, nullptr);
}

// ghost-layer primitives of the half-step state of every instance
__global__ void __launch_bounds__(kBlock) kb_prims_ghost(const Inst *tab, int count, idx_t total)
{
    const idx_t gb = xcd_block(total);
    if (gb >= total) return;
    idx_t lb;
    const Inst &I = find_inst(tab, count, kSlotGhost, gb, lb);
    if (retired(I)) return;
    const Geom g = I.g;
    const StateP st = const_view(I.half);
    const Prims P = I.P;
    prims_ghost_body(g, st, P, I.status, lb);
}

template <int RECON>
__global__ void __launch_bounds__(kBlock) kb_recon_x(const Inst *tab, int count, idx_t total)
{
    const idx_t gb = xcd_block(total);
    if (gb >= total) return;
    idx_t lb;
    const Inst &I = find_inst(tab, count, kSlotRow, gb, lb);
    if (retired(I)) return;
    const Geom g = I.g;
    const Prims P = I.P;
    const Flux F = I.F;
    recon_x_body<RECON>(g, const_view(I.half), P, F, I.in, I.out, I.dt, I.status, lb);
}

template <int D, int RECON>
__global__ void __launch_bounds__(kBlock, Recon<RECON>::kWaves) kb_march(const Inst *tab, int count, idx_t total)
{
    const idx_t gb = xcd_block(total);
    if (gb >= total) return;
    idx_t lb;
    const Inst &I = find_inst(tab, count, D == 1 ? kSlotMarch1 : kSlotMarch2, gb, lb);
    if (retired(I)) return;
    const Geom g = I.g;
    const Prims P = I.P;
    const Flux F = I.F;
    march_body<D, RECON>(g, const_view(I.half), P, F, I.out, I.dt, I.status, lb);
}

// DT: the CFL maxima of the new state ride along, one per block
template <bool DT>
__global__ void __launch_bounds__(kCtThreads, 4) kb_ct(const Inst *tab, int count, idx_t total)
{
    const idx_t gb = xcd_block(total);
    if (gb >= total) return;
    idx_t lb;
    const Inst &I = find_inst(tab, count, kSlotCt, gb, lb);
    if (retired(I)) return;
    const Geom g = I.g;
    const Prims P = I.P;
    const Flux F = I.F;
    ct_body<DT>(g, P, F, I.in, I.out, I.dt, I.status, lb, I.partial);
}

__global__ void __launch_bounds__(kBlock) kb_dt_partial(const Inst *tab, int count, idx_t total)
{
    // no XCD remap: the partial of block lb is written to partial[lb]
    const idx_t gb = blockIdx.x;
    if (gb >= total) return;
    idx_t lb;
    const Inst &I = find_inst(tab, count, kSlotDt, gb, lb);
    if (retired(I)) return;
    const Geom g = I.g;
    dt_partial_body(g, const_view(I.out), I.partial, I.status, lb);
}

// one block per instance: dt = cfl / max over that instance's partials (of the
// CT blocks, or of kb_dt_partial); an instance with an end time also advances
// its time by the step it took
__global__ void __launch_bounds__(1024) kb_dt_final(const Inst *tab, bool ct)
{
    const Inst &I = tab[blockIdx.x];
    if (retired(I)) return;
    const int n = (int)(ct ? nblk_ct(I.g) : nblk_dt(I.g));
    __shared__ double red[1024 / 64];
    double m = 0.0;
    for (int q = threadIdx.x; q < n; q += blockDim.x) m = fmax(m, I.partial[q]);
    m = wave_max(m);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) red[wv] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        double b = red[0];
        for (int q = 1; q < (int)(blockDim.x / 64); ++q) b = fmax(b, red[q]);
        I.next_dt[0] = I.g.cfl / b;
        if (I.t) I.t[0] += I.dt[0];
    }
}

// per-instance end times: instance i is active while t[i] < t_end[i] and then
// steps by min(dt[i], t_end[i] - t[i]) (the caller's clip of the last step)
__global__ void kb_clip(int count, const double *dt, const double *t, const double *t_end,
                        double *dt_eff, int *active)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const bool a = t[i] < t_end[i];
    active[i] = a ? 1 : 0;
    dt_eff[i] = a ? fmin(dt[i], t_end[i] - t[i]) : 0.0;
}

// ---------------------------------------------------------------------------
// host side: validation, workspace carving, launches
// ---------------------------------------------------------------------------




struct Layout {
    size_t half[8], prims, flux[3], partial, ct_partial, total;
    size_t prims_len, flux_len[3], npartial;
};

// partials the layout has always left room for (CT blocks of 64 x 8 columns and
// 4 to 32 planes): kept as the size is, so that workspace and scratch checks
// answer as before
static size_t partial_room(const Geom &g)
{
    const size_t cols = (size_t)((g.n[0] + (g.bc[0] == VLCT_BC_OUTFLOW) + 63) / 64) *
                        ((g.n[1] + (g.bc[1] == VLCT_BC_OUTFLOW) + 7) / 8);
    auto blocks = [&](int p) { return cols * ((g.n[2] + p - 1) / p); };
    int p = 32;
    while (p > 8 && blocks(p) < 1024) p /= 2;
    return blocks(p == 8 && blocks(8) < 256 ? 4 : p);
}

static Layout layout(const Geom &g)
{
    Layout L;
    size_t off = 0;
    for (int f = 0; f < 8; ++f) {
        L.half[f] = off;
        off += align_up(field_len(g.n, f) * sizeof(double));
    }
    L.prims_len = (size_t)g.p[0] * g.p[1] * g.p[2];
    L.prims = off;
    off += 8 * align_up(L.prims_len * sizeof(double));
    for (int d = 0; d < 3; ++d) {
        L.flux_len[d] = (size_t)flux_dim(g.n, d, 0) * flux_dim(g.n, d, 1) * flux_dim(g.n, d, 2);
        L.flux[d] = off;
        off += flux_axis_bytes(L.flux_len[d]);
    }
    const size_t N = (size_t)g.n[0] * g.n[1] * g.n[2];
    L.npartial = (N + kBlock - 1) / kBlock;  // partials of the CFL kernel
    L.partial = off;
    off += align_up(std::max(L.npartial, partial_room(g)) * sizeof(double));
    // one partial per CT block goes to the x axis' spare flux components
    L.ct_partial = L.flux[0] + 2 * align_up(L.flux_len[0] * sizeof(double));
    L.total = off;
    return L;
}


// launch observer of one vlct_step_observed call (diagnostics): set by that
// call on its own host thread for its duration only, so other calls and
// threads never see it
struct ObserverCtx {
    vlct_launch_observer cb;
    void *user;
};
static thread_local const ObserverCtx *t_observer = nullptr;

struct Observe {
    int kernel;
    hipStream_t s;
    Observe(int k, hipStream_t st) : kernel(k), s(st)
    {
        if (t_observer) t_observer->cb(t_observer->user, kernel, 0, static_cast<void *>(s));
    }
    ~Observe()
    {
        if (t_observer) t_observer->cb(t_observer->user, kernel, 1, static_cast<void *>(s));
    }
};

struct Bound {
    Prims P;
    Flux F;
    StateW half;
    double *partial, *ct_partial;  // CFL maxima per block of k_dt_partial, of the CT update
};

static Bound bind(const Layout &L, void *ws)
{
    char *b = static_cast<char *>(ws);
    Bound B;
    for (int f = 0; f < 8; ++f) {
        double *p = reinterpret_cast<double *>(b + L.half[f]);
        if (f < 5) B.half.u[f] = p; else B.half.b[f - 5] = p;
    }
    for (int f = 0; f < 8; ++f)
        B.P.w[f] = reinterpret_cast<double *>(b + L.prims + f * align_up(L.prims_len * sizeof(double)));
    B.F = bind_flux(b, L.flux, L.flux_len);
    B.partial = reinterpret_cast<double *>(b + L.partial);
    B.ct_partial = reinterpret_cast<double *>(b + L.ct_partial);
    return B;
}



int launch_prims(const Geom &g, const StateP &st, const Prims &P, uint32_t *status,
                 hipStream_t s)
{
    Observe o(VLCT_KERNEL_PRIMS, s);
    k_prims<<<xcd_grid(nblk_prims(g)), kBlock, 0, s>>>(g, st, P, status);
    return hipGetLastError() == hipSuccess ? VLCT_OK : VLCT_EHIP;
}

int launch_fluxes(const Geom &g, const StateP &st, const Prims &P, const Flux &F, int recon,
                  const StateP &base, const StateW &out, const double *dt_dev, uint32_t *status,
                  hipStream_t s)
{
    const int kid = recon == VLCT_RECON_PCM ? VLCT_KERNEL_FLUX_PCM : VLCT_KERNEL_FLUX_RECON;
#define VLCT_RECON3(R)                                                                        \
    {                                                                                         \
        { Observe o(kid, s); k_flux_recon_x<R><<<xcd_grid(nblk_row(g)), kBlock, 0, s>>>(g, st, P, F, base, out, dt_dev, status); } \
        { Observe o(kid, s); k_flux_recon_march<1, R><<<xcd_grid(nblk_march(g, 1)), kBlock, 0, s>>>(g, st, P, F, out, dt_dev, status); } \
        { Observe o(kid, s); k_flux_recon_march<2, R><<<xcd_grid(nblk_march(g, 2)), kBlock, 0, s>>>(g, st, P, F, out, dt_dev, status); } \
    }
    switch (recon) {
    case VLCT_RECON_PCM: VLCT_RECON3(VLCT_RECON_PCM) break;
    case VLCT_RECON_PLMC: VLCT_RECON3(VLCT_RECON_PLMC) break;
    case VLCT_RECON_PPMC: VLCT_RECON3(VLCT_RECON_PPMC) break;
    case VLCT_RECON_PLMP: VLCT_RECON3(VLCT_RECON_PLMP) break;
    default: VLCT_RECON3(VLCT_RECON_PPMP) break;
    }
#undef VLCT_RECON3
    return hipGetLastError() == hipSuccess ? VLCT_OK : VLCT_EHIP;
}

// the full step's CT edge fields and faces (Steps 8-9); with `partial` the CFL
// maxima of the new state, one per block
static int launch_ct(const Geom &g, const Prims &P, const Flux &F, const StateP &base,
                     const StateW &out, const double *dt_dev, uint32_t *status, double *partial,
                     hipStream_t s)
{
    Observe o(VLCT_KERNEL_UPDATE_FULL, s);
    if (partial)
        k_ct_update<true><<<xcd_grid(nblk_ct(g)), kCtThreads, 0, s>>>(g, P, F, base, out, dt_dev,
                                                                     status, partial);
    else
        k_ct_update<false><<<xcd_grid(nblk_ct(g)), kCtThreads, 0, s>>>(g, P, F, base, out, dt_dev,
                                                                      status, nullptr);
    return hipGetLastError() == hipSuccess ? VLCT_OK : VLCT_EHIP;
}

// the whole predictor (Steps 2-5) in one kernel: U^n -> U^{n+1/2}; with
// `side` (3 arrays, tape layout) it also records the faces' upwind sides
int launch_pred(const Geom &g, const StateP &st, const StateW &half, const Prims &P,
                const double *dt_dev, uint32_t *status, uint8_t *const *side, hipStream_t s)
{
    {
        Observe o(VLCT_KERNEL_PREDICTOR, s);
        uint8_t *s0 = side ? side[0] : nullptr, *s1 = side ? side[1] : nullptr,
                *s2 = side ? side[2] : nullptr;
        k_pred<<<xcd_grid(nblk_pred(g)), kPredThreads, 0, s>>>(g, st, half, P, dt_dev, status, s0,
                                                               s1, s2);
    }
    // ghost layers of the half-step primitives
    Observe o(VLCT_KERNEL_PRIMS, s);
    k_prims_ghost<<<xcd_grid((ghost_cells(g) + kBlock - 1) / kBlock), kBlock, 0, s>>>(
        g, as_const(half), P, status);
    return hipGetLastError() == hipSuccess ? VLCT_OK : VLCT_EHIP;
}

__global__ void k_pack_sides(Geom g, Flux F, uint8_t *s0, uint8_t *s1, uint8_t *s2)
{
    const idx_t N = (idx_t)g.n[0] * g.n[1] * g.n[2];
    const idx_t t = (idx_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= N) return;
    const int i = (int)(t % g.n[0]), j = (int)((t / g.n[0]) % g.n[1]),
              k = (int)(t / ((idx_t)g.n[0] * g.n[1]));
    s0[t] = side_code(F.sg[0][fidx(g, 0, i, j, k)]);
    s1[t] = side_code(F.sg[1][fidx(g, 1, i, j, k)]);
    s2[t] = side_code(F.sg[2][fidx(g, 2, i, j, k)]);
}

int launch_pack_sides(const Geom &g, const Flux &F, uint8_t *const side[3], hipStream_t s)
{
    const size_t N = (size_t)g.n[0] * g.n[1] * g.n[2];
    k_pack_sides<<<nblocks(N), kBlock, 0, s>>>(g, F, side[0], side[1], side[2]);
    return hipGetLastError() == hipSuccess ? VLCT_OK : VLCT_EHIP;
}

static int launch_dt(const Geom &g, const StateP &st, const Bound &B, const Layout &L,
                     double *dt_out, uint32_t *status, hipStream_t s)
{
    const size_t N = (size_t)g.n[0] * g.n[1] * g.n[2];
    Observe o(VLCT_KERNEL_DT, s);
    k_dt_partial<<<nblocks(N), kBlock, 0, s>>>(g, st, B.partial, status);
    k_dt_final<<<1, 1024, 0, s>>>(B.partial, (int)L.npartial, g.cfl, dt_out);
    return hipGetLastError() == hipSuccess ? VLCT_OK : VLCT_EHIP;
}

// the corrector (Steps 6-9) from the half-step state and its primitives in
// B.P, then the next CFL step: its reduction rides on the CT update unless the
// step is in place (it reads the base field on faces that other threads update)
static int corrector(const Geom &g, int recon, const StateP &half, const Bound &B, const Layout &L,
                     const StateP &base, const StateW &out, bool inplace, const double *dt_dev,
                     double *next_dt, uint32_t *status, uint8_t *const *side, hipStream_t s)
{
    const bool ride = next_dt && !inplace;
    int rc = launch_fluxes(g, half, B.P, B.F, recon, base, out, dt_dev, status, s);
    if (!rc)
        rc = launch_ct(g, B.P, B.F, base, out, dt_dev, status, ride ? B.ct_partial : nullptr, s);
    if (!rc && side) rc = launch_pack_sides(g, B.F, side, s);
    if (rc || !next_dt) return rc;
    if (!ride) return launch_dt(g, as_const(out), B, L, next_dt, status, s);
    Observe o(VLCT_KERNEL_DT_FINAL, s);
    k_dt_final<<<1, 1024, 0, s>>>(B.ct_partial, (int)nblk_ct(g), g.cfl, next_dt);
    return hipGetLastError() == hipSuccess ? VLCT_OK : VLCT_EHIP;
}

constexpr int kMaxBatch = 1 << 16;

// the instance table, then the clipped dt and active flag of every instance
// (used by vlct_step_batch_until)
static size_t batch_table_bytes(int count)
{
    return align_up((size_t)count * sizeof(Inst)) + align_up((size_t)count * sizeof(double)) +
           align_up((size_t)count * sizeof(int));
}
static double *batch_dt_eff(void *ws, int count)
{
    return reinterpret_cast<double *>(static_cast<char *>(ws) +
                                      align_up((size_t)count * sizeof(Inst)));
}
static int *batch_active(void *ws, int count)
{
    return reinterpret_cast<int *>(reinterpret_cast<char *>(batch_dt_eff(ws, count)) +
                                   align_up((size_t)count * sizeof(double)));
}

// an instance's tiles as its plan byte asks
static void plan_tiles(Geom &g, uint8_t plan)
{
    const int cv = plan & 15, mv = plan >> 4;
    if (cv > 0) {
        g.ct_tx = cv == 1 ? 30 : 14;
        g.ct_ty = kCtThreads / (g.ct_tx + 2) - 2;
    }
    const int m = mv == 1 ? 32 : 8;
    if (mv > 0 && march_fits(g, m)) g.march[1] = g.march[2] = m;
}

// an instance's share, by cells, of the blocks that run at a time: one
// predictor block per CU and two of the other kernels, more where the batch
// gives each of them more than 16 planes of a tile (against a whole chip each:
// 64 runs of 16..96 cells a side 3.83 -> 3.45 ms; 12 of 16..40 260 -> 165 us,
// 6 of 12..90, third order, 295)
static Slots batch_slots(const vlct_grid *vg, double cells)
{
    const double share = kNumCUs * ((double)vg->nx * vg->ny * vg->nz / cells);
    const double rounds = std::max(1.0, cells / (kNumCUs * 16.0 * kPredTx * kPredTy));
    auto part = [&](double f) { return std::max(1, (int)(share * f)); };
    return Slots{part(2.0), part(rounds), part(std::max(2.0, rounds))};
}

// instance records with workspace regions and flattened block offsets;
// returns the per-slot block totals through `total`
static void batch_records(int count, const vlct_grid *grids, const vlct_state *in,
                          const vlct_state *out, const double *dt_dev, double *next_dt_dev,
                          uint32_t *status_dev, const uint8_t *plan, void *ws, bool ride,
                          std::vector<Inst> &rec, idx_t total[kSlots])
{
    rec.resize(count);
    size_t off = batch_table_bytes(count);
    for (int s = 0; s < kSlots; ++s) total[s] = 0;
    double cells = 0.0;
    for (int i = 0; i < count; ++i) cells += (double)grids[i].nx * grids[i].ny * grids[i].nz;
    std::unordered_map<uint64_t, Geom> chosen;
    for (int i = 0; i < count; ++i) {
        Geom g = grid_geom(&grids[i]);
        // instances of the same size and boundaries share one choice
        uint64_t key = 0;
        for (int d = 0; d < 3; ++d) key = key << 14 | (uint64_t)g.n[d] << 1 | (uint64_t)g.bc[d];
        const auto [it, first] = chosen.try_emplace(key, g);
        if (first) choose_tiles(it->second, batch_slots(&grids[i], cells));
        copy_tiles(g, it->second);
        const Layout L = layout(g);
        plan_tiles(g, plan ? plan[i] : 0);
        const Bound B = bind(L, static_cast<char *>(ws) + off);
        off += L.total;
        Inst &r = rec[i];
        r.g = g;
        r.in = as_const(&in[i]);
        r.out = as_mut(&out[i]);
        r.half = B.half;
        r.P = B.P;
        r.F = B.F;
        r.partial = ride ? B.ct_partial : B.partial;
        r.dt = dt_dev + i;
        r.next_dt = next_dt_dev ? next_dt_dev + i : nullptr;
        r.status = status_dev ? status_dev + i : nullptr;
        r.active = nullptr;
        r.t = nullptr;
        idx_t nb[kSlots] = {};
        nb[kSlotPred] = nblk_pred(g);
        nb[kSlotGhost] = (ghost_cells(g) + kBlock - 1) / kBlock;
        nb[kSlotRow] = nblk_row(g);
        nb[kSlotMarch1] = nblk_march(g, 1);
        nb[kSlotMarch2] = nblk_march(g, 2);
        nb[kSlotCt] = nblk_ct(g);
        nb[kSlotDt] = nblk_dt(g);
        for (int s = 0; s < kSlots; ++s) {
            r.start[s] = total[s];
            total[s] += nb[s];
        }
    }
}

// every output array belongs to one instance, and an input array is shared
// only with the same field of its own instance's output (in-place)
static bool batch_aliasing_ok(int count, const vlct_state *in, const vlct_state *out)
{
    std::unordered_map<const void *, long> owner;  // pointer -> instance * 8 + field
    auto fields = [](const vlct_state &st, int f) -> const void * {
        const double *p[8] = {st.rho, st.mx, st.my, st.mz, st.E, st.bx, st.by, st.bz};
        return p[f];
    };
    for (int i = 0; i < count; ++i)
        for (int f = 0; f < 8; ++f)
            if (!owner.emplace(fields(out[i], f), (long)i * 8 + f).second) return false;
    for (int i = 0; i < count; ++i)
        for (int f = 0; f < 8; ++f) {
            auto it = owner.find(fields(in[i], f));
            if (it != owner.end() && it->second != (long)i * 8 + f) return false;
        }
    // an instance is either fully in place or fully out of place
    for (int i = 0; i < count; ++i) {
        int same = 0;
        for (int f = 0; f < 8; ++f) same += fields(in[i], f) == fields(out[i], f);
        if (same != 0 && same != 8) return false;
    }
    return true;
}

// ---------------------------------------------------------------------------
// static scratch of vlct_step_noalloc: the workspace of vlct_step in a
// file-scope device array, so a caller that cannot allocate device memory can
// still step a grid whose workspace fits.  Each device holds its own copy; its
// address comes from hipGetSymbolAddress once per device (the array's name in
// host code is a host-side stand-in, never a device address).  Nothing in the
// step's workspace has to start at zero: every kernel writes what a later one
// reads within the same call.
// ---------------------------------------------------------------------------
constexpr size_t kScratchBytes = VLCT_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
constexpr int kScratchDevices = 64;
static std::atomic<void *> g_scratch_addr[kScratchDevices];
static std::mutex g_scratch_mutex;

// device address of the current device's scratch array
static int scratch_address(void **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kScratchDevices) return VLCT_EHIP;
    void *p = g_scratch_addr[dev].load(std::memory_order_acquire);
    if (!p) {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        p = g_scratch_addr[dev].load(std::memory_order_relaxed);
        if (!p) {
            if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return VLCT_EHIP;
            g_scratch_addr[dev].store(p, std::memory_order_release);
        }
    }
    *out = p;
    return VLCT_OK;
}

// `out` must be `in` itself (all eight arrays the same) or use memory that no
// input array overlaps, and no two output arrays may overlap: compared as
// address ranges [p, p + bytes) of the grid's field sizes
static bool in_out_ok(const vlct_grid *vg, const vlct_state *in, const vlct_state *out,
                      bool &all_same)
{
    const int n[3] = {vg->nx, vg->ny, vg->nz};
    const double *pi[8] = {in->rho, in->mx, in->my, in->mz, in->E, in->bx, in->by, in->bz};
    const double *po[8] = {out->rho, out->mx, out->my, out->mz, out->E, out->bx, out->by, out->bz};
    auto overlap = [&](const double *a, int fa, const double *b, int fb) {
        const uintptr_t a0 = reinterpret_cast<uintptr_t>(a), b0 = reinterpret_cast<uintptr_t>(b);
        const uintptr_t a1 = a0 + field_len(n, fa) * sizeof(double);
        const uintptr_t b1 = b0 + field_len(n, fb) * sizeof(double);
        return a0 < b1 && b0 < a1;
    };
    all_same = true;
    for (int f = 0; f < 8; ++f) all_same &= pi[f] == po[f];
    for (int f = 0; f < 8; ++f)
        for (int h = f + 1; h < 8; ++h)
            if (overlap(po[f], f, po[h], h)) return false;
    if (all_same) return true;
    for (int f = 0; f < 8; ++f)
        for (int h = 0; h < 8; ++h)
            if (overlap(po[f], f, pi[h], h)) return false;
    return true;
}

}  // namespace vlct

using namespace vlct;

extern "C" {

size_t vlct_workspace_bytes(const vlct_grid *g)
{
    if (!grid_ok(g)) return 0;
    return layout(grid_geom(g)).total;
}

int vlct_cfl_dt(const vlct_grid *vg, const vlct_state *s, double *dt_dev, void *ws,
                size_t ws_bytes, void *stream)
{
    if (!grid_ok(vg) || !state_ok(s) || !dt_dev) return VLCT_EINVAL;
    const Geom g = grid_geom(vg);
    const Layout L = layout(g);
    if (!ws || ws_bytes < L.total) return VLCT_EWORKSPACE;
    const Bound B = bind(L, ws);
    return launch_dt(g, as_const(s), B, L, dt_dev, nullptr, static_cast<hipStream_t>(stream));
}

int vlct_step(const vlct_grid *vg, const vlct_state *in, const vlct_state *out,
              const double *dt_dev, double *next_dt_dev, uint32_t *status_dev, void *ws,
              size_t ws_bytes, void *stream)
{
    if (!grid_ok(vg) || !state_ok(in) || !state_ok(out) || !dt_dev) return VLCT_EINVAL;
    bool all_same = false;
    if (!in_out_ok(vg, in, out, all_same)) return VLCT_EINVAL;
    const Geom g = make_geom(vg);
    const Layout L = layout(g);
    if (!ws || ws_bytes < L.total) return VLCT_EWORKSPACE;
    const Bound B = bind(L, ws);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const StateP sin = as_const(in);
    // predictor (Steps 2-5), corrector (Steps 6-9)
    const int rc = launch_pred(g, sin, B.half, B.P, dt_dev, status_dev, nullptr, s);
    if (rc) return rc;
    return corrector(g, vg->recon, as_const(B.half), B, L, sin, as_mut(out), all_same, dt_dev,
                     next_dt_dev, status_dev, nullptr, s);
}

int vlct_step_noalloc(const vlct_grid *vg, const vlct_state *in, const vlct_state *out,
                      const double *dt_dev, double *next_dt_dev, uint32_t *status_dev,
                      void *stream)
{
    if (!grid_ok(vg) || !state_ok(in) || !state_ok(out) || !dt_dev) return VLCT_EINVAL;
    if (layout(grid_geom(vg)).total > kScratchBytes) return VLCT_ESCRATCH;
    void *ws = nullptr;
    const int rc = scratch_address(&ws);
    if (rc) return rc;
    return vlct_step(vg, in, out, dt_dev, next_dt_dev, status_dev, ws, kScratchBytes, stream);
}

size_t vlct_tape_bytes(const vlct_grid *g)
{
    if (!grid_ok(g)) return 0;
    const int n[3] = {g->nx, g->ny, g->nz};
    return tape_layout(n).total;
}

int vlct_step_taped(const vlct_grid *vg, const vlct_state *in, const vlct_state *out,
                    const double *dt_dev, double *next_dt_dev, uint32_t *status_dev, void *ws,
                    size_t ws_bytes, void *tape, size_t tape_bytes, void *stream)
{
    if (!grid_ok(vg) || !state_ok(in) || !state_ok(out) || !dt_dev) return VLCT_EINVAL;
    bool all_same = false;
    if (!in_out_ok(vg, in, out, all_same)) return VLCT_EINVAL;
    const Geom g = make_geom(vg);
    const Layout L = layout(g);
    const TapeLayout T = tape_layout(g.n);
    if (!ws || ws_bytes < L.total || !tape || tape_bytes < T.total) return VLCT_EWORKSPACE;
    const Bound B = bind(L, ws);
    char *tb = static_cast<char *>(tape);
    StateW half;
    for (int f = 0; f < 8; ++f) {
        double *a = reinterpret_cast<double *>(tb + T.half[f]);
        if (f < 5) half.u[f] = a; else half.b[f - 5] = a;
    }
    uint8_t *side[2][3];
    for (int h = 0; h < 2; ++h)
        for (int d = 0; d < 3; ++d) side[h][d] = reinterpret_cast<uint8_t *>(tb + T.side[h][d]);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const StateP sin = as_const(in);
    // the steps of vlct_step with the half-step state and both stages' upwind
    // sides kept in the tape
    const int rc = launch_pred(g, sin, half, B.P, dt_dev, status_dev, side[0], s);
    if (rc) return rc;
    return corrector(g, vg->recon, as_const(half), B, L, sin, as_mut(out), all_same, dt_dev,
                     next_dt_dev, status_dev, side[1], s);
}

const char *vlct_strerror(int code)
{
    switch (code) {
    case VLCT_OK: return "ok";
    case VLCT_EINVAL: return "invalid argument (grid descriptor, state pointers or dt)";
    case VLCT_EWORKSPACE: return "workspace missing or smaller than vlct_workspace_bytes()";
    case VLCT_EHIP: return "HIP launch or runtime error";
    case VLCT_EUNSUPPORTED: return "unsupported option";
    case VLCT_ESCRATCH:
        return "grid needs more workspace than the static scratch of vlct_step_noalloc "
               "(VLCT_NOALLOC_SCRATCH_BYTES)";
    default: return "unknown error code";
    }
}

int vlct_abi_version(void) { return VLCT_ABI_VERSION; }

int vlct_step_observed(const vlct_grid *g, const vlct_state *in, const vlct_state *out,
                       const double *dt_dev, double *next_dt_dev, uint32_t *status_dev, void *ws,
                       size_t ws_bytes, void *stream, vlct_launch_observer cb, void *user)
{
    if (!cb) return VLCT_EINVAL;
    const ObserverCtx ctx{cb, user};
    struct Scope {
        explicit Scope(const ObserverCtx *c) { t_observer = c; }
        ~Scope() { t_observer = nullptr; }
    } scope(&ctx);
    return vlct_step(g, in, out, dt_dev, next_dt_dev, status_dev, ws, ws_bytes, stream);
}

size_t vlct_batch_workspace_bytes(const vlct_grid *grids, int count)
{
    if (!grids || count < 1 || count > kMaxBatch) return 0;
    size_t tot = batch_table_bytes(count);
    for (int i = 0; i < count; ++i) {
        if (!grid_ok(&grids[i])) return 0;
        tot += layout(grid_geom(&grids[i])).total;
    }
    return tot;
}

int vlct_step_batch(int count, const vlct_grid *grids, const vlct_state *in,
                    const vlct_state *out, const double *dt_dev, double *next_dt_dev,
                    uint32_t *status_dev, void *ws, size_t ws_bytes, void *stream)
{
    return vlct_step_batch_plan(count, grids, in, out, dt_dev, next_dt_dev, status_dev, nullptr,
                                ws, ws_bytes, stream);
}

static int batch_args(int count, const vlct_grid *grids, const vlct_state *in,
                      const vlct_state *out, const double *dt_dev, const uint8_t *plan)
{
    if (count < 1 || count > kMaxBatch || !grids || !in || !out || !dt_dev) return VLCT_EINVAL;
    for (int i = 0; i < count; ++i)
        if (!grid_ok(&grids[i]) || !state_ok(&in[i]) || !state_ok(&out[i])) return VLCT_EINVAL;
    if (plan)
        for (int i = 0; i < count; ++i)
            if ((plan[i] & 15) >= kCtVariants || (plan[i] >> 4) >= kMarchVariants) return VLCT_EINVAL;
    for (int i = 1; i < count; ++i)
        if (grids[i].recon != grids[0].recon) return VLCT_EUNSUPPORTED;
    if (!batch_aliasing_ok(count, in, out)) return VLCT_EINVAL;
    return VLCT_OK;
}

// the batched step; with t_dev / t_end_dev (device, count each) every
// instance runs only while t < t_end, by min(dt, t_end - t), and advances t
static int batch_step(int count, const vlct_grid *grids, const vlct_state *in,
                      const vlct_state *out, const double *dt_dev, double *next_dt_dev,
                      uint32_t *status_dev, const uint8_t *plan, void *ws, size_t ws_bytes,
                      void *stream, double *t_dev, const double *t_end_dev)
{
    const int arc = batch_args(count, grids, in, out, dt_dev, plan);
    if (arc) return arc;
    const size_t need = vlct_batch_workspace_bytes(grids, count);
    if (!ws || ws_bytes < need) return VLCT_EWORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    std::vector<Inst> rec;
    idx_t tot[kSlots];
    // the CFL reduction rides on the CT update unless an instance steps in
    // place (it reads the base field on faces that other threads update)
    bool inplace = false;
    for (int i = 0; i < count; ++i) inplace |= in[i].rho == out[i].rho;
    const bool ride = next_dt_dev && !inplace;
    batch_records(count, grids, in, out, dt_dev, next_dt_dev, status_dev, plan, ws, ride, rec, tot);
    if (t_dev) {
        double *dt_eff = batch_dt_eff(ws, count);
        int *active = batch_active(ws, count);
        kb_clip<<<(count + 255) / 256, 256, 0, s>>>(count, dt_dev, t_dev, t_end_dev, dt_eff,
                                                    active);
        for (int i = 0; i < count; ++i) {
            rec[i].dt = dt_eff + i;
            rec[i].active = active + i;
            rec[i].t = t_dev + i;
        }
    }
    Inst *tab = static_cast<Inst *>(ws);
    for (int first = 0; first < count; first += kPackChunk) {
        PackArgs a;
        a.tab = tab;
        a.first = first;
        a.n = std::min(kPackChunk, count - first);
        for (int q = 0; q < a.n; ++q) a.rec[q] = rec[first + q];
        k_pack<<<1, 64, 0, s>>>(a);
    }
    const int recon = grids[0].recon;
    // predictor (Steps 2-5)
    {
        Observe o(VLCT_KERNEL_PREDICTOR, s);
        kb_pred<<<xcd_grid(tot[kSlotPred]), kPredThreads, 0, s>>>(tab, count, tot[kSlotPred]);
    }
    {
        Observe o(VLCT_KERNEL_PRIMS, s);
        kb_prims_ghost<<<xcd_grid(tot[kSlotGhost]), kBlock, 0, s>>>(tab, count, tot[kSlotGhost]);
    }
    // corrector (Steps 6-9); the predictor wrote the interior primitives
    const int kid = recon == VLCT_RECON_PCM ? VLCT_KERNEL_FLUX_PCM : VLCT_KERNEL_FLUX_RECON;
#define VLCT_BRECON(R)                                                                        \
    {                                                                                         \
        { Observe o(kid, s);                                                                  \
          kb_recon_x<R><<<xcd_grid(tot[kSlotRow]), kBlock, 0, s>>>(tab, count, tot[kSlotRow]); } \
        { Observe o(kid, s);                                                                  \
          kb_march<1, R><<<xcd_grid(tot[kSlotMarch1]), kBlock, 0, s>>>(tab, count, tot[kSlotMarch1]); } \
        { Observe o(kid, s);                                                                  \
          kb_march<2, R><<<xcd_grid(tot[kSlotMarch2]), kBlock, 0, s>>>(tab, count, tot[kSlotMarch2]); } \
    }
    switch (recon) {
    case VLCT_RECON_PCM: VLCT_BRECON(VLCT_RECON_PCM) break;
    case VLCT_RECON_PLMC: VLCT_BRECON(VLCT_RECON_PLMC) break;
    case VLCT_RECON_PPMC: VLCT_BRECON(VLCT_RECON_PPMC) break;
    case VLCT_RECON_PLMP: VLCT_BRECON(VLCT_RECON_PLMP) break;
    default: VLCT_BRECON(VLCT_RECON_PPMP) break;
    }
#undef VLCT_BRECON
    {
        Observe o(VLCT_KERNEL_UPDATE_FULL, s);
        if (ride)
            kb_ct<true><<<xcd_grid(tot[kSlotCt]), kCtThreads, 0, s>>>(tab, count, tot[kSlotCt]);
        else
            kb_ct<false><<<xcd_grid(tot[kSlotCt]), kCtThreads, 0, s>>>(tab, count, tot[kSlotCt]);
    }
    if (next_dt_dev) {
        Observe o(VLCT_KERNEL_DT, s);
        if (!ride)
            kb_dt_partial<<<(unsigned)tot[kSlotDt], kBlock, 0, s>>>(tab, count, tot[kSlotDt]);
        kb_dt_final<<<count, 1024, 0, s>>>(tab, ride);
    }
    return hipGetLastError() == hipSuccess ? VLCT_OK : VLCT_EHIP;
}

int vlct_step_batch_plan(int count, const vlct_grid *grids, const vlct_state *in,
                         const vlct_state *out, const double *dt_dev, double *next_dt_dev,
                         uint32_t *status_dev, const uint8_t *plan, void *ws, size_t ws_bytes,
                         void *stream)
{
    return batch_step(count, grids, in, out, dt_dev, next_dt_dev, status_dev, plan, ws, ws_bytes,
                      stream, nullptr, nullptr);
}

int vlct_step_batch_until(int count, const vlct_grid *grids, const vlct_state *states,
                          const double *dt_dev, double *next_dt_dev, uint32_t *status_dev,
                          double *t_dev, const double *t_end_dev, const uint8_t *plan, void *ws,
                          size_t ws_bytes, void *stream)
{
    if (!t_dev || !t_end_dev || !next_dt_dev) return VLCT_EINVAL;
    return batch_step(count, grids, states, states, dt_dev, next_dt_dev, status_dev, plan, ws,
                      ws_bytes, stream, t_dev, t_end_dev);
}

int vlct_batch_tune(int count, const vlct_grid *grids, const vlct_state *in,
                    const vlct_state *out, const double *dt_dev, void *ws, size_t ws_bytes,
                    void *stream, int reps, uint8_t *plan)
{
    const int arc = batch_args(count, grids, in, out, dt_dev, nullptr);
    if (arc) return arc;
    if (!plan || reps < 1 || reps > 100) return VLCT_EINVAL;
    // the trial steps write `out` and leave `in` unchanged
    for (int i = 0; i < count; ++i)
        if (in[i].rho == out[i].rho) return VLCT_EINVAL;
    if (!ws || ws_bytes < vlct_batch_workspace_bytes(grids, count)) return VLCT_EWORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return VLCT_EHIP;
    if (hipEventCreate(&e1) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return VLCT_EHIP;
    }
    // mean time of one batched step under plan p (one untimed step first)
    auto time_plan = [&](const std::vector<uint8_t> &p, float &ms) -> int {
        int rc = vlct_step_batch_plan(count, grids, in, out, dt_dev, nullptr, nullptr, p.data(),
                                      ws, ws_bytes, stream);
        if (rc) return rc;
        if (hipEventRecord(e0, s) != hipSuccess) return VLCT_EHIP;
        for (int r = 0; r < reps && !rc; ++r)
            rc = vlct_step_batch_plan(count, grids, in, out, dt_dev, nullptr, nullptr, p.data(),
                                      ws, ws_bytes, stream);
        if (rc) return rc;
        if (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
            hipEventElapsedTime(&ms, e0, e1) != hipSuccess)
            return VLCT_EHIP;
        ms /= (float)reps;
        return VLCT_OK;
    };
    std::vector<int> nx(count);
    for (int i = 0; i < count; ++i) nx[i] = grids[i].nx;
    std::vector<uint8_t> best;
    const int rc = tune_plan(nx, kCtVariants, kMarchVariants, time_plan, best);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc) return rc;
    std::copy(best.begin(), best.end(), plan);
    return VLCT_OK;
}

const char *vlct_kernel_name(int kernel)
{
    static const char *names[VLCT_KERNEL_COUNT] = {"prims",       "flux_pcm_hlld",
                                                   "flux_recon_hlld", "edges",
                                                   "update_half", "update_full",
                                                   "dt",          "dt_final",
                                                   "predictor"};
    return kernel >= 0 && kernel < VLCT_KERNEL_COUNT ? names[kernel] : "?";
}

}  // extern "C"
