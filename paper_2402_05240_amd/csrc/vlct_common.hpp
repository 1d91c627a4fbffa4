// vlct_common.hpp -- definitions shared by the step kernels (vlct.hip) and
// the adjoint kernels (vlct_adjoint.hip): launch geometry, index maps of the
// state and workspace arrays, state views and argument checks.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <cstring>

#include "../../include/vlct.h"

namespace vlct {

constexpr int kGhost = 3;          // ghost layers of the primitive workspace
constexpr int kBlock = 256;        // threads per block (4 wave64s)
constexpr int kMaxN = 4096;

using idx_t = long long;

// MI355X dispatches consecutive workgroups round-robin to its 8 XCDs, each with
// its own L2.  Kernels launched on xcd_grid(n) blocks read their logical block
// from xcd_block(n): hardware block b works on logical block
// (b mod 8) * ceil(n/8) + b / 8, so every XCD sweeps one contiguous slab of
// the domain and neighbouring rows and planes meet in the same L2.
constexpr int kXcd = 8;
__host__ __device__ __forceinline__ idx_t xcd_per(idx_t n) { return (n + kXcd - 1) / kXcd; }
__device__ __forceinline__ idx_t xcd_block(idx_t n)
{
    const idx_t b = blockIdx.x;
    return (b % kXcd) * xcd_per(n) + b / kXcd;
}

// Addressing.  A block touches a small box of each array, so its kernels form
// the box's origin once as a block-uniform 64-bit base (scalar registers) and
// address elements by 32-bit byte offsets from it: the load and store
// instructions take a scalar base plus a 32-bit vector offset, so an element
// costs one 32-bit add at most instead of a 64-bit index product and sum.
// Offsets stay below 4 GiB: the largest box is a z march's, its cells and six
// more padded planes of at most 4102^2 doubles; 16 cells always fit (3.0 GB),
// longer marches where march_fits says so.
// Accesses go through the global address space explicitly: pointers that a
// batched kernel reads from its instance table would otherwise be generic and
// take flat instructions, which have no scalar base.
using u32 = uint32_t;
#define VLCT_GLOBAL __attribute__((address_space(1)))
__device__ __forceinline__ double ld8(const double *base, u32 byte)
{
    const auto *p = (const VLCT_GLOBAL char *)(base) + byte;
    return *(const VLCT_GLOBAL double *)p;
}
__device__ __forceinline__ void st8(double *base, u32 byte, double v)
{
    auto *p = (VLCT_GLOBAL char *)(base) + byte;
    *(VLCT_GLOBAL double *)p = v;
}
__device__ __forceinline__ int ld1(const int8_t *base, u32 byte)
{
    return *((const VLCT_GLOBAL int8_t *)(base) + byte);
}
__device__ __forceinline__ void st1(int8_t *base, u32 byte, int8_t v)
{
    *((VLCT_GLOBAL int8_t *)(base) + byte) = v;
}
// a block-uniform value in scalar registers (one computed on the vector unit
// would hold vector registers for the whole kernel)
__device__ __forceinline__ double uniform(double x)
{
    const int lo = __builtin_amdgcn_readfirstlane(__double2loint(x));
    const int hi = __builtin_amdgcn_readfirstlane(__double2hiint(x));
    return __hiloint2double(hi, lo);
}
// Marks a thread's byte offset as changed (it is not): inside a loop over
// planes the compiler would otherwise hoist base + offset of every array as
// 64-bit vector pointers, which took 40 registers in the CT update and as many
// in the predictor, and would lose the scalar-base form of the accesses.
__device__ __forceinline__ void pin(u32 &o) { asm("" : "+v"(o)); }
// e / n for the position e of a thread past its block's first row of length n:
// rows longer than a block take no division
__device__ __forceinline__ u32 row_div(u32 e, u32 n) { return e < n ? 0u : (e - n < n ? 1u : e / n); }

// ---------------------------------------------------------------------------
// geometry shared by every kernel
// ---------------------------------------------------------------------------
struct Geom {
    int n[3];
    int bc[3];
    double dl[3], idl[3];  // cell widths and their reciprocals
    double gamma, gm1i, cfl;
    int p[3];  // padded primitive dims n + 2G
    int march[3];     // cells per segment of the corrector's marches along y and z ([1], [2])
    int pr_tx, pr_ty; // column tile of a predictor block
    int ct_tx, ct_ty; // column tile of a CT block
    int ct_planes;    // z planes a CT block marches through
    int pred_slab;    // z planes a predictor block marches through
};

__host__ __device__ __forceinline__ int map_cell(int i, int n, int bc)
{
    if (bc == VLCT_BC_PERIODIC) {
        // one period either side without an integer division
        if (i >= 0 && i < n) return i;
        if (i < 0 && i >= -n) return i + n;
        if (i >= n && i < 2 * n) return i - n;
        const int m = i % n;
        return m < 0 ? m + n : m;
    }
    return i < 0 ? 0 : (i >= n ? n - 1 : i);
}
// normal-face index: periodic faces wrap into [0, n-1], outflow clamps into [0, n]
__host__ __device__ __forceinline__ int map_face(int i, int n, int bc)
{
    if (bc == VLCT_BC_PERIODIC) return map_cell(i, n, bc);
    return i < 0 ? 0 : (i > n ? n : i);
}

// stored face arrays of the state: axis d has n_d + 1 faces along d
__device__ __forceinline__ idx_t face_store(const Geom &g, int d, int i, int j, int k)
{
    const idx_t nx = g.n[0] + (d == 0), ny = g.n[1] + (d == 1);
    return ((idx_t)k * ny + j) * nx + i;
}

__device__ __forceinline__ idx_t cell_store(const Geom &g, int i, int j, int k)
{
    return ((idx_t)k * g.n[1] + j) * g.n[0] + i;
}

// padded primitive index, i,j,k in [-G, n+G-1]
__device__ __forceinline__ idx_t pidx(const Geom &g, int i, int j, int k)
{
    return ((idx_t)(k + kGhost) * g.p[1] + (j + kGhost)) * g.p[0] + (i + kGhost);
}

// flux arrays of axis d: normal index in [0, n_d], transverse in [-1, n_e]
__host__ __device__ __forceinline__ idx_t flux_dim(const int n[3], int d, int e)
{
    return n[e] + (e == d ? 1 : 2);
}
__device__ __forceinline__ idx_t fidx(const Geom &g, int d, int i, int j, int k)
{
    const idx_t X = flux_dim(g.n, d, 0), Y = flux_dim(g.n, d, 1);
    return ((idx_t)(k + (d != 2)) * Y + (j + (d != 1))) * X + (i + (d != 0));
}

struct StateP {
    const double *u[5];
    const double *b[3];
};
struct StateW {
    double *u[5];
    double *b[3];
};
struct Prims {
    double *w[8];  // rho, vx, vy, vz, P, Bcx, Bcy, Bcz on padded cells
};
inline size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

// what the CT update needs of the corrector's face fluxes (the hydro parts go
// straight into the cells): the two EMFs of a face of axis d, -F[B_t1] (along
// t2) and F[B_t2] (along t1), and its CT upwind indicator (+1, -1, 0), the
// sign of S_M
struct Flux {
    double *e[3][2];
    int8_t *sg[3];
};

// bytes of one axis' share of the workspace: seven doubles and a byte per face.
// The EMFs take two of the seven; the size stays, so that every workspace and
// scratch check answers as it always has.
inline size_t flux_axis_bytes(size_t len)
{
    return 7 * align_up(len * sizeof(double)) + align_up(len);
}

inline Flux bind_flux(char *base, const size_t off[3], const size_t len[3])
{
    Flux F;
    for (int d = 0; d < 3; ++d) {
        for (int c = 0; c < 2; ++c)
            F.e[d][c] = reinterpret_cast<double *>(base + off[d] + c * align_up(len[d] * sizeof(double)));
        F.sg[d] = reinterpret_cast<int8_t *>(base + off[d] + 7 * align_up(len[d] * sizeof(double)));
    }
    return F;
}

// ---------------------------------------------------------------------------
// host helpers
// ---------------------------------------------------------------------------
inline bool grid_ok(const vlct_grid *g)
{
    if (!g) return false;
    const int n[3] = {g->nx, g->ny, g->nz};
    for (int d = 0; d < 3; ++d) {
        if (n[d] < 1 || n[d] > kMaxN) return false;
        if (g->bc[d] != VLCT_BC_PERIODIC && g->bc[d] != VLCT_BC_OUTFLOW) return false;
    }
    if (!(g->dx > 0.0) || !(g->dy > 0.0) || !(g->dz > 0.0)) return false;
    if (!(g->gamma > 1.0) || !(g->cfl > 0.0 && g->cfl <= 0.5)) return false;
    if (g->recon < VLCT_RECON_PCM || g->recon > VLCT_RECON_PPMP) return false;
    return true;
}

// Tile override for tests and tuning: the environment variable VLCT_TILES,
// read at every call, holds comma-separated key=value pairs (ct=N and pred=N or
// predslab=N planes per CT and predictor block, cttile=NX and predtile=NX columns
// along x of their tiles, march=N cells per corrector march segment, 1 to 32,
// admarch=N cells per adjoint march segment, 1 to 64) that replace the
// size-dependent choices.  Every choice computes the
// same per-cell and per-face arithmetic; the forward results are bitwise the
// same, the adjoint's equal to the summation order of its accumulations.
// Returns the value of `key` in that string, 0 when it is not set.
inline int tile_override(const char *env, const char *key)
{
    const size_t kl = std::strlen(key);
    for (const char *p = env; *p;) {
        if (std::strncmp(p, key, kl) == 0 && p[kl] == '=') return std::atoi(p + kl + 1);
        const char *c = std::strchr(p, ',');
        if (!c) break;
        p = c + 1;
    }
    return 0;
}

// blocks of the predictor and of the CT update: up to 512 threads, one per
// column of the tile and of its one-cell ring (32 x 13 columns: 34 x 15 = 510
// threads).  The predictor has one block per CU (133 KB of LDS, 256 VGPRs: two
// waves per SIMD), the CT update two.
constexpr int kPredTx = 32, kPredTy = 13, kTileThreads = 512;
constexpr int kPredBlocksPerCU = 1;
constexpr int kPredWavesPerSimd = 2;
constexpr int kNumCUs = 256;  // gfx950 (MI355X)

__host__ __device__ __forceinline__ long long pred_tiles(const Geom &g)
{
    const int ntx = (g.n[0] + (g.bc[0] == VLCT_BC_OUTFLOW) + g.pr_tx - 1) / g.pr_tx;
    const int nty = (g.n[1] + (g.bc[1] == VLCT_BC_OUTFLOW) + g.pr_ty - 1) / g.pr_ty;
    return (long long)ntx * nty;
}

__host__ __device__ __forceinline__ long long ct_tiles(const Geom &g)
{
    const int ntx = (g.n[0] + (g.bc[0] == VLCT_BC_OUTFLOW) + g.ct_tx - 1) / g.ct_tx;
    const int nty = (g.n[1] + (g.bc[1] == VLCT_BC_OUTFLOW) + g.ct_ty - 1) / g.ct_ty;
    return (long long)ntx * nty;
}

// Column tile and planes per block for a kernel that marches tiles along z:
// minimises the time of the launch, taken as rounds of one block per CU times
// (planes + 2) (a run of planes also evaluates the plane beyond each end) times
// `unit` of a round, over the tiles of at most kTileThreads columns (and of half
// of them: one wave per SIMD, a shorter plane but more blocks) and the planes
// that fill 1 to 6 rounds.  The 32-column tile stays unless another is 3% better.
// Tile counts along x go up by an eighth (4096 x 16 x 16: 57 -> 5 us of host time,
// the usual grids 2 to 4).
struct TileChoice {
    int tx, ty, planes;
    double cost;
};
template <class Unit>
inline TileChoice choose_tile(int ex, int ey, int nz, int slots, Unit unit)
{
    TileChoice best{0, 0, 0, 0.0};
    auto offer = [&](int tx, int threads) {
        int ty = threads / (tx + 2) - 2;
        if (ty < 1) return;
        const int nty = (ey + ty - 1) / ty;
        ty = (ey + nty - 1) / nty;
        const long long tiles = (long long)((ex + tx - 1) / tx) * nty;
        for (int r = 1; r <= 6; ++r) {
            const long long slabs = (long long)slots * r / tiles;
            if (slabs < 1) continue;
            const int p = slabs >= nz ? 1 : (int)((nz + slabs - 1) / slabs);
            if (p > 64) continue;
            const long long blocks = tiles * ((nz + p - 1) / p);
            const int rounds = (int)((blocks + slots - 1) / slots);
            const double cost = (p + 2) * unit((tx + 2) * (ty + 2), rounds);
            if (best.tx == 0 || cost < 0.97 * best.cost || (tx == best.tx && ty == best.ty && cost < best.cost))
                best = TileChoice{tx, ty, p, cost};
        }
    };
    offer(ex < kPredTx ? ex : kPredTx, kTileThreads);
    const int least = ex < 14 ? ex : 14;
    for (int threads = kTileThreads; threads >= kTileThreads / 2; threads /= 2)
        for (int ntx = (ex + 125) / 126; (ex + ntx - 1) / ntx >= least; ntx += 1 + ntx / 8) {
            offer((ex + ntx - 1) / ntx, threads);
            if (ntx >= ex) break;
        }
    return best;
}

// a march of m cells, with the stencil beyond either end, keeps its byte offsets
// (padded planes) below 2^32
inline bool march_fits(const Geom &g, int m)
{
    return (idx_t)g.p[0] * g.p[1] * 8 * (m + 6) < (idx_t)1 << 32;
}

// blocks of a grid that run at a time in each kernel, for the choices below
// (one per CU; a batched step: its instance's share)
struct Slots {
    int march = kNumCUs, pred = kNumCUs, ct = kNumCUs;
};

// the grid alone: what sizes, layouts and the kernels without tiles need.  The
// tiles are for choose_tiles, whose search takes the host 1 to 4 us a grid: a
// batched step makes it once per size and boundary (2048 runs of one cell,
// bound by the host: 4.01 ms with two searches per run, 1.93 so).
inline Geom grid_geom(const vlct_grid *vg)
{
    Geom g{};
    g.n[0] = vg->nx;
    g.n[1] = vg->ny;
    g.n[2] = vg->nz;
    for (int d = 0; d < 3; ++d) {
        g.bc[d] = vg->bc[d];
        g.p[d] = g.n[d] + 2 * kGhost;
    }
    g.dl[0] = vg->dx;
    g.dl[1] = vg->dy;
    g.dl[2] = vg->dz;
    for (int d = 0; d < 3; ++d) g.idl[d] = 1.0 / g.dl[d];
    g.gamma = vg->gamma;
    g.gm1i = 1.0 / (vg->gamma - 1.0);
    g.cfl = vg->cfl;
    return g;
}

inline void choose_tiles(Geom &g, const Slots &slots)
{
    const int ex = g.n[0] + (g.bc[0] == VLCT_BC_OUTFLOW), ey = g.n[1] + (g.bc[1] == VLCT_BC_OUTFLOW);
    const int nz = g.n[2];
    // corrector marches: 16 cells per segment where that is four blocks per CU
    // or more (256^3: 0.73 ms per axis, 0.75 with 8); below, the m up to 32 that
    // minimises rounds of blocks x (m + 1) Riemann solves in a row (against 8
    // everywhere: 32^3 step 125 -> 98 us with 1, 512 x 16 x 16 PPMC 180 -> 142
    // with 3, 64^3 142 -> 131 with 5, 128^3 608 -> 590 with 19)
    for (int d = 1; d <= 2; ++d) {
        const long long cols = ((long long)(g.n[0] + 2) * (g.n[3 - d] + 2) + kBlock - 1) / kBlock;
        auto blocks = [&](int m) { return cols * ((g.n[d] + m - 1) / m); };
        g.march[d] = 16;
        if (blocks(16) < 4 * slots.march) {
            long long best = 0;
            for (int m = 32; m >= 1; --m) {
                const long long cost = (blocks(m) + slots.march - 1) / slots.march * (m + 1);
                if (march_fits(g, m) && (best == 0 || cost < best)) {
                    best = cost;
                    g.march[d] = m;
                }
            }
        }
    }
    // fused predictor, one block per CU at a time: the 32 x 13 tile with the
    // planes (a power of two) of least cost where no choice fills at most six
    // rounds, else the cheapest choice.  A plane takes a lone block of 512
    // threads 7.0 us and one of 256 threads 4.6 (32^3: 4 planes of the 32 x 13
    // tile 45 us, 1 plane of a smaller one 19; 64^3 step 142 -> 135 us with 3
    // planes for 4, 80^3 220 -> 202 with 20 x 20 tiles of 5)
    g.pr_tx = kPredTx;
    g.pr_ty = kPredTy;
    double best = -1.0;
    for (int p = 64; p >= 4; p /= 2) {
        const long long blocks = pred_tiles(g) * ((nz + p - 1) / p);
        const double cost = (double)((blocks + slots.pred - 1) / slots.pred) * (p + 2);
        if (best < 0.0 || cost < best) {
            best = cost;
            g.pred_slab = p;
        }
    }
    const TileChoice pr = choose_tile(ex, ey, nz, slots.pred, [](int threads, int rounds) {
        return (threads > kTileThreads / 2 ? 1.0 : 0.66) * rounds;
    });
    if (pr.tx && pr.cost < best) {
        g.pr_tx = pr.tx;
        g.pr_ty = pr.ty;
        g.pred_slab = pr.planes;
    }
    // CT update: 8 to 32 planes of the 32 x 13 tile where that is four blocks
    // per CU or more; below, the cheapest choice, a lone block taking 1.65 us a
    // plane and a round of several per CU 1.4 (32^3 21 -> 10 us; 96^3 PPMC step
    // 402 -> 382 us with 5 planes for 8, 100 x 75 x 50 154 -> 145 with 20 x 20
    // tiles of 2)
    g.ct_tx = kPredTx;
    g.ct_ty = kPredTy;
    const long long cols = ct_tiles(g);
    auto ctblocks = [&](int p) { return cols * ((nz + p - 1) / p); };
    g.ct_planes = 32;
    while (g.ct_planes > 8 && ctblocks(g.ct_planes) < 4 * slots.ct) g.ct_planes /= 2;
    if (ctblocks(8) < 4 * slots.ct) {
        const TileChoice ct = choose_tile(ex, ey, nz, slots.ct, [](int threads, int rounds) {
            return rounds == 1 ? (threads > kTileThreads / 2 ? 1.2 : 1.0) : rounds;
        });
        if (ct.tx) {
            g.ct_tx = ct.tx;
            g.ct_ty = ct.ty;
            g.ct_planes = ct.planes;
        }
    }
    const char *env = std::getenv("VLCT_TILES");
    if (!env || !*env) return;
    auto forced = [env](const char *key, int &v, int lo, int hi) {
        const int o = tile_override(env, key);
        if (o >= lo && o <= hi) v = o;
    };
    forced("ct", g.ct_planes, 1, kMaxN);
    forced("pred", g.pred_slab, 1, kMaxN);
    forced("predslab", g.pred_slab, 1, kMaxN);
    int m = 0, ctx = 0, prx = 0;
    forced("march", m, 1, 32);
    if (m > 0 && march_fits(g, m)) g.march[1] = g.march[2] = m;
    forced("cttile", ctx, 1, kTileThreads / 3 - 2);
    if (ctx > 0) {
        g.ct_tx = ctx;
        g.ct_ty = kTileThreads / (ctx + 2) - 2;
    }
    forced("predtile", prx, 1, kTileThreads / 3 - 2);
    if (prx > 0) {
        g.pr_tx = prx;
        g.pr_ty = kTileThreads / (prx + 2) - 2;
    }
}

// the tiles chosen for a grid of the same size and boundaries
inline void copy_tiles(Geom &g, const Geom &from)
{
    g.march[1] = from.march[1];
    g.march[2] = from.march[2];
    g.pr_tx = from.pr_tx;
    g.pr_ty = from.pr_ty;
    g.pred_slab = from.pred_slab;
    g.ct_tx = from.ct_tx;
    g.ct_ty = from.ct_ty;
    g.ct_planes = from.ct_planes;
}

inline Geom make_geom(const vlct_grid *vg)
{
    Geom g = grid_geom(vg);
    choose_tiles(g, Slots());
    return g;
}

inline size_t field_len(const int n[3], int f)
{
    size_t nx = n[0], ny = n[1], nz = n[2];
    if (f < 5) return nx * ny * nz;
    if (f == 5) return (nx + 1) * ny * nz;
    if (f == 6) return nx * (ny + 1) * nz;
    return nx * ny * (nz + 1);
}

inline bool state_ok(const vlct_state *s)
{
    if (!s) return false;
    const double *p[8] = {s->rho, s->mx, s->my, s->mz, s->E, s->bx, s->by, s->bz};
    for (int f = 0; f < 8; ++f)
        if (!p[f]) return false;
    return true;
}

inline StateP as_const(const vlct_state *s)
{
    StateP p;
    p.u[0] = s->rho; p.u[1] = s->mx; p.u[2] = s->my; p.u[3] = s->mz; p.u[4] = s->E;
    p.b[0] = s->bx; p.b[1] = s->by; p.b[2] = s->bz;
    return p;
}

inline StateP as_const(const StateW &s)
{
    StateP p;
    for (int f = 0; f < 5; ++f) p.u[f] = s.u[f];
    for (int d = 0; d < 3; ++d) p.b[d] = s.b[d];
    return p;
}

inline StateW as_mut(const vlct_state *s)
{
    StateW p;
    p.u[0] = s->rho; p.u[1] = s->mx; p.u[2] = s->my; p.u[3] = s->mz; p.u[4] = s->E;
    p.b[0] = s->bx; p.b[1] = s->by; p.b[2] = s->bz;
    return p;
}


inline unsigned nblocks(size_t work) { return (unsigned)((work + kBlock - 1) / kBlock); }

// grid size (multiple of the XCD count) for a kernel that remaps with xcd_block
inline unsigned xcd_grid(size_t logical_blocks) { return (unsigned)(kXcd * xcd_per(logical_blocks)); }

// upwind side of a face from its CT indicator (the sign of S_M, Eq. emf-upwind):
// 0 for S_M > 0, 1 for S_M < 0, 2 for neither
__device__ __forceinline__ uint8_t side_code(int s)
{
    return s > 0 ? (uint8_t)0 : (s < 0 ? (uint8_t)1 : (uint8_t)2);
}

// tape of one step (vlct_step_taped): the half-step state and the upwind side
// of every interior face of both stages (one byte, at the index of the cell
// whose low face it is)
struct TapeLayout {
    size_t half[8], side[2][3], total;
};

inline TapeLayout tape_layout(const int n[3])
{
    TapeLayout T;
    size_t off = 0;
    for (int f = 0; f < 8; ++f) {
        T.half[f] = off;
        off += align_up(field_len(n, f) * sizeof(double));
    }
    const size_t N = (size_t)n[0] * n[1] * n[2];
    for (int h = 0; h < 2; ++h)
        for (int d = 0; d < 3; ++d) {
            T.side[h][d] = off;
            off += align_up(N);
        }
    T.total = off;
    return T;
}

// launches of the step kernels (vlct.hip), also used by the adjoint to
// recompute the forward intermediates
int launch_prims(const Geom &g, const StateP &st, const Prims &P, uint32_t *status,
                 hipStream_t s);
// Steps 2-5: U^n -> U^{n+1/2} and its primitives (ghost layers included); with
// `side` also the upwind sides of the interior faces
int launch_pred(const Geom &g, const StateP &st, const StateW &half, const Prims &P,
                const double *dt_dev, uint32_t *status, uint8_t *const *side, hipStream_t s);
// Steps 6-7 and the cells' part of Step 9: EMFs and indicators of the faces of
// st into F, the updated cells (base minus the flux differences) into out.u
int launch_fluxes(const Geom &g, const StateP &st, const Prims &P, const Flux &F, int recon,
                  const StateP &base, const StateW &out, const double *dt_dev, uint32_t *status,
                  hipStream_t s);
// upwind sides of the interior faces of F, per axis
int launch_pack_sides(const Geom &g, const Flux &F, uint8_t *const side[3], hipStream_t s);

}  // namespace vlct
