// vlct_adjoint.hip -- adjoint (reverse derivative) of one VL+CT step (Caddy &
// Schneider, "Cholla-MHD", Sec. 2.2) on gfx950:
//
//   lam_in = (d U^{n+1} / d U^n)^T lam_out
//
// for a step of fixed size dt (dt is a parameter, not differentiated), with
// every branch (HLLD wave regions, limiter cases, CT upwind sides, floors)
// taken as in the forward evaluation at U^n.  The step is the composition
//   U^n -> W^n -> PCM/HLLD fluxes -> CT edge fields -> U^{n+1/2}
//       -> W^{n+1/2} -> reconstruction/HLLD fluxes -> CT edge fields -> U^{n+1}
// with U^{n+1/2} = U^n + G1(U^n) and U^{n+1} = U^n + G2(U^{n+1/2}), so
//   lam_in = lam + mu + G1'^T mu,   mu = G2'^T lam.
// Each stage transpose runs, per cell or face and without a tape:
//   edges   : edge-field cotangents from the face cotangents (curl transposed)
//   faces   : flux cotangents (flux differences transposed; B_t1/B_t2 fluxes
//             gathered from the two edges that use each, with the upwind
//             weights of the forward fluxes), then HLLD reversed (x by rows,
//             y and z by column marches; each cell reconstructed once)
//   recon   : PLMC/PLMP/PPMC/PPMP reversed per cell and axis (corrector only)
//   prims   : reference fields -(v x B) gathered from the 12 edges around the
//             cell and reversed, then primitive recovery reversed (the
//             predictor's in the march of its z faces)
// The forward intermediates (primitives, fluxes with their upwind indicators,
// the half-step state) are recomputed by the step's own kernels.  Periodic
// boundaries: a ghost cell or ghost flux row holds exactly the values of its
// periodic image, so every cotangent is accumulated on the image directly.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "vlct_common.hpp"
#include "mhd_adjoint.hpp"

namespace vlct {

// cotangent arrays of one stage's transposes (interior cells, cell_store order)
struct AdStage {
    double *le[3];        // edge fields E_A at the edge indexed like its cell
    uint32_t *wcode;      // upwind sides of the edges' four faces, 8 bits per component
    double *lw[8];        // primitives (rho, v, P, B_cc)
    double *lrec[3][14];  // interface states per axis: low face (7), high face (7)
};

__device__ __forceinline__ int wrapc(int i, int n) { return map_cell(i, n, VLCT_BC_PERIODIC); }

// Flat indices are 32-bit: a field of 2^32 elements would be 32 GiB, and the
// adjoint's workspace alone holds more than 80 of them.  Coordinates passed
// here lie in the grid; neighbours are reached by adding a step that wraps.
__device__ __forceinline__ u32 cell_at(const Geom &g, int i, int j, int k)
{
    return ((u32)k * (u32)g.n[1] + (u32)j) * (u32)g.n[0] + (u32)i;
}
template <int D>
__device__ __forceinline__ u32 face_at(const Geom &g, int i, int j, int k)
{
    return ((u32)k * (u32)(g.n[1] + (D == 1)) + (u32)j) * (u32)(g.n[0] + (D == 0)) + (u32)i;
}
// padded primitive index, i, j, k in [-G, n + G - 1]
__device__ __forceinline__ u32 prim_at(const Geom &g, int i, int j, int k)
{
    return ((u32)(k + kGhost) * (u32)g.p[1] + (u32)(j + kGhost)) * (u32)g.p[0] + (u32)(i + kGhost);
}
__device__ __forceinline__ void cell_coords(const Geom &g, u32 t, int x[3])
{
    const u32 r = t / (u32)g.n[0], k = r / (u32)g.n[1];
    x[0] = (int)(t - r * (u32)g.n[0]);
    x[1] = (int)(r - k * (u32)g.n[1]);
    x[2] = (int)k;
}
template <int A>
__device__ __forceinline__ u32 cell_stride(const Geom &g)
{
    return A == 0 ? 1u : (A == 1 ? (u32)g.n[0] : (u32)g.n[0] * (u32)g.n[1]);
}
// steps of a flat cell index to the neighbour below and above along A
template <int A>
__device__ __forceinline__ u32 step_lo(const Geom &g, const int x[3])
{
    const u32 s = cell_stride<A>(g);
    return x[A] > 0 ? 0u - s : (u32)(g.n[A] - 1) * s;
}
template <int A>
__device__ __forceinline__ u32 step_hi(const Geom &g, const int x[3])
{
    const u32 s = cell_stride<A>(g);
    return x[A] < g.n[A] - 1 ? s : 0u - (u32)(g.n[A] - 1) * s;
}

// lab component of the primitive array for sweep-frame slot s of axis d:
// (rho, v_n, v_t1, v_t2, P, B_t1, B_t2) -> (0, 1+d, 1+t1, 1+t2, 4, 5+t1, 5+t2)
__host__ __device__ __forceinline__ int lab_slot(int d, int s)
{
    if (s == 0 || s == 4) return s;
    const int off = s < 4 ? 1 : 5;
    const int r = s < 4 ? s - 1 : s - 5 + 1;  // 0 normal, 1 t1, 2 t2
    return off + (d + r) % 3;
}
// lab conserved cell variable of sweep-frame flux component c (< 5) of axis d
__host__ __device__ __forceinline__ int lab_cons(int d, int c)
{
    if (c == 0 || c == 4) return c;
    return 1 + (d + c - 1) % 3;
}

__device__ __forceinline__ W7 w7_at(const Prims &P, int d, u32 o)
{
    return W7{P.w[0][o], P.w[lab_slot(d, 1)][o], P.w[lab_slot(d, 2)][o], P.w[lab_slot(d, 3)][o],
              P.w[4][o], P.w[lab_slot(d, 5)][o], P.w[lab_slot(d, 6)][o]};
}

// upwind sides of one stage's interior faces (side_code, per axis, at the
// index of the cell whose low face it is)
struct Sides {
    const uint8_t *s[3];
};

// 8-bit code of edge (A, x): the sides of the faces F_B(x), F_B(x - e_C),
// F_C(x), F_C(x - e_B) (the four upwind terms of the edge field)
template <int A>
__device__ __forceinline__ u32 edge_code(const Geom &g, const Sides &sd, const int x[3], u32 t)
{
    constexpr int B = (A + 1) % 3, C = (A + 2) % 3;
    return (u32)sd.s[B][t] | ((u32)sd.s[B][t + step_lo<C>(g, x)] << 2) | ((u32)sd.s[C][t] << 4) |
           ((u32)sd.s[C][t + step_lo<B>(g, x)] << 6);
}

// twice the weight (1, 0 or 1/2 by the side) of the low side of upwind term q
// of edge field A at flat cell index t; the high side has the rest
__device__ __forceinline__ int low2(u32 code, int q) { return (0x52 >> (2 * ((code >> (2 * q)) & 3u))) & 3; }
__device__ __forceinline__ int high2(u32 code, int q) { return 2 - low2(code, q); }

// the cotangent of the state that a stage starts from: before the stage's own
// terms it is that of the step's result (each periodic duplicate face folded
// into face 0, which the step copies to it) plus that of the half step (add),
// or nothing (the corrector's, whose input state enters through it alone)
struct AdBase {
    StateP lam, half;
    int add;
};
template <int D>
__device__ __forceinline__ double folded(const Geom &g, const StateP &lam, u32 f, const int x[3])
{
    double v = lam.b[D][f];
    if (x[D] == 0) {
        const u32 s = D == 0 ? 1u : (D == 1 ? (u32)g.n[0] : (u32)g.n[0] * (u32)g.n[1]);
        v += lam.b[D][f + (u32)g.n[D] * s];
    }
    return v;
}
template <int D>
__device__ __forceinline__ double base_face(const Geom &g, const AdBase &base, u32 f, const int x[3])
{
    return base.add ? folded<D>(g, base.lam, f, x) + base.half.b[D][f] : 0.0;
}
// the duplicate plane itself carries nothing
template <int D>
__device__ __forceinline__ void clear_duplicate(const Geom &g, const StateW &lacc, u32 f, const int x[3])
{
    if (x[D] == 0) {
        const u32 s = D == 0 ? 1u : (D == 1 ? (u32)g.n[0] : (u32)g.n[0] * (u32)g.n[1]);
        lacc.b[D][f + (u32)g.n[D] * s] = 0.0;
    }
}

// edge-field cotangents (curl of the face update transposed): the face update
// is b_x -= cy (Ez(j+1) - Ez(j)) - cz (Ey(k+1) - Ey(k)) and cyclically, and
// the upwind codes of the edges.  fold: lout's duplicate faces count for face 0.
// zero_lw: also clears the cell's primitive cotangents S.lw, into which the
// reconstruction transposes that follow add
__global__ void k_ad_edges(Geom g, StateP lout, int fold, Sides sd, AdStage S, const double *dt_dev,
                           double factor, int zero_lw)
{
    const u32 N = (u32)g.n[0] * (u32)g.n[1] * (u32)g.n[2];
    const u32 t = blockIdx.x * (u32)kBlock + threadIdx.x;
    if (t >= N) return;
    int x[3];
    cell_coords(g, t, x);
    const int i = x[0], j = x[1], k = x[2];
    const int im = i > 0 ? i - 1 : g.n[0] - 1, jm = j > 0 ? j - 1 : g.n[1] - 1,
              km = k > 0 ? k - 1 : g.n[2] - 1;
    const double cx = factor * dt_dev[0] / g.dl[0], cy = factor * dt_dev[0] / g.dl[1],
                 cz = factor * dt_dev[0] / g.dl[2];
    auto bx = [&](int a, int b, int c) {
        const u32 f = face_at<0>(g, a, b, c);
        return fold ? folded<0>(g, lout, f, x) : lout.b[0][f];
    };
    auto by = [&](int a, int b, int c) {
        const u32 f = face_at<1>(g, a, b, c);
        return fold ? folded<1>(g, lout, f, x) : lout.b[1][f];
    };
    auto bz = [&](int a, int b, int c) {
        const u32 f = face_at<2>(g, a, b, c);
        return fold ? folded<2>(g, lout, f, x) : lout.b[2][f];
    };
    const double x0 = bx(i, j, k), y0 = by(i, j, k), z0 = bz(i, j, k);
    S.le[0][t] = cz * (y0 - by(i, j, km)) + cy * (bz(i, jm, k) - z0);
    S.le[1][t] = cz * (bx(i, j, km) - x0) + cx * (z0 - bz(im, j, k));
    S.le[2][t] = cy * (x0 - bx(i, jm, k)) + cx * (by(im, j, k) - y0);
    S.wcode[t] = edge_code<0>(g, sd, x, t) | (edge_code<1>(g, sd, x, t) << 8) |
                 (edge_code<2>(g, sd, x, t) << 16);
    if (zero_lw)
        for (int f = 0; f < 8; ++f) S.lw[f][t] = 0.0;
}

// cotangents of the 7 fluxes of the face of axis D at x (the low face of cell
// x, flat index t): its loads, then its arithmetic, so that a march can issue
// the loads ahead of other work
struct FluxLoads {
    double hi[5], lo[5], e5x, e5y, e6x, e6y;
    u32 code, c5, c6;
};
template <int D>
__device__ __forceinline__ FluxLoads flux_loads(const Geom &g, const StateP &lout,
                                                const AdStage &S, const int x[3], u32 t)
{
    FluxLoads v;
    const u32 cl = t + step_lo<D>(g, x);
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        const int f = lab_cons(D, q);
        v.hi[q] = lout.u[f][t];
        v.lo[q] = lout.u[f][cl];
    }
    constexpr int A5 = (D + 2) % 3, C5 = (A5 + 2) % 3, A6 = (D + 1) % 3, B6 = (A6 + 1) % 3;
    const u32 y5 = t + step_hi<C5>(g, x), y6 = t + step_hi<B6>(g, x);
    v.code = S.wcode[t];
    v.c5 = S.wcode[y5];
    v.c6 = S.wcode[y6];
    v.e5x = S.le[A5][t];
    v.e5y = S.le[A5][y5];
    v.e6x = S.le[A6][t];
    v.e6y = S.le[A6][y6];
    return v;
}
template <int D>
__device__ __forceinline__ void flux_combine(const FluxLoads &v, double c, double lf[7])
{
    // cell update u -= c (F(x + e_D) - F(x))
#pragma unroll
    for (int q = 0; q < 5; ++q) lf[q] = c * (v.hi[q] - v.lo[q]);
    // F_D[B_t1] enters the edges E_A, A = D + 2, as -F: at x (weights of the
    // high sides of terms 3 and 4) and at x + e_C, C = D + 1 (low sides)
    {
        constexpr int A = (D + 2) % 3;
        const u32 cx = v.code >> (8 * A), cy = v.c5 >> (8 * A);
        const double wx = 1.0 + 0.5 * (double)(high2(cx, 2) + high2(cx, 3));
        const double wy = 1.0 + 0.5 * (double)(low2(cy, 2) + low2(cy, 3));
        lf[5] = -0.25 * wx * v.e5x + -0.25 * wy * v.e5y;
    }
    // F_D[B_t2] enters the edges E_A, A = D + 1, as +F: at x (high sides of
    // terms 1 and 2) and at x + e_B, B = D + 2 (low sides)
    {
        constexpr int A = (D + 1) % 3;
        const u32 cx = v.code >> (8 * A), cy = v.c6 >> (8 * A);
        const double wx = 1.0 + 0.5 * (double)(high2(cx, 0) + high2(cx, 1));
        const double wy = 1.0 + 0.5 * (double)(low2(cy, 0) + low2(cy, 1));
        lf[6] = 0.25 * wx * v.e6x + 0.25 * wy * v.e6y;
    }
}
template <int D>
__device__ __forceinline__ void flux_cotangent(const Geom &g, const StateP &lout,
                                               const AdStage &S, const int x[3], u32 t,
                                               double c, double lf[7])
{
    flux_combine<D>(flux_loads<D>(g, lout, S, x, t), c, lf);
}

// The cell reversal: its loads, then its arithmetic.
// Edge fields around cell x: E_A of the edges x, x + e_B, x + e_C and
// x + e_B + e_C, of which the cell is r00, r10, r01 and r11, and the upwind
// codes of the cell's seven edge positions (offset bits x, y, z).
struct CellLoads {
    double le[3][4], v[3], b[3], flo[3], fhi[3], u[5], base[5];
    u32 code[7];
};
template <int A>
__device__ __forceinline__ void edge_loads(const AdStage &S, u32 t, const u32 hi[3], double le[4])
{
    constexpr int B = (A + 1) % 3, C = (A + 2) % 3;
    le[0] = S.le[A][t];
    le[1] = S.le[A][t + hi[B]];
    le[2] = S.le[A][t + hi[C]];
    le[3] = S.le[A][t + hi[B] + hi[C]];
}
__device__ __forceinline__ CellLoads cell_loads(const Geom &g, const StateP &st, const Prims &P,
                                                const AdStage &S, const AdBase &base,
                                                const int x[3], u32 t)
{
    CellLoads c;
    const u32 hi[3] = {step_hi<0>(g, x), step_hi<1>(g, x), step_hi<2>(g, x)};
#pragma unroll
    for (int m = 0; m < 7; ++m)
        c.code[m] = S.wcode[t + (m & 1 ? hi[0] : 0u) + (m & 2 ? hi[1] : 0u) + (m & 4 ? hi[2] : 0u)];
    edge_loads<0>(S, t, hi, c.le[0]);
    edge_loads<1>(S, t, hi, c.le[1]);
    edge_loads<2>(S, t, hi, c.le[2]);
    const u32 o = prim_at(g, x[0], x[1], x[2]);
    const u32 f[3] = {face_at<0>(g, x[0], x[1], x[2]), face_at<1>(g, x[0], x[1], x[2]), t};
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        c.v[l] = P.w[1 + l][o];
        c.b[l] = P.w[5 + l][o];
        c.flo[l] = st.b[l][f[l]];
        c.fhi[l] = st.b[l][f[l] + hi[l]];
    }
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        c.u[q] = st.u[q][t];
        c.base[q] = base.add ? base.lam.u[q][t] + base.half.u[q][t] : 0.0;
    }
    return c;
}

// cotangent of -(v x B)_A at the cell from the four A-edges around it
template <int A>
__device__ __forceinline__ double eref_cotangent(const CellLoads &c)
{
    constexpr int B = (A + 1) % 3, C = (A + 2) % 3;
    auto code = [&](int m) { return c.code[m] >> (8 * A); };
    const u32 c0 = code(0), c1 = code(1 << B), c2 = code(1 << C), c3 = code((1 << B) + (1 << C));
    double acc = 0.5 * (double)(high2(c0, 0) + high2(c0, 2)) * c.le[A][0];
    acc += 0.5 * (double)(low2(c1, 0) + high2(c1, 3)) * c.le[A][1];
    acc += 0.5 * (double)(high2(c2, 1) + low2(c2, 2)) * c.le[A][2];
    acc += 0.5 * (double)(low2(c3, 1) + low2(c3, 3)) * c.le[A][3];
    return -0.25 * acc;
}

// reference fields -(v x B) and primitive recovery (Sec. 2.1; B_cc = face
// average) of a cell reversed: its primitive cotangents lw become those of its
// conserved variables, written to lacc.u on top of the base, and lb of each of
// its six faces (half to either side).  A floored quantity is a constant.
__device__ __forceinline__ void cell_rev(const Geom &g, const CellLoads &c, const AdBase &base,
                                         const StateW &lacc, u32 t, double lw[8], double lb[3])
{
    {
        const double vx = c.v[0], vy = c.v[1], vz = c.v[2];
        const double bx = c.b[0], by = c.b[1], bz = c.b[2];
        const double ex = eref_cotangent<0>(c), ey = eref_cotangent<1>(c), ez = eref_cotangent<2>(c);
        lw[1] += bz * ey - by * ez;
        lw[2] += -bz * ex + bx * ez;
        lw[3] += by * ex - bx * ey;
        lw[5] += -vz * ey + vy * ez;
        lw[6] += vz * ex - vx * ez;
        lw[7] += -vy * ex + vx * ey;
    }
    const double bc[3] = {0.5 * (c.flo[0] + c.fhi[0]), 0.5 * (c.flo[1] + c.fhi[1]),
                          0.5 * (c.flo[2] + c.fhi[2])};
    double d = c.u[0];
    const bool dfloor = !(d >= kFloorRho);
    if (dfloor) d = kFloorRho;
    const double id = mrcp(d);
    const double v[3] = {c.u[1] * id, c.u[2] * id, c.u[3] * id};
    const double ke = 0.5 * d * (v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
    const double me = 0.5 * (bc[0] * bc[0] + bc[1] * bc[1] + bc[2] * bc[2]);
    const double p = (g.gamma - 1.0) * (c.u[4] - ke - me);
    const bool pfloor = !(p >= kFloorP);
    const double gm1 = g.gamma - 1.0;
    const double lp = pfloor ? 0.0 : lw[4];
    const double v2 = v[0] * v[0] + v[1] * v[1] + v[2] * v[2];
    double lrho = dfloor ? 0.0 : lw[0] + lp * gm1 * 0.5 * v2;
    auto put = [&](int f, double a) { lacc.u[f][t] = base.add ? c.base[f] + a : a; };
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        if (!dfloor) lrho -= lw[1 + l] * v[l] * id;
        put(1 + l, lw[1 + l] * id - lp * gm1 * v[l]);
        lb[l] = 0.5 * (lw[5 + l] - lp * gm1 * bc[l]);
    }
    put(0, lrho);
    put(4, lp * gm1);
}

// a face's two states wait in LDS (each thread its own slots) while HLLD is
// reversed, which fetches them again (hlld_rev): 44 registers that two waves
// per SIMD would otherwise spill
template <int B>
struct ParkedStates {
    double (*s)[B];
    int tid;
    __device__ __forceinline__ void put(int o, const W7 &w) const
    {
        double v[7];
        to_arr(w, v);
#pragma unroll
        for (int q = 0; q < 7; ++q) s[o + q][tid] = v[q];
    }
    __device__ __forceinline__ W7 get(int o) const
    {
        return W7{s[o][tid],     s[o + 1][tid], s[o + 2][tid], s[o + 3][tid],
                  s[o + 4][tid], s[o + 5][tid], s[o + 6][tid]};
    }
    __device__ __forceinline__ void operator()(W7 &L, W7 &R) const
    {
        asm volatile("" ::: "memory");
        L = get(0);
        R = get(7);
    }
};

// PCM stage: flux cotangents, then HLLD reversed at the forward states (the
// cell primitives), then primitive recovery, without a pass over memory per
// face.  The x kernel writes the sum of the cotangents of a cell's two x-face
// states, the y march adds those of the y-faces, the z march those of the
// z-faces and reverses the finished cell: about 125 doubles moved per cell
// where storing both states' cotangents of every face moved 200.  The marches
// run one wave per SIMD, whose spare registers hold the next face's and the
// cell's loads during a reversal: 128^3 171 + 156 + 270 us, 222 + 406 for the
// marches without loads ahead (75% of their cycles waiting), 568 + 262 as face
// kernels and a gather; 64^3 26 + 26 + 42 us (80 + 36).
//
// x: items (row, face 0 .. nx) of every row in one flat sequence (face nx is
// face 0 again), blocks of kBlock items overlapping by one; the cotangent of a
// face's left state goes to the item on the left through LDS.  The x kernel
// also starts the z-faces' cotangents, which the z march's segments share.
__host__ __device__ __forceinline__ idx_t ad_pcm_row_blocks(const Geom &g)
{
    const idx_t items = (idx_t)(g.n[0] + 1) * g.n[1] * g.n[2];
    return (items - 1 + kBlock - 2) / (kBlock - 1);
}

__global__ __launch_bounds__(kBlock, 2) void k_ad_pcm_row(Geom g, Prims P, StateP st, StateP lout,
                                                          AdStage S, AdBase base, StateW lacc,
                                                          const double *dt_dev, double factor)
{
    __shared__ double lds[7][kBlock], park[14][kBlock];
    const u32 per_row = (u32)g.n[0] + 1, items = per_row * (u32)g.n[1] * (u32)g.n[2];
    const int tid = threadIdx.x;
    const u32 q = blockIdx.x * (u32)(kBlock - 1) + tid;
    const bool have = q < items;
    const u32 row = q / per_row, k = row / (u32)g.n[1];
    const int i = (int)(q - row * per_row);
    const int x[3] = {i < g.n[0] ? i : 0, (int)(row - k * (u32)g.n[1]), (int)k};
    W7 aL{0, 0, 0, 0, 0, 0, 0}, aR{0, 0, 0, 0, 0, 0, 0};
    const u32 t = cell_at(g, x[0], x[1], x[2]);
    const bool cell = have && i < g.n[0] && tid < kBlock - 1;
    if (have) {
        double lf[7];
        flux_cotangent<0>(g, lout, S, x, t, factor * dt_dev[0] / g.dl[0], lf);
        const u32 o = prim_at(g, i, x[1], x[2]);
        const u32 fo = face_at<0>(g, x[0], x[1], x[2]);
        double abn = 0.0;
        const ParkedStates<kBlock> states{park, tid};
        const W7 wl = w7_at(P, 0, o - 1), wr = w7_at(P, 0, o);
        states.put(0, wl);
        states.put(7, wr);
        hlld_rev(wl, wr, st.b[0][fo], g.gamma, g.gm1i, lf, aL, aR, abn, states);
        __builtin_amdgcn_sched_barrier(0);
        if (cell) {
            lacc.b[0][fo] = base_face<0>(g, base, fo, x) + abn;
            clear_duplicate<0>(g, lacc, fo, x);
        }
    }
    const double vl[7] = {aL.d, aL.u, aL.v, aL.w, aL.p, aL.by, aL.bz};
#pragma unroll
    for (int c = 0; c < 7; ++c) lds[c][tid] = vl[c];
    __syncthreads();
    if (!cell) return;
    const double vr[7] = {aR.d, aR.u, aR.v, aR.w, aR.p, aR.by, aR.bz};
#pragma unroll
    for (int c = 0; c < 7; ++c) S.lw[lab_slot(0, c)][t] = vr[c] + lds[c][tid + 1];
    lacc.b[2][t] = base_face<2>(g, base, t, x);
    clear_duplicate<2>(g, lacc, t, x);
}

// y and z: one thread per column and segment of M cells, which computes its
// faces and the one above it (whose left state is that of its top cell; the
// normal-field cotangent stays with the segment that owns the face) and
// carries each face's right-state cotangent to the next.
template <int D>
__global__ __launch_bounds__(kBlock, 1) void k_ad_pcm_march(Geom g, Prims P, StateP st, StateP lout,
                                                            AdStage S, AdBase base, StateW lacc,
                                                            const double *dt_dev, double factor,
                                                            int M)
{
    static_assert(D == 1 || D == 2, "columns march along y or z");
    constexpr int T = D == 1 ? 2 : 1;
    const int nD = g.n[D];
    const u32 cols = (u32)g.n[0] * (u32)g.n[T];
    const u32 ncb = (cols + kBlock - 1) / kBlock;
    const u32 seg = blockIdx.x / ncb;
    const u32 col = (blockIdx.x - seg * ncb) * kBlock + threadIdx.x;
    if (col >= cols) return;
    int x[3];
    x[T] = (int)(col / (u32)g.n[0]);
    x[0] = (int)(col - (u32)x[T] * (u32)g.n[0]);
    x[D] = 0;
    const int s0 = (int)seg * M, s1 = min(s0 + M, nD);  // cells [s0, s1)
    const double c = factor * dt_dev[0] / g.dl[D];
    const u32 tcol = cell_at(g, x[0], x[1], x[2]), tstep = cell_stride<D>(g);
    x[D] = s0 - 1;
    u32 po = prim_at(g, x[0], x[1], x[2]);
    const u32 pstep = D == 1 ? (u32)g.p[0] : (u32)g.p[0] * (u32)g.p[1];
    // the face's two states and the cotangent of the low-face state of the cell
    // below wait in LDS (thread-private)
    __shared__ double alow[7][kBlock], park[14][kBlock];
    const int tid = threadIdx.x;
    const ParkedStates<kBlock> states{park, tid};
    states.put(0, w7_at(P, D, po));
    double lbn = 0.0;
    // the loads of face a, a face ahead of its reversal
    FluxLoads fl;
    W7 wr;
    double bn;
    auto load_face = [&](int a) {
        x[D] = a < nD ? a : 0;
        fl = flux_loads<D>(g, lout, S, x, tcol + (u32)x[D] * tstep);
        bn = st.b[D][face_at<D>(g, x[0], x[1], x[2])];
        po += pstep;
        wr = w7_at(P, D, po);
    };
    load_face(s0);
    for (int a = s0; a <= s1; ++a) {
        double lf[7];
        flux_combine<D>(fl, c, lf);
        const double bna = bn;
        const W7 wra = wr;
        states.put(7, wra);
        if (a < s1) load_face(a + 1);
        // what this face and the cell below it read and add to
        double own = 0.0, lw[8];
        CellLoads cl;
        x[D] = a < nD ? a : 0;
        const u32 fo = face_at<D>(g, x[0], x[1], x[2]);
        if (D == 1 && a < s1) own = base_face<1>(g, base, fo, x);
        const u32 tc = tcol + (u32)(a - 1) * tstep;
        if (a > s0) {
#pragma unroll
            for (int f = 0; f < 8; ++f)
                if (D == 2 || (f != 5 && f != 6)) lw[f] = S.lw[f][tc];
            if (D == 2) {
                x[D] = a - 1;
                cl = cell_loads(g, st, P, S, base, x, tc);
                x[D] = a < nD ? a : 0;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        W7 aL{0, 0, 0, 0, 0, 0, 0}, aR{0, 0, 0, 0, 0, 0, 0};
        double abn = 0.0;
        hlld_rev(states.get(0), wra, bna, g.gamma, g.gm1i, lf, aL, aR, abn, states);
        states.put(0, states.get(7));
        if (D == 1 && a < s1) {
            lacc.b[1][fo] = own + abn;
            clear_duplicate<1>(g, lacc, fo, x);
        }
        if (a > s0) {
            // cell a - 1 has its face states' cotangents
            x[D] = a - 1;
            const double vl[7] = {aL.d, aL.u, aL.v, aL.w, aL.p, aL.by, aL.bz};
            if (D == 1) {
#pragma unroll
                for (int q = 0; q < 7; ++q) {
                    const int f = lab_slot(1, q);
                    // the x sweep has no B_x component
                    const double sum = alow[q][tid] + vl[q];
                    S.lw[f][tc] = f == 5 ? sum : lw[f] + sum;
                }
            } else {
#pragma unroll
                for (int q = 0; q < 7; ++q) lw[lab_slot(2, q)] += alow[q][tid] + vl[q];
                double lb[3];
                cell_rev(g, cl, base, lacc, tc, lw, lb);
                const u32 f0 = face_at<0>(g, x[0], x[1], x[2]), f1 = face_at<1>(g, x[0], x[1], x[2]);
                atomicAdd(&lacc.b[0][f0], lb[0]);
                atomicAdd(&lacc.b[0][f0 + step_hi<0>(g, x)], lb[0]);
                atomicAdd(&lacc.b[1][f1], lb[1]);
                atomicAdd(&lacc.b[1][f1 + step_hi<1>(g, x)], lb[1]);
                atomicAdd(&lacc.b[2][tc], lbn + lb[2]);
                lbn = lb[2];
            }
        }
        // the face's own term waits for the cell above it; the last one's (the
        // next segment's) does not count here
        if (D == 2) lbn = a < s1 ? lbn + abn : lbn;
        const double vr[7] = {aR.d, aR.u, aR.v, aR.w, aR.p, aR.by, aR.bz};
#pragma unroll
        for (int q = 0; q < 7; ++q) alow[q][tid] = vr[q];
    }
    if (D == 2) {
        x[D] = s1 < nD ? s1 : 0;
        atomicAdd(&lacc.b[2][tcol + (u32)x[D] * tstep], lbn);
    }
}

// faces of axis D = y or z with a parabolic corrector, one thread per
// column (i, j or k) and segment of M cells along D: each cell is
// reconstructed once and its high-face state carried to the next face.  Per
// face the same work as k_ad_faces_row.
__host__ __device__ __forceinline__ idx_t ad_march_blocks(const Geom &g, int D, int m)
{
    const int T = D == 1 ? 2 : 1;
    const idx_t cols = (idx_t)g.n[0] * g.n[T];
    return ((cols + kBlock - 1) / kBlock) * ((g.n[D] + m - 1) / m);
}

// cells per segment of the adjoint marches: `slots` blocks at a time and
// m + 1 reversals in a row in each, so the m up to 32 of least rounds x (m + 1)
// (64^3, third order, against 16 and 8: faces 131 -> 44 us an axis, reversed
// reconstructions 166 -> 104; 128^3, 32 and 16 are the same)
static int ad_march_segment(const Geom &g, int D, int slots)
{
    const char *env = std::getenv("VLCT_TILES");
    const int o = env ? tile_override(env, "admarch") : 0;
    if (o >= 1 && o <= 64) return o;
    idx_t best = 0;
    int len = 1;
    for (int m = 32; m >= 1; --m) {
        const idx_t cost = (ad_march_blocks(g, D, m) + slots - 1) / slots * (m + 1);
        if (best == 0 || cost < best) {
            best = cost;
            len = m;
        }
    }
    return len;
}

template <int D, int RECON>
__global__ __launch_bounds__(kBlock) void k_ad_faces_march(Geom g, Prims P, StateP st,
                                                           StateP lout, AdStage S,
                                                           StateW lacc, const double *dt_dev,
                                                           double factor, int M)
{
    static_assert(D == 1 || D == 2, "columns march along y or z");
    static_assert(RECON == VLCT_RECON_PPMC || RECON == VLCT_RECON_PPMP, "parabolic reconstructions");
    constexpr int T = D == 1 ? 2 : 1;
    constexpr bool kChar = RECON == VLCT_RECON_PPMC;
    constexpr int R = 2;
    const int nD = g.n[D];
    const u32 cols = (u32)g.n[0] * (u32)g.n[T];
    const u32 ncb = (cols + kBlock - 1) / kBlock;
    const u32 seg = blockIdx.x / ncb;
    const u32 col = (blockIdx.x - seg * ncb) * kBlock + threadIdx.x;
    if (col >= cols) return;
    int x[3];
    x[T] = (int)(col / (u32)g.n[0]);
    x[0] = (int)(col - (u32)x[T] * (u32)g.n[0]);
    x[D] = 0;
    const int s0 = (int)seg * M, s1 = min(s0 + M, nD);  // cells [s0, s1)
    const double c = factor * dt_dev[0] / g.dl[D];
    const u32 tcol = cell_at(g, x[0], x[1], x[2]), tstep = cell_stride<D>(g);
    x[D] = s0 - 1 - R;
    u32 po = prim_at(g, x[0], x[1], x[2]);
    const u32 pstep = D == 1 ? (u32)g.p[0] : (u32)g.p[0] * (u32)g.p[1];
    // stencil window of cells a - R .. a + R for a = s0 - 1
    W7 win[2 * R + 1];
    double bnc[2 * R + 1];
#pragma unroll
    for (int q = 0; q < 2 * R + 1; ++q) {
        win[q] = w7_at(P, D, po);
        bnc[q] = P.w[5 + D][po];
        po += pstep;
    }
    W7 prev{};
    uint32_t fprev = 0;
    for (int a = s0 - 1; a < s1; ++a) {
        W7 fm, fp;
        ppmc<kChar>(win[0], win[1], win[2], win[3], win[4], bnc[2], g.gamma, fm, fp);
        const uint32_t flo = floor_state(fm), fhi = floor_state(fp);
        if (a >= s0) {
            // the face a - 1/2 between the carried high state and this low state
            x[D] = a;
            const u32 t = tcol + (u32)a * tstep;
            double lf[7];
            flux_cotangent<D>(g, lout, S, x, t, c, lf);
            const u32 fo = face_at<D>(g, x[0], x[1], x[2]);
            W7 aL{0, 0, 0, 0, 0, 0, 0}, aR{0, 0, 0, 0, 0, 0, 0};
            double abn = 0.0;
            hlld_rev(prev, fm, st.b[D][fo], g.gamma, g.gm1i, lf, aL, aR, abn);
            lacc.b[D][fo] = abn;
            const u32 cl = t + step_lo<D>(g, x);
            const double vl[7] = {aL.d, aL.u, aL.v, aL.w, aL.p, aL.by, aL.bz};
            const double vr[7] = {aR.d, aR.u, aR.v, aR.w, aR.p, aR.by, aR.bz};
#pragma unroll
            for (int q = 0; q < 7; ++q) {
                double u = vl[q], v = vr[q];
                if (q == 0 && (fprev & kStatusDensityFloor)) u = 0.0;
                if (q == 4 && (fprev & kStatusPressureFloor)) u = 0.0;
                if (q == 0 && (flo & kStatusDensityFloor)) v = 0.0;
                if (q == 4 && (flo & kStatusPressureFloor)) v = 0.0;
                S.lrec[D][7 + q][cl] = u;  // high face of the cell below
                S.lrec[D][q][t] = v;       // low face of this cell
            }
        }
        prev = fp;
        fprev = fhi;
        if (a + 1 < s1) {
#pragma unroll
            for (int q = 0; q < 2 * R; ++q) {
                win[q] = win[q + 1];
                bnc[q] = bnc[q + 1];
            }
            win[2 * R] = w7_at(P, D, po);
            bnc[2 * R] = P.w[5 + D][po];
            po += pstep;
        }
    }
}

// blocks of the reconstructing x kernels: one wave, so that no barrier makes
// four waves of a CU wait for each other's loads (fused PLMC x kernel at 128^3
// 398 -> 366 us; 369 with 128 threads)
constexpr int kAdRow = 64;

// faces of axis x with a parabolic corrector: items (row, cell) with
// cells -1 .. nx-1 of every row in one flat sequence; a block reconstructs
// kAdRow consecutive items once each, hands the high-face states to the right
// neighbour through LDS, and each item with a left neighbour in its block and
// row takes the face between them (consecutive blocks overlap by one item).
// Per face: flux cotangents, HLLD reversed, the cotangents of the two floored
// states stored per cell and axis (a floored component carries none).
__host__ __device__ __forceinline__ idx_t ad_row_blocks(const Geom &g)
{
    const idx_t items = (idx_t)(g.n[0] + 1) * g.n[1] * g.n[2];
    return (items - 1 + kAdRow - 2) / (kAdRow - 1);
}

template <int RECON>
__global__ __launch_bounds__(kAdRow, 2) void k_ad_faces_row(Geom g, Prims P, StateP st,
                                                         StateP lout, AdStage S, StateW lacc,
                                                         const double *dt_dev, double factor)
{
    static_assert(RECON == VLCT_RECON_PPMC || RECON == VLCT_RECON_PPMP, "parabolic reconstructions");
    constexpr bool kChar = RECON == VLCT_RECON_PPMC;
    __shared__ double lds[7][kAdRow];
    __shared__ uint32_t lfl[kAdRow];
    const int nx = g.n[0];
    const u32 per_row = (u32)nx + 1, items = per_row * (u32)g.n[1] * (u32)g.n[2];
    const int t = threadIdx.x;
    const u32 q = blockIdx.x * (u32)(kAdRow - 1) + t;
    const bool have = q < items;
    const u32 row = q / per_row, plane = row / (u32)g.n[1];
    const int x[3] = {(int)(q - row * per_row) - 1, (int)(row - plane * (u32)g.n[1]), (int)plane};
    W7 fm{}, fp{};
    uint32_t flo = 0, fhi = 0;
    if (have) {
        const u32 po = prim_at(g, x[0], x[1], x[2]);
        auto at = [&](int off) { return po + (u32)off; };
        const double bn = P.w[5][at(0)];
        ppmc<kChar>(w7_at(P, 0, at(-2)), w7_at(P, 0, at(-1)), w7_at(P, 0, at(0)),
                    w7_at(P, 0, at(1)), w7_at(P, 0, at(2)), bn, g.gamma, fm, fp);
        flo = floor_state(fm);
        fhi = floor_state(fp);
    }
    lds[0][t] = fp.d; lds[1][t] = fp.u; lds[2][t] = fp.v; lds[3][t] = fp.w;
    lds[4][t] = fp.p; lds[5][t] = fp.by; lds[6][t] = fp.bz;
    lfl[t] = fhi;
    __syncthreads();
    if (t < 1 || !have || x[0] < 0) return;
    const W7 wl{lds[0][t - 1], lds[1][t - 1], lds[2][t - 1], lds[3][t - 1],
                lds[4][t - 1], lds[5][t - 1], lds[6][t - 1]};
    const uint32_t fl = lfl[t - 1];
    const u32 tc = cell_at(g, x[0], x[1], x[2]);
    double lf[7];
    flux_cotangent<0>(g, lout, S, x, tc, factor * dt_dev[0] / g.dl[0], lf);
    const u32 fo = face_at<0>(g, x[0], x[1], x[2]);
    W7 aL{0, 0, 0, 0, 0, 0, 0}, aR{0, 0, 0, 0, 0, 0, 0};
    double abn = 0.0;
    hlld_rev(wl, fm, st.b[0][fo], g.gamma, g.gm1i, lf, aL, aR, abn);
    lacc.b[0][fo] = abn;
    const u32 cl = tc + step_lo<0>(g, x);
    const double vl[7] = {aL.d, aL.u, aL.v, aL.w, aL.p, aL.by, aL.bz};
    const double vr[7] = {aR.d, aR.u, aR.v, aR.w, aR.p, aR.by, aR.bz};
#pragma unroll
    for (int c = 0; c < 7; ++c) {
        double u = vl[c], v = vr[c];
        if (c == 0 && (fl & kStatusDensityFloor)) u = 0.0;
        if (c == 4 && (fl & kStatusPressureFloor)) u = 0.0;
        if (c == 0 && (flo & kStatusDensityFloor)) v = 0.0;
        if (c == 4 && (flo & kStatusPressureFloor)) v = 0.0;
        S.lrec[0][7 + c][cl] = u;  // high face of the left cell
        S.lrec[0][c][tc] = v;      // low face of this cell
    }
}

// y and z faces of a linear-reconstruction stage with the reconstruction
// transposed in the same march: a segment computes its faces and the one
// above it (whose cotangent the top cell needs; its normal-field cotangent
// stays with the segment that owns it), and as soon as a cell has the
// cotangents of both its interface states it reverses its reconstruction.
// Bound by FP64 issue and by latency at one wave per SIMD (about 2000 of 3400
// vector instructions per face, 68% of cycles issuing): 128^3 PLMC 308 us per
// axis, 371 with 64-bit index arithmetic (4280); two waves per SIMD would spill
// 950 bytes (1295 us).
constexpr int kAdFusedWaves = 1;

template <int D, int RECON>
__global__ __launch_bounds__(kBlock, kAdFusedWaves) void k_ad_march_fused(
    Geom g, Prims P, StateP st, StateP lout, AdStage S, StateW lacc, const double *dt_dev,
    double factor, int M)
{
    static_assert(D == 1 || D == 2, "columns march along y or z");
    static_assert(RECON == VLCT_RECON_PLMC || RECON == VLCT_RECON_PLMP, "linear reconstructions");
    constexpr int T = D == 1 ? 2 : 1;
    constexpr bool kChar = RECON == VLCT_RECON_PLMC;
    const int nD = g.n[D];
    const u32 cols = (u32)g.n[0] * (u32)g.n[T];
    const u32 ncb = (cols + kBlock - 1) / kBlock;
    const u32 seg = blockIdx.x / ncb;
    const u32 col = (blockIdx.x - seg * ncb) * kBlock + threadIdx.x;
    if (col >= cols) return;
    int x[3];
    x[T] = (int)(col / (u32)g.n[0]);
    x[0] = (int)(col - (u32)x[T] * (u32)g.n[0]);
    x[D] = 0;
    const int s0 = (int)seg * M, s1 = min(s0 + M, nD);  // cells [s0, s1)
    const double c = factor * dt_dev[0] / g.dl[D];
    const u32 tcol = cell_at(g, x[0], x[1], x[2]), tstep = cell_stride<D>(g);
    auto cell = [&](int along) { return tcol + (u32)wrapc(along, nD) * tstep; };
    x[D] = s0 - 2;
    u32 po = prim_at(g, x[0], x[1], x[2]);
    const u32 pstep = D == 1 ? (u32)g.p[0] : (u32)g.p[0] * (u32)g.p[1];
    // What a thread keeps from cell to cell waits in LDS (its own slots), so
    // that the two reversals have the registers to themselves: the face's two
    // states (the low one's cell is a - 1), the high state of cell a, the
    // cotangent of the low state of cell a - 1, the cells a - 2 .. a + 1 of the
    // window (cell c in slot c & 3, with its B_n), and of the reversals (that of
    // cell m adds to the cells m - 1, m and m + 1) the sums of the two cells
    // still waiting for terms (cell c in slot c & 1): a cell leaves with one
    // atomic add per component (segments share the two cells at each end)
    constexpr int kNext = 14, kLow = 21, kPend = 28, kWin = 42;
    __shared__ double park[kWin + 32][kBlock];
    const int tid = threadIdx.x;
    const ParkedStates<kBlock> states{park, tid};
    auto win = [&](int c) { return states.get(kWin + 8 * (c & 3)); };
    auto winb = [&](int c) { return park[kWin + 8 * (c & 3) + 7][tid]; };
    auto load = [&](int c) {
        states.put(kWin + 8 * (c & 3), w7_at(P, D, po));
        park[kWin + 8 * (c & 3) + 7][tid] = P.w[5 + D][po];
        po += pstep;
    };
#pragma unroll
    for (int q = 0; q < 3; ++q) load(s0 - 2 + q);
#pragma unroll
    for (int k = 0; k < 14; ++k) park[kPend + k][tid] = 0.0;
    uint32_t fprev = 0;
    for (int a = s0 - 1; a <= s1; ++a) {
        // the loads of this face and of the window's next cell, ahead of the
        // reconstruction and the reversals
        x[D] = a < 0 ? nD - 1 : (a < nD ? a : 0);
        const u32 t = tcol + (u32)x[D] * tstep;
        const FluxLoads fl = flux_loads<D>(g, lout, S, x, t);
        const u32 fo = face_at<D>(g, x[0], x[1], x[2]);
        const double bn = st.b[D][fo];
        W7 ahead{0, 0, 0, 0, 0, 0, 0};
        double ahead_b = 0.0;
        if (a < s1) {
            ahead = w7_at(P, D, po);
            ahead_b = P.w[5 + D][po];
            po += pstep;
        }
        __builtin_amdgcn_sched_barrier(0);
        uint32_t flo, fhi;
        {
            W7 fm, fp;
            plmc<kChar>(win(a - 1), win(a), win(a + 1), winb(a), g.gamma, fm, fp);
            flo = floor_state(fm);
            fhi = floor_state(fp);
            states.put(7, fm);
            states.put(kNext, fp);
        }
        if (a >= s0) {
            // the face a - 1/2
            double lf[7];
            flux_combine<D>(fl, c, lf);
            W7 aL{0, 0, 0, 0, 0, 0, 0}, aR{0, 0, 0, 0, 0, 0, 0};
            double abn = 0.0;
            hlld_rev(states.get(0), states.get(7), bn, g.gamma, g.gm1i, lf, aL, aR, abn,
                     states);
            if (a < s1) lacc.b[D][fo] = abn;
            double alow[7];
#pragma unroll
            for (int k = 0; k < 7; ++k) alow[k] = park[kLow + k][tid];
            if (flo & kStatusDensityFloor) aR.d = 0.0;
            if (flo & kStatusPressureFloor) aR.p = 0.0;
            states.put(kLow, aR);
            if (a - 1 >= s0) {
                // cell a - 1 has both interface cotangents: reverse its PLM
                double ahigh[7] = {aL.d, aL.u, aL.v, aL.w, aL.p, aL.by, aL.bz};
                if (fprev & kStatusDensityFloor) ahigh[0] = 0.0;
                if (fprev & kStatusPressureFloor) ahigh[4] = 0.0;
                W7 am{0, 0, 0, 0, 0, 0, 0}, a0{0, 0, 0, 0, 0, 0, 0}, ap{0, 0, 0, 0, 0, 0, 0};
                double abc = 0.0;
                asm volatile("" ::: "memory");
                plmc_rev<kChar>(win(a - 2), win(a - 1), win(a), winb(a - 1), g.gamma, alow, ahigh,
                                am, a0, ap, abc);
                const double vm[7] = {am.d, am.u, am.v, am.w, am.p, am.by, am.bz};
                const double v0[7] = {a0.d, a0.u, a0.v, a0.w, a0.p, a0.by, a0.bz};
                const double vp[7] = {ap.d, ap.u, ap.v, ap.w, ap.p, ap.by, ap.bz};
                // slots of cells a - 2 (and a), a - 1
                const int so = kPend + 7 * ((a - 2) & 1), sn = kPend + 7 * ((a - 1) & 1);
                const u32 cm = cell(a - 2);
#pragma unroll
                for (int k = 0; k < 7; ++k) {
                    atomicAdd(&S.lw[lab_slot(D, k)][cm], park[so + k][tid] + vm[k]);
                    park[so + k][tid] = vp[k];
                    park[sn + k][tid] += v0[k];
                }
                atomicAdd(&S.lw[5 + D][cell(a - 1)], abc);
            }
        }
        states.put(0, states.get(kNext));
        fprev = fhi;
        states.put(kWin + 8 * ((a + 2) & 3), ahead);
        park[kWin + 8 * ((a + 2) & 3) + 7][tid] = ahead_b;
    }
    // the cells s1 - 1 and s1 (the last reversal was that of cell s1 - 1)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const u32 cc = cell(s1 - 1 + q);
        const int sl = kPend + 7 * ((s1 - 1 + q) & 1);
#pragma unroll
        for (int k = 0; k < 7; ++k) atomicAdd(&S.lw[lab_slot(D, k)][cc], park[sl + k][tid]);
    }
}

// x faces of a linear-reconstruction stage with the reconstruction transposed
// in the same kernel: items (row, cell) with cells -1 .. nx of every row in
// one flat sequence, blocks of kAdRow items overlapping by two.  Each item
// reconstructs its cell and hands the high-face state to the right through
// LDS; each item with a left neighbour in its block and row takes the face
// between them and hands the left state's cotangent back; each item whose
// faces both lie in the block and which is a cell of the grid then reverses
// its reconstruction.  A face computed twice (the last of a block, the
// periodic image at the end of a row) leaves its normal-field cotangent to
// the item that owns it.
__host__ __device__ __forceinline__ idx_t ad_row_fused_blocks(const Geom &g)
{
    const idx_t items = (idx_t)(g.n[0] + 2) * g.n[1] * g.n[2];
    return (items - 1 + kAdRow - 3) / (kAdRow - 2);  // items 1 .. items-1 at t in [1, kAdRow-2]
}

template <int RECON>
__global__ __launch_bounds__(kAdRow, kAdFusedWaves) void k_ad_row_fused(
    Geom g, Prims P, StateP st, StateP lout, AdStage S, StateW lacc, const double *dt_dev,
    double factor)
{
    static_assert(RECON == VLCT_RECON_PLMC || RECON == VLCT_RECON_PLMP, "linear reconstructions");
    constexpr bool kChar = RECON == VLCT_RECON_PLMC;
    __shared__ double lds[7][kAdRow];
    __shared__ double lds_p[7][kAdRow];
    __shared__ uint32_t lfl[kAdRow];
    __shared__ uint32_t lrev[kAdRow];
    const int nx = g.n[0];
    const u32 per_row = (u32)nx + 2, items = per_row * (u32)g.n[1] * (u32)g.n[2];
    const int t = threadIdx.x;
    const u32 q = blockIdx.x * (u32)(kAdRow - 2) + t;
    const bool have = q < items;
    const u32 row = q / per_row, plane = row / (u32)g.n[1];
    const int i = (int)(q - row * per_row) - 1;  // -1 .. nx
    // the cell, or its periodic image
    const int x[3] = {i < 0 ? nx - 1 : (i < nx ? i : 0), (int)(row - plane * (u32)g.n[1]), (int)plane};
    const u32 po = prim_at(g, i, x[1], x[2]), tc = cell_at(g, x[0], x[1], x[2]);
    auto at = [&](int off) { return po + (u32)off; };
    W7 fm{}, fp{};
    uint32_t flo = 0, fhi = 0;
    if (have) {
        plmc<kChar>(w7_at(P, 0, at(-1)), w7_at(P, 0, at(0)), w7_at(P, 0, at(1)),
                    P.w[5][at(0)], g.gamma, fm, fp);
        flo = floor_state(fm);
        fhi = floor_state(fp);
    }
    lds[0][t] = fp.d; lds[1][t] = fp.u; lds[2][t] = fp.v; lds[3][t] = fp.w;
    lds[4][t] = fp.p; lds[5][t] = fp.by; lds[6][t] = fp.bz;
    lfl[t] = fhi;
    __syncthreads();
    // the face x - 1/2 (x in 0 .. nx), between the item on the left and this one
    const bool face = t >= 1 && have && i >= 0;
    double alow[7] = {0, 0, 0, 0, 0, 0, 0}, ahigh_left[7] = {0, 0, 0, 0, 0, 0, 0};
    if (face) {
        const W7 wl{lds[0][t - 1], lds[1][t - 1], lds[2][t - 1], lds[3][t - 1],
                    lds[4][t - 1], lds[5][t - 1], lds[6][t - 1]};
        const uint32_t fl = lfl[t - 1];
        double lf[7];
        flux_cotangent<0>(g, lout, S, x, tc, factor * dt_dev[0] / g.dl[0], lf);
        const u32 fo = face_at<0>(g, x[0], x[1], x[2]);
        W7 aL{0, 0, 0, 0, 0, 0, 0}, aR{0, 0, 0, 0, 0, 0, 0};
        double abn = 0.0;
        hlld_rev(wl, fm, st.b[0][fo], g.gamma, g.gm1i, lf, aL, aR, abn);
        if (t <= kAdRow - 2 && i < nx) lacc.b[0][fo] = abn;
        const double vl[7] = {aL.d, aL.u, aL.v, aL.w, aL.p, aL.by, aL.bz};
        const double vr[7] = {aR.d, aR.u, aR.v, aR.w, aR.p, aR.by, aR.bz};
#pragma unroll
        for (int c = 0; c < 7; ++c) {
            ahigh_left[c] = vl[c];
            alow[c] = vr[c];
        }
        if (fl & kStatusDensityFloor) ahigh_left[0] = 0.0;
        if (fl & kStatusPressureFloor) ahigh_left[4] = 0.0;
        if (flo & kStatusDensityFloor) alow[0] = 0.0;
        if (flo & kStatusPressureFloor) alow[4] = 0.0;
    }
    __syncthreads();
    // hand the left state's cotangent to the item on the left
#pragma unroll
    for (int c = 0; c < 7; ++c) lds[c][t] = ahigh_left[c];
    __syncthreads();
    const bool rev = face && t <= kAdRow - 2 && i < nx;
    W7 am{0, 0, 0, 0, 0, 0, 0}, a0{0, 0, 0, 0, 0, 0, 0}, ap{0, 0, 0, 0, 0, 0, 0};
    double abc = 0.0;
    if (rev) {
        double ahigh[7];
#pragma unroll
        for (int c = 0; c < 7; ++c) ahigh[c] = lds[c][t + 1];
        plmc_rev<kChar>(w7_at(P, 0, at(-1)), w7_at(P, 0, at(0)), w7_at(P, 0, at(1)),
                        P.w[5][at(0)], g.gamma, alow, ahigh, am, a0, ap, abc);
    }
    __syncthreads();
    // the reversal adds to the cells x - 1, x and x + 1: the neighbours' terms
    // go through LDS to the item that owns the cell where it reversed too, so
    // that each cell leaves with one atomic add per component
    const double vm[7] = {am.d, am.u, am.v, am.w, am.p, am.by, am.bz};
    const double vp[7] = {ap.d, ap.u, ap.v, ap.w, ap.p, ap.by, ap.bz};
#pragma unroll
    for (int c = 0; c < 7; ++c) {
        lds[c][t] = vm[c];
        lds_p[c][t] = vp[c];
    }
    lrev[t] = rev ? 1u : 0u;
    __syncthreads();
    if (!rev) return;
    // an item that reversed on the left (right) is the cell x - 1 (x + 1) of this row
    const bool left_rev = t >= 1 && lrev[t - 1];
    const bool right_rev = lrev[t + 1] != 0u;
    const double v0[7] = {a0.d, a0.u, a0.v, a0.w, a0.p, a0.by, a0.bz};
#pragma unroll
    for (int c = 0; c < 7; ++c) {
        double v = v0[c];
        if (left_rev) v += lds_p[c][t - 1];
        if (right_rev) v += lds[c][t + 1];
        atomicAdd(&S.lw[lab_slot(0, c)][tc], v);
    }
    if (!left_rev) {
        const u32 cl = tc + step_lo<0>(g, x);
#pragma unroll
        for (int c = 0; c < 7; ++c) atomicAdd(&S.lw[lab_slot(0, c)][cl], vm[c]);
    }
    if (!right_rev) {
        const u32 cr = tc + step_hi<0>(g, x);
#pragma unroll
        for (int c = 0; c < 7; ++c) atomicAdd(&S.lw[lab_slot(0, c)][cr], vp[c]);
    }
    atomicAdd(&S.lw[5][tc], abc);
}

// parabolic reconstruction of each cell along x reversed, one thread per cell;
// the cotangents of the five stencil states go to their cells with one atomic
// add per component (neighbours in a row are neighbours in the wave).  Nothing
// passes between threads: an earlier form that handed the terms to the
// neighbours through LDS gave wrong cotangents, with or without -fapprox-func
// by the limiter's kind, for a reason that was not found.  The form with the
// exchange in one-wave blocks passed every check, but nothing showed why the
// other had not.  Bound by FP64 latency at one wave per SIMD (512 registers)
// and by the 36 adds: 64^3 PPMC 110 us and PPMP 95 us (87 and 71 with the
// exchange), 128^3 628 and 691 us (653 and 523).
template <int RECON>
__global__ __launch_bounds__(kAdRow) void k_ad_recon_row(Geom g, Prims P, AdStage S)
{
    static_assert(RECON == VLCT_RECON_PPMC || RECON == VLCT_RECON_PPMP, "parabolic reconstructions");
    constexpr bool kChar = RECON == VLCT_RECON_PPMC;
    __shared__ double win[35][kAdRow];
    const int nx = g.n[0], tid = threadIdx.x;
    const u32 N = (u32)nx * (u32)g.n[1] * (u32)g.n[2];
    const u32 t = blockIdx.x * (u32)kAdRow + tid;
    if (t >= N) return;
    int x[3];
    cell_coords(g, t, x);
    W7 ad[5];
#pragma unroll
    for (int q = 0; q < 5; ++q) ad[q] = W7{0, 0, 0, 0, 0, 0, 0};
    double abn = 0.0, afm[7], afp[7];
#pragma unroll
    for (int c = 0; c < 7; ++c) {
        afm[c] = S.lrec[0][c][t];
        afp[c] = S.lrec[0][7 + c][t];
    }
    // the stencil waits in LDS (each thread its own)
    const u32 o = prim_at(g, x[0], x[1], x[2]);
    const ParkedStates<kAdRow> cells{win, tid};
#pragma unroll
    for (int q = 0; q < 5; ++q) cells.put(7 * q, w7_at(P, 0, o + (u32)(q - 2)));
    ppmc_rev<kChar>(
        [&](int q) {
            asm volatile("" ::: "memory");  // not kept from the first fetch
            return cells.get(7 * q);
        },
        P.w[5][o], g.gamma, afm, afp, ad[0], ad[1], ad[2], ad[3], ad[4], abn);
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        const double v[7] = {ad[q].d, ad[q].u, ad[q].v, ad[q].w, ad[q].p, ad[q].by, ad[q].bz};
        const u32 cc = t - (u32)x[0] + (u32)wrapc(x[0] + q - 2, nx);
#pragma unroll
        for (int c = 0; c < 7; ++c) atomicAdd(&S.lw[lab_slot(0, c)][cc], v[c]);
    }
    atomicAdd(&S.lw[5][t], abn);
}

// Along y and z a thread marches a column segment of M cells and keeps the
// stencil's cells and the four cells still waiting for terms in LDS; a cell
// leaves with one atomic add per component once the reversal two cells above
// it is done (segments share two cells at each end, so every departure stays
// atomic).  The cell's own B_n cotangent comes from its reversal alone and is
// added in place.  64^3 PPMC, segments of 4: 104 -> 84 us with the stencil in
// LDS, fetched again by the last transposes (spills 304 -> 52 bytes).
template <int D, int RECON>
__global__ __launch_bounds__(kBlock) void k_ad_recon_march(Geom g, Prims P, AdStage S, int M)
{
    static_assert(D == 1 || D == 2, "columns march along y or z");
    static_assert(RECON == VLCT_RECON_PPMC || RECON == VLCT_RECON_PPMP, "parabolic reconstructions");
    constexpr int T = D == 1 ? 2 : 1;
    constexpr bool kChar = RECON == VLCT_RECON_PPMC;
    // the stencil's cells (with their B_n) and the cells waiting for terms, cell
    // c in slot c mod 5 (each thread its own column)
    __shared__ double pend[5][7][kBlock], win[40][kBlock];
    const int nD = g.n[D];
    const u32 cols = (u32)g.n[0] * (u32)g.n[T];
    const u32 ncb = (cols + kBlock - 1) / kBlock;
    const u32 seg = blockIdx.x / ncb;
    const u32 col = (blockIdx.x - seg * ncb) * kBlock + threadIdx.x;
    if (col >= cols) return;
    const int tid = threadIdx.x;
    int x[3];
    x[T] = (int)(col / (u32)g.n[0]);
    x[0] = (int)(col - (u32)x[T] * (u32)g.n[0]);
    x[D] = 0;
    const int s0 = (int)seg * M, s1 = min(s0 + M, nD);  // cells [s0, s1)
    const u32 tcol = cell_at(g, x[0], x[1], x[2]), tstep = cell_stride<D>(g);
    x[D] = s0 - 2;
    u32 pb = prim_at(g, x[0], x[1], x[2]);  // cell c - 2
    const u32 pstep = D == 1 ? (u32)g.p[0] : (u32)g.p[0] * (u32)g.p[1];
    auto slot = [](int c) { return (c + 10) % 5; };  // c >= -2
    auto cell = [&](int along) { return tcol + (u32)wrapc(along, nD) * tstep; };
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int k = 0; k < 7; ++k) pend[slot(s0 - 2 + q)][k][tid] = 0.0;
    const ParkedStates<kBlock> cells{win, tid};
    auto load = [&](int c, const W7 &w, double bn) {
        cells.put(8 * slot(c), w);
        win[8 * slot(c) + 7][tid] = bn;
    };
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        load(s0 - 2 + q, w7_at(P, D, pb), P.w[5 + D][pb]);
        pb += pstep;
    }
    for (int c = s0; c < s1; ++c) {
        const u32 t = tcol + (u32)c * tstep;
        double afm[7], afp[7];
#pragma unroll
        for (int k = 0; k < 7; ++k) {
            afm[k] = S.lrec[D][k][t];
            afp[k] = S.lrec[D][7 + k][t];
        }
        W7 ad[5];
#pragma unroll
        for (int q = 0; q < 5; ++q) ad[q] = W7{0, 0, 0, 0, 0, 0, 0};
        double abn = 0.0;
        const int sm = slot(c - 2), s1m = slot(c - 1), s00 = slot(c), s1p = slot(c + 1),
                  s2p = slot(c + 2);
        ppmc_rev<kChar>(
            [&](int q) {
                asm volatile("" ::: "memory");  // not kept from the first fetch
                return cells.get(8 * slot(c - 2 + q));
            },
            win[8 * s00 + 7][tid], g.gamma, afm, afp, ad[0], ad[1], ad[2], ad[3], ad[4], abn);
        double v[5][7];
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            v[q][0] = ad[q].d; v[q][1] = ad[q].u; v[q][2] = ad[q].v; v[q][3] = ad[q].w;
            v[q][4] = ad[q].p; v[q][5] = ad[q].by; v[q][6] = ad[q].bz;
        }
        const u32 cm = cell(c - 2);
#pragma unroll
        for (int k = 0; k < 7; ++k) {
            atomicAdd(&S.lw[lab_slot(D, k)][cm], pend[sm][k][tid] + v[0][k]);
            pend[s1m][k][tid] += v[1][k];
            pend[s00][k][tid] += v[2][k];
            pend[s1p][k][tid] += v[3][k];
            pend[s2p][k][tid] = v[4][k];
        }
        S.lw[5 + D][t] += abn;
        if (c + 1 < s1) {  // in the slot of cell c - 2
            load(c + 3, w7_at(P, D, pb), P.w[5 + D][pb]);
            pb += pstep;
        }
    }
    // the cells s1 - 2 .. s1 + 1 (the last reversal was that of cell s1 - 1)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const u32 cc = cell(s1 - 2 + q);
        const int sl = slot(s1 - 2 + q);
#pragma unroll
        for (int k = 0; k < 7; ++k) atomicAdd(&S.lw[lab_slot(D, k)][cc], pend[sl][k][tid]);
    }
}

// a cell of a reconstructing stage, whose primitive cotangents the
// reconstruction transposes have accumulated
__global__ __launch_bounds__(kBlock) void k_ad_prims(Geom g, StateP st, Prims P, AdStage S,
                                                     AdBase base, StateW lacc)
{
    const u32 N = (u32)g.n[0] * (u32)g.n[1] * (u32)g.n[2];
    const u32 t = blockIdx.x * (u32)kBlock + threadIdx.x;
    if (t >= N) return;
    int x[3];
    cell_coords(g, t, x);
    double lw[8], lb[3];
#pragma unroll
    for (int f = 0; f < 8; ++f) lw[f] = S.lw[f][t];
    cell_rev(g, cell_loads(g, st, P, S, base, x, t), base, lacc, t, lw, lb);
    const u32 f0 = face_at<0>(g, x[0], x[1], x[2]), f1 = face_at<1>(g, x[0], x[1], x[2]);
    atomicAdd(&lacc.b[0][f0], lb[0]);
    atomicAdd(&lacc.b[0][f0 + step_hi<0>(g, x)], lb[0]);
    atomicAdd(&lacc.b[1][f1], lb[1]);
    atomicAdd(&lacc.b[1][f1 + step_hi<1>(g, x)], lb[1]);
    atomicAdd(&lacc.b[2][t], lb[2]);
    atomicAdd(&lacc.b[2][t + step_hi<2>(g, x)], lb[2]);
}

// transposes of one stage: lout is the cotangent of the stage's output state
// (fold: its duplicate faces count for face 0), st/P/sd the stage's input
// state, primitives and upwind sides; lacc becomes the cotangent of the stage's
// input state, on top of `base`.
static void stage_adjoint(const Geom &g, double factor, const StateP &lout, bool fold,
                          const StateP &st, const Prims &P, const Sides &sd, int recon,
                          const AdStage &S, const AdBase &base, const StateW &lacc,
                          const double *dt, hipStream_t s)
{
    const unsigned gc = nblocks((size_t)g.n[0] * g.n[1] * g.n[2]);
    const unsigned gr = (unsigned)(((idx_t)g.n[0] * g.n[1] * g.n[2] + kAdRow - 1) / kAdRow);
    k_ad_edges<<<gc, kBlock, 0, s>>>(g, lout, fold, sd, S, dt, factor, recon != VLCT_RECON_PCM);
    const int slots = kNumCUs;
    const int m1 = ad_march_segment(g, 1, slots), m2 = ad_march_segment(g, 2, slots);
    const unsigned b1 = (unsigned)ad_march_blocks(g, 1, m1), b2 = (unsigned)ad_march_blocks(g, 2, m2);
#define VLCT_AD_FACES(R)                                                                   \
    k_ad_faces_row<R><<<(unsigned)ad_row_blocks(g), kAdRow, 0, s>>>(g, P, st, lout, S,     \
                                                                     lacc, dt, factor);    \
    k_ad_faces_march<1, R><<<b1, kBlock, 0, s>>>(g, P, st, lout, S, lacc, dt, factor, m1); \
    k_ad_faces_march<2, R><<<b2, kBlock, 0, s>>>(g, P, st, lout, S, lacc, dt, factor, m2);
#define VLCT_AD_FUSED(R)                                                                   \
    k_ad_row_fused<R><<<(unsigned)ad_row_fused_blocks(g), kAdRow, 0, s>>>(g, P, st, lout,  \
                                                                           S, lacc, dt,    \
                                                                           factor);        \
    k_ad_march_fused<1, R><<<b1, kBlock, 0, s>>>(g, P, st, lout, S, lacc, dt, factor, m1); \
    k_ad_march_fused<2, R><<<b2, kBlock, 0, s>>>(g, P, st, lout, S, lacc, dt, factor, m2);
#define VLCT_AD_RECON(R)                                                                   \
    k_ad_recon_row<R><<<gr, kAdRow, 0, s>>>(g, P, S);                                      \
    k_ad_recon_march<1, R><<<b1, kBlock, 0, s>>>(g, P, S, m1);                             \
    k_ad_recon_march<2, R><<<b2, kBlock, 0, s>>>(g, P, S, m2);
    if (recon == VLCT_RECON_PCM) {
        k_ad_pcm_row<<<(unsigned)ad_pcm_row_blocks(g), kBlock, 0, s>>>(g, P, st, lout, S, base,
                                                                       lacc, dt, factor);
        k_ad_pcm_march<1><<<b1, kBlock, 0, s>>>(g, P, st, lout, S, base, lacc, dt, factor, m1);
        k_ad_pcm_march<2><<<b2, kBlock, 0, s>>>(g, P, st, lout, S, base, lacc, dt, factor, m2);
    } else if (recon == VLCT_RECON_PLMC) {
        VLCT_AD_FUSED(VLCT_RECON_PLMC)
    } else if (recon == VLCT_RECON_PLMP) {
        VLCT_AD_FUSED(VLCT_RECON_PLMP)
    } else if (recon == VLCT_RECON_PPMC) {
        VLCT_AD_FACES(VLCT_RECON_PPMC)
        VLCT_AD_RECON(VLCT_RECON_PPMC)
    } else {
        VLCT_AD_FACES(VLCT_RECON_PPMP)
        VLCT_AD_RECON(VLCT_RECON_PPMP)
    }
#undef VLCT_AD_FACES
#undef VLCT_AD_FUSED
#undef VLCT_AD_RECON
    if (recon != VLCT_RECON_PCM) k_ad_prims<<<gc, kBlock, 0, s>>>(g, st, P, S, base, lacc);
}

// workspace of the adjoint: forward intermediates and cotangents.  Without a
// tape it also holds the recomputed fluxes, half-step state and upwind sides.
struct AdLayout {
    size_t prims[2], half[8], flux[3], side[2][3], le, wcode, lw, lrec, total;
    size_t prims_len, flux_len[3], cell_pitch;
    size_t lnext[8], lhalf[8];
};

static AdLayout ad_layout(const Geom &g, bool taped)
{
    AdLayout L;
    size_t off = 0;
    const size_t N = (size_t)g.n[0] * g.n[1] * g.n[2];
    L.cell_pitch = align_up(N * 8);
    L.prims_len = (size_t)g.p[0] * g.p[1] * g.p[2];
    for (int h = 0; h < 2; ++h) {
        L.prims[h] = off;
        off += 8 * align_up(L.prims_len * 8);
    }
    for (int d = 0; d < 3; ++d)
        L.flux_len[d] = (size_t)flux_dim(g.n, d, 0) * flux_dim(g.n, d, 1) * flux_dim(g.n, d, 2);
    if (!taped) {
        for (int f = 0; f < 8; ++f) {
            L.half[f] = off;
            off += align_up(field_len(g.n, f) * 8);
        }
        for (int d = 0; d < 3; ++d) {
            L.flux[d] = off;
            off += flux_axis_bytes(L.flux_len[d]);
        }
        for (int h = 0; h < 2; ++h)
            for (int d = 0; d < 3; ++d) {
                L.side[h][d] = off;
                off += align_up(N);
            }
    }
    for (int f = 0; f < 8; ++f) {
        L.lnext[f] = off;
        off += align_up(field_len(g.n, f) * 8);
    }
    for (int f = 0; f < 8; ++f) {
        L.lhalf[f] = off;
        off += align_up(field_len(g.n, f) * 8);
    }
    L.le = off;
    off += 3 * L.cell_pitch;
    L.wcode = off;
    off += align_up(N * sizeof(uint32_t));
    L.lw = off;
    off += 8 * L.cell_pitch;
    L.lrec = off;
    off += 42 * L.cell_pitch;
    L.total = off;
    return L;
}

// argument checks shared by both adjoint entry points
static int adjoint_args(const vlct_grid *vg, const vlct_state *in, const vlct_state *lam_out,
                        const vlct_state *lam_in, const double *dt_dev)
{
    if (!grid_ok(vg) || !state_ok(in) || !state_ok(lam_out) || !state_ok(lam_in) || !dt_dev)
        return VLCT_EINVAL;
    for (int d = 0; d < 3; ++d)
        if (vg->bc[d] != VLCT_BC_PERIODIC) return VLCT_EUNSUPPORTED;
    // no array of lam_in may overlap an array of `in` or `lam_out`, nor another of lam_in
    const int n[3] = {vg->nx, vg->ny, vg->nz};
    const vlct_state *sts[3] = {lam_in, in, lam_out};
    uintptr_t lo[3][8], hi[3][8];
    for (int q = 0; q < 3; ++q) {
        const double *p[8] = {sts[q]->rho, sts[q]->mx, sts[q]->my, sts[q]->mz, sts[q]->E,
                              sts[q]->bx, sts[q]->by, sts[q]->bz};
        for (int f = 0; f < 8; ++f) {
            lo[q][f] = reinterpret_cast<uintptr_t>(p[f]);
            hi[q][f] = lo[q][f] + field_len(n, f) * sizeof(double);
        }
    }
    for (int f = 0; f < 8; ++f)
        for (int q = 0; q < 3; ++q)
            for (int h = 0; h < 8; ++h) {
                if (q == 0 && h == f) continue;
                if (lo[0][f] < hi[q][h] && lo[q][h] < hi[0][f]) return VLCT_EINVAL;
            }
    return VLCT_OK;
}

// the adjoint of one step given the half-step state and both stages' upwind
// sides (from a tape, or recomputed into the workspace by the caller, who
// then has also computed both stages' primitives: have_prims)
static int adjoint_core(const vlct_grid *vg, const Geom &g, const AdLayout &L, char *b,
                        const StateP &sin, const StateP &hc, const Sides sides[2],
                        bool have_prims, const vlct_state *lam_out, const vlct_state *lam_in,
                        const double *dt_dev, hipStream_t s)
{
    auto arr = [&](size_t off) { return reinterpret_cast<double *>(b + off); };
    Prims P[2];
    for (int h = 0; h < 2; ++h)
        for (int f = 0; f < 8; ++f) P[h].w[f] = arr(L.prims[h] + f * align_up(L.prims_len * 8));
    StateW lhalf;
    for (int f = 0; f < 8; ++f) {
        double *e = arr(L.lhalf[f]);
        if (f < 5) lhalf.u[f] = e; else lhalf.b[f - 5] = e;
    }
    AdStage S;
    for (int a = 0; a < 3; ++a) S.le[a] = arr(L.le + a * L.cell_pitch);
    S.wcode = reinterpret_cast<uint32_t *>(b + L.wcode);
    for (int f = 0; f < 8; ++f) S.lw[f] = arr(L.lw + f * L.cell_pitch);
    for (int d = 0; d < 3; ++d)
        for (int c = 0; c < 14; ++c) S.lrec[d][c] = arr(L.lrec + (14 * d + c) * L.cell_pitch);

    // primitives of both stages' input states (same kernel as the step)
    if (!have_prims) {
        int rc = launch_prims(g, sin, P[0], nullptr, s);
        if (!rc) rc = launch_prims(g, hc, P[1], nullptr, s);
        if (rc) return rc;
    }

    // reverse: corrector stage into mu = lhalf, then lam_in = lam_out (U^{n+1}
    // contains U^n with unit weight) + mu + predictor^T mu
    const StateP lam = as_const(lam_out), mu = as_const(lhalf);
    stage_adjoint(g, 1.0, lam, true, hc, P[1], sides[1], vg->recon, S, AdBase{lam, mu, 0}, lhalf,
                  dt_dev, s);
    stage_adjoint(g, 0.5, mu, false, sin, P[0], sides[0], VLCT_RECON_PCM, S, AdBase{lam, mu, 1},
                  as_mut(lam_in), dt_dev, s);
    return hipGetLastError() == hipSuccess ? VLCT_OK : VLCT_EHIP;
}

// ---------------------------------------------------------------------------
// face fields from an edge-centred vector potential, B = curl_h A (periodic),
// and the transpose of that map.  A_x at (i, j-1/2, k-1/2), A_y at
// (i-1/2, j, k-1/2), A_z at (i-1/2, j-1/2, k), each stored like a cell array.
// ---------------------------------------------------------------------------
// (64-bit indices: unlike the adjoint's, these arrays alone may hold 2^32 cells)
__device__ __forceinline__ idx_t cell_of(const Geom &g, int i, int j, int k)
{
    return cell_store(g, wrapc(i, g.n[0]), wrapc(j, g.n[1]), wrapc(k, g.n[2]));
}
__device__ __forceinline__ void cell_coords(const Geom &g, idx_t t, int x[3])
{
    x[0] = (int)(t % g.n[0]);
    x[1] = (int)((t / g.n[0]) % g.n[1]);
    x[2] = (int)(t / ((idx_t)g.n[0] * g.n[1]));
}

__global__ void k_curl_potential(Geom g, const double *ax, const double *ay, const double *az,
                                 double *bx, double *by, double *bz)
{
    const idx_t N = (idx_t)g.n[0] * g.n[1] * g.n[2];
    const idx_t t = (idx_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= N) return;
    int x[3];
    cell_coords(g, t, x);
    const int i = x[0], j = x[1], k = x[2];
    const idx_t ip = cell_of(g, i + 1, j, k), jp = cell_of(g, i, j + 1, k),
                kp = cell_of(g, i, j, k + 1);
    const double vx = (az[jp] - az[t]) / g.dl[1] - (ay[kp] - ay[t]) / g.dl[2];
    const double vy = (ax[kp] - ax[t]) / g.dl[2] - (az[ip] - az[t]) / g.dl[0];
    const double vz = (ay[ip] - ay[t]) / g.dl[0] - (ax[jp] - ax[t]) / g.dl[1];
    bx[face_store(g, 0, i, j, k)] = vx;
    by[face_store(g, 1, i, j, k)] = vy;
    bz[face_store(g, 2, i, j, k)] = vz;
    // the duplicate periodic face planes
    if (i == 0) bx[face_store(g, 0, g.n[0], j, k)] = vx;
    if (j == 0) by[face_store(g, 1, i, g.n[1], k)] = vy;
    if (k == 0) bz[face_store(g, 2, i, j, g.n[2])] = vz;
}

__global__ void k_curl_potential_adjoint(Geom g, const double *lbx, const double *lby,
                                         const double *lbz, double *lax, double *lay, double *laz)
{
    const idx_t N = (idx_t)g.n[0] * g.n[1] * g.n[2];
    const idx_t t = (idx_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= N) return;
    int x[3];
    cell_coords(g, t, x);
    const int i = x[0], j = x[1], k = x[2];
    // cotangent of face (d; a, b, c) with the duplicate plane's folded onto plane 0
    auto lb = [&](int d, const double *p, int a, int b2, int c2) {
        const int q[3] = {wrapc(a, g.n[0]), wrapc(b2, g.n[1]), wrapc(c2, g.n[2])};
        double v = p[face_store(g, d, q[0], q[1], q[2])];
        if (q[d] == 0) {
            int r[3] = {q[0], q[1], q[2]};
            r[d] = g.n[d];
            v += p[face_store(g, d, r[0], r[1], r[2])];
        }
        return v;
    };
    lax[t] = (lb(1, lby, i, j, k - 1) - lb(1, lby, i, j, k)) / g.dl[2]
             + (lb(2, lbz, i, j, k) - lb(2, lbz, i, j - 1, k)) / g.dl[1];
    lay[t] = (lb(0, lbx, i, j, k) - lb(0, lbx, i, j, k - 1)) / g.dl[2]
             + (lb(2, lbz, i - 1, j, k) - lb(2, lbz, i, j, k)) / g.dl[0];
    laz[t] = (lb(0, lbx, i, j - 1, k) - lb(0, lbx, i, j, k)) / g.dl[1]
             + (lb(1, lby, i, j, k) - lb(1, lby, i - 1, j, k)) / g.dl[0];
}

}  // namespace vlct

using namespace vlct;

extern "C" {

static bool periodic_grid(const vlct_grid *g)
{
    return grid_ok(g) && g->bc[0] == VLCT_BC_PERIODIC && g->bc[1] == VLCT_BC_PERIODIC &&
           g->bc[2] == VLCT_BC_PERIODIC;
}

int vlct_curl_potential(const vlct_grid *vg, const double *ax, const double *ay, const double *az,
                        double *bx, double *by, double *bz, void *stream)
{
    if (!grid_ok(vg) || !ax || !ay || !az || !bx || !by || !bz) return VLCT_EINVAL;
    if (!periodic_grid(vg)) return VLCT_EUNSUPPORTED;
    const Geom g = grid_geom(vg);
    const size_t N = (size_t)g.n[0] * g.n[1] * g.n[2];
    k_curl_potential<<<nblocks(N), kBlock, 0, static_cast<hipStream_t>(stream)>>>(g, ax, ay, az,
                                                                                 bx, by, bz);
    return hipGetLastError() == hipSuccess ? VLCT_OK : VLCT_EHIP;
}

int vlct_curl_potential_adjoint(const vlct_grid *vg, const double *lbx, const double *lby,
                                const double *lbz, double *lax, double *lay, double *laz,
                                void *stream)
{
    if (!grid_ok(vg) || !lbx || !lby || !lbz || !lax || !lay || !laz) return VLCT_EINVAL;
    if (!periodic_grid(vg)) return VLCT_EUNSUPPORTED;
    const Geom g = grid_geom(vg);
    const size_t N = (size_t)g.n[0] * g.n[1] * g.n[2];
    k_curl_potential_adjoint<<<nblocks(N), kBlock, 0, static_cast<hipStream_t>(stream)>>>(
        g, lbx, lby, lbz, lax, lay, laz);
    return hipGetLastError() == hipSuccess ? VLCT_OK : VLCT_EHIP;
}

size_t vlct_adjoint_workspace_bytes(const vlct_grid *g)
{
    if (!grid_ok(g)) return 0;
    return ad_layout(grid_geom(g), false).total;
}

size_t vlct_adjoint_taped_workspace_bytes(const vlct_grid *g)
{
    if (!grid_ok(g)) return 0;
    return ad_layout(grid_geom(g), true).total;
}

int vlct_step_adjoint(const vlct_grid *vg, const vlct_state *in, const vlct_state *lam_out,
                      const vlct_state *lam_in, const double *dt_dev, void *ws, size_t ws_bytes,
                      void *stream)
{
    int rc = adjoint_args(vg, in, lam_out, lam_in, dt_dev);
    if (rc) return rc;
    const Geom g = make_geom(vg);
    const AdLayout L = ad_layout(g, false);
    if (!ws || ws_bytes < L.total) return VLCT_EWORKSPACE;
    char *b = static_cast<char *>(ws);
    hipStream_t s = static_cast<hipStream_t>(stream);
    auto arr = [&](size_t off) { return reinterpret_cast<double *>(b + off); };
    Prims P[2];
    for (int h = 0; h < 2; ++h)
        for (int f = 0; f < 8; ++f) P[h].w[f] = arr(L.prims[h] + f * align_up(L.prims_len * 8));
    StateW half;
    for (int f = 0; f < 8; ++f) {
        if (f < 5) half.u[f] = arr(L.half[f]); else half.b[f - 5] = arr(L.half[f]);
    }
    const Flux F = bind_flux(b, L.flux, L.flux_len);
    uint8_t *side[2][3];
    Sides sides[2];
    for (int h = 0; h < 2; ++h)
        for (int d = 0; d < 3; ++d) {
            side[h][d] = reinterpret_cast<uint8_t *>(b + L.side[h][d]);
            sides[h].s[d] = side[h][d];
        }
    // forward intermediates at U^n (the kernels of vlct_step); the cells that
    // the corrector fluxes update go to an array that nothing reads
    StateW unused;
    for (int f = 0; f < 8; ++f) {
        if (f < 5) unused.u[f] = arr(L.lnext[f]); else unused.b[f - 5] = arr(L.lnext[f]);
    }
    const StateP sin = as_const(in);
    rc = launch_prims(g, sin, P[0], nullptr, s);
    if (!rc) rc = launch_pred(g, sin, half, P[1], dt_dev, nullptr, side[0], s);
    const StateP hc = as_const(half);
    if (!rc) rc = launch_fluxes(g, hc, P[1], F, vg->recon, sin, unused, dt_dev, nullptr, s);
    if (!rc) rc = launch_pack_sides(g, F, side[1], s);
    if (rc) return rc;
    return adjoint_core(vg, g, L, b, sin, hc, sides, true, lam_out, lam_in, dt_dev, s);
}

int vlct_step_adjoint_taped(const vlct_grid *vg, const vlct_state *in, const vlct_state *lam_out,
                            const vlct_state *lam_in, const double *dt_dev, const void *tape,
                            size_t tape_bytes, void *ws, size_t ws_bytes, void *stream)
{
    int rc = adjoint_args(vg, in, lam_out, lam_in, dt_dev);
    if (rc) return rc;
    const Geom g = grid_geom(vg);
    const AdLayout L = ad_layout(g, true);
    const TapeLayout T = tape_layout(g.n);
    if (!ws || ws_bytes < L.total || !tape || tape_bytes < T.total) return VLCT_EWORKSPACE;
    const char *tb = static_cast<const char *>(tape);
    StateP hc;
    for (int f = 0; f < 8; ++f) {
        const double *a = reinterpret_cast<const double *>(tb + T.half[f]);
        if (f < 5) hc.u[f] = a; else hc.b[f - 5] = a;
    }
    Sides sides[2];
    for (int h = 0; h < 2; ++h)
        for (int d = 0; d < 3; ++d) sides[h].s[d] = reinterpret_cast<const uint8_t *>(tb + T.side[h][d]);
    return adjoint_core(vg, g, L, static_cast<char *>(ws), as_const(in), hc, sides, false,
                        lam_out, lam_in, dt_dev, static_cast<hipStream_t>(stream));
}

}  // extern "C"
