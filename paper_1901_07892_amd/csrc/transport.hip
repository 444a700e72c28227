// Face-density transport of the conservative scheme: the three-stage SSP-RK3
// update of the face densities (Sec. 4.2.2, eqs. eq_rk1, eq_rk2, eq_rk3),
//     rho1 = rho_n - dt R(u1, rho_n)
//     rho2 = 3/4 rho_n + 1/4 rho1 - 1/4 dt R(u2, rho1)
//     rho  = 1/3 rho_n + 2/3 rho2 - 2/3 dt R(u3, rho2),
// whose result is the face density that stokes_setup takes.  R(u, rho) is the
// divergence of u_adv rho_lim over the control volume of each face (one cell
// long in every direction, centred on the face):
//   - u_adv on a control-volume face normal to d is the mean of the two nearest
//     d-velocities (along the face's own axis the two faces around the cell
//     centre; across it the d-faces of the cells on either side of the edge);
//     wall-normal velocities are zero, so nothing crosses a wall;
//   - rho_lim is the CUI-limited cubic upwind value (Waterson and Deconinck
//     2007) from the far-upwind, upwind and downwind densities U, C, D along d:
//     r = (C - U)/(D - U), f = 3r on (0, 2/13], 5r/6 + 1/3 on (2/13, 4/5],
//     1 on (4/5, 1), r otherwise; rho_lim = U + f (D - U), or C when D = U;
//   - densities beyond a wall mirror the interior (homogeneous Neumann);
//   - wall-normal faces are not transported and hold rho_n in every stage.
//
// GPU mapping: one launch per stage in the caller's C-order layouts: a z-marching kernel
// that advances the three faces of each cell together (k_rk3_stage3) on large 3D grids, one
// thread per face otherwise (2D grids that fill them in tiles, k_rk3_stage2, else in rows,
// k_rk3_stage).  Every control-volume face flux is the same expression for both faces that
// share it, so the update is exactly conservative in the same sense as its definition.
#include "../../include/stokes.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace {

constexpr int kTrX = 64, kTrY = 4;           // cells (2D: faces) per block
// 3D grids march from 3 * 2^17 cells on where their tiles are at least 5/8 full (us per update,
// marching against a thread per face): 96^3 89 / 107, 128x128x24 48 / 52, 300x40x40 58 / 75,
// 24x200x200 (3/4 full) 111 / 119; but 64^3 41 / 35, 70^3 56 / 52, 65x65x1000 (0.61 full)
// 590 / 536, 16x300x300 (half full) 226 / 174, 2x2x500000 5900 / 310.
constexpr double kTrMarch = 393216, kTrMarchFill = 0.625;
// 2D grids take tiles that are at least 3/4 full (tiles against rows): 1500^2 112 / 159,
// 100000x8 46 / 63; but 33x20000 (half full) 63 / 41, 8x100000 253 / 46.
constexpr double kTrTileFill = 0.75;
constexpr int kTrBlocks = 4096;              // blocks that a marching launch aims at

struct TrGrid {
    int dim;
    int n[3];
    double ih[3];
};

struct StageArgs {
    double a_n, a_s, c_dt;                   // out = a_n rho_n + a_s rho_s - c_dt R(u, rho_s)
    const double *rn[3], *rs[3], *u[3];
    double *out[3];
};

// Flux a rho_lim through a control-volume face with the densities r0 .. r3 around it
// (r1 | r2 next to it): rho_lim is the CUI-limited value from far-upwind U, upwind C and
// downwind D.  With N = C - U and A = D - U (r = N/A), f(r) A is N outside 0 < r < 1 and
// inside it the least in magnitude of 3 N, 5/6 N + A/3 and A, since f is concave there;
// so the limiter is two minima of magnitudes and needs no division and no branch (the
// upwind side and the branch differ from lane to lane).
// Where a comparison of r is undefined (a NaN, an infinity) the value is C where A = 0 (a
// NaN of C stays one) or where a NaN of A leaves N >= 0, else D, as the chain of branches
// gives it: N's sign is selected by A > 0, the last minimum is a selection of D.
__device__ inline double cui_flux(double a, double r0, double r1, double r2, double r3) {
    const bool up = a > 0.0;
    const double U = up ? r0 : r3, C = up ? r1 : r2, D = up ? r2 : r1;
    const double A = D - U, N = C - U, An = fabs(A);
    const double Nn = A > 0.0 ? N : -N;                   // N sign(A)
    const double w = fmin(3.0 * Nn, __builtin_fma(5.0 / 6.0, Nn, An * (1.0 / 3.0)));
    const double v = w < An ? U + copysign(w, A) : D;
    return a * (Nn <= 0.0 || Nn >= An || A == 0.0 ? C : v);          // r <= 0, r >= 1 or D = U: upwind
}

// Index of entry m along an axis (mirrored beyond a wall: about the wall face along the
// component's own axis, about the wall across it) for an array of extent E >= 2,
// -2 <= m <= E + 1.
template <bool FACE>
__device__ inline int mirror(int m, int E) {
    if (FACE) {
        m = abs(m);
        return E - 1 - abs(E - 1 - m);
    }
    m ^= m >> 31;                                // -1 - m where negative
    const int q = E - 1 - m;
    return E - 1 - (q ^ (q >> 31));
}

// One face (i, j, k) of component C, neighbours from cache
template <int DIM, int C>
__device__ inline void stage_face(const TrGrid &g, const StageArgs &s, int i, int j, int k) {
    const int p[3] = {i, j, k};
    const int E[3] = {g.n[0] + (C == 0), g.n[1] + (C == 1), DIM == 3 ? g.n[2] + (C == 2) : 1};
    if (i >= E[0] || j >= E[1] || k >= E[2]) return;
    const int st[3] = {1, E[0], E[0] * E[1]};
    const int t = i + st[1] * j + st[2] * k;
    const double rn = s.rn[C][t];
    if (p[C] == 0 || p[C] == g.n[C]) {                  // wall-normal face: not transported
        s.out[C][t] = rn;
        return;
    }
    const double *rc = s.rs[C];
    const double r2 = rc[t];
    double R = 0.0;
    auto axis = [&](auto axis_) {
        constexpr int d = decltype(axis_)::value;
        constexpr bool fa = d == C;
        const int m = p[d], base = t - m * st[d];
        // densities at m-2 .. m+2 along d
        const double r0 = rc[base + mirror<fa>(m - 2, E[d]) * st[d]], r1 = rc[base + mirror<fa>(m - 1, E[d]) * st[d]];
        const double r3 = rc[base + mirror<fa>(m + 1, E[d]) * st[d]], r4 = rc[base + mirror<fa>(m + 2, E[d]) * st[d]];
        // advective velocities on the control-volume faces m (lower) and m+1 (upper)
        double alo, ahi;
        const double *ud = s.u[d];
        if constexpr (fa) {
            // c-faces around the cell centres m-1 | m and m | m+1 (interior faces have both)
            const double uc = ud[t];
            alo = 0.5 * (ud[t - st[d]] + uc);
            ahi = 0.5 * (uc + ud[t + st[d]]);
        } else {
            // d-faces of the cells p[C]-1 and p[C] at edge index m and m+1 along d
            const int e0 = g.n[0] + (d == 0), e1 = g.n[1] + (d == 1);
            const int sd[3] = {1, e0, e0 * e1};
            const int q = i + sd[1] * j + sd[2] * k, qm = q - sd[C];
            alo = 0.5 * (ud[qm] + ud[q]);
            ahi = 0.5 * (ud[qm + sd[d]] + ud[q + sd[d]]);
        }
        R += (cui_flux(ahi, r1, r2, r3, r4) - cui_flux(alo, r0, r1, r2, r3)) * g.ih[d];
    };
    axis(std::integral_constant<int, 0>{});
    axis(std::integral_constant<int, 1>{});
    if constexpr (DIM == 3) axis(std::integral_constant<int, 2>{});
    s.out[C][t] = s.a_n * rn + s.a_s * r2 - s.c_dt * R;
}

// One thread per face, the faces of a component (blockIdx.y) numbered in a row: every thread
// has work whatever the grid's proportions.
template <int DIM>
__global__ void __launch_bounds__(kTrX *kTrY) k_rk3_stage(TrGrid g, StageArgs s) {
    const unsigned t = blockIdx.x * (kTrX * kTrY) + threadIdx.x;
    const unsigned E0 = g.n[0] + (blockIdx.y == 0), E1 = g.n[1] + (blockIdx.y == 1);
    const unsigned row = t / E0, k = row / E1;
    const int i = (int)(t - row * E0), j = (int)(row - k * E1);
    if (blockIdx.y == 0) stage_face<DIM, 0>(g, s, i, j, (int)k);
    else if (blockIdx.y == 1) stage_face<DIM, 1>(g, s, i, j, (int)k);
    else if constexpr (DIM == 3) stage_face<DIM, 2>(g, s, i, j, (int)k);
}

// 2D in tiles of 64 x 4 faces, x fastest, a block taking every gridDim.x-th tile: the rows
// above and below a face are read by the same block.
__global__ void __launch_bounds__(kTrX *kTrY) k_rk3_stage2(TrGrid g, StageArgs s, int gx, unsigned tiles) {
    for (unsigned t = blockIdx.x; t < tiles; t += gridDim.x) {
        const int i = (int)(t % gx) * kTrX + threadIdx.x, j = (int)(t / gx) * kTrY + threadIdx.y;
        if (blockIdx.y == 0) stage_face<2, 0>(g, s, i, j, 0);
        else stage_face<2, 1>(g, s, i, j, 0);
    }
}

// 3D, marching in z: a thread owns the cell column (i, j) over a chunk of kc planes and
// advances the cell's x-face i, y-face j and z-face k together.  Each component's
// densities at k-2 .. k+2 slide through registers, and so do the velocities of the plane
// below and the flux through the control-volume face below (the upper flux of one plane
// is the lower one of the next); x- and y-neighbours are other threads' columns, from
// cache.  So a face costs 5 limited values instead of 6 and about 14 loads instead of 30,
// and of the 12 arrays that a stage has to move (density, velocity, rho_n, result) each
// plane comes from memory once: one thread per face of one component re-read the planes
// k-2 .. k+2 of a density from beyond L2 (its five planes of every array in flight exceed
// an XCD's 4 MB) and was bound by that: 968 us per stage at 256^3, now 545 (3.0 TB/s of
// those 12 arrays).  166 registers, three wavefronts per SIMD; at 128 it spills (940 us).
// What is left is about equal parts of vector instructions (0.3 ms) and cache accesses.
// The wall faces i = Nx, j = Ny, k = Nz hold rho_n and are written by the last cells.
template <int TX>
__global__ void __launch_bounds__(kTrX *kTrY) k_rk3_stage3(TrGrid g, StageArgs s, int gx, int gy, int kc) {
    // tiles in x, y, then chunks; each XCD takes a contiguous range
    const unsigned G = gridDim.x, b = blockIdx.x, per = G >> 3, rest = G & 7, xcd = b & 7, loc = b >> 3;
    const unsigned t = xcd < rest ? xcd * (per + 1) + loc : rest * (per + 1) + (xcd - rest) * per + loc;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    const int i = (int)(t % gx) * TX + threadIdx.x, j = (int)(t / gx % gy) * (kTrX * kTrY / TX) + threadIdx.y;
    const int k0 = (int)(t / gx / gy) * kc, k1 = min(k0 + kc, nz);
    if (i >= nx || j >= ny) return;
    // row and plane strides of the three face arrays
    const int sy0 = nx + 1, sy1 = nx, sy2 = nx;
    const int sz0 = sy0 * ny, sz1 = sy1 * (ny + 1), sz2 = sy2 * ny;
    // mirrored neighbours at -2, -1, +1, +2 (as offsets), across the own axis and along it
    const int xf0 = mirror<true>(i - 2, nx + 1) - i, xf1 = mirror<true>(i - 1, nx + 1) - i;
    const int xf3 = mirror<true>(i + 1, nx + 1) - i, xf4 = mirror<true>(i + 2, nx + 1) - i;
    const int xc0 = mirror<false>(i - 2, nx) - i, xc1 = mirror<false>(i - 1, nx) - i;
    const int xc3 = mirror<false>(i + 1, nx) - i, xc4 = mirror<false>(i + 2, nx) - i;
    const int yf0 = mirror<true>(j - 2, ny + 1) - j, yf1 = mirror<true>(j - 1, ny + 1) - j;
    const int yf3 = mirror<true>(j + 1, ny + 1) - j, yf4 = mirror<true>(j + 2, ny + 1) - j;
    const int yc0 = mirror<false>(j - 2, ny) - j, yc1 = mirror<false>(j - 1, ny) - j;
    const int yc3 = mirror<false>(j + 1, ny) - j, yc4 = mirror<false>(j + 2, ny) - j;
    const int im = i > 0 ? 1 : 0, jm = j > 0 ? 1 : 0;    // the cells west and south (wall faces do not use them)
    const double *u = s.u[0], *v = s.u[1], *w = s.u[2];
    const int c0 = i + sy0 * j, c1 = i + sy1 * j, c2 = i + sy2 * j;     // the column in each array
    const bool same = s.rn[0] == s.rs[0];                // the first stage: rho_n is the stage density
    // densities at k-2 .. k+2
    auto col = [&](const double *r, int c, int sz, int k, auto face) {
        constexpr bool f = decltype(face)::value;
        return r[c + sz * mirror<f>(k, f ? nz + 1 : nz)];
    };
    using F = std::true_type;
    using N = std::false_type;
    double a0 = col(s.rs[0], c0, sz0, k0 - 2, N{}), a1 = col(s.rs[0], c0, sz0, k0 - 1, N{}), a2 = col(s.rs[0], c0, sz0, k0, N{}), a3 = col(s.rs[0], c0, sz0, k0 + 1, N{});
    double b0 = col(s.rs[1], c1, sz1, k0 - 2, N{}), b1 = col(s.rs[1], c1, sz1, k0 - 1, N{}), b2 = col(s.rs[1], c1, sz1, k0, N{}), b3 = col(s.rs[1], c1, sz1, k0 + 1, N{});
    double d0 = col(s.rs[2], c2, sz2, k0 - 2, F{}), d1 = col(s.rs[2], c2, sz2, k0 - 1, F{}), d2 = col(s.rs[2], c2, sz2, k0, F{}), d3 = col(s.rs[2], c2, sz2, k0 + 1, F{});
    // velocities of the plane below and the lower fluxes of plane k0
    const int km = max(k0 - 1, 0);
    double u_lo = u[c0 + sz0 * km], ue_lo = u[c0 + 1 + sz0 * km];
    double v_lo = v[c1 + sz1 * km], vn_lo = v[c1 + sy1 + sz1 * km];
    double w0 = w[c2 + sz2 * k0], ww0 = w[c2 - im + sz2 * k0], ws0 = w[c2 - jm * sy2 + sz2 * k0];
    double fa = cui_flux(0.5 * (ww0 + w0), a0, a1, a2, a3);
    double fb = cui_flux(0.5 * (ws0 + w0), b0, b1, b2, b3);
    double fd = cui_flux(0.5 * (w[c2 + sz2 * km] + w0), d0, d1, d2, d3);
    const double ihx = g.ih[0], ihy = g.ih[1], ihz = g.ih[2];
    for (int k = k0; k < k1; ++k) {
        const int q0 = c0 + sz0 * k, q1 = c1 + sz1 * k, q2 = c2 + sz2 * k;
        const double a4 = col(s.rs[0], c0, sz0, k + 2, N{}), b4 = col(s.rs[1], c1, sz1, k + 2, N{}), d4 = col(s.rs[2], c2, sz2, k + 2, F{});
        const double w1 = w[q2 + sz2], ww1 = w[q2 + sz2 - im], ws1 = w[q2 + sz2 - jm * sy2];
        const double uc = u[q0], uw = u[q0 - im], ue = u[q0 + 1], us = u[q0 - jm * sy0], ues = u[q0 + 1 - jm * sy0];
        const double vc = v[q1], vs = v[q1 - jm * sy1], vn = v[q1 + sy1], vw = v[q1 - im], vnw = v[q1 + sy1 - im];
        const double *ra = s.rs[0] + q0, *rb = s.rs[1] + q1, *rd = s.rs[2] + q2;
        const double na = same ? a2 : s.rn[0][q0], nb = same ? b2 : s.rn[1][q1], nd = same ? d2 : s.rn[2][q2];
        // x-face i
        {
            const double x0 = ra[xf0], x1 = ra[xf1], x3 = ra[xf3], x4 = ra[xf4];
            const double y0 = ra[yc0 * sy0], y1 = ra[yc1 * sy0], y3 = ra[yc3 * sy0], y4 = ra[yc4 * sy0];
            const double hi = cui_flux(0.5 * (ww1 + w1), a1, a2, a3, a4);
            double R = (cui_flux(0.5 * (uc + ue), x1, a2, x3, x4) - cui_flux(0.5 * (uw + uc), x0, x1, a2, x3)) * ihx;
            R += (cui_flux(0.5 * (vnw + vn), y1, a2, y3, y4) - cui_flux(0.5 * (vw + vc), y0, y1, a2, y3)) * ihy;
            R += (hi - fa) * ihz;
            fa = hi;
            s.out[0][q0] = i == 0 ? na : s.a_n * na + s.a_s * a2 - s.c_dt * R;
            if (i == nx - 1) s.out[0][q0 + 1] = s.rn[0][q0 + 1];
        }
        // y-face j
        {
            const double x0 = rb[xc0], x1 = rb[xc1], x3 = rb[xc3], x4 = rb[xc4];
            const double y0 = rb[yf0 * sy1], y1 = rb[yf1 * sy1], y3 = rb[yf3 * sy1], y4 = rb[yf4 * sy1];
            const double hi = cui_flux(0.5 * (ws1 + w1), b1, b2, b3, b4);
            double R = (cui_flux(0.5 * (ues + ue), x1, b2, x3, x4) - cui_flux(0.5 * (us + uc), x0, x1, b2, x3)) * ihx;
            R += (cui_flux(0.5 * (vc + vn), y1, b2, y3, y4) - cui_flux(0.5 * (vs + vc), y0, y1, b2, y3)) * ihy;
            R += (hi - fb) * ihz;
            fb = hi;
            s.out[1][q1] = j == 0 ? nb : s.a_n * nb + s.a_s * b2 - s.c_dt * R;
            if (j == ny - 1) s.out[1][q1 + sy1] = s.rn[1][q1 + sy1];
        }
        // z-face k
        {
            const double x0 = rd[xc0], x1 = rd[xc1], x3 = rd[xc3], x4 = rd[xc4];
            const double y0 = rd[yc0 * sy2], y1 = rd[yc1 * sy2], y3 = rd[yc3 * sy2], y4 = rd[yc4 * sy2];
            const double hi = cui_flux(0.5 * (w0 + w1), d1, d2, d3, d4);
            double R = (cui_flux(0.5 * (ue_lo + ue), x1, d2, x3, x4) - cui_flux(0.5 * (u_lo + uc), x0, x1, d2, x3)) * ihx;
            R += (cui_flux(0.5 * (vn_lo + vn), y1, d2, y3, y4) - cui_flux(0.5 * (v_lo + vc), y0, y1, d2, y3)) * ihy;
            R += (hi - fd) * ihz;
            fd = hi;
            s.out[2][q2] = k == 0 ? nd : s.a_n * nd + s.a_s * d2 - s.c_dt * R;
            if (k == nz - 1) s.out[2][q2 + sz2] = s.rn[2][q2 + sz2];
        }
        a0 = a1; a1 = a2; a2 = a3; a3 = a4;
        b0 = b1; b1 = b2; b2 = b3; b3 = b4;
        d0 = d1; d1 = d2; d2 = d3; d3 = d4;
        u_lo = uc; ue_lo = ue; v_lo = vc; vn_lo = vn;
        w0 = w1; ww0 = ww1; ws0 = ws1;
    }
}

size_t face_count(const stokes_grid *g, int c) {
    const int d = g->dim;
    size_t n = 1;
    for (int a = 0; a < d; ++a) n *= (size_t)g->n[a] + (a == c ? 1 : 0);
    return n;
}

// True when a face array would hold 2^31 faces or more (32-bit thread and face
// indices); counted in double, since a product of 32-bit extents can exceed 64 bits.
bool too_many_faces(const stokes_grid *g) {
    for (int c = 0; c < g->dim; ++c) {
        double n = 1.0;
        for (int a = 0; a < g->dim; ++a) n *= (double)g->n[a] + (a == c ? 1.0 : 0.0);
        if (n >= 2147483648.0) return true;
    }
    return false;
}

}  // namespace

extern "C" size_t stokes_density_workspace_size(const stokes_grid *grid) {
    if (!grid || (grid->dim != 2 && grid->dim != 3)) return 0;
    for (int a = 0; a < grid->dim; ++a)
        if (grid->n[a] < 2) return 0;
    if (too_many_faces(grid)) return 0;
    size_t tot = 0;
    for (int c = 0; c < grid->dim; ++c) tot += face_count(grid, c);
    return tot * sizeof(double);
}

extern "C" stokes_status stokes_density_rk3(const stokes_grid *grid, double dt, const double *const rho_n[3],
                                            const double *const u_stage[9], double *const rho_out[3],
                                            void *workspace, size_t ws_bytes, void *stream) {
    if (!grid || !rho_n || !u_stage || !rho_out) return STOKES_EINVAL;
    const int dim = grid->dim;
    if (dim != 2 && dim != 3) return STOKES_EINVAL;
    for (int d = 0; d < dim; ++d)
        if (grid->periodic[d]) return STOKES_EINVAL;     // walls only
    if (!(dt > 0.0) || !std::isfinite(dt)) return STOKES_EINVAL;
    TrGrid g{};
    g.dim = dim;
    for (int a = 0; a < 3; ++a) {
        g.n[a] = a < dim ? grid->n[a] : 1;
        g.ih[a] = 0.0;
    }
    for (int a = 0; a < dim; ++a) {
        if (grid->n[a] < 2) return STOKES_ESHAPE;
        if (!(grid->h[a] > 0.0) || !std::isfinite(grid->h[a])) return STOKES_EINVAL;
        g.ih[a] = 1.0 / grid->h[a];
    }
    if (too_many_faces(grid)) return STOKES_ESHAPE;
    for (int c = 0; c < dim; ++c) {
        if (!rho_n[c] || !rho_out[c]) return STOKES_EINVAL;
        for (int st = 0; st < 3; ++st)
            if (!u_stage[3 * st + c]) return STOKES_EINVAL;
    }
    const size_t need = stokes_density_workspace_size(grid);
    if (!workspace) return STOKES_EINVAL;
    if (ws_bytes < need) return STOKES_ENOMEM;
    // rho1 lives in rho_out, rho2 in the workspace
    double *r2[3] = {nullptr, nullptr, nullptr};
    {
        double *w = static_cast<double *>(workspace);
        for (int c = 0; c < dim; ++c) {
            r2[c] = w;
            w += face_count(grid, c);
        }
    }
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    // share of the threads of tiles of tx x ty cells (2D: faces) that have one
    const int past = dim == 3 ? 0 : 1;
    auto fill = [&](int tx, int ty) {
        const double x = g.n[0] + past, y = g.n[1] + past;
        return x * y / (std::ceil(x / tx) * tx * std::ceil(y / ty) * ty);
    };
    // tiles of 64 x 4 cells, or 32 x 8 where those leave fewer threads idle
    const bool narrow = dim == 3 && fill(kTrX / 2, 2 * kTrY) > fill(kTrX, kTrY);
    const int tx = narrow ? kTrX / 2 : kTrX, ty = narrow ? 2 * kTrY : kTrY;
    const bool march = dim == 3 && (double)g.n[0] * g.n[1] * g.n[2] >= kTrMarch && fill(tx, ty) >= kTrMarchFill;
    const bool tiled = dim == 2 && fill(tx, ty) >= kTrTileFill;
    const int gx = (g.n[0] + past + tx - 1) / tx, gy = (g.n[1] + past + ty - 1) / ty;
    // z chunks of a marching block: halved down to 3 or 4 planes (a chunk reads four more planes of
    // density and one of velocity) while there are fewer than kTrBlocks blocks
    int kc = g.n[2];
    while (kc > 4 && (double)gx * gy * ((g.n[2] + kc - 1) / kc) < kTrBlocks) kc = (kc + 1) / 2;
    const unsigned tiles = (unsigned)gx * (unsigned)gy;
    // one thread per face of the largest component array, fewer than 2^31
    size_t most = 0;
    for (int c = 0; c < dim; ++c) most = std::max(most, face_count(grid, c));
    const unsigned rows = (unsigned)((most + kTrX * kTrY - 1) / (kTrX * kTrY));
    auto stage = [&](double a_n, double a_s, double c_dt, const double *const rs[3], int st, double *const out[3]) {
        StageArgs a{};
        a.a_n = a_n;
        a.a_s = a_s;
        a.c_dt = c_dt;
        for (int c = 0; c < 3; ++c) {
            a.rn[c] = c < dim ? rho_n[c] : nullptr;
            a.rs[c] = c < dim ? rs[c] : nullptr;
            a.u[c] = c < dim ? u_stage[3 * st + c] : nullptr;
            a.out[c] = c < dim ? out[c] : nullptr;
        }
        const dim3 tile(tx, ty), face(rows, dim);
        const unsigned chunks = tiles * (unsigned)((g.n[2] + kc - 1) / kc);
        if (march && narrow) k_rk3_stage3<kTrX / 2><<<chunks, tile, 0, s>>>(g, a, gx, gy, kc);
        else if (march) k_rk3_stage3<kTrX><<<chunks, tile, 0, s>>>(g, a, gx, gy, kc);
        else if (tiled) k_rk3_stage2<<<dim3(std::min(tiles, 1u << 25), 2), tile, 0, s>>>(g, a, gx, tiles);
        else if (dim == 3) k_rk3_stage<3><<<face, kTrX * kTrY, 0, s>>>(g, a);
        else k_rk3_stage<2><<<face, kTrX * kTrY, 0, s>>>(g, a);
    };
    stage(0.0, 1.0, dt, rho_n, 0, rho_out);
    stage(0.75, 0.25, 0.25 * dt, rho_out, 1, r2);
    stage(1.0 / 3.0, 2.0 / 3.0, (2.0 / 3.0) * dt, r2, 2, rho_out);
    return hipGetLastError() == hipSuccess ? STOKES_OK : STOKES_EHIP;
}
