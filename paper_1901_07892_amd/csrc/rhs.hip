// Explicit momentum right-hand side of one time step.
//
// Moving the explicit terms of the discrete momentum equations to the right
// (Sec. 4.2.2, eq_nc_discrete_momentum, and eq_c_discrete_momentum with the old
// density), with the viscous term split as theta (new) + (1 - theta) (old),
// gives on every interior face
//     f = (rho/dt) u^n + (1 - theta) L_mu u^n + rho_force g,
// L_mu u = div[mu (grad u + grad u^T)] the strain-rate operator of the solve
// (shear viscosity on cell edges = harmonic mean of the four cells around the
// edge, out-of-domain cells mirrored; no-slip walls: wall-normal velocity zero,
// tangential ghost = minus the interior value).  theta = 1/2 is the paper's
// Crank-Nicolson split; rho_force is the flow-only density for the
// well-balanced gravity force (Sec. 5).  The convective term is the caller's.
//
// Two kernels: in 3D, a z-marching one with the old velocity, the viscosity and the
// shear stresses of a plane in LDS (k_explicit_rhs3_z, below); in 2D, one thread per point
// (i, j) of the (Nx+1)(Ny+1) index space, which holds the x-face i and the
// y-face j of cell (i, j), neighbours from cache (k_explicit_rhs2).  All arrays
// are the caller's C-order layouts.
#include "../../include/stokes.h"

#include <hip/hip_runtime.h>

#include <cmath>

namespace {

constexpr int kRhsBlock = 256;

struct RhsArgs {
    int dim, nx, ny, nz;
    double ihx, ihy, ihz;
    double idt, expl;        // 1/dt, 1 - theta
    double g[3];
    const double *u, *v, *w, *mu;
    const double *rx, *ry, *rz;      // density of the mass term
    const double *fx, *fy, *fz;      // density of the gravity force (may be null)
};

struct Fields {
    const RhsArgs &a;
    __device__ int cx(int i) const { return min(max(i, 0), a.nx - 1); }
    __device__ int cy(int j) const { return min(max(j, 0), a.ny - 1); }
    __device__ int cz(int k) const { return min(max(k, 0), a.nz - 1); }
    __device__ double M(int i, int j, int k) const {        // cell viscosity, mirrored outside
        return a.mu[cx(i) + a.nx * (cy(j) + a.ny * cz(k))];
    }
    // harmonic mean of four viscosities, 4 / (1/p + 1/q + 1/r + 1/s), with one
    // division: 4 pq rs / ((p + q) rs + (r + s) pq); 0 if any of them is 0
    __device__ static double hm4(double p, double q, double r, double s) {
        const double pq = p * q, rs = r * s;
        const double num = pq * rs;
        return num == 0.0 ? 0.0 : 4.0 * num / ((p + q) * rs + (r + s) * pq);
    }
    __device__ double Mxy(int i, int j, int k) const {
        return hm4(M(i - 1, j - 1, k), M(i, j - 1, k), M(i - 1, j, k), M(i, j, k));
    }
    // velocity components with the wall rules: wall-normal entries read as 0,
    // tangential ghosts beyond a wall are minus the mirrored interior value
    __device__ double U(int i, int j, int k) const {
        if (i <= 0 || i >= a.nx) return 0.0;
        double s = 1.0;
        if (j < 0) { j = -1 - j; s = -s; } else if (j >= a.ny) { j = 2 * a.ny - 1 - j; s = -s; }
        if (a.dim == 3) { if (k < 0) { k = -1 - k; s = -s; } else if (k >= a.nz) { k = 2 * a.nz - 1 - k; s = -s; } }
        return s * a.u[i + (a.nx + 1) * (j + a.ny * k)];
    }
    __device__ double V(int i, int j, int k) const {
        if (j <= 0 || j >= a.ny) return 0.0;
        double s = 1.0;
        if (i < 0) { i = -1 - i; s = -s; } else if (i >= a.nx) { i = 2 * a.nx - 1 - i; s = -s; }
        if (a.dim == 3) { if (k < 0) { k = -1 - k; s = -s; } else if (k >= a.nz) { k = 2 * a.nz - 1 - k; s = -s; } }
        return s * a.v[i + a.nx * (j + (a.ny + 1) * k)];
    }
    __device__ double W(int i, int j, int k) const {
        if (a.dim != 3 || k <= 0 || k >= a.nz) return 0.0;
        double s = 1.0;
        if (i < 0) { i = -1 - i; s = -s; } else if (i >= a.nx) { i = 2 * a.nx - 1 - i; s = -s; }
        if (j < 0) { j = -1 - j; s = -s; } else if (j >= a.ny) { j = 2 * a.ny - 1 - j; s = -s; }
        return s * a.w[i + a.nx * (j + a.ny * k)];
    }
};

__global__ void __launch_bounds__(kRhsBlock) k_explicit_rhs2(RhsArgs a, double *__restrict__ ox,
                                                             double *__restrict__ oy) {
    const int px = a.nx + 1, py = a.ny + 1;
    const int p = blockIdx.x * kRhsBlock + threadIdx.x;
    if (p >= px * py) return;
    const int i = p % px, j = p / px;
    const Fields F{a};
    const double hx = a.ihx, hy = a.ihy;
    // x-face i of row j
    if (j < a.ny) {
        double r = 0.0;
        if (i > 0 && i < a.nx) {
            const double u0 = F.U(i, j, 0);
            double L = 2.0 * hx * hx * (F.M(i, j, 0) * (F.U(i + 1, j, 0) - u0) - F.M(i - 1, j, 0) * (u0 - F.U(i - 1, j, 0)));
            L += hy * (F.Mxy(i, j + 1, 0) * ((F.U(i, j + 1, 0) - u0) * hy + (F.V(i, j + 1, 0) - F.V(i - 1, j + 1, 0)) * hx) -
                       F.Mxy(i, j, 0) * ((u0 - F.U(i, j - 1, 0)) * hy + (F.V(i, j, 0) - F.V(i - 1, j, 0)) * hx));
            const int o = i + px * j;
            r = a.rx[o] * a.idt * u0 + a.expl * L;
            if (a.fx) r += a.fx[o] * a.g[0];
        }
        ox[i + px * j] = r;
    }
    // y-face j of column i
    if (i < a.nx) {
        double r = 0.0;
        if (j > 0 && j < a.ny) {
            const double v0 = F.V(i, j, 0);
            double L = 2.0 * hy * hy * (F.M(i, j, 0) * (F.V(i, j + 1, 0) - v0) - F.M(i, j - 1, 0) * (v0 - F.V(i, j - 1, 0)));
            L += hx * (F.Mxy(i + 1, j, 0) * ((F.V(i + 1, j, 0) - v0) * hx + (F.U(i + 1, j, 0) - F.U(i + 1, j - 1, 0)) * hy) -
                       F.Mxy(i, j, 0) * ((v0 - F.V(i - 1, j, 0)) * hx + (F.U(i, j, 0) - F.U(i, j - 1, 0)) * hy));
            const int o = i + a.nx * j;
            r = a.ry[o] * a.idt * v0 + a.expl * L;
            if (a.fy) r += a.fy[o] * a.g[1];
        }
        oy[i + a.nx * j] = r;
    }
}

// 3D form, marching in z: a block of 32 x 8 threads covers a tile of points with one
// point of overlap on every side, so that 30 x 6 of its threads write results.  Every
// thread loads the velocities and viscosity of its own point one plane ahead, with the
// wall rules applied (wall-normal entries 0, tangential ghosts odd, viscosity mirrored);
// in-plane neighbours come from LDS, the plane below from registers.  A thread evaluates
// the three shear stresses on the edges through its point's lower corner once (three
// harmonic means, i.e. divisions, per point) and shares them through LDS: the rows of
// the x-, y- and z-face of a cell are differences of these and of normal stresses.
// The stress differences along z need the edges of the next plane, so plane k is written
// in the step of plane k + 1.  Bound by the latency of a plane step, its loads and two
// barriers: 250 x 190 x 131 in 315 us with loads waited for in the same step, nine
// harmonic means per point and one 512-thread block per CU; 191 us now (3.4 TB/s), with 136
// registers and three wavefronts per SIMD.  Of
// the blocks tried (64 x 16, 64 x 8, 32 x 32, 32 x 16, 32 x 8, 16 x 16) the small one
// wins although its overlap is the larger: three of them share a CU.
// The wall-normal faces beyond the last cell of a row, column or stack (i = Nx, j = Ny,
// k = Nz) hold zero and are written by that last cell's thread.
constexpr int kZX = 32, kZY = 8;
constexpr int kOX = kZX - 2, kOY = kZY - 2;      // results per block and plane
constexpr int kRhsBlocks = 2048;                 // blocks that a launch aims at

__global__ void __launch_bounds__(kZX *kZY) k_explicit_rhs3_z(RhsArgs a, int gx, int gy, int kc,
        double *__restrict__ ox, double *__restrict__ oy, double *__restrict__ oz) {
    __shared__ double sU[2][kZX * kZY], sV[2][kZX * kZY], sW[2][kZX * kZY], sM[2][kZX * kZY];
    __shared__ double sXY[kZX * kZY], sXZ[kZX * kZY], sYZ[kZX * kZY];
    // tiles in x, y, then chunks of kc planes; each XCD takes a contiguous range
    const unsigned G = gridDim.x, b = blockIdx.x, per = G >> 3, rest = G & 7, xcd = b & 7, loc = b >> 3;
    const unsigned t = xcd < rest ? xcd * (per + 1) + loc : rest * (per + 1) + (xcd - rest) * per + loc;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int tx = threadIdx.x, ty = threadIdx.y, tid = tx + kZX * ty;
    const int i = (int)(t % gx) * kOX + tx - 1, j = (int)(t / gx % gy) * kOY + ty - 1;
    const int k0 = (int)(t / gx / gy) * kc, k1 = min(k0 + kc, nz);
    const bool out = tx >= 1 && tx <= kOX && ty >= 1 && ty <= kOY && i < nx && j < ny;
    // this point's offset in a plane of each array (mirrored beyond the walls) and sign
    const int im = i < 0 ? 0 : i >= nx ? 2 * nx - 1 - i : i, jm = j < 0 ? 0 : j >= ny ? 2 * ny - 1 - j : j;
    const bool near = i <= nx && j <= ny;        // farther points are never used
    const double su = near && i > 0 && i < nx ? (j < 0 || j >= ny ? -1.0 : 1.0) : 0.0;
    const double sv = near && j > 0 && j < ny ? (i < 0 || i >= nx ? -1.0 : 1.0) : 0.0;
    const double sw = near ? ((i < 0 || i >= nx) != (j < 0 || j >= ny) ? -1.0 : 1.0) : 0.0;
    const int qu = su != 0.0 ? i + (nx + 1) * jm : 0, qv = sv != 0.0 ? im + nx * j : 0, qw = sw != 0.0 ? im + nx * jm : 0;
    const int zu = (nx + 1) * ny, zv = nx * (ny + 1), zw = nx * ny;      // plane strides
    const int qm = near ? min(max(i, 0), nx - 1) + nx * min(max(j, 0), ny - 1) : 0;
    double u, v, w, m;                           // own point at the plane being loaded, -1 .. nz
    auto load = [&](int k) {
        const int kk = k < 0 ? 0 : k >= nz ? nz - 1 : k;
        const double sz = k < 0 || k >= nz ? -1.0 : 1.0;
        // (a wall-normal entry is not read as 0 times whatever it holds)
        u = su != 0.0 ? su * sz * a.u[qu + zu * kk] : 0.0;
        v = sv != 0.0 ? sv * sz * a.v[qv + zv * kk] : 0.0;
        w = sw != 0.0 && k > 0 && k < nz ? sw * a.w[qw + zw * k] : 0.0;
        m = a.mu[qm + zw * kk];
    };
    const double hx = a.ihx, hy = a.ihy, hz = a.ihz;
    // plane k - 1: own values, viscosities to the west and south, z-edge stresses, and what
    // the rows of that plane already have
    double ul = 0.0, vl = 0.0, wl = 0.0, ml = 0.0, mwl = 0.0, msl = 0.0, wll = 0.0, mll = 0.0;
    double xzl = 0.0, yzl = 0.0, Lx = 0.0, Ly = 0.0, Lzx = 0.0, Lzy = 0.0;
    double rxn = 0.0, ryn = 0.0, rzn = 0.0, fxn = 0.0, fyn = 0.0, fzn = 0.0;
    load(k0 - 1);
    for (int k = k0 - 1; k <= k1; ++k) {
        const int s = k & 1;
        const double uc = u, vc = v, wc = w, mc = m;
        sU[s][tid] = uc;
        sV[s][tid] = vc;
        sW[s][tid] = wc;
        sM[s][tid] = mc;
        // the next plane, and this plane's densities for its rows, which end in the next step
        if (k < k1) load(k + 1);
        const bool write = out && k > k0;
        const double rx = rxn, ry = ryn, rz = rzn, fx = fxn, fy = fyn, fz = fzn;
        if (out && k >= k0 && k < k1) {
            const int ku = i + (nx + 1) * (j + ny * k), kv = i + nx * (j + (ny + 1) * k), kw = i + nx * (j + ny * k);
            rxn = a.rx[ku];
            ryn = a.ry[kv];
            rzn = a.rz[kw];
            if (a.fx) {
                fxn = a.fx[ku];
                fyn = a.fy[kv];
                fzn = a.fz[kw];
            }
        }
        __syncthreads();
        // neighbours west and south (threads at the tile's rim read any valid slot: their
        // stresses are not used)
        const int tw = tx > 0 ? tid - 1 : tid, ts = ty > 0 ? tid - kZX : tid, tws = tx > 0 && ty > 0 ? tid - kZX - 1 : tid;
        const double us = sU[s][ts], vw = sV[s][tw], ww = sW[s][tw], ws = sW[s][ts];
        const double mw = sM[s][tw], ms = sM[s][ts], mws = sM[s][tws];
        const double xy = Fields::hm4(mws, ms, mw, mc) * ((uc - us) * hy + (vc - vw) * hx);
        const double xz = Fields::hm4(mwl, ml, mw, mc) * ((uc - ul) * hz + (wc - ww) * hx);
        const double yz = Fields::hm4(msl, ml, ms, mc) * ((vc - vl) * hz + (wc - ws) * hy);
        sXY[tid] = xy;
        sXZ[tid] = xz;
        sYZ[tid] = yz;
        __syncthreads();
        if (write) {
            // rows of plane k - 1
            const int ku = i + (nx + 1) * (j + ny * (k - 1)), kv = i + nx * (j + (ny + 1) * (k - 1)), kw = i + nx * (j + ny * (k - 1));
            const double Lxk = Lx + hz * (xz - xzl), Lyk = Ly + hz * (yz - yzl);
            double r = i > 0 ? rx * a.idt * ul + a.expl * Lxk + fx * a.g[0] : 0.0;
            ox[ku] = r;
            if (i == nx - 1) ox[ku + 1] = 0.0;               // wall face i = nx
            r = j > 0 ? ry * a.idt * vl + a.expl * Lyk + fy * a.g[1] : 0.0;
            oy[kv] = r;
            if (j == ny - 1) oy[kv + nx] = 0.0;              // wall face j = ny
            double L = 2.0 * hz * hz * (ml * (wc - wl) - mll * (wl - wll));
            L += Lzx;
            L += Lzy;
            r = k > 1 ? rz * a.idt * wl + a.expl * L + fz * a.g[2] : 0.0;
            oz[kw] = r;
            if (k == nz) oz[kw + nx * ny] = 0.0;             // wall face k = nz
        }
        if (out) {
            const double ue = sU[s][tid + 1], uw = sU[s][tid - 1], vn = sV[s][tid + kZX], vs = sV[s][tid - kZX];
            Lx = 2.0 * hx * hx * (mc * (ue - uc) - mw * (uc - uw)) + hy * (sXY[tid + kZX] - xy);
            Ly = 2.0 * hy * hy * (mc * (vn - vc) - ms * (vc - vs)) + hx * (sXY[tid + 1] - xy);
            Lzx = hx * (sXZ[tid + 1] - xz);
            Lzy = hy * (sYZ[tid + kZX] - yz);
        }
        xzl = xz;
        yzl = yz;
        wll = wl;
        mll = ml;
        ul = uc;
        vl = vc;
        wl = wc;
        ml = mc;
        mwl = mw;
        msl = ms;
    }
}

bool finite_pos(double v) { return std::isfinite(v) && v > 0.0; }

}  // namespace

extern "C" stokes_status stokes_explicit_rhs(const stokes_grid *grid, const double *const rho_face[3],
        const double *mu_cell, double dt, double theta, const double *const u_n[3],
        const double *const rho_force[3], const double gravity[3], double *const f[3], void *stream) {
    if (!grid || !rho_face || !mu_cell || !u_n || !f) return STOKES_EINVAL;
    const int dim = grid->dim;
    if (dim != 2 && dim != 3) return STOKES_EINVAL;
    for (int d = 0; d < dim; ++d) {
        if (grid->periodic[d]) return STOKES_EINVAL;     // walls only
        if (grid->n[d] < 2) return STOKES_ESHAPE;
        if (!finite_pos(grid->h[d])) return STOKES_EINVAL;
        if (!rho_face[d] || !u_n[d] || !f[d] || (rho_force && !rho_force[d])) return STOKES_EINVAL;
    }
    if (!finite_pos(dt) || !std::isfinite(theta) || theta < 0.0 || theta > 1.0) return STOKES_EINVAL;
    if (rho_force && (!gravity || !std::isfinite(gravity[0]) || !std::isfinite(gravity[1]) ||
                      (dim == 3 && !std::isfinite(gravity[2]))))
        return STOKES_EINVAL;
    const long long nz = dim == 3 ? grid->n[2] : 1;
    // point count in double: a product of three 32-bit extents can exceed 64 bits
    const double pts = ((double)grid->n[0] + 1) * ((double)grid->n[1] + 1) * (dim == 3 ? (double)nz + 1 : 1.0);
    if (pts >= (double)((1LL << 31) - kRhsBlock)) return STOKES_ESHAPE;   // 32-bit point and array indices
    RhsArgs a{};
    a.dim = dim;
    a.nx = grid->n[0];
    a.ny = grid->n[1];
    a.nz = (int)nz;
    a.ihx = 1.0 / grid->h[0];
    a.ihy = 1.0 / grid->h[1];
    a.ihz = dim == 3 ? 1.0 / grid->h[2] : 0.0;
    a.idt = 1.0 / dt;
    a.expl = 1.0 - theta;
    a.u = u_n[0];
    a.v = u_n[1];
    a.w = dim == 3 ? u_n[2] : nullptr;
    a.mu = mu_cell;
    a.rx = rho_face[0];
    a.ry = rho_face[1];
    a.rz = dim == 3 ? rho_face[2] : nullptr;
    if (rho_force) {
        a.fx = rho_force[0];
        a.fy = rho_force[1];
        a.fz = dim == 3 ? rho_force[2] : nullptr;
        for (int d = 0; d < 3; ++d) a.g[d] = d < dim ? gravity[d] : 0.0;
    }
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (dim == 3) {
        // z chunks halved down to 3 or 4 planes (a chunk loads two more) while there are fewer than
        // kRhsBlocks blocks; with 1024 / 2048 / 4096 of them aimed at: 128^3 62 / 64 / 65 us, 200^3
        // 247 / 243 / 256, 250 x 190 x 131 207 / 183 / 198, 256^3 580 / 508 / 493, 1024 x 96 x 96 305 / 260 / 273
        const int gx = (a.nx + kOX - 1) / kOX, gy = (a.ny + kOY - 1) / kOY;
        int kc = a.nz;
        while (kc > 4 && (double)gx * gy * ((a.nz + kc - 1) / kc) < kRhsBlocks) kc = (kc + 1) / 2;
        const unsigned blocks = (unsigned)gx * (unsigned)gy * (unsigned)((a.nz + kc - 1) / kc);
        // (a launch holds fewer than 2^32 threads along an axis, and the runtime takes more without
        // an error: blocks of 32 x 8, since a thin grid can have 4e7 of them)
        k_explicit_rhs3_z<<<blocks, dim3(kZX, kZY), 0, s>>>(a, gx, gy, kc, f[0], f[1], f[2]);
    } else {
        const unsigned blocks = (unsigned)((pts + kRhsBlock - 1) / kRhsBlock);
        k_explicit_rhs2<<<blocks, kRhsBlock, 0, s>>>(a, f[0], f[1]);
    }
    return hipGetLastError() == hipSuccess ? STOKES_OK : STOKES_EHIP;
}
