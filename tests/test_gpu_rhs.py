"""Parity of the device explicit right-hand side (stokes_explicit_rhs) with the
oracle (oracle/assemble.py: explicit_rhs, built on the assembled strain-rate
operator), element by element, and at 256^3 an identity with the solver's own
matvec.

Tolerance: both sides evaluate the same stencil in FP64 (different summation
order and harmonic-mean rounding): |gpu - oracle| <= 1e-12 * max|oracle| per
component; the viscous-dominated cases (dt = 1e3, so rho/dt ~ 1) pin the
viscous part at that level."""
import numpy as np
import pytest

import workloads as W
from oracle import assemble as A
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


def _device(dim, n, h, rho, mu, dt, theta, un, rf, gv):
    import torch
    import paper_1901_07892_amd as S
    grid = S._binding.make_grid(dim, n, h)
    f = [torch.full(W.face_shape(n, c), float("nan"), dtype=torch.float64, device="cuda") for c in range(dim)]
    print("stokes_explicit_rhs dim=%d n=%s theta=%g gravity=%s" % (dim, tuple(n), theta, rf is not None), flush=True)
    S.stokes_explicit_rhs(grid, [to_dev(a) for a in rho], to_dev(mu), dt, theta, [to_dev(a) for a in un], f,
                          [to_dev(a) for a in rf] if rf is not None else None, gv)
    torch.cuda.synchronize()
    return [to_host(a) for a in f]


def _inputs(dim, n, seed, viscous=False):
    rng = np.random.default_rng(seed)
    rho = [rng.uniform(1.0, 1000.0, W.face_shape(n, c)) for c in range(dim)]
    mu = rng.uniform(1e-5, 1e-3, W.cell_shape(n))
    mu[rng.random(mu.shape) < 0.05] = 0.0                    # zero viscosity is allowed
    un = [rng.standard_normal(W.face_shape(n, c)) for c in range(dim)]
    for c in range(dim):                                     # garbage on wall-normal faces: ignored
        for end in (0, -1):
            sl = [slice(None)] * 3
            sl[2 - c] = end
            un[c][tuple(sl)] = 1e6 * rng.standard_normal(un[c][tuple(sl)].shape)
    rf = [rng.uniform(1.0, 1000.0, W.face_shape(n, c)) for c in range(dim)]
    return rho, mu, un, rf


CASES = [(2, (64, 64, 1)), (2, (33, 17, 1)), (3, (13, 11, 9)), (3, (32, 24, 20)), (3, (2, 3, 2))]


@pytest.mark.parametrize("theta,dt,grav", [(0.5, 1e-4, True), (0.0, 1e3, False), (1.0, 1e-3, True),
                                           (0.5, 1e3, True)])
@pytest.mark.parametrize("dim,n", CASES)
def test_explicit_rhs_matches_oracle(dim, n, theta, dt, grav):
    h = tuple(1.0 / max(n[:dim]) * s for s in (1.0, 1.1, 0.9))
    rho, mu, un, rf = _inputs(dim, n, 7 + sum(n))
    gv = (0.4, -9.81, 2.0)
    got = _device(dim, n, h, rho, mu, dt, theta, un, rf if grav else None, gv if grav else None)
    g = A.OGrid(dim, tuple(n), h)
    want = A.explicit_rhs(g, rho, mu, dt, theta, un, rf if grav else None, gv)
    for c in range(dim):
        scale = max(float(np.abs(want[c]).max()), 1e-300)
        np.testing.assert_allclose(got[c], want[c], rtol=0, atol=1e-12 * scale)


def test_explicit_rhs_matches_solver_matvec_at_headline_size():
    """256^3 headline coefficients with dt = 1e3 (viscous terms comparable to the
    mass term): f(theta = 0) + A_1 u^n = 2 (rho/dt) u^n, with A_1 = rho/dt - L_mu
    applied by the solver's matvec (stokes_apply with visc_scale 1), which is
    pinned to the oracle at this size elsewhere."""
    import torch
    import paper_1901_07892_amd as S
    p = W.config5()
    dt = 1e3
    rng = np.random.default_rng(900001)
    un = [rng.standard_normal(W.face_shape(p.n, c)) for c in range(3)]
    for c in range(3):
        for end in (0, -1):
            sl = [slice(None)] * 3
            sl[2 - c] = end
            un[c][tuple(sl)] = 0.0
    f = _device(3, p.n, p.h, p.rho_faces, p.mu, dt, 0.0, un, None, None)
    s = S.StokesSolver(3, p.n, p.h, [to_dev(r) for r in p.rho_faces], to_dev(p.mu), dt, restart=2)
    xd = [to_dev(a) for a in un]
    yd = [torch.zeros_like(a) for a in xd]
    yp = torch.zeros(W.cell_shape(p.n), dtype=torch.float64, device="cuda")
    s.apply(xd, torch.zeros_like(yp), yd, yp)
    torch.cuda.synchronize()
    s.close()
    for c in range(3):
        lhs = f[c] + to_host(yd[c])
        rhs = 2.0 * p.rho_faces[c] / dt * un[c]
        inner = [slice(None)] * 3
        inner[2 - c] = slice(1, -1)
        inner = tuple(inner)
        scale = float(np.abs(f[c]).max())
        assert np.abs(lhs[inner] - rhs[inner]).max() <= 1e-12 * scale


@pytest.mark.parametrize("n", [(30, 6, 4), (31, 7, 5), (61, 13, 9), (60, 12, 33), (2, 2, 40), (29, 5, 17)],
                         ids=lambda n: "x".join(map(str, n)))
def test_explicit_rhs_tile_edges_match_oracle(n):
    """Grids at the edges of the 30 x 6 result tiles and of the z chunks of the 3D kernel, with
    NaN on the wall-normal faces, which are not read."""
    h = (0.01, 0.011, 0.009)
    rho, mu, un, rf = _inputs(3, n, 3)
    clean = [a.copy() for a in un]
    for c in range(3):
        for end in (0, -1):
            sl = [slice(None)] * 3
            sl[2 - c] = end
            un[c][tuple(sl)] = np.nan
            clean[c][tuple(sl)] = 0.0
    got = _device(3, n, h, rho, mu, 1e3, 0.5, un, rf, (0.4, -9.81, 2.0))
    want = A.explicit_rhs(A.OGrid(3, n, h), rho, mu, 1e3, 0.5, clean, rf, (0.4, -9.81, 2.0))
    for c in range(3):
        assert np.abs(got[c] - want[c]).max() <= 1e-12 * np.abs(want[c]).max()


def test_explicit_rhs_on_a_grid_of_more_blocks_than_2_to_24():
    """2 x 101 000 000 x 2 cells: the tiles of such a grid are more than 2^32 threads in a row.
    All inputs are ones, so every row away from the ends holds the values of a short grid's."""
    import torch
    import paper_1901_07892_amd as S
    h, g = (0.25, 0.5, 0.2), (0.0, 0.0, -9.81)

    def run(ny):
        grid = S._binding.make_grid(3, (2, ny, 2), h)
        one = torch.ones(6 * ny + 4, dtype=torch.float64, device="cuda")
        f = [torch.full(s, np.nan, dtype=torch.float64, device="cuda") for s in ((2, ny, 3), (2, ny + 1, 2), (3, ny, 2))]
        S.stokes_explicit_rhs(grid, [one] * 3, one, 0.1, 0.5, [one] * 3, f, [one] * 3, g)
        torch.cuda.synchronize()
        return f
    ny = 101_000_000
    if torch.cuda.mem_get_info()[0] < 10 ** 11:
        pytest.skip("needs 20 GB of device memory")
    print("explicit rhs 2x%dx2" % ny, flush=True)
    small, big = run(32), run(ny)
    for a, b in zip(small, big):
        assert torch.equal(a[:, :8], b[:, :8]) and torch.equal(a[:, -8:], b[:, -8:])
        assert bool((b[:, 8:-8] == a[:, 16:17]).all())
