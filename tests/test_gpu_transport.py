"""GPU parity of the SSP-RK3 face-density transport (stokes_density_rk3) with the
oracle (oracle/transport.py), element by element, and its invariants at the
256^3 headline size.

Tolerance: both sides evaluate the same fluxes in FP64 with the same limiter
branches; they differ only in rounding order (and, at a limiter break point,
by the limiter's continuity), so |gpu - oracle| <= 1e-13 max|rho|."""
import numpy as np
import pytest

import workloads as W
from oracle import transport as OT
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


def _gpu(dim, n, h, dt, rho, stages):
    import torch
    import paper_1901_07892_amd as S
    grid = S._binding.make_grid(dim, n, h)
    rd = [to_dev(a) for a in rho]
    ud = [[to_dev(a) for a in st] for st in stages]
    out = [torch.full_like(a, np.nan) for a in rd]
    ws = torch.empty(S.stokes_density_workspace_size(grid), dtype=torch.uint8, device="cuda")
    print("stokes_density_rk3 dim=%d n=%s dt=%g" % (dim, tuple(n), dt), flush=True)
    S.stokes_density_rk3(grid, dt, rd, ud, out, ws)
    torch.cuda.synchronize()
    return [to_host(a) for a in out]


def _stages(dim, n, h, seed, margin=0):
    return [W.stream_velocity(n, h, dim, seed + s, margin=margin) for s in range(3)]


def _random_stages(dim, n, seed):
    """Arbitrary (not divergence-free) stage velocities with zero wall-normal entries."""
    out = []
    for s in range(3):
        xs, _ = W.random_vector(n, dim, seed + s)
        out.append(xs[:dim])
    return out


def _check(got, want, dim):
    scale = max(np.abs(w).max() for w in want)
    errs = [float(np.abs(got[c] - want[c]).max() / scale) for c in range(dim)]
    print("  max |gpu - oracle| / max|rho| per component", ["%.1e" % e for e in errs], flush=True)
    for c in range(dim):
        assert np.all(np.isfinite(got[c]))
    assert max(errs) <= 1e-13, errs


CASES = [
    # config 1's densities (air/water/solid, ratio 833) in a divergence-free flow, CFL 0.4
    ("config1_64", lambda: W.config1(), "stream", 0.4),
    # config 2's wavy interface and three discs at a quarter of its size
    ("config2_128", lambda: W.config2(scale=4), "stream", 0.4),
    # config 3's dam break at 32^3
    ("config3_32", lambda: W.config3(scale=4), "stream", 0.3),
    # the headline recipe at 48^3 with arbitrary (not divergence-free) stage velocities
    ("config5_48_random_u", lambda: W.config5(n_cells=48), "random", 0.2),
]


@pytest.mark.parametrize("name,maker,kind,cfl", CASES)
def test_density_transport_matches_oracle(name, maker, kind, cfl):
    prob = maker()
    dim, n, h = prob.dim, prob.n, prob.h
    rho = [prob.rho_faces[c] for c in range(dim)]
    stages = _stages(dim, n, h, 11) if kind == "stream" else _random_stages(dim, n, 21)
    umax = max(float(np.abs(a).max()) for st in stages for a in st)
    dt = cfl * min(h[:dim]) / umax
    got = _gpu(dim, n, h, dt, rho, stages)
    want = OT.ssp_rk3(dim, h, dt, rho, stages)
    _check(got, want, dim)
    moved = max(float(np.abs(want[c] - rho[c]).max()) for c in range(dim))
    assert moved > 1e-3 * max(float(np.abs(r).max()) for r in rho)     # the interface did move


@pytest.mark.parametrize("dim,n", [(2, (7, 5, 1)), (3, (5, 9, 6)), (3, (2, 2, 2)), (3, (3, 2, 4))])
def test_density_transport_ragged_and_minimal_grids(dim, n):
    rng = np.random.default_rng(sum(n))
    h = (0.2, 0.15, 0.1)
    rho = [rng.uniform(1.0, 1000.0, size=W.face_shape(n, c)) for c in range(dim)]
    stages = _random_stages(dim, n, 3)
    got = _gpu(dim, n, h, 0.01, rho, stages)
    _check(got, OT.ssp_rk3(dim, h, 0.01, rho, stages), dim)


def test_density_transport_full_size_headline():
    """The 256^3 headline densities (two solids, density ratio 1000): element by
    element against the oracle, and mass conserved to round-off by a flow that
    vanishes near the walls."""
    prob = W.config5()
    dim, n, h = 3, prob.n, prob.h
    rho = [prob.rho_faces[c] for c in range(3)]
    stages = _stages(dim, n, h, 31, margin=2)
    dt = 0.3 * h[0]                                       # max |u| = 1
    got = _gpu(dim, n, h, dt, rho, stages)
    print("  oracle at 256^3 ...", flush=True)
    want = OT.ssp_rk3(dim, h, dt, rho, stages)
    _check(got, want, dim)
    for c in range(3):
        m0, m1 = float(rho[c].sum()), float(got[c].sum())
        print("  component %d: mass %.15e -> %.15e" % (c, m0, m1), flush=True)
        assert abs(m1 - m0) <= 1e-12 * m0


def test_density_transport_argument_errors():
    import torch
    import paper_1901_07892_amd as S
    n, h = (4, 4, 4), (0.25,) * 3
    grid = S._binding.make_grid(3, n, h)
    rho = [torch.ones(W.face_shape(n, c), dtype=torch.float64, device="cuda") for c in range(3)]
    u = [[torch.zeros_like(a) for a in rho] for _ in range(3)]
    out = [torch.zeros_like(a) for a in rho]
    ws = torch.empty(S.stokes_density_workspace_size(grid), dtype=torch.uint8, device="cuda")
    with pytest.raises(S.StokesError) as e:
        S.stokes_density_rk3(grid, -1.0, rho, u, out, ws)
    assert e.value.status == -1
    with pytest.raises(S.StokesError) as e:
        S.stokes_density_rk3(grid, 0.1, rho, u, out, ws[:8])
    assert e.value.status == -3
    bad = S._binding.make_grid(3, (1, 4, 4), h)
    with pytest.raises(S.StokesError) as e:
        S.stokes_density_rk3(bad, 0.1, rho, u, out, ws)
    assert e.value.status == -2


@pytest.mark.parametrize("n", [(2, 2, 2), (65, 3, 33), (70, 9, 1), (2, 3, 1), (64, 64, 32), (65, 67, 31), (129, 31, 37), (40, 100, 34), (2, 2, 32768)],
                         ids=lambda n: "x".join(map(str, n)))
def test_rk3_tile_edges_match_oracle(n):
    """Small and 2D grids (one thread per face) and grids of at least 2^17 cells around the
    64 x 4 and 32 x 8 tiles and the z chunks of the marching kernel (one cell past a tile, a
    last chunk of fewer planes, columns of 2 cells), with jumps of 1 to 1000 so that every
    branch of the limiter is taken."""
    dim = 2 if n[2] == 1 else 3
    h = (1.0 / 64,) * 3
    rng = np.random.default_rng(n[0])
    rho = [10.0 ** rng.uniform(0.0, 3.0, W.face_shape(n, c)) for c in range(dim)]
    stages = _random_stages(dim, n, 7)
    dt = 0.05 * h[0] / max(float(np.abs(a).max()) for st in stages for a in st)
    _check(_gpu(dim, n, h, dt, rho, stages), OT.ssp_rk3(dim, h, dt, rho, stages), dim)


def _cui_by_branches(U, C, D):
    """The limiter as its chain of branches, whose comparisons also decide for NaN and infinities."""
    with np.errstate(invalid="ignore"):
        A, N = D - U, C - U
        An, Nn = np.abs(A), np.where(A > 0.0, N, -N)
        return np.select([A == 0.0, (Nn <= 0.0) | (Nn >= An), 13.0 * Nn <= 2.0 * An, 5.0 * Nn <= 4.0 * An],
                         [C, C, U + 3.0 * N, U + (5.0 / 6.0) * N + A / 3.0], D)


@pytest.mark.parametrize("n", [(24, 18, 1), (9, 7, 6), (64, 64, 40), (96, 64, 64), (254, 130, 1)], ids=lambda n: "x".join(map(str, n)))
def test_rk3_carries_nan_and_infinities(n, monkeypatch):
    """Invalid densities reach the same faces as through the limiter's branches: a NaN in a region
    of equal densities spreads to the faces downstream of it.  Half of the grid holds one density,
    the other half random ones; finite results within the module's bound."""
    dim = 2 if n[2] == 1 else 3
    h = (1.0 / 64,) * 3
    rng = np.random.default_rng(5)
    rho = []
    for c in range(dim):
        r = rng.uniform(1.0, 1000.0, W.face_shape(n, c))
        r[:, :n[1] // 2] = 700.0
        at = rng.choice(r.size, 12, replace=False)
        r.reshape(-1)[at] = [np.nan] * 8 + [np.inf] * 4
        rho.append(r)
    stages = _random_stages(dim, n, 7)
    dt = 0.05 * h[0] / max(float(np.abs(a).max()) for st in stages for a in st)
    monkeypatch.setattr(OT, "cui_face", _cui_by_branches)
    with np.errstate(invalid="ignore"):
        want = OT.ssp_rk3(dim, h, dt, rho, stages)
    got = _gpu(dim, n, h, dt, rho, stages)
    for c in range(dim):
        fin = np.isfinite(want[c])
        assert 0 < np.isnan(want[c]).sum() < want[c].size // 2
        assert np.array_equal(np.isnan(got[c]), np.isnan(want[c])), c
        assert np.array_equal(got[c][np.isinf(want[c])], want[c][np.isinf(want[c])]), c
        assert np.abs(got[c][fin] - want[c][fin]).max() <= 1e-13 * 1000.0


@pytest.mark.parametrize("n", [(128, 64, 48), (129, 61, 51), (90, 67, 66), (44, 100, 91), (1024, 200, 2), (65, 65, 94), (255, 6, 1),
                               (255, 3, 1), (63, 3, 1), (64, 3, 1), (9, 70, 1)], ids=lambda n: "x".join(map(str, n)))
def test_rk3_routes_match_oracle(n):
    """Both sides of the rules that choose the kernel: 3D grids of 3 * 2^17 cells and more with 64 x 4
    tiles, 32 x 8 tiles, one cell past a tile, a shorter last z chunk and columns of 2 cells, and one
    whose tiles are too empty; 2D grids with full, half empty and nearly empty tiles.  The inputs of
    the test of the tile edges."""
    dim = 2 if n[2] == 1 else 3
    h = (1.0 / 64,) * 3
    rng = np.random.default_rng(n[0])
    rho = [10.0 ** rng.uniform(0.0, 3.0, W.face_shape(n, c)) for c in range(dim)]
    stages = _random_stages(dim, n, 7)
    dt = 0.05 * h[0] / max(float(np.abs(a).max()) for st in stages for a in st)
    _check(_gpu(dim, n, h, dt, rho, stages), OT.ssp_rk3(dim, h, dt, rho, stages), dim)


@pytest.mark.parametrize("n,like", [((2, 2, 33000), (64, 64, 32)), ((4, 4, 5000), (50, 50, 32)), ((4, 200, 200), (64, 64, 39)),
                                    ((8, 100000, 1), (900, 900, 1))],
                         ids=lambda n: "x".join(map(str, n)))
def test_rk3_narrow_grids_cost_what_their_faces_do(n, like):
    """Grids a few cells wide take no tiles that leave most threads idle: at most four times
    as long as a grid of other proportions with as many cells (launches in both)."""
    import torch
    import paper_1901_07892_amd as S

    def us(m):
        dim = 2 if m[2] == 1 else 3
        grid = S._binding.make_grid(dim, m, (1.0 / 64,) * 3)
        mk = lambda v: [torch.full(W.face_shape(m, c), v, dtype=torch.float64, device="cuda") for c in range(dim)]
        rho, u, out = mk(2.0), [mk(0.1) for _ in range(3)], mk(0.0)
        ws = torch.empty(S.stokes_density_workspace_size(grid), dtype=torch.uint8, device="cuda")
        best = float("inf")
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                S.stokes_density_rk3(grid, 1e-4, rho, u, out, ws)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 100.0)
        return best
    t, ref = us(n), us(like)
    print("  density %s %.1f us, %s %.1f us" % (n, t, like, ref), flush=True)
    assert t <= 4.0 * ref
