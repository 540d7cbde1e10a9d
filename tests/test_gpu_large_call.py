"""The kernels of large calls at few particles, where they can be compared with the
oracle: interpolation over aligned tiles (ragged and narrow last tiles, the smallest
grid, tiles that take several passes, odd Nz, the derivative route) and the general
sort.  Calls this small take other kernels by default (variant "large_call").

Tolerances as in the tests of the same quantities: interpolation 1e-13 in FP64 and
2e-6 in FP32, applies 1e-10 and 1e-5; both sorts are stable, so the grids spread
after them have the same bits.
"""
import numpy as np
import pytest

import workloads
from workloads import Box

from _parity import oracle_apply, oracle_interp, particle_err, rel_err
from oracle import torque_deriv

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TILES = {
    "bw48": ("bw", 32.0, 32.0, 8.0, 48, 48, 32),
    "sc40x56": ("sc", 20.0, 28.0, 7.0, 40, 56, 24),
    "bw68x70": ("bw", 34.0, 35.0, 6.0, 68, 70, 17),       # narrow last tiles: a window meets three
    "sc100x36": ("sc", 50.0, 18.0, 6.0, 100, 36, 13),
    "bw40x22": ("bw", 20.0, 11.0, 5.0, 40, 22, 12),       # the smallest
}


def _dev(a, precision):
    dt = torch.float64 if precision == "fp64" else torch.float32
    return torch.tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")


def _np(t):
    torch.cuda.synchronize()
    return t.cpu().numpy().astype(np.float64)


def _solver(box, precision, cap):
    from paper_2210_01837_amd import Solver
    s = Solver.from_box(box, precision=precision, max_particles=cap)
    s.set_variant("large_call", 1)
    return s


def _particles(box, n, seed, precision, crowd=0):
    """n particles, `crowd` of them in 4 x 4 cells across the seam in x."""
    alpha = 3 * box.h
    zhi = box.H - alpha - 0.05 if box.geometry == "bw" else box.H - 0.2
    pos, F, T = workloads.random_particles(box, n, seed, 0.2, zhi)
    pos[0, :2] = [box.Lx - 1e-3, 0.3]
    pos[1, :2] = [0.2, box.Ly - 0.7 * box.h]
    pos[2, 2] = 0.4 * alpha
    if crowd:
        pos[-crowd:, 0] = (box.Lx - 2 * box.h + 4 * box.h * pos[-crowd:, 0] / box.Lx) % box.Lx
        pos[-crowd:, 1] = 5.0 + 4 * box.h * pos[-crowd:, 1] / box.Ly
    if precision == "mixed":
        pos, F, T = (a.astype(np.float32).astype(np.float64) for a in (pos, F, T))
    return pos, F, T


@pytest.mark.parametrize("crowd", [0, 400])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("name", list(TILES))
def test_interpolation_tiles(name, precision, crowd):
    box = Box(*TILES[name])
    pos, _, _ = _particles(box, 150 + crowd, 61, precision, crowd)
    grid = workloads.random_array((6, box.Nz, box.Ny, box.Nx), 62)
    if precision == "mixed":
        grid = grid.astype(np.float32).astype(np.float64)
    print(f"[large call interp] {name} {precision} crowd {crowd}", flush=True)
    s = _solver(box, precision, 600)
    P, G = _dev(pos, precision), _dev(grid, precision)
    U, Om = s.stage_interp(P, G)
    U2, O2 = s.stage_interp(P, G)
    torch.cuda.synchronize()
    assert torch.equal(U, U2) and torch.equal(Om, O2)
    s.set_variant("large_call", 0)                        # one wavefront per particle
    Uw, Ow = s.stage_interp(P, G)
    rU, rO = oracle_interp(box, pos, grid)
    tol = 1e-13 if precision == "fp64" else 2e-6
    for got, wave, ref in ((U, Uw, rU), (Om, Ow, rO)):
        assert rel_err(_np(got), ref) < tol and particle_err(_np(got), ref) < 4 * tol
        assert rel_err(_np(wave), ref) < tol and particle_err(_np(wave), ref) < 4 * tol
    s.close()


@pytest.mark.parametrize("crowd", [0, 400])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("route", ["curl", "derivative"])
@pytest.mark.parametrize("name", list(TILES))
def test_applies(name, route, precision, crowd):
    box = Box(*TILES[name], torque_route=route)
    pos, F, T = _particles(box, 200 + crowd, 63, precision, crowd)
    print(f"[large call apply] {name} {route} {precision} crowd {crowd}", flush=True)
    if route == "derivative":
        rU, rO = torque_deriv.DerivativeSolver(box).apply(pos, F, T)
    else:
        rU, rO = oracle_apply(box, pos, F, T)
    s = _solver(box, precision, 600)
    P, Fd, Td = (_dev(a, precision) for a in (pos, F, T))
    U, Om = s.apply(P, Fd, Td)
    tol = 1e-10 if precision == "fp64" else 1e-5
    for got, ref in ((U, rU), (Om, rO)):
        assert rel_err(_np(got), ref) < tol and particle_err(_np(got), ref) < 10 * tol
    U3, _ = s.apply(P, Fd, Td, want_omega=False)
    torch.cuda.synchronize()
    assert torch.equal(U, U3)
    s.close()


@pytest.mark.parametrize("n", [1, 64, 65, 2047, 2049, 4096])
@pytest.mark.parametrize("nx,ny", [(14, 16), (48, 44), (320, 324)])   # 1, 2 and 3 digits
def test_sorts_agree(nx, ny, n):
    """The general sort against one workgroup's: crowded and empty cells, particles
    outside the domain, none inside."""
    box = Box("bw", nx * 0.5, ny * 0.5, 6.0, nx, ny, 12)
    rng = np.random.default_rng(64)
    pos = np.stack([rng.uniform(0, box.Lx, n), rng.uniform(0, box.Ly, n),
                    rng.uniform(0.2, 4.0, n)], axis=1)
    pos[: n // 3, :2] = [1.3, 2.4]                        # one cell
    pos[::7, 2] = -1.0                                    # outside
    F, T = rng.standard_normal((2, n, 3))
    print(f"[sorts] {nx}x{ny} n={n}", flush=True)
    s = _solver(box, "fp64", n)
    for p in (pos, np.where([[False, False, True]], -1.0, pos)):
        got = []
        for large in (1, 0):
            s.set_variant("large_call", large)
            g = s.stage_spread(_dev(p, "fp64"), _dev(F, "fp64"), _dev(T, "fp64"))
            got.append((g, s.status()))
        assert torch.equal(got[0][0], got[1][0]) and got[0][1] == got[1][1]
        assert got[0][1][1] == int((p[:, 2] < 0).sum())
    s.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_particles_outside_the_domain(precision):
    box = Box(*TILES["bw68x70"])
    pos, F, T = _particles(box, 60, 65, precision)
    pos[4, 2], pos[7, 2] = -0.1, box.H - 0.5
    s = _solver(box, precision, 60)
    U, Om = (_np(a) for a in s.apply(*(_dev(a, precision) for a in (pos, F, T))))
    assert s.status() == (-2, 2)
    out = np.isnan(U).all(axis=1)
    assert np.array_equal(np.nonzero(out)[0], [4, 7]) and np.isnan(Om[out]).all()
    rU, rO = oracle_apply(box, pos[~out], F[~out], T[~out])
    tol = 1e-10 if precision == "fp64" else 1e-5
    assert rel_err(U[~out], rU) < tol and rel_err(Om[~out], rO) < tol
    s.close()
