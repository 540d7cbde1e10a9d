"""The lines between the kernels of one step, and the edges of their tiles.

Column solve: coefficient counts of every instantiation (Nz 8, 20 | 21, 32 |
33, 48 | 49, 64), bands that end in a tail of one to four nodes or not, a
spectrum that is no whole number of 16-column groups.  Row transforms: every
radix of the run-time plans, both precisions.  Particles: one workgroup's sort
against the general one and its two forms of offsets, one wavefront per
particle against the tiles.  Spread: rings that overflow, odd Nz, rows that are
not 16-byte aligned, in FP64 and with the FP64 vertical force.

Tolerances: FP64 column solve and transforms as in the other stage tests
(1e-11, 1e-14); an FP32 Chebyshev transform sums at most 32 + 32 rounded
products, 64 * 6e-8 = 4e-6 of the result, and the solve may amplify that a few
times on node data that are rough in z: 2e-5.  FP32 row transforms: 2e-6.  The
same particles on two paths differ by the order of the sums only: 1e-12.
"""
import numpy as np
import pytest

import workloads
from workloads import Box

from _parity import oracle_apply, oracle_solve, rel_err

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _solver(box, precision, cap=1 << 10):
    from paper_2210_01837_amd import Solver
    return Solver.from_box(box, precision=precision, max_particles=cap)


def _dev(a, precision):
    dt = torch.float64 if precision == "fp64" else torch.float32
    return torch.tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")


def _np(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy().astype(
        np.complex128 if t.is_complex() else np.float64)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("geometry", ["bw", "sc"])
@pytest.mark.parametrize("nz,lo,hi", [
    (8, 0, 7), (20, 3, 19), (21, 0, 20), (32, 12, 31), (32, 15, 31), (32, 11, 31),
    (32, 20, 20), (33, 0, 32), (48, 29, 47), (49, 5, 48), (64, 0, 63)])
def test_column_solve_sizes(nz, lo, hi, geometry, precision):
    box = Box(geometry, 13.0, 11.0, 6.0, 26, 22, nz)
    sp = workloads.random_array((6, nz, 14, 22), 40 + nz, complex_=True)
    if precision == "mixed":
        sp = sp.astype(np.complex64).astype(np.complex128)
    print(f"[column sizes] {geometry} Nz={nz} band {lo}..{hi} {precision}", flush=True)
    s = _solver(box, precision)
    dt = torch.complex128 if precision == "fp64" else torch.complex64
    got = _np(s.stage_solve(torch.tensor(sp, dtype=dt, device="cuda"), lo, hi))
    ref = oracle_solve(box, sp, lo, hi)
    sl = slice(lo, hi + 1)
    tol = 1e-11 if precision == "fp64" else 2e-5
    for ch in range(6):
        assert rel_err(got[ch, sl], ref[ch, sl]) < tol, ch


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("nx,ny", [
    (8, 8), (18, 14), (20, 24), (28, 30), (32, 22), (34, 52), (182, 204), (192, 450),
    (756, 512), (1250, 1176)])
def test_row_transform_radices(nx, ny, precision):
    box = Box("bw", nx * 0.5, ny * 0.5, 4.0, nx, ny, 8)
    lo = hi = 3
    nkx = nx // 2 + 1
    real = np.float64 if precision == "fp64" else np.float32
    cplx = np.complex128 if precision == "fp64" else np.complex64
    print(f"[row transforms] {nx}x{ny} {precision}", flush=True)
    plane = workloads.random_array((6, ny, nx), 41).astype(real)
    grid = torch.zeros((6, box.Nz, ny, nx), dtype=getattr(torch, real.__name__),
                       device="cuda")
    grid[:, lo] = torch.from_numpy(plane).cuda()
    ref = np.transpose(np.fft.rfft2(plane.astype(np.float64), axes=(-2, -1)), (0, 2, 1))
    sp = workloads.random_array((6, nkx, ny), 42, complex_=True).astype(cplx)
    spec = torch.zeros((6, box.Nz, nkx, ny), dtype=getattr(torch, cplx.__name__),
                       device="cuda")
    spec[:, lo] = torch.from_numpy(sp).cuda()
    back = np.fft.irfft2(np.transpose(sp.astype(np.complex128), (0, 2, 1)), s=(ny, nx),
                         axes=(-2, -1)) * (nx * ny)
    s = _solver(box, precision)
    tol = 1e-14 if precision == "fp64" else 2e-6
    assert rel_err(_np(s.stage_fft_forward(grid, lo, hi))[:, lo], ref) < tol
    assert rel_err(_np(s.stage_fft_inverse(spec, lo, hi))[:, lo], back) < tol


@pytest.mark.parametrize("n", [63, 4096, 8192, 131072])
def test_particle_paths_agree_across_their_line(n):
    """n particles, and the same with one more that carries no force: the two
    calls take different kernels for the sort (4096; the offsets at 131072)
    and the interpolation (8192)."""
    box = Box("bw", 128.0, 128.0, 8.0, 192, 192, 16)
    rng = np.random.default_rng(43)
    pos = np.stack([rng.uniform(0, 128, n + 1), rng.uniform(0, 128, n + 1),
                    rng.uniform(0.3, 5.5, n + 1)], axis=1)
    pos[5, 2] = -1.0                                  # outside the domain
    F, T = rng.standard_normal((2, n + 1, 3))
    F[n], T[n] = 0.0, 0.0
    print(f"[particle paths] n={n}", flush=True)
    s = _solver(box, "fp64", cap=n + 1)
    P, Fd, Td = (_dev(a, "fp64") for a in (pos, F, T))
    U0, O0 = (_np(a) for a in s.apply(P[:n].contiguous(), Fd[:n].contiguous(),
                                      Td[:n].contiguous()))
    assert s.status()[1] == 1
    U1, O1 = (_np(a) for a in s.apply(P, Fd, Td))
    assert s.status()[1] == 1
    for a, b in ((U0, U1[:n]), (O0, O1[:n])):
        assert np.array_equal(np.isnan(a), np.isnan(b)) and np.isnan(a).sum() == 3
        assert rel_err(np.nan_to_num(a), np.nan_to_num(b)) < 1e-12


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("geometry,nz", [("bw", 27), ("sc", 25), ("sc", 24)])
@pytest.mark.parametrize("torques", [True, False])
def test_spread_of_a_dense_cluster(geometry, nz, torques, precision):
    box = Box(geometry, 25.0, 22.0, 7.0, 50, 44, nz)
    n = 300
    pos, F, T = workloads.random_particles(box, n, 44, 0.3, 5.2)
    pos[:260, 0] = 24.2 + 1.6 * (pos[:260, 0] / 25.0)    # across the seam in x
    pos[:260, 1] = 9.0 + 1.2 * (pos[:260, 1] / 22.0)
    if precision == "mixed":
        pos, F, T = (a.astype(np.float32).astype(np.float64) for a in (pos, F, T))
    if not torques:
        T = np.zeros_like(T)
    print(f"[cluster] {geometry} Nz={nz} {precision} torques {torques}", flush=True)
    s = _solver(box, precision)
    U, Om = s.apply(_dev(pos, precision), _dev(F, precision),
                    _dev(T, precision) if torques else None)
    rU, rO = oracle_apply(box, pos, F, T)
    tol = 1e-10 if precision == "fp64" else 1e-5
    assert rel_err(_np(U), rU) < tol and rel_err(_np(Om), rO) < tol
