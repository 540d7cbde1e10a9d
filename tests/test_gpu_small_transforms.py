"""xy transforms of small grids: the two-buffer kernels that they take by default
in FP64 up to the lines of that rule and just beyond it, and the row kernels at the
same sizes (rows per workgroup asked for), every radix of their run-time plans; and
rows so long that one full batch of them fits a CU, whole and ragged batches.

Tolerances as for the other row transforms, FP64 1e-14, FP32 2e-6."""
import numpy as np
import pytest

import workloads
from workloads import Box

from _parity import rel_err

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _check(nx, ny, nz, lo, hi, precision, rows=None):
    from paper_2210_01837_amd import Solver
    box = Box("bw", nx * 0.5, ny * 0.5, max(4.0, 0.25 * nz), nx, ny, nz)
    real = np.float64 if precision == "fp64" else np.float32
    cplx = np.complex128 if precision == "fp64" else np.complex64
    nkx, sl = nx // 2 + 1, slice(lo, hi + 1)
    s = Solver.from_box(box, precision=precision, max_particles=16)
    if rows:
        s.set_variant("fft_rows_x", rows[0])
        s.set_variant("fft_rows_y", rows[1])
    tol = 1e-14 if precision == "fp64" else 2e-6
    grid = workloads.random_array((6, nz, ny, nx), 51).astype(real)
    spec = _np(s.stage_fft_forward(torch.from_numpy(grid).cuda(), lo, hi))
    ref = np.fft.rfft2(grid[:, sl].astype(np.float64), axes=(-2, -1))
    assert rel_err(spec[:, sl], np.transpose(ref, (0, 1, 3, 2))) < tol
    sp = workloads.random_array((6, nz, nkx, ny), 52, complex_=True).astype(cplx)
    back = _np(s.stage_fft_inverse(torch.from_numpy(sp).cuda(), lo, hi))
    x = np.transpose(sp[:, sl].astype(np.complex128), (0, 1, 3, 2))
    ref = np.fft.irfft2(x, s=(ny, nx), axes=(-2, -1)) * (nx * ny)
    assert rel_err(back[:, sl], ref) < tol
    s.close()


def _np(t):
    torch.cuda.synchronize()
    return t.cpu().numpy().astype(np.complex128 if t.is_complex() else np.float64)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("nx,ny,nz,lo,hi", [
    (8, 8, 8, 4, 7), (24, 26, 32, 8, 31), (34, 22, 17, 0, 16), (80, 80, 32, 30, 31),
    (80, 80, 33, 30, 32), (64, 128, 25, 3, 3), (64, 130, 24, 3, 3), (48, 192, 32, 9, 10),
    (48, 196, 32, 9, 10), (320, 40, 16, 2, 4), (324, 40, 16, 2, 4)])
def test_small_grids(nx, ny, nz, lo, hi, precision):
    print(f"[small transforms] {nx}x{ny}x{nz} {precision}", flush=True)
    _check(nx, ny, nz, lo, hi, precision)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("full", [True, False])
@pytest.mark.parametrize("nx,ny", [
    (8, 8), (18, 14), (20, 24), (28, 30), (32, 22), (34, 52), (182, 34), (180, 128)])
def test_row_kernels_at_small_sizes(nx, ny, full, precision):
    """Every radix from 2 to 17, whole and ragged batches and single rows."""
    print(f"[small row transforms] {nx}x{ny} {precision} full {full}", flush=True)
    rows = (16 if precision == "mixed" else 8, 8) if full else (1, 1)
    _check(nx, ny, 8, 5, 6, precision, rows)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("nx,ny", [(1274, 24), (1280, 32), (1320, 26), (2520, 22), (2592, 20)])
def test_long_rows(nx, ny, precision):
    print(f"[long rows] {nx}x{ny} {precision}", flush=True)
    _check(nx, ny, 8, 4, 5, precision)
