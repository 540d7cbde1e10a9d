"""Spread of few particles on FP64 grids: the gather up to one particle in 1024
cells, the matrix cores beyond it, and both block sizes of the latter there too.
Tolerance 1e-13, as for the other FP64 spreads."""
import numpy as np
import pytest

import workloads
from workloads import Box

from _parity import max_rel, oracle_spread, rel_err

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("torques", [True, False])
@pytest.mark.parametrize("rows", [0, 8, 16])
@pytest.mark.parametrize("geometry,nx,ny,nz,n", [
    ("bw", 64, 64, 24, 4), ("bw", 64, 64, 24, 5), ("sc", 90, 50, 27, 1),
    ("sc", 90, 50, 27, 4), ("sc", 90, 50, 27, 5), ("bw", 24, 88, 32, 2)])
def test_few_particles(geometry, nx, ny, nz, n, rows, torques):
    from paper_2210_01837_amd import Solver
    box = Box(geometry, nx * 0.5, ny * 0.5, 8.0, nx, ny, nz)
    pos, F, T = workloads.random_particles(box, n, 81, 0.2, 6.4)
    pos[0, :2] = [box.Lx - 1e-3, 0.3]                     # across both seams
    print(f"[sparse spread] {geometry} {nx}x{ny}x{nz} n={n} rows {rows}", flush=True)
    s = Solver.from_box(box, precision="fp64", max_particles=8)
    if rows:
        s.set_variant("spread_block_rows", rows)
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda")   # noqa: E731
    got = s.stage_spread(dev(pos), dev(F), dev(T) if torques else None)
    torch.cuda.synchronize()
    ref = oracle_spread(box, pos, F, T if torques else np.zeros_like(T))
    got = got.cpu().numpy()
    assert rel_err(got, ref) < 1e-13 and max_rel(got, ref) < 1e-13
    s.close()
