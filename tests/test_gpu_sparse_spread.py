"""Spread of few and of crowded particles on FP64 grids.  Few: the gather up to one
particle in 1024 cells, the matrix cores beyond it, and both block sizes of the
latter there too.  Crowded, on tall grids: the gather from three particles in five
cells on.  Tolerance 1e-13, as for the other FP64 spreads."""
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


@pytest.mark.parametrize("torques", [True, False])
@pytest.mark.parametrize("nz,n,gather", [(41, 48384, True), (41, 48383, False),
                                         (40, 48384, False)])
def test_crowded_tall_grid(nz, n, gather, torques):
    """Default against the gather (its bits where it is the default) and the matrix
    cores."""
    from paper_2210_01837_amd import Solver
    box = Box("sc", 144.0, 140.0, 12.0, 288, 280, nz)
    rng = np.random.default_rng(82)
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda")   # noqa: E731
    P = dev(rng.random((n, 3)) * [box.Lx, box.Ly, box.H])
    F, T = dev(rng.standard_normal((n, 3))), dev(rng.standard_normal((n, 3)))
    print(f"[crowded spread] Nz={nz} n={n} torques {torques}", flush=True)
    s = Solver.from_box(box, precision="fp64", max_particles=n)
    out = []
    for name, value in ((None, 0), ("wave_spread", 1), ("spread_block_rows", 8)):
        if name:
            s.set_variant(name, value)
        out.append(s.stage_spread(P, F, T if torques else None))
        if name:
            s.set_variant(name, 0)
    torch.cuda.synchronize()
    assert torch.equal(out[0], out[1]) == gather
    for other in out[1:]:
        assert float((out[0] - other).norm() / other.norm()) < 1e-13
    s.close()
