"""Viscosities and units of length other than one.

The result of a call is finite and as accurate in any of them: SI units, water in
micrometres, nanometres, a very viscous fluid.  Tolerances as in the other apply
tests: 1e-10 in FP64, 1e-5 in mixed precision.  A change of units by powers of
two changes no rounding by itself, only what leaves a type's range: the scaled
result agrees to 1e-6, a few roundings in FP32.
"""
import numpy as np
import pytest

import workloads
from workloads import Box

from _parity import oracle_apply, rel_err

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# length of a grid cell, height, grid size, viscosity, force
UNITS = {
    "water_um": (1.0, 20.0, 32, 1e-3, 1.0),
    "water_um_wide": (1.0, 100.0, 128, 1e-3, 1.0),
    "nm": (400.0, 8000.0, 48, 1.0, 1.0),
    "nm_thin": (4.0, 100.0, 100, 1e-9, 1e-3),
    "si": (1e-6, 2e-5, 32, 8.9e-4, 1e-14),
    "syrup": (1.0, 20.0, 32, 1e3, 1.0),
}


def _run(box, precision, pos, F, T):
    from paper_2210_01837_amd import Solver
    dt = torch.float64 if precision == "fp64" else torch.float32
    s = Solver.from_box(box, precision=precision, max_particles=len(pos))
    dev = lambda a: torch.tensor(a, dtype=dt, device="cuda")   # noqa: E731
    U, Om = s.apply(dev(pos), dev(F), None if T is None else dev(T))
    torch.cuda.synchronize()
    return (t.cpu().numpy().astype(np.float64) for t in (U, Om))


def _particles(box, n, seed, precision):
    pos, F, T = workloads.random_particles(box, n, seed, 0.1 * box.H, 0.7 * box.H)
    if precision == "mixed":
        pos, F, T = (a.astype(np.float32).astype(np.float64) for a in (pos, F, T))
    return pos, F, T


@pytest.mark.parametrize("torques", [True, False])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("geometry", ["bw", "sc"])
@pytest.mark.parametrize("name", list(UNITS))
def test_units_against_oracle(name, geometry, precision, torques):
    h, H, n, eta, force = UNITS[name]
    box = Box(geometry, n * h, n * h, H, n, n, 32, eta=eta)
    pos, F, T = _particles(box, 40, 71, precision)
    F = (F * force).astype(np.float32).astype(np.float64)
    T = (T * (force * h)).astype(np.float32).astype(np.float64)
    print(f"[units] {name} {geometry} {precision} torques {torques}", flush=True)
    U, Om = _run(box, precision, pos, F, T if torques else None)
    rU, rO = oracle_apply(box, pos, F, T if torques else np.zeros_like(T))
    tol = 1e-10 if precision == "fp64" else 1e-5
    assert rel_err(U, rU) < tol and rel_err(Om, rO) < tol


@pytest.mark.parametrize("geometry", ["bw", "sc"])
@pytest.mark.parametrize("length,visc", [(-20, -10), (-10, 0), (13, 0), (0, -40), (0, 40)])
def test_change_of_units(length, visc, geometry):
    """Lengths times 2^length, viscosity times 2^visc, torques with the lengths:
    U goes with 1 / (viscosity length), Omega with 1 / (viscosity length^2)."""
    box = Box(geometry, 24.0, 20.0, 9.0, 48, 40, 24)
    pos, F, T = _particles(box, 60, 72, "mixed")
    a, b = 2.0 ** length, 2.0 ** visc
    print(f"[change of units] {geometry} 2^{length} 2^{visc}", flush=True)
    U, Om = _run(box, "mixed", pos, F, T)
    other = Box(geometry, 24.0 * a, 20.0 * a, 9.0 * a, 48, 40, 24, eta=b)
    V, Nu = _run(other, "mixed", pos * a, F, T * a)
    assert rel_err(V * (a * b), U) < 1e-6 and rel_err(Nu * (a * a * b), Om) < 1e-6


@pytest.mark.parametrize("geometry", ["bw", "sc"])
@pytest.mark.parametrize("name", ["water_um", "nm", "nm_thin"])
def test_units_with_many_nodes(name, geometry):
    """Nz > 32: FP64 transforms of FP32 data."""
    h, H, n, eta, force = UNITS[name]
    box = Box(geometry, n * h, n * h, H, n, n, 40, eta=eta)
    pos, F, T = _particles(box, 40, 73, "mixed")
    F = (F * force).astype(np.float32).astype(np.float64)
    T = (T * (force * h)).astype(np.float32).astype(np.float64)
    print(f"[units, 40 nodes] {name} {geometry}", flush=True)
    U, Om = _run(box, "mixed", pos, F, T)
    rU, rO = oracle_apply(box, pos, F, T)
    assert rel_err(U, rU) < 1e-5 and rel_err(Om, rO) < 1e-5
