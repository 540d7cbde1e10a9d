"""xy transforms that run over groups of channels (spectra beyond the last-level
cache): groups of one, two and three channels, and an uneven last group.

Tolerances as for the other row transforms, FP64 1e-14, FP32 2e-6."""
import numpy as np
import pytest

from workloads import Box

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,precision", [(768, "mixed"), (1176, "mixed"), (768, "fp64")])
def test_transforms_by_channel_groups(n, precision):
    from paper_2210_01837_amd import Solver
    print(f"[fft groups] {n} {precision}", flush=True)
    box = Box("bw", n * 0.5, n * 0.5, 8.0, n, n, 32)
    s = Solver.from_box(box, precision=precision, max_particles=16)
    real = torch.float64 if precision == "fp64" else torch.float32
    tol = 1e-14 if precision == "fp64" else 2e-6
    lo, hi = 9, 11
    gen = torch.Generator(device="cuda").manual_seed(5)
    grid = torch.randn((6, 32, n, n), generator=gen, device="cuda", dtype=real)
    spec = s.stage_fft_forward(grid, lo, hi)[:, lo:hi + 1]
    for ch in range(6):
        ref = torch.fft.rfft2(grid[ch, lo:hi + 1].double()).transpose(1, 2)
        err = ((spec[ch] - ref).abs().square().sum() / ref.abs().square().sum()).sqrt()
        assert float(err) < tol, ch
    full = torch.zeros((6, 32, n // 2 + 1, n), device="cuda",
                       dtype=torch.complex128 if precision == "fp64" else torch.complex64)
    full[:, lo:hi + 1] = spec
    back = s.stage_fft_inverse(full, lo, hi)[:, lo:hi + 1].double() / (n * n)
    ref = grid[:, lo:hi + 1].double()
    for ch in range(6):
        err = (back[ch] - ref[ch]).norm() / ref[ch].norm()
        assert float(err) < 2 * tol, ch              # there and back


def test_uneven_group_same_bits():
    """Three channels in FP64 (groups of two and one) against six (two each):
    zero torques leave the bits of U."""
    from paper_2210_01837_amd import Solver
    box = Box("bw", 384.0, 384.0, 8.0, 768, 768, 32)
    s = Solver.from_box(box, precision="fp64", max_particles=4096)
    rng = np.random.default_rng(6)
    pos = np.stack([rng.uniform(0, 384, 4096), rng.uniform(0, 384, 4096),
                    rng.uniform(0.3, 5.5, 4096)], axis=1)
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda")   # noqa: E731
    pos, F = dev(pos), dev(rng.standard_normal((4096, 3)))
    U0, _ = s.apply(pos, F, None, want_omega=False)
    U1, _ = s.apply(pos, F, torch.zeros_like(F), want_omega=True)
    assert torch.isfinite(U0).all() and torch.equal(U0, U1)
