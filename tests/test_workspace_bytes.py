"""fcmdp_workspace_bytes against the buffers and tables of a solver: particle and
grid buffers, Chebyshev tables, the root tables of the transforms and the
per-stage twiddles of the run-time plans (all but the first stage's: at least
n - 17 of them)."""
import pytest


def _needed(n, nx, ny, nz, word):
    m, nkx = nx // 2, nx // 2 + 1
    blocks = -(-n // 2048)
    buffers = [6 * nz * ny * nx * word, 12 * nz * nkx * ny * word, 4 * n, 4 * n, 4 * n, 4 * n,
               1024 * (blocks + 1), 4 * (nx * ny + 1), 16 * n, 32 * n * word, 8 * n * word,
               2 * n * nz * word, 8, 4]
    tables = [8 * nz, 8 * nz * nz, 8 * nz * nz, word * nz, 8 * 120, word * 120,
              2 * word * m, 2 * word * ny, 2 * word * (m + 1),
              2 * word * max(0, m - 17), 2 * word * max(0, ny - 17)]
    return sum(buffers) + sum(tables)


@pytest.mark.parametrize("precision,word", [("fp64", 8), ("mixed", 4)])
@pytest.mark.parametrize("n,nx,ny,nz", [
    (1, 8, 8, 8), (1000, 96, 90, 32), (4097, 1536, 1536, 8), (1 << 20, 2176, 2176, 32),
    (1, 10000, 4992, 8), (1, 5000, 5000, 64)])
def test_covers_every_buffer(n, nx, ny, nz, precision, word):
    from paper_2210_01837_amd import workspace_bytes
    got = workspace_bytes(n, geometry="bw", Lx=nx * 0.5, Ly=ny * 0.5, H=6.0, Nx=nx, Ny=ny,
                          Nz=nz, precision=precision)
    need = _needed(n, nx, ny, nz, word)
    assert need <= got <= need + 200 * 1024
