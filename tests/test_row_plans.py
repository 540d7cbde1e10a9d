"""Every grid size that the factors and the LDS of the transforms allow is accepted
in both precisions, so the search for a run-time plan finds one that fits a
workgroup for each of them (creation refuses a size without one)."""
import ctypes

import pytest


def _smooth(n):
    for p in (2, 3, 5, 7, 11, 13, 17):
        while n % p == 0:
            n //= p
    return n == 1


@pytest.mark.parametrize("precision,word", [("fp64", 16), ("mixed", 8)])
def test_every_supported_length_has_a_row_plan(precision, word):
    from paper_2210_01837_amd import _lib, make_params
    L = _lib.lib()
    lds = 160 * 1024
    nb = ctypes.c_size_t(0)

    def code(nx, ny):
        p = make_params("bw", nx * 0.5, ny * 0.5, 4.0, nx, ny, 8, precision=precision)
        return L.fcmdp_workspace_bytes(ctypes.byref(p), 1, ctypes.byref(nb))

    wrong = []
    for n in range(8, 2 * lds // word + 64, 2):
        x_ok = _smooth(n // 2) and (n + 1) * word <= lds
        y_ok = _smooth(n) and 2 * n * word <= lds
        if (code(n, 8) == _lib.OK) != x_ok or (code(8, n) == _lib.OK) != y_ok:
            wrong.append(n)
    assert wrong == []
