"""Four r-z steps per launch against single steps: bitwise the same fields and
wakes for every remainder of the step count, strips and chunks cut by the
grid's edges, and chunks shorter than their halos."""
import numpy as np
import pytest

from paper_0901_1053_amd import inputs, tete

pytestmark = pytest.mark.gpu

DZ = 1e-3


def _run(nr, nz, mode, precision, kernel, rows, counts):
    dr = DZ if mode else 1.25 * DZ
    G = tete.RZGrid(nr, nz, dr, DZ, DZ, mode, precision=precision)
    G.set_pec_cells(inputs.rz_random_cells(nr, nz, 61))
    G.set_fields(inputs.rz_random_fields(G.shape, 62))
    j0 = 0 if mode == 0 else min(5, nr - 2)
    jw = min(max(1, j0), nr - 3) if nr > 3 else 1
    if nr > 3:
        G.set_bunch(1e-9, 2.0 * DZ, j0, 12, jw, -4, 40)
    G.set_tuning(rows, 0, kernel, 0)
    for n in counts:
        G.step(n)
    out = G.get_fields()
    if nr > 3:
        out["wpar"], out["wperp"] = G.wake()
    G.close()
    return out


# a strip owns 56 k; chunks of 8 rows are half their halo
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("nr,nz,mode,rows", [(2, 2, 1, 0), (9, 55, 0, 0), (40, 56, 1, 8), (33, 113, 2, 11),
                                             (70, 600, 0, 0), (17, 1200, 3, 16)])
def test_four_steps_equal_single_steps(precision, nr, nz, mode, rows):
    print("rz four", precision, nr, nz, mode, rows, flush=True)
    a = _run(nr, nz, mode, precision, "fused", rows, [23])
    for counts in ([23], [4, 6, 13], [1, 8, 2, 12]):
        b = _run(nr, nz, mode, precision, "auto", rows, counts)
        for k in a:
            assert np.array_equal(a[k], b[k]), (counts, k)
