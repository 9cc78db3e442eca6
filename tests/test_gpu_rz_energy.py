"""The r-z energy sum: strips of 64 entries cut by the grid's edge, items of one row,
of a few and of sixteen with a short last one, against the oracle's sum."""
import numpy as np
import pytest

from oracle import rz_oracle as Z
from paper_0901_1053_amd import inputs, tete

pytestmark = pytest.mark.gpu

DZ = 1e-3


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("nr,nz", [(2, 2), (5, 62), (5, 63), (6, 64), (3, 129), (300, 300), (16390, 40), (2700, 1000)])
def test_energy_matches_oracle(nr, nz, mode):
    print("r-z energy", nr, nz, mode, flush=True)
    dr = DZ if mode else 1.25 * DZ
    g = Z.RZGeom(nr, nz, dr, DZ, DZ, mode)
    cells = inputs.rz_random_cells(nr, nz, 63)
    m = Z.materials(g, cells)
    f = inputs.rz_random_fields((nr + 1, nz + 1), 64)
    Z.apply_pec(g, m, f)
    want = Z.energy(g, m, f)
    for precision, tol in (("fp64", 1e-12), ("fp32", 1e-5)):
        G = tete.RZGrid(nr, nz, dr, DZ, DZ, mode, precision=precision)
        G.set_pec_cells(cells)
        G.set_fields(f)
        got = [G.energy()[0] for _ in range(2)]
        assert got[0] == got[1] and abs(got[0] - want) <= tol * abs(want), precision
        G.close()
