"""Plane solves of the implicit scheme taken several iterations per pass:
tiles cut exactly and one row, entry or plane over, one pass and many, and work
items wholly in metal between items that are not, against the LU oracle."""
import numpy as np
import pytest

from oracle import implicit_oracle as IM
from oracle import oracle as O
from paper_0901_1053_amd import inputs, tete
from tests import parity as P

pytestmark = pytest.mark.gpu

DZ = 1e-3
COARSE, MIDDLE, FINE = 8e-3, 2e-3, 0.3e-3     # dx = dy: 4 to about 90 iterations


# FP32 tiles own 38 rows, FP64 tiles 24; rows of 64 and 65 entries take one and
# two waves; chunks hold at most 64 planes
@pytest.mark.parametrize("shape,mesh,metal", [
    ((5, 37, 63), COARSE, False), ((4, 38, 64), MIDDLE, False), ((3, 23, 20), MIDDLE, False), ((3, 24, 20), FINE, False),
    ((3, 47, 9), FINE, False), ((3, 77, 5), MIDDLE, False), ((150, 5, 5), MIDDLE, True), ((63, 4, 70), MIDDLE, True),
    ((64, 4, 4), COARSE, False),
])
def test_passes_match_oracle(shape, mesh, metal):
    print("implicit passes", shape, mesh, metal, flush=True)
    nx, ny, nz = shape
    cells = inputs.random_cells(nx, ny, nz, 91, frac=0.1)
    if metal:
        cells[nx // 3:(5 * nx) // 6] = 1
    f0 = inputs.random_fields((nx + 1, ny + 1, nz + 1), 92)
    g = O.Geom(nx, ny, nz, mesh, 1.1 * mesh, DZ, DZ)
    m = O.vacuum_materials(g, cells)
    ref = {k: v.copy() for k, v in f0.items()}
    O.apply_pec(g, m, ref)
    S = IM.Implicit(g, m)
    for _ in range(7):
        S.step(ref)
    for precision, tol in (("fp64", 1e-12), ("fp32", 2e-5)):
        G = tete.Grid(nx, ny, nz, mesh, 1.1 * mesh, DZ, DZ, precision=precision, implicit=True)
        G.set_pec_cells(cells)
        G.set_fields(f0)
        G.step(7)
        got = G.get_fields()
        assert P.field_rel_err(got, ref) <= tol, precision
        # nothing is kept between solves: the same fields again, other steps between
        G.step(3)
        G.set_fields(f0)
        G.step(7)
        again = G.get_fields()
        for k in got:
            assert np.array_equal(got[k], again[k]), (precision, k)
        G.close()
