"""The two ways the implicit scheme's plane solves run: one iteration per launch over
lists of rows, and several per pass over work items of several planes (with a last
one cut short, and cut again where metal leaves few items).  A step is checked by
putting the state after it into the scheme's own equations (16): the error of the
solves is at most the residual, since (I - alpha T) does not shrink a vector in the
scheme's energy norm."""
import numpy as np
import pytest

from oracle import implicit_oracle as IM
from oracle import oracle as O
from paper_0901_1053_amd import inputs, tete

DZ = 1e-3
TOL = {"fp64": 1e-13, "fp32": 1e-5}    # about 50 roundings of sums of ten terms below 4


def _fwd(f, ax):
    d = np.zeros_like(f)
    lo, hi = [slice(None)] * 3, [slice(None)] * 3
    lo[ax], hi[ax] = slice(0, -1), slice(1, None)
    d[...] = -f
    d[tuple(lo)] += f[tuple(hi)]
    return d


def _bwd(f, ax):
    lo, hi = [slice(None)] * 3, [slice(None)] * 3
    lo[ax], hi[ax] = slice(0, -1), slice(1, None)
    d = -f
    d[tuple(hi)] += f[tuple(lo)]
    return d


def residual(m, cdt, f0, f1):
    """Largest residual of (16) over both half steps, by the largest field value."""
    a = 0.5 * cdt
    t0 = lambda f: {"hx": -m["hx"] * _fwd(f["ez"], 1), "hy": m["hy"] * _fwd(f["ez"], 0),
                    "ez": m["ez"] * (_bwd(f["hx"], 1) - _bwd(f["hy"], 0))}
    t1 = lambda f: {"ex": -m["ex"] * _bwd(f["hz"], 1), "ey": m["ey"] * _bwd(f["hz"], 0),
                    "hz": m["hz"] * (_fwd(f["ex"], 1) - _fwd(f["ey"], 0))}
    lv = {"hx": m["hx"] * _fwd(f0["ey"], 2), "hy": -m["hy"] * _fwd(f0["ex"], 2), "ez": 0.0}
    lu = {"ex": m["ex"] * _bwd(f1["hy"], 2), "ey": -m["ey"] * _bwd(f1["hx"], 2), "hz": 0.0}
    worst = 0.0
    for t, far in ((t0, lv), (t1, lu)):
        old, new = t(f0), t(f1)
        for k in old:
            r = (f1[k] - a * new[k]) - (f0[k] + a * old[k] + cdt * far[k])
            worst = max(worst, float(np.max(np.abs(r))))
    return worst / max(float(np.max(np.abs(v))) for v in f1.values())


def _cells(shape, metal):
    nx = shape[0]
    cells = inputs.random_cells(*shape, 93, frac=0.003)
    if metal:
        cells[int(nx * (1 - metal)):] = 1
    return cells


def _materials(shape, cells):
    return O.vacuum_materials(O.Geom(*shape, DZ, 1.1 * DZ, DZ, DZ), cells)


def test_residual_of_the_oracle():
    """The LU oracle's step leaves a residual of a few roundings, and a step wrong in one entry does not."""
    shape = (7, 6, 9)
    cells = inputs.random_cells(*shape, 94, frac=0.1)
    g = O.Geom(*shape, DZ, 1.1 * DZ, DZ, DZ)
    m = O.vacuum_materials(g, cells)
    f = inputs.random_fields(g.shape, 95)
    O.apply_pec(g, m, f)
    f0 = {k: v.copy() for k, v in f.items()}
    IM.Implicit(g, m).step(f)
    assert residual(m, g.cdt, f0, f) <= TOL["fp64"]
    f["hz"][3, 3, 4] += 1e-6
    assert residual(m, g.cdt, f0, f) >= 1e-7


# FP32 rows of 38, FP64 of 24 to a tile.  Passes: chunks of 2 planes, the last of 1;
# chunks of 6 (5) planes cut to 2 for the items that metal leaves; of 2 cut to 1.
# Lists of rows: the smallest grids, and grids with few iterations' worth of rows
@pytest.mark.gpu
@pytest.mark.parametrize("shape,precision,metal", [
    ((80, 60, 127), "fp32", 0), ((150, 100, 191), "fp32", 0.45), ((60, 60, 127), "fp32", 0),
    ((100, 36, 127), "fp64", 0), ((60, 140, 191), "fp64", 0.55), ((60, 60, 127), "fp64", 0),
    ((30, 26, 100), "fp32", 0), ((30, 26, 100), "fp64", 0.3), ((80, 80, 64), "fp64", 0), ((2, 2, 2), "fp32", 0),
])
def test_both_ways_solve_the_scheme(shape, precision, metal):
    print("implicit ways", shape, precision, metal, flush=True)
    cells = _cells(shape, metal)
    m = _materials(shape, cells)
    G = tete.Grid(*shape, DZ, 1.1 * DZ, DZ, DZ, precision=precision, implicit=True)
    G.set_pec_cells(cells)
    G.set_fields(inputs.random_fields(G.shape, 96))
    f0 = G.get_fields()
    for step in range(3):
        G.step(1)
        f1 = G.get_fields()
        assert residual(m, DZ, f0, f1) <= TOL[precision], step
        f0 = f1
    G.close()


# a grid whose geometry changes between one that takes passes and one that takes lists:
# neither way uses what the other left
@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_geometry_changes_the_way(precision):
    shape = (60, 60, 127)
    print("implicit geometry", precision, flush=True)
    G = tete.Grid(*shape, DZ, 1.1 * DZ, DZ, DZ, precision=precision, implicit=True)
    for metal in (0, 0.9, 0, 0.6):
        cells = _cells(shape, metal)
        m = _materials(shape, cells)
        G.set_pec_cells(cells)
        G.set_fields(inputs.random_fields(G.shape, 97))
        G.step(3)
        f0 = G.get_fields()
        G.step(1)
        assert residual(m, DZ, f0, G.get_fields()) <= TOL[precision], metal
    G.close()
