"""The two-step kernel's march along x: chunk lengths that end it at every place
of its unrolled loop, tiles with and without the source row, against the
single-step kernel (materials by class: against one chunk), bitwise."""
import numpy as np
import pytest

from paper_0901_1053_amd import inputs, tete

pytestmark = pytest.mark.gpu

DZ = 1e-3
SHAPE = (25, 40, 70)


def _fields(orc, precision, kernel, xchunk, rows, bunch_row, classes):
    nx, ny, nz = SHAPE
    cells = inputs.random_cells(nx, ny, nz, 61)
    G = tete.Grid(nx, ny, nz, 2 * DZ, 2 * DZ, DZ, DZ, precision=precision, materials=classes)
    G.set_pec_cells(cells)
    if classes:
        g = orc.Geom(nx, ny, nz, 2 * DZ, 2 * DZ, DZ, DZ)
        vac = orc.vacuum_materials(g, cells)
        rng = np.random.default_rng(62)
        table = np.array([[vac[k].max() for k in inputs.KEYS]] * 4) * rng.uniform(0.6, 1.0, size=(4, 6))
        G.set_material_classes(rng.integers(0, 4, size=g.shape).astype(np.uint8), table)
    G.set_fields(inputs.random_fields(G.shape, 63))
    G.set_bunch(1e-9, 2.0 * DZ, nx // 2, bunch_row, 12, -90, 120)
    G.set_tuning(kernel, rows, xchunk, 0, 0)
    G.step(4)
    out = G.get_fields()
    out["wake"] = G.wake()
    G.close()
    return out


@pytest.mark.parametrize("precision,rows,classes", [("fp32", 16, False), ("fp32", 24, False), ("fp32", 32, False),
                                                    ("fp32", 0, True), ("fp64", 16, False), ("fp64", 0, True)])
def test_every_end_of_the_march(orc, precision, rows, classes):
    # bunch in the first rows, at the edge of two 16-row tiles, in a later tile
    for bunch_row in (2, 9, 33):
        base = _fields(orc, precision, "fused2" if classes else "fused", 10 ** 6, 0, bunch_row, classes)
        for xchunk in (1, 2, 3, 4, 5, 6, 13, 26):
            print("march", precision, rows, bunch_row, xchunk, flush=True)
            got = _fields(orc, precision, "fused2", xchunk, rows, bunch_row, classes)
            for k in base:
                assert np.array_equal(got[k], base[k]), (bunch_row, xchunk, k)
        assert np.any(base["wake"] != 0)


# one tile of 18 owned rows by 28 entries exactly, one more, two tiles; with and
# without the second state's sample
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("ny,nz,every", [(17, 27, 1), (18, 28, 2), (35, 55, 1), (36, 56, 2), (9, 83, 3)])
def test_energy_samples_at_tile_edges(precision, ny, nz, every):
    nx = 9
    print("energy tiles", precision, ny, nz, every, flush=True)
    out = []
    for kernel in ("fused2", "fused"):
        G = tete.Grid(nx, ny, nz, 2 * DZ, 2 * DZ, DZ, DZ, precision=precision, max_series=32)
        G.set_pec_cells(inputs.random_cells(nx, ny, nz, 64))
        G.set_fields(inputs.random_fields(G.shape, 65))
        G.set_tuning(kernel, 0, 0, 0, 0)
        G.set_diagnostics(every)
        G.step(9)
        out.append((G.energy_series(), G.get_fields()))
        G.close()
    a, b = out[0][0], out[1][0]
    assert len(a) == len(b) and np.max(np.abs(a - b)) <= 1e-13 * np.max(np.abs(b))   # FP64 sums of the same terms
    for k in out[0][1]:
        assert np.array_equal(out[0][1][k], out[1][1][k]), k


def _single(orc, precision, xchunk, bunch_row, arrays, shape):
    nx, ny, nz = shape
    cells = inputs.random_cells(nx, ny, nz, 66)
    G = tete.Grid(nx, ny, nz, 2 * DZ, 2 * DZ, DZ, DZ, precision=precision, materials=arrays)
    G.set_pec_cells(cells)
    if arrays:
        g = orc.Geom(nx, ny, nz, 2 * DZ, 2 * DZ, DZ, DZ)
        vac = orc.vacuum_materials(g, cells)
        rng = np.random.default_rng(67)
        G.set_materials({k: v * rng.uniform(0.6, 1.0, size=v.shape) for k, v in vac.items()})
    G.set_fields(inputs.random_fields(G.shape, 68))
    G.set_bunch(1e-9, 2.0 * DZ, nx // 2, bunch_row, 12, -90, 120)
    G.set_tuning("split" if xchunk < 0 else "fused", 0, max(xchunk, 0), 0, 0)
    G.step(3)
    out = G.get_fields()
    out["wake"] = G.wake()
    G.close()
    return out


# the single step: every end of its march, tiles of 8, 12 and 20 owned rows by 62
# and 30 entries; against the two-kernel step within 1e-12 / 2e-5, and bitwise
# between chunk lengths
@pytest.mark.parametrize("precision,arrays", [("fp32", False), ("fp64", False), ("fp32", True), ("fp64", True)])
@pytest.mark.parametrize("shape", [(25, 40, 70), (9, 19, 29), (9, 20, 61), (4, 41, 62)])
def test_every_end_of_the_single_step(orc, precision, arrays, shape):
    tol = 1e-12 if precision == "fp64" else 2e-5
    for bunch_row in (2, shape[1] // 2, shape[1] - 1):
        print("single march", precision, arrays, shape, bunch_row, flush=True)
        ref = _single(orc, precision, -1, bunch_row, arrays, shape)
        base = _single(orc, precision, 10 ** 6, bunch_row, arrays, shape)
        for k in ref:
            assert np.max(np.abs(base[k] - ref[k])) <= tol * max(np.max(np.abs(ref[k])), 1e-300), k
        for xchunk in (1, 2, 3, 4, 5, 6):
            got = _single(orc, precision, xchunk, bunch_row, arrays, shape)
            for k in base:
                assert np.array_equal(got[k], base[k]), (bunch_row, xchunk, k)


# 270 tiles of 16 rows are two rounds of workgroups, 162 of 24 rows one; 54 and 36
# tiles one round either way: the FP32 instances with 24 and with 16 rows
@pytest.mark.parametrize("shape", [(6, 95, 735), (6, 95, 150)])
@pytest.mark.parametrize("kind", ["energy", "arrays"])
def test_rows_of_the_larger_instances(orc, kind, shape):
    nx, ny, nz = shape
    print("16 or 24 rows", kind, shape, flush=True)
    cells = inputs.random_cells(nx, ny, nz, 81)
    out = []
    for kernel in ("fused2", "fused"):
        G = tete.Grid(nx, ny, nz, 2 * DZ, 2 * DZ, DZ, DZ, precision="fp32", materials=kind == "arrays", max_series=32)
        G.set_pec_cells(cells)
        if kind == "arrays":
            vac = orc.vacuum_materials(orc.Geom(nx, ny, nz, 2 * DZ, 2 * DZ, DZ, DZ), cells)
            rng = np.random.default_rng(82)
            G.set_materials({k: v * rng.uniform(0.6, 1.0, size=v.shape) for k, v in vac.items()})
        else:
            G.set_diagnostics(1)
        G.set_fields(inputs.random_fields(G.shape, 83))
        G.set_bunch(1e-9, 2.0 * DZ, nx // 2, 41, 12, -90, 120)
        G.set_tuning(kernel, 0, 10 ** 6, 0, 0)
        G.step(5)
        out.append((G.get_fields(), G.wake(), G.energy_series() if kind == "energy" else np.ones(1)))
        G.close()
    for k in out[0][0]:
        assert np.array_equal(out[0][0][k], out[1][0][k]), k
    assert np.array_equal(out[0][1], out[1][1])
    a, b = out[0][2], out[1][2]
    assert len(a) == len(b) and np.max(np.abs(a - b)) <= 1e-13 * np.max(np.abs(b))   # FP64 sums of the same terms
