"""Single steps of grids that leave out static tiles: the list's chunks fill the CUs
as those of the full launch do, of at most 32 planes, and the steps equal those of
every tile, bitwise."""
import numpy as np
import pytest

from paper_0901_1053_amd import inputs, tete
from tests import host_plan

pytestmark = pytest.mark.gpu

DZ = 1e-3


def _cells(shape):
    """A pipe along z: metal outside a few rows and entries about the middle."""
    nx, ny, nz = shape
    c = np.ones(shape, np.uint8)
    c[nx // 4:nx - nx // 4, ny // 2 - 3:ny // 2 + 3] = 0
    return c


# owned rows and entries of a tile: FP32 12 x 62, FP64 8 x 62 from PEC codes, 20 x 30
# with materials; grids of fewer tiles than CUs, of one plane's chunk and of several
# rounds
@pytest.mark.parametrize("precision,arrays,rows,lanes", [("fp32", False, 12, 62), ("fp64", False, 8, 62),
                                                         ("fp32", True, 12, 62), ("fp64", True, 20, 30)])
@pytest.mark.parametrize("shape", [(40, 40, 100), (64, 25, 64), (5, 30, 40), (70, 95, 250)])
def test_lists_of_single_steps(orc, precision, arrays, rows, lanes, shape):
    print("skip single", precision, arrays, shape, flush=True)
    nx, ny, nz = shape
    cells = _cells(shape)
    out = []
    for skip in (True, False):
        G = tete.Grid(*shape, 2 * DZ, 2 * DZ, DZ, DZ, precision=precision, materials=arrays, skip_static=skip)
        G.set_pec_cells(cells)
        if arrays:
            vac = orc.vacuum_materials(orc.Geom(*shape, 2 * DZ, 2 * DZ, DZ, DZ), cells)
            rng = np.random.default_rng(98)
            G.set_materials({k: v * rng.uniform(0.6, 1.0, size=v.shape) for k, v in vac.items()})
        G.set_fields(inputs.random_fields(G.shape, 99))
        G.set_bunch(1e-9, 2.0 * DZ, nx // 2, ny // 2, 12, -90, 120)
        G.set_tuning("fused", 0, 0, 0, 0)
        G.step(7)
        out.append((G.get_fields(), G.wake()))
        if skip:
            tiles = ((ny + rows) // rows) * ((nz + lanes) // lanes)
            chunks = host_plan.plan(tiles, nx + 1, 32, 6, 1, 1)[1]
            skipped, total = G.static_tiles()
            assert total == tiles * chunks and 0 <= skipped < total
            assert chunks * 32 >= nx + 1 and (tiles * chunks > 128 or chunks == nx + 1)
        G.close()
    for k in tete.KEYS:
        assert np.array_equal(out[0][0][k], out[1][0][k]), k
    assert np.array_equal(out[0][1], out[1][1])
