"""Energy samples of FP32 pairs in tiles of 24 rows of 32 lanes (18 by 28 entries
owned), taken where 16 rows would need a second round of workgroups: grids cut
exactly at such tiles and one row or entry over, without and with witness lines,
against single steps: fields, wakes and lines bitwise, energies to their FP64
rounding."""
import numpy as np
import pytest

from paper_0901_1053_amd import inputs, tete

pytestmark = pytest.mark.gpu

DZ = 1e-3


@pytest.mark.parametrize("witness", [False, True])
@pytest.mark.parametrize("every", [1, 2, 3])
@pytest.mark.parametrize("ny,nz", [(89, 839), (90, 840), (89, 840), (90, 839)])
def test_24_rows_at_tile_edges(ny, nz, every, witness):
    nx = 7
    tiles = [((ny + r) // r) * ((nz + 28) // 28) for r in (10, 18)]
    assert tiles[0] > 256 >= tiles[1]      # two rounds of 16-row tiles, one of 24-row tiles
    print("24 rows", ny, nz, every, witness, flush=True)
    cells = inputs.random_cells(nx, ny, nz, 101)
    out = []
    for kernel in ("fused2", "fused"):
        G = tete.Grid(nx, ny, nz, 2 * DZ, 2 * DZ, DZ, DZ, precision="fp32", max_series=32)
        G.set_pec_cells(cells)
        G.set_fields(inputs.random_fields(G.shape, 102))
        G.set_bunch(1e-9, 2.0 * DZ, nx // 2, 54, 12, -90, 120)
        if witness:
            G.set_witness(nx // 2, 55)
        G.set_diagnostics(every)
        G.set_tuning(kernel, 0, 10 ** 6, 0, 0)
        G.step(9)
        out.append((G.get_fields(), G.energy_series(), [G.wake()] + (list(G.witness_wake()) if witness else [])))
        G.close()
    for k in tete.KEYS:
        assert np.array_equal(out[0][0][k], out[1][0][k]), k
    for a, b in zip(out[0][2], out[1][2]):
        assert np.array_equal(a, b) and np.any(a != 0)
    a, b = out[0][1], out[1][1]
    assert len(a) == len(b) and np.max(np.abs(a - b)) <= 1e-13 * np.max(np.abs(b))   # FP64 sums of the same terms
