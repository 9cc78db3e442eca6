"""The cross-section's potential at the sizes where its iterations change their
kernel (one workgroup with 4, 7, 10, 14 or 17 nodes per thread, or one launch per
sub-step): the pipe state against the oracle's, every entry within 1e-12 of the
largest (the device iterates to a residual of 1e-16, the oracle factorises)."""
import numpy as np
import pytest

from oracle import oracle as O
from oracle import pipe_oracle as PO
from paper_0901_1053_amd import tete

pytestmark = pytest.mark.gpu

DZ = 1e-3


# nodes (nx + 1)(ny + 1): 9, 4096, 4097, 7168, 7169, 10240, 10241, 14336, 14337,
# 17408, 17536; rows of 511 and 512 nodes
@pytest.mark.parametrize("nx,ny", [(2, 2), (63, 63), (16, 240), (63, 111), (66, 106), (63, 159), (76, 132), (111, 127),
                                   (80, 176), (127, 135), (127, 136), (7, 510), (7, 511)])
def test_potential_at_the_plane_sizes(nx, ny):
    print("pipe plane", nx, ny, flush=True)
    nz, M, n0, src = 8, 3, 4, (nx // 2, ny // 2)
    g = O.Geom(nx, ny, nz, 2 * DZ, 1.8 * DZ, DZ, DZ)
    cells = np.zeros((nx, ny, nz), np.uint8)
    if nx > 8 and ny > 8:
        cells[:2, :5] = 1
        cells[nx - 2:, ny - 4:] = 1
    m = O.vacuum_materials(g, cells)
    phi = PO.potential(g, PO.pec_nodes(m), *src)
    ref = PO.self_field(g, m, phi, O.bunch_cells(1e-9, 1.5 * DZ, DZ, M), M, n0)
    G = tete.Grid(nx, ny, nz, g.dx, g.dy, g.dz, g.cdt, precision="fp64")
    G.set_pec_cells(cells)
    G.set_bunch(1e-9, 1.5 * DZ, src[0], src[1], M, -M, 20)
    it = G.set_open_pipes(n0)
    assert 0 < it <= 20 * (nx + ny) + 1000
    f = G.get_fields()
    scale = max(np.abs(ref[k]).max() for k in tete.KEYS)
    for k in tete.KEYS:
        assert np.abs(f[k] - ref[k]).max() <= 1e-12 * scale, k
