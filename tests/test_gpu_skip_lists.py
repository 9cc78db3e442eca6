"""The lists of active tiles of two-step launches: the count left out with the chunk
length the library chose equals the one derived from the oracle's PEC edges."""
import pytest

from paper_0901_1053_amd import inputs, tete
from tests.test_gpu_skip import _expected_static
from tests.test_gpu_skip_chunks import DZ, _cells

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("kind,shape", [("vacuum", (90, 25, 130)), ("metal", (40, 25, 130)), ("slab", (61, 35, 130)),
                                        ("post", (90, 35, 130)), ("post", (7, 35, 130)), ("post", (150, 95, 300))])
def test_tiles_left_out(precision, kind, shape):
    print("skip lists", precision, kind, shape, flush=True)
    nx, ny, nz = shape
    cells = _cells(kind, shape)
    G = tete.Grid(*shape, 2 * DZ, 2 * DZ, DZ, DZ, precision=precision, skip_static=True)
    G.set_pec_cells(cells)
    G.set_fields(inputs.random_fields(G.shape, 103))
    G.step(4)
    skipped, total = G.static_tiles()
    tiles = ((ny + 10) // 10) * ((nz + (60 if precision == "fp32" else 28)) // (60 if precision == "fp32" else 28))
    assert total % tiles == 0
    chunks = total // tiles
    xc = -(-(nx + 1) // chunks)
    assert -(-(nx + 1) // xc) == chunks
    assert (skipped, total) == tuple(_expected_static(shape, cells, precision, 0, xc))
    if kind in ("slab", "post"):
        assert skipped > 0
    G.close()
