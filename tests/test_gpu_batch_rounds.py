"""Two-step batch launches of several rounds of workgroups: members of uneven
length along x, a last round that is full, nearly empty or the only one, a member
with its own chunk length, and batches on both sides of the chunk length's rule,
each against the member stepped alone, bitwise."""
import numpy as np
import pytest

from paper_0901_1053_amd import inputs, tete

pytestmark = pytest.mark.gpu

DZ = 1e-3


def _grid(shape, precision, seed, xchunk):
    nx, ny, nz = shape
    G = tete.Grid(nx, ny, nz, 2 * DZ, 2 * DZ, DZ, DZ, precision=precision)
    G.set_pec_cells(inputs.random_cells(nx, ny, nz, seed))
    G.set_fields(inputs.random_fields(G.shape, seed + 1))
    G.set_bunch(1e-9, 2.0 * DZ, nx // 2, ny // 2, 12, -90, 120)
    if xchunk:
        G.set_tuning("fused2", 0, xchunk, 0, 0)
    return G


# tiles of 10 rows by 60 (FP32) or 28 (FP64) entries: 100 tiles each in the first
# two (several rounds), 128 each (full rounds only), 257 (one item in the second
# round), a few (a part of one round)
@pytest.mark.parametrize("precision,ny,nz,nxs,xchunk", [
    ("fp32", 95, 595, (3, 30, 7, 19, 11, 24, 2, 15, 9), 0), ("fp64", 95, 275, (3, 30, 7, 19, 11, 24, 2, 15, 9), 0),
    ("fp32", 95, 595, (17, 5, 12), 4), ("fp32", 79, 959, (8, 8, 8, 8), 0), ("fp32", 9, 257 * 60 - 1, (6,), 0),
    ("fp64", 9, 40, (70, 3), 0),
    # 2040 and 2060 tiles: chunks of at most 48 and of at most 24 planes
    ("fp32", 9, 1020 * 60 - 1, (50, 3), 0), ("fp32", 9, 1030 * 60 - 1, (50, 3), 0),
])
def test_rounds_equal_alone(precision, ny, nz, nxs, xchunk):
    print("batch rounds", precision, ny, nz, nxs, flush=True)
    ref = []
    for i, nx in enumerate(nxs):
        G = _grid((nx, ny, nz), precision, 71 + i, 0)
        G.step(5)
        ref.append((G.get_fields(dtype=precision), G.wake()))
        G.close()
    B = tete.Batch(precision)
    grids = [_grid((nx, ny, nz), precision, 71 + i, xchunk if i == 1 else 0) for i, nx in enumerate(nxs)]
    for i, G in enumerate(grids):
        B.set(i, G)
    B.step(5)
    for G, (f_ref, w_ref) in zip(grids, ref):
        f = G.get_fields(dtype=precision)
        for k in tete.KEYS:
            assert np.array_equal(f[k], f_ref[k]), k
        assert np.array_equal(G.wake(), w_ref)
