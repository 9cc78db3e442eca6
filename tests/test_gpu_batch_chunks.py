"""Batches whose chunks are planned for all members: launches of one round and of
several, single steps and pairs, with a member that asks for its own chunk length,
each against the member stepped alone, bitwise."""
import numpy as np
import pytest

from paper_0901_1053_amd import inputs, tete

pytestmark = pytest.mark.gpu

DZ = 1e-3


def _grid(shape, precision, seed, xchunk, kernel):
    nx, ny, nz = shape
    G = tete.Grid(nx, ny, nz, 2 * DZ, 2 * DZ, DZ, DZ, precision=precision)
    G.set_pec_cells(inputs.random_cells(nx, ny, nz, seed))
    G.set_fields(inputs.random_fields(G.shape, seed + 1))
    G.set_bunch(1e-9, 2.0 * DZ, nx // 2, ny // 2, 12, -90, 120)
    if xchunk:
        G.set_tuning(kernel, 0, xchunk, 0, 0)
    return G


# a few tiles (one round of short chunks), one member of 117 FP32 tiles over 129
# planes (one round of long ones), several rounds; 5 steps: pairs and a single step
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("kernel", ["fused2", "fused"])
@pytest.mark.parametrize("shapes,xchunk", [([(30, 24, 70), (41, 9, 100), (2, 30, 20)], 0), ([(128, 128, 520)], 0),
                                           ([(128, 60, 300), (20, 95, 595), (75, 31, 130)], 0),
                                           ([(128, 60, 300), (60, 95, 595), (75, 31, 130)], 64)])
def test_members_equal_alone(precision, kernel, shapes, xchunk):
    print("batch chunks", precision, kernel, shapes, xchunk, flush=True)
    ref = []
    for i, s in enumerate(shapes):
        G = _grid(s, precision, 51 + i, 0, kernel)
        G.step(5)
        ref.append((G.get_fields(dtype=precision), G.wake()))
        G.close()
    B = tete.Batch(precision)
    B.set_launch(kernel=kernel)
    grids = [_grid(s, precision, 51 + i, xchunk if i == 0 else 0, kernel) for i, s in enumerate(shapes)]
    for i, G in enumerate(grids):
        B.set(i, G)
    B.step(5)
    for G, (f_ref, w_ref) in zip(grids, ref):
        f = G.get_fields(dtype=precision)
        for k in tete.KEYS:
            assert np.array_equal(f[k], f_ref[k]), k
        assert np.array_equal(G.wake(), w_ref)
    B.close()
    for G in grids:
        G.close()
