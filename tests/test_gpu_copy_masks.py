"""Which entries tete_set_fields and tete_rz_set_fields keep, against masks from the
cells and materials on the host: grids small enough for one entry per thread and
large enough for two and four, counts that leave a remainder, caller arrays on and
off 16-byte alignment, every pair of types."""
import numpy as np
import pytest

from oracle import oracle as O
from oracle import rz_oracle as Z
from paper_0901_1053_amd import inputs, tete
from tests.test_gpu_copy import TD, _offset

pytestmark = pytest.mark.gpu

DZ = 1e-3


def _case(kind, shape, precision):
    """A grid, its keys, fields to set and the entries that are kept (bool per key)."""
    if kind == "rz":
        nr, nz, mode = shape
        G = tete.RZGrid(nr, nz, 1.25 * DZ, DZ, DZ, mode, precision=precision)
        cells = inputs.rz_random_cells(nr, nz, 81)
        G.set_pec_cells(cells)
        g = Z.RZGeom(nr, nz, 1.25 * DZ, DZ, DZ, mode)
        one = {k: np.ones(G.shape) for k in tete.RZ_KEYS}
        Z.apply_pec(g, Z.materials(g, cells), one)
        return G, tete.RZ_KEYS, inputs.rz_random_fields(G.shape, 82), {k: v != 0 for k, v in one.items()}
    G = tete.Grid(*shape, 2 * DZ, 2 * DZ, DZ, DZ, precision=precision, materials=kind == "mat")
    cells = inputs.random_cells(*shape, 81)
    G.set_pec_cells(cells)
    m = O.vacuum_materials(O.Geom(*shape, 2 * DZ, 2 * DZ, DZ, DZ), cells)
    if kind == "mat":
        rng = np.random.default_rng(83)
        m = {k: 0.5 * v for k, v in m.items()}
        for k in tete.KEYS[:3]:
            m[k][rng.random(G.shape) < 0.2] = 0.0
        G.set_materials(m)
    return G, tete.KEYS, inputs.random_fields(G.shape, 82), {k: v != 0 for k, v in m.items()}


# entries: 27 to a few hundred; past 2^20, where two and four a thread begin, with
# remainders modulo four of 3, 0, 2 and 1 (the last at 2^20 + 1)
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("dtype", ["fp32", "fp64"])
@pytest.mark.parametrize("kind,shape", [
    ("vac", (2, 2, 2)), ("vac", (4, 3, 6)), ("mat", (4, 3, 6)), ("vac", (100, 100, 102)), ("mat", (100, 100, 102)),
    ("vac", (5, 9, 17500)), ("rz", (2, 2, 0)), ("rz", (6, 11, 1)), ("rz", (1029, 1018, 0)), ("rz", (16, 61680, 1)),
])
def test_kept_entries(kind, shape, precision, dtype):
    import torch as t
    print("kept entries", kind, shape, precision, dtype, flush=True)
    td = {"fp32": t.float32, "fp64": t.float64}[dtype]
    G, keys, f, kept = _case(kind, shape, precision)
    f = {k: np.where(v == 0, 1.0, v).astype(TD[dtype]) for k, v in f.items()}
    want = {k: np.where(kept[k], f[k].astype(TD[precision]).astype(TD[dtype]), 0) for k in keys}
    get = "tete_rz_get_fields" if kind == "rz" else "tete_get_fields"
    put = "tete_rz_set_fields" if kind == "rz" else "tete_set_fields"
    code = tete.FP32 if dtype == "fp32" else tete.FP64
    for off in (0, 1):
        src = [_offset(t, f[k], td, off * (1 + c % 3)) for c, k in enumerate(keys)]
        tete._chk(put, getattr(tete.load(), put)(G.h, tete.P6(*[a.data_ptr() for a in src]), code))
        dst = [_offset(t, np.full(G.np, 7.0), td, off * (1 + c % 2)) for c in range(6)]
        tete._chk(get, getattr(tete.load(), get)(G.h, tete.P6(*[a.data_ptr() for a in dst]), code))
        t.cuda.synchronize()
        for k, a in zip(keys, dst):
            assert np.array_equal(a.cpu().numpy().reshape(G.shape), want[k]), (off, k)
    G.close()
