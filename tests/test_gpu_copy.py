"""Fields in and out of the library (four entries per thread, 16-byte accesses
where the caller's arrays allow them): caller arrays off 16-byte alignment,
entry counts that leave 1, 2 and 3 entries over, every pair of types."""
import numpy as np
import pytest

from paper_0901_1053_amd import inputs, tete

pytestmark = pytest.mark.gpu

DZ = 1e-3
TD = {"fp32": np.float32, "fp64": np.float64}


def _grid(kind, shape, precision):
    if kind == "rz":
        G = tete.RZGrid(shape[0], shape[1], 1.25 * DZ, DZ, DZ, shape[2], precision=precision)
        G.set_pec_cells(inputs.rz_random_cells(shape[0], shape[1], 71))
        return G, tete.RZ_KEYS, inputs.rz_random_fields(G.shape, 72)
    G = tete.Grid(*shape, 2 * DZ, 2 * DZ, DZ, DZ, precision=precision, materials=kind == "mat")
    cells = inputs.random_cells(*shape, 71)
    G.set_pec_cells(cells)
    f = inputs.random_fields(G.shape, 72)
    if kind == "mat":
        vac = (DZ / DZ ** 2, DZ / DZ ** 2, DZ / (2 * DZ) ** 2)
        m = {}
        rng = np.random.default_rng(73)
        for c, k in enumerate(tete.KEYS):
            m[k] = 0.4 * vac[c % 3] * (0.5 + 0.5 * rng.random(G.shape))
        for k in tete.KEYS[:3]:
            m[k][rng.random(G.shape) < 0.2] = 0.0
        G.set_materials(m)
    return G, tete.KEYS, f


def _offset(t, a, dtype, off):
    """A device copy of a that starts off elements past an aligned address."""
    buf = t.zeros(a.size + 8, dtype=dtype, device="cuda:0")
    buf[off:off + a.size] = t.from_numpy(np.ascontiguousarray(a).reshape(-1)).to("cuda:0", dtype)
    return buf[off:off + a.size]


# np mod 4: 1 (5*3*5), 2 (5*3*6), 3 (3*5*9), 0 (4*6*5); a single thread's worth (3*3*3 = 27)
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("dtype", ["fp32", "fp64"])
@pytest.mark.parametrize("kind,shape", [("vac", (4, 2, 4)), ("vac", (4, 2, 5)), ("vac", (2, 4, 8)), ("vac", (3, 5, 4)),
                                        ("vac", (2, 2, 2)), ("mat", (4, 2, 5)), ("mat", (6, 7, 40)),
                                        ("rz", (2, 2, 0)), ("rz", (4, 6, 1)), ("rz", (6, 4, 0)), ("rz", (30, 70, 2))])
def test_unaligned_fields(kind, shape, precision, dtype):
    import torch as t
    td = {"fp32": t.float32, "fp64": t.float64}[dtype]
    G, keys, f = _grid(kind, shape, precision)
    f = {k: v.astype(TD[dtype]) for k, v in f.items()}
    G.set_fields(f, dtype=dtype)
    want = G.get_fields(dtype=dtype)
    # kept entries come back as given (rounded to the grid's type), the others as zero
    for k in keys:
        kept = want[k] != 0
        assert np.array_equal(want[k][kept], f[k].astype(TD[precision]).astype(TD[dtype])[kept]), k
        assert kept.any() or min(shape[:2]) == 2, k
    G.set_fields({k: np.zeros_like(v) for k, v in f.items()}, dtype=dtype)
    get = "tete_rz_get_fields" if kind == "rz" else "tete_get_fields"
    put = "tete_rz_set_fields" if kind == "rz" else "tete_set_fields"
    code = tete.FP32 if dtype == "fp32" else tete.FP64
    src = [_offset(t, f[k], td, 1 + c % 3) for c, k in enumerate(keys)]
    tete._chk(put, getattr(tete.load(), put)(G.h, tete.P6(*[a.data_ptr() for a in src]), code))
    dst = [_offset(t, np.full(G.np, 7.0), td, 1 + c % 2) for c in range(6)]
    tete._chk(get, getattr(tete.load(), get)(G.h, tete.P6(*[a.data_ptr() for a in dst]), code))
    t.cuda.synchronize()
    for k, a in zip(keys, dst):
        assert np.array_equal(a.cpu().numpy().reshape(G.shape), want[k]), k
    G.close()
