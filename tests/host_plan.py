"""The host-side launch choices of csrc/tete_plan.h, compiled by the host compiler
alone and called through ctypes."""
import ctypes as C
import functools
import os
import subprocess
import tempfile

import numpy as np

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_0901_1053_amd", "csrc")

SHIM = r'''
#include "tete_plan.h"
using namespace tete;
extern "C" {
int implicit(int real_bytes, int iters, int stages, int64_t rows, int64_t ie, int64_t ih, int xc)
{
    return implicit_passes(real_bytes, iters, stages, rows, ie, ih, xc);
}
int rz_rows(int nr1, int64_t nzt, int fp32) { return rz_chunk_rows(nr1, nzt, fp32 != 0); }
int rz_energy(int nr1, int64_t nzt) { return rz_energy_rows(nr1, nzt); }
void plan(int64_t tiles, int nplanes, int64_t xmax, int fill, int unroll, int tail, int* out)
{
    const ChunkPlan p = plan_chunks(tiles, nplanes, xmax, fill, unroll, tail != 0);
    const int v[6] = {p.xchunk, p.nxc, p.nfull, p.nblk, p.tsplit, p.tchunk};
    for (int q = 0; q < 6; ++q) out[q] = v[q];
}
int active(const int* next, int tiles, int planes, int xmax)
{
    return active_chunk(ActiveTiles{next, tiles, planes}, xmax);
}
int batch(const int64_t* tiles, const int* planes, int n, int grid, int cap, int fill, int* one)
{
    const BatchPlan p = plan_batch(tiles, planes, n, grid, cap, fill);
    *one = p.one_round;
    return p.chunk;
}
}
'''


@functools.lru_cache(maxsize=None)
def lib():
    d = tempfile.mkdtemp(prefix="tete_plan_")
    src, so = os.path.join(d, "shim.cpp"), os.path.join(d, "shim.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", so, src])
    L = C.CDLL(so)
    L.implicit.argtypes = [C.c_int] * 3 + [C.c_int64] * 3 + [C.c_int]
    L.rz_rows.argtypes = [C.c_int, C.c_int64, C.c_int]
    L.rz_energy.argtypes = [C.c_int, C.c_int64]
    L.plan.argtypes = [C.c_int64, C.c_int, C.c_int64, C.c_int, C.c_int, C.c_int, C.POINTER(C.c_int)]
    L.batch.argtypes = [C.POINTER(C.c_int64), C.POINTER(C.c_int), C.c_int, C.c_int, C.c_int, C.c_int, C.POINTER(C.c_int)]
    L.active.argtypes = [C.c_void_p] + [C.c_int] * 3
    return L


def active(on, xmax):
    """Planes per chunk for on[plane, tile], True where the tile is not static."""
    planes, tiles = on.shape
    nxt = np.full((planes + 1, tiles), planes, np.int32)
    for q in range(planes - 1, -1, -1):
        nxt[q] = np.where(on[q], q, nxt[q + 1])
    return lib().active(nxt.ctypes.data, tiles, planes, xmax)


def batch(members, grid, cap, fill):
    """(planes per chunk, one round) for members (tiles, planes)"""
    n, one = len(members), C.c_int()
    c = lib().batch((C.c_int64 * n)(*[m[0] for m in members]), (C.c_int * n)(*[m[1] for m in members]), n, grid, cap,
                    fill, C.byref(one))
    return c, bool(one.value)


def plan(tiles, nplanes, xmax, fill, unroll, tail):
    """(xchunk, nxc, nfull, nblk, tsplit, tchunk)"""
    out = (C.c_int * 6)()
    lib().plan(tiles, nplanes, xmax, fill, unroll, tail, out)
    return tuple(out)
