// Device helpers shared by the fused step kernels: raw buffer loads and
// stores, whole-wave lane shifts, the XCD-aware workgroup remap and the tile
// schedule.
#pragma once

#include <stdint.h>

#include <algorithm>

#include <hip/hip_runtime.h>

#include "tete_impl.h"
#include "tete_plan.h"

namespace tete {
namespace {

// Raw buffer load of one field value at byte offset off (vector) + soff
// (scalar); a lane whose off is past the buffer's size reads 0.
template <typename R>
__device__ __forceinline__ R bload(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff = 0);
template <>
__device__ __forceinline__ float bload<float>(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, soff, 0));
}
template <>
__device__ __forceinline__ double bload<double>(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff)
{
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, 0));
}
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
template <typename R>
__device__ __forceinline__ void bstore(__amdgpu_buffer_rsrc_t r, uint32_t off, R v);
template <>
__device__ __forceinline__ void bstore<float>(__amdgpu_buffer_rsrc_t r, uint32_t off, float v)
{
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, off, 0, 0);
}
template <>
__device__ __forceinline__ void bstore<double>(__amdgpu_buffer_rsrc_t r, uint32_t off, double v)
{
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, off, 0, 0);
}

// Neighbours along k are the neighbouring lanes of the wave: DPP whole-wave
// shifts by one lane (lane 0 / lane 63 receive 0; both are halo lanes).  The
// bound control writes the 0, so no register has to be cleared first.
__device__ __forceinline__ int dpp_prev(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xf, 0xf, true); }
__device__ __forceinline__ int dpp_next(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x130, 0xf, 0xf, true); }
__device__ __forceinline__ float lane_prev(float v) { return __builtin_bit_cast(float, dpp_prev(__builtin_bit_cast(int, v))); }
__device__ __forceinline__ float lane_next(float v) { return __builtin_bit_cast(float, dpp_next(__builtin_bit_cast(int, v))); }
typedef int i32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ double lane_prev(double v)
{
    i32x2 w = __builtin_bit_cast(i32x2, v);
    w.x = dpp_prev(w.x);
    w.y = dpp_prev(w.y);
    return __builtin_bit_cast(double, w);
}
__device__ __forceinline__ double lane_next(double v)
{
    i32x2 w = __builtin_bit_cast(i32x2, v);
    w.x = dpp_next(w.x);
    w.y = dpp_next(w.y);
    return __builtin_bit_cast(double, w);
}

// Logical tile of a workgroup.  Consecutive hardware workgroups are spread
// round-robin over the eight XCDs; the remap gives each XCD a contiguous range
// of logical tiles so that neighbouring j-tiles (which share halo rows) run on
// the same XCD and share its L2.
__device__ __forceinline__ int xcd_remap(int b, int n)
{
    const int nx = 8;
    int x = b % nx, r = b / nx;
    int base = n / nx, extra = n % nx;
    return x < extra ? x * (base + 1) + r : extra * (base + 1) + (x - extra) * base + r;
}

// The same for a launch whose workgroups fill a CU each: kRound of them run at
// a time, and the remap is taken within each round.  The running workgroups
// then cover one contiguous range of tiles (whole rows of neighbouring bands),
// an eighth of it per XCD.  With the range split over the whole launch the
// eight XCDs worked in eight distant bands: 4.14 against 3.90 ms per step on
// the 512 x 512 x 2048 grid in FP32 (k-tiles first), 7.44 against 7.00 ms in FP64.
__device__ __forceinline__ int xcd_rounds(int b, int n)
{
    const int r0 = b / kRound * kRound;
    return r0 + xcd_remap(b - r0, min(kRound, n - r0));
}

// Tile (ty, tz) and x-chunk cx of logical workgroup lb.  order 2: k-tiles
// fastest, so the tiles of one band of rows, which together cover whole
// contiguous rows, run together; order 1: j-tiles fastest; orders 3-6: blocks
// of BZ k-tiles by BY j-tiles (8 x 4, 16 x 2, 4 x 8, 2 x 16: 32 workgroups, one
// XCD's worth) fastest, so that neighbouring row bands, which share halo rows,
// also run together and share the XCD's L2.  Order 0 is order 2: with the
// rounds above it is the fastest (the blocks read up to 13 % fewer bytes but
// took 1 to 5 % longer, padded or not).  Returns false for the padding
// workgroups of the blocked orders.
__host__ __device__ __forceinline__ bool blocked_order(int order) { return order >= 3 && order <= 6; }
__host__ __device__ __forceinline__ int block_z(int order)
{
    return order == 3 ? 8 : order == 4 ? 16 : order == 5 ? 4 : 2;
}
__host__ __device__ __forceinline__ int block_y(int order) { return 32 / block_z(order); }
// Workgroups of one launch: tiles (padded to whole blocks for the blocked
// orders) times x-chunks.
__host__ __device__ __forceinline__ int launch_tiles(int order, int nyt, int nzt, int nxc)
{
    if (!blocked_order(order)) return nyt * nzt * nxc;
    const int BZ = block_z(order), BY = block_y(order);
    return ((nzt + BZ - 1) / BZ) * ((nyt + BY - 1) / BY) * BZ * BY * nxc;
}
__host__ __device__ __forceinline__ bool tile_of(int lb, int order, int nyt, int nzt, int& ty, int& tz, int& cx)
{
    if (order == 2) {
        tz = lb % nzt;
        ty = (lb / nzt) % nyt;
        cx = lb / (nzt * nyt);
        return true;
    }
    if (blocked_order(order)) {
        const int BZ = block_z(order), BY = block_y(order);
        const int nbz = (nzt + BZ - 1) / BZ, nby = (nyt + BY - 1) / BY;
        const int w = lb % (BZ * BY), b = lb / (BZ * BY);
        tz = (b % nbz) * BZ + w % BZ;
        ty = ((b / nbz) % nby) * BY + w / BZ;
        cx = b / (nbz * nby);
        return tz < nzt && ty < nyt;
    }
    ty = lb % nyt;
    tz = (lb / nyt) % nzt;
    cx = lb / (nyt * nzt);
    return true;
}

// A work item: tile (ty, tz), planes xs .. xe-1.
struct Tile {
    int ty, tz, xs, xe;
};

// Work item lb of a launch of A.nblk; false for an item without planes (the
// padding of the blocked orders, a tail item past the end of a short chunk).
template <typename R>
__device__ __forceinline__ bool tile_at(const FArgs<R>& A, int lb, Tile& t)
{
    int sub = -1;
    if (lb >= A.nfull) {
        const int ntail = (A.nblk - A.nfull) / A.tsplit, q = lb - A.nfull;
        sub = q / ntail;
        lb = A.nfull + q % ntail;
    }
    int cx;
    if (!tile_of(lb, A.order, A.nyt, A.nzt, t.ty, t.tz, cx)) return false;
    t.xs = cx * A.xchunk;
    t.xe = min(t.xs + A.xchunk, A.g.nx + 1);
    if (sub >= 0) {
        t.xs += sub * A.tchunk;
        t.xe = min(t.xs + A.tchunk, t.xe);
    }
    return t.xs < t.xe;
}

// Work item of an entry of a list of active tiles, (cx nyt + ty) nzt + tz.
template <typename R>
__device__ __forceinline__ Tile listed_tile(const FArgs<R>& A, int e)
{
    Tile t;
    t.tz = e % A.nzt;
    t.ty = (e / A.nzt) % A.nyt;
    t.xs = e / (A.nzt * A.nyt) * A.xchunk;
    t.xe = min(t.xs + A.xchunk, A.g.nx + 1);
    return t;
}

// Fills the tiling of A: the x-chunk asked for (clipped to xmax planes), or
// where xchunk is 0 the plan for a launch of this grid alone (plan_chunks).
template <typename R>
inline void set_chunks(FArgs<R>& A, int xchunk, int order, int64_t xmax, int fill, int unroll)
{
    A.order = order != 0 ? order : 2;
    const int nplanes = A.g.nx + 1, tiles = launch_tiles(A.order, A.nyt, A.nzt, 1);
    if (xchunk <= 0) {
        const ChunkPlan p = plan_chunks(tiles, nplanes, xmax, fill, unroll, !blocked_order(A.order));
        A.xchunk = p.xchunk;
        A.nxc = p.nxc;
        A.nfull = p.nfull;
        A.nblk = p.nblk;
        A.tsplit = p.tsplit;
        A.tchunk = p.tchunk;
        return;
    }
    A.xchunk = (int)std::min<int64_t>(xchunk, xmax);
    A.nxc = (nplanes + A.xchunk - 1) / A.xchunk;
    A.nblk = A.nfull = launch_tiles(A.order, A.nyt, A.nzt, A.nxc);
    A.tsplit = 1;
    A.tchunk = A.xchunk;
}

}  // namespace
}  // namespace tete
