// Fused explicit TE/TM step (scheme (23), the ten sub-updates of Sec. 4.2) in
// one kernel, for vacuum cells with staircase PEC codes.
//
// Work decomposition.  A workgroup owns a tile of TY rows (j) by 62 entries
// (k) of the grid and marches along x through a chunk of planes.  Each wave is
// one j-row of 64 consecutive k (lanes), the tile plus a halo of one k below
// and one above; the workgroup holds TY + 4 rows, the tile plus a halo of two
// rows below and two above.  Along k, neighbours come from lane shuffles;
// along j, from LDS; along x, from registers, because the march visits the
// planes in order.  Every value of the step is therefore computed in
// registers and each field entry is read once from HBM and written once.
//
// The ten sub-updates form a pipeline over the planes.  With old data of plane
// p loaded at iteration p, the sub-updates run at plane lags
//   S1 (h_x^n)          p        S2 (h_y^n)        p-1    S3 (e_z^{n+1/2}) p-1
//   S4 (h_x^{n+1/2})    p-2      S5 (h_y^{n+1/2})  p-2
//   S6 (e_x^{n+1/2})    p-2      S7 (e_y^{n+1/2})  p-2    S8 (h_z^{n+1})   p-3
//   S9 (e_x^{n+1})      p-4      S10 (e_y^{n+1})   p-3
// chosen so that every j-neighbour a sub-update needs was produced in an
// earlier iteration (or loaded in this one): one LDS write phase and a single
// barrier per plane suffice, with the LDS double-buffered by plane parity.
// The halo rows, halo lanes and the first planes of a chunk compute values
// that are never stored; only the tile's own entries are written.

#include <algorithm>
#include <vector>

#include "tete_stage.h"

namespace tete {
namespace {

// k entries owned per row of lw lanes (two halo lanes)
__host__ __device__ constexpr int owned_k(int lw) { return lw - 2; }

// LDS of one workgroup: six double-buffered j-exchange planes of TYH + 2 rows.
template <typename R, int TYH, int LW = 64>
struct Lds {
    R x[6][2][TYH + 2][LW];
};

// Per-entry materials (kappa_x, kappa_y, kappa_z, mu_x, mu_y, mu_z arrays,
// zero on PEC edges and outside each component's range) for the MAT instance.
template <typename R>
struct MatA {
    const R* m[6];
};

// One work item (tile and x-chunk) of one step of the grid described by A.
// Every thread of the workgroup must call it (it contains barriers).  MAT:
// the coefficients come from the per-entry arrays of MA, loaded with the
// fields of each plane and carried to the lags where the sub-updates use them
// (kappa_z to p-1, mu_x to p-2, mu_y to p-2, kappa_y to p-3, mu_z to p-3,
// kappa_x to p-4), instead of the vacuum scalars and the PEC codes.
//
// What bounds it: memory, if the vector instructions stay few.  As in the
// two-step kernel plane addresses are scalar (a buffer resource per access, whose
// range is 0 for a plane without data or outside the chunk), LDS slots are
// immediate offsets from two bases, the march is unrolled by whole turns of the
// prefetch buffers and leaves at its exact end, PEC masks are a bit-field extract
// and an and, only a tile that holds the source row tests for it, and material
// coefficients are multiplied by a or 2a once, when their plane is taken.  us per
// launch before and after: materials FP64 160 x 160 x 640 673 (12 rows of 64 lanes)
// and 589, 4.1 TB/s of fields and coefficients; vacuum FP64 256 x 256 x 512 787 and
// 777 (16 rows, one plane ahead: 949 and 806), FP32 436 and 435.
template <typename R, int TYH, int PD, bool MAT = false, int LW = 64>
__device__ __forceinline__ void fused_tile(const FArgs<R>& A, const Tile& t, Lds<R, TYH, LW>& L,
                                           const MatA<R>& MA = MatA<R>{})
{
    constexpr int TY = TYH - 4, KT = owned_k(LW);
    // Lane shifts act on the whole wave; with two rows per wave (LW = 32) the
    // shift across the row boundary only feeds halo lanes.
    const Geo g = A.g;

    const int kl = threadIdx.x % LW;
    const int jl = threadIdx.x / LW;
    const int j = t.ty * TY - 2 + jl;
    const int k = t.tz * KT - 1 + kl;
    const bool jin = (unsigned)j <= (unsigned)g.ny;
    const bool kin = (unsigned)k <= (unsigned)g.nz;
    const bool node = jin && kin;
    const bool owned = node && jl >= 2 && jl < 2 + TY && kl >= 1 && kl <= KT;
    const int roff = k + j * g.sz;

    // index-range masks of the h components in j and k; along x they need none:
    // outside their range every e their update reads is 0
    const bool hx_jk = node && j < g.ny && k < g.nz;
    const bool hy_k = node && k < g.nz;
    const bool hz_j = node && j < g.ny;

    const int xs = t.xs, xe = t.xe;
    const int xload_end = min(xe + 1, g.nx);    // last plane whose old data is needed
    const int pb = max(0, xs - 2);              // first one

    const R a = A.a, a2 = A.a + A.a;
    const bool src_row = A.src.on && (LW == 64 ? __builtin_amdgcn_readfirstlane(j) : j) == A.src.j0;

    constexpr uint32_t RB = sizeof(R);
    constexpr uint32_t OOB = 0x80000000u;
    const uint32_t plane_bytes = (uint32_t)g.sp * RB;      // below 2^31 (fused_fits)
    auto mk = [](const void* base, int64_t off, uint32_t bytes) {
        return __builtin_amdgcn_make_buffer_rsrc((char*)const_cast<void*>(base) + off, (short)0, (int)bytes, 0x00020000);
    };
    const uint32_t in_ld = (uint32_t)roff * RB;
    const uint32_t vld = node ? in_ld : OOB, vcode = node ? (uint32_t)roff : OOB, vst = owned ? in_ld : OOB;
    auto xown = [&](int q) { return q >= xs && q < xe; };
    auto has_old = [&](int q) { return q >= pb && q <= xload_end; };
    auto st = [&](R* base, int q, R v) {
        bstore(mk(base, (int64_t)q * plane_bytes, xown(q) ? plane_bytes : 0u), vst, v);
    };
    const uint32_t cfix = node ? 0u : 7u;              // outside the grid: PEC

    // Prefetch: the old data of planes p+1 .. p+PD are in flight while plane p
    // is processed.  The PD+1 plane buffers are used round-robin by the unrolled
    // loop, so a buffer that a load is writing is never copied (a copy would
    // have to wait for that load).
    struct PR {
        R ex, ey, ez, hx, hy, hz;
        uint32_t c;
        R m[MAT ? 6 : 1];
    };
    auto load_plane = [&](int i, PR& d) {
        const bool pv = has_old(i);
        const uint32_t nb = pv ? plane_bytes : 0u;
        const int64_t po = (int64_t)i * plane_bytes;
        d.ex = bload<R>(mk(A.ex, po, nb), vld);
        d.ey = bload<R>(mk(A.ey, po, nb), vld);
        d.ez = bload<R>(mk(A.ez, po, nb), vld);
        d.hx = bload<R>(mk(A.hx, po, nb), vld);
        d.hy = bload<R>(mk(A.hy, po, nb), vld);
        d.hz = bload<R>(mk(A.hz, po, nb), vld);
        if constexpr (MAT) {
#pragma unroll
            for (int c = 0; c < 6; ++c) d.m[c] = bload<R>(mk(MA.m[c], po, nb), vld);
            d.c = 0u;
        } else {
            d.c = __builtin_amdgcn_raw_buffer_load_b8(mk(A.code, (int64_t)i * g.sp, pv ? (uint32_t)g.sp : 0u), vcode, 0, 0);
        }
    };

    Stage<R> S = {};
    uint32_t ch = 0x7777u;       // PEC codes of planes p-1 .. p-4, four bits each
    // carried coefficients of the MAT instance, multiplied by a or 2a (index:
    // planes behind p)
    R KXc[MAT ? 5 : 1] = {}, KYc[MAT ? 4 : 1] = {}, KZc[MAT ? 2 : 1] = {}, MXc[MAT ? 3 : 1] = {}, MYc[MAT ? 3 : 1] = {},
      MZc[MAT ? 4 : 1] = {};
    const R amx = hx_jk ? a * A.mx : R(0), amy = hy_k ? a * A.my : R(0), a2mz = hz_j ? a2 * A.mz : R(0);
    const R akx = a * A.kx, aky = a * A.ky, a2kz = a2 * A.kz;

    // exchange slot of quantity q, parity s, row jl + r
    typedef __attribute__((address_space(3))) R* LP;
    LP lp0 = (LP)&L.x[0][0][0][0] + threadIdx.x, lp1 = lp0 + 65536 / sizeof(R);
    asm("" : "+v"(lp0));
    asm("" : "+v"(lp1));
    auto ex = [&](int q, int s, int r) -> LP {
        const int off = ((2 * q + s) * (TYH + 2) + r) * LW;
        return off * (int)sizeof(R) < 65536 ? lp0 + off : lp1 + (off - 65536 / (int)sizeof(R));
    };

    PR buf[PD + 1];
#pragma unroll
    for (int d = 0; d < PD; ++d) load_plane(xs - 2 + d, buf[d]);

    const int pend = xe + 3;
    auto body = [&](auto src_tile, const int p, const int s, const PR& cur, PR& nxt) {
        constexpr bool SRC = decltype(src_tile)::value;
        load_plane(p + PD, nxt);
        if constexpr (MAT) {
            KXc[0] = a * cur.m[0]; KYc[0] = a * cur.m[1]; KZc[0] = a2 * cur.m[2];
            MXc[0] = a * cur.m[3]; MYc[0] = a * cur.m[4]; MZc[0] = a2 * cur.m[5];
        }
        // outside the grid, or a plane without old data: PEC on all edges
        const uint32_t c0 = (cur.c & 7u) | cfix | (has_old(p) ? 0u : 7u);

        // j-exchange through LDS (row r of the tile is LDS row r+1).  Rows 0 and
        // TYH+1 are never written: what they hold reaches only rows 0, 1,
        // TYH-2 and TYH-1 of the tile, which are never stored.
        *ex(0, s, 1) = cur.ez;
        *ex(1, s, 1) = S.hxn_m1;
        *ex(2, s, 1) = S.ezh_m2;
        *ex(3, s, 1) = S.HZm2;
        *ex(4, s, 1) = S.exh_m3;
        *ex(5, s, 1) = S.hzn_m4;
        __syncthreads();
        const Nb<R> nb = {*ex(0, s, 2), *ex(1, s, 0), *ex(2, s, 2), *ex(3, s, 0), *ex(4, s, 2), *ex(5, s, 0)};

        Co<R> f;
        if constexpr (MAT) {
            f.mx0 = MXc[0]; f.mx2 = MXc[2]; f.my1 = MYc[1]; f.my2 = MYc[2]; f.mz3 = MZc[3];
            f.kz1 = KZc[1]; f.ky2 = KYc[2]; f.kx2 = KXc[2]; f.ky3 = KYc[3]; f.kx4 = KXc[4];
        } else {
            f.mx0 = f.mx2 = amx;
            f.my1 = f.my2 = amy;
            f.mz3 = a2mz;
            f.kz1 = sel_free<2>(ch, a2kz);
            f.ky2 = sel_free<5>(ch, aky);
            f.kx2 = sel_free<4>(ch, akx);
            f.ky3 = sel_free<9>(ch, aky);
            f.kx4 = sel_free<12>(ch, akx);
        }
        // S3 of the source plane: the bunch current of step n on edge k, rounded
        // on its own before it is subtracted
        const bool src = SRC && src_row && p - 1 == A.src.i0 && kin && k < g.nz;
        R inj = 0;
        if (src) {
            const int64_t m = (int64_t)k - A.src.n + A.src.M;   // cell m crosses edge k in step n
            if (m >= -A.src.M && m <= A.src.M) {
#pragma clang fp contract(off)
                R kz;
                if constexpr (MAT) kz = MA.m[2][(int64_t)(p - 1) * g.sp + roff];
                else kz = sel_free<2>(ch, A.kz);
                inj = (R)((double)kz * A.src.lam[m + A.src.M]);
            }
        }
        const Out<R> o = stage_plane<SRC>(S, In<R>{cur.ex, cur.ey, cur.ez, cur.hx, cur.hy, cur.hz}, nb, f, inj);
        if (src && owned && xown(p - 1) && k < A.src.kend) {
            const int64_t js = A.src.n - k - A.src.M;      // wake sample of edge k
            if (js >= A.src.jmin && js < (int64_t)A.src.jmin + A.src.nw)
                A.src.wacc[js - A.src.jmin] += -0.5 * ((double)o.ezold1 + (double)o.ezh1);
        }

        st(A.ez1, p - 1, o.ezh1);
        st(A.hx1, p - 2, o.hxh2);
        st(A.hy1, p - 2, o.hyh2);
        st(A.hz1, p - 3, o.hzn3);
        st(A.ey1, p - 3, o.ey13);
        st(A.ex1, p - 4, o.ex14);

        ch = (ch << 4) | c0;
        if constexpr (MAT) {
#pragma unroll
            for (int d = 4; d > 0; --d) KXc[d] = KXc[d - 1];
#pragma unroll
            for (int d = 3; d > 0; --d) { KYc[d] = KYc[d - 1]; MZc[d] = MZc[d - 1]; }
#pragma unroll
            for (int d = 2; d > 0; --d) { MXc[d] = MXc[d - 1]; MYc[d] = MYc[d - 1]; }
            KZc[1] = KZc[0];
        }
    };

    constexpr int U = PD == 2 ? 6 : PD == 1 && sizeof(R) == 8 ? 2 : 4;
    static_assert(U % 2 == 0 && U % (PD + 1) == 0, "whole turns of the parity and of the prefetch buffers");
    auto march = [&](auto src_tile) {
        int p = xs - 2;
        for (;;) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                body(src_tile, p, u & 1, buf[u % (PD + 1)], buf[(u + PD) % (PD + 1)]);
                if (p++ == pend) return;
            }
        }
    };
    const int srow = A.src.j0 - (t.ty * TY - 2);
    if (A.src.on && srow >= 0 && srow < TYH) march(std::true_type{});
    else march(std::false_type{});
}

// One step of one grid: one workgroup per (tile, x-chunk).
template <typename R, int TYH, int PD>
__global__ __launch_bounds__(64 * TYH) void k_fused(FArgs<R> A, const int* act)
{
    __shared__ Lds<R, TYH> L;
    Tile t;
    if (act) t = listed_tile(A, act[xcd_rounds(blockIdx.x, gridDim.x)]);   // the active tiles only
    else if (!tile_at(A, xcd_rounds(blockIdx.x, A.nblk), t)) return;       // whole group
    fused_tile<R, TYH, PD>(A, t, L);
}

// The same step with per-entry materials.  act (or null): the tiles that are
// not static, (cx nyt + ty) nzt + tz in the launch's tile order
// (fused_static_tiles), one workgroup each, remapped over the XCDs.
template <typename R, int TYH, int LW, int PD>
__global__ __launch_bounds__(LW * TYH) void k_fused_mat(FArgs<R> A, MatA<R> MA, const int* act)
{
    __shared__ Lds<R, TYH, LW> L;
    Tile t;
    if (act) t = listed_tile(A, act[xcd_rounds(blockIdx.x, gridDim.x)]);
    else if (!tile_at(A, xcd_rounds(blockIdx.x, A.nblk), t)) return;   // whole group
    fused_tile<R, TYH, PD, true, LW>(A, t, L, MA);
}

// A tile of the materials step is static when every entry it loads (rows
// ty TY - 2 .., TYH of them, lanes tz KT - 1 .., LW of them, planes
// max(0, xs-2) .. min(xe+1, nx)) has kappa zero on its three e edges (PEC, or
// outside the component's range): e stays zero and h constant there, and the
// step leaves every entry the tile owns unchanged.  One workgroup per tile.
// kx null: the vacuum step, static where the PEC code of every entry is 7
// (three e edges PEC or absent), so that e stays zero and h constant.
template <typename R>
__global__ __launch_bounds__(256) void k_static_mat(const R* kx, const R* ky, const R* kz, const uint8_t* code, Geo g,
                                                    int TYH, int LW, int xchunk, int nyt, int nzt, uint8_t* out)
{
    __shared__ int active;
    const int t = blockIdx.x;
    const int tz = t % nzt, ty = (t / nzt) % nyt, cx = t / (nzt * nyt);
    if (threadIdx.x == 0) active = 0;
    __syncthreads();
    const int xs = cx * xchunk, xe = min(xs + xchunk, g.nx + 1);
    const int pb = max(0, xs - 2), pe = min(xe + 1, g.nx);
    const int TY = TYH - 4, KT = owned_k(LW);
    const int64_t per_plane = (int64_t)TYH * LW;
    const int64_t n = (int64_t)(pe - pb + 1) * per_plane;
    bool found = false;
    for (int64_t e = threadIdx.x; e < n && !found; e += blockDim.x) {
        const int q = pb + (int)(e / per_plane);
        const int r = (int)(e % per_plane);
        const int j = ty * TY - 2 + r / LW, k = tz * KT - 1 + r % LW;
        if (j < 0 || j > g.ny || k < 0 || k > g.nz) continue;
        const int64_t i = (int64_t)q * g.sp + (int64_t)j * g.sz + k;
        if (kx ? (kx[i] != R(0) || ky[i] != R(0) || kz[i] != R(0)) : (code[i] & 7u) != 7u) found = true;
    }
    if (found) atomicOr(&active, 1);
    __syncthreads();
    if (threadIdx.x == 0) out[t] = active ? 0 : 1;
}

// One step of every active instance of a batch, by a persistent grid: work
// item w (instance, tile, x-chunk) is taken by workgroup w mod gridDim.x in
// round w / gridDim.x.  Within a round the items are remapped over the XCDs
// like the tiles of one grid, so that neighbouring tiles share an L2.  The
// instance's step index and the ping-pong parity come from the table, which
// the host may rewrite between launches (a captured graph stays valid); this
// launch follows `flips` launches and `steps` steps of the current block.
template <typename R, int TYH, int PD>
__global__ __launch_bounds__(64 * TYH) void k_fused_batch(const BatchTable<R>* Tg, int flips, int steps)
{
    __shared__ Lds<R, TYH> L;
    // The table is read-only during the launch: reading it through the
    // constant address space makes its (uniform) fields scalar loads into
    // scalar registers instead of vector loads that would occupy VGPRs.
    typedef const __attribute__((address_space(4))) BatchTable<R>* CTable;
    typedef const __attribute__((address_space(4))) uint32_t* CWords;
    const CTable T = (CTable)Tg;
    const int total = T->total;
    const int ninst = T->ninst;
    const int parity = (T->phase + flips) & 1;
    for (int round = 0; round * (int)gridDim.x < total; ++round) {
        const int base = round * (int)gridDim.x;
        const int span = min((int)gridDim.x, total - base);
        if ((int)blockIdx.x >= span) break;
        // work item and instance are uniform over the workgroup: keep them (and
        // the instance's arguments) in scalar registers
        const int w = __builtin_amdgcn_readfirstlane(base + xcd_remap(blockIdx.x, span));
        int lo = 0, hi = ninst - 1;               // last instance whose first item is <= w
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (T->offset[mid] <= w) lo = mid;
            else hi = mid - 1;
        }
        const int inst = __builtin_amdgcn_readfirstlane(lo);
        FArgs<R> A;
        {
            const CWords src = (CWords)&T->item[inst].a[parity];
            uint32_t* dst = (uint32_t*)&A;
#pragma unroll
            for (int i = 0; i < (int)(sizeof(FArgs<R>) / 4); ++i) dst[i] = src[i];
        }
        A.src.n = T->step[inst] + steps;
        Tile t;
        if (tile_at(A, w - T->offset[inst], t)) fused_tile<R, TYH, PD>(A, t, L);
        __syncthreads();   // the LDS is reused by the next item
    }
}

// After a block: advance every instance's step index, and the phase by the
// number of launches (each launch swaps the ping-pong sets once).
template <typename R>
__global__ void k_batch_advance(BatchTable<R>* T, int steps, int flips)
{
    const int i = threadIdx.x + blockIdx.x * blockDim.x;
    if (i < T->ninst) T->step[i] += steps;
    if (i == 0) T->phase = (T->phase + flips) & 1;
}

// Planes loaded ahead where three are asked for: two in FP64, whose registers do
// not hold a third (31 spill, 856 against 777 us per step on 256 x 256 x 512).
template <typename R>
constexpr int deepest() { return sizeof(R) == 8 ? 2 : 3; }

template <typename R, int TYH, int PD>
hipError_t launch_fused_t(const FArgs<R>& A, const int* act, int nact, hipStream_t s)
{
    if (!act) k_fused<R, TYH, PD><<<A.nblk, 64 * TYH, 0, s>>>(A, nullptr);
    else if (nact > 0) k_fused<R, TYH, PD><<<nact, 64 * TYH, 0, s>>>(A, act);
    return hipGetLastError();
}

}  // namespace

int fused_default_rows(int real_bytes) { return real_bytes == 8 ? 12 : 16; }   // FP64 at 16 rows spills

// Shape of the materials instance: FP32 16 rows of 64 lanes; FP64 24 rows of 32,
// the 768 threads whose 168 VGPRs hold its carried coefficients: 600 of 768
// entries owned against 496 with 12 rows of 64.
inline int mat_rows(int real_bytes) { return real_bytes == 8 ? 24 : 16; }
inline int mat_lanes(int real_bytes) { return real_bytes == 8 ? 32 : 64; }

template <typename R>
bool fused_setup(FArgs<R>& A, int rows, int xchunk, int order, bool mat, int longest)
{
    if (rows == 0) rows = fused_default_rows(sizeof(R));
    if (mat) rows = mat_rows(sizeof(R));
    else if (rows != 12 && rows != 16) return false;
    const int TY = rows - 4, KT = owned_k(mat ? mat_lanes(sizeof(R)) : 64);
    A.nyt = (A.g.ny + 1 + TY - 1) / TY;
    A.nzt = (A.g.nz + 1 + KT - 1) / KT;
    // chunks of less than 2^31 bytes with their halo; longer ones gain nothing
    const int64_t plane_bytes = (int64_t)A.g.sp * sizeof(R);
    int64_t xmax = ((int64_t(1) << 31) - 1) / plane_bytes - 4;
    if (xmax < 1) return false;
    if (xchunk == 0 && longest > 0) xmax = std::min<int64_t>(xmax, longest);
    set_chunks(A, xchunk, order, xmax, kFusedFill, 1);
    return true;
}

template <typename R>
FArgs<R> fused_args(Fields<R> o, Fields<R> nf, Mat<R> M, Geo g, R alpha, Src src)
{
    FArgs<R> A;
    A.ex = o.c[0]; A.ey = o.c[1]; A.ez = o.c[2]; A.hx = o.c[3]; A.hy = o.c[4]; A.hz = o.c[5];
    A.ex1 = nf.c[0]; A.ey1 = nf.c[1]; A.ez1 = nf.c[2]; A.hx1 = nf.c[3]; A.hy1 = nf.c[4]; A.hz1 = nf.c[5];
    A.code = M.code;
    A.cls = M.cls;
    A.ctab = M.ctab;
    A.g = g;
    A.a = alpha;
    A.kx = M.k[0]; A.ky = M.k[1]; A.kz = M.k[2];
    A.mx = M.m[0]; A.my = M.m[1]; A.mz = M.m[2];
    A.src = src;
    A.nyt = A.nzt = A.nxc = A.xchunk = A.nblk = A.order = A.nfull = A.tsplit = A.tchunk = 0;
    return A;
}

template <typename R>
hipError_t launch_batch_step(BatchTable<R>* T, int rows, int depth, int grid, int flips, int steps, hipStream_t s)
{
    if (rows == 0) rows = fused_default_rows(sizeof(R));
    const int threads = 64 * rows;
    if (rows == 12) {
        if (depth == 1) k_fused_batch<R, 12, 1><<<grid, threads, 0, s>>>(T, flips, steps);
        else if (depth == 3) k_fused_batch<R, 12, deepest<R>()><<<grid, threads, 0, s>>>(T, flips, steps);
        else k_fused_batch<R, 12, 2><<<grid, threads, 0, s>>>(T, flips, steps);
    } else {
        if (depth == 1) k_fused_batch<R, 16, 1><<<grid, threads, 0, s>>>(T, flips, steps);
        else if (depth == 3) k_fused_batch<R, 16, deepest<R>()><<<grid, threads, 0, s>>>(T, flips, steps);
        else k_fused_batch<R, 16, 2><<<grid, threads, 0, s>>>(T, flips, steps);
    }
    return hipGetLastError();
}

template <typename R>
hipError_t launch_batch_advance(BatchTable<R>* T, int steps, int flips, hipStream_t s)
{
    k_batch_advance<R><<<(TETE_MAX_BATCH + 255) / 256, 256, 0, s>>>(T, steps, flips);
    return hipGetLastError();
}

bool fused_fits(Geo g, int real_bytes)
{
    return (int64_t)g.sp * real_bytes * 5 < (int64_t(1) << 31);
}

int64_t fused_tile_cap(Geo g)
{
    // the smallest owned shapes, 8 rows (12-row tiles) by 62 entries and 20 rows by
    // 30 (FP64 materials), over tiles of single planes
    auto tiles = [&](int ty, int kt) { return (int64_t)((g.ny + ty) / ty) * ((g.nz + kt) / kt); };
    return (int64_t)(g.nx + 1) * std::max(tiles(8, owned_k(64)), tiles(20, owned_k(32)));
}

// Planes per chunk of a list of active tiles, at most, where the tuning gives none:
// short chunks find more tiles wholly in the metal.  us per step with the chunks
// that fill the CUs, of at most 32 planes, with equal chunks of at most 32, and with
// 32: 40 x 40 x 100 FP32 13.0, 27.8, 43.1; 64 x 64 x 64 FP32 materials 16.3, 33.1, 49.7;
// 160 x 160 x 320 FP32 122, 124, 130.
constexpr int kListChunk = 32;

template <typename R>
hipError_t fused_static_tiles(const R* const kap[3], const uint8_t* code, Geo g, int rows, int xchunk, int order,
                              uint8_t* tab, int* act, int64_t cap, int64_t* ntiles, int* nact, hipStream_t s)
{
    FArgs<R> A = fused_args<R>(Fields<R>{}, Fields<R>{}, Mat<R>{}, g, R(0), Src{});
    if (kap) rows = mat_rows(sizeof(R));   // the materials instance: its one shape
    else if (rows == 0) rows = fused_default_rows(sizeof(R));
    if (!fused_setup<R>(A, rows, xchunk, order, kap != nullptr, kListChunk)) return hipErrorInvalidValue;
    const int64_t nt = (int64_t)A.nyt * A.nzt * A.nxc;
    if (nt > cap || nt > 0x7fffffff) return hipErrorInvalidValue;
    if (!kap && !code) return hipErrorInvalidValue;
    k_static_mat<R><<<(int)nt, 256, 0, s>>>(kap ? kap[0] : nullptr, kap ? kap[1] : nullptr, kap ? kap[2] : nullptr,
                                            code, g, rows, kap ? mat_lanes(sizeof(R)) : 64, A.xchunk, A.nyt, A.nzt,
                                            tab);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    std::vector<uint8_t> h((size_t)nt);
    if ((e = hipMemcpyAsync(h.data(), tab, (size_t)nt, hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
    // the active tiles in the order the full launch takes them
    std::vector<int> list;
    list.reserve((size_t)nt);
    const int nlb = launch_tiles(A.order, A.nyt, A.nzt, A.nxc);
    for (int lb = 0; lb < nlb; ++lb) {
        int ty, tz, cx;
        if (!tile_of(lb, A.order, A.nyt, A.nzt, ty, tz, cx)) continue;
        const int t = (cx * A.nyt + ty) * A.nzt + tz;
        if (!h[(size_t)t]) list.push_back(t);
    }
    if (!list.empty()) {
        if ((e = hipMemcpyAsync(act, list.data(), sizeof(int) * list.size(), hipMemcpyHostToDevice, s)) !=
            hipSuccess)
            return e;
        if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;   // list is a host temporary
    }
    *ntiles = nt;
    *nact = (int)list.size();
    return hipSuccess;
}

template <typename R>
hipError_t launch_step_fused(Fields<R> o, Fields<R> nf, Mat<R> M, Geo g, R alpha, Src src, int rows, int xchunk,
                             int depth, int order, hipStream_t s, hipEvent_t* ev, const int* act, int nact)
{
    FArgs<R> A = fused_args<R>(o, nf, M, g, alpha, src);
    const bool mat = M.arr[0] != nullptr;   // per-entry materials: one shape, one plane prefetched
    if (rows == 0) rows = fused_default_rows(sizeof(R));
    if (!fused_setup<R>(A, rows, xchunk, order, mat, act ? kListChunk : 0)) return hipErrorInvalidValue;
    hipError_t e;
    if (ev && (e = hipEventRecord(ev[0], s)) != hipSuccess) return e;
    if (mat) {
        MatA<R> MA;
        for (int c = 0; c < 6; ++c) {
            if (!M.arr[c]) return hipErrorInvalidValue;
            MA.m[c] = M.arr[c];
        }
        constexpr int TYH = sizeof(R) == 8 ? 24 : 16, LW = sizeof(R) == 8 ? 32 : 64;
        // with a list of active tiles, one workgroup per entry (none: every
        // tile is static and the new set already holds the result)
        if (!act) k_fused_mat<R, TYH, LW, 1><<<A.nblk, LW * TYH, 0, s>>>(A, MA, nullptr);
        else if (nact > 0) k_fused_mat<R, TYH, LW, 1><<<nact, LW * TYH, 0, s>>>(A, MA, act);
        e = hipGetLastError();
    } else if (rows == 12) {
        if (depth == 1) e = launch_fused_t<R, 12, 1>(A, act, nact, s);
        else if (depth == 3) e = launch_fused_t<R, 12, deepest<R>()>(A, act, nact, s);
        else e = launch_fused_t<R, 12, 2>(A, act, nact, s);
    } else {
        if (depth == 1) e = launch_fused_t<R, 16, 1>(A, act, nact, s);
        else if (depth == 3) e = launch_fused_t<R, 16, deepest<R>()>(A, act, nact, s);
        else e = launch_fused_t<R, 16, 2>(A, act, nact, s);
    }
    if (e != hipSuccess) return e;
    if (ev && (e = hipEventRecord(ev[1], s)) != hipSuccess) return e;
    if (ev && (e = hipEventRecord(ev[2], s)) != hipSuccess) return e;
    return hipSuccess;
}

#define TETE_FUSED_INST(R)                                                                                     \
    template bool fused_setup<R>(FArgs<R>&, int, int, int, bool, int);                                            \
    template FArgs<R> fused_args<R>(Fields<R>, Fields<R>, Mat<R>, Geo, R, Src);                                 \
    template hipError_t launch_batch_step<R>(BatchTable<R>*, int, int, int, int, int, hipStream_t);            \
    template hipError_t launch_batch_advance<R>(BatchTable<R>*, int, int, hipStream_t);
TETE_FUSED_INST(float)
TETE_FUSED_INST(double)

template hipError_t launch_step_fused<float>(Fields<float>, Fields<float>, Mat<float>, Geo, float, Src, int, int,
                                             int, int, hipStream_t, hipEvent_t*, const int*, int);
template hipError_t launch_step_fused<double>(Fields<double>, Fields<double>, Mat<double>, Geo, double, Src, int,
                                              int, int, int, hipStream_t, hipEvent_t*, const int*, int);
template hipError_t fused_static_tiles<float>(const float* const[3], const uint8_t*, Geo, int, int, int, uint8_t*,
                                              int*, int64_t, int64_t*, int*, hipStream_t);
template hipError_t fused_static_tiles<double>(const double* const[3], const uint8_t*, Geo, int, int, int, uint8_t*,
                                               int*, int64_t, int64_t*, int*, hipStream_t);

}  // namespace tete
