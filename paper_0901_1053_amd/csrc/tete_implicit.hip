// The implicit TE/TM scheme (16) of Sec. 4.1 as a measured comparator of the
// explicit scheme: each half step solves (I - alpha T_i) x = rhs, where T_i
// holds the transverse curls, taken at the mean of the old and new level.
//
// Solving.  Eliminating the transverse components leaves, per z-plane, one
// positive definite system for e_z (first half) and for h_z (second half):
//     (I + alpha^2 kappa_z (P_y^T mu_x P_y + P_x^T mu_y P_x)) e_z = b_e,
//     (I + alpha^2 mu_z (P_y kappa_x P_y^T + P_x kappa_y P_x^T)) h_z = b_h,
// after which h_x, h_y (e_x, e_y) follow from the new e_z (h_z).  Their
// spectra lie in [1, 1 + alpha^2 (4/dx^2 + 4/dy^2)] (Gershgorin, vacuum and
// staircase PEC), so Chebyshev iteration with these bounds converges at a known
// rate: a fixed number of iterations, no inner products, no reductions, and the
// same result for any launch shape.  The right-hand sides and the back
// substitution are grid-stride passes over the entries, z fastest; the solves
// take several iterations per pass over work items, or, where those leave the chip
// idle, one per launch over lists of rows (implicit_passes).

#include <math.h>

#include <algorithm>
#include <vector>

#include "tete_dev.h"

namespace tete {
namespace {

constexpr int TBI = 256;
constexpr int kListChunk = 8192;   // entries counted and listed by one block

struct IGeo {
    int nx, ny, nz, sz, sp, np;
};

__device__ __forceinline__ void dec(const IGeo& g, int idx, int& i, int& j, int& k)
{
    i = idx / g.sp;
    const int r = idx - i * g.sp;
    j = r / g.sz;
    k = r - j * g.sz;
}

template <typename R>
struct ICoef {
    R kx, ky, kz, mx, my, mz;   // vacuum kappa and mu
    R a, dt;                    // alpha = dtau / 2, dtau
};

// entry values with zero outside the array (the kept-zero out-of-range
// entries of each component hold zero already)
template <typename R>
__device__ __forceinline__ R val(const R* f, const IGeo& g, int i, int j, int k)
{
    if (i < 0 || j < 0 || k < 0 || i > g.nx || j > g.ny || k > g.nz) return (R)0;
    return f[k + g.sz * j + g.sp * i];
}

// coefficients that vanish outside the component's range and on PEC edges
template <typename R>
__device__ __forceinline__ R kap_x(const uint8_t* code, const IGeo& g, const ICoef<R>& c, int i, int j, int k)
{
    if (i < 0 || j < 0 || k < 0 || i >= g.nx || j > g.ny || k > g.nz) return (R)0;
    return (code[k + g.sz * j + g.sp * i] & 1u) ? (R)0 : c.kx;
}
template <typename R>
__device__ __forceinline__ R kap_y(const uint8_t* code, const IGeo& g, const ICoef<R>& c, int i, int j, int k)
{
    if (i < 0 || j < 0 || k < 0 || i > g.nx || j >= g.ny || k > g.nz) return (R)0;
    return (code[k + g.sz * j + g.sp * i] & 2u) ? (R)0 : c.ky;
}
template <typename R>
__device__ __forceinline__ R kap_z(const uint8_t* code, const IGeo& g, const ICoef<R>& c, int i, int j, int k)
{
    if (i < 0 || j < 0 || k < 0 || i > g.nx || j > g.ny || k >= g.nz) return (R)0;
    return (code[k + g.sz * j + g.sp * i] & 4u) ? (R)0 : c.kz;
}
template <typename R>
__device__ __forceinline__ R mu_x(const IGeo& g, const ICoef<R>& c, int i, int j, int k)
{
    return (i < 0 || j < 0 || k < 0 || i > g.nx || j >= g.ny || k >= g.nz) ? (R)0 : c.mx;
}
template <typename R>
__device__ __forceinline__ R mu_y(const IGeo& g, const ICoef<R>& c, int i, int j, int k)
{
    return (i < 0 || j < 0 || k < 0 || i >= g.nx || j > g.ny || k >= g.nz) ? (R)0 : c.my;
}
template <typename R>
__device__ __forceinline__ R mu_z(const IGeo& g, const ICoef<R>& c, int i, int j, int k)
{
    return (i < 0 || j < 0 || k < 0 || i >= g.nx || j >= g.ny || k > g.nz) ? (R)0 : c.mz;
}

// Right-hand sides of the first half step, (I + alpha T_0) u^{n-1/2} +
// dtau (L v^n + j_u^n): r_hx, r_hy into w.hx, w.hy, r_ez into B; the initial
// iterate for e_z is e_z^{n-1/2}.
template <typename R>
__global__ void k_imp_rhs_u(Fields<R> o, Fields<R> w, R* B, const uint8_t* code, IGeo g, ICoef<R> c, Src src)
{
    const R *ex = o.c[0], *ey = o.c[1], *ez = o.c[2], *hx = o.c[3], *hy = o.c[4];
    for (int idx = blockIdx.x * blockDim.x + threadIdx.x; idx < g.np; idx += gridDim.x * blockDim.x) {
        int i, j, k;
        dec(g, idx, i, j, k);
        const R mx = mu_x(g, c, i, j, k), my = mu_y(g, c, i, j, k), kz = kap_z(code, g, c, i, j, k);
        const R e0 = ez[idx];
        // h_x: -alpha mu_x P_y e_z + dtau mu_x P_z e_y
        w.c[3][idx] = mx == (R)0 ? (R)0
                                 : hx[idx] - c.a * mx * (val(ez, g, i, j + 1, k) - e0) +
                                       c.dt * mx * (val(ey, g, i, j, k + 1) - ey[idx]);
        // h_y: +alpha mu_y P_x e_z - dtau mu_y P_z e_x
        w.c[4][idx] = my == (R)0 ? (R)0
                                 : hy[idx] + c.a * my * (val(ez, g, i + 1, j, k) - e0) -
                                       c.dt * my * (val(ex, g, i, j, k + 1) - ex[idx]);
        if (kz == (R)0) {
            B[idx] = (R)0;
            w.c[2][idx] = (R)0;
            continue;
        }
        // e_z: +alpha kappa_z (P_y^T h_x - P_x^T h_y) - dtau kappa_z j_z
        R b = e0 + c.a * kz * ((val(hx, g, i, j - 1, k) - hx[idx]) - (val(hy, g, i - 1, j, k) - hy[idx]));
        if (src.on && i == src.i0 && j == src.j0) {
            const int64_t m = (int64_t)k - src.n + src.M;     // cell m crosses edge k in step n
            if (m >= -src.M && m <= src.M) {
#pragma clang fp contract(off)
                b -= (R)((double)kz * src.lam[m + src.M]);
            }
        }
        B[idx] = b;
        w.c[2][idx] = e0;
    }
}

// b_e = r_ez + alpha kappa_z (P_y^T r_hx - P_x^T r_hy), in place on B
template <typename R>
__global__ void k_imp_b_u(Fields<R> w, R* B, const uint8_t* code, IGeo g, ICoef<R> c)
{
    const R *rhx = w.c[3], *rhy = w.c[4];
    for (int idx = blockIdx.x * blockDim.x + threadIdx.x; idx < g.np; idx += gridDim.x * blockDim.x) {
        int i, j, k;
        dec(g, idx, i, j, k);
        const R kz = kap_z(code, g, c, i, j, k);
        if (kz == (R)0) continue;
        B[idx] += c.a * kz * ((val(rhx, g, i, j - 1, k) - rhx[idx]) - (val(rhy, g, i - 1, j, k) - rhy[idx]));
    }
}

// One iteration per launch, over lists of the rows that hold unknowns.

// (A x) of the e_z system at a free entry: x + alpha^2 kappa_z r0 x
template <typename R>
__device__ __forceinline__ R apply_e(const R* x, const uint8_t* code, const IGeo& g, const ICoef<R>& c, int i, int j,
                                     int k, int idx, R kz)
{
    const R x0 = x[idx];
    const R r = mu_x(g, c, i, j - 1, k) * (x0 - val(x, g, i, j - 1, k)) - mu_x(g, c, i, j, k) * (val(x, g, i, j + 1, k) - x0) +
                mu_y(g, c, i - 1, j, k) * (x0 - val(x, g, i - 1, j, k)) - mu_y(g, c, i, j, k) * (val(x, g, i + 1, j, k) - x0);
    return x0 + c.a * c.a * kz * r;
}

// (A x) of the h_z system at an in-range entry: x + alpha^2 mu_z r1 x
template <typename R>
__device__ __forceinline__ R apply_h(const R* x, const uint8_t* code, const IGeo& g, const ICoef<R>& c, int i, int j,
                                     int k, int idx, R mz)
{
    const R x0 = x[idx];
    const R r = kap_x(code, g, c, i, j + 1, k) * (x0 - val(x, g, i, j + 1, k)) -
                kap_x(code, g, c, i, j, k) * (val(x, g, i, j - 1, k) - x0) +
                kap_y(code, g, c, i + 1, j, k) * (x0 - val(x, g, i + 1, j, k)) -
                kap_y(code, g, c, i, j, k) * (val(x, g, i - 1, j, k) - x0);
    return x0 + c.a * c.a * mz * r;
}

// An h_z row whose four surrounding e edges are all PEC (inside the metal) is
// the identity and decoupled from every other unknown: its neighbours reach it
// only through one of those edges, whose kappa is zero.  Its solution is b.
template <typename R>
__device__ __forceinline__ bool h_coupled(const uint8_t* code, const IGeo& g, const ICoef<R>& c, int i, int j, int k)
{
    return kap_x(code, g, c, i, j + 1, k) != (R)0 || kap_x(code, g, c, i, j, k) != (R)0 ||
           kap_y(code, g, c, i + 1, j, k) != (R)0 || kap_y(code, g, c, i, j, k) != (R)0;
}

// Row lists (built once per geometry, ascending): the free e_z edges and the
// coupled h_z rows.  Chunk b of `chunk` entries is counted by block b, the
// host turns the counts into offsets, and block b writes its chunk's rows
// in order (wave ballots and a scan over the block's waves).
template <typename R>
__device__ __forceinline__ void row_flags(const uint8_t* code, const IGeo& g, const ICoef<R>& c, int idx, bool& fe,
                                          bool& fh)
{
    int i, j, k;
    dec(g, idx, i, j, k);
    fe = kap_z(code, g, c, i, j, k) != (R)0;
    fh = mu_z(g, c, i, j, k) != (R)0 && h_coupled(code, g, c, i, j, k);
}

template <typename R>
__global__ __launch_bounds__(TBI) void k_list_count(const uint8_t* code, IGeo g, ICoef<R> c, int chunk, int* cnt)
{
    __shared__ int se[TBI], sh[TBI];
    const int lo = blockIdx.x * chunk, hi = min(lo + chunk, g.np);
    int ne = 0, nh = 0;
    for (int idx = lo + (int)threadIdx.x; idx < hi; idx += TBI) {
        bool fe, fh;
        row_flags(code, g, c, idx, fe, fh);
        ne += fe;
        nh += fh;
    }
    se[threadIdx.x] = ne;
    sh[threadIdx.x] = nh;
    __syncthreads();
    for (int w = TBI / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            se[threadIdx.x] += se[threadIdx.x + w];
            sh[threadIdx.x] += sh[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        cnt[2 * blockIdx.x] = se[0];
        cnt[2 * blockIdx.x + 1] = sh[0];
    }
}

template <typename R>
__global__ __launch_bounds__(TBI) void k_list_write(const uint8_t* code, IGeo g, ICoef<R> c, int chunk,
                                                    const int* off, int* le, int* lh)
{
    constexpr int NW = TBI / 64;
    __shared__ int we[NW], wh[NW];
    const int lo = blockIdx.x * chunk, hi = min(lo + chunk, g.np);
    const int wave = threadIdx.x / 64;
    const unsigned long long below = __lanemask_lt();
    int oe = off[2 * blockIdx.x], oh = off[2 * blockIdx.x + 1];
    for (int base = lo; base < hi; base += TBI) {       // same trip count for every thread
        const int idx = base + (int)threadIdx.x;
        bool fe = false, fh = false;
        if (idx < hi) row_flags(code, g, c, idx, fe, fh);
        const unsigned long long me = __ballot(fe), mh = __ballot(fh);
        if ((threadIdx.x & 63) == 0) {
            we[wave] = __popcll(me);
            wh[wave] = __popcll(mh);
        }
        __syncthreads();
        int pe = oe, ph = oh, te = 0, th = 0;
        for (int w = 0; w < NW; ++w) {
            if (w < wave) {
                pe += we[w];
                ph += wh[w];
            }
            te += we[w];
            th += wh[w];
        }
        if (fe) le[pe + __popcll(me & below)] = idx;
        if (fh) lh[ph + __popcll(mh & below)] = idx;
        oe += te;
        oh += th;
        __syncthreads();                                 // the counts are rewritten next round
    }
}

// Chebyshev start on the rows of the list: r = b - A x, d = r / theta.  Rows
// outside the list (PEC e_z edges, h_z outside its range or inside the
// metal) are not unknowns: their x is fixed (0, or h_z^n, which equals b on an
// identity row) and their directions are zero in both buffers of the
// ping-pong pair, which the e_z and h_z solves share: every solve zeroes its
// own rows in both buffers in its last iteration.
template <typename R, bool H>
__global__ void k_cheb_init(const R* X, const R* B, R* Rr, R* D, const int* list, int n, const uint8_t* code, IGeo g,
                            ICoef<R> c, R inv_theta)
{
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) {
        const int idx = list[t];
        int i, j, k;
        dec(g, idx, i, j, k);
        const R s = H ? mu_z(g, c, i, j, k) : kap_z(code, g, c, i, j, k);
        const R ax = H ? apply_h(X, code, g, c, i, j, k, idx, s) : apply_e(X, code, g, c, i, j, k, idx, s);
        const R r = B[idx] - ax;
        Rr[idx] = r;
        D[idx] = r * inv_theta;
    }
}

// One Chebyshev step: x += d; unless last: r -= A d, d' = c1 d + c2 r; in the
// last step both direction buffers are cleared on the list's rows
template <typename R, bool H>
__global__ void k_cheb_iter(R* X, R* Rr, R* D, R* Dn, const int* list, int n, const uint8_t* code, IGeo g, ICoef<R> c,
                            R c1, R c2, int last)
{
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) {
        const int idx = list[t];
        int i, j, k;
        dec(g, idx, i, j, k);
        const R s = H ? mu_z(g, c, i, j, k) : kap_z(code, g, c, i, j, k);
        const R d = D[idx];
        X[idx] += d;
        if (last) {   // no thread reads the directions any more
            D[idx] = (R)0;
            Dn[idx] = (R)0;
            continue;
        }
        const R ad = H ? apply_h(D, code, g, c, i, j, k, idx, s) : apply_e(D, code, g, c, i, j, k, idx, s);
        const R r = Rr[idx] - ad;
        Rr[idx] = r;
        Dn[idx] = c1 * d + c2 * r;
    }
}

// The plane solves: several Chebyshev iterations per pass over memory.  A
// workgroup marches along x over a chunk of planes with a tile of rows (several
// per thread) by up to 64 entries; entries of different k are decoupled, so
// there is no halo along k.  With the pass's input of plane p loaded, stage t
// (one iteration, or the start of the iteration in its place) runs at plane
// p-t-1: it needs its direction at the planes before and after, which the march
// holds in registers, and at the rows before and after, which come from the
// thread's other rows or through LDS (double-buffered, one barrier per plane).
// Each stage costs one row at each edge of the tile and one plane at each end of
// the chunk.  x, r and d are read and written once per pass: 24 bytes per row
// and pass (FP32) instead of 28 per row and iteration over a list of rows.
// 21 vector instructions per row and stage for e_z, 31 for h_z, two waves a SIMD: on
// the 512 x 512 x 2048 taper the vector units are 45 to 67 % busy while the passes move
// 3.8 to 4.9 TB/s (a copy takes 5.0).  160 x 160 x 512 on cubic cells (15 iterations), FP32: a solve
// of e_z 1.17 -> 0.35 ms, of h_z 1.43 -> 0.43 ms.  Eight waves of 256 registers
// hold six rows a thread without spilling, 16 waves of 128 registers three.
constexpr int kChebWaves = 8;
constexpr int kMaxStages = 5;
// Stages per pass and rows per thread: the state of a stage is four values per
// row, and a workgroup of eight waves has 256 registers a thread.  FP64 with four
// rows spills 2 to 14 of them in the passes between the first and the last and in
// the last at four stages, 51 to 66 at five; with six rows 149 to 180 at four.
template <typename R> constexpr int kStages = sizeof(R) == 4 ? 5 : 4;
template <typename R> constexpr int kRJ = sizeof(R) == 4 ? 6 : 4;
template <typename R> constexpr int kOwn = kRJ<R> * kChebWaves - 2 * kStages<R>;   // rows a tile owns

// Tiles of a pass of NS stages: OWN rows by kt entries, chunks of xc planes;
// work item (cx nyt + ty) nzt + tz.
struct ChebTiles {
    int nyt, nzt, kt, xc, nxc;
};

template <typename R>
struct ChebArgs {
    const R* x0;            // first pass: the iterate it starts from
    R* x;                   // the iterate (first pass: written only)
    const R *r, *d;         // residual (first pass: the right-hand side) and direction
    R *r1, *d1;             // the same after the pass
    const uint8_t* code;
    const int* list;        // work items that hold unknowns
    IGeo g;
    ICoef<R> c;
    ChebTiles T;
    R inv_theta;
    // d' = c1 d + c2 r and on = 1 of a stage that iterates; 1, 0 and 0 of one that
    // hands on its input
    R c1[kMaxStages], c2[kMaxStages], on[kMaxStages];
};

// H: the h_z system, else e_z.  Free e edges are the PEC codes' clear bits (set
// outside a component's range); rows outside the unknowns (PEC e_z edges, h_z
// outside its range or with its four e edges PEC, where the system is the
// identity and decoupled) have residual and direction 0.
template <typename R, bool H, bool FIRST, bool LAST, int NS>
__global__ __launch_bounds__(64 * kChebWaves) void k_cheb_pass(ChebArgs<R> A)
{
    constexpr int RJ = kRJ<R>, OWN = kOwn<R>;
    constexpr int NC = H ? RJ + 1 : RJ;    // rows of codes: kappa_x of the row above too
    constexpr int CB = H ? 2 : 1;          // code bits kept per plane
    __shared__ R ex[2][NS][2 * kChebWaves][64];   // each thread's first and last row
    const IGeo g = A.g;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int it = A.list[blockIdx.x];
    const int tz = it % A.T.nzt, ty = it / A.T.nzt % A.T.nyt, cx = it / (A.T.nzt * A.T.nyt);
    const int row0 = RJ * wave;
    const int j0 = ty * OWN - NS + row0, k0 = tz * A.T.kt;
    const int nk = min(A.T.kt, g.nz + 1 - k0);
    const bool kin = lane < nk;
    const uint32_t kmask = kin ? ~0u : 0u;
    const int xs = cx * A.T.xc, xe = min(xs + A.T.xc, g.nx + 1);

    // Rows and planes are uniform over a wave: a scalar address per array and
    // row, the lane as the offset.  Rows outside the grid read entry 0 and lanes
    // past the tile its last entry, without branches; what they return is masked.
    const uint32_t lo = (uint32_t)min(lane, nk - 1);
    auto in_grid = [&](int r, int p) { return (unsigned)(j0 + r) <= (unsigned)g.ny && (unsigned)p <= (unsigned)g.nx; };
    auto base = [&](int r, int p) -> int64_t {
        return in_grid(r, p) ? (int64_t)k0 + (int64_t)g.sz * (j0 + r) + (int64_t)g.sp * p : 0;
    };
    auto at = [&](const R* a, int64_t b) { return *(const R*)((const char*)(a + b) + lo * (uint32_t)sizeof(R)); };
    struct In {
        R d[RJ], r[RJ], x[RJ];
    };
    auto load = [&](int p, In& v) {
#pragma unroll
        for (int r = 0; r < RJ; ++r) {
            const int64_t b = base(r, p);
            v.r[r] = at(A.r, b);
            if constexpr (FIRST) {
                v.d[r] = at(A.x0, b);
            } else {
                v.d[r] = at(A.d, b);
                v.x[r] = at(A.x, b);
            }
        }
    };
    // free edges of plane p: H: e_x (bit 0) and e_y (bit 1), else e_z (bit 0)
    auto code = [&](int p, uint32_t (&cw)[NC]) {
#pragma unroll
        for (int r = 0; r < NC; ++r) {
            const uint32_t v = *(A.code + base(r, p) + lo);
            cw[r] = in_grid(r, p) ? (H ? ~v & 3u : (~v >> 2) & 1u) : 0u;
        }
    };

    // the same of planes p+1 (lowest bits), p, p-1, ... per row, 0 outside the
    // grid; as a mask for bit b of plane p-back
    uint32_t hist[NC] = {};
    auto bit = [&](int r, int back, int b) -> uint32_t {
        return (uint32_t)((int32_t)(hist[r] << (31 - (CB * (back + 1) + b))) >> 31);
    };
    // row r of plane p-back holds an unknown (h_z rows outside their range have
    // no free edge)
    auto unknown = [&](int r, int back) -> uint32_t {
        if constexpr (H) return bit(r, back, 0) | bit(r + 1, back, 0) | bit(r, back, 1) | bit(r, back - 1, 1);
        else return bit(r, back, 0);
    };
    auto keep = [](uint32_t m, R v) {
        if constexpr (sizeof(R) == 4) {
            return __builtin_bit_cast(R, __builtin_bit_cast(uint32_t, v) & m);
        } else {
            const uint64_t m2 = ((uint64_t)m << 32) | m;
            return __builtin_bit_cast(R, __builtin_bit_cast(uint64_t, v) & m2);
        }
    };
    const R s2 = A.c.a * A.c.a * (H ? A.c.mz : A.c.kz);

    // per stage: direction at its plane and the plane before, residual and
    // iterate at its plane
    R dq[NS][RJ] = {}, dm[NS][RJ] = {}, rq[NS][RJ] = {}, xq[NS][RJ] = {};

    const int pa = xs - NS, pe = xe - 1 + NS;
    uint32_t cnxt[NC];
    code(pa, cnxt);
#pragma unroll
    for (int r = 0; r < NC; ++r) hist[r] = cnxt[r] & kmask;
    code(pa + 1, cnxt);
    In nxt;
    auto plane = [&](const int p) {
        const In cur = nxt;
#pragma unroll
        for (int r = 0; r < NC; ++r) hist[r] = (hist[r] << CB) | (cnxt[r] & kmask);
        load(p + 1, nxt);
        code(p + 2, cnxt);

        const int s = p & 1;
#pragma unroll
        for (int t = 0; t < NS; ++t) {
            ex[s][t][2 * wave][lane] = dq[t][0];
            ex[s][t][2 * wave + 1][lane] = dq[t][RJ - 1];
        }
        __syncthreads();

        R di[RJ], ri[RJ], xi[RJ];
#pragma unroll
        for (int r = 0; r < RJ; ++r) {
            const uint32_t u = unknown(r, 0);
            if constexpr (FIRST) {
                // the iterate itself: any entry of the grid
                di[r] = xi[r] = keep(in_grid(r, p) ? kmask : 0u, cur.d[r]);
            } else {
                di[r] = keep(u, cur.d[r]);
                xi[r] = cur.x[r];
            }
            ri[r] = keep(u, cur.r[r]);
        }
#pragma unroll
        for (int t = 0; t < NS; ++t) {
            // the rows outside the tile read one inside it: such values reach
            // only halo rows
            const R below = ex[s][t][max(2 * wave - 1, 0)][lane],
                    above = ex[s][t][min(2 * wave + 2, 2 * kChebWaves - 1)][lane];
            R dn[RJ], rn[RJ], xn[RJ];
#pragma unroll
            for (int r = 0; r < RJ; ++r) {
                const R d0 = dq[t][r];
                const R jm = r == 0 ? below : dq[t][r - 1], jp = r == RJ - 1 ? above : dq[t][r + 1];
                const R im = dm[t][r], ip = di[r];
                const uint32_t u = unknown(r, t + 1);
                R q;
                if constexpr (H) {
                    const R kxp = keep(bit(r + 1, t + 1, 0), A.c.kx), kx0 = keep(bit(r, t + 1, 0), A.c.kx);
                    const R kyp = keep(bit(r, t, 1), A.c.ky), ky0 = keep(bit(r, t + 1, 1), A.c.ky);
                    q = kxp * (d0 - jp) - kx0 * (jm - d0) + kyp * (d0 - ip) - ky0 * (im - d0);
                } else {
                    q = A.c.mx * (d0 - jm) - A.c.mx * (jp - d0) + A.c.my * (d0 - im) - A.c.my * (ip - d0);
                }
                const R ad = d0 + s2 * q;
                if (FIRST && t == 0) {
                    rn[r] = keep(u, rq[t][r] - ad);
                    dn[r] = rn[r] * A.inv_theta;
                    xn[r] = xq[t][r];
                } else {
                    const R rv = rq[t][r] - A.on[t] * ad;
                    rn[r] = keep(u, rv);
                    dn[r] = keep(u, A.c1[t] * d0 + A.c2[t] * rv);
                    xn[r] = xq[t][r] + A.on[t] * d0;
                }
            }
#pragma unroll
            for (int r = 0; r < RJ; ++r) {
                dm[t][r] = dq[t][r];
                dq[t][r] = di[r];
                rq[t][r] = ri[r];
                xq[t][r] = xi[r];
                di[r] = dn[r];
                ri[r] = rn[r];
                xi[r] = xn[r];
            }
            // the stages in turn: overlapped, their masks and temporaries spill
            __builtin_amdgcn_sched_barrier(0);
        }
        const int q = p - NS;
        if (q >= xs && q < xe) {
#pragma unroll
            for (int r = 0; r < RJ; ++r) {
                if (row0 + r < NS || row0 + r >= NS + OWN || !in_grid(r, q) || !kin) continue;
                const int64_t b = base(r, q);
                auto put = [&](R* a, R v) { *(R*)((char*)(a + b) + lo * (uint32_t)sizeof(R)) = v; };
                // the last iteration's x += d needs nothing else
                put(A.x, LAST ? xi[r] + di[r] : xi[r]);
                if constexpr (!LAST) {
                    put(A.r1, ri[r]);
                    put(A.d1, di[r]);
                }
            }
        }
    };
    load(pa, nxt);
    for (int p = pa; p <= pe; ++p) plane(p);
}

// Work items: act[2 it] counts the unknowns of the e_z system, act[2 it + 1] is 1
// where the item holds some of h_z (which touch a free e_x or e_y edge), else 0.
// One workgroup per item.
__global__ __launch_bounds__(TBI) void k_cheb_active(const uint8_t* code, IGeo g, ChebTiles T, int own, int* act)
{
    __shared__ int ne, nh;
    const int it = blockIdx.x;
    const int tz = it % T.nzt, ty = it / T.nzt % T.nyt, cx = it / (T.nzt * T.nyt);
    if (threadIdx.x == 0) ne = nh = 0;
    __syncthreads();
    const int k0 = tz * T.kt, nk = min(T.kt, g.nz + 1 - k0);
    // an h_z row's e edges reach one row and one plane further
    const int ja = ty * own, nj = min(own + 1, g.ny + 1 - ja), xs = cx * T.xc, nx = min(T.xc + 1, g.nx + 1 - xs);
    int fe = 0, fh = 0;
    for (int jx = threadIdx.x / 64; jx < nj * nx; jx += TBI / 64) {
        const int j = jx % nj, i = jx / nj, kk = threadIdx.x & 63;
        if (kk >= nk) continue;
        const uint32_t free = ~(uint32_t)code[k0 + kk + g.sz * (ja + j) + g.sp * (xs + i)];
        if ((free & 4u) && j < own && i < T.xc) ++fe;
        if (free & 3u) fh = 1;
    }
    if (fe) atomicAdd(&ne, fe);
    if (fh) atomicOr(&nh, 1);
    __syncthreads();
    if (threadIdx.x == 0) {
        act[2 * it] = ne;
        act[2 * it + 1] = nh;
    }
}

// h_x = r_hx - alpha mu_x P_y e_z, h_y = r_hy + alpha mu_y P_x e_z (new e_z);
// the wake takes -1/2 (e_z^{n-1/2} + e_z^{n+1/2}) on the bunch line
template <typename R>
__global__ void k_imp_back_u(Fields<R> o, Fields<R> w, const uint8_t* code, IGeo g, ICoef<R> c, Src src)
{
    const R* ez = w.c[2];
    for (int idx = blockIdx.x * blockDim.x + threadIdx.x; idx < g.np; idx += gridDim.x * blockDim.x) {
        int i, j, k;
        dec(g, idx, i, j, k);
        const R mx = mu_x(g, c, i, j, k), my = mu_y(g, c, i, j, k);
        const R e0 = ez[idx];
        if (mx != (R)0) w.c[3][idx] -= c.a * mx * (val(ez, g, i, j + 1, k) - e0);
        if (my != (R)0) w.c[4][idx] += c.a * my * (val(ez, g, i + 1, j, k) - e0);
        if (src.on && i == src.i0 && j == src.j0 && k < src.kend) {
            const int64_t js = src.n - k - src.M;            // wake sample of edge k
            if (js >= src.jmin && js < (int64_t)src.jmin + src.nw)
                src.wacc[js - src.jmin] += -0.5 * ((double)o.c[2][idx] + (double)e0);
        }
    }
}

// Right-hand sides of the second half step, (I + alpha T_1) v^n - dtau L^T
// u^{n+1/2}: r_ex, r_ey into w.ex, w.ey, r_hz into B; initial iterate h_z^n.
template <typename R>
__global__ void k_imp_rhs_v(Fields<R> o, Fields<R> w, R* B, const uint8_t* code, IGeo g, ICoef<R> c)
{
    const R *ex = o.c[0], *ey = o.c[1], *hz = o.c[5], *hx1 = w.c[3], *hy1 = w.c[4];
    for (int idx = blockIdx.x * blockDim.x + threadIdx.x; idx < g.np; idx += gridDim.x * blockDim.x) {
        int i, j, k;
        dec(g, idx, i, j, k);
        const R kx = kap_x(code, g, c, i, j, k), ky = kap_y(code, g, c, i, j, k), mz = mu_z(g, c, i, j, k);
        const R h0 = hz[idx];
        // e_x: -alpha kappa_x P_y^T h_z + dtau kappa_x P_z^T h_y
        w.c[0][idx] = kx == (R)0 ? (R)0
                                 : ex[idx] - c.a * kx * (val(hz, g, i, j - 1, k) - h0) +
                                       c.dt * kx * (val(hy1, g, i, j, k - 1) - hy1[idx]);
        // e_y: +alpha kappa_y P_x^T h_z - dtau kappa_y P_z^T h_x
        w.c[1][idx] = ky == (R)0 ? (R)0
                                 : ey[idx] + c.a * ky * (val(hz, g, i - 1, j, k) - h0) -
                                       c.dt * ky * (val(hx1, g, i, j, k - 1) - hx1[idx]);
        if (mz == (R)0) {
            B[idx] = (R)0;
            w.c[5][idx] = (R)0;
            continue;
        }
        // h_z: +alpha mu_z (P_y e_x - P_x e_y)
        B[idx] = h0 + c.a * mz * ((val(ex, g, i, j + 1, k) - ex[idx]) - (val(ey, g, i + 1, j, k) - ey[idx]));
        w.c[5][idx] = h0;
    }
}

// b_h = r_hz + alpha mu_z (P_y r_ex - P_x r_ey), in place on B
template <typename R>
__global__ void k_imp_b_v(Fields<R> w, R* B, IGeo g, ICoef<R> c)
{
    const R *rex = w.c[0], *rey = w.c[1];
    for (int idx = blockIdx.x * blockDim.x + threadIdx.x; idx < g.np; idx += gridDim.x * blockDim.x) {
        int i, j, k;
        dec(g, idx, i, j, k);
        const R mz = mu_z(g, c, i, j, k);
        if (mz == (R)0) continue;
        B[idx] += c.a * mz * ((val(rex, g, i, j + 1, k) - rex[idx]) - (val(rey, g, i + 1, j, k) - rey[idx]));
    }
}

// e_x = r_ex - alpha kappa_x P_y^T h_z, e_y = r_ey + alpha kappa_y P_x^T h_z (new h_z)
template <typename R>
__global__ void k_imp_back_v(Fields<R> w, const uint8_t* code, IGeo g, ICoef<R> c)
{
    const R* hz = w.c[5];
    for (int idx = blockIdx.x * blockDim.x + threadIdx.x; idx < g.np; idx += gridDim.x * blockDim.x) {
        int i, j, k;
        dec(g, idx, i, j, k);
        const R kx = kap_x(code, g, c, i, j, k), ky = kap_y(code, g, c, i, j, k);
        const R h0 = hz[idx];
        if (kx != (R)0) w.c[0][idx] -= c.a * kx * (val(hz, g, i, j - 1, k) - h0);
        if (ky != (R)0) w.c[1][idx] += c.a * ky * (val(hz, g, i - 1, j, k) - h0);
    }
}

int iblocks(int np) { return std::min(16384, std::max(1, (np + TBI - 1) / TBI)); }

// Chebyshev coefficients for spectrum [1, lmax]: (c1, c2) of each step after
// the first (Saad, Iterative Methods for Sparse Linear Systems, Alg. 12.1).
struct Cheb {
    double inv_theta;
    std::vector<double> c1, c2;
};

Cheb cheb_plan(double lmax, int iters)
{
    Cheb p;
    const double theta = 0.5 * (lmax + 1.0), delta = 0.5 * (lmax - 1.0);
    p.inv_theta = 1.0 / theta;
    const double s1 = theta / delta;
    double rho = 1.0 / s1;
    for (int t = 1; t < iters; ++t) {
        const double rn = 1.0 / (2.0 * s1 - rho);
        p.c1.push_back(rn * rho);
        p.c2.push_back(2.0 * rn / delta);
        rho = rn;
    }
    return p;
}

// Tiles of `own` rows: entries split evenly over waves of at most 64 lanes;
// chunks that fill whole rounds of the 256 CUs, of at most 64 planes so that
// items wholly in the metal are found.
// xc: planes per chunk, or 0 for chunks that fill whole rounds.
ChebTiles cheb_tiles(const IGeo& g, int own, int stages, int xc = 0)
{
    ChebTiles T;
    T.nyt = (g.ny + own) / own;
    const int w = (g.sz + 63) / 64;
    T.kt = (g.sz + w - 1) / w;
    T.nzt = (g.sz + T.kt - 1) / T.kt;
    if (xc > 0) {
        T.xc = xc;
        T.nxc = (g.nx + xc) / xc;
        return T;
    }
    const ChunkPlan p = plan_chunks((int64_t)T.nyt * T.nzt, g.nx + 1, 64, 2 * stages, 1, false);
    T.xc = p.xchunk;
    T.nxc = p.nxc;
    return T;
}

// x of one system, which holds the iterate to start from, one iteration per launch
// over the list of its rows.
template <typename R, bool H>
hipError_t cheb_solve_rows(R* x, const ImpWork<R>& wk, const uint8_t* code, const IGeo& g, const ICoef<R>& c,
                           const Cheb& p, int iters, hipStream_t s)
{
    const int* list = H ? wk.lh : wk.le;
    const int n = H ? wk.nh : wk.ne;
    if (n == 0) return hipSuccess;   // no unknowns: x stays as set
    const int nb = iblocks(n);
    k_cheb_init<R, H><<<nb, TBI, 0, s>>>(x, wk.b, wk.r, wk.d[0], list, n, code, g, c, (R)p.inv_theta);
    for (int t = 0; t < iters; ++t) {
        const bool last = t == iters - 1;
        const R c1 = last ? (R)0 : (R)p.c1[t], c2 = last ? (R)0 : (R)p.c2[t];
        k_cheb_iter<R, H><<<nb, TBI, 0, s>>>(x, wk.r, wk.d[t & 1], wk.d[(t + 1) & 1], list, n, code, g, c, c1, c2,
                                             last);
    }
    return hipGetLastError();
}

// x of one system: iters iterations from x0 with right-hand side b.  The start
// (r = b - A x0, d = r / theta) and iters - 1 iterations (x += d, r -= A d, d' =
// c1 d + c2 r) are the stages, shared evenly among the passes; the last x += d
// is part of the last pass's stores.  Passes read and write two buffer pairs in
// turn; every row outside the unknowns is masked on load, so the buffers need no
// particular content.
template <typename R, bool H>
hipError_t cheb_solve(const R* x0, R* x, const ImpWork<R>& wk, const uint8_t* code, const IGeo& g, const ICoef<R>& c,
                      const Cheb& p, int iters, hipStream_t s)
{
    if (wk.xc == 0) return cheb_solve_rows<R, H>(x, wk, code, g, c, p, iters, s);   // x holds x0
    constexpr int NS = kStages<R>;
    ChebArgs<R> A;
    const int items = H ? wk.nh : wk.ne;
    if (items == 0) return hipSuccess;   // no unknowns: x stays as set
    A.x0 = x0;
    A.x = x;
    A.code = code;
    A.list = H ? wk.lh : wk.le;
    A.g = g;
    A.c = c;
    A.T = cheb_tiles(g, kOwn<R>, kStages<R>, wk.xc);
    A.inv_theta = (R)p.inv_theta;
    const int passes = (iters + NS - 1) / NS;
    R* pair[2][2] = {{wk.r, wk.d[0]}, {wk.b, wk.d[1]}};
    int done = 0;
    for (int q = 0; q < passes; ++q) {
        const bool first = q == 0, last = q == passes - 1;
        const int n = iters / passes + (q < iters % passes ? 1 : 0);
        for (int t = 0; t < kMaxStages; ++t) {
            const int m = done + t - 1;   // stage 0 of all is the start
            const bool on = t < n && m >= 0;
            A.c1[t] = on ? (R)p.c1[m] : R(1);
            A.c2[t] = on ? (R)p.c2[m] : R(0);
            A.on[t] = on ? R(1) : R(0);
        }
        A.r = first ? wk.b : pair[(q + 1) & 1][0];
        A.d = pair[(q + 1) & 1][1];
        A.r1 = pair[q & 1][0];
        A.d1 = pair[q & 1][1];
        const int tb = 64 * kChebWaves;
        if (first && last) k_cheb_pass<R, H, true, true, NS><<<items, tb, 0, s>>>(A);
        else if (first) k_cheb_pass<R, H, true, false, NS><<<items, tb, 0, s>>>(A);
        else if (last) k_cheb_pass<R, H, false, true, NS><<<items, tb, 0, s>>>(A);
        else k_cheb_pass<R, H, false, false, NS><<<items, tb, 0, s>>>(A);
        done += n;
    }
    return hipGetLastError();
}

}  // namespace

// Largest eigenvalue bound 1 + alpha^2 (4/dx^2 + 4/dy^2) and the iterations
// that bring the Chebyshev error factor 2 ((sqrt k - 1)/(sqrt k + 1))^n below
// the precision's tolerance (1e-17 for FP64, 1e-8 for FP32).
int implicit_iters(const Geo& g, double dx, double dy, double alpha, int fp32, double* lmax_out)
{
    (void)g;
    const double lmax = 1.0 + alpha * alpha * (4.0 / (dx * dx) + 4.0 / (dy * dy));
    const double sk = sqrt(lmax), rho = (sk - 1.0) / (sk + 1.0);
    const double tol = fp32 ? 1e-8 : 1e-17;
    int n = rho > 0.0 ? (int)ceil(log(tol / 2.0) / log(rho)) : 1;
    if (lmax_out) *lmax_out = lmax;
    return std::max(1, std::min(n, 10000));
}

int implicit_list_chunks(int64_t np) { return (int)((np + kListChunk - 1) / kListChunk); }

// Lists of rows for one iteration per launch: free e_z edges and coupled h_z rows.
// The directions of all other rows have to be zero: they are in a new workspace and
// after every solve over lists, not after passes (wk.xc > 0).
template <typename R>
hipError_t build_row_lists(const Mat<R>& M, const IGeo& g, const ImpWork<R>& wk, int* cnt, int* le, int* lh, int* ne,
                           int* nh, hipStream_t s)
{
    const ICoef<R> c{M.k[0], M.k[1], M.k[2], M.m[0], M.m[1], M.m[2], (R)0, (R)0};
    const int nch = implicit_list_chunks(g.np);
    hipError_t e;
    for (int q = 0; q < 2 && wk.xc > 0; ++q)
        if ((e = launch_zero_bytes(wk.d[q], sizeof(R) * (size_t)g.np, s)) != hipSuccess) return e;
    k_list_count<R><<<nch, TBI, 0, s>>>(M.code, g, c, kListChunk, cnt);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    std::vector<int> h(2 * (size_t)nch);
    if ((e = hipMemcpyAsync(h.data(), cnt, sizeof(int) * h.size(), hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
    int64_t te = 0, th = 0;                      // exclusive scan of the chunk counts
    for (int b = 0; b < nch; ++b) {
        const int ce = h[2 * b], chh = h[2 * b + 1];
        h[2 * b] = (int)te;
        h[2 * b + 1] = (int)th;
        te += ce;
        th += chh;
    }
    if (te > g.np || th > g.np) return hipErrorInvalidValue;
    if ((e = hipMemcpyAsync(cnt, h.data(), sizeof(int) * h.size(), hipMemcpyHostToDevice, s)) != hipSuccess) return e;
    k_list_write<R><<<nch, TBI, 0, s>>>(M.code, g, c, kListChunk, cnt, le, lh);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;   // h is released on return
    *ne = (int)te;
    *nh = (int)th;
    return hipSuccess;
}

template <typename R>
hipError_t implicit_build_lists(Mat<R> M, Geo geo, int iters, const ImpWork<R>& wk, int* cnt, int* le, int* lh, int* ne,
                                int* nh, int* xc, hipStream_t s)
{
    IGeo g{geo.nx, geo.ny, geo.nz, geo.sz, geo.sp, geo.np};
    // With few active items the march of one item is the pass's time: then
    // shorter chunks, as many as leave a CU for each.  104 x 89 x 758 taper FP32, 12
    // steps with samples: 7.97 ms with the chunks of the full tiling; 461 us per step
    // with these.
    ChebTiles T = cheb_tiles(g, kOwn<R>, kStages<R>);
    hipError_t e;
    auto by_rows = [&] {
        const hipError_t r = build_row_lists<R>(M, g, wk, cnt, le, lh, ne, nh, s);
        if (r == hipSuccess) *xc = 0;
        return r;
    };
    // not even passes of a single plane would do for every row there can be: no need
    // to look for items
    if (!implicit_passes(sizeof(R), iters, kStages<R>, 2 * (int64_t)geo.np, 1, 1, 1)) return by_rows();
    std::vector<int> a[2];
    int64_t rows = 0;   // free e_z edges
    for (int turn = 0; turn < 2; ++turn) {
        const int64_t items = (int64_t)T.nyt * T.nzt * T.nxc;
        if (2 * items > geo.np) return hipErrorInvalidValue;   // an item covers far more than two entries
        k_cheb_active<<<(int)items, TBI, 0, s>>>(M.code, g, T, kOwn<R>, le);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        std::vector<int> h(2 * (size_t)items);
        if ((e = hipMemcpyAsync(h.data(), le, sizeof(int) * h.size(), hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
        if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
        rows = 0;
        for (int64_t t = 0; t < items; ++t) rows += h[2 * t];
        for (int b = 0; b < 2; ++b) {
            a[b].clear();
            for (int64_t t = 0; t < items; ++t)
                if (h[2 * t + b]) a[b].push_back((int)t);
        }
        const int64_t na = (int64_t)std::max(a[0].size(), a[1].size());
        if (turn > 0 || na == 0 || 2 * na > kRound || T.xc == 1) break;
        const ChebTiles S = cheb_tiles(g, kOwn<R>, kStages<R>, std::max(1, (int)(T.xc * na / kRound)));
        if (2 * (int64_t)S.nyt * S.nzt * S.nxc > geo.np) break;
        T = S;
    }
    // the h_z system has about as many rows as e_z
    if (!implicit_passes(sizeof(R), iters, kStages<R>, 2 * rows, (int64_t)a[0].size(), (int64_t)a[1].size(), T.xc))
        return by_rows();
    *xc = T.xc;
    int* const out[2] = {le, lh};
    for (int b = 0; b < 2; ++b)
        if (!a[b].empty() &&
            (e = hipMemcpyAsync(out[b], a[b].data(), sizeof(int) * a[b].size(), hipMemcpyHostToDevice, s)) != hipSuccess)
            return e;
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;   // host temporaries
    *ne = (int)a[0].size();
    *nh = (int)a[1].size();
    return hipSuccess;
}

template <typename R>
hipError_t launch_step_implicit(Fields<R> o, Fields<R> w, Mat<R> M, Geo geo, double dx, double dy, R alpha, Src src,
                                ImpWork<R> wk, hipStream_t s, hipEvent_t* ev)
{
    IGeo g{geo.nx, geo.ny, geo.nz, geo.sz, geo.sp, geo.np};
    ICoef<R> c{M.k[0], M.k[1], M.k[2], M.m[0], M.m[1], M.m[2], alpha, alpha + alpha};
    double lmax;
    const int iters = implicit_iters(geo, dx, dy, (double)alpha, sizeof(R) == 4, &lmax);
    const Cheb plan = cheb_plan(lmax, iters);
    const int nb = iblocks(g.np);
    hipError_t e;
    if (ev && (e = hipEventRecord(ev[0], s)) != hipSuccess) return e;
    k_imp_rhs_u<R><<<nb, TBI, 0, s>>>(o, w, wk.b, M.code, g, c, src);
    k_imp_b_u<R><<<nb, TBI, 0, s>>>(w, wk.b, M.code, g, c);
    if ((e = cheb_solve<R, false>(o.c[2], w.c[2], wk, M.code, g, c, plan, iters, s)) != hipSuccess) return e;
    k_imp_back_u<R><<<nb, TBI, 0, s>>>(o, w, M.code, g, c, src);
    if (ev && (e = hipEventRecord(ev[1], s)) != hipSuccess) return e;
    k_imp_rhs_v<R><<<nb, TBI, 0, s>>>(o, w, wk.b, M.code, g, c);
    k_imp_b_v<R><<<nb, TBI, 0, s>>>(w, wk.b, g, c);
    if ((e = cheb_solve<R, true>(o.c[5], w.c[5], wk, M.code, g, c, plan, iters, s)) != hipSuccess) return e;
    k_imp_back_v<R><<<nb, TBI, 0, s>>>(w, M.code, g, c);
    if (ev && (e = hipEventRecord(ev[2], s)) != hipSuccess) return e;
    return hipGetLastError();
}

template hipError_t implicit_build_lists<float>(Mat<float>, Geo, int, const ImpWork<float>&, int*, int*, int*, int*, int*,
                                                int*, hipStream_t);
template hipError_t implicit_build_lists<double>(Mat<double>, Geo, int, const ImpWork<double>&, int*, int*, int*, int*, int*,
                                                int*, hipStream_t);
template hipError_t launch_step_implicit<float>(Fields<float>, Fields<float>, Mat<float>, Geo, double, double, float,
                                                Src, ImpWork<float>, hipStream_t, hipEvent_t*);
template hipError_t launch_step_implicit<double>(Fields<double>, Fields<double>, Mat<double>, Geo, double, double,
                                                 double, Src, ImpWork<double>, hipStream_t, hipEvent_t*);

}  // namespace tete
