// Open entrance and exit pipes (the infinite pipes of the structure of Sec. 5,
// for which the paper gives no method): the bunch's own field in a uniform
// entrance pipe, written as the state a run starts from.
//
// In a pipe whose cross-section does not change along z, a bunch moving at
// v = c on the node line (i0, j0) with dtau = dz carries the field
//   e_x = -(P_x phi) F(k - n),             e_y = -(P_y phi) F(k - n),
//   h_x = (dx/dy) (P_y phi) F(k + 1 - n),  h_y = -(dy/dx) (P_x phi) F(k + 1 - n),
//   e_z = h_z = 0
// one cell per step through the ten sub-updates of scheme (23) (Sec. 4.2):
// along z each transverse edge sees the one-dimensional leapfrog at Courant
// number one; S8 keeps h_z = 0 because the transverse e is a gradient; S3
// keeps e_z = 0 because the transverse divergence of h at step n is the bunch
// current.  phi is the cross-section's potential,
//   (dy/dx)(2 phi - phi(i+1,j) - phi(i-1,j)) + (dx/dy)(2 phi - phi(i,j+1) - phi(i,j-1)) = delta_(i0,j0)
// on the nodes whose e_z edge is not PEC, phi = 0 on the others, solved here
// by conjugate gradients in FP64; F is tied to the current,
//   (F(p) + F(p+1)) / 2 = lam[p + 2M] / dtau (bunch cell p + M crosses edge
//   k in step n, p = k - n), F(p) = 0 for p > 0,
// and continues below p = -2M - 1 as the checkerboard F(p) = -F(p+1).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tete_impl.h"

namespace tete {
namespace {

constexpr int PT = 256;              // threads of the plane kernels
constexpr int PB = RED_BLOCKS;       // most blocks of a reduction pass

__host__ __device__ inline int pblocks(int64_t n) { return (int)(n / PT + 1 < PB ? n / PT + 1 : PB); }

__device__ __forceinline__ double wsum(double v)
{
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    return v;
}

// Sum over the block in a fixed order (waves, then the four wave sums).
__device__ __forceinline__ double bsum(double v)
{
    __shared__ double red[PT / 64];
    v = wsum(v);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) red[w] = v;
    __syncthreads();
    double r = red[0];
    for (int t = 1; t < PT / 64; ++t) r += red[t];
    __syncthreads();
    return r;
}

// Free-node weight of the cross-section (1: the e_z edge of plane 0 is not
// PEC, 0: PEC), node (i, j) at t = j + (ny + 1) i.
__global__ void k_pipe_mask(double* w, const uint8_t* code, CgPlane P, int sp, int sz)
{
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < P.n; t += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)(t / (P.ny + 1)), j = (int)(t % (P.ny + 1));
        w[t] = (code[(int64_t)i * sp + (int64_t)j * sz] & 4) ? 0.0 : 1.0;
    }
}

// Cell planes 0 .. kst-1 uniform: every code of a node line repeats its
// first plane (e_z bit from plane 0, e_x and e_y bits from plane 1, as plane 0
// of e_x, e_y lies on the wall).  Any difference sets *bad.
__global__ void k_pipe_uniform(const uint8_t* code, CgPlane P, int sp, int sz, int kst, int* bad)
{
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < P.n; t += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)(t / (P.ny + 1)), j = (int)(t % (P.ny + 1));
        const uint8_t* c = code + (int64_t)i * sp + (int64_t)j * sz;
        const int z0 = c[0] & 4, t1 = c[1] & 3;
        int diff = 0;
        for (int k = 1; k < kst; ++k) diff |= ((c[k] & 4) != z0) | ((c[k] & 3) != t1);
        if (diff) *bad = 1;
    }
}

// Laplacian of the cross-section applied to p on the free nodes (0 on the
// others); partial[block] = sum of p q.
__global__ __launch_bounds__(PT) void k_cg_apply(double* q, const double* p, const double* w, CgPlane P,
                                                 double* partial)
{
    const int sy = P.ny + 1;
    double s = 0.0;
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < P.n; t += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)(t / sy), j = (int)(t % sy);
        double v = 0.0;
        if (w[t] != 0.0) {
            // free nodes lie strictly inside the plane (the walls are PEC), so
            // every neighbour exists; the tests keep the reads in bounds anyway
            const double pim = i > 0 ? p[t - sy] : 0.0, pip = i < P.nx ? p[t + sy] : 0.0;
            const double pjm = j > 0 ? p[t - 1] : 0.0, pjp = j < P.ny ? p[t + 1] : 0.0;
            v = P.wx * ((p[t] - pip) + (p[t] - pim)) + P.wy * ((p[t] - pjp) + (p[t] - pjm));
        }
        q[t] = v;
        s += p[t] * v;
    }
    s = bsum(s);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// Scalars of the iteration in sc: rr = |r|^2, alpha, beta, done flag, tol.
enum { CG_RR = 0, CG_ALPHA = 1, CG_BETA = 2, CG_DONE = 3, CG_TOL = 4, CG_ITER = 5 };

__global__ __launch_bounds__(PT) void k_cg_alpha(const double* partial, int nb, double* sc)
{
    double v = 0.0;
    for (int t = threadIdx.x; t < nb; t += blockDim.x) v += partial[t];
    const double pq = bsum(v);
    if (threadIdx.x == 0) sc[CG_ALPHA] = (sc[CG_DONE] != 0.0 || pq == 0.0) ? 0.0 : sc[CG_RR] / pq;
}

__global__ __launch_bounds__(PT) void k_cg_update(double* x, double* r, const double* p, const double* q,
                                                  const double* sc, CgPlane P, double* partial)
{
    const double a = sc[CG_ALPHA];
    double s = 0.0;
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < P.n; t += (int64_t)gridDim.x * blockDim.x) {
        x[t] += a * p[t];
        const double rv = r[t] - a * q[t];
        r[t] = rv;
        s += rv * rv;
    }
    s = bsum(s);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// New |r|^2 and beta; once |r|^2 <= tol the iteration is done and every later
// alpha and beta is 0, which freezes x at the first iterate that met tol.
__global__ __launch_bounds__(PT) void k_cg_beta(const double* partial, int nb, double* sc)
{
    double v = 0.0;
    for (int t = threadIdx.x; t < nb; t += blockDim.x) v += partial[t];
    const double rn = bsum(v);
    if (threadIdx.x == 0) {
        if (sc[CG_DONE] != 0.0) {
            sc[CG_BETA] = 0.0;
        } else {
            sc[CG_BETA] = sc[CG_RR] != 0.0 ? rn / sc[CG_RR] : 0.0;
            sc[CG_RR] = rn;
            sc[CG_ITER] += 1.0;
            if (rn <= sc[CG_TOL]) sc[CG_DONE] = 1.0;
        }
    }
}

__global__ void k_cg_dir(double* p, const double* r, const double* sc, CgPlane P)
{
    const double b = sc[CG_BETA];
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < P.n; t += (int64_t)gridDim.x * blockDim.x)
        p[t] = r[t] + b * p[t];
}

// The iterations of a plane that one workgroup holds: r, q and x of node
// t = 1024 m + thread in registers (m < M), p in LDS with zeros around it.  A
// launch per sub-step took 18.3 us per iteration whatever the plane, five launches
// as long as a launch takes; here the sub-steps are three barriers apart: 2.5 us on
// 64 x 64 nodes, 4.0 on 97 x 97, 6.7 on 112 x 128, most of it LDS reads of the
// five-point stencil and the sums.  17 nodes per thread fill the LDS; a larger
// plane takes the launches.  The sums are
// those of the kernels above in the same order (waves of 64 nodes by the shuffle
// tree, four waves, then the blocks of 256 nodes by the same rule), so the
// iterates and their number are bitwise the same.
constexpr int CGT = 1024;        // threads
constexpr int CGP = 512;         // most zeros before and after p: row length + 1

__device__ __forceinline__ double cg_pair(uint32_t al, uint32_t ah) { return __hiloint2double((int)ah, (int)al); }
// One level of the shuffle tree for two values at a time: lanes below 32 (even
// rows of 16) of the result hold a's sums, the others b's.
__device__ __forceinline__ double cg_fold32(double a, double b)
{
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)__double2loint(a), (uint32_t)__double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)__double2hiint(a), (uint32_t)__double2hiint(b), false, false);
    return cg_pair(lo[0], hi[0]) + cg_pair(lo[1], hi[1]);
}
__device__ __forceinline__ double cg_fold16(double a, double b)
{
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)__double2loint(a), (uint32_t)__double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)__double2hiint(a), (uint32_t)__double2hiint(b), false, false);
    return cg_pair(lo[0], hi[0]) + cg_pair(lo[1], hi[1]);
}
template <int N>
__device__ __forceinline__ double cg_row(double v)      // v of lane + N within a row of 16
{
    return cg_pair((uint32_t)__builtin_amdgcn_mov_dpp(__double2loint(v), 0x100 + N, 0xf, 0xf, true),
                   (uint32_t)__builtin_amdgcn_mov_dpp(__double2hiint(v), 0x100 + N, 0xf, 0xf, true));
}
__device__ __forceinline__ double cg_rows(double v)
{
    v += cg_row<8>(v);
    v += cg_row<4>(v);
    v += cg_row<2>(v);
    v += cg_row<1>(v);
    return v;
}

// Sums of the M values per thread over the workgroup, as k_cg_apply and
// k_cg_alpha (k_cg_update and k_cg_beta) form them; ws: 16 M doubles.  Every
// thread returns the sum.
template <int M>
__device__ __forceinline__ double cg_sum(const double (&v)[M], double* ws)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int m = 0; m < M; m += 4) {
        // row 0 of the result holds v[m], row 1 v[m+2], row 2 v[m+1], row 3 v[m+3]
        const double a = cg_fold32(v[m], m + 1 < M ? v[m + 1] : 0.0);
        const double b = cg_fold32(m + 2 < M ? v[m + 2] : 0.0, m + 3 < M ? v[m + 3] : 0.0);
        const double s = cg_rows(cg_fold16(a, b));
        const int row = lane >> 4, mm = m + (row >> 1) + (row & 1) * 2;
        if ((lane & 15) == 0 && mm < M) ws[mm * 16 + wave] = s;
    }
    __syncthreads();
    // block b of 256 nodes: its four waves in order; blocks by the tree of 64
    double part[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int b = 64 * h + lane;
        part[h] = 0.0;
        if (b < 4 * M) part[h] += ((ws[4 * b] + ws[4 * b + 1]) + ws[4 * b + 2]) + ws[4 * b + 3];
    }
    const double s = cg_fold32(part[0], part[1]);
    const double t = cg_rows(cg_fold16(s, s));
    const double r0 = cg_pair((uint32_t)__builtin_amdgcn_readlane(__double2loint(t), 0),
                              (uint32_t)__builtin_amdgcn_readlane(__double2hiint(t), 0));
    const double r1 = cg_pair((uint32_t)__builtin_amdgcn_readlane(__double2loint(t), 32),
                              (uint32_t)__builtin_amdgcn_readlane(__double2hiint(t), 32));
    return r0 + r1;
}

template <int M>
__global__ __launch_bounds__(CGT) void k_cg_block(CgWork W, CgPlane P, int iters)
{
    __shared__ double pl[M * CGT + 2 * CGP];
    __shared__ double ws[2][16 * M];
    const int tid = threadIdx.x, n = (int)P.n, sy = P.ny + 1;
    double* const p = pl + CGP;
    double x[M], r[M];
    uint32_t freem = 0;
    for (int t = tid; t < M * CGT + 2 * CGP; t += CGT) pl[t] = 0.0;
    __syncthreads();
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const int t = m * CGT + tid;
        x[m] = r[m] = 0.0;
        if (t < n) {
            x[m] = W.x[t];
            r[m] = W.r[t];
            p[t] = W.p[t];
            if (W.w[t] != 0.0) freem |= 1u << m;
        }
    }
    double rr = W.sc[CG_RR], alpha = W.sc[CG_ALPHA], beta = W.sc[CG_BETA], it = W.sc[CG_ITER];
    const double tol = W.sc[CG_TOL];
    bool done = W.sc[CG_DONE] != 0.0;
    __syncthreads();
    for (int k = 0; k < iters && !done && rr == rr; ++k) {
        double q[M], s[M];
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const int t = m * CGT + tid;
            double v = 0.0;
            const double c = p[t];
            // free nodes lie strictly inside the plane; the zeros around p keep
            // the others' reads in bounds
            if (freem >> m & 1) v = P.wx * ((c - p[t + sy]) + (c - p[t - sy])) + P.wy * ((c - p[t + 1]) + (c - p[t - 1]));
            q[m] = v;
            s[m] = c * v;
        }
        const double pq = cg_sum<M>(s, ws[0]);
        alpha = pq == 0.0 ? 0.0 : rr / pq;
#pragma unroll
        for (int m = 0; m < M; ++m) {
            x[m] += alpha * p[m * CGT + tid];
            r[m] = r[m] - alpha * q[m];
            s[m] = r[m] * r[m];
        }
        const double rn = cg_sum<M>(s, ws[1]);     // its barrier: every read of p above is done
        beta = rr != 0.0 ? rn / rr : 0.0;
        rr = rn;
        it += 1.0;
        done = rn <= tol;
#pragma unroll
        for (int m = 0; m < M; ++m) p[m * CGT + tid] = r[m] + beta * p[m * CGT + tid];
        __syncthreads();
    }
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const int t = m * CGT + tid;
        if (t < n) {
            W.x[t] = x[m];
            W.r[t] = r[m];
            W.p[t] = p[t];
        }
    }
    if (tid == 0) {
        W.sc[CG_RR] = rr;
        W.sc[CG_ALPHA] = alpha;
        W.sc[CG_BETA] = beta;
        W.sc[CG_DONE] = done ? 1.0 : 0.0;
        W.sc[CG_ITER] = it;
    }
}

// x = 0, r = p = delta at the bunch node; sc as for a fresh iteration.
__global__ void k_cg_init(double* x, double* r, double* p, CgPlane P, int64_t src, double tol, double* sc)
{
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < P.n; t += (int64_t)gridDim.x * blockDim.x) {
        const double v = t == src ? 1.0 : 0.0;
        x[t] = 0.0;
        r[t] = v;
        p[t] = v;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc[CG_RR] = 1.0;
        sc[CG_ALPHA] = sc[CG_BETA] = 0.0;
        sc[CG_DONE] = 0.0;
        sc[CG_TOL] = tol;
        sc[CG_ITER] = 0.0;
    }
}

// Profile table of the bunch current: F[p - lo] for p = lo .. 1, lo = -2M-1,
// from the head down (one thread: the recurrence is sequential).
__global__ void k_pipe_profile(double* F, const double* lam, int M, double dtau)
{
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    const int lo = -2 * M - 1;
    F[1 - lo] = 0.0;
    for (int q = 0; q >= lo; --q) {
        const double cur = q >= -2 * M ? lam[q + 2 * M] / dtau : 0.0;
        F[q - lo] = 2.0 * cur - F[q + 1 - lo];
    }
}

__device__ __forceinline__ double prof(const double* F, int lo, int64_t p)
{
    if (p > 0) return 0.0;
    if (p >= lo) return F[p - lo];
    return ((lo - p) & 1) ? -F[0] : F[0];
}

// The state y^{n0} of the field above, every entry of the six arrays (e_z,
// h_z, out-of-range entries and PEC edges 0).
template <typename R>
__global__ void k_pipe_field(Fields<R> f, const uint8_t* code, const double* phi, const double* F, int lo, int64_t n0,
                             double rxy, double ryx, Geo g)
{
    const int sy = g.ny + 1;
    for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < g.np;
         idx += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)(idx / g.sp), j = (int)((idx / g.sz) % sy), k = (int)(idx % g.sz);
        const uint8_t c = code[idx];
        const double fe = prof(F, lo, (int64_t)k - n0), fh = prof(F, lo, (int64_t)k + 1 - n0);
        const double* ph = phi + (int64_t)i * sy + j;
        // Ex = -(P_x phi), Ey = -(P_y phi) at this entry's x- and y-edges
        const double Ex = i < g.nx ? -(ph[sy] - ph[0]) : 0.0;
        const double Ey = j < g.ny ? -(ph[1] - ph[0]) : 0.0;
        f.c[0][idx] = (c & 1) ? R(0) : (R)(Ex * fe);
        f.c[1][idx] = (c & 2) ? R(0) : (R)(Ey * fe);
        f.c[2][idx] = R(0);
        f.c[3][idx] = (j < g.ny && k < g.nz) ? (R)((-rxy * Ey) * fh) : R(0);
        f.c[4][idx] = (i < g.nx && k < g.nz) ? (R)((ryx * Ex) * fh) : R(0);
        f.c[5][idx] = R(0);
    }
}

}  // namespace

hipError_t launch_pipe_check(double* w, const uint8_t* code, Geo g, CgPlane P, int kst, int* bad, hipStream_t s)
{
    if (kst < 1 || kst > g.nz) return hipErrorInvalidValue;
    const int nb = pblocks(P.n);
    k_pipe_mask<<<nb, PT, 0, s>>>(w, code, P, g.sp, g.sz);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_pipe_uniform<<<nb, PT, 0, s>>>(code, P, g.sp, g.sz, kst, bad);
    return hipGetLastError();
}

hipError_t launch_cg_init(CgWork W, CgPlane P, int64_t src, double tol, hipStream_t s)
{
    if (src < 0 || src >= P.n) return hipErrorInvalidValue;
    k_cg_init<<<pblocks(P.n), PT, 0, s>>>(W.x, W.r, W.p, P, src, tol, W.sc);
    return hipGetLastError();
}

bool cg_one_block(CgPlane P) { return P.n <= 17 * CGT && P.ny + 2 <= CGP; }

hipError_t launch_cg_iterations(CgWork W, CgPlane P, int iters, hipStream_t s)
{
    if (cg_one_block(P)) {
        if (P.n <= 4 * CGT) k_cg_block<4><<<1, CGT, 0, s>>>(W, P, iters);
        else if (P.n <= 7 * CGT) k_cg_block<7><<<1, CGT, 0, s>>>(W, P, iters);
        else if (P.n <= 10 * CGT) k_cg_block<10><<<1, CGT, 0, s>>>(W, P, iters);
        else if (P.n <= 14 * CGT) k_cg_block<14><<<1, CGT, 0, s>>>(W, P, iters);
        else k_cg_block<17><<<1, CGT, 0, s>>>(W, P, iters);
        return hipGetLastError();
    }
    const int nb = pblocks(P.n);
    for (int it = 0; it < iters; ++it) {
        k_cg_apply<<<nb, PT, 0, s>>>(W.q, W.p, W.w, P, W.partial);
        k_cg_alpha<<<1, PT, 0, s>>>(W.partial, nb, W.sc);
        k_cg_update<<<nb, PT, 0, s>>>(W.x, W.r, W.p, W.q, W.sc, P, W.partial);
        k_cg_beta<<<1, PT, 0, s>>>(W.partial, nb, W.sc);
        k_cg_dir<<<nb, PT, 0, s>>>(W.p, W.r, W.sc, P);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_pipe_profile(double* F, const double* lam, int M, double dtau, hipStream_t s)
{
    k_pipe_profile<<<1, 64, 0, s>>>(F, lam, M, dtau);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_pipe_field(Fields<R> f, const uint8_t* code, const double* phi, const double* F, int M, int64_t n0,
                             double rxy, double ryx, Geo g, hipStream_t s)
{
    const int64_t nb = (int64_t)g.np / PT + 1;
    k_pipe_field<R><<<(int)(nb < 65536 ? nb : 65536), PT, 0, s>>>(f, code, phi, F, -2 * M - 1, n0, rxy, ryx, g);
    return hipGetLastError();
}

template hipError_t launch_pipe_field<float>(Fields<float>, const uint8_t*, const double*, const double*, int, int64_t,
                                             double, double, Geo, hipStream_t);
template hipError_t launch_pipe_field<double>(Fields<double>, const uint8_t*, const double*, const double*, int,
                                              int64_t, double, double, Geo, hipStream_t);

}  // namespace tete
