// Conversion of six field arrays between the caller's device arrays and the
// library's, four consecutive entries per thread and array: 16-byte accesses
// and one index division per four entries.  HBM bounds both directions
// (512 x 512 x 2048, FP32: out 7.69 -> 4.78 ms, 5.42 TB/s; in 5.86 -> 4.98 ms against
// one entry per thread).
#pragma once

#include <stdint.h>

#include <hip/hip_runtime.h>

namespace tete {
namespace {

template <typename R>
struct Six {
    R* c[6];
};

constexpr int kCopyThreads = 256;

// Entries e .. e+3 of p (e a multiple of 4); VEC: p is 16-byte aligned.
template <bool VEC, typename R>
__device__ __forceinline__ void load4(const R* p, int64_t e, R (&v)[4])
{
    if constexpr (VEC && sizeof(R) == 4) {
        const float4 a = *(const float4*)(p + e);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    } else if constexpr (VEC) {
        const double2 a = *(const double2*)(p + e), b = *(const double2*)(p + e + 2);
        v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = p[e + u];
    }
}

template <bool VEC, typename R>
__device__ __forceinline__ void store4(R* p, int64_t e, const R (&v)[4])
{
    if constexpr (VEC && sizeof(R) == 4) {
        *(float4*)(p + e) = make_float4(v[0], v[1], v[2], v[3]);
    } else if constexpr (VEC) {
        *(double2*)(p + e) = make_double2(v[0], v[1]);
        *(double2*)(p + e + 2) = make_double2(v[2], v[3]);
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) p[e + u] = v[u];
    }
}

// dst_c = src_c, n entries.  VEC: every caller array is 16-byte aligned (the
// library's arrays always are).
template <bool VEC, typename D, typename S>
__global__ __launch_bounds__(kCopyThreads) void k_export6(Six<D> dst, Six<const S> src, int64_t n)
{
    const int64_t e = 4 * (blockIdx.x * (int64_t)kCopyThreads + threadIdx.x);
    if (e + 4 <= n) {
        S v[6][4];
#pragma unroll
        for (int c = 0; c < 6; ++c) load4<true>(src.c[c], e, v[c]);
#pragma unroll
        for (int c = 0; c < 6; ++c) {
            const D w[4] = {(D)v[c][0], (D)v[c][1], (D)v[c][2], (D)v[c][3]};
            store4<VEC>(dst.c[c], e, w);
        }
    } else {
        for (int64_t i = e; i < n; ++i)
            for (int c = 0; c < 6; ++c) dst.c[c][i] = (D)src.c[c][i];
    }
}

// dst_c = src_c where the entry is kept, else 0.  keep(e, m) gives the bits
// (component c: bit c) of entries e .. e+3, of which those past the array's end
// are not used.
template <bool VEC, typename D, typename S, class KEEP>
__global__ __launch_bounds__(kCopyThreads) void k_import6(Six<D> dst, Six<const S> src, int64_t n, KEEP keep)
{
    const int64_t e = 4 * (blockIdx.x * (int64_t)kCopyThreads + threadIdx.x);
    if (e >= n) return;
    uint32_t m[4];
    if (e + 4 <= n) {
        S v[6][4];
#pragma unroll
        for (int c = 0; c < 6; ++c) load4<VEC>(src.c[c], e, v[c]);
        keep(e, m);
#pragma unroll
        for (int c = 0; c < 6; ++c) {
            D w[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) w[u] = (m[u] >> c) & 1u ? (D)v[c][u] : D(0);
            store4<true>(dst.c[c], e, w);
        }
    } else {
        keep(e, m);
        for (int u = 0; e + u < n; ++u)
            for (int c = 0; c < 6; ++c) dst.c[c][e + u] = (m[u] >> c) & 1u ? (D)src.c[c][e + u] : D(0);
    }
}

inline bool aligned16(const void* const p[6])
{
    for (int c = 0; c < 6; ++c)
        if ((uintptr_t)p[c] & 15) return false;
    return true;
}

inline unsigned copy_blocks(int64_t n) { return (unsigned)((n + 4 * kCopyThreads - 1) / (4 * kCopyThreads)); }

template <typename R>
Six<R> six(R* const p[6])
{
    Six<R> s;
    for (int c = 0; c < 6; ++c) s.c[c] = p[c];
    return s;
}

template <typename D, typename S>
void run_export6(void* const dst[6], Six<const S> src, int64_t n, hipStream_t s)
{
    Six<D> d;
    for (int c = 0; c < 6; ++c) d.c[c] = (D*)dst[c];
    if (aligned16((const void* const*)dst)) k_export6<true, D, S><<<copy_blocks(n), kCopyThreads, 0, s>>>(d, src, n);
    else k_export6<false, D, S><<<copy_blocks(n), kCopyThreads, 0, s>>>(d, src, n);
}

template <typename D, typename S, class KEEP>
void run_import6(Six<D> dst, const void* const src[6], int64_t n, KEEP keep, hipStream_t s)
{
    Six<const S> a;
    for (int c = 0; c < 6; ++c) a.c[c] = (const S*)src[c];
    if (aligned16(src)) k_import6<true, D, S><<<copy_blocks(n), kCopyThreads, 0, s>>>(dst, a, n, keep);
    else k_import6<false, D, S><<<copy_blocks(n), kCopyThreads, 0, s>>>(dst, a, n, keep);
}

}  // namespace
}  // namespace tete
