// Conversion of six field arrays between the caller's device arrays and the
// library's, four consecutive entries per thread and array, or two where a type is
// FP64: 16-byte accesses next to one another, and one index division per thread (some
// imports one entry, below).  HBM bounds both directions (512 x 512 x 2048, FP32: out 7.69 -> 4.78 ms, 5.42 TB/s; in
// 5.86 -> 4.98 ms against one entry per thread).
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

// Entries per thread and array: 16 bytes of the wider type.
template <typename D, typename S>
constexpr int kPer = sizeof(D) == 8 || sizeof(S) == 8 ? 2 : 4;

template <typename R, int N>
struct alignas(sizeof(R) * N) Pack {
    R v[N];
};

// Entries e .. e+N-1 of p (e a multiple of N); VEC: p is 16-byte aligned.
template <bool VEC, int N, typename R>
__device__ __forceinline__ void load_n(const R* p, int64_t e, R (&v)[N])
{
    if constexpr (VEC) {
        const Pack<R, N> a = *(const Pack<R, N>*)(p + e);
#pragma unroll
        for (int u = 0; u < N; ++u) v[u] = a.v[u];
    } else {
#pragma unroll
        for (int u = 0; u < N; ++u) v[u] = p[e + u];
    }
}

template <bool VEC, int N, typename R>
__device__ __forceinline__ void store_n(R* p, int64_t e, const R (&v)[N])
{
    if constexpr (VEC) {
        Pack<R, N> a;
#pragma unroll
        for (int u = 0; u < N; ++u) a.v[u] = v[u];
        *(Pack<R, N>*)(p + e) = a;
    } else {
#pragma unroll
        for (int u = 0; u < N; ++u) p[e + u] = v[u];
    }
}

// Code bytes of entries e .. e+N-1, lowest first (e a multiple of N; up to three
// bytes past the last code lie in the array's padding).
template <int N>
__device__ __forceinline__ uint32_t load_codes(const uint8_t* code, int64_t e)
{
    if constexpr (N == 4) return *(const uint32_t*)(code + e);
    else if constexpr (N == 2) return *(const uint16_t*)(code + e);
    else return code[e];
}

// dst_c = src_c, n entries.  VEC: every caller array is 16-byte aligned (the
// library's arrays always are).
template <bool VEC, typename D, typename S>
__global__ __launch_bounds__(kCopyThreads) void k_export6(Six<D> dst, Six<const S> src, int64_t n)
{
    constexpr int N = kPer<D, S>;
    const int64_t e = N * (blockIdx.x * (int64_t)kCopyThreads + threadIdx.x);
    if (e + N <= n) {
        S v[6][N];
#pragma unroll
        for (int c = 0; c < 6; ++c) load_n<true, N>(src.c[c], e, v[c]);
#pragma unroll
        for (int c = 0; c < 6; ++c) {
            D w[N];
#pragma unroll
            for (int u = 0; u < N; ++u) w[u] = (D)v[c][u];
            store_n<VEC, N>(dst.c[c], e, w);
        }
    } else {
        for (int64_t i = e; i < n; ++i)
            for (int c = 0; c < 6; ++c) dst.c[c][i] = (D)src.c[c][i];
    }
}

// dst_c = src_c where the entry is kept, else 0.  keep(e, m) gives the bits
// (component c: bit c) of the thread's entries from e on, of which those past the
// array's end are not used.
template <int N, bool VEC, typename D, typename S, class KEEP>
__global__ __launch_bounds__(kCopyThreads) void k_import6(Six<D> dst, Six<const S> src, int64_t n, KEEP keep)
{
    const int64_t e = N * (blockIdx.x * (int64_t)kCopyThreads + threadIdx.x);
    if (e >= n) return;
    uint32_t m[N];
    if constexpr (N == 1) {
        keep(e, m);
#pragma unroll
        for (int c = 0; c < 6; ++c) dst.c[c][e] = (m[0] >> c) & 1u ? (D)src.c[c][e] : D(0);
    } else if (e + N <= n) {
        S v[6][N];
#pragma unroll
        for (int c = 0; c < 6; ++c) load_n<VEC, N>(src.c[c], e, v[c]);
        keep(e, m);
#pragma unroll
        for (int c = 0; c < 6; ++c) {
            D w[N];
#pragma unroll
            for (int u = 0; u < N; ++u) w[u] = (m[u] >> c) & 1u ? (D)v[c][u] : D(0);
            store_n<true, N>(dst.c[c], e, w);
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

// Imports that take one entry per thread, one array after the other: FP64 from FP64,
// where a wave's loads from six arrays at once only spread its traffic over more
// memory pages (kernel on 256 x 256 x 512: one entry, array by array 538 us, all loads
// first 564, two entries 586; with per-entry materials 662, 701, 752; 400 x 400 x 1200
// 3131, 3385, 3452), and grids of less than 1024 workgroups of four entries, which wait
// for the loads of few waves (64 x 64 x 64 FP32 with materials 24.1 us a call with four,
// 22.8 with one).
inline bool import_one_entry(int64_t n, size_t dst, size_t src)
{
    return (dst == 8 && src == 8) || n < 4 * (int64_t)kCopyThreads * 1024;
}

inline unsigned copy_blocks(int64_t n, int per) { return (unsigned)((n + per * kCopyThreads - 1) / (per * kCopyThreads)); }

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
    if (aligned16((const void* const*)dst)) k_export6<true, D, S><<<copy_blocks(n, kPer<D, S>), kCopyThreads, 0, s>>>(d, src, n);
    else k_export6<false, D, S><<<copy_blocks(n, kPer<D, S>), kCopyThreads, 0, s>>>(d, src, n);
}

template <typename D, typename S, class KEEP>
void run_import6(Six<D> dst, const void* const src[6], int64_t n, KEEP keep, hipStream_t s)
{
    Six<const S> a;
    for (int c = 0; c < 6; ++c) a.c[c] = (const S*)src[c];
    constexpr int N = kPer<D, S>;
    if (import_one_entry(n, sizeof(D), sizeof(S)))
        k_import6<1, true, D, S><<<copy_blocks(n, 1), kCopyThreads, 0, s>>>(dst, a, n, keep);
    else if (aligned16(src)) k_import6<N, true, D, S><<<copy_blocks(n, N), kCopyThreads, 0, s>>>(dst, a, n, keep);
    else k_import6<N, false, D, S><<<copy_blocks(n, N), kCopyThreads, 0, s>>>(dst, a, n, keep);
}

}  // namespace
}  // namespace tete
