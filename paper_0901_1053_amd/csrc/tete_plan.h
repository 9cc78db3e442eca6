// Launch choices made on the host from sizes alone, with no GPU code: plain
// functions that a host compiler can build by itself.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace tete {
namespace {

constexpr int kRound = 256;   // workgroups running at a time: one per CU
// lead-in and drain of a chunk, in planes: the single step's (planes xs-2 .. xe+3)
// and the two-step kernel's (xs-4 .. xe+7, of which the first and the last few are
// cheaper)
constexpr int kFusedFill = 6, kFused2Fill = 10;

// X-chunks of a launch whose workgroups fill a CU each.  A workgroup's time is
// the planes of its chunk and `fill` more (the pipeline's lead-in and drain),
// in steps of `unroll` planes.  The launch takes as many rounds of kRound
// workgroups; the items of a last, partly filled round are cut along x so that
// they fill it (the tail).  Chosen is the count of chunks with the smallest
// time; a quarter of the work over all CUs is added, which decides between
// equal times for the fewer chunks.  Measured with chunks as few as fill half
// the CUs against this rule, us per step (two-step kernel): 24 x 24 x 48
// FP64 24.9, 10.6; 64 x 64 x 256 FP32 20.4, 16.4; 192 x 192 x 1024 FP32 371, 295;
// 192 x 192 x 768 FP32 by class 363, 249; 97 x 131 x 801 FP64 179, 163; with the
// rounds above 512 x 512 x 2048 FP32 4144, 3723.
struct ChunkPlan {
    int xchunk, nxc, nfull, nblk, tsplit, tchunk;
};
inline ChunkPlan plan_chunks(int64_t tiles, int nplanes, int64_t xmax, int fill, int unroll, bool tail)
{
    auto planes = [&](int xc) { return (double)((xc + fill + unroll - 1) / unroll * unroll); };
    ChunkPlan best = {};
    double best_cost = 0.0;
    for (int xc = (int)std::min<int64_t>(nplanes, xmax); xc >= 1;) {
        const int nxc = (nplanes + xc - 1) / xc;
        xc = (nplanes + nxc - 1) / nxc;                 // equal chunks, as many
        const int64_t items = tiles * nxc;
        // beyond 32 rounds more chunks only add lead-in planes
        if (best.nblk > 0 && items > 32 * (int64_t)kRound) break;
        if (items > 0x3fffffff) break;
        const int rem = (int)(items % kRound);
        ChunkPlan p = {xc, nxc, (int)items, (int)items, 1, xc};
        double rounds = (double)((items + kRound - 1) / kRound) * planes(xc);
        if (tail && rem > 0 && items > kRound) {
            const double base = (double)(items / kRound) * planes(xc);
            for (int s = 2; s * rem <= kRound && s <= xc; ++s) {
                const int tc = (xc + s - 1) / s;
                if (base + planes(tc) < rounds) {
                    rounds = base + planes(tc);
                    p.nfull = (int)(items - rem);
                    p.tsplit = (xc + tc - 1) / tc;
                    p.tchunk = tc;
                    p.nblk = p.nfull + rem * p.tsplit;
                }
            }
        }
        const double cost = rounds + 0.25 * (double)items * planes(xc) / kRound;
        if (best.nblk == 0 || cost < best_cost) {
            best = p;
            best_cost = cost;
        }
        --xc;                                           // the next count of chunks that makes them shorter
    }
    return best;
}

// Tiles of the two-step kernel that are not static over a chunk: next[q tiles + t] is
// the first plane from q on that is not static in tile t (planes where there is
// none; a row past the last plane holds that too).  A chunk xs .. xe-1 loads planes
// xs-4 .. xe+3.
struct ActiveTiles {
    const int* next;
    int tiles, planes;
    bool operator()(int t, int cx, int xc) const
    {
        const int xs = cx * xc, xe = std::min(xs + xc, planes);
        return next[(int64_t)std::max(0, xs - 4) * tiles + t] <= std::min(xe + 3, planes - 1);
    }
    int64_t count(int xc) const
    {
        int64_t v = 0;
        for (int cx = 0; cx * xc < planes; ++cx)
            for (int t = 0; t < tiles; ++t) v += (*this)(t, cx, xc);
        return v;
    }
};

// Chunk length of the active tiles where the tuning gives none, at most xmax: the
// launch runs them in rounds of kRound, each as long as a chunk and ten planes; equal
// chunks, as many as make that shortest (a quarter of the work over all CUs added, as
// in plan_chunks).  Shorter chunks leave out more metal, so several rounds are no
// reason to stop before 32 planes; below, the ten planes weigh more.  us per launch
// with 32 planes whatever the grid and with this rule: 96 x 96 x 512 open pipe FP32
// 72.6, 64.2; 512 x 512 x 2048 taper FP64 1750, 1637 (129 planes, where a search that
// stops at eight rounds ends, 2033), FP32 990, 890.
inline int active_chunk(const ActiveTiles& a, int xmax)
{
    int best = 0;
    double best_cost = 0.0;
    for (int xc = std::min(a.planes, xmax); xc >= 1; --xc) {
        const int c = (a.planes + xc - 1) / xc;
        xc = (a.planes + c - 1) / c;                  // equal chunks, as many
        const int64_t items = a.count(xc);
        const double cost =
            ((double)((items + kRound - 1) / kRound) + 0.25 * (double)items / kRound) * (double)(xc + kFused2Fill);
        if (best == 0 || cost < best_cost) {
            best_cost = cost;
            best = xc;
        }
        if (items == 0) break;
        if (items > 8 * (int64_t)kRound && xc <= 32) break;
    }
    return best;
}

// Chunks of a batch's launch: planes per chunk of every member, at most, where `grid`
// persistent workgroups take the items of n members of tiles[i] tiles over
// planes[i] planes; `fill` as above.  Chosen is the count of rounds whose items are
// the shortest in all.  In several rounds the workgroups drift apart along x, and
// neighbouring tiles far apart read their halo rows from memory again: chunks are
// then at most `cap` planes.
struct BatchPlan {
    int chunk;
    bool one_round;
};
inline BatchPlan plan_batch(const int64_t* tiles, const int* planes, int n, int grid, int cap, int fill)
{
    int longest = 1;
    for (int i = 0; i < n; ++i) longest = std::max(longest, planes[i]);
    auto items = [&](int c) {
        int64_t v = 0;
        for (int i = 0; i < n; ++i) v += tiles[i] * ((planes[i] + c - 1) / c);
        return v;
    };
    // shortest chunk of at most `most` planes with at most k rounds of items, or 0
    auto shortest = [&](int64_t k, int most) {
        if (items(most) > k * grid) return 0;
        int lo = 1, hi = most;
        while (lo < hi) {
            const int mid = (lo + hi) / 2;
            if (items(mid) <= k * grid) hi = mid;
            else lo = mid + 1;
        }
        return lo;
    };
    const int c1 = shortest(1, longest);
    BatchPlan best = {c1, c1 > 0};
    int64_t best_cost = c1 + fill;
    cap = std::min(cap, longest);
    const int64_t k0 = std::max<int64_t>(2, (items(cap) + grid - 1) / grid);
    for (int64_t k = k0; k < k0 + 4; ++k) {
        const int c = shortest(k, cap);
        if (c > 0 && (best.chunk == 0 || k * (c + fill) < best_cost)) {
            best = {c, false};
            best_cost = k * (c + fill);
        }
    }
    return best;
}

// Whether a plane solve of the implicit scheme takes several Chebyshev iterations
// per pass over memory (k_cheb_pass, `stages` of them, items_e and items_h work
// items of xc planes) or one per launch over lists of rows (k_cheb_iter, `rows` of
// both systems together).  A launch over a list takes 3.9 us or its rows' memory
// traffic, a pass as long as one item's march in each round of the workgroups,
// whose lead-in planes are cheaper than the others.  The rates below fit 29 grids
// measured with either within 12 % (18 % on 160 x 160 x 512); lists are kept unless
// passes take 8 % less.  us per step with lists and with passes, FP32: 24 x 24 x 48
// 147, 174; 40 x 40 x 200 186, 204; 60 x 60 x 400 taper 207, 360; 64 x 64 x 256 with
// 6 iterations 170, 180; 80 x 80 x 64 215, 208; 60 x 60 x 400 457, 274; 104 x 89 x
// 758 taper 489, 447; 160 x 160 x 512 2899, 1200.  FP64: 24 x 24 x 48 273, 407; 60 x
// 60 x 400 taper 404, 870; 80 x 80 x 64 500, 562; 60 x 60 x 400 1310, 830.
inline bool implicit_passes(int real_bytes, int iters, int stages, int64_t rows, int64_t items_e, int64_t items_h,
                            int xc)
{
    const bool f32 = real_bytes == 4;
    const double row = f32 ? 5.9e-6 : 10.1e-6, plane = f32 ? 2.78 : 4.14, lead = f32 ? 8.7 : 5.0;   // us, us, planes
    const double lists = (iters + 1) * (2 * 3.9 + row * (double)rows);
    const double rounds = (double)((items_e + kRound - 1) / kRound + (items_h + kRound - 1) / kRound);
    const double passes = (double)((iters + stages - 1) / stages) * rounds * (xc + lead) * plane;
    return passes < 0.92 * lists;
}

// Rows per r-chunk of the r-z kernel taking four steps per launch, on nr1 rows and
// nzt z-strips, a wave each.  A wave marches its rows and 16 halo
// rows.  With n waves a SIMD a row takes, us: FP32 1.1, 1.2, 1.2, 1.5, 1.9, 2.1
// for n = 1 .. 6 (500 x 9000), as much as three for less and in proportion for more;
// FP64, whose registers hold two, 1.45, 2.1, 3.5, 4.1, rounds of two.  Fewer than 12
// rows spend most of the march on the halo, and the chunk after the first then holds
// a ring or wake line near the axis too.  us per step with the rows chosen and with
// others: 1000 x 18183 FP32 112 rows 56.3, 84 60.1, 167 64.5, 28 61.1, FP64 167 99.1,
// 84 101; 500 x 9000 FP32 28 rows 13.6, 42 17.5; 700 x 14000 FP32 59 rows 32.1, 88
// 36.1; 1000 x 4000 FP32 24 rows 12.6, 36 13.0; 333 x 4001 FP64 12 rows 9.9, 32 15.0;
// 300 x 300 FP32 12 rows 6.3, 9 7.8; 100000 x 40 FP32 33 rows 20.7, 131 37.3.
inline int rz_chunk_rows(int nr1, int64_t nzt, bool fp32)
{
    int best = 12;
    int64_t best_cost = 0;
    for (int64_t chunks = 1; chunks <= (nr1 + 11) / 12;) {
        const int rows = std::max(12, (int)((nr1 + chunks - 1) / chunks));
        const int64_t n = (nzt * ((nr1 + rows - 1) / rows) + 4 * kRound - 1) / (4 * kRound);
        const int64_t cost = (rows + 16) * (fp32 ? std::max<int64_t>(3, n) : (n + 1) / 2 * 2);
        if (best_cost == 0 || cost < best_cost) {
            best = rows;
            best_cost = cost;
        }
        if (rows <= 12) break;
        chunks = (nr1 + rows - 2) / (rows - 1);   // the next count with fewer rows
    }
    return best;
}

// Rows a wave of the r-z energy sum marches, on nr1 rows and nzt strips of 64
// entries along z: 16 (a row's loads wait for one another, so a march is paid in
// latency), fewer where the chip's 8192 waves would not have one item each.  us per
// read-out with the host's call, 16 rows of 256 entries an item and this: 60 x 700
// FP32 33.0, 25.2; 300 x 300 FP64 33.4, 25.5; 100000 x 40 FP64 90, 63; a grid-stride
// sum took 26.3, 26.6 and 74.
inline int rz_energy_rows(int nr1, int64_t nzt)
{
    return (int)std::min<int64_t>(16, std::max<int64_t>(1, nzt * nr1 / 8192));
}

}  // namespace
}  // namespace tete
