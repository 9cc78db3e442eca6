// Launch choices made on the host from sizes alone, with no GPU code: plain
// functions that a host compiler can build by itself.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace tete {
namespace {

constexpr int kRound = 256;   // workgroups running at a time: one per CU

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

}  // namespace
}  // namespace tete
