// One plane of one step of scheme (23) for one entry per thread: the ten
// sub-updates at their plane lags, the carried state between planes, and the
// neighbour values along j.  The single-step kernel runs one such stage, the
// two-step kernel two.
#pragma once

#include "tete_dev.h"

namespace tete {
namespace {

// Carried pipeline state of one stage, named by plane lag behind the stage's
// input plane q (m1 = q-1, ...), as in the single-step kernel.  The z
// differences of the old e_x and e_y are formed again when needed (a lane
// shift and a subtraction) rather than carried, which saves registers.
template <typename R>
struct Stage {
    R EXm1, EXm2;
    R EYm1, EYm2;
    R EZm1, HYm1;
    R HZm1, HZm2, HZm3;
    R hxn_m1, hxn_m2, hyn_m2, ezh_m2;
    R pztHX_m3, pztHY_m3, pztHY_m4;
    R exh_m3, exh_m4, eyh_m3, hzn_m4;
};

// Input plane of a stage (fields of the step it starts from).
template <typename R>
struct In {
    R ex, ey, ez, hx, hy, hz;
};
// j-neighbours read from LDS: e_z (j+1) at q, h_x^n (j-1) at q-1, e_z^{n+1/2}
// (j+1) at q-2, h_z^n (j-1) at q-2, e_x^{n+1/2} (j+1) at q-3, h_z^{n+1} (j-1)
// at q-4.
template <typename R>
struct Nb {
    R ez0_jp, hxn1_jm, ezh2_jp, hz2_jm, exh3_jp, hzn4_jm;
};
// Coefficients of the sub-updates of one iteration, each already multiplied
// by its factor a or 2a (the product the single-step kernel forms first, so
// the arithmetic is the same): mu masked by the index ranges of the h
// components, kappa zero on PEC edges.
template <typename R>
struct Co {
    R mx0, mx2, my1, my2, mz3, kz1, ky2, kx2, ky3, kx4;
};
// Results of one iteration: e_z^{n-1/2} and e_z^{n+1/2} at q-1, h_x^{n+1/2}
// and h_y^{n+1/2} at q-2, h_z^{n+1} and e_y^{n+1} at q-3, e_x^{n+1} at q-4.
template <typename R>
struct Out {
    R ezold1, ezh1, hxh2, hyh2, hzn3, ey13, ex14;
};

// One iteration of a stage: the ten sub-updates at their lags, then the
// rotation of the carried state by one plane.  inj is the bunch current term
// taken off e_z^{n+1/2} (zero off the source line; x - 0 is exact).
template <bool SRC, typename R>
__device__ __forceinline__ Out<R> stage_plane(Stage<R>& S, const In<R>& c, const Nb<R>& nb, const Co<R>& f,
                                              const R inj)
{
    // S1 at q: h_x^n = h_x^{n-1/2} + a mu_x [P_z e_y^n - P_y e_z^{n-1/2}]
    const R pzEY0 = lane_next(c.ey) - c.ey;
    const R hxn0 = c.hx + f.mx0 * (pzEY0 - (nb.ez0_jp - c.ez));
    // S2 at q-1: h_y^n = h_y^{n-1/2} + a mu_y [-P_z e_x^n + P_x e_z^{n-1/2}]
    const R pzEXm1 = lane_next(S.EXm1) - S.EXm1;
    const R hyn_m1 = S.HYm1 + f.my1 * (-pzEXm1 + (c.ez - S.EZm1));
    // S3 at q-1: e_z^{n+1/2} = e_z^{n-1/2} + 2a kappa_z [P_y^T h_x^n - P_x^T h_y^n - j_z^n]
    R ezh_m1 = S.EZm1 + f.kz1 * ((nb.hxn1_jm - S.hxn_m1) - (S.hyn_m2 - hyn_m1));
    if constexpr (SRC) {
#pragma clang fp contract(off)
        ezh_m1 -= inj;
    }
    // S4 at q-2: h_x^{n+1/2} = h_x^n + a mu_x [P_z e_y^n - P_y e_z^{n+1/2}]
    const R pzEYm2 = lane_next(S.EYm2) - S.EYm2;
    const R hxh_m2 = S.hxn_m2 + f.mx2 * (pzEYm2 - (nb.ezh2_jp - S.ezh_m2));
    // S5 at q-2: h_y^{n+1/2} = h_y^n + a mu_y [-P_z e_x^n + P_x e_z^{n+1/2}]
    const R pzEXm2 = lane_next(S.EXm2) - S.EXm2;
    const R hyh_m2 = S.hyn_m2 + f.my2 * (-pzEXm2 + (ezh_m1 - S.ezh_m2));
    // S7 at q-2: e_y^{n+1/2} = e_y^n + a kappa_y [-P_z^T h_x^{n+1/2} + P_x^T h_z^n]
    const R pztHX_m2 = lane_prev(hxh_m2) - hxh_m2;
    const R eyh_m2 = S.EYm2 + f.ky2 * (-pztHX_m2 + (S.HZm3 - S.HZm2));
    // S6 at q-2: e_x^{n+1/2} = e_x^n + a kappa_x [P_z^T h_y^{n+1/2} - P_y^T h_z^n]
    const R pztHY_m2 = lane_prev(hyh_m2) - hyh_m2;
    const R exh_m2 = S.EXm2 + f.kx2 * (pztHY_m2 - (nb.hz2_jm - S.HZm2));
    // S8 at q-3: h_z^{n+1} = h_z^n + 2a mu_z [P_y e_x^{n+1/2} - P_x e_y^{n+1/2}]
    const R hzn_m3 = S.HZm3 + f.mz3 * ((nb.exh3_jp - S.exh_m3) - (eyh_m2 - S.eyh_m3));
    // S9 at q-4: e_x^{n+1} = e_x^{n+1/2} + a kappa_x [P_z^T h_y^{n+1/2} - P_y^T h_z^{n+1}]
    const R ex1_m4 = S.exh_m4 + f.kx4 * (S.pztHY_m4 - (nb.hzn4_jm - S.hzn_m4));
    // S10 at q-3: e_y^{n+1} = e_y^{n+1/2} + a kappa_y [-P_z^T h_x^{n+1/2} + P_x^T h_z^{n+1}]
    const R ey1_m3 = S.eyh_m3 + f.ky3 * (-S.pztHX_m3 + (S.hzn_m4 - hzn_m3));

    const Out<R> o = {S.EZm1, ezh_m1, hxh_m2, hyh_m2, hzn_m3, ey1_m3, ex1_m4};

    S.EXm2 = S.EXm1; S.EXm1 = c.ex;
    S.EYm2 = S.EYm1; S.EYm1 = c.ey;
    S.EZm1 = c.ez; S.HYm1 = c.hy;
    S.HZm3 = S.HZm2; S.HZm2 = S.HZm1; S.HZm1 = c.hz;
    S.hxn_m2 = S.hxn_m1; S.hxn_m1 = hxn0;
    S.hyn_m2 = hyn_m1;
    S.ezh_m2 = ezh_m1;
    S.pztHX_m3 = pztHX_m2;
    S.pztHY_m4 = S.pztHY_m3; S.pztHY_m3 = pztHY_m2;
    S.exh_m4 = S.exh_m3; S.exh_m3 = exh_m2;
    S.eyh_m3 = eyh_m2;
    S.hzn_m4 = hzn_m3;
    return o;
}

// v, or 0 where bit B of the code history is set (a PEC edge): two vector
// instructions (written as shifts, the mask becomes a compare and a select).
template <int B, typename R>
__device__ __forceinline__ R sel_free(uint32_t hist, R v)
{
    uint32_t m;
    asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(m) : "v"(hist), "n"(B));
    if constexpr (sizeof(R) == 4) {
        return __builtin_bit_cast(R, __builtin_bit_cast(uint32_t, v) & ~m);
    } else {
        const uint64_t m2 = ((uint64_t)m << 32) | m;
        return __builtin_bit_cast(R, __builtin_bit_cast(uint64_t, v) & ~m2);
    }
}

}  // namespace
}  // namespace tete
