// ade_pair.h -- the pair term of a uniform flow (kernels_pair.hip states it), the
// candidate it is evaluated on and the end of a target's sum; shared by the
// kernels that walk row windows and those that walk neighbour lists.
#pragma once

#include "ade_walk.h"

namespace ade {

// One candidate: the pair term, evaluated without a branch (the lanes of a
// wavefront almost never all fail the predicate together); the kernel factor
// vanishes outside the support, and a candidate at r = 0 adds nothing.
// the constant the kernel factor of the pair term leaves out: its value at q = 0
template <int KERN>
constexpr double kPolyScale = (KERN == 4) ? 6.0 : 1.0;

// the bracket is A0 + S (E . x / r)^2 with S = +-1 (PlumeDev::dterm; in 2D
// S = +1 always).  The term forms S times it, (E . x / r)^2 + S A0, and
// finish_target multiplies the sum by S.
// ZC (zero separations): two distinct particles may share a position, so a
// candidate at r = 0 is cut by a select.  Without ZC the only candidate at
// r = 0 is the target's own record (a padding slot re-reads it): r^2 starts
// from a tiny offset (2^-40 in FP32), far below half a unit in the last place
// of any r^2 >= 1 (grid units), so it changes such an r^2 only where the
// exact sum sits on a rounding tie (then by one unit in the last place); it
// keeps the self term finite, and the self term is w (C_a - C_a) = 0 exactly.
template <typename real>
constexpr real kTinyR2 = sizeof(real) == 4 ? (real)9.094947017729282e-13 : (real)7.888609052210118e-31;  // 2^-40, 2^-100
template <int DIM, typename real, int KERN, bool ZC>
struct PairTerm {
    real invHu, a0s, ex, ey, ez;
    __device__ __forceinline__ void operator()(const Target& T, real Ca, uint32_t bx, uint32_t by,
                                               uint32_t bz, real Cb, real& acc) const {
        (*this)(T, Ca, bx, by, bz, Cb, true, acc);
    }
    // the same, added only if keep (a padding slot of a walk shared by two
    // targets)
    __device__ __forceinline__ void operator()(const Target& T, real Ca, uint32_t bx, uint32_t by,
                                               uint32_t bz, real Cb, bool keep, real& acc) const {
        const real dx = (real)(int32_t)(T.ux - bx);
        const real dy = (real)(int32_t)(T.uy - by);
        const real dz = (DIM == 3) ? (real)(int32_t)(T.uz - bz) : (real)0;
        sep(dx, dy, dz, Ca, Cb, keep, acc);
    }
    // the same from the separation (dx, dy, dz) = x_a - x_b in grid units
    __device__ __forceinline__ void sep(real dx, real dy, real dz, real Ca, real Cb, bool keep, real& acc) const {
        real r2 = ZC ? dx * dx : fmar(dx, dx, kTinyR2<real>);
        r2 = fmar(dy, dy, r2);
        if (DIM == 3) r2 = fmar(dz, dz, r2);
        // with ZC, r2 = 0 (the target itself, a padding slot, a coincident
        // particle) is cut by the select below; the support r <= H by the
        // clamp of 1 - q at 0, which zeroes the kernel factor outside it (W is
        // 0 at q = 1, so where the rounding of r puts 1 - q on the other side
        // of 0 the term is below 1e-28 of a typical one either way)
        const bool inside = ZC ? (keep && r2 > (real)0) : keep;
        const real rinv = rsqrt_r(r2);
        const real r = r2 * rinv;
        const real omq = clamp_unit(fmar(-r, invHu, (real)1));
        real f;
        if (KERN == 4) {  // (1 - q)^5 (1 + 5q) / 6
            const real o2 = omq * omq;
            f = (o2 * o2) * fmar((real)(-5.0 / 6.0), o2, omq);
        } else {
            f = omq * omq * omq;
        }
        real p = ex * dx;
        p = fmar(ey, dy, p);
        if (DIM == 3) p = fmar(ez, dz, p);
        const real pr = p * rinv;
        const real A = fmar(pr, pr, a0s);  // S times the bracket
        const real w = inside ? A * f : (real)0;
        acc = fmar(w, Ca - Cb, acc);
    }
};

// the constants come from the plume table as they are (FP32 copies for FP32),
// so they stay in scalar registers
template <int DIM, typename real, int KERN, bool ZC>
__device__ __forceinline__ PairTerm<DIM, real, KERN, ZC> make_term(const PlumeDev& P) {
    PairTerm<DIM, real, KERN, ZC> t;
    real c[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) c[k] = (sizeof(real) == 4) ? (real)P.fterm[k] : (real)P.dterm[k];
    t.invHu = c[1];
    t.a0s = c[3] * c[4];
    t.ex = c[5];
    t.ey = c[6];
    t.ez = c[7];
    return t;
}


template <typename real>
struct Cand {
    uint32_t x, y, z;
    real C;
};

template <int DIM, typename real>
__device__ __forceinline__ Cand<real> unpack(const uint4& r) {
    return Cand<real>{r.x, r.y, (DIM == 3) ? r.z : 0u, Rec<DIM, real>::conc(r)};
}

// The end of a target's pair sum acc: rhs mode writes the right-hand side
// (vphi * acc) in id order; update mode the new concentration Cbase +
// scale dt rhs with its candidate record, in cell order.  A uniform flow
// moves every particle of a plume by the same displacement, so neither the
// order of the particles nor the cells of the build change (positions are
// kept in the plume's frame, ade_internal.h).  (x, y, z, C) is the target's
// record, C its concentration in Cpair.
template <int DIM, typename real, int KERN, int MODE>
__device__ __forceinline__ void finish_target(const PairLaunch& a, const PlumeDev& P, const Cand<real>& t, uint32_t i,
                                              real acc) {
    constexpr bool kRec = Rec<DIM, real>::kStageable;
    // the kernel factor's constant and the bracket's sign S (the pair term
    // sums S times the bracket)
    const double kS = kPolyScale<KERN> * P.dterm[4];
    if ((MODE & ~kModeExact) == kModeRhs) {
        static_cast<real*>(a.out)[a.sid[i]] = (real)(kS * P.vphi) * acc;
        return;
    }
    const real sc = (real)(a.scale * P.dt * P.vphi * kS);
    const real C = a.Cbase == a.Cpair ? t.C : static_cast<const real*>(a.Cbase)[i];
    const real Cn = fmar(sc, acc, C);
    static_cast<real*>(a.out)[i] = Cn;
    if (kRec) a.out_rec[i] = Rec<DIM, real>::pack(t.x, t.y, t.z, Cn);
}

// The step counter, advanced by one thread of the launch that ends a step
// (no kernel of the launch reads it).
__device__ __forceinline__ void advance_step(const PairLaunch& a) {
    if (a.step && blockIdx.x == 0 && threadIdx.x == 0) *a.step += 1;
}

}  // namespace ade
