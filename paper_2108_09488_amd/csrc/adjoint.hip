// adjoint.hip -- sensor interpolation and the discrete adjoint of the explicit
// SPH advection-dispersion step (Klapp et al., arXiv:2108.09488, Eqs. 3-5),
// giving dJ/d(alpha_L, alpha_T, D_m) for the misfit J = sum_s (C_s - d_s)^2.
//
// With rhs = L C and the explicit step C^{n+1} = C^n + dt L^n C^n,
//     lambda^N = dJ/dC^N,  lambda^n = lambda^{n+1} + dt (L^n)^T lambda^{n+1},
//     dJ/dtheta_k = sum_n dt lambda^{n+1} . (dL^n/dtheta_k) C^n.
// For equal particle volumes and a uniform tensor the pair weights are
// symmetric (w_ab = w_ba), so (L^n)^T = L^n: the adjoint kernel applies the
// same pair sum to lambda.
// The predictor-corrector step (Eqs. 8-9) is C^{n+1} = (I + dt L + dt^2/2 L^2)
// C^n: a uniform flow moves every particle by the same displacement, so the
// operator of the corrector stage is that of the predictor.  Its adjoint is
// the same two stages applied to lambda,
//     mu = lambda + dt/2 L lambda,  lambda^n = lambda + dt L mu,
// and with C^h = C^n + dt/2 L C^n the gradient gains
//     dt [lambda . L_k C^h + (mu - lambda) . L_k C^n]
// (= dt lambda . L_k C^n + dt^2/2 (lambda . L_k L C^n + L lambda . L_k C^n)).
// kAdjHalf forms mu, C^h and the second term; kAdjFull forms lambda^n and
// the first.  L depends on theta only through D (Eq. 3), which
// is linear in theta: dD/dalpha_L = v v^T/|v|, dD/dalpha_T = |v| I - v v^T/|v|,
// dD/dD_m = I.  With p = (x_ab . v)^2 / (|v|^2 r^2) the factor
// A = Gamma x^T M x / r^2 - tr M of the pair term becomes
//     alpha_L: |v| (Gamma p - 1),  alpha_T: |v| (Gamma (1 - p) - (d - 1)),
//     D_m: Gamma - d.
// The forward states are recomputed from checkpoints segment by segment
// (the cell build and the pair sums are deterministic, so the recompute is
// bit-identical to the forward run), and the gradient is accumulated in FP64
// per workgroup in a fixed order.  In a uniform flow the particles keep their
// order and their relative positions, so a state is its C alone, lambda stays
// in cell order, and when the states of all steps fit the workspace that the
// checkpoints take nothing is recomputed.
//
// Sensors: Shepard interpolation C_s = sum_b W(r_sb) C_b / sum_b W(r_sb) with
// the kernel of Eq. (7) (its normalisation cancels); its transpose seeds
// lambda^N = sum_s 2 (C_s - d_s) W(r_sb) / sum_b' W(r_sb').
#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "ade_list.h"
#include "ctx.h"

namespace ade {

// Kernel shape of Eq. (7) without its normalisation at distance r, as two
// factors: (1 - q)^6 and (1 + 6 q + 35/3 q^2) for C4, (1 - q)^4 and (1 + 4 q) for
// C2, q = r / H.
template <typename real, int KERN>
__device__ __forceinline__ void kernel_factors(real r, real invHu, real& a, real& b) {
    const real q = r * invHu;
    const real omq = pos_unit(fmar(-r, invHu, (real)1));
    const real o2 = omq * omq;
    a = (KERN == 4) ? o2 * (o2 * o2) : o2 * o2;
    b = (KERN == 4) ? fmar(q, fmar((real)(35.0 / 3.0), q, (real)6), (real)1) : fmar((real)4, q, (real)1);
}

template <int DIM>
__device__ __forceinline__ uint32_t to_fixed(double x, double L) {
    return (uint32_t)(int64_t)rint((x / L) * 4294967296.0);
}

// ---------------------------------------------------------------------------
// sensors
// ---------------------------------------------------------------------------
// One wavefront per sensor: its lanes list the row windows together, evaluate 64
// candidates at a time, and add the terms up in the order of the windows, one
// after the other (a lane per sensor waited for its windows' records in turn: 27
// against 8 us for 64 sensors; the sums are the same).
template <int DIM, typename real, int KERN>
__global__ __launch_bounds__(256) void k_sensor_fwd(const PlumeDev* __restrict__ plumes,
                                                   const double* __restrict__ xs, int ns,
                                                   StateArrays S, const FrameStep* __restrict__ frame,
                                                   const uint32_t* __restrict__ cs,
                                                   real* __restrict__ pred, real* __restrict__ den) {
    // the windows of a wavefront's sensor: first record and records before it
    __shared__ uint2 win[256 / kWave][2 * kMaxRowOffsets + 1];
    const int s = (int)(blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave);
    if (s >= ns) return;  // the whole wavefront
    uint2* w = win[threadIdx.x / kWave];
    const PlumeDev P = plumes[0];
    const uint32_t lane = threadIdx.x & (kWave - 1);
    uint32_t u[3] = {0u, 0u, 0u};
    for (int c = 0; c < DIM; ++c) u[c] = to_fixed<DIM>(xs[(size_t)c * ns + s], P.L) - frame_shift(P, frame, c);
    const Target T = make_target<DIM>(P, u[0], u[1], u[2]);
    const real H2 = h2_of<real>(P), invHu = (real)P.invHu;
    const uint32_t* px = S.pos[0];
    const uint32_t* py = S.pos[1];
    const uint32_t* pz = S.pos[2];
    const real* C = static_cast<const real*>(S.C);
    const int span = 2 * P.R + 1, noff = (DIM == 3) ? span * span : span;
    uint32_t total = 0;
    for (int j0 = 0; j0 < noff; j0 += kWave) {
        const int j = j0 + (int)lane;
        RowRanges r{0u, 0u, 0u, 0u};
        if (j < noff) r = row_ranges<DIM>(P, cs, T, j, span);
        const uint32_t n0 = r.e0 > r.s0 ? r.e0 - r.s0 : 0u, n1 = r.e1 > r.s1 ? r.e1 - r.s1 : 0u;
        const uint32_t incl = wave_inclusive_scan(n0 + n1), at = total + incl - n0 - n1;
        if (j < noff) {
            w[2 * j] = make_uint2(r.s0, at);
            w[2 * j + 1] = make_uint2(r.s1, at + n0);
        }
        total += (uint32_t)__shfl((int)incl, kWave - 1, kWave);
    }
    __builtin_amdgcn_wave_barrier();  // (the LDS writes of a wavefront take effect in program order)
    asm volatile("" ::: "memory");
    real num = 0, dsum = 0;
    uint32_t q = 0;  // the window of this lane's candidate (they ascend)
    for (uint32_t k0 = 0; k0 < total; k0 += kWave) {
        const uint32_t k = k0 + lane;
        real fa = 0, fb = 0, Cb = 0;
        if (k < total) {
            while (q + 1 < 2u * (uint32_t)noff && w[q + 1].y <= k) ++q;
            const uint32_t b = w[q].x + (k - w[q].y);
            const real dx = (real)(int32_t)(T.ux - px[b]);
            const real dy = (real)(int32_t)(T.uy - py[b]);
            const real dz = (DIM == 3) ? (real)(int32_t)(T.uz - pz[b]) : (real)0;
            real r2 = dx * dx;
            r2 = fmar(dy, dy, r2);
            if (DIM == 3) r2 = fmar(dz, dz, r2);
            if (r2 <= H2) {
                kernel_factors<real, KERN>(sqrt(r2), invHu, fa, fb);
                Cb = C[b];
            }
        }
        // a candidate outside the support adds exact zeros
        const int n = (int)min(total - k0, (uint32_t)kWave);
        for (int l = 0; l < n; ++l) {
            const real al = __shfl(fa, l, kWave), bl = __shfl(fb, l, kWave);
            num = fmar(al * bl, __shfl(Cb, l, kWave), num);
            dsum = fmar(al, bl, dsum);
        }
    }
    if (lane != 0) return;
    pred[s] = dsum > (real)0 ? num / dsum : (real)0;
    if (den) den[s] = dsum;
}

// One lane per sensor, for many sensors (kWaveSensors32): the same terms in the same
// order.
template <int DIM, typename real, int KERN>
__global__ __launch_bounds__(256) void k_sensor_lane(const PlumeDev* __restrict__ plumes,
                                                    const double* __restrict__ xs, int ns,
                                                    StateArrays S, const FrameStep* __restrict__ frame,
                                                    const uint32_t* __restrict__ cs,
                                                    real* __restrict__ pred, real* __restrict__ den) {
    const int s = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (s >= ns) return;
    const PlumeDev P = plumes[0];
    uint32_t u[3] = {0u, 0u, 0u};
    for (int c = 0; c < DIM; ++c) u[c] = to_fixed<DIM>(xs[(size_t)c * ns + s], P.L) - frame_shift(P, frame, c);
    const Target T = make_target<DIM>(P, u[0], u[1], u[2]);
    const real H2 = h2_of<real>(P), invHu = (real)P.invHu;
    const uint32_t* px = S.pos[0];
    const uint32_t* py = S.pos[1];
    const uint32_t* pz = S.pos[2];
    const real* C = static_cast<const real*>(S.C);
    const int span = 2 * P.R + 1, noff = (DIM == 3) ? span * span : span;
    real num = 0, dsum = 0;
    for (int j = 0; j < noff; ++j) {
        const RowRanges r = row_ranges<DIM>(P, cs, T, j, span);
        for (int part = 0; part < 2; ++part) {
            const uint32_t b0 = part ? r.s1 : r.s0, b1 = part ? r.e1 : r.e0;
            for (uint32_t b = b0; b < b1; ++b) {
                const real dx = (real)(int32_t)(T.ux - px[b]);
                const real dy = (real)(int32_t)(T.uy - py[b]);
                const real dz = (DIM == 3) ? (real)(int32_t)(T.uz - pz[b]) : (real)0;
                real r2 = dx * dx;
                r2 = fmar(dy, dy, r2);
                if (DIM == 3) r2 = fmar(dz, dz, r2);
                if (r2 <= H2) {
                    real fa, fb;
                    kernel_factors<real, KERN>(sqrt(r2), invHu, fa, fb);
                    num = fmar(fa * fb, C[b], num);
                    dsum = fmar(fa, fb, dsum);
                }
            }
        }
    }
    pred[s] = dsum > (real)0 ? num / dsum : (real)0;
    if (den) den[s] = dsum;
}

// residual weights r_s = 2 (C_s - d_s) / sum_b W_sb and J (FP64, fixed order)
template <typename real>
__global__ __launch_bounds__(256) void k_sensor_resid(int ns, const real* __restrict__ pred,
                                                     const real* __restrict__ den,
                                                     const real* __restrict__ obs,
                                                     real* __restrict__ rw, double* __restrict__ J) {
    __shared__ double lds[256 / kWave];
    double acc = 0.0;
    for (int s = threadIdx.x; s < ns; s += blockDim.x) {
        const double d = (double)pred[s] - (double)obs[s];
        acc += d * d;
        rw[s] = den[s] > (real)0 ? (real)(2.0 * d / (double)den[s]) : (real)0;
    }
    acc = block_sum(acc, lds);
    if (threadIdx.x == 0) *J = acc;
}

// lambda^N of particle b = sum_s r_s W(r_sb), sensors staged through LDS in
// chunks; in id order for a velocity field, in cell order in a frame
template <int DIM, typename real, int KERN>
__global__ __launch_bounds__(256) void k_sensor_seed(const PlumeDev* __restrict__ plumes,
                                                    const double* __restrict__ xs, int ns,
                                                    const real* __restrict__ rw, StateArrays S,
                                                    const FrameStep* __restrict__ frame, uint32_t N,
                                                    real* __restrict__ lam) {
    __shared__ uint32_t su[256][3];
    __shared__ real sr[256];
    __shared__ uint32_t scan[256 / kWave];
    __shared__ int ext[6];  // the workgroup's particles relative to its first: smallest and largest per axis
    const PlumeDev P = plumes[0];
    const uint32_t i0 = blockIdx.x * blockDim.x, i = i0 + threadIdx.x;
    const bool active = i < N;
    uint32_t u[3] = {0u, 0u, 0u}, u0[3];
    if (active)
        for (int c = 0; c < DIM; ++c) u[c] = S.pos[c][i];
    if (threadIdx.x < 6) ext[threadIdx.x] = 0;
    __syncthreads();
    for (int c = 0; c < DIM; ++c) {
        u0[c] = S.pos[c][i0];
        if (active) {
            atomicMin(&ext[2 * c], (int)(u[c] - u0[c]));
            atomicMax(&ext[2 * c + 1], (int)(u[c] - u0[c]));
        }
    }
    __syncthreads();
    // whether a sensor can be within the support of a particle of the workgroup
    // (consecutive in cell order, so close together): along every axis, at the
    // separation or one box length from it
    auto near = [&](const uint32_t (&q)[3]) {
        bool in = true;
        for (int c = 0; c < DIM; ++c) {
            const int64_t d = (int32_t)(q[c] - u0[c]), lo = (int64_t)ext[2 * c] - P.hx, hi = (int64_t)ext[2 * c + 1] + P.hx;
            const int64_t box = int64_t(1) << 32;
            in = in && ((d >= lo && d <= hi) || (d - box >= lo && d - box <= hi) || (d + box >= lo && d + box <= hi));
        }
        return in;
    };
    const real H2 = h2_of<real>(P), invHu = (real)P.invHu;
    real acc = 0;
    for (int s0 = 0; s0 < ns; s0 += 256) {
        const int s = s0 + threadIdx.x;
        uint32_t q[3] = {0u, 0u, 0u};
        bool keep = false;
        if (s < ns) {
            for (int c = 0; c < DIM; ++c) q[c] = to_fixed<DIM>(xs[(size_t)c * ns + s], P.L) - frame_shift(P, frame, c);
            keep = near(q);
        }
        // the sensors kept, in their order (the scan's barriers also separate
        // the last chunk's reads from these writes)
        uint32_t cnt;
        const uint32_t at = block_exclusive_scan(keep ? 1u : 0u, scan, cnt);
        if (keep) {
            for (int c = 0; c < DIM; ++c) su[at][c] = q[c];
            sr[at] = rw[s];
        }
        __syncthreads();
        if (active) {
            for (uint32_t k = 0; k < cnt; ++k) {
                // separation sensor - particle, as in the forward interpolation
                const real dx = (real)(int32_t)(su[k][0] - u[0]);
                const real dy = (real)(int32_t)(su[k][1] - u[1]);
                const real dz = (DIM == 3) ? (real)(int32_t)(su[k][2] - u[2]) : (real)0;
                real r2 = dx * dx;
                r2 = fmar(dy, dy, r2);
                if (DIM == 3) r2 = fmar(dz, dz, r2);
                if (r2 <= H2) {
                    real fa, fb;
                    kernel_factors<real, KERN>(sqrt(r2), invHu, fa, fb);
                    acc = fmar(sr[k], fa * fb, acc);
                }
            }
        }
        __syncthreads();
    }
    if (active) lam[frame ? i : S.id[i]] = acc;
}

// ---------------------------------------------------------------------------
// adjoint step
// ---------------------------------------------------------------------------
// The adjoint passes walk the neighbour lists of the forward kernels, or, for a
// plume without lists, its row windows (one lane per target).  A candidate
// carries its position and the pass's two values: X (the state in
// the gradient terms) and u (the vector the operator is applied to).  In 2D
// FP32 they travel as one 16-byte record (x, y, X, u) written just before
// the pass; otherwise they are read from the arrays.
template <typename real>
struct ACand {
    uint32_t x, y, z;
    real X, u;
};

template <int DIM, typename real>
struct ARec {
    static constexpr bool kPacked = DIM == 2 && sizeof(real) == 4;
};

__device__ __forceinline__ uint32_t fbits(float v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ float bitsf(uint32_t v) { return __builtin_bit_cast(float, v); }

// velocity field: lambda from id order into the cell order of a snapshot
template <typename real>
__global__ __launch_bounds__(256) void k_adj_gather(StateArrays S, const real* __restrict__ lam_id, uint32_t N,
                                                   real* __restrict__ lam_s) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N) lam_s[i] = lam_id[S.id[i]];
}

// uniform flow, 2D FP32: the records (x, y, X, u) of the first pass
__global__ __launch_bounds__(256) void k_adj_pack(StateArrays S, const float* __restrict__ X,
                                                 const float* __restrict__ u, uint32_t N, uint4* __restrict__ arec) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N) arec[i] = make_uint4(S.pos[0][i], S.pos[1][i], fbits(X[i]), fbits(u[i]));
}

// kAdjEuler: out = lambda^n = lam + dt L lam, gradient dt lam . L_k X.
// kAdjHalf:  out = mu = lam + dt/2 L lam, xh_out = C^h = X + dt/2 L X,
//            arec_out = their records, gradient dt (mu - lam) . L_k X.
// kAdjFull:  out = lambda^n = lam + dt L u (u = mu), gradient dt lam . L_k X
//            (X = C^h).
// Everything in cell order.  Given Xnext = C^(n-1), the passes that end a step
// also write the next step's records (x, y, Xnext, lambda^n).
// A workgroup takes blockDim.x consecutive targets of a tile; its gradient
// partials go to gpart[3 * blockIdx.x ..].
enum AdjMode { kAdjEuler = 0, kAdjHalf = 1, kAdjFull = 2 };

struct AdjLaunch {
    const PlumeDev* plumes;
    const TileDev* tiles;
    uint32_t ntiles;
    StateArrays S;
    const uint32_t* cs;
    const void* u;       // the vector the operator is applied to
    const void* lam;
    const void* X;       // the state in the gradient terms
    const uint4* arec;   // 2D FP32: records (x, y, X, u)
    void* lam_out;
    void* xh_out;
    const void* Xnext;
    uint4* arec_out;
    double speed;        // |v|
    double* gpart;
    // neighbour lists of the launch shape (list null: row windows)
    const uint32_t* list;
    const ListWave* waves;
};

// The pass's term of one pair: sums of a target.
template <int DIM, typename real, int KERN, int AMODE>
struct AdjTerm {
    real H2, invHu, a0, a1, gam, spd, vx, vy, vz;
    struct Sums {
        real al = 0, cl = 0, g1 = 0, g2 = 0, g3 = 0;
    };
    __device__ __forceinline__ AdjTerm(const PlumeDev& P, double speed)
        : H2(h2_of<real>(P)), invHu((real)P.invHu), a0((real)P.a0), a1((real)P.a1), gam((real)(DIM + 2)),
          spd((real)speed), vx((real)P.ehat[0]), vy((real)P.ehat[1]), vz((real)P.ehat[2]) {}
    // the target t and a candidate c at the separation (dx, dy, dz) = x_t - x_c.
    // Branch-free: outside the support (and at r2 = 0, where 1/r is infinite) f
    // and p are replaced by 0, so every term is exactly 0
    __device__ __forceinline__ void operator()(real dx, real dy, real dz, const ACand<real>& t, const ACand<real>& c,
                                               bool keep, Sums& s) const {
        real r2 = dx * dx;
        r2 = fmar(dy, dy, r2);
        if (DIM == 3) r2 = fmar(dz, dz, r2);
        const bool in = keep && r2 > (real)0 && r2 <= H2;
        const real rinv = rsqrt_r(r2);
        const real q = r2 * rinv * invHu;
        real omq = (real)1 - q;
        omq = pos_unit(omq);
        real f;
        if (KERN == 4) {
            const real o2 = omq * omq;
            f = o2 * o2 * omq * fmar((real)5, q, (real)1);
        } else {
            f = omq * omq * omq;
        }
        // Gamma x^T D x / r^2 - tr D = a0 + a1 p, p = (e . x / r)^2
        const real xv = fmar(dz, vz, fmar(dy, vy, dx * vx));
        real p = xv * xv * (rinv * rinv);
        f = in ? f : (real)0;
        p = in ? p : (real)0;
        const real A = fmar(a1, p, a0);
        const real dCf = (t.X - c.X) * f;
        s.al = fmar(A * f, t.u - c.u, s.al);
        if (AMODE == kAdjHalf) s.cl = fmar(A, dCf, s.cl);
        s.g1 = fmar(spd * fmar(gam, p, (real)-1), dCf, s.g1);
        s.g2 = fmar(spd * fmar(-gam, p, gam - (real)(DIM - 1)), dCf, s.g2);
        s.g3 = fmar(gam - (real)DIM, dCf, s.g3);
    }
};

template <int DIM, typename real>
__device__ __forceinline__ ACand<real> adj_part(const AdjLaunch& a, uint32_t k) {
    if constexpr (ARec<DIM, real>::kPacked) {
        const uint4 r = a.arec[k];
        return ACand<real>{r.x, r.y, 0u, (real)bitsf(r.z), (real)bitsf(r.w)};
    } else {
        return ACand<real>{a.S.pos[0][k], a.S.pos[1][k], (DIM == 3) ? a.S.pos[2][k] : 0u,
                           static_cast<const real*>(a.X)[k], static_cast<const real*>(a.u)[k]};
    }
}

// The end of target i of a pass; returns its multiplier of the gradient sums.
template <int DIM, typename real, int AMODE, typename Sums>
__device__ __forceinline__ double adj_finish(const AdjLaunch& a, const PlumeDev& P, const ACand<real>& t, uint32_t i,
                                             const Sums& s) {
    constexpr bool kPacked = ARec<DIM, real>::kPacked;
    const double sd = P.dt * P.vphi;
    const real li = static_cast<const real*>(a.lam)[i];
    if (AMODE == kAdjHalf) {
        const real h = (real)(0.5 * sd);
        const real mu = fmar(h, s.al, li), xh = fmar(h, s.cl, t.X);
        static_cast<real*>(a.lam_out)[i] = mu;
        static_cast<real*>(a.xh_out)[i] = xh;
        if constexpr (kPacked) a.arec_out[i] = make_uint4(t.x, t.y, fbits(xh), fbits(mu));
        return 0.5 * sd * (double)s.al;  // mu - lambda
    }
    const real ln = fmar((real)sd, s.al, li);
    static_cast<real*>(a.lam_out)[i] = ln;
    if constexpr (kPacked)
        if (a.Xnext) a.arec_out[i] = make_uint4(t.x, t.y, fbits(static_cast<const real*>(a.Xnext)[i]), fbits(ln));
    return (double)li;
}

// per-workgroup gradient partials, accumulated over the steps in FP64
__device__ __forceinline__ void adj_partials(double c1, double c2, double c3, double* lds, double* gpart) {
    c1 = block_sum(c1, lds);
    c2 = block_sum(c2, lds);
    c3 = block_sum(c3, lds);
    if (threadIdx.x == 0) {
        gpart[3 * blockIdx.x + 0] += c1;
        gpart[3 * blockIdx.x + 1] += c2;
        gpart[3 * blockIdx.x + 2] += c3;
    }
}

// over the row windows, one lane per target
template <int DIM, typename real, int KERN, int AMODE>
__global__ __launch_bounds__(256) void k_adjoint(AdjLaunch a, const PlumeDev* __restrict__ plumes,
                                                const TileDev* __restrict__ tiles) {
    extern __shared__ uint2 lds_list[];
    __shared__ double lds[kTile / kWave];
    const uint32_t tpb = blockDim.x, subs = kTile / tpb;
    const TileDev t = tiles[blockIdx.x / subs];
    const uint32_t i0 = t.start + (blockIdx.x % subs) * tpb;
    if (i0 >= t.end) return;  // whole workgroup: ragged last tile
    const uint32_t i1 = min(t.end, i0 + tpb);
    const PlumeDev P = plumes[t.plume];
    const bool active = i0 + threadIdx.x < i1;
    const uint32_t i = active ? i0 + threadIdx.x : i0;
    const ACand<real> self = adj_part<DIM, real>(a, i);
    const Target T = make_target<DIM>(P, self.x, self.y, self.z);
    uint2* list = lds_list + threadIdx.x;
    uint32_t total = 0;
    if (active) total = build_list<DIM, 1>(P, a.cs, T, list, tpb);
    else list[0] = make_uint2(kListEndStart, kListEndEnd);
    const AdjTerm<DIM, real, KERN, AMODE> term(P, a.speed);
    typename AdjTerm<DIM, real, KERN, AMODE>::Sums s;
    walk_stream<4>(
        list, tpb, total, i, [&](uint32_t k) { return adj_part<DIM, real>(a, k / kRecBytes); },
        [&](const ACand<real>& c, bool keep) {
            term((real)(int32_t)(T.ux - c.x), (real)(int32_t)(T.uy - c.y),
                 (DIM == 3) ? (real)(int32_t)(T.uz - c.z) : (real)0, self, c, keep, s);
        });
    double m = 0.0;
    if (active) m = P.dt * P.vphi * adj_finish<DIM, real, AMODE>(a, P, self, i, s);
    adj_partials(m * (double)s.g1, m * (double)s.g2, m * (double)s.g3, lds, a.gpart);
}

// over the neighbour lists of the launch shape: blockDim.x / G * T targets of a
// tile a workgroup.  256^2 plume (26 neighbours, four lanes a target): 14.9 us a
// pass over the windows with one lane a target, 7.2 us here.
template <int DIM, typename real, int KERN, int AMODE, int G, int T>
__global__ __launch_bounds__(256) void k_adjoint_list(AdjLaunch a, const PlumeDev* __restrict__ plumes,
                                                     const TileDev* __restrict__) {
    __shared__ double lds[kTile / kWave];
    const uint32_t wv = __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave);
    const ListWave head = a.waves[wv];
    const PlumeDev P = plumes[head.plume];
    double c1 = 0.0, c2 = 0.0, c3 = 0.0;
    if (head.i0 < head.end) {  // the wavefront has targets (ragged last tile)
        const ListTargets<G, T> q(head.i0, head.end);
        const AdjTerm<DIM, real, KERN, AMODE> term(P, a.speed);
        typename AdjTerm<DIM, real, KERN, AMODE>::Sums sA, sB;
        walk_lists<DIM, G, T>(
            a.list, head, P, q,
            [&](uint32_t k) { return adj_part<DIM, real>(a, k / kRecBytes); },
            [&](uint32_t k0, uint32_t k1, bool second, auto&& walk) {
                const ACand<real> T0 = adj_part<DIM, real>(a, k0), T1 = adj_part<DIM, real>(a, k1);
                typename AdjTerm<DIM, real, KERN, AMODE>::Sums s0, s1;
                walk([&](const ACand<real>& c, bool keep) {
                    // a slot past the end of the list holds target k0: no term for it
                    term((real)(int32_t)(T0.x - c.x), (real)(int32_t)(T0.y - c.y),
                         (DIM == 3) ? (real)(int32_t)(T0.z - c.z) : (real)0, T0, c, true, s0);
                    if (T == 2)
                        term((real)(int32_t)(T1.x - c.x), (real)(int32_t)(T1.y - c.y),
                             (DIM == 3) ? (real)(int32_t)(T1.z - c.z) : (real)0, T1, c, keep, s1);
                });
                if (second) {
                    sB = s0;
                } else {
                    sA = s0;
                    sB = s1;
                }
            });
        auto end = [&](auto& s, bool mine, uint32_t i) {
            s.al = group_sum<G>(s.al);
            if (AMODE == kAdjHalf) s.cl = group_sum<G>(s.cl);
            s.g1 = group_sum<G>(s.g1);
            s.g2 = group_sum<G>(s.g2);
            s.g3 = group_sum<G>(s.g3);
            if (!mine) return;
            const double m = P.dt * P.vphi * adj_finish<DIM, real, AMODE>(a, P, adj_part<DIM, real>(a, i), i, s);
            c1 += m * (double)s.g1;
            c2 += m * (double)s.g2;
            c3 += m * (double)s.g3;
        };
        end(sA, q.lj == 0 && q.actA, q.iA);
        if (T == 2) end(sB, q.lj == (G == 1 ? 0u : 1u) && q.actB, q.iB);
    }
    adj_partials(c1, c2, c3, lds, a.gpart);
}

__global__ __launch_bounds__(256) void k_grad_reduce(const double* __restrict__ gpart, uint32_t nb,
                                                    double* __restrict__ out) {
    __shared__ double lds[256 / kWave];
    for (int k = 0; k < 3; ++k) {
        double s = 0.0;
        for (uint32_t b = threadIdx.x; b < nb; b += blockDim.x) s += gpart[3 * b + k];
        s = block_sum(s, lds);
        if (threadIdx.x == 0) out[k] = s;
    }
}

// copy of a state snapshot: positions, C (as 32-bit words), ids, records,
// the cell table and the step counter
struct SnapCopy {
    uint32_t* dpos[3];
    const uint32_t* spos[3];
    uint32_t* dC;
    const uint32_t* sC;
    uint32_t* did;
    const uint32_t* sid;
    uint4* drec;
    const uint4* srec;
    uint32_t* dcs;
    const uint32_t* scs;
    int64_t* dstep;
    const int64_t* sstep;
    uint32_t n, ncs, cwords;
    // velocity field: the per-particle arrays (velocities, tensor reciprocals,
    // 2D FP32 records) as 32-bit words, xn[e] words each
    uint32_t* dx[10];
    const uint32_t* sx[10];
    uint32_t xn[10];
    int nx;
};

__global__ __launch_bounds__(256) void k_copy_snap(SnapCopy a) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) *a.dstep = *a.sstep;
    if (i < a.n * a.cwords) a.dC[i] = a.sC[i];
    if (i < a.ncs) a.dcs[i] = a.scs[i];
    if (i >= a.n) return;
#pragma unroll
    for (int d = 0; d < 3; ++d)
        if (a.dpos[d]) a.dpos[d][i] = a.spos[d][i];
    a.did[i] = a.sid[i];
    if (a.drec) a.drec[i] = a.srec[i];
}

// the velocity-field arrays of a snapshot copy (a separate launch: the
// 32-byte records make them the largest arrays)
__global__ __launch_bounds__(256) void k_copy_snap_x(SnapCopy a) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    for (int e = 0; e < a.nx; ++e)
        if (i < a.xn[e]) a.dx[e][i] = a.sx[e][i];
}

namespace {

#define ADE_DISPATCH3(dim, rb, kern, CALL)                              \
    do {                                                                \
        if (dim == 2 && rb == 4 && kern == 4) { CALL(2, float, 4); }    \
        else if (dim == 2 && rb == 4) { CALL(2, float, 2); }            \
        else if (dim == 2 && kern == 4) { CALL(2, double, 4); }         \
        else if (dim == 2) { CALL(2, double, 2); }                      \
        else if (rb == 4 && kern == 4) { CALL(3, float, 4); }           \
        else if (rb == 4) { CALL(3, float, 2); }                        \
        else if (kern == 4) { CALL(3, double, 4); }                     \
        else { CALL(3, double, 2); }                                    \
    } while (0)

// One state snapshot of a velocity field: the sorted particle state and its
// cell table.
struct Snap {
    uint32_t* pos[3];
    void* C;
    uint32_t* id;
    uint4* rec;
    uint32_t* cs;
    int64_t* step;
    void* vel[3];  // velocity field only (null otherwise)
    void* rD[6];
    uint4* grec;
};

constexpr uint32_t kAdjMaxSubs = 4;  // workgroups per tile of the adjoint passes (64 threads)
// the velocity-field pass: 256 threads, four lanes per target, so 64 targets
// and kAdjMaxSubs workgroups per tile
constexpr uint32_t kGenAdjBlock = 256;

// threads per workgroup of the adjoint passes: the largest of 256, 128, 64
// whose candidate lists fit in 64 KiB of LDS
uint32_t adj_block(const Plan& pl) {
    for (uint32_t b = 256; b > 64; b /= 2)
        if ((size_t)b * (size_t)pl.list_cap * 8u <= kPairLdsMax) return b;
    return 64;
}

// count snapshots laid out one after the other, `stride` bytes apart (every
// snapshot of a context has the same size and starts 256-byte aligned)
struct SnapSeq {
    Snap first{};
    size_t stride = 0;
    size_t count = 0;
    Snap operator[](size_t k) const {
        Snap s = first;
        const size_t d = k * stride;
        auto shift = [d](auto*& p) {
            if (p) p = reinterpret_cast<std::remove_reference_t<decltype(p)>>(reinterpret_cast<char*>(p) + d);
        };
        for (int i = 0; i < 3; ++i) shift(s.pos[i]);
        shift(s.C);
        shift(s.id);
        shift(s.rec);
        shift(s.cs);
        shift(s.step);
        for (int i = 0; i < 3; ++i) shift(s.vel[i]);
        for (int i = 0; i < 6; ++i) shift(s.rD[i]);
        shift(s.grec);
        return s;
    }
};

struct AdjLayout {
    size_t bytes = 0;
    // velocity field: snapshots; a uniform flow keeps its states in their place
    char* pool = nullptr;
    size_t pool_bytes = 0;
    SnapSeq ck;    // checkpoints (every K steps, plus the final state)
    SnapSeq seg;   // states of one segment
    SnapSeq segh;  // velocity field with the predictor-corrector: their half-step states
    void* y;                // ... and y = L lambda of the corrector stage (id order)
    void* lam[2];
    void* lam_s;
    void* mu_s;  // predictor-corrector: mu and C^h of the step (cell order)
    void* ch_s;
    uint4* arec;   // 2D FP32, uniform flow: candidate records of the pass (x, y, X, u)
    uint4* arec2;  // predictor-corrector: those of the second pass
    void* pred;
    void* den;
    void* rw;
    double* J;
    double* gpart;
    double* grad;
};

void take_snap(char* base, size_t& off, const ade_ctx* c, Snap& s) {
    auto take = [&](size_t bytes) -> char* {
        off = (off + 255) & ~size_t(255);
        char* p = base ? base + off : nullptr;
        off += bytes;
        return p;
    };
    const Plan& pl = c->plan;
    const size_t N = (size_t)pl.N;
    for (int d = 0; d < 3; ++d) s.pos[d] = (d < pl.dim) ? (uint32_t*)take(N * 4) : nullptr;
    s.C = take(N * pl.real_bytes);
    s.id = (uint32_t*)take(N * 4);
    s.rec = c->S.rec ? (uint4*)take(N * 16) : nullptr;
    s.cs = (uint32_t*)take((pl.ncell + 1) * 4);
    s.step = (int64_t*)take(8);
    for (int d = 0; d < 3; ++d) s.vel[d] = c->S.vel[d] ? take(N * pl.real_bytes) : nullptr;
    for (int d = 0; d < 6; ++d) s.rD[d] = c->S.rD[d] ? take(N * pl.real_bytes) : nullptr;
    s.grec = keeps_gen_rec(pl) ? (uint4*)take(N * 32) : nullptr;
}

void adj_layout(const ade_ctx* c, int64_t nsteps, int32_t K, int32_t ns, char* base, AdjLayout& L) {
    size_t off = 0;
    auto take = [&](size_t bytes) -> char* {
        off = (off + 255) & ~size_t(255);
        char* p = base ? base + off : nullptr;
        off += bytes;
        return p;
    };
    const Plan& pl = c->plan;
    const int64_t nck = (nsteps + K - 1) / K + 1;
    // one snapshot's size, as take_snap lays it out from an aligned offset
    size_t snap_bytes = 0;
    {
        Snap probe;
        take_snap(nullptr, snap_bytes, c, probe);
        snap_bytes = (snap_bytes + 255) & ~size_t(255);
    }
    const bool gpc = pl.general && pl.integrator == ADE_PC;
    auto seq = [&](SnapSeq& q, size_t count) {
        q.count = count;
        q.stride = snap_bytes;
        off = (off + 255) & ~size_t(255);
        size_t o = off;
        if (count) take_snap(base, o, c, q.first);
        off += count * snap_bytes;
    };
    seq(L.ck, (size_t)nck);
    L.pool = base;
    seq(L.seg, (size_t)K);
    L.pool_bytes = off;
    seq(L.segh, gpc ? (size_t)K : 0);
    const size_t N = (size_t)pl.N, rb = (size_t)pl.real_bytes;
    L.lam[0] = take(N * rb);
    L.lam[1] = take(N * rb);
    L.lam_s = take(N * rb);
    L.y = gpc ? take(N * rb) : nullptr;
    const bool pc = pl.integrator == ADE_PC;
    const bool packed = pl.dim == 2 && pl.real_bytes == 4;
    L.mu_s = pc ? take(N * rb) : nullptr;
    L.ch_s = pc ? take(N * rb) : nullptr;
    L.arec = packed ? (uint4*)take(N * 16) : nullptr;
    L.arec2 = (packed && pc) ? (uint4*)take(N * 16) : nullptr;
    L.pred = take((size_t)ns * rb);
    L.den = take((size_t)ns * rb);
    L.rw = take((size_t)ns * rb);
    L.J = (double*)take(8);
    L.gpart = (double*)take((size_t)pl.ntiles * kAdjMaxSubs * 3 * 8);
    L.grad = (double*)take(3 * 8);
    L.bytes = off + 256;
}

// one launch per snapshot (the arrays are small for the adjoint's problem
// sizes, so separate copies would be launch-bound)
int copy_state(const ade_ctx* c, const Snap& dst, const Snap& src) {
    const Plan& pl = c->plan;
    const uint32_t N = (uint32_t)pl.N, nc = (uint32_t)pl.ncell + 1;
    const uint32_t words = (uint32_t)pl.real_bytes / 4;
    SnapCopy a;
    for (int d = 0; d < 3; ++d) {
        a.dpos[d] = (d < pl.dim) ? dst.pos[d] : nullptr;
        a.spos[d] = (d < pl.dim) ? src.pos[d] : nullptr;
    }
    a.dC = static_cast<uint32_t*>(dst.C);
    a.sC = static_cast<const uint32_t*>(src.C);
    a.did = dst.id;
    a.sid = src.id;
    a.drec = (dst.rec && src.rec) ? dst.rec : nullptr;
    a.srec = src.rec;
    a.dcs = dst.cs;
    a.scs = src.cs;
    a.dstep = dst.step;
    a.sstep = src.step;
    a.n = N;
    a.ncs = nc;
    a.cwords = words;
    const uint32_t items = std::max(N * words, nc);
    a.nx = 0;
    uint32_t xitems = 0;
    auto extra = [&](void* d, const void* s, uint32_t nw) {
        if (!d || !s) return;
        a.dx[a.nx] = static_cast<uint32_t*>(d);
        a.sx[a.nx] = static_cast<const uint32_t*>(s);
        a.xn[a.nx] = nw;
        ++a.nx;
        xitems = std::max(xitems, nw);
    };
    for (int d = 0; d < 3; ++d) extra(dst.vel[d], src.vel[d], N * words);
    for (int d = 0; d < 6; ++d) extra(dst.rD[d], src.rD[d], N * words);
    extra(dst.grec, src.grec, N * 8);
    hipLaunchKernelGGL(k_copy_snap, dim3((items + 255) / 256), dim3(256), 0, c->stream, a);
    HIPCHK(hipGetLastError());
    if (a.nx > 0) {
        hipLaunchKernelGGL(k_copy_snap_x, dim3((xitems + 255) / 256), dim3(256), 0, c->stream, a);
        HIPCHK(hipGetLastError());
    }
    return ADE_OK;
}

Snap live(ade_ctx* c) {
    Snap s;
    for (int d = 0; d < 3; ++d) s.pos[d] = c->S.pos[d];
    s.C = c->S.C;
    s.id = c->S.id;
    s.rec = c->S.rec;
    s.cs = c->cell_start;
    s.step = c->step;
    for (int d = 0; d < 3; ++d) s.vel[d] = c->S.vel[d];
    for (int d = 0; d < 6; ++d) s.rD[d] = c->S.rD[d];
    s.grec = keeps_gen_rec(c->plan) ? c->S.grec : nullptr;
    return s;
}

StateArrays snap_arrays(const ade_ctx* c, const Snap& s) {
    StateArrays a = c->S;
    for (int d = 0; d < 3; ++d) a.pos[d] = s.pos[d] ? s.pos[d] : s.pos[0];
    a.C = s.C;
    a.id = s.id;
    a.rec = s.rec;
    for (int d = 0; d < 3; ++d) a.vel[d] = s.vel[d];
    for (int d = 0; d < 6; ++d) a.rD[d] = s.rD[d];
    a.grec = s.grec;
    return a;
}

int check_sensor_args(const ade_ctx* c, const double* d_xs, int32_t ns) {
    if (!c) return fail(ADE_EINVAL, "null ctx");
    if (!d_xs || ns <= 0) return fail(ADE_EINVAL, "sensors: null positions or n_sensors <= 0");
    if (c->plan.P != 1) return fail(ADE_EINVAL, "sensors and the adjoint need a single-plume context");
    if (!c->built) return fail(ADE_ESTATE, "cells not built");
    return ADE_OK;
}

// Sensors up to which each has a wavefront; more have a lane each.  A sensor's
// wavefront costs the same however many there are (it lists the rows with few of its
// lanes and adds 64 terms one after the other), a kernel of lanes takes the time of the
// slowest lane until they fill the chip.  The two are equal at about 20000 sensors
// (FP32, 64^2 to 512^2: 16384 sensors 23 and 28 us with 16 neighbours, 43 and 49 with
// 46; 32768 39 and 27, 81 and 59; a million-particle or a 3D plume at 33000 to 40000),
// in FP64 at 11000 (512^2: 8192 sensors 43 and 50 us, 16384 78 and 68; 3D 16000);
// 262144 sensors of 46 neighbours 604 and 214 us, in FP64 1160 and 225.
constexpr int kWaveSensors32 = 20480, kWaveSensors64 = 10240;

int launch_sensor_fwd(ade_ctx* c, const double* d_xs, int32_t ns, const StateArrays& S,
                      const uint32_t* cs, void* pred, void* den) {
    const Plan& pl = c->plan;
    const bool lane = ns > (pl.real_bytes == 4 ? kWaveSensors32 : kWaveSensors64);
    dim3 g(lane ? (ns + 255) / 256 : (ns + 3) / 4), b(256);
#define CALL(D, R, K)                                                                        \
    do {                                                                                     \
        auto kern = lane ? k_sensor_lane<D, R, K> : k_sensor_fwd<D, R, K>;                   \
        hipLaunchKernelGGL(kern, g, b, 0, c->stream, c->plumes, d_xs, ns, S, frame_of(c), cs, (R*)pred, (R*)den); \
    } while (0)
    ADE_DISPATCH3(pl.dim, pl.real_bytes, pl.kernel, CALL);
#undef CALL
    HIPCHK(hipGetLastError());
    return ADE_OK;
}

}  // namespace
}  // namespace ade

using namespace ade;

extern "C" {

int ade_sensor_interp(ade_ctx* c, const double* d_xs, int32_t n_sensors, void* d_Cs) {
    int rc = check_sensor_args(c, d_xs, n_sensors);
    if (rc) return rc;
    if (!d_Cs) return fail(ADE_EINVAL, "null output");
    return launch_sensor_fwd(c, d_xs, n_sensors, c->S, c->cell_start, d_Cs, nullptr);
}

int ade_adjoint_workspace_bytes(const ade_ctx* c, int64_t nsteps, int32_t ckpt_every, int32_t n_sensors,
                                size_t* bytes) {
    if (!c || !bytes) return fail(ADE_EINVAL, "null argument");
    if (nsteps < 1 || ckpt_every < 1 || n_sensors < 1)
        return fail(ADE_EINVAL, "nsteps, ckpt_every and n_sensors must be positive");
    AdjLayout L;
    adj_layout(c, nsteps, ckpt_every, n_sensors, nullptr, L);
    *bytes = L.bytes;
    return ADE_OK;
}

}  // extern "C"

namespace {

// misfit of the state S and the adjoint seed of its last step in lam
int misfit_and_seed(ade_ctx* c, const AdjLayout& L, const StateArrays& S, const double* d_xs, int32_t ns,
                    const void* d_obs, void* lam) {
    const Plan& pl = c->plan;
    const uint32_t N = (uint32_t)pl.N;
    hipStream_t st = c->stream;
    int rc;
    if ((rc = launch_sensor_fwd(c, d_xs, ns, S, c->cell_start, L.pred, L.den))) return rc;
    if (pl.real_bytes == 4)
        hipLaunchKernelGGL((k_sensor_resid<float>), dim3(1), dim3(256), 0, st, ns, (const float*)L.pred,
                           (const float*)L.den, (const float*)d_obs, (float*)L.rw, L.J);
    else
        hipLaunchKernelGGL((k_sensor_resid<double>), dim3(1), dim3(256), 0, st, ns, (const double*)L.pred,
                           (const double*)L.den, (const double*)d_obs, (double*)L.rw, L.J);
    HIPCHK(hipGetLastError());
    dim3 g((N + 255) / 256), b(256);
#define CALL(D, R, KK)                                                                             \
    hipLaunchKernelGGL((k_sensor_seed<D, R, KK>), g, b, 0, st, c->plumes, d_xs, ns, (const R*)L.rw, \
                       S, frame_of(c), N, (R*)lam)
    ADE_DISPATCH3(pl.dim, pl.real_bytes, pl.kernel, CALL);
#undef CALL
    HIPCHK(hipGetLastError());
    HIPCHK(hipMemsetAsync(L.gpart, 0, (size_t)pl.ntiles * kAdjMaxSubs * 3 * 8, st));
    return ADE_OK;
}

// the gradient from its nparts workgroup partials, and J, to the host
int reduce_to_host(ade_ctx* c, const AdjLayout& L, uint32_t nparts, double* h_J, double* h_grad) {
    hipStream_t st = c->stream;
    hipLaunchKernelGGL(k_grad_reduce, dim3(1), dim3(256), 0, st, L.gpart, nparts, L.grad);
    HIPCHK(hipGetLastError());
    double hostv[4];
    HIPCHK(hipMemcpyAsync(hostv, L.grad, 3 * 8, hipMemcpyDeviceToHost, st));
    HIPCHK(hipMemcpyAsync(hostv + 3, L.J, 8, hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
    for (int k = 0; k < 3; ++k) h_grad[k] = hostv[k];
    *h_J = hostv[3];
    return ADE_OK;
}

// The adjoint of a uniform flow.  The snapshots' part of the workspace holds
// the states (C only): all of them when they fit, else the checkpoints and one
// segment.
int adjoint_uniform(ade_ctx* c, const AdjLayout& L, int64_t nsteps, int32_t K, const double* d_xs, int32_t ns,
                    const void* d_obs, double* h_J, double* h_grad) {
    const Plan& pl = c->plan;
    const uint32_t N = (uint32_t)pl.N;
    const size_t sbytes = (size_t)N * (size_t)pl.real_bytes, slot = (sbytes + 255) & ~size_t(255);
    hipStream_t st = c->stream;
    const bool pc = pl.integrator == ADE_PC, packed = pl.dim == 2 && pl.real_bytes == 4;
    const uint32_t ab = adj_block(pl), asubs = kTile / ab;
    const size_t ashm = (size_t)ab * (size_t)pl.list_cap * 8u;
    if (ashm > kPairLdsMax) return fail(ADE_EINVAL, "candidate lists of the adjoint do not fit in LDS");

    char* pool = L.pool;
    size_t room = L.pool_bytes;
    uint4* arecs[2] = {L.arec, L.arec2};  // the passes' records, read and written in turn
    if (packed && !pc) {
        arecs[1] = reinterpret_cast<uint4*>(pool);
        const size_t rbytes = ((size_t)N * 16 + 255) & ~size_t(255);
        pool += rbytes;
        room -= rbytes;
    }
    const int64_t nck = (nsteps + K - 1) / K;
    const bool all = room / slot >= (size_t)nsteps + 1;
    if (!all && room / slot < (size_t)(nck + 1 + K)) return fail(ADE_EWORKSPACE, "adjoint workspace too small");
    // where state n lives: checkpoints 0 .. nck (the last one the final
    // state), then the segment's states by n mod K
    auto state = [&](int64_t n) -> void* {
        size_t k;
        if (all) k = (size_t)n;
        else if (n == nsteps) k = (size_t)nck;
        else if (n % K == 0) k = (size_t)(n / K);
        else k = (size_t)(nck + 1 + n % K);
        return pool + k * slot;
    };
    int rc = settle_lists(c);
    if (rc) return rc;
    // states n0 + 1 .. n1 from state n0, whose records S.rec holds
    auto advance = [&](int64_t n0, int64_t n1, bool count) -> int {
        uint4* rec[2] = {c->S.rec, pc ? c->S.rec : c->aux_rec};
        for (int64_t n = n0; n < n1; ++n)
            if ((rc = enqueue_uniform(c, state(n), rec[(n - n0) & 1], state(n + 1), rec[(n - n0 + 1) & 1], count)))
                return rc;
        return ADE_OK;
    };

    HIPCHK(hipMemcpyAsync(state(0), c->S.C, sbytes, hipMemcpyDeviceToDevice, st));
    if ((rc = advance(0, nsteps, true))) return rc;
    StateArrays fin = c->S;
    fin.C = state(nsteps);
    if ((rc = misfit_and_seed(c, L, fin, d_xs, ns, d_obs, L.lam[0]))) return rc;

    AdjLaunch base{};
    base.plumes = c->plumes;
    base.tiles = c->tiles;
    base.ntiles = pl.ntiles;
    base.S = c->S;
    base.cs = c->cell_start;
    base.gpart = L.gpart;
    {
        const PlumeDev& P = pl.plumes[0];
        double sp = 0;
        for (int k = 0; k < pl.dim; ++k) sp += P.vel[k] * P.vel[k];
        base.speed = std::sqrt(sp);
    }
    // the lists of the forward run, if the plume has them; the wavefronts of a tile in
    // at most kAdjMaxSubs workgroups: of 64 threads with one lane to one or two targets, of
    // 128 with two lanes to one or four to two, of 256 with four to one
    const PairLaunch fwd = pair_args(c, c->S.C, c->S.rec, c->S.C, 1.0, nullptr, nullptr);
    base.list = fwd.list;
    base.waves = fwd.waves;
    const uint32_t lwaves = (uint32_t)(kTile / 64) * (uint32_t)fwd.lanes / (uint32_t)fwd.targets;  // per tile
    const uint32_t lsubs = std::min(lwaves, kAdjMaxSubs), lblock = 64 * (lwaves / lsubs);
    const uint32_t parts = pl.ntiles * (fwd.list ? lsubs : asubs);
    auto run = [&](int mode, const void* u, const void* lam, const void* X, const uint4* rec, void* out, void* xh,
                   const void* next, uint4* rec_out) -> int {
        AdjLaunch a = base;
        a.u = u;
        a.lam = lam;
        a.X = X;
        a.arec = rec;
        a.lam_out = out;
        a.xh_out = xh;
        a.Xnext = next;
        a.arec_out = rec_out;
#define SHAPE(D, R, KK, M)                                                                                       \
    do {                                                                                                         \
        auto kern = k_adjoint_list<D, R, KK, M, 1, 1>;                                                           \
        if (fwd.targets == 2) kern = fwd.lanes == 4 ? k_adjoint_list<D, R, KK, M, 4, 2> : k_adjoint_list<D, R, KK, M, 1, 2>; \
        else if (fwd.lanes == 4) kern = k_adjoint_list<D, R, KK, M, 4, 1>;                                       \
        else if (fwd.lanes == 2) kern = k_adjoint_list<D, R, KK, M, 2, 1>;                                       \
        if (a.list) hipLaunchKernelGGL(kern, dim3(parts), dim3(lblock), 0, st, a, a.plumes, a.tiles);            \
        else hipLaunchKernelGGL((k_adjoint<D, R, KK, M>), dim3(parts), dim3(ab), (uint32_t)ashm, st, a, a.plumes, a.tiles); \
    } while (0)
#define CALL(D, R, KK)                                  \
    if (mode == kAdjEuler) SHAPE(D, R, KK, kAdjEuler);  \
    else if (mode == kAdjHalf) SHAPE(D, R, KK, kAdjHalf); \
    else SHAPE(D, R, KK, kAdjFull)
        ADE_DISPATCH3(pl.dim, pl.real_bytes, pl.kernel, CALL);
#undef CALL
#undef SHAPE
        HIPCHK(hipGetLastError());
        return ADE_OK;
    };
    const dim3 g((N + 255) / 256), b(256);
    int li = 0, ri = 0;
    for (int64_t n = nsteps - 1; n >= 0; --n) {
        const bool top = n == nsteps - 1;
        // entering an earlier segment: its states are recomputed (those of the
        // last one are still there)
        const bool enter = !all && !top && (n + 1) % K == 0;
        if (enter && n % K != 0) {
            const int64_t n0 = n / K * K;
            HIPCHK(launch_set_state(pl.dim, pl.real_bytes, c->S, state(n0), N, st));
            if ((rc = advance(n0, n, false))) return rc;
        }
        if (packed && (top || enter)) {
            hipLaunchKernelGGL(k_adj_pack, g, b, 0, st, c->S, (const float*)state(n), (const float*)L.lam[li], N,
                               arecs[ri]);
            HIPCHK(hipGetLastError());
        }
        const void* next = (n > 0 && (all || n % K != 0)) ? state(n - 1) : nullptr;
        if (pc) {
            if ((rc = run(kAdjHalf, L.lam[li], L.lam[li], state(n), arecs[0], L.mu_s, L.ch_s, nullptr, arecs[1])) ||
                (rc = run(kAdjFull, L.mu_s, L.lam[li], L.ch_s, arecs[1], L.lam[1 - li], nullptr, next, arecs[0])))
                return rc;
        } else {
            if ((rc = run(kAdjEuler, L.lam[li], L.lam[li], state(n), arecs[ri], L.lam[1 - li], nullptr, next,
                          arecs[1 - ri])))
                return rc;
            ri = 1 - ri;
        }
        li = 1 - li;
    }
    // leave the context at step nsteps (the forward run counted its steps)
    HIPCHK(launch_set_state(pl.dim, pl.real_bytes, c->S, state(nsteps), N, st));
    c->since += nsteps;
    return reduce_to_host(c, L, parts, h_J, h_grad);
}

// The adjoint of a velocity field over kept states.  A state is built where it is
// kept: the checkpoint at the start of each segment but the last, and all states of
// the last segment, by the forward run; the other states of a segment when the
// reverse sweep comes to it.  (Copied from the context's own arrays, and with the
// last segment run twice, a 128^2 adjoint of 60 steps made 68 more copies of two
// launches and 22 more steps of four.)
// The pass at a state hands lambda on in the order of the next pass's state, found
// from the inverse order that the placement leaves in the kept state's unused
// candidate records; 3D FP64 keeps none and gathers in a launch of its own.
int adjoint_field(ade_ctx* c, const AdjLayout& L, int64_t nsteps, int32_t K, const double* d_xs, int32_t ns,
                  const void* d_obs, double* h_J, double* h_grad) {
    int rc = ADE_OK;
    const Plan& pl = c->plan;
    const uint32_t N = (uint32_t)pl.N;
    hipStream_t st = c->stream;
    const int64_t nck = (nsteps + K - 1) / K, last0 = (nck - 1) * K;
    const bool pc = pl.integrator == ADE_PC;
    if ((size_t)kGenAdjBlock / 4 * (size_t)pl.list_cap * 8u > kPairLdsMax)
        return fail(ADE_EINVAL, "candidate lists of the adjoint do not fit in LDS");

    // the arrays of a kept state; records that it has no room for are those of the
    // last build
    auto kept = [&](const Snap& s) {
        GenState g{snap_arrays(c, s), s.cs, (uint32_t)pl.ncell + 1, s.step, reinterpret_cast<uint32_t*>(s.rec)};
        g.S.rec = nullptr;
        if (!keeps_gen_rec(pl)) g.S.grec = c->S.grec;
        return g;
    };
    // state n + 1 into `to` from state n, its half-step state into `half`
    auto step = [&](const GenState& from, const GenState& half, const GenState& to) -> int {
        if (!pc) {
            if ((rc = run_gen(c, kModeStep, nullptr, from))) return rc;
        } else {
            if ((rc = run_gen(c, kModeHalf, nullptr, from)) || (rc = enqueue_build_into(c, half, nullptr))) return rc;
            GenState mid = half;
            mid.step = from.step;
            if ((rc = run_gen(c, kModeFull, nullptr, mid))) return rc;
        }
        return enqueue_build_into(c, to, from.step);
    };
    const Snap first = last0 == 0 ? L.seg[0] : L.ck[0];
    if ((rc = copy_state(c, first, live(c)))) return rc;
    auto forward_home = [&](int64_t n) {
        if (n == nsteps) return gen_live(c);
        if (n >= last0) return kept(L.seg[(size_t)(n - last0)]);
        return n % K == 0 ? kept(L.ck[(size_t)(n / K)]) : gen_live(c);
    };
    for (int64_t n = 0; n < nsteps; ++n) {
        const GenState half = pc && n >= last0 ? kept(L.segh[(size_t)(n - last0)]) : gen_live(c);
        if ((rc = step(forward_home(n), half, forward_home(n + 1)))) return rc;
    }
    if ((rc = misfit_and_seed(c, L, c->S, d_xs, ns, d_obs, L.lam[0]))) return rc;

    // lambda of id order in a state's cell order
    auto gather = [&](const StateArrays& S, const void* lam, void* out) -> int {
        dim3 g((N + 255) / 256), b(256);
        if (pl.real_bytes == 4)
            hipLaunchKernelGGL((k_adj_gather<float>), g, b, 0, st, S, (const float*)lam, N, (float*)out);
        else
            hipLaunchKernelGGL((k_adj_gather<double>), g, b, 0, st, S, (const double*)lam, N, (double*)out);
        HIPCHK(hipGetLastError());
        return ADE_OK;
    };
    // a pass at state `at` over `in` (its cell order); the output goes to next in
    // the order that inv gives, and to `id` in id order
    auto pass = [&](int mode, const GenState& at, const void* in, const void* lam_id, void* id, void* next,
                    const uint32_t* inv) -> int {
        AdjGenLaunch g;
        g.plumes = c->plumes;
        g.tiles = c->tiles;
        g.ntiles = pl.ntiles;
        g.list_cap = pl.list_cap;
        g.S = at.S;
        g.cell_start = at.cell_start;
        g.lam_s = in;
        g.lam_id = lam_id;
        g.lam_out = id;
        g.lam_next = inv ? next : nullptr;
        g.inv = inv;
        g.gpart = L.gpart;
        HIPCHK(launch_adjoint_gen(pl.dim, pl.real_bytes, pl.kernel, mode, g, kGenAdjBlock, st));
        return ADE_OK;
    };

    // reverse sweep, segment by segment
    void* sorted[2] = {L.lam_s, L.lam[1]};  // Euler: lambda in cell order, in turn (id order: lam[0])
    int li = 0;  // predictor-corrector: lambda in id order in lam[li], in cell order in lam_s
    for (int64_t n0 = last0; n0 >= 0; n0 -= K) {
        const int64_t n1 = std::min<int64_t>(n0 + K, nsteps);
        auto home = [&](int64_t n) {
            return kept(n == n0 && n0 != last0 ? L.ck[(size_t)(n0 / K)] : L.seg[(size_t)(n - n0)]);
        };
        auto half = [&](int64_t n) { return pc ? kept(L.segh[(size_t)(n - n0)]) : gen_live(c); };
        if (n0 != last0) {
            if (!keeps_gen_rec(pl)) HIPCHK(launch_gen_rec(pl.dim, pl.real_bytes, home(n0).S, N, st));
            for (int64_t n = n0; n + 1 < n1; ++n)
                if ((rc = step(home(n), half(n), home(n + 1)))) return rc;
            if (pc && ((rc = run_gen(c, kModeHalf, nullptr, home(n1 - 1))) ||
                       (rc = enqueue_build_into(c, half(n1 - 1), nullptr))))
                return rc;
        }
        bool ready = false;  // lambda is in the cell order of the next pass
        for (int64_t n = n1 - 1; n >= n0; --n) {
            const GenState at = home(n);
            // state 0 was copied, without its inverse order
            const uint32_t* inv = n > 0 ? at.inv : nullptr;
            if (pc) {
                // y = L2 lambda at the half-step state (its own cells and
                // order), then lambda^n = lambda + dt y + dt^2/2 L1 y here
                const GenState mid = half(n);
                if (!ready && (rc = gather(mid.S, L.lam[li], L.lam_s))) return rc;
                if ((rc = pass(kAdjGenHalf, mid, L.lam_s, nullptr, inv ? nullptr : L.y, L.y, inv))) return rc;
                if (!inv && (rc = gather(at.S, L.y, L.lam_s))) return rc;
                const uint32_t* inv_next = n > n0 ? half(n - 1).inv : nullptr;
                if ((rc = pass(kAdjGenFull, at, inv ? L.y : L.lam_s, L.lam[li], L.lam[1 - li], L.lam_s, inv_next)))
                    return rc;
                li = 1 - li;
                ready = inv_next != nullptr;
            } else {
                if (!ready && (rc = gather(at.S, L.lam[0], sorted[0]))) return rc;
                const uint32_t* inv_next = n - 1 > 0 && n > n0 ? home(n - 1).inv : nullptr;
                if ((rc = pass(kAdjGenEuler, at, sorted[0], nullptr, inv_next ? nullptr : L.lam[0], sorted[1], inv_next)))
                    return rc;
                if (inv_next) std::swap(sorted[0], sorted[1]);
                ready = inv_next != nullptr;
            }
        }
    }
    // the context is at step nsteps; its records, where the sweep made others
    if (!keeps_gen_rec(pl) && nck > 1) HIPCHK(launch_gen_rec(pl.dim, pl.real_bytes, c->S, N, st));
    return reduce_to_host(c, L, pl.ntiles * kAdjMaxSubs, h_J, h_grad);
}

// The adjoint run of ade_adjoint over a workspace of ws_bytes at d_ws
// (256-byte aligned; arguments checked by the caller).
int adjoint_run(ade_ctx* c, int64_t nsteps, int32_t K, const double* d_xs, int32_t ns, const void* d_obs,
                void* d_ws, size_t ws_bytes, double* h_J, double* h_grad) {
    AdjLayout L;
    adj_layout(c, nsteps, K, ns, nullptr, L);
    if (ws_bytes < L.bytes) return fail(ADE_EWORKSPACE, "adjoint workspace too small: need %zu bytes", L.bytes);
    adj_layout(c, nsteps, K, ns, static_cast<char*>(d_ws), L);
    if (c->plan.general) return adjoint_field(c, L, nsteps, K, d_xs, ns, d_obs, h_J, h_grad);
    return adjoint_uniform(c, L, nsteps, K, d_xs, ns, d_obs, h_J, h_grad);
}

int check_adjoint_args(ade_ctx* c, int64_t nsteps, int32_t K, const double* d_xs, int32_t ns, const void* d_obs,
                       double* h_J, double* h_grad) {
    int rc = check_sensor_args(c, d_xs, ns);
    if (rc) return rc;
    if (!d_obs || !h_J || !h_grad) return fail(ADE_EINVAL, "null argument");
    if (nsteps < 1 || K < 1) return fail(ADE_EINVAL, "nsteps and ckpt_every must be positive");
    return ADE_OK;
}

// Adjoint workspace of the allocation-free entry point: a fixed array in the
// library's device memory (one copy per GPU, held until the process ends).
// Host code reaches it only through the address hipGetSymbolAddress gives
// on each device, never through the array's name.
constexpr size_t kNoAllocScratchBytes = size_t(64) << 20;
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];

// The scratch array's address on the device of stream st (looked up once per
// device, with that device current).
int scratch_on(hipStream_t st, void** out) {
    int cur = 0, dev = 0;
    HIPCHK(hipGetDevice(&cur));
    dev = cur;
    if (st) HIPCHK(hipStreamGetDevice(st, &dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(ADE_EINVAL, "device %d out of range", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        if (dev != cur) HIPCHK(hipSetDevice(dev));
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (dev != cur) HIPCHK(hipSetDevice(cur));
        if (e != hipSuccess || !p)
            return fail(ADE_EHIP, "hipGetSymbolAddress of the scratch array: %s", hipGetErrorString(e));
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return ADE_OK;
}

}  // namespace

extern "C" {

int ade_adjoint(ade_ctx* c, int64_t nsteps, int32_t K, const double* d_xs, int32_t ns, const void* d_obs,
                void* d_ws, size_t ws_bytes, double* h_J, double* h_grad) {
    int rc = check_adjoint_args(c, nsteps, K, d_xs, ns, d_obs, h_J, h_grad);
    if (rc) return rc;
    if (!d_ws) return fail(ADE_EINVAL, "null workspace");
    if (reinterpret_cast<uintptr_t>(d_ws) & 255u) return fail(ADE_EINVAL, "workspace must be 256-byte aligned");
    return adjoint_run(c, nsteps, K, d_xs, ns, d_obs, d_ws, ws_bytes, h_J, h_grad);
}

int ade_adjoint_noalloc_max_bytes(size_t* bytes) {
    if (!bytes) return fail(ADE_EINVAL, "null argument");
    *bytes = kNoAllocScratchBytes;
    return ADE_OK;
}

int ade_adjoint_noalloc(ade_ctx* c, int64_t nsteps, int32_t K, const double* d_xs, int32_t ns, const void* d_obs,
                        double* h_J, double* h_grad) {
    int rc = check_adjoint_args(c, nsteps, K, d_xs, ns, d_obs, h_J, h_grad);
    if (rc) return rc;
    AdjLayout L;
    adj_layout(c, nsteps, K, ns, nullptr, L);
    if (L.bytes > kNoAllocScratchBytes)
        return fail(ADE_EWORKSPACE,
                    "ade_adjoint_noalloc: this run needs %zu bytes of adjoint workspace, above the %zu bytes of "
                    "the library's static scratch array; use ade_adjoint with a workspace",
                    L.bytes, kNoAllocScratchBytes);
    void* ws = nullptr;
    if ((rc = scratch_on(c->stream, &ws))) return rc;
    return adjoint_run(c, nsteps, K, d_xs, ns, d_obs, ws, kNoAllocScratchBytes, h_J, h_grad);
}

}  // extern "C"
