// ade_list.h -- the walk of a wavefront's neighbour lists (kernels_list.hip
// describes their layout and builds them); shared by the pair sum and the adjoint
// of a uniform flow.
#pragma once

#include <type_traits>

#include "ade_walk.h"

namespace ade {

// rows before the entries: the counts, which only a second target needs
template <int T>
constexpr uint32_t kCountRows = T == 2 ? 1u : 0u;

template <int DIM>
struct Entry {
    static constexpr int kPerRow = DIM == 2 ? 2 : 1;
};

// rows of nb batches
template <int DIM>
__device__ __forceinline__ uint32_t batch_rows(uint32_t nb) {
    return nb * (kListBatch / Entry<DIM>::kPerRow);
}

// Entry p of a group stands in slot p / G of this lane of it: the lanes take entries in
// turn, two lanes in alternating order (0 1, 1 0, 0 1, ...).  Consecutive entries lie side
// by side along x; if one of two lanes always took the left one of each pair, the first-order
// terms of a concentration gradient would pile up in the partial sums and cancel only
// between the lanes (400^2 in FP32, error of the right-hand side against 64 bits: 50
// neighbours 1.228e-6 in turn, 1.171e-6 alternating, 1.152e-6 over the row windows,
// whose other candidates mix the turns; 21 neighbours 9.87e-7, 9.63e-7, 9.64e-7).  Four lanes
// are no worse in turn (1.173e-6; alternating 1.182e-6).
template <int G>
__device__ __forceinline__ uint32_t entry_lane(uint32_t p) {
    return G == 2 ? (p ^ (p >> 1)) & 1u : p % G;
}
// a lane's share of its group's m entries
template <int G>
__device__ __forceinline__ uint32_t lane_share(uint32_t m, uint32_t lj) {
    if (G == 2) return m / 2u + ((m & 1u) && entry_lane<2>(m - 1u) == lj ? 1u : 0u);
    return m > lj ? (m - lj + G - 1) / G : 0u;
}

// The targets of a lane's group in the wavefront whose first target is i0 (end:
// past the tile's last).
template <int G, int T>
struct ListTargets {
    uint32_t lane, lj, iA, iB;
    bool actA, actB;
    __device__ __forceinline__ ListTargets(uint32_t i0, uint32_t end) {
        lane = threadIdx.x & (kWave - 1);
        lj = lane % G;
        const uint32_t ia = i0 + T * (lane / G), ib = ia + T - 1;
        actA = ia < end;
        actB = T == 2 && ib < end;
        // past the end of a ragged tile a group keeps a copy of a valid target
        // (its sums are discarded)
        iA = actA ? ia : i0;
        iB = actB ? ib : iA;
    }
};

// sum over the lanes of a group (fixed order: deterministic)
template <int G, typename real>
__device__ __forceinline__ real group_sum(real v) {
    if (G >= 2) v += __shfl_xor(v, 1, kWave);
    if (G >= 4) v += __shfl_xor(v, 2, kWave);
    return v;
}

// Walks the lists of a wavefront.  pass(k0, k1, second,
// walk) is called once with the group's two targets (T = 1: twice the same), or,
// where the wavefront holds a pair too far apart, with (a, a) and then (second)
// (b, b); it calls walk(one), and one(c, keep) gets every record of the list,
// fetch(k) of its byte offset among 16-byte records.  keep false: a slot past
// the end of the lane's list, which holds the record of target k0.
template <int DIM, int G, int T, typename Fetch, typename Pass>
__device__ __forceinline__ void walk_lists(const uint32_t* __restrict__ list, const ListWave& head, const PlumeDev& P,
                                           const ListTargets<G, T>& q, Fetch&& fetch, Pass&& pass) {
    constexpr int B = kListBatch, kPer = Entry<DIM>::kPerRow, RB = B / kPer;
    using CandT = decltype(fetch(0u));
    const uint32_t* __restrict__ rows = list + (size_t)head.row * kWave;
    const uint32_t words = T == 2 ? rows[q.lane] : 0u;
    // 2D: entries count from the wavefront's base; a window past the end of
    // the plume goes on at its start
    const bool wraps = DIM == 2 && P.n > 65536u && head.base + 65536u > P.n;
    const bool merged = T == 1 || !(head.nb & ListWave::kTwoPasses);
    uint32_t row = kCountRows<T>;
    const int npass = merged ? 1 : 2;
    for (int ps = 0; ps < npass; ++ps) {
        const bool second = ps == 1;
        const uint32_t k0 = second ? q.iB : q.iA, k1 = merged ? q.iB : k0;
        const uint32_t own = lane_share<G>(second ? words >> 16 : words & 0xffffu, q.lj);
        const uint32_t nb = second ? head.nb2 : head.nb & ~ListWave::kTwoPasses;
        // batches in which every lane has entries of its own: the second
        // target needs no end-of-list test there (T = 1 needs none at all)
        const uint32_t nfull = T == 1 ? nb : second ? head.full >> 16 : head.full & 0xffffu;
        const uint32_t* __restrict__ L = rows + (size_t)row * kWave;  // uniform; the lane is added to the load
        pass(k0, k1, second, [&](auto&& one) {
            auto walk = [&](auto wrap) {
                constexpr bool kWrap = decltype(wrap)::value;
                const uint32_t origin = DIM == 2 ? (P.poff + (kWrap ? 0u : head.base)) * kRecBytes : 0u;
                uint32_t e0[RB], e1[RB];
                CandT c0[B], c1[B];
                auto load = [&](uint32_t(&e)[RB], uint32_t it) {
#pragma unroll
                    for (int r = 0; r < RB; ++r) e[r] = L[(it * RB + r) * kWave + q.lane];
                };
                auto get = [&](CandT(&c)[B], const uint32_t(&e)[RB]) {
#pragma unroll
                    for (int k = 0; k < B; ++k) {
                        uint32_t at;
                        if (DIM == 2) {
                            uint32_t i = (k & 1) ? e[k / kPer] >> 16 : e[k / kPer] & 0xffffu;
                            if (kWrap) {
                                i += head.base;
                                i = min(i, i - P.n);
                            }
                            at = i * kRecBytes + origin;
                        } else {
                            at = e[k];
                        }
                        c[k] = fetch(at);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                };
                auto eval = [&](const CandT(&c)[B], uint32_t it) {
                    if (it < nfull) {
#pragma unroll
                        for (int k = 0; k < B; ++k) one(c[k], true);
                    } else {
#pragma unroll
                        for (int k = 0; k < B; ++k) one(c[k], it * B + k < own);
                    }
                };
                // entries two batches ahead of their evaluation, records one (the
                // lists end with room for the entries read past the last batch)
                load(e0, 0u);
                load(e1, 1u);
                get(c0, e0);
                load(e0, 2u);
                for (uint32_t it = 1;; it += 2) {
                    if (it >= nb) {
                        eval(c0, it - 1);
                        break;
                    }
                    get(c1, e1);
                    load(e1, it + 2);
                    eval(c0, it - 1);
                    if (it + 1 >= nb) {
                        eval(c1, it);
                        break;
                    }
                    get(c0, e0);
                    load(e0, it + 3);
                    eval(c1, it);
                }
            };
            if (nb > 0) {
                if (DIM == 2 && wraps) walk(std::integral_constant<bool, true>{});
                else walk(std::integral_constant<bool, false>{});
            }
        });
        row += batch_rows<DIM>(nb);
    }
}

}  // namespace ade
