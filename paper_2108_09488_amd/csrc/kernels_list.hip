// kernels_list.hip -- neighbour lists of a uniform flow and the pair sum over
// them (gfx950).
//
// A uniform flow keeps the relative positions of a plume's particles, so their
// neighbours are those of the build for the whole run.  k_list writes, once per
// build, what a group of lanes (G lanes serving T neighbouring targets, the
// launch shape) has to read: the records within the support of any of its
// targets.  k_pair_list then evaluates only those, step after step, where the
// row windows of kernels_pair.hip hold 1.5 (2D) to 2 (3D) candidates per
// neighbour and cost a window search and a cursor per launch.
//
// What bounds it: VALU issue (86% of the slots in 3D, 65% in the 2D sweep), with
// the L1 lookups of the gathers close behind in 2D.  The list costs 2 bytes (2D) or
// 4 (3D) per entry and launch.
// Measured per update launch against the row windows: 128^3 plume (256
// neighbours) 870 -> 475 us, the six-plume sweep 96 -> 68 us, the 256-plume
// ensemble 235 -> 201 us, a 512^2 plume (46 neighbours) 24 -> 13.5 us; the build
// takes about two such launches.  Measured and not taken: the group's records
// copied to LDS first with one target a group (3D 618 us, sweep 81 us, ensemble
// 213 us: the copy's latency per workgroup outweighed the cheaper gathers), and
// 2 entries a batch (sweep +6%).
//
// Layout.  A wavefront's lists are `rows` rows of 64 words, one word per lane:
// with two targets a group row 0 holds the entry counts of the lane's group, then
// come the entries, which the group's lanes take in turn (entry_lane).  Every load of a row is coalesced; what is uniform, ListWave, comes
// through the scalar unit.  2D: two 16-bit entries a word,
// record numbers from the wavefront's base (a window of 65536 records around its
// targets, modulo the plume's particles).  3D: one 32-bit byte offset a word (a
// window of pencils spans too many records).  Entries past a lane's count up to
// the wavefront's last batch are the group's own target, whose term is zero.
//
// A wavefront holding two targets too far apart to share separations
// (pair_rows) stores the two targets' own lists one after the other; both
// kernels then take two passes.
#include <hip/hip_ext.h>

#include "ade_list.h"
#include "ade_pair.h"

namespace ade {

namespace {

__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, o, kWave));
    return __builtin_amdgcn_readfirstlane(v);
}
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v = min(v, (uint32_t)__shfl_xor((int)v, o, kWave));
    return __builtin_amdgcn_readfirstlane(v);
}

// position of record k (byte offset / 16)
template <int DIM, typename real>
__device__ __forceinline__ uint3 pos_at(const uint4* __restrict__ rec, const uint32_t* const (&pos)[3], uint32_t k) {
    if constexpr (Rec<DIM, real>::kStageable) {
        const uint4 r = rec[k];
        return make_uint3(r.x, r.y, (DIM == 3) ? r.z : 0u);
    } else {
        return make_uint3(pos[0][k], pos[1][k], (DIM == 3) ? pos[2][k] : 0u);
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// list build: one wavefront per workgroup, over the row windows of
// kernels_pair.hip
// ---------------------------------------------------------------------------
template <int DIM, typename real, int G, int T>
__global__ __launch_bounds__(64) void k_list(ListBuild a, const PlumeDev* __restrict__ plumes,
                                             const TileDev* __restrict__ tiles) {
    extern __shared__ uint2 lds_list[];
    constexpr uint32_t kGroups = kWave / G, kTargets = kGroups * T, kWaves = kTile / kTargets;
    const TileDev t = tiles[blockIdx.x / kWaves];
    const uint32_t i0 = t.start + (blockIdx.x % kWaves) * kTargets;
    const ListPlume lp = a.lplumes[t.plume];
    ListWave head{i0, t.end, t.plume, 0u, 0u, 0u, 0u, 0u};
    if (i0 >= t.end || lp.rows == 0u) {  // no targets, or a plume without lists
        head.end = 0u;
        if (threadIdx.x == 0) a.waves[blockIdx.x] = head;
        return;
    }
    const PlumeDev P = plumes[t.plume];
    head.row = lp.row0 + (i0 - P.poff) / kTargets * lp.rows;
    uint32_t* out = a.list + (size_t)head.row * kWave;
    uint16_t* out2 = reinterpret_cast<uint16_t*>(out);

    const uint32_t lane = threadIdx.x, g = lane / G, lj = lane % G;
    const uint32_t ia = i0 + T * g, ib = ia + T - 1;
    const bool actA = ia < t.end, actB = ib < t.end;
    const uint32_t iA = actA ? ia : i0, iB = actB ? ib : iA;
    const uint4* __restrict__ rec = a.rec;
    auto target = [&](uint32_t k) {
        const uint3 p = pos_at<DIM, real>(rec, a.spos, k);
        return make_target<DIM>(P, p.x, p.y, p.z);
    };

    // 2D: the first record of the wavefront's window: the start of the row
    // below the lowest one that a target of it can reach (the targets ascend
    // in rows; one row more for a pair whose second target is the lower one)
    uint32_t base = 0;
    if (DIM == 2 && P.n > 65536u) {
        const Target first = target(i0);
        const int row = wrap_row(P, first.ry - P.R - 1);
        base = cell_start_at(a.cell_start, row_base(P, row, 0)) - P.poff;
    }
    base = __builtin_amdgcn_readfirstlane(base);
    head.base = base;

    int pry = 0, prz = 0;
    const bool close = T == 1 || pair_rows<DIM>(P, target(iA), target(iB), pry, prz);
    const bool merged = __builtin_amdgcn_ballot_w64(!close) == 0ull;
    const int npass = merged ? 1 : 2;
    uint2* list = lds_list + g;
    // a little beyond the support: the pair sum forms the second target's
    // separation as here, with one rounding more
    const real H2 = h2_of<real>(P) * (real)(1.0 + 9.5367431640625e-07);
    const uint32_t cap = lp.rows;
    uint32_t row = kCountRows<T>, words = 0;
    bool bad = false;
    auto entry = [&](uint32_t k) {  // 2D: the 16-bit entry of record byte offset k
        uint32_t e = k / kRecBytes - P.poff - base;
        if ((int32_t)e < 0) e += P.n;
        if (e > 0xffffu) bad = true;
        return e;
    };
    auto put = [&](uint32_t s, uint32_t dst, uint32_t k) {  // slot s of lane dst: record byte offset k
        const uint32_t r = row + s / Entry<DIM>::kPerRow;
        if (r >= cap) {
            bad = true;
        } else if (DIM == 2) {
            out2[(r * kWave + dst) * 2u + (s & 1u)] = (uint16_t)entry(k);
        } else {
            out[r * kWave + dst] = k;
        }
    };
    for (int pass = 0; pass < npass; ++pass) {
        const bool second = pass == 1;
        const uint32_t k0 = second ? iB : iA, k1 = merged ? iB : k0;
        const Target T0 = target(k0), T1 = target(k1);
        const bool active = actA && !(second && !actB);
        uint32_t total = 0;
        if (!active) {
            list[0] = make_uint2(kListEndStart, kListEndEnd);
        } else if (T == 2 && merged) {
            if (G == 1) {
                total = build_union<DIM>(P, a.cell_start, T0, T1, pry, prz, list, kGroups);
            } else {
                const int ny = 2 * P.R + 1 + (pry != 0 ? 1 : 0);
                const int nz = (DIM == 3) ? 2 * P.R + 1 + (prz != 0 ? 1 : 0) : 1;
                const float dxc = (float)(int32_t)(T1.ux - T0.ux) * P.cellx;
                total = build_rows_quad(
                    [&](int oy, int oz) { return union_row<DIM>(P, a.cell_start, T0, T1, dxc, pry, prz, oy, oz); },
                    ny, nz, min(0, pry) - P.R, (DIM == 3) ? min(0, prz) - P.R : 0, list, kGroups);
            }
        } else {
            total = build_list<DIM, G>(P, a.cell_start, T0, list, kGroups);
        }
        const real bx = (real)(int32_t)(T1.ux - T0.ux);
        const real by = (real)(int32_t)(T1.uy - T0.uy);
        const real bz = (DIM == 3) ? (real)(int32_t)(T1.uz - T0.uz) : (real)0;
        uint32_t m = 0;     // the group's entries so far (the same in its lanes)
        uint32_t half = 0;  // 2D, G = 1: the even entry of a word that is not complete
        struct At {
            uint32_t k;
            uint3 p;
        };
        walk_list_fn<G, 4>(
            k0, list, kGroups, total, lj,
            [&](uint32_t k) { return At{k, pos_at<DIM, real>(rec, a.spos, k / kRecBytes)}; },
            [&](const At& c, bool keep) {
                const real dx = (real)(int32_t)(T0.ux - c.p.x);
                const real dy = (real)(int32_t)(T0.uy - c.p.y);
                const real dz = (DIM == 3) ? (real)(int32_t)(T0.uz - c.p.z) : (real)0;
                real r2 = dx * dx;
                r2 = fmar(dy, dy, r2);
                if (DIM == 3) r2 = fmar(dz, dz, r2);
                bool hit;
                if (T == 2) {
                    // the targets themselves are listed too: their own terms are 0
                    const real ex = dx + bx, ey = dy + by, ez = dz + bz;
                    real q2 = ex * ex;
                    q2 = fmar(ey, ey, q2);
                    if (DIM == 3) q2 = fmar(ez, ez, q2);
                    hit = keep && (r2 < q2 ? r2 : q2) <= H2;
                } else {
                    hit = keep && r2 > (real)0 && r2 <= H2;
                }
                if (G == 1) {
                    if (hit) {
                        if (DIM == 2) {
                            const uint32_t e = entry(c.k), r = row + m / 2u;
                            if (m & 1u) {
                                if (r < cap) out[r * kWave + lane] = half | (e << 16);
                                else bad = true;
                            }
                            half = e;
                        } else {
                            put(m, lane, c.k);
                        }
                        ++m;
                    }
                } else {
                    // hits of the lower lanes of the wavefront, less those
                    // below the group
                    const uint64_t bal = __builtin_amdgcn_ballot_w64(hit);
                    const uint32_t lower = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
                    const uint32_t upto = lower + (hit ? 1u : 0u);
                    const uint32_t first = quad_perm<G == 4 ? 0x00 : 0xA0>(lower);  // [0,0,0,0] / [0,0,2,2]
                    const uint32_t last = quad_perm<G == 4 ? 0xFF : 0xF5>(upto);    // [3,3,3,3] / [1,1,3,3]
                    const uint32_t p = m + lower - first;
                    if (hit) put(p / G, (lane & ~(uint32_t)(G - 1)) + entry_lane<G>(p), c.k);
                    m += last - first;
                }
            });
        // up to the wavefront's last batch: the pass's own target
        const uint32_t own = lane_share<G>(m, lj);
        const uint32_t nb = (wave_max(own) + kListBatch - 1) / kListBatch;
        if (DIM == 2 && G == 1 && (m & 1u)) put(m - 1u, lane, (half + base) % P.n * kRecBytes + P.poff * kRecBytes);
        for (uint32_t s = own; s < nb * kListBatch; ++s) put(s, lane, k0 * kRecBytes);
        if (m > 0xffffu) bad = true;
        words |= (m & 0xffffu) << (second ? 16 : 0);
        row += batch_rows<DIM>(nb);
        const uint32_t full = wave_min(own) / kListBatch;
        if (second) {
            head.nb2 = nb;
            head.full |= full << 16;
        } else {
            head.nb = nb | (merged ? 0u : ListWave::kTwoPasses);
            head.full = full;
        }
    }
    if (T == 2) out[lane] = words;
    if (!Rec<DIM, real>::kStageable && lj == 0) {  // 3D FP64: the targets' position records
        auto pack = [&](uint32_t k) { a.pos[k] = make_uint4(a.spos[0][k], a.spos[1][k], a.spos[2][k], 0u); };
        if (actA) pack(iA);
        if (T == 2 && actB) pack(iB);
    }
    if (lane == 0) a.waves[blockIdx.x] = head;
    if (bad) a.over[t.plume] = 1u;
}

// ---------------------------------------------------------------------------
// the pair sum over the lists
// ---------------------------------------------------------------------------
template <int DIM, typename real, int KERN, int MODE, int G, int T, bool ZC>
__device__ __forceinline__ void list_item(const PairLaunch& a, const PlumeDev* __restrict__ plumes,
                                          uint32_t w) {
    // The wavefront's number among all: a workgroup holds a whole number of them.
    // Its head comes in one scalar load; by way of its tile, its plume's lists and
    // then their head (three loads in a chain) the 47^3 FP64 kernel takes 37 us (35
    // now), the 128-plume ensemble's quads 270 us (257).
    const uint32_t wv = __builtin_amdgcn_readfirstlane(w * ((uint32_t)a.block / kWave) + threadIdx.x / kWave);
    const ListWave head = a.waves[wv];
    if (head.i0 >= head.end) return;  // ragged last tile, or a plume whose row windows are walked
    const PlumeDev P = plumes[head.plume];
    const ListTargets<G, T> q(head.i0, head.end);
    const real* __restrict__ Cp = static_cast<const real*>(a.Cpair);
    constexpr bool kRec = Rec<DIM, real>::kStageable;
    const uint4* __restrict__ rec = kRec ? a.rec : a.list_pos;
    // a particle, from its record (3D FP64: its position record and its C)
    auto fetch = [&](uint32_t k) {  // 32-bit byte offset from a uniform base
        const uint4 r = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(rec) + k);
        if constexpr (kRec) return unpack<DIM, real>(r);
        else return Cand<real>{r.x, r.y, r.z, *reinterpret_cast<const real*>(reinterpret_cast<const char*>(Cp) + k / 2u)};
    };
    auto part = [&](uint32_t k) { return fetch(k * kRecBytes); };
    const PairTerm<DIM, real, KERN, ZC> term = make_term<DIM, real, KERN, ZC>(P);
    real accA = (real)0, accB = (real)0;
    walk_lists<DIM, G, T>(a.list, head, P, q, fetch, [&](uint32_t k0, uint32_t k1, bool second, auto&& walk) {
        const Cand<real> T0 = part(k0), T1 = part(k1);
        const real bx = (real)(int32_t)(T1.x - T0.x);
        const real by = (real)(int32_t)(T1.y - T0.y);
        const real bz = (DIM == 3) ? (real)(int32_t)(T1.z - T0.z) : (real)0;
        real acc0 = (real)0, acc1 = (real)0;
        walk([&](const Cand<real>& c, bool keep) {
            const real dx = (real)(int32_t)(T0.x - c.x);
            const real dy = (real)(int32_t)(T0.y - c.y);
            const real dz = (DIM == 3) ? (real)(int32_t)(T0.z - c.z) : (real)0;
            term.sep(dx, dy, dz, T0.C, c.C, true, acc0);
            if constexpr ((MODE & kModeExact) != 0)
                term.sep((real)(int32_t)(T1.x - c.x), (real)(int32_t)(T1.y - c.y), (real)0, T1.C, c.C, keep, acc1);
            else if (T == 2)
                term.sep(dx + bx, dy + by, dz + bz, T1.C, c.C, keep, acc1);
        });
        if (second) {
            accB = acc0;
        } else {
            accA = acc0;
            accB = acc1;
        }
    });
    accA = group_sum<G>(accA);
    if (T == 2) accB = group_sum<G>(accB);
    if (q.lj == 0 && q.actA) finish_target<DIM, real, KERN, MODE>(a, P, part(q.iA), q.iA, accA);
    if (T == 2 && q.lj == (G == 1 ? 0u : 1u) && q.actB) finish_target<DIM, real, KERN, MODE>(a, P, part(q.iB), q.iB, accB);
}

template <int DIM, typename real, int KERN, int MODE, int G, int T, bool ZC>
__global__ __launch_bounds__(256) void k_pair_list(PairLaunch a, const PlumeDev* __restrict__ plumes,
                                                   uint32_t nwork) {
    advance_step(a);
    if (a.persistent == 0) {
        list_item<DIM, real, KERN, MODE, G, T, ZC>(a, plumes, xcd_remap(blockIdx.x, gridDim.x, a.xcd_group));
        return;
    }
    const uint32_t nx = 8, x = blockIdx.x % nx, k = blockIdx.x / nx;
    const uint32_t per_x = (gridDim.x + nx - 1 - x) / nx;
    for (uint32_t m = k;; m += per_x) {
        const uint32_t w = xcd_item(x, m, nwork, a.xcd_group);
        if (w >= nwork) break;
        list_item<DIM, real, KERN, MODE, G, T, ZC>(a, plumes, w);
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <int DIM, typename real, int G, int T>
static void launch_list_s(const ListBuild& a, hipStream_t s) {
    constexpr uint32_t kWaves = kTile / (kWave / G * T);
    const size_t shm = (size_t)(kWave / G) * (size_t)a.list_cap * 8u;
    hipLaunchKernelGGL((k_list<DIM, real, G, T>), dim3(a.ntiles * kWaves), dim3(kWave), shm, s, a, a.plumes, a.tiles);
}

template <int DIM, typename real>
static void launch_list_t(const ListBuild& a, hipStream_t s) {
    if (a.targets == 2 && a.lanes == 4) launch_list_s<DIM, real, 4, 2>(a, s);
    else if (a.targets == 2) launch_list_s<DIM, real, 1, 2>(a, s);
    else if (a.lanes == 4) launch_list_s<DIM, real, 4, 1>(a, s);
    else if (a.lanes == 2) launch_list_s<DIM, real, 2, 1>(a, s);
    else launch_list_s<DIM, real, 1, 1>(a, s);
}

hipError_t launch_list(int dim, int real_bytes, const ListBuild& a, hipStream_t s) {
    if (pair_lds_bytes(kWave, a.lanes, a.list_cap) > kPairLdsMax) return hipErrorInvalidValue;
    if (dim == 2 && real_bytes == 4) launch_list_t<2, float>(a, s);
    else if (dim == 2) launch_list_t<2, double>(a, s);
    else if (real_bytes == 4) launch_list_t<3, float>(a, s);
    else launch_list_t<3, double>(a, s);
    return hipGetLastError();
}

template <int DIM, typename real, int KERN, int G, int T, bool ZC, int X = 0>
static void launch_pair_list_x(int mode, const PairLaunch& a, hipStream_t s) {
    const uint32_t tpb = (uint32_t)a.block / G * T;
    const uint32_t nwork = a.ntiles * (kTile / tpb);
    PairLaunch c = a;
    if (nwork < 8) c.persistent = 0;  // a persistent grid needs a workgroup on every XCD
    const uint32_t grid = (c.persistent > 0) ? max(8u, min(nwork, (uint32_t)c.persistent)) : nwork;
    dim3 gr(grid), b(a.block);
    auto kern = (mode == kModeRhs) ? k_pair_list<DIM, real, KERN, kModeRhs + X, G, T, ZC>
                                   : k_pair_list<DIM, real, KERN, kModeStep + X, G, T, ZC>;
    if (c.ev0)
        hipExtLaunchKernelGGL(kern, gr, b, 0u, s, c.ev0, c.ev1, 0u, c, c.plumes, nwork);
    else
        hipLaunchKernelGGL(kern, gr, b, 0, s, c, c.plumes, nwork);
}

template <int DIM, typename real, int KERN, int G, int T, bool ZC>
static void launch_pair_list_s(int mode, const PairLaunch& a, hipStream_t s) {
    if constexpr (T == 2 && DIM == 2 && sizeof(real) == 4) {
        if (a.exact) {
            launch_pair_list_x<DIM, real, KERN, G, T, ZC, kModeExact>(mode, a, s);
            return;
        }
    }
    launch_pair_list_x<DIM, real, KERN, G, T, ZC>(mode, a, s);
}

// one target a group: its list holds no record at r = 0 but the padding (the
// target itself); two targets may find one of theirs coinciding with the other
template <int DIM, typename real, int KERN>
static void launch_pair_list_t(int mode, const PairLaunch& a, hipStream_t s) {
    if (a.targets == 2 && a.lanes == 4) {
        if constexpr (sizeof(real) == 4) {
            if (a.zc) launch_pair_list_s<DIM, real, KERN, 4, 2, true>(mode, a, s);
            else launch_pair_list_s<DIM, real, KERN, 4, 2, false>(mode, a, s);
        }
    } else if (a.targets == 2) {
        if (a.zc) launch_pair_list_s<DIM, real, KERN, 1, 2, true>(mode, a, s);
        else launch_pair_list_s<DIM, real, KERN, 1, 2, false>(mode, a, s);
    } else if (a.lanes == 4) launch_pair_list_s<DIM, real, KERN, 4, 1, false>(mode, a, s);
    else if (a.lanes == 2) launch_pair_list_s<DIM, real, KERN, 2, 1, false>(mode, a, s);
    else launch_pair_list_s<DIM, real, KERN, 1, 1, false>(mode, a, s);
}

hipError_t launch_pair_list(int dim, int real_bytes, int kernel, int mode, const PairLaunch& a, hipStream_t s) {
    if (dim == 2) {
        if (real_bytes == 4) {
            if (kernel == 4) launch_pair_list_t<2, float, 4>(mode, a, s);
            else launch_pair_list_t<2, float, 2>(mode, a, s);
        } else {
            if (kernel == 4) launch_pair_list_t<2, double, 4>(mode, a, s);
            else launch_pair_list_t<2, double, 2>(mode, a, s);
        }
    } else {
        if (real_bytes == 4) {
            if (kernel == 4) launch_pair_list_t<3, float, 4>(mode, a, s);
            else launch_pair_list_t<3, float, 2>(mode, a, s);
        } else {
            if (kernel == 4) launch_pair_list_t<3, double, 4>(mode, a, s);
            else launch_pair_list_t<3, double, 2>(mode, a, s);
        }
    }
    return hipGetLastError();
}

}  // namespace ade
