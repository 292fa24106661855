// ade_device.h -- device helpers shared by the kernels (gfx950, wave64).
#pragma once

#include "ade_internal.h"

namespace ade {

constexpr int kWave = 64;

// Workgroups of one launch are dispatched round-robin over the 8 XCDs of the
// chip (workgroup b runs on XCD b % 8).  Items are dealt to the XCDs in turns
// of `group` consecutive items, so that neighbouring items (which share
// candidate cells) share an L2 while every XCD still gets an even share of
// every part of the item list (plumes of an ensemble differ in cost per item).
// A bijection of [0, n): the last incomplete round keeps the identity.
__device__ __forceinline__ uint32_t xcd_remap(uint32_t b, uint32_t n, uint32_t group) {
    const uint32_t nx = 8, round = nx * group;
    const uint32_t full = n / round * round;
    if (b >= full) return b;
    const uint32_t g = b / round, r = b % round;
    return g * round + (r % nx) * group + r / nx;
}

// The m-th item (m = 0, 1, ...) that xcd_remap deals to XCD x, or n when
// XCD x has fewer than m + 1 items (the persistent grid walks this list).
__device__ __forceinline__ uint32_t xcd_item(uint32_t x, uint32_t m, uint32_t n, uint32_t group) {
    const uint32_t nx = 8, round = nx * group;
    const uint32_t full = n / round * round;
    const uint32_t per = full / nx;  // items of XCD x in complete rounds
    if (m < per) return (m / group) * round + x * group + m % group;
    const uint32_t t = full + x + (m - per) * nx;  // the identity tail, round-robin
    return t < n ? t : n;
}

// Cell of a fixed-point position: rows of the (y[, z]) grid, x cells inside a
// row, sub-rows (in y) inside an x cell; the position inside the row is the
// low word of uy * nr.
template <int DIM>
__device__ __forceinline__ uint32_t cell_key(const PlumeDev& P, uint32_t ux, uint32_t uy,
                                             uint32_t uz) {
    const uint32_t fx = __umulhi(ux, P.nfx);
    const uint32_t ry = __umulhi(uy, P.nr);
    const uint32_t rz = (DIM == 3) ? __umulhi(uz, P.nr) : 0u;
    const uint32_t sy = __umulhi(uy * P.nr, P.nsub);
    return P.cbase + ((rz * P.nr + ry) * P.nfx + fx) * P.nsub + sy;
}

// Counting pass: count the particle with this id in its cell and record the
// id in the cell's bucket, or past kBucket in the overflow list.
__device__ __forceinline__ void enlist(const CellLists& L, uint32_t key, uint32_t id) {
    const uint32_t t = atomicAdd(&L.count[key], 1u);
    if (t < kBucket) {
        L.bucket[(size_t)key * kBucket + t] = id;
    } else {
        const uint32_t p = atomicAdd(&L.ovf_count[0], 1u);
        L.ovf[p] = make_uint2(key, id);
    }
}

template <typename T>
__device__ __forceinline__ T wave_inclusive_scan(T x) {
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        T y = __shfl_up(x, o, kWave);
        if (lane >= o) x += y;
    }
    return x;
}

template <typename T>
__device__ __forceinline__ T wave_sum(T x) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) x += __shfl_xor(x, o, kWave);
    return x;
}

// Exclusive scan over the block (blockDim.x a multiple of 64, at most 1024).
// lds must hold blockDim.x / 64 elements; returns the block total in total.
template <typename T>
__device__ __forceinline__ T block_exclusive_scan(T v, T* lds, T& total) {
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const int nw = blockDim.x / kWave;
    T x = wave_inclusive_scan(v);
    if (lane == kWave - 1) lds[w] = x;
    __syncthreads();
    T pre = 0, tot = 0;
    for (int i = 0; i < nw; ++i) {
        T s = lds[i];
        pre += (i < w) ? s : T(0);
        tot += s;
    }
    __syncthreads();
    total = tot;
    return pre + x - v;
}

// Sum over the block in a fixed order (deterministic); result valid in all threads.
template <typename T>
__device__ __forceinline__ T block_sum(T v, T* lds) {
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const int nw = blockDim.x / kWave;
    T x = wave_sum(v);
    if (lane == 0) lds[w] = x;
    __syncthreads();
    T tot = 0;
    for (int i = 0; i < nw; ++i) tot += lds[i];
    __syncthreads();
    return tot;
}

// 16-byte record of a particle for the candidate loops: fixed-point position
// and concentration (2D: x, y, C[, C high word]; 3D FP32: x, y, z, C).  3D FP64
// does not fit and uses the structure-of-arrays state instead.
template <int DIM, typename real>
struct Rec {
    static constexpr bool kStageable = !(DIM == 3 && sizeof(real) == 8);
    static __device__ __forceinline__ uint4 pack(uint32_t x, uint32_t y, uint32_t z, real c) {
        uint4 r;
        r.x = x;
        r.y = y;
        if (sizeof(real) == 4) {
            const uint32_t cb = __float_as_uint((float)c);
            r.z = (DIM == 3) ? z : cb;
            r.w = (DIM == 3) ? cb : 0u;
        } else {
            const unsigned long long cb = (unsigned long long)__double_as_longlong((double)c);
            r.z = (uint32_t)cb;
            r.w = (uint32_t)(cb >> 32);
        }
        return r;
    }
    static __device__ __forceinline__ real conc(const uint4& r) {
        if (sizeof(real) == 4) return (real)__uint_as_float(DIM == 3 ? r.w : r.z);
        return (real)__longlong_as_double((long long)(((unsigned long long)r.w << 32) | r.z));
    }
};

// Candidate record of a velocity-field particle: its position words, then C, the
// velocity and the reciprocals of the tensor components in the working precision,
// padded to a multiple of 32 bytes (2D FP32: {x, y, C, v_x} {v_y, 1/D_xx, 1/D_xy,
// 1/D_yy}, 32 bytes; 3D FP32 and 2D FP64 64; 3D FP64 96, its position in four words).
template <int DIM, typename real>
struct GenRec {
    static constexpr int kVals = 1 + DIM + (DIM == 2 ? 3 : 6);
    static constexpr int kPer = sizeof(real) / 4;
    static constexpr int kPos = (kPer == 2 && DIM == 3) ? 4 : DIM;  // doubles on even words
    static constexpr int kWords = kPos + kVals * kPer;
    static constexpr int kQuads = (kWords + 7) / 8 * 2;
    static __device__ __forceinline__ real value(const uint32_t* w, int j) {
        if constexpr (sizeof(real) == 4) return __uint_as_float(w[kPos + j]);
        else return __hiloint2double((int)w[kPos + 2 * j + 1], (int)w[kPos + 2 * j]);
    }
    // the words of record k: 16-byte loads and one for the rest
    static __device__ __forceinline__ void load(const uint4* __restrict__ rec, uint32_t k, uint32_t (&w)[kWords]) {
        // 2D FP32: a 32-bit byte offset from a uniform base (such a context
        // holds fewer than 2^27 particles)
        const char* base = reinterpret_cast<const char*>(rec) +
                           (kQuads == 2 ? (size_t)(k << 5) : (size_t)k * (kQuads * 16));
#pragma unroll
        for (int q = 0; q < kWords / 4; ++q) {
            const uint4 v = *reinterpret_cast<const uint4*>(base + 16 * q);
            w[4 * q] = v.x;
            w[4 * q + 1] = v.y;
            w[4 * q + 2] = v.z;
            w[4 * q + 3] = v.w;
        }
        constexpr int kRest = kWords / 4 * 4;
        if constexpr (kWords % 4 == 2) {
            const uint2 v = *reinterpret_cast<const uint2*>(base + 4 * kRest);
            w[kRest] = v.x;
            w[kRest + 1] = v.y;
        } else if constexpr (kWords % 4 == 1) {
            w[kRest] = *reinterpret_cast<const uint32_t*>(base + 4 * kRest);
        }
    }
    // vals: velocity and reciprocals
    static __device__ __forceinline__ void store(uint4* __restrict__ rec, uint32_t k, const uint32_t* u, real C,
                                                 const real* vals) {
        uint32_t w[kQuads * 4] = {};
#pragma unroll
        for (int c = 0; c < DIM; ++c) w[c] = u[c];
#pragma unroll
        for (int j = 0; j < kVals; ++j) {
            const real v = j == 0 ? C : vals[j > 0 ? j - 1 : 0];
            if constexpr (sizeof(real) == 4) {
                w[kPos + j] = __float_as_uint((float)v);
            } else {
                w[kPos + 2 * j] = (uint32_t)__double2loint((double)v);
                w[kPos + 2 * j + 1] = (uint32_t)__double2hiint((double)v);
            }
        }
#pragma unroll
        for (int q = 0; q < kQuads; ++q)
            rec[(size_t)k * kQuads + q] = make_uint4(w[4 * q], w[4 * q + 1], w[4 * q + 2], w[4 * q + 3]);
    }
};

}  // namespace ade
