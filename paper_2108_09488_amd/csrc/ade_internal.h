// ade_internal.h -- device-side tables and kernel launch declarations shared
// by the kernels and the C-ABI host code of the SPH advection-dispersion
// library (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ade {

constexpr int kTile = 256;          // particles per tile (a tile never spans two plumes)
constexpr int kScanPerThread = 16;  // counting-sort scan: elements per thread
constexpr int kScanBlock = 256;
constexpr int kScanChunk = kScanPerThread * kScanBlock;
constexpr int kCellChunk = 1024;    // cell-count scan: 256 threads x 4 counts per workgroup

// cell tables are padded to a whole number of scan chunks (plus the sentinel)
inline uint64_t cell_pad(uint64_t ncell) { return (ncell + 1 + kCellChunk - 1) / kCellChunk * kCellChunk; }

// Per-plume constants.  Positions are uint32 fractions of the box, so all
// lengths below are in grid units (L / 2^32).
struct PlumeDev {
    uint32_t poff, n;       // particles [poff, poff + n) in the concatenated order
    uint32_t cbase, ncell;  // cells [cbase, cbase + ncell) of the global cell table
    uint32_t nfx, nr;       // cells per row along x; rows per side in y (and z)
    int32_t R;              // rows to each side that can hold neighbours
    uint32_t hx;            // half-width of the x search window (>= H_u (1 + 2^-16))
    uint32_t tfirst, tcount;// tiles of this plume
    uint32_t nsub;          // sub-rows per row (cells of a row: nfx x-cells of nsub sub-rows each)
    uint32_t pad1;
    double Hu;              // support radius in grid units
    double H2d;             // Hu^2 (double)
    float H2f;              // Hu^2 rounded to float
    float cellx;            // x cells per grid unit, nfx * 2^-32 (float)
    double invHu;
    float Hc2f;             // square of the search radius Hc = H_u (1 + 2^-16) + 2
    float rowh2f;           // square of the row height in grid units, (2^32 / nr)^2
    float cslack;           // slack of a candidate window in x cells (covers float rounding)
    float pad4;
    double a0, a1;          // Gamma x^T D x / r^2 - tr D = a0 + a1 (e . x / r)^2 (Eq. 3 tensor)
    double ehat[3];         // unit flow direction e (x axis when |v| = 0)
    double pad3;
    // pair-term constants as the pair kernel uses them: Hu^2, 1/Hu, 5/Hu,
    // A0, S, E_x, E_y, E_z with the bracket A = A0 + S (E . x / r)^2,
    // E = sqrt|a1| e, S = sign of a1 (in 2D always +1: a negative a1 is
    // folded into A0 and E normal to the flow)
    double dterm[8];
    float fterm[8];         // the same in FP32
    double trD;             // trace of D
    double vphi;            // V * (kernel derivative prefactor): rhs = vphi * sum
    double dt;
    double ushift[3];       // displacement per step in grid units
    double vel[3];          // flow velocity (physical units)
    double mass;            // particle mass
    double L;
    double aL, aT, Dm;      // alpha_L, alpha_T, D_m (per-particle tensors of a velocity field)
};

struct TileDev {
    uint32_t plume, start, end, pad;
};

// Particle state in structure-of-arrays form.
struct StateArrays {
    uint32_t* pos[3];
    uint4* rec;      // 16-byte candidate records (sorted buffer S only; null if unused)
    void* C;
    uint32_t* id;
    uint32_t* key;   // cell key (hashed buffer U only)
    // velocity field only (null otherwise): per-particle velocity (DIM
    // components) and the reciprocals of the components of the dispersion
    // tensor of Eq. (3) it gives (2D: xx, xy, yy; 3D: xx, xy, xz, yy, yz, zz;
    // 1/0 = inf), in the working precision
    void* vel[3];
    void* rD[6];
    // velocity field with the predictor-corrector: C^n carried through the
    // predictor's build (null otherwise)
    void* Cb;
    // velocity field, sorted buffer S only (null otherwise): the candidate
    // records of the pair sum (GenRec, ade_device.h)
    uint4* grec;
};

// Counting pass of the cell build: the number of particles per cell and
// their ids -- the first kBucket of a cell in its bucket, any further ones in
// an overflow list of (key, id) pairs.
constexpr uint32_t kBucket = 8;
struct CellLists {
    uint32_t* count;      // per cell (cleared by the scan)
    uint32_t* bucket;     // kBucket entries per cell: particle ids
    uint2* ovf;           // overflow pairs (key, id), up to N
    uint32_t* ovf_count;  // [0] pairs added since the last scan, [1] pairs of the current build
};

// kModeStep: the update of C (a uniform flow: C + scale dt rhs; a velocity
// field: also the moves and the next build's counts), kModeRhs: the
// right-hand side; kModeHalf and kModeFull: the predictor and the corrector
// of the velocity-field predictor-corrector step
enum PairMode { kModeStep = 0, kModeHalf = 1, kModeRhs = 2, kModeFull = 3 };
// added to the mode of a two-target kernel over lists in 2D FP32: the second
// target's separations as PairLaunch::exact has them
constexpr int kModeExact = 4;

// A uniform flow moves every particle of a plume by the same displacement
// rint((k+1) u) - rint(k u) (u = PlumeDev::ushift) at step k.  The sorted
// state of such a context therefore keeps the positions of one step, the
// frame's origin k0 (0 after a build), with the order and the cell table
// built from them; the position at step k is the stored one plus frame_shift.
// The context's step counter is the pair (k, k0).  Separations, hence
// neighbour sets and pair sums, are the same in the frame.  A step is then one
// launch with no sort behind it: per step 53.5 -> 27.3 us (512^2 plume, 46
// neighbours), 149 -> 106 us (six-plume sweep), 417 -> 249 us (256-plume
// ensemble), 22 -> 8.4 us (64^2 FP64), against a rebuild in every step.
struct FrameStep {
    int64_t k, k0;
};

// Neighbour lists (kernels_list.hip): where a plume's lists stand for the
// launch shape they were built for.
struct ListPlume {
    uint32_t row0;   // first row (64 words) of the plume's lists
    uint32_t rows;   // rows per wavefront (0: the plume keeps no lists)
};
// What is uniform in a wavefront's lists, in the order of the pair kernel's work
// items: one scalar load leads to everything that the wavefront reads.
struct alignas(32) ListWave {
    static constexpr uint32_t kTwoPasses = 0x80000000u;
    uint32_t i0, end;  // its targets' tile: the first target and past the last (i0 >= end: none)
    uint32_t plume;
    uint32_t row;   // first row of its lists
    uint32_t base;  // 2D: the record that its entries count from
    uint32_t nb;    // batches, and whether a second pass follows (kTwoPasses)
    uint32_t nb2;   // batches of the second pass
    uint32_t full;  // batches in which every lane has entries (16 bits a pass)
};
// entries a lane evaluates per batch, and rows read past a wavefront's last
constexpr int kListBatch = 4;
constexpr uint32_t kListSlack = 4 * kListBatch;

struct PairLaunch {
    const PlumeDev* plumes;
    const TileDev* tiles;
    uint32_t ntiles;
    int block;              // threads per workgroup
    int lanes;              // lanes per target particle (1, 2 or 4)
    int targets;            // target particles per lane: 1, or 2 (one lane, block <= 128)
    int list_cap;           // candidate-list entries per target in LDS (list_cap_for)
    int persistent;         // 0: one workgroup per work item; > 0: that many workgroups loop
    uint32_t xcd_group;     // consecutive work items an XCD takes in turn (>= 1)
    int zc;                 // 1: two distinct particles may share a position, so every
                            // candidate is tested for r > 0; 0: the only candidate at
                            // r = 0 is the target's own record (FP32 C4 kernels skip the test)
    int exact;              // lists in 2D FP32: 1: both targets of a pair form their separations
                            // from integers (kModeExact); 0: the second's from the first's
    const uint4* rec;       // candidate records (position + C of Cpair), or null: SoA reads
    const uint32_t* spos[3];
    const uint32_t* sid;
    const void* Cpair;      // concentrations entering C_a - C_b
    const void* Cbase;      // concentrations updated (update mode)
    const uint32_t* cell_start;
    double scale;           // fraction of the plume's dt: step 1, predictor 0.5 (unused for rhs)
    void* out;              // update: S-order output; rhs: id-order output
    uint4* out_rec;         // update: candidate records with the new C (S order)
    int64_t* step;          // update: the step counter, advanced by this launch (null: left)
    // neighbour lists (list null: walk the row windows)
    const uint32_t* list;
    const ListWave* waves;
    const uint4* list_pos;  // 3D FP64: positions as 16-byte records
    hipEvent_t ev0, ev1;    // if set: events stamped at the kernel's start and end
};

// candidate-list capacity per target for plumes of span = 2R + 1 neighbour
// rows per axis: span + 2 entries per plane of rows (see build_list), plus a
// sentinel and one entry read past it
inline int list_cap_for(int dim, int span) { return (dim == 3 ? span : 1) * (span + 2) + 2; }
// the same for the merged list of a lane's two targets (span + 1 rows per
// plane, span + 1 planes in 3D; n + 2 ranges per plane of n rows)
inline int list_cap_pair_for(int dim, int span) { return (dim == 3 ? span + 1 : 1) * (span + 3) + 2; }
// LDS bytes of the pair kernel's candidate lists for a workgroup
inline size_t pair_lds_bytes(int block, int lanes, int list_cap) {
    return (size_t)(block / lanes) * (size_t)list_cap * 8u;
}
constexpr size_t kPairLdsMax = 65536;

// Build of the neighbour lists of a launch shape.
struct ListBuild {
    const PlumeDev* plumes;
    const TileDev* tiles;
    uint32_t ntiles;
    int lanes, targets;     // the launch shape
    int list_cap;           // candidate-list entries per group in LDS
    const ListPlume* lplumes;
    const uint4* rec;       // candidate records, or null: positions from spos
    const uint32_t* spos[3];
    const uint32_t* cell_start;
    uint32_t* list;
    ListWave* waves;
    uint4* pos;             // 3D FP64: positions as 16-byte records, written with the lists
    uint32_t* over;         // per plume: set when its lists do not fit
};
hipError_t launch_list(int dim, int real_bytes, const ListBuild& a, hipStream_t s);
hipError_t launch_pair_list(int dim, int real_bytes, int kernel, int mode, const PairLaunch& a, hipStream_t s);

// kernel launchers (kernels_*.hip); all return hipError_t of the launch
hipError_t launch_init(int dim, int real_bytes, const PlumeDev* plumes, const TileDev* tiles,
                       uint32_t ntiles, const double* x, const void* C, uint32_t N,
                       StateArrays U, CellLists lists, hipStream_t s);
// nout: entries of cell_start to write, ncell + 1 up to cell_pad(ncell)
hipError_t launch_scan(CellLists lists, uint32_t* cell_start, uint32_t nout, uint32_t* partial, uint32_t ncell,
                       hipStream_t s);
hipError_t launch_place(int dim, int real_bytes, StateArrays U, StateArrays S, CellLists lists,
                        const uint32_t* cell_start, uint32_t N, const int64_t* step, int64_t* step_out,
                        uint32_t* inv, hipStream_t s);
// Velocity field (per-particle velocities, general Eq. 4): the pair sum with
// per-pair harmonic means and the convective term, one lane per target.
struct GenLaunch {
    const PlumeDev* plumes;
    const TileDev* tiles;
    uint32_t ntiles;
    int list_cap;
    int lanes;              // lanes per target particle: 1, 2 or 4 (per two targets: 4)
    int targets;            // targets per group of lanes: 1, or 2 (four lanes, 2D FP32)
    int block;              // threads per workgroup: 64, 128 or 256 (its lists fit in LDS)
    StateArrays S, U;
    const uint32_t* cell_start;
    CellLists lists;
    const int64_t* step;
    void* out;              // rhs mode: id-order output
    hipEvent_t ev0, ev1;    // if set: events stamped at the kernel's start and end
};
hipError_t launch_gen_rec(int dim, int real_bytes, StateArrays S, uint32_t N, hipStream_t s);
hipError_t launch_setvel(int dim, int real_bytes, const PlumeDev* plumes, const TileDev* tiles, uint32_t ntiles,
                         const double* v, uint32_t N, StateArrays U, hipStream_t s);
// Adjoint pass of the velocity-field Euler step over a state snapshot S:
// lam_out (id order) = lambda + dt L^T lambda, gradient partials per
// workgroup added to gpart[3 * workgroup + k].
struct AdjGenLaunch {
    const PlumeDev* plumes;
    const TileDev* tiles;
    uint32_t ntiles;
    int list_cap;
    StateArrays S;
    const uint32_t* cell_start;
    const void* lam_s;  // the vector the pass applies the operator to, in the snapshot's cell order
    const void* lam_id; // corrector pass: lambda^(n+1) in id order
    void* lam_out;      // the pass's output in id order (null: not written)
    void* lam_next;     // its output in the cell order of the next pass's state (null: not written),
    const uint32_t* inv;  // where particle id is in that order
    double* gpart;
};
// passes: Euler (lambda + dt L lambda), and the predictor-corrector's two:
// at the half-step snapshot y = L lambda, at the step's snapshot
// lambda + dt y + dt^2/2 L y
enum AdjGenMode { kAdjGenEuler = 0, kAdjGenHalf = 1, kAdjGenFull = 2 };
hipError_t launch_adjoint_gen(int dim, int real_bytes, int kernel, int mode, const AdjGenLaunch& a,
                              uint32_t block, hipStream_t s);
hipError_t launch_pair_gen(int dim, int real_bytes, int kernel, int mode, const GenLaunch& g, hipStream_t s);
hipError_t launch_pair(int dim, int real_bytes, int kernel, int mode, const PairLaunch& a, hipStream_t s);
// C and candidate records of the sorted state from (C, rec)
hipError_t launch_set_state(int dim, int real_bytes, StateArrays S, const void* C, uint32_t N, hipStream_t s);
hipError_t launch_read_C(int real_bytes, StateArrays S, uint32_t N, void* out, hipStream_t s);
hipError_t launch_coincident(int dim, const PlumeDev* plumes, const TileDev* tiles, uint32_t ntiles,
                             StateArrays S, const uint32_t* cell_start, uint32_t* flag, hipStream_t s);
hipError_t launch_read_x(int dim, const PlumeDev* plumes, const TileDev* tiles, uint32_t ntiles,
                         StateArrays S, const FrameStep* frame, uint32_t N, double* out, hipStream_t s);
hipError_t launch_mass(int real_bytes, const PlumeDev* plumes, int nplumes, const TileDev* tiles,
                       uint32_t ntiles, StateArrays S, double* partial, double* out,
                       hipStream_t s);
hipError_t launch_nbr(int dim, int real_bytes, int fill, const PlumeDev* plumes,
                      const TileDev* tiles, uint32_t ntiles, StateArrays S,
                      const uint32_t* cell_start, int64_t* offsets, int32_t* ids, hipStream_t s);
hipError_t launch_scan64(int64_t* data, uint32_t n, int64_t* partial, hipStream_t s);

}  // namespace ade
