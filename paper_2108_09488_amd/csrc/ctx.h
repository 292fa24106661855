// ctx.h -- host-side context of the C ABI shared by the API translation
// units: the plan of a context (per-plume tables), the context itself and the
// launch sequences every entry point builds on.
#pragma once

#include <hip/hip_runtime.h>

#include <string>
#include <vector>

#include "../../include/adesph.h"
#include "ade_internal.h"

namespace ade {

// records a thread-local error message and returns code
int fail(int code, const char* fmt, ...);

#define HIPCHK(expr)                                                                     \
    do {                                                                                 \
        hipError_t e_ = (expr);                                                          \
        if (e_ != hipSuccess)                                                            \
            return fail(ADE_EHIP, "%s failed: %s", #expr, hipGetErrorString(e_));       \
    } while (0)

struct Plan {
    int dim = 0, real_bytes = 0, kernel = 0, integrator = 0, P = 0;
    int64_t N = 0;
    uint64_t ncell = 0;
    uint32_t ntiles = 0, nscan = 0;
    int list_cap = 0;       // candidate-list entries per target (largest plume)
    int list_cap_pair = 0;  // the same for a lane's merged list of two targets
    double nbar_max = 0.0;  // largest expected neighbours per particle of a plume
    double pairs = 0.0;     // expected neighbours of all particles
    bool general = false;   // velocity field: per-particle velocities (ADE_VELOCITY_FIELD)
    bool check_finite = false;  // ADE_CHECK_FINITE on any plume
    std::vector<PlumeDev> plumes;
    std::vector<double> nbar;   // expected neighbours per particle of each plume
    std::vector<TileDev> tiles;
    std::vector<TileDev> pair_tiles;  // the tiles in the pair kernel's order (costliest plumes first)
};

// 16-byte words of a velocity field's candidate record (GenRec::kQuads)
inline size_t gen_rec_quads(const Plan& pl) {
    return pl.real_bytes == 4 ? (pl.dim == 2 ? 2 : 4) : (pl.dim == 2 ? 4 : 6);
}
// whether saved states and snapshots hold the records; elsewhere they are made
// again from the arrays
inline bool keeps_gen_rec(const Plan& pl) { return pl.general && pl.dim == 2 && pl.real_bytes == 4; }

// The neighbour lists of a plan for a launch shape: each plume's place, and the
// sizes of the arrays they take (bytes 0: no plume keeps any).
struct ListPlan {
    size_t rows = 0, waves = 0, bytes = 0;
    std::vector<ListPlume> place;
};
ListPlan list_plan(const Plan& pl, int lanes, int targets);

// D of Eq. (3) for a uniform flow (row stride 3); returns its trace.
double trace_D(int dim, double aL, double aT, double Dm, const double* v, double D[9]);

}  // namespace ade

struct ade_ctx {
    ade::Plan plan;
    hipStream_t stream = nullptr;
    ade_tuning tuning{256, 2, 0, 0};
    ade_tuning window{256, 2, 0, 0};  // the shape of launches over row windows (tuning, once it is set)
    ade::PlumeDev* plumes = nullptr;
    ade::TileDev* tiles = nullptr;
    ade::TileDev* pair_tiles = nullptr;
    ade::StateArrays S{}, U{};
    ade::CellLists lists{};
    uint32_t* count = nullptr;
    uint32_t* cell_start = nullptr;
    void* scan_partial = nullptr;
    void* aux = nullptr;
    uint4* aux_rec = nullptr;
    double* mass_partial = nullptr;
    double* range_partial = nullptr;  // per tile: min and max of C
    int64_t* step = nullptr;  // the step counter (uniform flow: a FrameStep, k then k0)
    // checks: [0] a non-finite concentration or coincident particles, [1 + plume] its lists do not fit
    uint32_t* flags = nullptr;
    size_t zero_bytes = 0;  // from step on: what a new state starts from zero
    // neighbour lists (uniform flow), in the buffers that only a build uses
    char* list_mem = nullptr;
    size_t list_bytes = 0;  // 0: the context keeps none
    ade::ListPlume* lplumes = nullptr;
    ade::TileDev* win_tiles = nullptr;  // tiles of the plumes without lists, when some plumes have them
    ade::ListPlan lists_of;  // the lists that are there
    int list_shape = 0;      // launch shape (shape_of) they, or their absence, were settled for; 0: not since the build
    int place_shape = 0;     // launch shape lplumes holds the places of (0: none)
    uint32_t win_ntiles = 0;
    bool list_on = false;    // some plume has lists
    bool list_use = false;   // the kernels of the current call read them
    bool list_used = false;  // a call on the particles of the last build read them, or would have
    int list_runs = 0;       // sets of particles before these whose steps did, in a row (at most 2)
    int64_t since = 0;       // steps the host launched since the step of the cells' build
    bool graph_lists = false;  // the captured steps read lists
    bool graph_tiles = false;  // and walk the windows of win_tiles
    uint32_t h_total = 0;  // host copy of N for the cell-start sentinel
    bool initialized = false, built = false;
    // two particles of a plume share a position (the pair kernels then test
    // every candidate for r > 0); true until a cell build has checked
    bool coincident = true;
    bool vel_set = false;  // velocity field: ade_set_velocities called since init
    hipGraph_t graph = nullptr;
    hipGraphExec_t graph_exec = nullptr;
    bool capturing = false;
    // pair-kernel timing
    bool timing = false;
    std::vector<hipEvent_t> events;
    size_t ev_used = 0;
    double timed_ms = 0.0;
    int64_t timed_launches = 0;
};

namespace ade {

// settles whether the kernels of a call of nsteps steps (-1: of another call) read
// neighbour lists, and builds them for the current launch shape if they are not there
int settle_lists(ade_ctx* c, int64_t nsteps = -1);
// enqueue a pair kernel (timed when timing is on)
int run_pair(ade_ctx* c, int mode, const PairLaunch& a);
// launch arguments of a pair kernel over the sorted particles of c: rec the
// candidate records carrying Cpair
PairLaunch pair_args(ade_ctx* c, const void* Cpair, const uint4* rec, const void* Cbase, double scale, void* out,
                     uint4* out_rec);
// one step of a uniform flow from the concentrations (C, rec) to (Cn, recn),
// which differ from them; advances the step counter if asked
int enqueue_uniform(ade_ctx* c, const void* C, const uint4* rec, void* Cn, uint4* recn, bool count);
// the frame of a uniform flow (null for a velocity field)
inline const FrameStep* frame_of(const ade_ctx* c) {
    return c->plan.general ? nullptr : reinterpret_cast<const FrameStep*>(c->step);
}
// counting sort of the hashed U buffer into S and the cell-start table
int enqueue_build(ade_ctx* c, int inc_step);
// A velocity field's sorted state: the context's own, or one kept by the adjoint.
struct GenState {
    StateArrays S;
    uint32_t* cell_start;
    uint32_t ncs;   // entries of cell_start
    int64_t* step;  // its step counter
    uint32_t* inv;  // where particle id is in its order (null: not kept)
};
GenState gen_live(const ade_ctx* c);
// the counting sort into `to`; its step counter becomes *step + 1 (step null: left)
int enqueue_build_into(ade_ctx* c, const GenState& to, const int64_t* step);
// n explicit steps (velocity field: pair sum, update and rebuild each)
int enqueue_steps(ade_ctx* c, int64_t n);
// launch arguments of the velocity-field pair kernel over the sorted state of c
GenLaunch gen_args(ade_ctx* c, void* out);
// enqueue the velocity-field pair kernel (timed when timing is on)
int run_gen(ade_ctx* c, int mode, void* out, const GenState& at);

}  // namespace ade
