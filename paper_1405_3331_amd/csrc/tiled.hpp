// tiled.hpp -- temporally blocked, LDS-tiled step kernel: interface used by the host side.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cuesim.h"
#include "internal.hpp"

namespace cuesim {

constexpr int kDefaultBlockSteps = 8;   // of a batch that no planned shape fits

// How a workgroup steps a tile (kernels_tiled.hip).
enum TileShape { kPair, kTwoPair, kTwo, kWide };

// Tile geometry chosen once per simulation.
struct TiledPlan {
    int dim = 2;
    int block_steps = 1;     // B: steps advanced per launch (1 = tiling unavailable)
    int halo = 0;            // H: cells loaded around each tile core
    int core_x = 0, core_y = 0;
    int tiles_x = 0, tiles_y = 0;
    int n_tiles = 0;
    int height = 0;          // loaded tile height (rows), core_y + 2 * halo
    int move = 0;            // cells a tip can travel in one launch, ceil(B * s / dx)
    int cpl = 2;             // columns per lane: loaded tile width is 64 * cpl
    TileShape shape = kPair;
    int cone_rows = 15;      // strip rows traded per occupied cone slot (load balance)
    int n_species = 1;
    int nx = 0, ny = 0, nz = 1;
    float inv_dx = 1.0f;
    StencilCoef coef[SIM_MAX_SPECIES] = {};
    size_t lds_bytes = 0;
};

// Candidate part sizes of a crowded tile (kernels_tiled.hip).
constexpr int kPartSizes = 5;

// Launch-to-launch state of the tiled kernel, in device memory: completed steps, which half
// of every ping-pong pair is the input (parity) and which third of the cone counts (phase),
// the counters a launch resets by itself, and the crowded tiles' further parts, counted per
// candidate size while the cones were put into their buckets ([phase], listed in
// TiledState::extra).  The first group is read by every workgroup and so kept off the lines
// that the atomics change.
struct alignas(128) LaunchState {
    uint32_t step;
    int32_t parity, phase, unused;
    alignas(128) int32_t next;   // the persistent queue
    int32_t arrived;             // workgroups that have read the group above
    alignas(128) int32_t extra_n[3][8];
};

struct TiledArgs2D;

// Device buffers owned by the tiled path.
struct TiledState {
    float4* bucket[2] = {nullptr, nullptr};    // per tile: cone slots (x, y, theta, id)
    char* memory = nullptr;                    // launch state, counts, lists and per-tile tables
    int32_t* count[3] = {nullptr, nullptr, nullptr};   // cones per tile
    int cur = 0;                               // bucket buffer holding the live cones
    int phase = 0;                             // and their counts (the device state's copies)
    int capacity = 0;                          // slots per tile
    TiledArgs2D* args = nullptr;               // this simulation's arguments (host memory)
    LaunchState* launch = nullptr;             // device launch state
    int4* extra = nullptr;                     // further parts of crowded tiles, (simulation,
                                               // tile, part, 0): [parity][size][extra_cap]
    int extra_cap = 0;
    int room = 0;                              // workgroups resident beside one per tile
};

// Choose B (up to block_steps; 0: the planner's choice) and the tile shape; block_steps = 1 in the
// result means no tiling fits.
// force_cpl != 0 restricts the row width to 64 * force_cpl columns, force_height != 0 the
// loaded tile height; a forced shape that does not fit falls back to the planner's choice.
// alone: the simulation has launches of its own; a batch's members do not, and the launch that
// they share has one row width, so that only the height falls back.
TiledPlan tiled_plan(int dim, int nx, int ny, int nz, int n_species, double step_cells,
                     int block_steps, int n_cones, int force_cpl = 0, int force_height = 0,
                     bool alone = true);
// Depth and tile heights for a batch of simulations with row width 64 * cpl: the depth (theirs
// where they ask for one; 0 if no shape fits them all) and each simulation's loaded height (its
// tile_height where it gives one that fits at any depth).
int tiled_batch_shape(const sim_params* const* params, int n, int cpl, std::vector<int>& height);
// The row width and depth with which every member of a batch can be planned, and their plans.
// Returns -1, or a member that no common shape fits.
struct BatchPlan {
    int cpl = 2, block_steps = 0;
    std::vector<TiledPlan> members;
};
int tiled_batch_plan(const sim_params* const* params, int n, BatchPlan& plan);
// Allocate buckets and per-tile tables and upload the argument table; fields[s][b] are the
// simulation's ping-pong field buffers, cones its caller-order arrays.
hipError_t tiled_allocate(const TiledPlan& plan, TiledState& st, int n_cones,
                          const ConeRules& rules, const sim_params* p, float* const fields[][2],
                          ConeArrays cones, hipStream_t stream);
// Set the device launch state (step counter; parity = input half of the ping-pong pairs).
hipError_t tiled_set_launch_state(TiledState& st, uint32_t step, int parity, hipStream_t stream);
// The host's copies (st.cur, st.phase) from the device launch state.
hipError_t tiled_get_launch_state(TiledState& st);
// Record mode: while tape is non-null every launch also writes the state after each of its
// sub-steps to tape + ((step - n0) * n_species + s) * cells and every cone step's record to
// `cones` (step - n0) (null: off).
void tiled_set_record(TiledState& st, float* tape, const ConeTape& cones, uint32_t n0);
void tiled_release(TiledState& st);
// Move active cones from the caller-order arrays into the tile buckets (which hold none:
// new, or dropped).  In a batch `launch` and `extra` are the batch's and sim its index.
hipError_t tiled_bucket(const TiledPlan& plan, TiledState& st, ConeArrays cones,
                        hipStream_t stream);
hipError_t tiled_bucket_batch(const TiledPlan& plan, TiledState& st, ConeArrays cones,
                              int sim, LaunchState* launch, int4* extra, int extra_cap,
                              hipStream_t stream);
// Copy the active cones from the tile buckets into the caller-order arrays; the buckets stay
// valid, so stepping goes on without bucketing again, unless `drop` empties them.
hipError_t tiled_sync_cones(const TiledPlan& plan, TiledState& st, ConeArrays cones,
                            hipStream_t stream, bool drop);
// Advance `steps` (<= plan.block_steps) steps in one launch; flips st.cur like the device
// parity.
// start/stop (may be null): events the launch records around the kernel (timing).
hipError_t tiled_launch(const TiledPlan& plan, TiledState& st, int steps, hipStream_t stream,
                        hipEvent_t start = nullptr, hipEvent_t stop = nullptr);

// Mirror launches that ran without tiled_launch (a batch's) in the host-side state.
void tiled_advanced(TiledState& st, int launches);

// Size in bytes of one argument-table entry (for batching several simulations).
size_t tiled_table_entry_bytes();
// One persistent launch over the work items of a batch whose argument tables are
// concatenated in `table`; all simulations share n_species, cpl and `launch`.  base lists
// every (simulation, tile); extra the further parts of crowded tiles.
hipError_t tiled_launch_batch(const TiledArgs2D* table, int4* extra, const int2* base,
                              int n_base, int extra_cap, int n_species, int cpl,
                              size_t lds_bytes, int steps, LaunchState* launch,
                              hipStream_t stream);
// Bound on the further parts of tiles holding n_cones cones in total, in full parts.
int tiled_extra_capacity(int64_t n_cones);
constexpr int kBatchPartLists = 1;   // a batch lists full parts only: extra is
                                     // [parity][extra_cap]
// Number of workgroups of the persistent batch launch for a given dynamic LDS size.
int tiled_persistent_grid(size_t lds_bytes);
// Allow the batch kernel variant lds_bytes of dynamic LDS (call before launching or
// capturing it).
hipError_t tiled_prepare_batch(int n_species, int cpl, size_t lds_bytes);

}  // namespace cuesim
