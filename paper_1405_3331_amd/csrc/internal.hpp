// internal.hpp -- launchers shared between the host side of the library and the kernel
// translation units.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "cuesim.h"
#include "device.hpp"

namespace cuesim {

// Stencil coefficients of one species: c' = (c - kdt*c) + r*(sum(neighbours) - 2 dim c).
// Keeping decay and diffusion as separate terms (rather than folding them into one centre
// weight 1 - 2 dim r - k dt, whose FP32 rounding shifts the effective decay rate and is
// amplified ~1/(k dt) in the steady state) leaves only unbiased rounding.
struct StencilCoef {
    float r, kdt;
};

// Cone state in the caller's order (structure of arrays).
struct ConeArrays {
    float* pos;          // [M][dim]
    float* dir;          // 2D [M]; 3D [M][3]
    int32_t* status;
    int32_t* target;
    int32_t* event_step;
    int n;
};

// Fill the near map of a target grid (its dimensions and targets set) of `words` words.
hipError_t launch_near_map(int dim, const TargetGrid& tg, uint32_t* near, size_t words,
                           int n_targets, hipStream_t stream);

// 2D field step of every species in one launch, sources included (kernels_field2d.hip).
// Field2DStep holds the per-box source lists (row, column in the box, amount) built once by
// field2d_prepare from the merged, pre-scaled sources of each species.
struct Field2DStep {
    int nx = 0, ny = 0, n_species = 0, n_boxes = 0;
    char* memory = nullptr;         // every list below
    int32_t* src_start = nullptr;   // [n_boxes + 1]
    int32_t* src_row = nullptr;     // per entry: row j
    int32_t* src_col = nullptr;     // per entry: thread of the box owning the cell
    float* src_q = nullptr;         // per entry: amount / dx^2
    // two steps per launch (launch_field2d_pair): per box of 256 x 4 cells, the sources on
    // the box and its one-cell ring, as (tile position, amount / dx^2)
    int n_pair_boxes = 0;
    int32_t* pair_start = nullptr;  // [n_pair_boxes + 1]
    int32_t* pair_pos = nullptr;    // per entry: row * 258 + column within the ringed box
    float* pair_q = nullptr;
};
struct Field2DStepArgs {
    const float* in[2];
    float* out[2];
    StencilCoef coef[2];
    int nx, ny, n_species;
    int tx, ty, per_xcd;
    const int32_t* src_start;
    const int32_t* src_row;
    const int32_t* src_col;
    const float* src_q;
};
Field2DStepArgs field2d_args(const Field2DStep& f, const float* const* in, float* const* out,
                             const StencilCoef* coef);
hipError_t field2d_prepare(Field2DStep& f, int nx, int ny, int n_species,
                           const std::vector<int32_t>* cells, const std::vector<float>* q);
void field2d_release(Field2DStep& f);
// Two steps: out1 = the state after one step, out2 after two (every species).
hipError_t launch_field2d_pair(const Field2DStep& f, const float* const* in, float* const* out1,
                               float* const* out2, const StencilCoef* coef, hipStream_t stream);
// start/stop (may be null): events the launch itself records.
hipError_t launch_field2d_rows(const Field2DStep& f, const float* const* in, float* const* out,
                               const StencilCoef* coef, hipStream_t stream,
                               hipEvent_t start = nullptr, hipEvent_t stop = nullptr);

// One 2D step's cones in the caller's order (kernels_plain.hip); with `tape` they are recorded
// as its step t.
hipError_t launch_cones2d(const ConeRules& rules, const float* f0, const float* f1,
                          ConeArrays cones, uint32_t step, hipStream_t stream,
                          const ConeTape* tape = nullptr, size_t t = 0);
// The same (unrecorded), and in the same launch the next field step, from the fields that the
// cones read.
hipError_t launch_step2d(const ConeRules& rules, ConeArrays cones, uint32_t step,
                         const Field2DStepArgs& next, hipStream_t stream);

// 3D field step of every species in one launch, sources included (kernels_field3d.hip).
// Field3D holds the per-box source lists (plane, thread, amount) built once by
// field3d_prepare from the merged, pre-scaled sources of each species.
struct Field3D {
    int nx = 0, ny = 0, nz = 0, n_species = 0, n_boxes = 0;
    char* memory = nullptr;          // every list below
    int32_t* src_start = nullptr;    // [n_boxes + 1]
    int32_t* src_plane = nullptr;    // per entry: plane index l
    int32_t* src_thread = nullptr;   // per entry: thread of the box owning the cell
    float* src_q = nullptr;          // per entry: amount / dx^3
};
struct Field3DArgs {
    const float* in[2];
    float* out[2];
    StencilCoef coef[2];
    int nx, ny, nz, n_species;
    int tx, ty, tz, planes, per_xcd;
    const int32_t* src_start;
    const int32_t* src_plane;
    const int32_t* src_thread;
    const float* src_q;
};
Field3DArgs field3d_args(const Field3D& f, const float* const* in, float* const* out,
                         const StencilCoef* coef);
hipError_t field3d_prepare(Field3D& f, int nx, int ny, int nz, int n_species,
                           const std::vector<int32_t>* cells, const std::vector<float>* q);
void field3d_release(Field3D& f);
// start/stop (may be null): events the launch itself records.
hipError_t launch_field3d(const Field3D& f, const float* const* in, float* const* out,
                          const StencilCoef* coef, hipStream_t stream,
                          hipEvent_t start = nullptr, hipEvent_t stop = nullptr);

// Active 3D cones in spatial order (kernels_cones3d.hip): per cone the tip (x, y, z, id)
// and heading (hx, hy, hz, 0), ping-pong halves, with the radix-sort keys, slots and scratch.
// Stopped cones carry id -1 and the key `inactive`, past every active one.
struct ConeOrder3D {
    char* memory = nullptr;   // every array below
    float4* tip[2] = {};
    float4* dir[2] = {};
    uint32_t* key[2] = {};
    int32_t* slot[2] = {};
    int32_t* scratch = nullptr;   // counting-sort histograms (sort_pairs)
    int cur = 0;
    int n = 0;
    int x_bits = 0;   // of the key
    uint32_t inactive = 0;
    int end_bit = 1;
};
hipError_t order3d_allocate(ConeOrder3D& o, int n, int nx, int ny, int nz);
void order3d_release(ConeOrder3D& o);
// Caller-order arrays -> ordered state (pack, sort, gather).
hipError_t order3d_begin(ConeOrder3D& o, const ConeRules& r, ConeArrays cones,
                         hipStream_t stream);
// Re-sort the ordered state by the current tips.
hipError_t order3d_refresh(ConeOrder3D& o, const ConeRules& r, hipStream_t stream);
// One step of the ordered cones; stopping cones are written to `cones` at once.
hipError_t launch_cones3d_ordered(const ConeRules& r, const float* f0, const float* f1,
                                  ConeOrder3D& o, ConeArrays cones, uint32_t step,
                                  hipStream_t stream);
// The same, and in the same launch the next field step, from the fields that the cones read.
hipError_t launch_step3d(const ConeRules& r, ConeOrder3D& o, ConeArrays cones, uint32_t step,
                         const Field3DArgs& next, hipStream_t stream);
// Tips and headings of the still-active ordered cones back into the caller-order arrays.
hipError_t order3d_end(const ConeOrder3D& o, ConeArrays cones, hipStream_t stream);

// Sample adjoints of one reverse step held as 64-bit fixed-point sums, so that the sum in a
// cell does not depend on the order in which the cones' contributions arrive (integer
// addition is associative): value = q * 2^(e - kFixedBits), where 2^e bounds the step's
// largest |contribution| (step_max[t] holds its FP32 bits, 0 for a step without any).
// Every contribution is at most 2^kFixedBits in magnitude after scaling, so up to
// 2^(62 - kFixedBits) of them can meet in one cell without overflow.
constexpr int kFixedBits = 40;

__device__ __forceinline__ int fixed_exponent(uint32_t max_bits) {
    if (max_bits == 0u) return 0;
    int e;
    (void)frexpf(__uint_as_float(max_bits), &e);   // max = f 2^e, 0.5 <= f < 1
    return e;
}

// Reverse pass of the 2D step, segment by segment (kernels_adjoint.hip for the cones,
// kernels_reverse2d.hip for the fields).
constexpr int kRevSteps = 8;   // reverse field steps per launch

// One checkpoint segment of `len` steps from step seg0 and what its reverse works on.  Field
// state c^t of species s (after t steps of the segment, t = 0 .. len) is
// fields + (t * n_species + s) * cells.
struct ReverseSegment {
    ConeRules rules;
    StencilCoef coef[2];
    int nx, ny, n_species, M, len;
    uint32_t seg0;
    const float* fields;
    ConeTape tape;         // the segment's cone steps
    float2* ag;            // [len][M]: adjoint of the cone's sampled gradient, before the
                           // species' signs
    float4* boxes;         // [launch][M]: box of the tips (x from, x to, y from, y to) whose
                           // samples have an adjoint in the launch's steps
    uint32_t* step_max;    // [len], zero before the segment's launches
    int32_t* list_end;     // [launch][tile]: where the tile's cones end in the launch's list
    int32_t* list;         // [launch][list_cap]
    size_t list_cap;
    // accumulators over the whole sweep: [species][tile], and one per source
    double* acc_D;
    double* acc_k;
    double* acc_q;
    const int32_t* q_start;   // [species][tile + 1] into q_entry (reverse_sources)
    const int2* q_entry;
};
// The reverse of a segment's cone steps from step t_from of its len (t_from = len - 1 - a multiple
// of kRevSteps) on, for every cone of `tape` (the segment's steps): sample adjoints and boxes as
// in ReverseSegment, the cones' own adjoints in acone.  start_status: the cones' status at the
// segment's first step, seg0; status and event_step: the handle's, run_status and run_event: at the
// run's end (the tape holds no steps past a cone's stop, whatever was written since).
struct ConeChain {
    ConeTape tape;
    uint32_t seg0;
    int len, t_from;
    float2* ag;
    float4* boxes;
    const int32_t* start_status;
    const int32_t* status;
    const int32_t* event_step;
    const int32_t* run_status;
    const int32_t* run_event;
    float* acone;   // [M][3]
};
// Column and row of a tile, tiles_x to a row.  A division, once per workgroup: the high word of
// tile * ceil(2^32 / tiles_x) is one too large from tile * (ceil(2^32 / tiles_x) * tiles_x - 2^32)
// = 2^32 on, which grids a few hundred thousand columns wide reach.
__host__ __device__ __forceinline__ int2 tile_place(int tile, int tiles_x) {
    const int row = tile / tiles_x;
    return make_int2(tile - row * tiles_x, row);
}
// A launch over n_tiles tiles: per_slice workgroups (a multiple of the dies, which take contiguous
// stretches) for each of `slices` slices of the grid's z axis, so that no axis has more than 2^32
// threads (a row of cells 2^30 wide has 9.6 million tiles of 512 threads).
struct ReverseGrid {
    int slices, per_slice;
    // tile of workgroup x of slice z (none from n_tiles on)
    __host__ __device__ __forceinline__ int tile(int x, int z) const {
        return z * per_slice + (x % 8) * (per_slice / 8) + x / 8;
    }
};
ReverseGrid reverse_grid(int n_tiles);
int reverse_tiles(int nx, int ny);
int reverse_launches(int len);
// Entries that the list of one launch can need: M cones moving at most step_cells per step.
size_t reverse_list_capacity(int nx, int ny, int M, double step_cells);
// Append one species' sources, numbered from `first`, listed by the tile of their cell.
void reverse_sources(int nx, int ny, const std::vector<int32_t>& cells, int first,
                     std::vector<int32_t>& start, std::vector<int2>& entry);
// The cones that can touch each tile, for every launch of the segment (after the cones'
// reverse).
hipError_t launch_reverse_lists(const ReverseSegment& g, double step_cells, hipStream_t stream);
// Launch `launch` of reverse_launches(len): the field adjoint of every species from a_in to
// a_out, kRevSteps steps back (fewer in the last launch); with `chain`, beside it kRevSteps steps
// of that chain.
hipError_t launch_field_reverse2d(const ReverseSegment& g, int launch, const float* const* a_in,
                                  float* const* a_out, const ConeChain* chain,
                                  hipStream_t stream);
int adjoint_cone_blocks(int n);
// Forward re-run of segments seg_first .. seg_first + n_seg - 1 of a run checkpointed every
// `every` of its n_steps steps from step n0; run step t's fields are at
// fields + ((t - t_base) * n_species + s) * cells and its cone steps are recorded as step
// t - t_base of `tape`.
hipError_t launch_cones_segments2d(const ConeRules& rules, const float* fields, size_t cells,
                                   int n_species, int t_base, int seg_first, int n_seg,
                                   int every, int n_steps, uint32_t n0, const float* ckpt_pos,
                                   const float* ckpt_dir, const int32_t* ckpt_int, int M,
                                   const ConeTape& tape, hipStream_t stream);
// The rest of a segment's chain, down to its first step, in a launch of its own.
hipError_t launch_cone_chain2d(const ConeRules& rules, const ConeChain& c, hipStream_t stream);
// Every step's largest contribution to a cell (step_max), once the segment's chain is done.
hipError_t launch_sample_max2d(const ReverseSegment& g, hipStream_t stream);
// Loss partials and the seed of the cones' adjoints; with stop (2 n words) the cones' status and
// event step go there.
hipError_t launch_adjoint_seed2d(const ConeArrays& cones, const float* tip_target,
                                 const float* weight, float* acone, double* partial,
                                 int32_t* stop, hipStream_t stream);

// Adjacency list of the connections and its breadth-first levels (kernels_graph.hip).
struct GraphBuffers {
    int32_t* owner = nullptr;          // [M] neuron owning each cone
    int32_t* target_owner = nullptr;   // [T] neuron owning each target
    int32_t* key = nullptr;            // [M] sort keys / values and their sorted copies
    int32_t* cone = nullptr;
    int32_t* key_sorted = nullptr;
    int32_t* cone_sorted = nullptr;
    int32_t* degree = nullptr;         // [N]
    int32_t* row_start = nullptr;      // [N + 1]  (V_a)
    int32_t* edges = nullptr;          // [M]      (E_a; the first row_start[N] are used)
    int32_t* level = nullptr;          // [N]
    int32_t* grew = nullptr;           // [1]
    int32_t* scratch = nullptr;        // counting-sort histograms (sort_pairs)
    int n_neurons = 0;
    int n_edges = 0;                   // of the adjacency list last read back
};
hipError_t launch_adjacency(const GraphBuffers& g, const int32_t* status, const int32_t* target,
                            int n_cones, int n_neurons, hipStream_t stream);

// Host side of the connectivity build (sim.hip), shared by the entry points that build it:
// the argument checks, and the build itself into caller-provided device buffers g (owners
// uploaded, adjacency built on the handle's stream, copied into the caller's arrays).
sim_status connectivity_validate(sim_handle* h, int32_t n_neurons, const int32_t* cone_owner,
                                 const int32_t* target_owner, const int32_t* row_start,
                                 const int32_t* edges, int64_t edge_capacity,
                                 const int64_t* n_edges);
sim_status connectivity_build(sim_handle* h, GraphBuffers& g, const int32_t* cone_owner,
                              const int32_t* target_owner, int32_t* row_start, int32_t* edges,
                              int64_t edge_capacity, int64_t* n_edges);
sim_status handle_fail(sim_handle* h, sim_status st, const char* msg);
int handle_cones(const sim_handle* h);
int handle_targets(const sim_handle* h);
int handle_device(const sim_handle* h);   // the device the handle was created on
// The neuron that owns each edge of the list (the sorted keys).
const int32_t* adjacency_from(const GraphBuffers& g);
// Levels of every vertex in one launch, for graphs that bfs_in_one_launch admits.
bool bfs_in_one_launch(int n, int64_t n_edges);
hipError_t launch_bfs(const GraphBuffers& g, int n_edges, int root, hipStream_t stream);
hipError_t launch_bfs_init(int32_t* level, int n, int root, hipStream_t stream);
hipError_t launch_bfs_level(const int32_t* row_start, const int32_t* edges, int n, int depth,
                            int32_t* level, int32_t* grew, hipStream_t stream);

// Stable sort of n (key, value) pairs by the low key_bits bits of the keys (every key must
// be below 2^key_bits) with the project's counting passes (kernels_sort.hip).  keys/vals
// hold the input; keys_alt/vals_alt (same sizes) are the other half of each pass's
// ping-pong; *in_alt tells which pair holds the result.  scratch holds
// sort_pairs_scratch_bytes(n) bytes.
size_t sort_pairs_scratch_bytes(int n);
bool sort_in_alt(int key_bits);   // whether such a sort ends in the alternate arrays
hipError_t sort_pairs(uint32_t* keys, int32_t* vals, uint32_t* keys_alt, int32_t* vals_alt,
                      int n, int key_bits, int32_t* scratch, hipStream_t stream, bool* in_alt);

// Up to kMaxSpans device-to-device copies of whole 4-byte words in one launch: span k copies
// word_end[k] - word_end[k - 1] words from src[k] to dst[k] (word_end is cumulative).
constexpr int kMaxSpans = 8;
struct CopySpans {
    const void* src[kMaxSpans];
    void* dst[kMaxSpans];
    size_t word_end[kMaxSpans];
    int n;
};
hipError_t launch_copy_spans(const CopySpans& c, hipStream_t stream);

// Sum of a field in FP64 (deterministic two-pass reduction) into *out (device); when
// nonfinite is given, a non-finite sum sets *nonfinite = 1 (device).
hipError_t launch_mass(const float* field, int64_t n, double* partial, int n_partial,
                       double* out, hipStream_t stream, int32_t* nonfinite = nullptr);
constexpr int kMassPartials = 1024;

}  // namespace cuesim
