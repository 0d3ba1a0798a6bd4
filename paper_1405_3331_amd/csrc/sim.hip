// sim.hip -- host side of the C ABI (include/cuesim.h): parameter validation, device
// allocation and upload, the step loop, state read-back and write, error reporting.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <new>
#include <string>
#include <vector>

#include "cuesim.h"
#include "internal.hpp"
#include "memory.hpp"
#include "validate.hpp"
#include "tiled.hpp"

using namespace cuesim;

namespace {

thread_local std::string g_create_error;

// Steps between refreshes of the spatial order of 3D cones (a cone moves step_len per step;
// 8, 16, 32 and 64 were measured at 256^3, 32 was fastest).
constexpr int kOrderRefresh = 32;
}  // namespace

// Record of the last sim_adjoint_run: checkpoints every `every` steps of the forward run
// (fields and caller-order cone state), the loss's per-cone target tips and weights.
struct AdjointRun {
    int64_t n0 = 0, n_steps = 0;
    int every = 1, n_ckpt = 0;
    float* ckpt_field = nullptr;        // [n_ckpt][n_species][n_cells]
    float* ckpt_pos = nullptr;          // [n_ckpt][M][2]
    float* ckpt_dir = nullptr;          // [n_ckpt][M]
    int32_t* ckpt_int = nullptr;        // [n_ckpt][3][M]: status, target, event_step
    int32_t* stop = nullptr;            // [2][M]: status and event step at the run's end
    float* tip_target = nullptr;        // [M][2]: t_a(i)
    float* weight = nullptr;            // [M]
    float* acone = nullptr;             // [M][3]
    double* loss_partial = nullptr;     // [cone workgroups]
    float* tape = nullptr;              // [n_steps + 1][n_species][n_cells]: every field state
                                        // of the run, recorded as it ran (null: not recorded)
    float4* cone_tape = nullptr;        // and every cone step (ConeTape; null: the fields alone)
    float4* cone_unkept = nullptr;      // [M]: where the run puts cone steps that are not kept
    // The reverse sweep's workspace, allocated by its first call and kept for further calls
    // on the same record (freed with the record).
    struct Work {
        bool ready = false;
        bool whole = false;             // the field window is the whole run (else one segment)
        int cone_segs = 1;              // segments of the cone window
        float* tape_own = nullptr;      // the windows' field states and cone steps, where the run
        float4* tape_cones = nullptr;   // did not record them
        float2* ag = nullptr;           // two segments' sample adjoints [2][K][M]
        uint32_t* step_max = nullptr;   // [K]
        float4* boxes = nullptr;        // the cones' tips per launch, and the cones that touch
        int32_t* list_end = nullptr;    // each tile
        int32_t* list = nullptr;
        float* afield = nullptr;        // the field adjoint, ping-pong per species
        double* acc = nullptr;          // FP64 accumulators
        int32_t* q_start = nullptr;     // the sources listed per tile
        int2* q_entry = nullptr;
    } work;
};


struct sim_handle {
    // geometry and coefficients
    int dim = 2, nx = 0, ny = 0, nz = 1;
    int64_t n_cells = 0;
    double dx = 1.0, dt = 1.0;
    int n_species = 1;
    StencilCoef coef[SIM_MAX_SPECIES] = {};
    int n_cones = 0, n_targets = 0;
    ConeRules rules = {};

    hipStream_t stream = nullptr;
    bool own_stream = false;
    int device = 0;

    // device state
    float* field[SIM_MAX_SPECIES][2] = {};
    int cur[SIM_MAX_SPECIES] = {0, 0};
    Field2DStep field2d = {};   // 2D un-blocked field step with its per-box source lists
    ConeArrays cones = {};
    char* cone_memory = nullptr;     // the arrays of `cones`
    char* target_memory = nullptr;   // the target grid
    uint32_t* near_map = nullptr;    // and its near map, with the mass check's flag behind it
    double* mass_partial = nullptr;
    double* mass_out = nullptr;
    // periodic mass check: every mass_every steps (0: off) sim_step enqueues the FP64 mass of
    // every species; a non-finite total raises the device flag mass_flag, copied to the
    // pinned host word behind the event of mass_host.  `nonfinite` is sticky:
    // set by a check that saw a non-finite total, cleared by a SIM_MASS read whose totals
    // are all finite.
    int64_t mass_every = 0;
    int32_t* mass_flag = nullptr;
    HostFlag mass_host;   // mass_flag's copy
    bool mass_pending = false;
    bool nonfinite = false;

    // temporal blocking
    int block_steps = 1;
    TiledPlan plan = {};
    TiledState tiled = {};
    bool cones_bucketed = false;   // active cones live in the tile buckets
    bool cones_synced = true;      // the caller-order arrays hold the active cones' state
    bool captured = false;         // launches were captured: a caller's graph may replay them

    // 3D: field step with its per-box source lists; active cones in spatial order,
    // refreshed every kOrderRefresh steps
    Field3D field3d = {};
    ConeOrder3D order3d = {};
    bool cones_ordered = false;    // tips and headings of active cones live in order3d
    int since_refresh = 0;

    int64_t step = 0;
    bool poisoned = false;
    std::string err;

    // caller-order inputs the adjoint needs
    std::vector<float> target_host;                          // [T][dim]
    std::vector<int32_t> src_caller_cell[SIM_MAX_SPECIES];   // per source, caller order
    std::vector<int32_t> src_merged_cell[SIM_MAX_SPECIES];   // merged, sorted by cell
    std::vector<float> src_merged_q[SIM_MAX_SPECIES];        // their amounts / dx^dim
    AdjointRun* adj = nullptr;
    int64_t adj_tape_limit = 0;   // bytes the gradient may record (0: half the free memory)
    float* record = nullptr;      // recording a run (per-step path): tape of its field states
    ConeTape cone_record = {};    // and of its cone steps
    int64_t record_n0 = 0;        // step of the tape's first state
    GraphBuffers graph = {};                                 // last sim_connectivity
    int graph_cones = 0;

    // timing of the step kernel
    bool timing = false;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> events;
    double timed_ms = 0.0;
    int64_t timed_launches = 0;
};

namespace {

sim_status fail(sim_handle* h, sim_status st, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (h)
        h->err = buf;
    else
        g_create_error = buf;
    return st;
}

bool sticky(hipError_t e) {
    return e == hipErrorIllegalAddress || e == hipErrorLaunchFailure ||
           e == hipErrorAssert || e == hipErrorECCNotCorrectable;
}

sim_status device_fail(sim_handle* h, hipError_t e, const char* what) {
    if (h && sticky(e)) h->poisoned = true;
    return fail(h, e == hipErrorOutOfMemory ? SIM_ENOMEM : SIM_EDEVICE, "%s: %s (%d)", what,
                hipGetErrorString(e), (int)e);
}

#define HIP_TRY(h, expr)                                       \
    do {                                                       \
        hipError_t e_ = (expr);                                \
        if (e_ != hipSuccess) return device_fail(h, e_, #expr); \
    } while (0)

template <class T>
hipError_t dalloc(T** p, size_t count) {
    *p = nullptr;
    if (count == 0) return hipSuccess;
    return device_malloc((void**)p, count * sizeof(T));
}

template <class T>
void dfree(T*& p) {
    device_free(p);
    p = nullptr;
}

void drop_events(sim_handle* h) {
    for (auto& ev : h->events) {
        (void)hipEventDestroy(ev.first);
        (void)hipEventDestroy(ev.second);
    }
    h->events.clear();
}

static void adjoint_work_release(AdjointRun::Work& w) {
    dfree(w.tape_own);
    dfree(w.tape_cones);
    dfree(w.ag);
    dfree(w.step_max);
    dfree(w.boxes);
    dfree(w.list_end);
    dfree(w.list);
    dfree(w.afield);
    dfree(w.acc);
    dfree(w.q_start);
    dfree(w.q_entry);
    w = AdjointRun::Work();
}

// (the handle's stream may still be at work on what is given back: wait for it)
void adjoint_release(sim_handle* h) {
    AdjointRun* a = h->adj;
    if (!a) return;
    (void)hipStreamSynchronize(h->stream);
    dfree(a->ckpt_field);
    dfree(a->ckpt_pos);
    dfree(a->ckpt_dir);
    dfree(a->ckpt_int);
    dfree(a->stop);
    dfree(a->tip_target);
    dfree(a->weight);
    dfree(a->acone);
    dfree(a->loss_partial);
    dfree(a->tape);
    dfree(a->cone_tape);
    dfree(a->cone_unkept);
    adjoint_work_release(a->work);
    delete a;
    h->adj = nullptr;
}

void graph_release(sim_handle* h) {
    GraphBuffers& g = h->graph;
    if (g.row_start) (void)hipStreamSynchronize(h->stream);
    dfree(g.owner);
    dfree(g.target_owner);
    dfree(g.key);
    dfree(g.cone);
    dfree(g.key_sorted);
    dfree(g.cone_sorted);
    dfree(g.degree);
    dfree(g.row_start);
    dfree(g.edges);
    dfree(g.level);
    dfree(g.grew);
    dfree(g.scratch);
    g = GraphBuffers{};
}

void release(sim_handle* h) {
    // what is given back may be reused at once: wait for all work on the device, the caller's
    // on a view of a field among it
    int current = h->device;
    (void)hipGetDevice(&current);
    if (current != h->device) (void)hipSetDevice(h->device);
    (void)hipDeviceSynchronize();
    if (current != h->device) (void)hipSetDevice(current);
    adjoint_release(h);
    graph_release(h);
    for (int s = 0; s < SIM_MAX_SPECIES; ++s) {
        for (int b = 0; b < 2; ++b) dfree(h->field[s][b]);
    }
    dfree(h->cone_memory);
    dfree(h->target_memory);
    dfree(h->near_map);
    dfree(h->mass_partial);   // and mass_out
    host_flag_free(h->mass_host);
    h->mass_host = HostFlag{};
    tiled_release(h->tiled);
    order3d_release(h->order3d);
    field3d_release(h->field3d);
    field2d_release(h->field2d);
    drop_events(h);
    if (h->own_stream && h->stream) (void)hipStreamDestroy(h->stream);
    h->stream = nullptr;
    device_memory_user(-1);
}

// Fold a finished periodic mass check into the sticky flag (never waits).
void poll_mass_check(sim_handle* h) {
    if (!h->mass_pending || hipEventQuery(h->mass_host.event) != hipSuccess) return;
    h->mass_pending = false;
    if (*(volatile int32_t*)h->mass_host.word) h->nonfinite = true;
}

sim_status nonfinite_fail(sim_handle* h) {
    return fail(h, SIM_ENONFINITE,
                "a mass check found a non-finite total: replace the state (sim_write_state) "
                "and read SIM_MASS to clear");
}

int dir_width(int dim) { return dim == 2 ? 1 : 3; }

// Validate the parameter struct (validate.cpp).  Returns SIM_OK or an error with
// g_create_error set.
sim_status validate(const sim_params* p) {
    char msg[512];
    const sim_status st = validate_params(p, msg, sizeof msg);
    if (st != SIM_OK) return fail(nullptr, st, "%s", msg);
    return SIM_OK;
}

// Bucket targets into cubic cells of side >= contact radius (host counting sort, once).
sim_status build_targets(sim_handle* h, const sim_params* p) {
    const int dim = p->dim;
    const double L[3] = {h->nx * h->dx, h->ny * h->dx, h->nz * h->dx};
    const double longest = std::max(L[0], std::max(L[1], dim == 3 ? L[2] : 0.0));
    const int max_per_axis = dim == 2 ? 512 : 128;
    double cell = std::max(p->contact_radius, longest / max_per_axis);
    if (!(cell > 0)) cell = longest;
    int g[3] = {1, 1, 1};
    for (int a = 0; a < dim; ++a) g[a] = std::max(1, (int)std::ceil(L[a] / cell));
    const int64_t n_cells = (int64_t)g[0] * g[1] * g[2];
    std::vector<int32_t> start(n_cells + 1, 0);
    std::vector<int64_t> key(p->n_targets);
    for (int t = 0; t < p->n_targets; ++t) {
        int c[3] = {0, 0, 0};
        for (int a = 0; a < dim; ++a) {
            const double v = std::floor((double)p->target_pos[(int64_t)t * dim + a] / cell);
            c[a] = (int)std::min<double>(std::max<double>(v, 0.0), g[a] - 1);
        }
        key[t] = ((int64_t)c[2] * g[1] + c[1]) * g[0] + c[0];
        start[key[t] + 1] += 1;
    }
    for (int64_t c = 0; c < n_cells; ++c) start[c + 1] += start[c];
    std::vector<float4> pts(std::max(1, p->n_targets));
    std::vector<int32_t> fill(start.begin(), start.end() - 1);
    for (int t = 0; t < p->n_targets; ++t) {
        const float* tp = p->target_pos + (int64_t)t * dim;
        float4 v;
        v.x = tp[0];
        v.y = tp[1];
        v.z = dim == 3 ? tp[2] : 0.0f;
        int32_t idx = t;
        std::memcpy(&v.w, &idx, sizeof idx);
        pts[fill[key[t]]++] = v;
    }
    UploadBlock up;
    const size_t at_pts = up.add(pts), at_start = up.add(start);
    HIP_TRY(h, up.upload(&h->target_memory));
    TargetGrid& tg = h->rules.targets;
    tg.pts = (const float4*)(h->target_memory + at_pts);
    tg.cell_start = (const int32_t*)(h->target_memory + at_start);
    tg.gx = g[0];
    tg.gy = g[1];
    tg.gz = g[2];
    tg.inv_cell = (float)(1.0 / cell);
    tg.r = (float)p->contact_radius;
    tg.r2 = (float)(p->contact_radius * p->contact_radius);
    // the near map: cells of the contact radius where that gives at most 2048 (3D: 256) per
    // axis (512 KB, 2 MB), so that few tips share a cell with a target's reach
    const double near = std::max(p->contact_radius, longest / (dim == 2 ? 2048 : 256));
    int n[3] = {1, 1, 1};
    for (int a = 0; a < dim; ++a) n[a] = std::max(1, (int)std::ceil(L[a] / near));
    tg.near_nx = n[0];
    tg.near_ny = n[1];
    tg.near_nz = n[2];
    tg.near_inv = (float)(1.0 / near);
    tg.near_wx = (n[0] + (dim == 2 ? 7 : 3)) / (dim == 2 ? 8 : 4);
    tg.near_wy = (n[1] + 3) / 4;
    const size_t words = (size_t)tg.near_wx * tg.near_wy * (size_t)((n[2] + 1) / 2);
    HIP_TRY(h, dalloc(&h->near_map, words + 1));
    tg.near = h->near_map;
    h->mass_flag = (int32_t*)(h->near_map + words);   // zeroed with the map
    HIP_TRY(h, launch_near_map(dim, tg, h->near_map, words + 1, p->n_targets, h->stream));
    return SIM_OK;
}

// Merge sources sharing a cell (amounts summed in double) and scale by 1/dx^dim; the field
// kernels take them from these host lists.
void merge_sources(sim_handle* h, const sim_params* p, int s) {
    std::map<int32_t, double> merged;
    const double vol = std::pow(p->dx, p->dim);
    for (int m = 0; m < p->n_sources[s]; ++m)
        merged[p->source_cell[s][m]] += (double)p->source_q[s][m] / vol;
    h->src_merged_cell[s].clear();
    h->src_merged_q[s].clear();
    for (auto& kv : merged) {
        h->src_merged_cell[s].push_back(kv.first);
        h->src_merged_q[s].push_back((float)kv.second);
    }
}

sim_status item_size(sim_handle* h, sim_item what, int32_t index, size_t* bytes) {
    const size_t M = (size_t)h->n_cones;
    switch (what) {
        case SIM_FIELD:
            if (index < 0 || index >= h->n_species)
                return fail(h, SIM_EINVAL, "species index %d out of range", index);
            *bytes = (size_t)h->n_cells * sizeof(float);
            return SIM_OK;
        case SIM_CONE_POS: *bytes = M * h->dim * sizeof(float); break;
        case SIM_CONE_DIR: *bytes = M * dir_width(h->dim) * sizeof(float); break;
        case SIM_CONE_STATUS:
        case SIM_CONE_TARGET:
        case SIM_CONE_EVENT_STEP: *bytes = M * sizeof(int32_t); break;
        case SIM_MASS: *bytes = (size_t)h->n_species * sizeof(double); break;
        case SIM_STEP: *bytes = sizeof(int64_t); break;
        case SIM_COUNTS: *bytes = 3 * sizeof(int32_t); break;
        case SIM_KERNEL_TIME: *bytes = 2 * sizeof(double); break;
        case SIM_TILING: *bytes = 8 * sizeof(int32_t); break;
        case SIM_EVENTS: *bytes = 0; break;  // computed by the caller of item_size
        default: return fail(h, SIM_EINVAL, "unknown item %d", (int)what);
    }
    if (index != 0) return fail(h, SIM_EINVAL, "index must be 0 for item %d", (int)what);
    return SIM_OK;
}

// Where a caller's graph may have replayed launches, the host's copies of the launch state (which
// half of the fields and buckets is current, which third of the counts) are taken from the device's.
sim_status follow_replays(sim_handle* h) {
    if (!h->captured) return SIM_OK;
    HIP_TRY(h, hipStreamSynchronize(h->stream));
    HIP_TRY(h, tiled_get_launch_state(h->tiled));
    for (int s = 0; s < h->n_species; ++s) h->cur[s] = h->tiled.cur;
    h->cones_synced = !h->cones_bucketed;
    return SIM_OK;
}

// Bring the caller-order arrays up to date with the active cones' working copies (the tile
// buckets, or the 3D spatial order), which stay valid: stepping goes on from them.
sim_status sync_cones(sim_handle* h) {
    const sim_status st = follow_replays(h);
    if (st != SIM_OK) return st;
    if (h->cones_synced) return SIM_OK;
    if (h->cones_ordered) HIP_TRY(h, order3d_end(h->order3d, h->cones, h->stream));
    if (h->cones_bucketed)
        HIP_TRY(h, tiled_sync_cones(h->plan, h->tiled, h->cones, h->stream, false));
    h->cones_synced = true;
    return SIM_OK;
}

// The same, and the working copies are given up: the caller-order arrays are about to change.
sim_status unbucket(sim_handle* h) {
    sim_status st = follow_replays(h);
    if (st != SIM_OK) return st;
    if (h->cones_bucketed) {
        HIP_TRY(h, tiled_sync_cones(h->plan, h->tiled, h->cones, h->stream, true));
        h->cones_bucketed = false;
    } else {
        st = sync_cones(h);
        if (st != SIM_OK) return st;
    }
    h->cones_ordered = false;
    h->cones_synced = true;
    return SIM_OK;
}

// A start/stop event pair for the next timed launch (both null when timing is off).  The
// launch records them itself (hipExtLaunchKernel: the dispatch packet carries the
// timestamps), so timing adds no commands between launches.
sim_status timing_events(sim_handle* h, hipEvent_t* start, hipEvent_t* stop) {
    *start = *stop = nullptr;
    if (!h->timing) return SIM_OK;
    HIP_TRY(h, hipEventCreate(start));
    HIP_TRY(h, hipEventCreate(stop));
    h->events.emplace_back(*start, *stop);
    return SIM_OK;
}

sim_status collect_timing(sim_handle* h) {
    for (auto& ev : h->events) {
        float ms = 0.0f;
        HIP_TRY(h, hipEventSynchronize(ev.second));
        HIP_TRY(h, hipEventElapsedTime(&ms, ev.first, ev.second));
        h->timed_ms += ms;
        h->timed_launches += 1;
    }
    drop_events(h);
    return SIM_OK;
}

// The field step of every species in one launch, sources included.
sim_status plain_field(sim_handle* h) {
    hipEvent_t t0, t1;
    sim_status st = timing_events(h, &t0, &t1);
    if (st != SIM_OK) return st;
    const float* in[SIM_MAX_SPECIES] = {};
    float* out[SIM_MAX_SPECIES] = {};
    for (int s = 0; s < h->n_species; ++s) {
        in[s] = h->field[s][h->cur[s]];
        out[s] = h->field[s][h->cur[s] ^ 1];
    }
    if (h->dim == 3)
        HIP_TRY(h, launch_field3d(h->field3d, in, out, h->coef, h->stream, t0, t1));
    else
        HIP_TRY(h, launch_field2d_rows(h->field2d, in, out, h->coef, h->stream, t0, t1));
    for (int s = 0; s < h->n_species; ++s) h->cur[s] ^= 1;
    if (h->record)   // recording a run: the new state goes to the tape
        for (int s = 0; s < h->n_species; ++s)
            HIP_TRY(h, hipMemcpyAsync(h->record + ((size_t)(h->step + 1 - h->record_n0) *
                                                       h->n_species + s) * h->n_cells,
                                      h->field[s][h->cur[s]], (size_t)h->n_cells * 4,
                                      hipMemcpyDeviceToDevice, h->stream));
    return SIM_OK;
}

// n un-blocked steps: each is the field step, then the cones against the new fields (2D: in
// caller order; 3D: in spatial order).  The cones change no field, so a step's cones and the
// next step's field share a launch; with launches timed (each then times a field step alone) or
// a run recorded, every part has its own.
sim_status plain_steps(sim_handle* h, int64_t n) {
    const bool shared = !h->timing && !h->record && h->cones.n > 0;
    for (int64_t i = 0; i < n; ++i) {
        if (i == 0 || !shared) {
            const sim_status st = plain_field(h);
            if (st != SIM_OK) return st;
        }
        const float* f[SIM_MAX_SPECIES] = {};
        float* out[SIM_MAX_SPECIES] = {};
        for (int s = 0; s < h->n_species; ++s) {
            f[s] = h->field[s][h->cur[s]];
            out[s] = h->field[s][h->cur[s] ^ 1];
        }
        const float* f1 = h->n_species > 1 ? f[1] : f[0];
        const bool with_field = shared && i + 1 < n;
        const uint32_t step = (uint32_t)h->step;
        if (h->dim == 2) {
            if (with_field)
                HIP_TRY(h, launch_step2d(h->rules, h->cones, step,
                                         field2d_args(h->field2d, f, out, h->coef), h->stream));
            else
                HIP_TRY(h, launch_cones2d(h->rules, f[0], f1, h->cones, step, h->stream,
                                          h->record ? &h->cone_record : nullptr,
                                          (size_t)(h->step - h->record_n0)));
        } else if (h->order3d.n > 0) {
            if (!h->cones_ordered) {
                HIP_TRY(h, order3d_begin(h->order3d, h->rules, h->cones, h->stream));
                h->cones_ordered = true;
                h->since_refresh = 0;
            } else if (h->since_refresh >= kOrderRefresh) {
                HIP_TRY(h, order3d_refresh(h->order3d, h->rules, h->stream));
                h->since_refresh = 0;
            }
            if (with_field)
                HIP_TRY(h, launch_step3d(h->rules, h->order3d, h->cones, step,
                                         field3d_args(h->field3d, f, out, h->coef), h->stream));
            else
                HIP_TRY(h, launch_cones3d_ordered(h->rules, f[0], f1, h->order3d, h->cones, step,
                                                  h->stream));
            h->since_refresh += 1;
        }
        if (with_field)
            for (int s = 0; s < h->n_species; ++s) h->cur[s] ^= 1;
        h->step += 1;
        h->cones_synced = h->dim == 2;   // a 2D step works on the caller-order arrays
    }
    return SIM_OK;
}

sim_status tiled_steps(sim_handle* h, int64_t n) {
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(h->stream, &capture) != hipSuccess) (void)hipGetLastError();
    if (capture != hipStreamCaptureStatusNone) {
        h->captured = true;
    } else if (!h->cones_bucketed || h->mass_every > 0) {   // what uses the host's copies
        const sim_status st = follow_replays(h);
        if (st != SIM_OK) return st;
    }
    if (!h->cones_bucketed) {
        HIP_TRY(h, tiled_bucket(h->plan, h->tiled, h->cones, h->stream));
        h->cones_bucketed = true;
    }
    while (n > 0) {
        const int b = (int)std::min<int64_t>(n, h->plan.block_steps);
        hipEvent_t t0, t1;
        sim_status st = timing_events(h, &t0, &t1);
        if (st != SIM_OK) return st;
        HIP_TRY(h, tiled_launch(h->plan, h->tiled, b, h->stream, t0, t1));
        h->cones_synced = false;
        for (int s = 0; s < h->n_species; ++s) h->cur[s] ^= 1;
        h->step += b;
        n -= b;
    }
    return SIM_OK;
}

// sim_create, with `member` as the tiling of a batch's member.
sim_status create_impl(const sim_params* p, void* hip_stream, const TiledPlan* member,
                       sim_handle** out) {
    if (!out) return fail(nullptr, SIM_EINVAL, "out is NULL");
    *out = nullptr;
    sim_status st = validate(p);
    if (st != SIM_OK) return st;
    sim_handle* h = new (std::nothrow) sim_handle();
    if (!h) return fail(nullptr, SIM_ENOMEM, "host allocation failed");
    device_memory_user(1);
    auto bail = [&](sim_status s) {
        g_create_error = h->err;
        release(h);
        delete h;
        return s;
    };
    h->dim = p->dim;
    h->nx = p->nx;
    h->ny = p->ny;
    h->nz = p->dim == 3 ? p->nz : 1;
    h->n_cells = (int64_t)h->nx * h->ny * h->nz;
    h->dx = p->dx;
    h->dt = p->dt;
    h->n_species = p->n_species;
    h->n_cones = p->n_cones;
    h->n_targets = p->n_targets;
    hipError_t e = hipGetDevice(&h->device);
    if (e != hipSuccess) return bail(device_fail(h, e, "hipGetDevice"));
    if (hip_stream) {
        h->stream = (hipStream_t)hip_stream;
    } else {
        e = hipStreamCreateWithFlags(&h->stream, hipStreamNonBlocking);
        if (e != hipSuccess) return bail(device_fail(h, e, "hipStreamCreate"));
        h->own_stream = true;
    }
    for (int s = 0; s < p->n_species; ++s) {
        const double r = p->D[s] * p->dt / (p->dx * p->dx);
        h->coef[s].r = (float)r;
        h->coef[s].kdt = (float)(p->k[s] * p->dt);
    }
    ConeRules& R = h->rules;
    R.nx = h->nx;
    R.ny = h->ny;
    R.nz = h->nz;
    R.inv_dx = (float)(1.0 / p->dx);
    R.half_inv_dx = (float)(0.5 / p->dx);
    R.Lx = (float)(h->nx * p->dx);
    R.Ly = (float)(h->ny * p->dx);
    R.Lz = (float)(h->nz * p->dx);
    R.step_len = (float)p->step_len;
    R.gain = (float)p->turn_gain;
    R.max_turn = (float)p->max_turn;
    R.turn_law = p->turn_law;
    R.snr_coef = (float)(p->snr_scale * p->cone_width);
    R.inv_kd = p->turn_law == SIM_TURN_SNR ? (float)(1.0 / p->kd) : 0.0f;
    R.c_min = (float)p->c_min;
    R.c_max = (float)p->c_max;
    R.tan_max = p->max_turn <= kSmallCap ? (float)std::tan(p->max_turn) : 0.0f;
    R.sigma = (float)p->noise_sigma;
    R.sign0 = (float)p->sign[0];
    R.sign1 = p->n_species > 1 ? (float)p->sign[1] : 0.0f;
    R.n_species = p->n_species;
    R.key.k0 = (uint32_t)(p->seed & 0xffffffffu);
    R.key.k1 = (uint32_t)(p->seed >> 32);
    R.key.sim_index = p->sim_index;

    // fields
    for (int s = 0; s < p->n_species; ++s) {
        for (int b = 0; b < 2; ++b) {
            e = dalloc(&h->field[s][b], (size_t)h->n_cells);
            if (e != hipSuccess) return bail(device_fail(h, e, "field allocation"));
        }
        if (p->init_field[s])
            e = hipMemcpy(h->field[s][0], p->init_field[s], h->n_cells * sizeof(float),
                          hipMemcpyHostToDevice);
        else
            e = hipMemset(h->field[s][0], 0, h->n_cells * sizeof(float));
        if (e != hipSuccess) return bail(device_fail(h, e, "field upload"));
        merge_sources(h, p, s);
        h->src_caller_cell[s].assign(p->source_cell[s], p->source_cell[s] + p->n_sources[s]);
    }
    // cones (caller order)
    const size_t M = (size_t)p->n_cones;
    h->cones.n = p->n_cones;
    {
        const std::vector<int32_t> active(M, kActive), minus1(M, -1);
        UploadBlock up;
        const size_t at_pos = up.add(p->cone_pos, M * p->dim),
                     at_dir = up.add(p->cone_dir, M * dir_width(p->dim)),
                     at_status = up.add(active), at_target = up.add(minus1),
                     at_event = up.add(minus1);
        e = up.upload(&h->cone_memory);
        if (e != hipSuccess) return bail(device_fail(h, e, "cone upload"));
        h->cones.pos = (float*)(h->cone_memory + at_pos);
        h->cones.dir = (float*)(h->cone_memory + at_dir);
        h->cones.status = (int32_t*)(h->cone_memory + at_status);
        h->cones.target = (int32_t*)(h->cone_memory + at_target);
        h->cones.event_step = (int32_t*)(h->cone_memory + at_event);
    }
    // The mass check's memory is made here (its flag with the near map), so that none of its calls
    // needs any.
    if ((e = dalloc(&h->mass_partial, kMassPartials + SIM_MAX_SPECIES)) != hipSuccess ||
        (e = host_flag(&h->mass_host)) != hipSuccess)
        return bail(device_fail(h, e, "mass check set-up"));
    h->mass_out = h->mass_partial + kMassPartials;
    if (p->dim == 3)
        e = field3d_prepare(h->field3d, h->nx, h->ny, h->nz, h->n_species, h->src_merged_cell,
                            h->src_merged_q);
    else
        e = field2d_prepare(h->field2d, h->nx, h->ny, h->n_species, h->src_merged_cell,
                            h->src_merged_q);
    if (e != hipSuccess) return bail(device_fail(h, e, "field step set-up"));
    if (p->dim == 3 && M > 0) {
        e = order3d_allocate(h->order3d, p->n_cones, h->nx, h->ny, h->nz);
        if (e != hipSuccess) return bail(device_fail(h, e, "cone order allocation"));
    }
    st = build_targets(h, p);
    if (st != SIM_OK) return bail(st);
    h->target_host.assign(p->target_pos, p->target_pos + (size_t)p->n_targets * p->dim);
    // temporal blocking plan
    h->block_steps = p->block_steps;   // 0: the planner's choice
    if (h->block_steps != 1) {
        h->plan = member ? *member
                         : tiled_plan(h->dim, h->nx, h->ny, h->nz, h->n_species,
                                      p->step_len / p->dx, h->block_steps, h->n_cones,
                                      p->tile_cols_per_lane, p->tile_height);
        h->plan.inv_dx = h->rules.inv_dx;
        for (int s = 0; s < h->n_species; ++s) h->plan.coef[s] = h->coef[s];
        if (h->plan.block_steps <= 1) {
            h->block_steps = 1;   // no tile shape fits: fall back to one step per launch
        } else {
            h->block_steps = h->plan.block_steps;
            e = tiled_allocate(h->plan, h->tiled, h->n_cones, h->rules, p, h->field, h->cones,
                               h->stream);
            if (e != hipSuccess) return bail(device_fail(h, e, "tiled state allocation"));
        }
    }
    e = hipDeviceSynchronize();
    if (e != hipSuccess) return bail(device_fail(h, e, "create synchronisation"));
    *out = h;
    return SIM_OK;
}

}  // namespace

struct sim_batch {
    std::vector<sim_handle*> sims;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    void* table = nullptr;            // concatenated device argument tables
    int2* base = nullptr;             // every (simulation, tile), largest simulations first
    int n_base = 0;
    int4* extra = nullptr;            // further parts of crowded tiles, [parity][extra_cap]
    int extra_cap = 0;
    LaunchState* launch = nullptr;
    int n_species = 1, cpl = 2, block_steps = 1;
    size_t lds_bytes = 0;
    int64_t step = 0;
    int graph_launches = 0;           // launches captured in `graph` (0: no graph)
    hipGraph_t graph = nullptr;
    hipGraphExec_t graph_exec = nullptr;
    std::string err;
};

namespace {

sim_status batch_fail(sim_batch* b, sim_status st, const char* msg) {
    if (b)
        b->err = msg;
    else
        g_create_error = msg;
    return st;
}

#define BATCH_TRY(b, expr)                                                        \
    do {                                                                          \
        hipError_t e_ = (expr);                                                   \
        if (e_ != hipSuccess) {                                                   \
            char m_[256];                                                         \
            snprintf(m_, sizeof m_, "%s: %s (%d)", #expr, hipGetErrorString(e_), (int)e_); \
            return batch_fail(b, e_ == hipErrorOutOfMemory ? SIM_ENOMEM : SIM_EDEVICE, m_); \
        }                                                                         \
    } while (0)

void batch_release(sim_batch* b) {
    if (b->graph_exec) (void)hipGraphExecDestroy(b->graph_exec);
    if (b->graph) (void)hipGraphDestroy(b->graph);
    b->graph_exec = nullptr;
    b->graph = nullptr;
    for (sim_handle* h : b->sims) {
        if (!h) continue;
        release(h);
        delete h;
    }
    b->sims.clear();
    device_free(b->table);
    device_free(b->extra);
    device_free(b->base);
    device_free(b->launch);
    b->table = nullptr;
    b->extra = nullptr;
    b->base = nullptr;
    b->launch = nullptr;
    if (b->own_stream && b->stream) (void)hipStreamDestroy(b->stream);
    b->stream = nullptr;
}

// One launch of `steps` steps for every simulation of the batch.
sim_status batch_launch(sim_batch* b, int steps) {
    BATCH_TRY(b, tiled_launch_batch((const TiledArgs2D*)b->table, b->extra, b->base,
                                    b->n_base, b->extra_cap, b->n_species, b->cpl,
                                    b->lds_bytes, steps, b->launch, b->stream));
    return SIM_OK;
}

// Mirror a completed launch of `steps` steps in every simulation's host-side state.
void batch_advance(sim_batch* b, int steps, int launches) {
    for (sim_handle* h : b->sims) {
        for (int s = 0; s < h->n_species; ++s) h->cur[s] ^= launches & 1;
        tiled_advanced(h->tiled, launches);
        h->cones_synced = false;
        h->step += (int64_t)steps * launches;
    }
    b->step += (int64_t)steps * launches;
}

}  // namespace

namespace cuesim {

sim_status handle_fail(sim_handle* h, sim_status st, const char* msg) {
    return fail(h, st, "%s", msg);
}

int handle_cones(const sim_handle* h) { return h->n_cones; }

int handle_targets(const sim_handle* h) { return h->n_targets; }

int handle_device(const sim_handle* h) { return h->device; }

sim_status connectivity_validate(sim_handle* h, int32_t n_neurons, const int32_t* cone_owner,
                                 const int32_t* target_owner, const int32_t* row_start,
                                 const int32_t* edges, int64_t edge_capacity,
                                 const int64_t* n_edges) {
    if (!h) return fail(nullptr, SIM_EINVAL, "handle is NULL");
    if (h->poisoned) return fail(h, SIM_ESTATE, "handle poisoned by an earlier device error");
    const int M = h->n_cones, T = h->n_targets;
    if (n_neurons < 1) return fail(h, SIM_EINVAL, "n_neurons < 1");
    if (!row_start || !n_edges || edge_capacity < 0 || (edge_capacity > 0 && !edges) ||
        (M > 0 && !cone_owner) || (T > 0 && !target_owner))
        return fail(h, SIM_EINVAL, "NULL pointer or negative capacity");
    for (int i = 0; i < M; ++i)
        if (cone_owner[i] < 0 || cone_owner[i] >= n_neurons)
            return fail(h, SIM_EINVAL, "cone_owner[%d] = %d out of range", i, cone_owner[i]);
    for (int t = 0; t < T; ++t)
        if (target_owner[t] < 0 || target_owner[t] >= n_neurons)
            return fail(h, SIM_EINVAL, "target_owner[%d] = %d out of range", t, target_owner[t]);
    return SIM_OK;
}

sim_status connectivity_build(sim_handle* h, GraphBuffers& g, const int32_t* cone_owner,
                              const int32_t* target_owner, int32_t* row_start, int32_t* edges,
                              int64_t edge_capacity, int64_t* n_edges) {
    const int M = h->n_cones, T = h->n_targets;
    const size_t N = (size_t)g.n_neurons;
    if (M > 0)
        HIP_TRY(h, hipMemcpyAsync(g.owner, cone_owner, (size_t)M * 4, hipMemcpyHostToDevice,
                                  h->stream));
    if (T > 0)
        HIP_TRY(h, hipMemcpyAsync(g.target_owner, target_owner, (size_t)T * 4,
                                  hipMemcpyHostToDevice, h->stream));
    // stopped cones keep their final status and target in the caller-order arrays
    HIP_TRY(h, launch_adjacency(g, h->cones.status, h->cones.target, M, g.n_neurons,
                                h->stream));
    HIP_TRY(h, hipMemcpyAsync(row_start, g.row_start, (N + 1) * 4, hipMemcpyDeviceToHost,
                              h->stream));
    HIP_TRY(h, hipStreamSynchronize(h->stream));
    const int64_t E = row_start[g.n_neurons];
    *n_edges = E;
    g.n_edges = (int)E;   // at most the cones
    if (E > edge_capacity)
        return fail(h, SIM_ERANGE, "edge buffer holds %lld edges, %lld needed",
                    (long long)edge_capacity, (long long)E);
    if (E > 0) {
        HIP_TRY(h, hipMemcpyAsync(edges, g.edges, (size_t)E * 4, hipMemcpyDeviceToHost,
                                  h->stream));
        HIP_TRY(h, hipStreamSynchronize(h->stream));
    }
    return SIM_OK;
}

}  // namespace cuesim

extern "C" {


sim_status sim_create(const sim_params* p, void* hip_stream, sim_handle** out) {
    return create_impl(p, hip_stream, nullptr, out);
}

sim_status sim_step(sim_handle* h, int64_t n_steps) {
    if (!h) return fail(nullptr, SIM_EINVAL, "handle is NULL");
    if (h->poisoned) return fail(h, SIM_ESTATE, "handle poisoned by an earlier device error");
    if (n_steps < 0) return fail(h, SIM_EINVAL, "n_steps < 0");
    if (h->step + n_steps > 2147483647LL)
        return fail(h, SIM_EINVAL, "step count would exceed 2^31-1");
    poll_mass_check(h);
    if (h->nonfinite) return nonfinite_fail(h);
    if (n_steps == 0) return SIM_OK;
    while (n_steps > 0) {
        // with the periodic mass check on, stop at the next multiple of mass_every
        int64_t n = n_steps;
        if (h->mass_every > 0) n = std::min(n, h->mass_every - h->step % h->mass_every);
        sim_status st = SIM_OK;
        if (h->block_steps > 1) {
            st = tiled_steps(h, n);
        } else {
            st = plain_steps(h, n);
        }
        if (st != SIM_OK) return st;
        n_steps -= n;
        if (h->mass_every > 0 && h->step % h->mass_every == 0) {
            for (int s = 0; s < h->n_species; ++s)
                HIP_TRY(h, launch_mass(h->field[s][h->cur[s]], h->n_cells, h->mass_partial,
                                       kMassPartials, h->mass_out + s, h->stream,
                                       h->mass_flag));
            HIP_TRY(h, hipMemcpyAsync(h->mass_host.word, h->mass_flag, sizeof(int32_t),
                                      hipMemcpyDeviceToHost, h->stream));
            HIP_TRY(h, hipEventRecord(h->mass_host.event, h->stream));
            h->mass_pending = true;
        }
    }
    return SIM_OK;
}

sim_status sim_set_mass_check(sim_handle* h, int64_t every) {
    if (!h) return fail(nullptr, SIM_EINVAL, "handle is NULL");
    if (h->poisoned) return fail(h, SIM_ESTATE, "handle poisoned by an earlier device error");
    if (every < 0) return fail(h, SIM_EINVAL, "every < 0");
    h->mass_every = every;
    return SIM_OK;
}

sim_status sim_read_state(sim_handle* h, sim_item what, int32_t index, void* dst,
                          size_t dst_bytes, size_t* bytes_written) {
    if (!h) return fail(nullptr, SIM_EINVAL, "handle is NULL");
    if (h->poisoned) return fail(h, SIM_ESTATE, "handle poisoned by an earlier device error");
    size_t need = 0;
    sim_status st = item_size(h, what, index, &need);
    if (st != SIM_OK) return st;
    const size_t M = (size_t)h->n_cones;
    if (what == SIM_EVENTS || what == SIM_COUNTS) {
        st = sync_cones(h);
        if (st != SIM_OK) return st;
        HIP_TRY(h, hipStreamSynchronize(h->stream));
        std::vector<int32_t> status(M), target(M), ev(M);
        if (M) {
            HIP_TRY(h, hipMemcpy(status.data(), h->cones.status, M * 4, hipMemcpyDeviceToHost));
            HIP_TRY(h, hipMemcpy(target.data(), h->cones.target, M * 4, hipMemcpyDeviceToHost));
            HIP_TRY(h, hipMemcpy(ev.data(), h->cones.event_step, M * 4, hipMemcpyDeviceToHost));
        }
        if (what == SIM_COUNTS) {
            int32_t counts[3] = {0, 0, 0};
            for (size_t i = 0; i < M; ++i)
                if (status[i] >= 0 && status[i] <= 2) counts[status[i]] += 1;
            if (bytes_written) *bytes_written = sizeof counts;
            if (dst_bytes < sizeof counts) return fail(h, SIM_ERANGE, "buffer too small");
            if (!dst) return fail(h, SIM_EINVAL, "dst is NULL");
            std::memcpy(dst, counts, sizeof counts);
            return SIM_OK;
        }
        std::vector<int32_t> rows;
        std::vector<size_t> order;
        for (size_t i = 0; i < M; ++i)
            if (status[i] != kActive) order.push_back(i);
        std::stable_sort(order.begin(), order.end(),
                         [&](size_t a, size_t b) { return ev[a] < ev[b]; });
        for (size_t i : order) {
            rows.push_back((int32_t)i);
            rows.push_back(target[i]);
            rows.push_back(ev[i]);
            rows.push_back(status[i]);
        }
        need = rows.size() * sizeof(int32_t);
        if (bytes_written) *bytes_written = need;
        if (dst_bytes < need) return fail(h, SIM_ERANGE, "buffer too small: need %zu", need);
        if (need && !dst) return fail(h, SIM_EINVAL, "dst is NULL");
        if (need) std::memcpy(dst, rows.data(), need);
        return SIM_OK;
    }
    if (bytes_written) *bytes_written = need;
    if (dst_bytes < need) return fail(h, SIM_ERANGE, "buffer too small: need %zu", need);
    if (need && !dst) return fail(h, SIM_EINVAL, "dst is NULL");
    switch (what) {
        case SIM_FIELD:
            st = follow_replays(h);
            if (st != SIM_OK) return st;
            HIP_TRY(h, hipStreamSynchronize(h->stream));
            HIP_TRY(h, hipMemcpy(dst, h->field[index][h->cur[index]], need, hipMemcpyDeviceToHost));
            return SIM_OK;
        case SIM_CONE_POS:
        case SIM_CONE_DIR:
        case SIM_CONE_STATUS:
        case SIM_CONE_TARGET:
        case SIM_CONE_EVENT_STEP: {
            st = sync_cones(h);
            if (st != SIM_OK) return st;
            HIP_TRY(h, hipStreamSynchronize(h->stream));
            const void* src = what == SIM_CONE_POS      ? (const void*)h->cones.pos
                              : what == SIM_CONE_DIR    ? (const void*)h->cones.dir
                              : what == SIM_CONE_STATUS ? (const void*)h->cones.status
                              : what == SIM_CONE_TARGET ? (const void*)h->cones.target
                                                        : (const void*)h->cones.event_step;
            if (need) HIP_TRY(h, hipMemcpy(dst, src, need, hipMemcpyDeviceToHost));
            return SIM_OK;
        }
        case SIM_MASS: {
            st = follow_replays(h);
            if (st != SIM_OK) return st;
            for (int s = 0; s < h->n_species; ++s)
                HIP_TRY(h, launch_mass(h->field[s][h->cur[s]], h->n_cells, h->mass_partial,
                                       kMassPartials, h->mass_out + s, h->stream));
            HIP_TRY(h, hipStreamSynchronize(h->stream));
            double m[SIM_MAX_SPECIES];
            HIP_TRY(h, hipMemcpy(m, h->mass_out, h->n_species * sizeof(double),
                                 hipMemcpyDeviceToHost));
            const double vol = std::pow(h->dx, h->dim);
            bool finite = true;
            for (int s = 0; s < h->n_species; ++s) {
                m[s] *= vol;
                finite = finite && std::isfinite(m[s]);
            }
            std::memcpy(dst, m, need);
            // this check supersedes any earlier one: the flag follows what it found
            HIP_TRY(h, hipMemsetAsync(h->mass_flag, 0, sizeof(int32_t), h->stream));
            HIP_TRY(h, hipStreamSynchronize(h->stream));
            *h->mass_host.word = 0;
            h->mass_pending = false;
            h->nonfinite = !finite;
            if (!finite) return nonfinite_fail(h);
            return SIM_OK;
        }
        case SIM_STEP:
            std::memcpy(dst, &h->step, sizeof(int64_t));
            return SIM_OK;
        case SIM_TILING: {
            const TiledPlan& t = h->plan;
            const bool tiled = h->block_steps > 1;
            int32_t v[8] = {tiled ? t.block_steps : 1, tiled ? t.halo : 0, tiled ? t.core_x : 0,
                            tiled ? t.core_y : 0, tiled ? t.n_tiles : 0, tiled ? t.cpl : 0,
                            tiled ? t.height : 0, tiled ? (int32_t)t.lds_bytes : 0};
            std::memcpy(dst, v, sizeof v);
            return SIM_OK;
        }
        case SIM_KERNEL_TIME: {
            HIP_TRY(h, hipStreamSynchronize(h->stream));
            st = collect_timing(h);
            if (st != SIM_OK) return st;
            double v[2] = {h->timed_ms, (double)h->timed_launches};
            std::memcpy(dst, v, sizeof v);
            return SIM_OK;
        }
        default:
            return fail(h, SIM_EINVAL, "item %d is not readable", (int)what);
    }
}

sim_status sim_write_state(sim_handle* h, sim_item what, int32_t index, const void* src,
                           size_t bytes) {
    if (!h) return fail(nullptr, SIM_EINVAL, "handle is NULL");
    if (h->poisoned) return fail(h, SIM_ESTATE, "handle poisoned by an earlier device error");
    size_t need = 0;
    sim_status st = item_size(h, what, index, &need);
    if (st != SIM_OK) return st;
    if (bytes != need) return fail(h, SIM_EINVAL, "size %zu != item size %zu", bytes, need);
    if (need && !src) return fail(h, SIM_EINVAL, "src is NULL");
    switch (what) {
        case SIM_FIELD:
            st = follow_replays(h);
            if (st != SIM_OK) return st;
            HIP_TRY(h, hipStreamSynchronize(h->stream));
            HIP_TRY(h, hipMemcpy(h->field[index][h->cur[index]], src, need, hipMemcpyHostToDevice));
            return SIM_OK;
        case SIM_CONE_POS:
        case SIM_CONE_DIR:
        case SIM_CONE_STATUS:
        case SIM_CONE_TARGET:
        case SIM_CONE_EVENT_STEP: {
            st = unbucket(h);
            if (st != SIM_OK) return st;
            HIP_TRY(h, hipStreamSynchronize(h->stream));
            void* d = what == SIM_CONE_POS      ? (void*)h->cones.pos
                      : what == SIM_CONE_DIR    ? (void*)h->cones.dir
                      : what == SIM_CONE_STATUS ? (void*)h->cones.status
                      : what == SIM_CONE_TARGET ? (void*)h->cones.target
                                                : (void*)h->cones.event_step;
            if (need) HIP_TRY(h, hipMemcpy(d, src, need, hipMemcpyHostToDevice));
            return SIM_OK;
        }
        case SIM_STEP: {
            int64_t v;
            std::memcpy(&v, src, sizeof v);
            if (v < 0 || v > 2147483647LL) return fail(h, SIM_EINVAL, "step out of range");
            st = follow_replays(h);
            if (st != SIM_OK) return st;
            HIP_TRY(h, hipStreamSynchronize(h->stream));
            h->step = v;
            if (h->block_steps > 1)
                HIP_TRY(h, tiled_set_launch_state(h->tiled, (uint32_t)v, h->cur[0], h->stream));
            return SIM_OK;
        }
        default:
            return fail(h, SIM_EINVAL, "item %d is not writable", (int)what);
    }
}

sim_status sim_device_ptr(sim_handle* h, sim_item what, int32_t index, void** dev_ptr,
                          size_t* bytes) {
    if (!h || !dev_ptr) return fail(h, SIM_EINVAL, "NULL argument");
    if (h->poisoned) return fail(h, SIM_ESTATE, "handle poisoned by an earlier device error");
    if (what != SIM_FIELD) return fail(h, SIM_EINVAL, "only SIM_FIELD has a device view");
    size_t need = 0;
    sim_status st = item_size(h, what, index, &need);
    if (st == SIM_OK) st = follow_replays(h);
    if (st != SIM_OK) return st;
    *dev_ptr = h->field[index][h->cur[index]];
    if (bytes) *bytes = need;
    return SIM_OK;
}

sim_status sim_set_timing(sim_handle* h, int32_t enable) {
    if (!h) return fail(nullptr, SIM_EINVAL, "handle is NULL");
    if (h->poisoned) return fail(h, SIM_ESTATE, "handle poisoned by an earlier device error");
    HIP_TRY(h, hipStreamSynchronize(h->stream));
    drop_events(h);
    h->timing = enable != 0;
    h->timed_ms = 0.0;
    h->timed_launches = 0;
    return SIM_OK;
}

sim_status sim_synchronize(sim_handle* h) {
    if (!h) return fail(nullptr, SIM_EINVAL, "handle is NULL");
    if (h->poisoned) return fail(h, SIM_ESTATE, "handle poisoned by an earlier device error");
    HIP_TRY(h, hipStreamSynchronize(h->stream));
    poll_mass_check(h);
    if (h->nonfinite) return nonfinite_fail(h);
    return SIM_OK;
}

sim_status sim_destroy(sim_handle* h) {
    if (!h) return SIM_OK;
    hipError_t e = hipSuccess;
    if (h->stream) e = hipStreamSynchronize(h->stream);
    release(h);
    const bool bad = e != hipSuccess || h->poisoned;
    delete h;
    if (bad) return fail(nullptr, SIM_EDEVICE, "device error pending at destroy");
    return SIM_OK;
}

sim_status sim_release_memory(void) {
    const hipError_t e = release_device_memory();
    if (e != hipSuccess) return device_fail(nullptr, e, "sim_release_memory");
    return SIM_OK;
}

const char* sim_last_error(const sim_handle* h) {
    return h ? h->err.c_str() : g_create_error.c_str();
}

// ------------------------------------------------------------------------------------
// Trajectory-loss gradient (2D)
// ------------------------------------------------------------------------------------
namespace {

static int64_t cone_blocks(const sim_handle* h) { return adjoint_cone_blocks(std::max(h->n_cones, 1)); }

// Loss seed from the current (final) cone state: a_p = 2 w (p - t), a_theta = 0; the
// per-workgroup loss partials are left in adj->loss_partial.  At the run's end (`stop` given) also
// where the cones stopped.
static sim_status adjoint_seed(sim_handle* h, int32_t* stop = nullptr) {
    sim_status st = sync_cones(h);
    if (st != SIM_OK) return st;
    AdjointRun* a = h->adj;
    HIP_TRY(h, launch_adjoint_seed2d(h->cones, a->tip_target, a->weight, a->acone,
                                     a->loss_partial, stop, h->stream));
    return SIM_OK;
}

// Cone tape entries of a window of n_steps steps.
static size_t cone_tape_size(const sim_handle* h, int64_t n_steps) {
    return (size_t)(kConePlanes + 2 * h->n_species) * (size_t)n_steps *
           std::max<size_t>((size_t)h->n_cones, 1);
}
static ConeTape cone_tape_view(const sim_handle* h, float4* base, int64_t n_steps) {
    return ConeTape{base, (size_t)n_steps * (size_t)h->n_cones, h->n_cones};
}

// Bytes of every field state of a run of n_steps and of its cone steps; or of the field states and
// a float4 per cone step, which go towards a window of several segments' cone steps.
static size_t adjoint_field_bytes(const sim_handle* h, int64_t n_steps) {
    return (size_t)(n_steps + 1) * (size_t)h->n_species * (size_t)h->n_cells * 4;
}
static size_t adjoint_whole_bytes(const sim_handle* h, int64_t n_steps) {
    return adjoint_field_bytes(h, n_steps) + cone_tape_size(h, n_steps) * sizeof(float4);
}
static size_t adjoint_fields_alone_bytes(const sim_handle* h, int64_t n_steps) {
    return adjoint_field_bytes(h, n_steps) + (size_t)n_steps * (size_t)h->n_cones * sizeof(float4);
}

// The handle's tape limit (sim_adjoint_set_tape_limit), or half the free device memory.
static size_t adjoint_tape_limit(const sim_handle* h) {
    if (h->adj_tape_limit > 0) return (size_t)h->adj_tape_limit;
    size_t free_bytes = 0, total_bytes = 0;
    if (hipMemGetInfo(&free_bytes, &total_bytes) != hipSuccess) free_bytes = 0;
    return (free_bytes + device_idle_bytes(h->device)) / 2;
}

// Drops the handle's record when it goes out of scope: that of a run that failed on the way holds
// less than its length says.
struct RecordUndo {
    sim_handle* h;
    ~RecordUndo() {
        if (h) adjoint_release(h);
    }
};

// Ends the recording of a run's field states (both paths) when it goes out of scope.
struct RecordGuard {
    sim_handle* h = nullptr;
    ~RecordGuard() {
        if (!h) return;
        h->record = nullptr;
        if (h->block_steps > 1) tiled_set_record(h->tiled, nullptr, ConeTape{}, 0);
    }
};

}  // namespace

sim_status sim_adjoint_run(sim_handle* h, int64_t n_steps, int32_t checkpoint_every,
                           const int32_t* assign, const float* weight, double* loss) {
    if (!h) return fail(nullptr, SIM_EINVAL, "handle is NULL");
    if (h->poisoned) return fail(h, SIM_ESTATE, "handle poisoned by an earlier device error");
    if (h->dim != 2) return fail(h, SIM_EINVAL, "the trajectory-loss gradient is 2D only");
    if (h->rules.turn_law != SIM_TURN_VECTOR)
        return fail(h, SIM_EINVAL, "the trajectory-loss gradient needs the vector turn law");
    if (n_steps < 0 || checkpoint_every < 1)
        return fail(h, SIM_EINVAL, "n_steps < 0 or checkpoint_every < 1");
    if (h->step + n_steps > 2147483647LL)
        return fail(h, SIM_EINVAL, "step count would exceed 2^31-1");
    if (!loss) return fail(h, SIM_EINVAL, "loss is NULL");
    const int M = h->n_cones;
    const int T = h->n_targets;
    if (M > 0 && (!assign || !weight)) return fail(h, SIM_EINVAL, "assign or weight is NULL");
    std::vector<float> tips((size_t)2 * M);
    for (int i = 0; i < M; ++i) {
        if (assign[i] < 0 || assign[i] >= T)
            return fail(h, SIM_EINVAL, "assign[%d] = %d is not a target index", i, assign[i]);
        if (!std::isfinite(weight[i])) return fail(h, SIM_EINVAL, "weight[%d] not finite", i);
        tips[2 * i] = h->target_host[(size_t)assign[i] * 2];
        tips[2 * i + 1] = h->target_host[(size_t)assign[i] * 2 + 1];
    }
    sim_status st = follow_replays(h);
    if (st != SIM_OK) return st;
    adjoint_release(h);
    AdjointRun* a = new (std::nothrow) AdjointRun();
    if (!a) return fail(h, SIM_ENOMEM, "adjoint record");
    h->adj = a;
    RecordUndo undo{h};
    a->n0 = h->step;
    a->n_steps = n_steps;
    a->every = checkpoint_every;
    a->n_ckpt = (int)((n_steps + checkpoint_every - 1) / checkpoint_every);
    const size_t ns = (size_t)h->n_species, cells = (size_t)h->n_cells, Ms = (size_t)M;
    const size_t nck = (size_t)a->n_ckpt;
    hipError_t e;
    if ((e = dalloc(&a->ckpt_field, nck * ns * cells)) != hipSuccess ||
        (e = dalloc(&a->ckpt_pos, nck * Ms * 2)) != hipSuccess ||
        (e = dalloc(&a->ckpt_dir, nck * Ms)) != hipSuccess ||
        (e = dalloc(&a->ckpt_int, nck * 3 * Ms)) != hipSuccess ||
        (e = dalloc(&a->stop, 2 * Ms)) != hipSuccess ||
        (e = dalloc(&a->tip_target, Ms * 2)) != hipSuccess ||
        (e = dalloc(&a->weight, Ms)) != hipSuccess ||
        (e = dalloc(&a->acone, Ms * 3)) != hipSuccess ||
        (e = dalloc(&a->loss_partial, (size_t)cone_blocks(h))) != hipSuccess) {
        if (e == hipErrorOutOfMemory)
            return fail(h, SIM_ENOMEM, "adjoint checkpoints: out of device memory");
        return device_fail(h, e, "adjoint allocation");
    }
    if (M > 0) {
        HIP_TRY(h, hipMemcpyAsync(a->tip_target, tips.data(), Ms * 2 * 4, hipMemcpyHostToDevice,
                                  h->stream));
        HIP_TRY(h, hipMemcpyAsync(a->weight, weight, Ms * 4, hipMemcpyHostToDevice, h->stream));
    }
    // When the whole run's states fit the tape limit, record every field state and cone step
    // as the run goes, or the field states alone where the cone steps do not fit beside them;
    // what was not recorded, or whose tape cannot be had, the sweep re-runs from the checkpoints.
    RecordGuard recording;
    const size_t limit = a->n_ckpt > 1 ? adjoint_tape_limit(h) : 0;
    if (adjoint_fields_alone_bytes(h, n_steps) < limit) {
        if (adjoint_whole_bytes(h, n_steps) < limit &&
            dalloc(&a->cone_tape, cone_tape_size(h, n_steps)) != hipSuccess)
            (void)hipGetLastError();
        if ((!a->cone_tape && dalloc(&a->cone_unkept, std::max<size_t>(Ms, 1)) != hipSuccess) ||
            dalloc(&a->tape, (size_t)(n_steps + 1) * ns * cells) != hipSuccess) {
            (void)hipGetLastError();
            dfree(a->cone_tape);
        } else {
            for (size_t s = 0; s < ns; ++s)
                HIP_TRY(h, hipMemcpyAsync(a->tape + s * cells, h->field[s][h->cur[s]], cells * 4,
                                          hipMemcpyDeviceToDevice, h->stream));
            recording.h = h;
            h->record = a->tape;
            h->record_n0 = h->step;
            // (the recording kernels write every cone step's record: all of them into one, where
            // they are not kept, since a branch there costs 6% of such a launch)
            h->cone_record = a->cone_tape ? cone_tape_view(h, a->cone_tape, n_steps)
                                          : ConeTape{a->cone_unkept, 0, 0};
            if (h->block_steps > 1)
                tiled_set_record(h->tiled, a->tape, h->cone_record, (uint32_t)h->step);
        }
    }
    for (int j = 0; j < a->n_ckpt; ++j) {
        st = sync_cones(h);
        if (st != SIM_OK) return st;
        // the checkpoint: fields and cone arrays in one copy launch
        CopySpans cp = {};
        size_t words = 0;
        auto span = [&](const void* src, void* dst, size_t bytes) {
            cp.src[cp.n] = src;
            cp.dst[cp.n] = dst;
            words += bytes / 4;
            cp.word_end[cp.n++] = words;
        };
        for (size_t s = 0; s < ns; ++s)
            span(h->field[s][h->cur[s]], a->ckpt_field + ((size_t)j * ns + s) * cells, cells * 4);
        if (M > 0) {
            int32_t* ci = a->ckpt_int + (size_t)j * 3 * Ms;
            span(h->cones.pos, a->ckpt_pos + (size_t)j * Ms * 2, Ms * 8);
            span(h->cones.dir, a->ckpt_dir + (size_t)j * Ms, Ms * 4);
            span(h->cones.status, ci, Ms * 4);
            span(h->cones.target, ci + Ms, Ms * 4);
            span(h->cones.event_step, ci + 2 * Ms, Ms * 4);
        }
        HIP_TRY(h, launch_copy_spans(cp, h->stream));
        const int64_t len = std::min<int64_t>(checkpoint_every, n_steps - (int64_t)j * checkpoint_every);
        st = sim_step(h, len);
        if (st != SIM_OK) return st;
    }
    st = adjoint_seed(h, a->stop);
    if (st != SIM_OK) return st;
    std::vector<double> part((size_t)cone_blocks(h), 0.0);
    if (M > 0)
        HIP_TRY(h, hipMemcpyAsync(part.data(), a->loss_partial, part.size() * sizeof(double),
                                  hipMemcpyDeviceToHost, h->stream));
    HIP_TRY(h, hipStreamSynchronize(h->stream));
    double L = 0.0;
    for (double v : part) L += v;
    *loss = M > 0 ? L : 0.0;
    undo.h = nullptr;
    return SIM_OK;
}

sim_status sim_adjoint_backward(sim_handle* h, double* dL_dq, double* dL_dD, double* dL_dk) {
    if (!h) return fail(nullptr, SIM_EINVAL, "handle is NULL");
    if (h->poisoned) return fail(h, SIM_ESTATE, "handle poisoned by an earlier device error");
    AdjointRun* a = h->adj;
    if (!a) return fail(h, SIM_ESTATE, "no sim_adjoint_run to differentiate");
    if (h->step != a->n0 + a->n_steps)
        return fail(h, SIM_ESTATE, "the simulation was stepped after sim_adjoint_run");
    if (!dL_dq || !dL_dD || !dL_dk) return fail(h, SIM_EINVAL, "output pointer is NULL");
    const int ns = h->n_species, M = h->n_cones, nx = h->nx, ny = h->ny;
    const size_t cells = (size_t)h->n_cells, Ms = (size_t)M;
    const int K = (int)std::min<int64_t>(a->every, std::max<int64_t>(a->n_steps, 1));
    const int fb = reverse_tiles(nx, ny);   // accumulator slots per species
    int n_q[SIM_MAX_SPECIES] = {0, 0}, q_off[SIM_MAX_SPECIES] = {0, 0};
    for (int s = 0; s < ns; ++s) n_q[s] = (int)h->src_caller_cell[s].size();
    q_off[1] = n_q[0];
    const int nq_all = n_q[0] + (ns > 1 ? n_q[1] : 0);

    // Workspace.  One segment's per-step sample adjoints and the lists of the cones that touch
    // each tile, the field adjoint (ping-pong per species), FP64 accumulators and what the run did
    // not record of its field states and cone steps, for a window of segments: the whole run if
    // both fit the limit after all (re-run once, one thread per segment and cone for the cones),
    // else a segment after the other; with the field states recorded, as many segments' cone steps
    // as a float4 per cone step of the run holds, and one more.
    const int n_seg = a->n_ckpt;
    const int64_t n_run = a->n_steps;
    const bool fields_recorded = a->tape != nullptr, cones_recorded = a->cone_tape != nullptr;
    AdjointRun::Work& w = a->work;
    const bool fresh = !w.ready;   // first sweep of this record: allocate the workspace
    if (fresh) {
        constexpr int kMostSegs = 32768;   // of one re-run launch
        const bool fits = n_seg > 1 && adjoint_whole_bytes(h, n_run) < adjoint_tape_limit(h);
        w.whole = fields_recorded || fits;
        w.cone_segs = cones_recorded ? n_seg
                      : !w.whole     ? 1
                      : fits         ? std::min(n_seg, kMostSegs)
                                     : std::min(1 + n_seg / (kConePlanes + 2 * ns), kMostSegs);
    }
    const bool whole = w.whole;
    const int64_t window = whole ? n_run : K;   // steps: of the fields, and of the cones
    const int64_t cone_window =
        std::min<int64_t>(n_run, (int64_t)std::max(w.cone_segs, 1) * a->every);
    float*& tape_own = w.tape_own;
    float4*& tape_cones = w.tape_cones;
    uint32_t*& step_max = w.step_max;
    float*& afield = w.afield;
    double*& acc = w.acc;
    int32_t*& q_start = w.q_start;
    int2*& q_entry = w.q_entry;
    // on a device error the workspace is dropped (the next call allocates it again)
    auto free_all = [&]() {
        (void)hipStreamSynchronize(h->stream);
        adjoint_work_release(w);
    };
    std::vector<int32_t> q_start_h;
    std::vector<int2> q_entry_h;
    for (int s = 0; s < ns; ++s)
        reverse_sources(nx, ny, h->src_caller_cell[s], q_off[s], q_start_h, q_entry_h);
    const size_t launches = (size_t)reverse_launches(K);
    const double step_cells = h->rules.step_len * h->rules.inv_dx;
    const size_t list_cap = reverse_list_capacity(nx, ny, std::max(M, 1), step_cells);
    hipError_t e = hipSuccess;
    const size_t acc_n = (size_t)2 * ns * fb + (size_t)std::max(nq_all, 1);
    if (fresh &&
        ((!fields_recorded &&
          (e = dalloc(&tape_own, (size_t)(window + 1) * ns * cells)) != hipSuccess) ||
         (!cones_recorded &&
          (e = dalloc(&tape_cones, cone_tape_size(h, cone_window))) != hipSuccess) ||
        (e = dalloc(&w.ag, (size_t)2 * K * std::max<size_t>(Ms, 1))) != hipSuccess ||
        (e = dalloc(&step_max, (size_t)K)) != hipSuccess ||
        (e = dalloc(&w.boxes, launches * std::max<size_t>(Ms, 1))) != hipSuccess ||
        (e = dalloc(&w.list_end, launches * fb)) != hipSuccess ||
        (e = dalloc(&w.list, launches * list_cap)) != hipSuccess ||
        (e = dalloc(&afield, (size_t)2 * ns * cells)) != hipSuccess ||
        (e = dalloc(&acc, acc_n)) != hipSuccess ||
        (e = dalloc(&q_start, q_start_h.size())) != hipSuccess ||
        (e = dalloc(&q_entry, std::max<size_t>(q_entry_h.size(), 1))) != hipSuccess)) {
        free_all();
        if (e == hipErrorOutOfMemory)
            return fail(h, SIM_ENOMEM, "adjoint workspace: out of device memory");
        return device_fail(h, e, "adjoint workspace");
    }
#define ADJ_TRY(expr)                                                       \
    do {                                                                    \
        hipError_t e_ = (expr);                                             \
        if (e_ != hipSuccess) {                                             \
            free_all();                                                     \
            return device_fail(h, e_, #expr);                               \
        }                                                                   \
    } while (0)
    if (fresh) {
        ADJ_TRY(hipMemcpyAsync(q_start, q_start_h.data(), q_start_h.size() * 4,
                               hipMemcpyHostToDevice, h->stream));
        if (!q_entry_h.empty())
            ADJ_TRY(hipMemcpyAsync(q_entry, q_entry_h.data(), q_entry_h.size() * sizeof(int2),
                                   hipMemcpyHostToDevice, h->stream));
        w.ready = true;
    }
    ADJ_TRY(hipMemsetAsync(afield, 0, (size_t)2 * ns * cells * sizeof(float), h->stream));
    ADJ_TRY(hipMemsetAsync(acc, 0, acc_n * sizeof(double), h->stream));
    double* acc_D = acc;
    double* acc_k = acc + (size_t)ns * fb;
    double* acc_q = acc + (size_t)2 * ns * fb;
    sim_status st = adjoint_seed(h);   // final statuses now in h->cones (caller order)
    if (st != SIM_OK) {
        free_all();
        return st;
    }
    int64_t t_base = 0;   // run step whose field state is at the start of the field window
    float* const tape = fields_recorded ? a->tape : tape_own;
    auto field_at = [&](int64_t t, int s) {
        return tape + ((size_t)(t - t_base) * ns + s) * cells;
    };
    int cur = 0;
    auto afield_at = [&](int s, int half) { return afield + ((size_t)s * 2 + half) * cells; };
    const ConeTape tape_of_cones = cones_recorded ? cone_tape_view(h, a->cone_tape, n_run)
                                                  : cone_tape_view(h, tape_cones, cone_window);
    // re-run the fields of run steps [t0, t0 + len) from the checkpoint of segment j
    auto rerun_fields = [&](int j, int64_t t0, int64_t len) -> hipError_t {
        hipError_t r = hipMemcpyAsync(field_at(t0, 0), a->ckpt_field + (size_t)j * ns * cells,
                                      (size_t)ns * cells * 4, hipMemcpyDeviceToDevice,
                                      h->stream);
        // two steps per launch (every state is kept), the last one alone if odd
        int64_t t = t0;
        for (; t + 2 <= t0 + len && r == hipSuccess; t += 2) {
            const float* in[SIM_MAX_SPECIES] = {field_at(t, 0), field_at(t, ns - 1)};
            float* out1[SIM_MAX_SPECIES] = {field_at(t + 1, 0), field_at(t + 1, ns - 1)};
            float* out2[SIM_MAX_SPECIES] = {field_at(t + 2, 0), field_at(t + 2, ns - 1)};
            r = launch_field2d_pair(h->field2d, in, out1, out2, h->coef, h->stream);
        }
        if (t < t0 + len && r == hipSuccess) {
            const float* in[SIM_MAX_SPECIES] = {field_at(t, 0), field_at(t, ns - 1)};
            float* out[SIM_MAX_SPECIES] = {field_at(t + 1, 0), field_at(t + 1, ns - 1)};
            r = launch_field2d_rows(h->field2d, in, out, h->coef, h->stream);
        }
        return r;
    };
    // and the cone steps of segments c_lo .. j, which the cone window then holds
    int c_lo = cones_recorded ? 0 : n_seg;   // first segment in the window
    auto rerun_cones = [&](int j) -> hipError_t {
        c_lo = std::max(0, j - w.cone_segs + 1);
        const int64_t c0 = (int64_t)c_lo * a->every;
        return launch_cones_segments2d(h->rules, field_at(c0, 0), cells, ns, (int)c0, c_lo,
                                       j - c_lo + 1, a->every, (int)n_run, (uint32_t)a->n0,
                                       a->ckpt_pos, a->ckpt_dir, a->ckpt_int, M, tape_of_cones,
                                       h->stream);
    };
    if (whole && !fields_recorded) ADJ_TRY(rerun_fields(0, 0, n_run));
    // segment j, and the chain of its cones from its last step
    auto segment = [&](int j) {
        const int64_t t0 = (int64_t)j * a->every;
        ReverseSegment g = {};
        g.rules = h->rules;
        for (int s = 0; s < ns; ++s) g.coef[s] = h->coef[s];
        g.nx = nx;
        g.ny = ny;
        g.n_species = ns;
        g.M = M;
        g.len = (int)std::min<int64_t>(a->every, n_run - t0);
        g.seg0 = (uint32_t)(a->n0 + t0);
        g.fields = field_at(t0, 0);
        g.tape = tape_of_cones;
        g.tape.base += (size_t)(t0 - (int64_t)c_lo * a->every) * Ms;
        g.ag = w.ag + (size_t)(j & 1) * K * Ms;
        g.step_max = step_max;
        g.boxes = w.boxes;
        g.list_end = w.list_end;
        g.list = w.list;
        g.list_cap = list_cap;
        g.acc_D = acc_D;
        g.acc_k = acc_k;
        g.acc_q = acc_q;
        g.q_start = q_start;
        g.q_entry = q_entry;
        return g;
    };
    auto chain_of = [&](int j, const ReverseSegment& g) {
        ConeChain c = {};
        c.tape = g.tape;
        c.tape.M = M;
        c.seg0 = g.seg0;
        c.len = g.len;
        c.t_from = g.len - 1;
        c.ag = g.ag;
        c.boxes = g.boxes;
        c.start_status = a->ckpt_int + (size_t)j * 3 * Ms;
        c.status = h->cones.status;
        c.event_step = h->cones.event_step;
        c.run_status = a->stop;
        c.run_event = a->stop + Ms;
        c.acone = a->acone;
        return c;
    };
    // The cones' chain needs no field adjoint: that of a segment whose cone steps are there already
    // runs beside the field steps of the segment after it, kRevSteps steps per launch (a few CUs
    // for 55 us per 100 steps of 8192 cones otherwise).
    ConeChain next = {};
    next.t_from = -1;
    bool beside = false;   // the chain of segment j has begun
    for (int j = n_seg - 1; j >= 0; --j) {
        if (!whole) {
            t_base = (int64_t)j * a->every;
            ADJ_TRY(rerun_fields(j, t_base, std::min<int64_t>(a->every, n_run - t_base)));
        }
        if (j < c_lo) ADJ_TRY(rerun_cones(j));
        const ReverseSegment g = segment(j);
        if (!beside) next = chain_of(j, g);
        ADJ_TRY(launch_cone_chain2d(h->rules, next, h->stream));   // what is left of it
        ADJ_TRY(hipMemsetAsync(step_max, 0, (size_t)K * sizeof(uint32_t), h->stream));
        ADJ_TRY(launch_sample_max2d(g, h->stream));
        // the tiles the segment's cones touch, then the field steps
        ADJ_TRY(launch_reverse_lists(g, step_cells, h->stream));
        beside = j > c_lo && M > 0;
        if (beside) next = chain_of(j - 1, segment(j - 1));
        for (int l = 0; l < reverse_launches(g.len); ++l) {
            const float* in[SIM_MAX_SPECIES] = {afield_at(0, cur), afield_at(ns - 1, cur)};
            float* out[SIM_MAX_SPECIES] = {afield_at(0, cur ^ 1), afield_at(ns - 1, cur ^ 1)};
            const bool more = beside && next.t_from >= 0;
            ADJ_TRY(launch_field_reverse2d(g, l, in, out, more ? &next : nullptr, h->stream));
            if (more) next.t_from -= kRevSteps;
            cur ^= 1;
        }
    }
    std::vector<double> host(acc_n);
    ADJ_TRY(hipMemcpyAsync(host.data(), acc, acc_n * sizeof(double), hipMemcpyDeviceToHost,
                           h->stream));
    ADJ_TRY(hipStreamSynchronize(h->stream));
#undef ADJ_TRY
    const double dx2 = h->dx * h->dx;
    for (int s = 0; s < ns; ++s) {
        double sD = 0.0, sk = 0.0;
        for (int b = 0; b < fb; ++b) {
            sD += host[(size_t)s * fb + b];
            sk += host[(size_t)(ns + s) * fb + b];
        }
        dL_dD[s] = sD * h->dt / dx2;
        dL_dk[s] = -h->dt * sk;
    }
    for (int m = 0; m < nq_all; ++m) dL_dq[m] = host[(size_t)2 * ns * fb + m] / dx2;
    return SIM_OK;
}

sim_status sim_adjoint_set_tape_limit(sim_handle* h, int64_t max_bytes) {
    if (!h) return fail(nullptr, SIM_EINVAL, "handle is NULL");
    if (max_bytes < 0) return fail(h, SIM_EINVAL, "max_bytes < 0");
    h->adj_tape_limit = max_bytes;
    return SIM_OK;
}

// ------------------------------------------------------------------------------------
// Connectivity: adjacency list of the contacts and breadth-first levels
// ------------------------------------------------------------------------------------
sim_status sim_connectivity(sim_handle* h, int32_t n_neurons, const int32_t* cone_owner,
                            const int32_t* target_owner, int32_t* row_start, int32_t* edges,
                            int64_t edge_capacity, int64_t* n_edges) {
    sim_status st = connectivity_validate(h, n_neurons, cone_owner, target_owner, row_start,
                                          edges, edge_capacity, n_edges);
    if (st != SIM_OK) return st;
    const int M = h->n_cones, T = h->n_targets;
    graph_release(h);
    GraphBuffers& g = h->graph;
    const size_t Ms = (size_t)std::max(M, 1), N = (size_t)n_neurons;
    g.n_neurons = n_neurons;
    hipError_t e;
    if ((e = dalloc(&g.owner, Ms)) != hipSuccess ||
        (e = dalloc(&g.target_owner, (size_t)std::max(T, 1))) != hipSuccess ||
        (e = dalloc(&g.key, Ms)) != hipSuccess || (e = dalloc(&g.cone, Ms)) != hipSuccess ||
        (e = dalloc(&g.key_sorted, Ms)) != hipSuccess ||
        (e = dalloc(&g.cone_sorted, Ms)) != hipSuccess ||
        (e = dalloc(&g.degree, N)) != hipSuccess || (e = dalloc(&g.row_start, N + 1)) != hipSuccess ||
        (e = dalloc(&g.edges, Ms)) != hipSuccess || (e = dalloc(&g.level, N)) != hipSuccess ||
        (e = dalloc(&g.grew, 1)) != hipSuccess ||
        (e = device_malloc((void**)&g.scratch, sort_pairs_scratch_bytes(M))) != hipSuccess) {
        graph_release(h);
        if (e == hipErrorOutOfMemory) return fail(h, SIM_ENOMEM, "connectivity buffers");
        return device_fail(h, e, "connectivity allocation");
    }
    h->graph_cones = M;
    return connectivity_build(h, g, cone_owner, target_owner, row_start, edges, edge_capacity,
                              n_edges);
}

sim_status sim_bfs_levels(sim_handle* h, int32_t root, int32_t* level) {
    if (!h) return fail(nullptr, SIM_EINVAL, "handle is NULL");
    if (h->poisoned) return fail(h, SIM_ESTATE, "handle poisoned by an earlier device error");
    GraphBuffers& g = h->graph;
    if (!g.row_start) return fail(h, SIM_ESTATE, "no sim_connectivity graph to traverse");
    if (!level) return fail(h, SIM_EINVAL, "level is NULL");
    const int N = g.n_neurons;
    if (root < 0 || root >= N) return fail(h, SIM_EINVAL, "root %d out of range", root);
    const bool one_launch = bfs_in_one_launch(N, g.n_edges);
    HIP_TRY(h, one_launch ? launch_bfs(g, g.n_edges, root, h->stream)
                          : launch_bfs_init(g.level, N, root, h->stream));
    for (int depth = 0; depth < N && !one_launch; ++depth) {
        int32_t grew = 0;
        HIP_TRY(h, hipMemsetAsync(g.grew, 0, sizeof(int32_t), h->stream));
        HIP_TRY(h, launch_bfs_level(g.row_start, g.edges, N, depth, g.level, g.grew, h->stream));
        HIP_TRY(h, hipMemcpyAsync(&grew, g.grew, sizeof grew, hipMemcpyDeviceToHost, h->stream));
        HIP_TRY(h, hipStreamSynchronize(h->stream));
        if (!grew) break;
    }
    HIP_TRY(h, hipMemcpyAsync(level, g.level, (size_t)N * 4, hipMemcpyDeviceToHost, h->stream));
    HIP_TRY(h, hipStreamSynchronize(h->stream));
    return SIM_OK;
}

sim_status sim_batch_create(const sim_params* const* params, int32_t n, void* hip_stream,
                            int32_t graph_launches, sim_batch** out) {
    if (!out) return batch_fail(nullptr, SIM_EINVAL, "out is NULL");
    *out = nullptr;
    if (!params || n < 1) return batch_fail(nullptr, SIM_EINVAL, "need at least one simulation");
    if (graph_launches < 0 || graph_launches > 1024)
        return batch_fail(nullptr, SIM_EINVAL, "graph_launches must be in [0, 1024]");
    for (int i = 0; i < n; ++i) {
        if (!params[i]) return batch_fail(nullptr, SIM_EINVAL, "params[i] is NULL");
        if (params[i]->dim != 2) return batch_fail(nullptr, SIM_EINVAL, "batches are 2D only");
        if (params[i]->n_species != params[0]->n_species)
            return batch_fail(nullptr, SIM_EINVAL, "all simulations need the same n_species");
        if (params[i]->block_steps != params[0]->block_steps)
            return batch_fail(nullptr, SIM_EINVAL, "all simulations need the same block_steps");
        if (params[i]->tile_cols_per_lane != params[0]->tile_cols_per_lane)
            return batch_fail(nullptr, SIM_EINVAL,
                              "all simulations need the same tile_cols_per_lane");
    }
    if (params[0]->tile_cols_per_lane != 0 && params[0]->tile_cols_per_lane != 2 &&
        params[0]->tile_cols_per_lane != 4)
        return batch_fail(nullptr, SIM_EINVAL, "tile_cols_per_lane must be 0, 2 or 4");
    sim_batch* b = new (std::nothrow) sim_batch();
    if (!b) return batch_fail(nullptr, SIM_ENOMEM, "host allocation failed");
    auto bail = [&](sim_status st) {
        const std::string msg = b->err.empty() ? g_create_error : b->err;
        batch_release(b);
        delete b;
        g_create_error = msg;
        return st;
    };
    hipError_t e;
    if (hip_stream) {
        b->stream = (hipStream_t)hip_stream;
    } else {
        if ((e = hipStreamCreateWithFlags(&b->stream, hipStreamNonBlocking)) != hipSuccess)
            return bail(batch_fail(b, SIM_EDEVICE, "hipStreamCreate failed"));
        b->own_stream = true;
    }
    b->n_species = params[0]->n_species;
    int64_t total_cones = 0;
    for (int i = 0; i < n; ++i) {   // the shape is planned from checked parameters
        const sim_status st = validate(params[i]);
        if (st != SIM_OK) return bail(st);
    }
    BatchPlan shape;
    const int misfit = tiled_batch_plan(params, n, shape);
    if (misfit >= 0) {
        char m[160];
        snprintf(m, sizeof m, "simulation %d: no tiling that fits all members fits it", misfit);
        return bail(batch_fail(b, SIM_EINVAL, m));
    }
    b->cpl = shape.cpl;
    b->block_steps = shape.block_steps;
    for (int i = 0; i < n; ++i) {
        sim_params q = *params[i];
        q.block_steps = shape.block_steps;
        sim_handle* h = nullptr;
        sim_status st = create_impl(&q, b->stream, &shape.members[i], &h);
        if (st != SIM_OK) return bail(st);
        b->sims.push_back(h);
        b->lds_bytes = std::max(b->lds_bytes, h->plan.lds_bytes);
        b->n_base += h->plan.n_tiles;
        total_cones += h->n_cones;
    }
    if (total_cones > INT32_MAX / 2)
        return bail(batch_fail(b, SIM_EINVAL, "too many cones in the batch"));
    b->extra_cap = tiled_extra_capacity(total_cones);
    // concatenated argument tables, tiles, shared launch state
    const size_t entry = tiled_table_entry_bytes();
    std::vector<int2> items;
    items.reserve(b->n_base);
    for (int i = 0; i < n; ++i)
        for (int t = 0; t < b->sims[i]->plan.n_tiles; ++t) items.push_back(make_int2(i, t));
    // largest simulations first, so the persistent grid finishes with small work items
    std::stable_sort(items.begin(), items.end(), [&](const int2& x, const int2& y) {
        return b->sims[x.x]->plan.height * b->sims[x.x]->n_cones >
               b->sims[y.x]->plan.height * b->sims[y.x]->n_cones;
    });
    if ((e = device_malloc(&b->table, entry * n)) != hipSuccess ||
        (e = device_malloc((void**)&b->base, sizeof(int2) * items.size())) != hipSuccess ||
        (e = device_malloc((void**)&b->extra, sizeof(int4) * 2 * kBatchPartLists * b->extra_cap)) !=
            hipSuccess ||
        (e = device_malloc((void**)&b->launch, sizeof(LaunchState))) != hipSuccess)
        return bail(batch_fail(b, SIM_ENOMEM, "batch allocation failed"));
    for (int i = 0; i < n; ++i)
        if ((e = hipMemcpy((char*)b->table + entry * i, b->sims[i]->tiled.args, entry,
                           hipMemcpyHostToDevice)) != hipSuccess)
            return bail(batch_fail(b, SIM_EDEVICE, "table upload failed"));
    if ((e = hipMemcpy(b->base, items.data(), sizeof(int2) * items.size(),
                       hipMemcpyHostToDevice)) != hipSuccess)
        return bail(batch_fail(b, SIM_EDEVICE, "item upload failed"));
    const LaunchState ls = {};
    if ((e = hipMemcpy(b->launch, &ls, sizeof ls, hipMemcpyHostToDevice)) != hipSuccess)
        return bail(batch_fail(b, SIM_EDEVICE, "launch state upload failed"));
    if ((e = tiled_prepare_batch(b->n_species, b->cpl, b->lds_bytes)) != hipSuccess)
        return bail(batch_fail(b, SIM_EDEVICE, "kernel attribute failed"));
    // initial bucketing of every simulation's cones
    for (int i = 0; i < n; ++i) {
        sim_handle* h = b->sims[i];
        if ((e = tiled_bucket_batch(h->plan, h->tiled, h->cones, i, b->launch, b->extra,
                                    b->extra_cap, b->stream)) != hipSuccess)
            return bail(batch_fail(b, SIM_EDEVICE, "bucketing failed"));
        h->cones_bucketed = true;
    }
    // optional graph of `graph_launches` full-depth launches, replayed by sim_batch_step
    if (graph_launches > 0) {
        if ((e = hipStreamBeginCapture(b->stream, hipStreamCaptureModeThreadLocal)) != hipSuccess)
            return bail(batch_fail(b, SIM_EDEVICE, "graph capture failed to start"));
        for (int l = 0; l < graph_launches; ++l) {
            e = tiled_launch_batch((const TiledArgs2D*)b->table, b->extra, b->base,
                                   b->n_base, b->extra_cap, b->n_species, b->cpl,
                                   b->lds_bytes, b->block_steps, b->launch, b->stream);
            if (e != hipSuccess) break;
        }
        hipGraph_t g = nullptr;
        const hipError_t e2 = hipStreamEndCapture(b->stream, &g);
        if (e != hipSuccess || e2 != hipSuccess)
            return bail(batch_fail(b, SIM_EDEVICE, "graph capture failed"));
        b->graph = g;
        if ((e = hipGraphInstantiate(&b->graph_exec, g, nullptr, nullptr, 0)) != hipSuccess)
            return bail(batch_fail(b, SIM_EDEVICE, "graph instantiation failed"));
        b->graph_launches = graph_launches;
    }
    if ((e = hipStreamSynchronize(b->stream)) != hipSuccess)
        return bail(batch_fail(b, SIM_EDEVICE, "create synchronisation failed"));
    *out = b;
    return SIM_OK;
}

sim_status sim_batch_step(sim_batch* b, int64_t n_steps) {
    if (!b) return batch_fail(nullptr, SIM_EINVAL, "batch is NULL");
    if (n_steps < 0) return batch_fail(b, SIM_EINVAL, "n_steps < 0");
    if (b->step + n_steps > 2147483647LL)
        return batch_fail(b, SIM_EINVAL, "step count would exceed 2^31-1");
    for (sim_handle* h : b->sims)
        if (h->poisoned) return batch_fail(b, SIM_ESTATE, "a simulation hit a device error");
    const int64_t per_graph = (int64_t)b->graph_launches * b->block_steps;
    while (per_graph > 0 && n_steps >= per_graph) {
        BATCH_TRY(b, hipGraphLaunch(b->graph_exec, b->stream));
        batch_advance(b, b->block_steps, b->graph_launches);
        n_steps -= per_graph;
    }
    while (n_steps > 0) {
        const int steps = (int)std::min<int64_t>(n_steps, b->block_steps);
        sim_status st = batch_launch(b, steps);
        if (st != SIM_OK) return st;
        batch_advance(b, steps, 1);
        n_steps -= steps;
    }
    return SIM_OK;
}

sim_status sim_batch_read_state(sim_batch* b, int32_t sim, sim_item what, int32_t index,
                                void* dst, size_t dst_bytes, size_t* bytes_written) {
    if (!b) return batch_fail(nullptr, SIM_EINVAL, "batch is NULL");
    if (sim < 0 || sim >= (int32_t)b->sims.size())
        return batch_fail(b, SIM_EINVAL, "simulation index out of range");
    sim_handle* h = b->sims[sim];
    const sim_status st = sim_read_state(h, what, index, dst, dst_bytes, bytes_written);
    if (st != SIM_OK) b->err = h->err;
    return st;
}

sim_status sim_batch_synchronize(sim_batch* b) {
    if (!b) return batch_fail(nullptr, SIM_EINVAL, "batch is NULL");
    BATCH_TRY(b, hipStreamSynchronize(b->stream));
    return SIM_OK;
}

sim_status sim_batch_destroy(sim_batch* b) {
    if (!b) return SIM_OK;
    hipError_t e = hipSuccess;
    if (b->stream) e = hipStreamSynchronize(b->stream);
    batch_release(b);
    delete b;
    if (e != hipSuccess) return batch_fail(nullptr, SIM_EDEVICE, "device error pending at destroy");
    return SIM_OK;
}

const char* sim_batch_last_error(const sim_batch* b) {
    return b ? b->err.c_str() : g_create_error.c_str();
}

}  // extern "C"
