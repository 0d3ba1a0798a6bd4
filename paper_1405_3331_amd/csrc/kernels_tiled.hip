// kernels_tiled.hip -- temporally blocked, LDS-tiled step kernel for 2D grids.
//
// One launch advances B steps.  Each workgroup owns one tile: a core of TX x TY cells plus
// a halo of H cells on every side, loaded once from HBM into LDS.  Each sub-step updates
// the whole tile in LDS (the valid region shrinks by one cell per sub-step), adds the
// sources that fall in the tile, and then steps the growth cones bucketed to the tile
// against the just-updated LDS field -- the field update precedes the cone step within a
// step, as in the paper's time step.  After B sub-steps the core is written back and every
// surviving cone is appended to the bucket of the tile that now holds its tip.
//
// Halo: a cone bucketed to the core at block start is at most ceil((B-1) s / dx) cells away
// from the core before its last sub-step and samples cells up to 2 away from its own cell,
// while the valid region after sub-step b is the core grown by H - b; so
// H = B + ceil((B-1) s / dx) + 2 keeps every sample inside valid cells.  H is rounded up to
// a multiple of the per-lane segment width so that segments stay aligned to the grid.
//
// Layout of a tile row in LDS: one wavefront spans the loaded width W = 64 * CPL, lane l
// owning columns CPL*l .. CPL*l + CPL-1.  The wavefronts of a workgroup own
// consecutive strips of rows and update them in place or into a
// second copy of the tile (see strip_update).
//
// HBM traffic per launch: the tile with its halo is read once and the core written once,
// instead of B reads and B writes of every cell.
#include <hip/hip_ext.h>

#include "memory.hpp"
#include "rows.hpp"
#include "tiled.hpp"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstddef>
#include <cstring>
#include <map>
#include <new>
#include <vector>

namespace cuesim {

namespace {

// How a workgroup steps its tile (TileShape of a plan):
//   kPair      8 wavefronts, one copy of the tile, two workgroups to a CU;
//   kTwoPair   the same with two copies;
//   kTwo       12 wavefronts, two copies, a CU's LDS to itself;
//   kWide      16 wavefronts, one copy, a CU's LDS to itself.
// With two copies of the tile a sub-step goes from one to the other, so that neither the strips'
// edge rows nor the cones' reads of the field have to be kept apart from the next sub-step's
// writes: one barrier per sub-step instead of three.  It is used where all tiles still start at
// once.  Per step, over 6400 steps: 777 x 389, two species 3.05 -> 2.72 us, 1000 x 600 2.42 ->
// 2.12, 1024^2 2.51 -> 2.10, 1500 x 1100 with 30,000 cones 3.31 -> 2.76; 128 x 128 1.66 -> 1.55.
// Twelve wavefronts against eight in kTwo: 1024^2 2.04 -> 1.99, 1500 x 1100 2.57 -> 2.48 (sixteen:
// 2.08, 2.55); where two workgroups share a CU eight are better (128 x 128 1.56 against 1.63).  A
// second cone per thread in kTwo, so that crowded tiles need fewer parts, costs every tile:
// 1024^2 2.17.
// kWide: on the largest grids a tile twice as wide spends less on its halo: 2048^2 with 65,536
// cones, 10,000 steps after 200: depth 14, 138 rows of 256 columns 3.98 us per step, two tiles of
// 143 rows of 128 columns per CU, depth 12, 4.46 (the first 1000: 3.82 and 3.87; 143 rows of 256
// columns stepped by 8 wavefronts 4.8).  Short tiles lose by it (777 x 389, two species, 56
// rows: 5.0 against 4.2 us).  Past one round of tiles it still gains (over steps 48 to 624; the
// best of 128 columns, of heights up to 296 and of 143 at depth 12): 3000^2 6.3 us against 7.1,
// 4096^2 10.0 against 11.0, 6000 x 5000 18.4 against 18.5; at 8192^2 it no longer does (40.8, 37.8).
constexpr int kWideRows = 96;
constexpr size_t kCuLds = 160 * 1024;
constexpr int kMaxTileTargets = 256;        // targets staged in LDS per tile
constexpr size_t kLdsBudget = 154 * 1024;   // dynamic LDS; the rest is static (targets,
                                            // re-bucketing counters)
constexpr int kLoadBatch = 10;              // tile rows a wavefront has in flight at load
constexpr int kConeSlots = 1;               // cones per thread held in registers: a second
                                            // one costs every tile (above).  Without the loops
                                            // over them the kernels are allotted other registers:
                                            // 128 x 128 2.6% faster, 777 x 389 with two species 1
                                            // to 2% slower
constexpr int kPartCones = 512;             // cones that a part steps (kWide: twice as many)
constexpr size_t kStaticLds = kMaxTileTargets * 16 + 3 * 9 * 4 + 16;   // static LDS per tile
constexpr int kSmallest = 192;              // and when a tile's cones are split furthest
constexpr int kHeadItems = 64;              // sources and targets of a tile kept at a fixed
                                            // stride, found from the tile number alone
constexpr int kSpecCones = 128;             // cone slots read before the tile's count is known
constexpr int kGuardRows = 4;               // one above and three below each species plane
constexpr int kXcds = 8;                    // dies (XCDs); workgroup b of a launch runs on die
                                            // b % kXcds

// Wavefronts and copies of the tile of each shape, and cones per part in units of kPartCones (in
// kTwo the wavefronts past the eighth hold none and take more rows).
constexpr int waves_of(int shape) { return shape == kWide ? 16 : shape == kTwo ? 12 : 8; }
constexpr bool two_copies(int shape) { return shape == kTwoPair || shape == kTwo; }
constexpr int part_units(int shape) { return shape == kWide ? 2 : 1; }

}  // namespace

// Static description of one simulation for the tiled kernel (device-resident table entry).
// Everything that changes from launch to launch lives in LaunchState.
struct TiledArgs2D {
    float* field[SIM_MAX_SPECIES][2];   // [species][ping-pong buffer]
    StencilCoef coef[SIM_MAX_SPECIES];
    int nx, ny;
    int tiles_x, n_tiles;
    int tx_core, ty_core, halo, height;   // TX, TY, H, loaded height HL
    const int4* head;          // per tile: first target, targets, first source, sources
    const int2* src_entry;     // (LDS index within the species plane, species)
    const float* src_amount;
    const float4* tgt_pts;     // targets within reach of the tile's cones this launch
    const int2* head_src;      // per tile, kHeadItems each: the first sources, (LDS index |
                               // species << 24, amount bits), and the first targets
    const float4* head_tgt;
    float4* bucket[2];         // per tile: cone slots (x, y, theta, id); the launch reads one
                               // half and fills the other
    int32_t* count[3];         // cones per tile: this launch's input, its output, and last
                               // launch's input, zeroed for the next launch's output
    int capacity;
    int cone_rows;             // stencil rows a wavefront gives up per cone slot it steps
    ConeArrays cones;
    ConeRules rules;
    float* record;             // non-null: every sub-step's field also goes to
                               // record + ((step - record_n0) * NS + s) * cells (a tape of
                               // every state of a run, for the trajectory-loss gradient)
    ConeTape cone_record;      // and what the reverse needs of every cone step
    uint32_t record_n0;
};

namespace {

// Load a tile plane (HL rows from grid row y0) into LDS rows 0 .. HL-1 at `dst`, the rows
// strided over the wavefronts, kLoadBatch rows in flight per wavefront: the batch's loads
// are all issued before the first is used.  A batch running past the tile re-reads its last
// row and parks the copy in guard row HL, which is never meaningful.  Cells outside the grid
// read as zero; cells inside never use them (they take their own value for out-of-grid
// neighbours).
// issued() runs once the first batch's loads are on their way (before the wait for them).
template <int CPL, int WAVES, bool ALIGNED, class Issued>
__device__ __forceinline__ void load_tile(float* dst, GlobalPtr<const float> f, int nx, int ny,
                                          int y0, int HL, int gx0, int cx, int wave,
                                          const bool (&col_in)[CPL], const Issued& issued) {
    using V = typename Row<CPL>::T;
    constexpr int W = 64 * CPL;
    for (int ly0 = wave; ly0 < HL; ly0 += kLoadBatch * WAVES) {
        RowVec<CPL> v[kLoadBatch];
#pragma unroll
        for (int r = 0; r < kLoadBatch; ++r)
            v[r] = load_row<CPL, ALIGNED>(f, nx, ny, y0 + min(ly0 + r * WAVES, HL - 1), gx0);
        if (ly0 == wave) issued();
#pragma unroll
        for (int r = 0; r < kLoadBatch; ++r) {
            const int ly = min(ly0 + r * WAVES, HL);
            const bool row_in = (unsigned)(y0 + ly) < (unsigned)ny;
            V out;
#pragma unroll
            for (int k = 0; k < CPL; ++k) set_comp(out, k, row_in && col_in[k] ? v[r][k] : 0.0f);
            *(V*)&dst[ly * W + cx] = out;
        }
    }
}

// LDS view of one species: a tile of width x height cells whose first is cell (x0, y0).
struct LdsField2D {
    const float* L;
    int x0, y0, width, height;
};

// One stencil + decay sub-step of one species over a wavefront's strip of rows
// [ybeg, yend), into `to`: L itself (in place) or the other copy.  L points at tile row 0; rows
// -1 and HL .. HL+2 are guard rows (never meaningful) so reads, which reach at most two rows
// past the strip, need no clamping.  In place, every LDS read of a row is issued within a
// wavefront before that row's write, so interior rows are overwritten as soon as they are
// computed; the strip's first and last rows are read by the neighbouring wavefronts and are
// returned for writing after a barrier.  Four row registers cycle through their roles (above / at / below /
// prefetched), so rows are prefetched two ahead with no register moves: a prefetched row
// is either this strip's, still unmodified, or a neighbour's first row, written only after
// the barrier (or is never used).  The first and last rows are peeled off, so the loop body
// has no branches and the LDS wait counter can let prefetches stay in flight.  A strip
// never reaches outside the grid's rows; `top` (`bottom`) says that its first (last) row is
// the grid's first (last), whose missing neighbour is the row itself.
template <int CPL>
struct StripEdges {
    typename Row<CPL>::T first, last;
};

template <int CPL, int COLS>
__device__ __forceinline__ StripEdges<CPL> strip_update(const float* L, float* to, int ybeg,
                                                        int yend, int cx, int gx0, int nx,
                                                        bool top, bool bottom, StencilCoef cf) {
    using V = typename Row<CPL>::T;
    constexpr int W = 64 * CPL;
    const float* rd = L + cx;
    float* wr = to + cx;
    auto load = [&](int yy) { return *(const V*)&rd[yy * W]; };
    auto store = [&](int yy, const V& v) { *(V*)&wr[yy * W] = v; };
    auto upd = [&](const V& s, const V& c, const V& n, int) {
        return row_update<CPL, COLS>(s, c, n, gx0, nx, cf);
    };
    StripEdges<CPL> out;
    V A = load(ybeg - 1), Bv = load(ybeg), C = load(ybeg + 1), D = load(ybeg + 2);
    // the strip's first row (returned, written after the barrier)
    if (yend - ybeg == 1) {
        out.first = upd(top ? Bv : A, Bv, bottom ? Bv : C, ybeg);
        out.last = out.first;
        return out;
    }
    out.first = upd(top ? Bv : A, Bv, C, ybeg);
    A = load(ybeg + 3);
    // interior rows [ybeg + 1, yend - 1), written in place: a branch-free body of four rows,
    // the registers (Bv, C, D, A) holding rows y - 1 .. y + 2 at its top
    int y = ybeg + 1;
    const int yin = yend - 1;
    for (; y + 4 <= yin; y += 4) {
        V nv = upd(Bv, C, D, y);
        Bv = load(y + 3);
        store(y, nv);
        nv = upd(C, D, A, y + 1);
        C = load(y + 4);
        store(y + 1, nv);
        nv = upd(D, A, Bv, y + 2);
        D = load(y + 5);
        store(y + 2, nv);
        nv = upd(A, Bv, C, y + 3);
        A = load(y + 6);
        store(y + 3, nv);
    }
    // 0..3 remaining interior rows, then the last row (returned)
    const int r = yin - y;
    if (r == 0) {
        out.last = upd(Bv, C, bottom ? C : D, y);
    } else if (r == 1) {
        store(y, upd(Bv, C, D, y));
        out.last = upd(C, D, bottom ? D : A, y + 1);
    } else if (r == 2) {
        const V v0 = upd(Bv, C, D, y);
        Bv = load(y + 3);
        store(y, v0);
        store(y + 1, upd(C, D, A, y + 1));
        out.last = upd(D, A, bottom ? A : Bv, y + 2);
    } else {
        const V v0 = upd(Bv, C, D, y);
        Bv = load(y + 3);
        store(y, v0);
        const V v1 = upd(C, D, A, y + 1);
        C = load(y + 4);
        store(y + 1, v1);
        store(y + 2, upd(D, A, Bv, y + 2));
        out.last = upd(A, Bv, bottom ? Bv : C, y + 3);
    }
    return out;
}

// Contact test against the targets staged for this tile (a superset of every target within
// the contact radius of any tip the tile's cones can reach in this launch), or against the
// whole grid when the tile's list did not fit in LDS.
struct TileContact {
    const float4* pts;
    int n;
    bool staged;
    const TargetGrid* grid;
    template <int dim>
    __device__ int find(float x, float y, float z) const {
        return staged ? contact_in_list<dim>(pts, n, grid->r2, x, y, z)
                      : contact_target<dim>(*grid, x, y, z);
    }
};

// The gradient footprint of a tip read from the LDS tile.  Its 12 cells lie between one
// cell before and two after the corner cell (i0, j0) along each axis, so one base address
// and constant offsets reach them all; at a grid wall the outer cell is the wall cell itself
// (the zero-flux ghost), substituted afterwards.  The base is clamped so that every read
// stays inside the tile: a tip bucketed to the tile never needs the clamp (the halo covers
// its footprint), and with it no tip can read outside the tile.
__device__ __forceinline__ Footprint2D footprint_lds(const LdsField2D& f, const ConeRules& r,
                                                    float x, float y) {
    Footprint2D p;
    corner(x, r.inv_dx, r.nx, p.i0, p.fx);
    corner(y, r.inv_dx, r.ny, p.j0, p.fy);
    p.im = max(p.i0 - 1, 0);
    p.ip = min(p.i0 + 2, r.nx - 1);
    p.jm = max(p.j0 - 1, 0);
    p.jp = min(p.j0 + 2, r.ny - 1);
    const int W = f.width;
    const int lx = min(max(p.i0 - f.x0, 1), W - 3);
    const int ly = min(max(p.j0 - f.y0, 1), f.height - 3);
    const float* b = f.L + ly * W + lx;
    p.a0 = b[-1];
    p.a1 = b[0];
    p.a2 = b[1];
    p.a3 = b[2];
    p.b0 = b[W - 1];
    p.b1 = b[W];
    p.b2 = b[W + 1];
    p.b3 = b[W + 2];
    p.c0 = b[-W];
    p.c1 = b[1 - W];
    p.d0 = b[2 * W];
    p.d1 = b[2 * W + 1];
    if (p.im == p.i0) {   // left wall
        p.a0 = p.a1;
        p.b0 = p.b1;
    }
    if (p.ip == p.i0 + 1) {   // right wall
        p.a3 = p.a2;
        p.b3 = p.b2;
    }
    if (p.jm == p.j0) {   // bottom wall
        p.c0 = p.a1;
        p.c1 = p.a2;
    }
    if (p.jp == p.j0 + 1) {   // top wall
        p.d0 = p.b1;
        p.d1 = p.b2;
    }
    return p;
}

// The cone step in two parts.  The first samples the signed gradient g at the tip from the
// LDS field (the only part that reads the field); the second turns, adds noise, advances
// and tests exit and contact using g and registers only, so it may run while the next
// sub-step already overwrites the field.
// The sample is (g_x, g_y, concentration of species 0; the last only under the SNR law).
// RECORD: the sample's part of the cone's record goes to the run's cone tape (step t of it).
template <int NS, bool RECORD>
__device__ __forceinline__ float3 tile_cone_gradient(const float4& st, const LdsField2D& f0,
                                                     const LdsField2D& f1,
                                                     const ConeRules& rules,
                                                     const ConeTape& tape, size_t t) {
    float gxv = 0.0f, gyv = 0.0f, conc = 0.0f;
    const int id = __float_as_int(st.w);
    if (id < 0) return make_float3(gxv, gyv, conc);
    const Footprint2D p0 = footprint_lds(f0, rules, st.x, st.y);
    const CornerGradients2D g0 = corner_gradients_2d(p0, rules);
    if (RECORD) tape.sample(0, t, id, g0);
    gradient_from_2d(p0, g0, gxv, gyv, rules.turn_law == 1 ? &conc : nullptr);
    gxv *= rules.sign0;
    gyv *= rules.sign0;
    if (NS > 1) {
        float hx, hy;
        const Footprint2D p1 = footprint_lds(f1, rules, st.x, st.y);
        const CornerGradients2D g1 = corner_gradients_2d(p1, rules);
        if (RECORD) tape.sample(1, t, id, g1);
        gradient_from_2d(p1, g1, hx, hy, nullptr);
        gxv = fmaf(rules.sign1, hx, gxv);
        gyv = fmaf(rules.sign1, hy, gyv);
    }
    if (RECORD) tape.put(2, t, id, make_float4(gxv, gyv, p0.fx, p0.fy));
    return make_float3(gxv, gyv, conc);
}

// Second part; a stopped cone has its final state written to the caller-order arrays and
// the sign bit of its id set.  One Philox block serves an even step and the next odd one:
// the odd step's two words wait in `spare` (`fresh`: no even step of this launch has
// filled them yet).
template <bool RECORD>
__device__ __forceinline__ void tile_cone_advance(float4& st, float2& sc, uint2& spare,
                                                  float3 g, const ConeRules& rules,
                                                  uint32_t step, bool fresh,
                                                  const TileContact& contact,
                                                  const ConeArrays& cones,
                                                  const ConeTape& tape, size_t t) {
    int id = __float_as_int(st.w);
    if (id < 0) return;
    float z[2];
    if ((step & 1u) == 0u || fresh) {
        const uint4 blk = noise_block_2d(rules.key, (uint32_t)id, step);
        if (step & 1u) {
            normal_pair(blk.z, blk.w, z);
        } else {
            normal_pair(blk.x, blk.y, z);
            spare = make_uint2(blk.z, blk.w);
        }
    } else {
        normal_pair(spare.x, spare.y, z);
    }
    float x = st.x, y = st.y, th = st.z;
    const float2 before = sc;
    const ConeEvent ev =
        cone_step_2d(rules, g.x, g.y, g.z, z, x, y, th, sc.x, sc.y, contact);
    if (RECORD)
        record_turn(tape, t, id, rules, st.x, st.y, before.x, before.y, g.x, g.y, sc.x, sc.y);
    if (ev.status != kActive) {
        cones.pos[2 * id] = x;
        cones.pos[2 * id + 1] = y;
        cones.dir[id] = th;
        cones.status[id] = ev.status;
        cones.target[id] = ev.target;
        cones.event_step[id] = (int32_t)(step + 1);
        id = (int)((unsigned)id | 0x80000000u);
    }
    st = make_float4(x, y, th, __int_as_float(id));
}

// Cell of a coordinate, clamped to the grid (as a float first: a NaN tip maps to cell 0).
__device__ __forceinline__ int cell_of(float p, float inv_dx, int n) {
    return (int)fminf(fmaxf(floorf(p * inv_dx), 0.0f), (float)(n - 1));
}

// Destination tile of a cone's tip after a launch, restricted to the 3x3 neighbourhood of
// the tile it was stepped in (the halo guarantees it never moves further).
__device__ __forceinline__ int2 next_tile(const float4& st, int tx, int ty, int tiles_x,
                                          int tiles_y, float inv_dx, int nx, int ny,
                                          int tx_core, int ty_core) {
    int ntx = cell_of(st.x, inv_dx, nx) / tx_core;
    int nty = cell_of(st.y, inv_dx, ny) / ty_core;
    ntx = min(max(ntx, max(tx - 1, 0)), min(tx + 1, tiles_x - 1));
    nty = min(max(nty, max(ty - 1, 0)), min(ty + 1, tiles_y - 1));
    return make_int2(ntx, nty);
}

// The core of a tile from LDS to the fields dst[s] (row-major, the grid's row length),
// through global-address-space stores.  The tile's rows are strided over the wavefronts.
// STREAM: non-temporal stores, for the run tape, which is read only by a later reverse sweep
// (the recording forward run of a 1024^2 gradient: 8.1 against 8.4 ms).
template <int NS, int CPL, int WAVES, bool STREAM = false>
__device__ __forceinline__ void store_core(float* const dst[], const float* from,
                                           const TiledArgs2D& a, int tx, int ty, int plane,
                                           int cx, int wave, bool aligned) {
    using V = typename Row<CPL>::T;
    constexpr int W = 64 * CPL;
    const int H = a.halo;
    const int cx0 = tx * a.tx_core, cy0 = ty * a.ty_core;
    for (int ly = wave; ly < a.ty_core; ly += WAVES) {
        const int gy = cy0 + ly;
        if (gy >= a.ny) break;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const V v = *(const V*)&from[s * plane + (ly + H + 1) * W + cx];
            const GlobalPtr<float> row = gbl(dst[s]) + (size_t)gy * a.nx + cx0;
            if (aligned) {
                const int lx = cx - H;   // the segment is wholly inside or outside the core
                if (lx >= 0 && lx < a.tx_core && cx0 + lx < a.nx) {
                    RowVec<CPL> x;
#pragma unroll
                    for (int k = 0; k < CPL; ++k) x[k] = comp(v, k);
                    if (STREAM)
                        __builtin_nontemporal_store(x, (GlobalPtr<RowVec<CPL>>)(row + lx));
                    else
                        *(GlobalPtr<RowVec<CPL>>)(row + lx) = x;
                }
                continue;
            }
#pragma unroll
            for (int k = 0; k < CPL; ++k) {
                const int lx = cx + k - H;   // core column of this lane's k-th cell
                if (lx >= 0 && lx < a.tx_core && cx0 + lx < a.nx) {
                    if (STREAM)
                        __builtin_nontemporal_store(comp(v, k), row + lx);
                    else
                        row[lx] = comp(v, k);
                }
            }
        }
    }
}

// Candidate part sizes of a crowded tile, largest first: the parts that a launch steps it in
// take at most this many times `units` cones each.  A persistent launch, whose queue balances
// itself, uses the first only.
static_assert(kPartCones == 512, "candidate part sizes assume 512-cone parts");
__device__ __forceinline__ int tile_parts(int c, int p) { return max(1, (c + p - 1) / p); }
// Parts of a tile of c cones under candidate j (constant divisors: no integer division).
__device__ __forceinline__ int candidate_parts(int c, int j, int units) {
    if (units == 2) c = (c + 1) / 2;   // ceil(ceil(c / u) / p) == ceil(c / (u p))
    switch (j) {
        case 1: return tile_parts(c, 384);
        case 2: return tile_parts(c, 320);
        case 3: return tile_parts(c, 256);
        case 4: return tile_parts(c, 192);
        default: return tile_parts(c, kPartCones);
    }
}
static_assert(kSmallest == 192, "the smallest candidate");

// Where the cones put into the next launch's buckets list the further parts of the tiles
// they crowd.
struct PartLists {
    LaunchState* ls;
    int4* list;   // the next launch's lists, one per candidate size, `cap` entries each
    int cap;
    int phase;    // of the next launch
    int sizes;    // candidates in use
    int sim;
    int units;    // of a part's size
};

// A tile's count has gone from `before` to `now` cones by one atomic addition: every part
// that these cones opened goes to the candidates' lists.  Additions to one count follow one
// another, so each part is listed once, whatever their order; a part's cones are decided
// from the final count by the launch that steps them.  A list longer than `cap` is not used
// (kPartSizes: the full-part list always fits).
__device__ __forceinline__ void list_parts(const PartLists& to, int tile, int before, int now) {
    if (now <= kSmallest) return;
    for (int j = 0; j < to.sizes; ++j) {
        const int a = candidate_parts(before, j, to.units);
        const int b = candidate_parts(now, j, to.units);
        if (b <= a) continue;
        const int at = atomicAdd(&to.ls->extra_n[to.phase][j], b - a);
        for (int q = a; q < b; ++q)
            if (at + q - a < to.cap)
                to.list[j * to.cap + at + q - a] = make_int4(to.sim, tile, q, 0);
    }
}

// A workgroup's place in the launch: which tile and part it steps, and the launch's state as
// every workgroup read it.
struct TileWork {
    int tile, part, chosen;   // chosen: candidate part size in use
    int steps;
    uint32_t first_step;
    int par, phase;
};

// Advance the launch state for the next launch: by the last workgroup to have read it.
__device__ __forceinline__ void advance_launch(LaunchState* ls, uint32_t next_step, int par,
                                               int phase) {
    ls->step = next_step;
    ls->parity = par ^ 1;
    ls->phase = phase == 2 ? 0 : phase + 1;
}

// Count this workgroup (one thread of it) as having read the launch state: its place in the
// order.  The counter wraps to zero at the last one.  (The compiler turns an addition into a
// wavefront-wide one and waits for its answer on the spot, 1.5 us where every workgroup
// starts at once; it leaves the wrapping increment alone.)
__device__ __forceinline__ int arrive(LaunchState* ls) {
    return (int)__builtin_amdgcn_atomic_inc32((uint32_t*)&ls->arrived, gridDim.x - 1,
                                              __ATOMIC_RELAXED, "agent");
}

// One work item: one part of one tile of one simulation for `steps` sub-steps.  Every part
// of a tile computes the tile's field; each part steps its even share of the tile's cones
// (at most one per thread), and only part 0 writes the field back, so a tile crowded with cones
// is spread over several workgroups.  par selects the input half of every ping-pong pair
// (fields and cone buckets; the other half is written), phase the input third of the counts.
//
// What a workgroup reads before its first sub-step is found from the tile number and the
// launch state alone (count, header, the first sources and targets at a fixed stride, the
// first cone slots), so that it all travels together with the tile's rows; before, headers,
// targets and sources were read one after the other's answer (about 3 us of a launch).
// (with LISTED the item comes from a persistent launch's queue)
template <int NS, int CPL, int SHAPE, bool RECORD, bool LISTED>
__device__ __forceinline__ void tile_body(const TiledArgs2D& a, const TileWork& w,
                                          const PartLists& lists) {
    using V = typename Row<CPL>::T;
    constexpr int W = 64 * CPL;
    constexpr int WAVES = waves_of(SHAPE), kThreads = 64 * WAVES;
    constexpr bool TWO = two_copies(SHAPE);
    extern __shared__ __align__(16) float lds[];
    __shared__ int dest_count[9];
    __shared__ int dest_base[9];
    __shared__ int dest_fill[9];
    __shared__ float4 tile_targets[kMaxTileTargets];
    const int tile = w.tile, steps = w.steps, par = w.par;
    const uint32_t first_step = w.first_step;
    const float* in[SIM_MAX_SPECIES] = {a.field[0][par], a.field[NS > 1 ? 1 : 0][par]};
    float* out[SIM_MAX_SPECIES] = {a.field[0][par ^ 1], a.field[NS > 1 ? 1 : 0][par ^ 1]};
    float4* const bucket_out = a.bucket[par ^ 1];
    int32_t* const count_in = a.count[w.phase];
    int32_t* const count_out = a.count[lists.phase];
    int32_t* const count_next = a.count[3 - w.phase - lists.phase];

    const int tx = tile % a.tiles_x, ty = tile / a.tiles_x;
    const int tiles_y = a.n_tiles / a.tiles_x;
    const int HL = a.height, H = a.halo;
    const int x0 = tx * a.tx_core - H, y0 = ty * a.ty_core - H;
    // species plane: guard row, HL tile rows, three guard rows; row 0 at offset W
    const int plane = W * (HL + kGuardRows);
    // the wavefront index is uniform across a wavefront: keep it (and the strip bounds
    // derived from it) in scalar registers so strip bookkeeping is scalar work
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int cx = CPL * lane;
    const int gx0 = x0 + cx;

    // 0. the tile's count and header, its first sources (every wavefront keeps them, one per
    //    lane) and targets, and the first cone slots, requested together with the tile's
    //    rows.  Every cone of the part stays in registers for the whole launch: cone i sits
    //    in thread i % kThreads, slot i / kThreads (a part holds at most kConeSlots *
    //    kThreads cones).
    const bool first_part = w.part == 0;
    const GlobalPtr<const float4> live = gbl((const float4*)a.bucket[par]) +
                                         (size_t)tile * a.capacity;
    const bool spec = first_part && (int)threadIdx.x < min(kSpecCones, a.capacity);
    float4 mine[kConeSlots];
#pragma unroll
    for (int k = 0; k < kConeSlots; ++k) mine[k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (spec) mine[0] = gload(live + threadIdx.x);
    const int2 hs = gload(gbl(a.head_src) + (size_t)tile * kHeadItems + lane);
    float4 ht = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (wave == WAVES - 1) ht = gload(gbl(a.head_tgt) + (size_t)tile * kHeadItems + lane);
    const int n_all = *gbl(count_in + tile);
    const i4v head = *(GlobalPtr<const i4v>)gbl(a.head + tile);
    const int t_lo = head.x, n_tt = head.y, src_lo = head.z, n_src = head.w;
    const TileContact contact{tile_targets, n_tt, n_tt <= kMaxTileTargets, &a.rules.targets};
    int n_cones = 0;
    // the part's share of the tile's cones (the first n_all % parts parts take one more), and
    // its remaining cones, once the count is there
    auto rest = [&]() {
        const int parts = candidate_parts(n_all, w.chosen, part_units(SHAPE));
        const int each = parts == 1 ? n_all : n_all / parts, more = n_all - each * parts;
        n_cones = each + (w.part < more ? 1 : 0);
        const int first = w.part * each + min(w.part, more);
#pragma unroll
        for (int k = 0; k < kConeSlots; ++k) {
            const int i = threadIdx.x + k * kThreads;
            if (i < n_cones) {
                if (k > 0 || !spec) mine[k] = gload(live + first + i);
            } else {
                mine[k].w = __int_as_float(-1);
            }
        }
    };

    // 1. load the tile, kLoadBatch rows in flight per wavefront; cells outside the grid
    //    read as zero and are never used by cells inside it, which take their own value
    //    for out-of-grid neighbours
    bool col_in[CPL];
#pragma unroll
    for (int k = 0; k < CPL; ++k) col_in[k] = (unsigned)(gx0 + k) < (unsigned)a.nx;
    // whole-segment vector loads and stores when segments cannot straddle the grid edge
    const bool aligned = (x0 % CPL) == 0 && (a.nx % CPL) == 0 && (a.tx_core % CPL) == 0;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const GlobalPtr<const float> f = gbl((const float*)in[s]);
        float* const dst = lds + s * plane + W;
        if (aligned)
            load_tile<CPL, WAVES, true>(dst, f, a.nx, a.ny, y0, HL, gx0, cx, wave, col_in,
                                 [&] { if (s == 0) rest(); });
        else
            load_tile<CPL, WAVES, false>(dst, f, a.nx, a.ny, y0, HL, gx0, cx, wave, col_in,
                                  [&] { if (s == 0) rest(); });
    }
    if (contact.staged) {
        if (wave == WAVES - 1 && lane < n_tt) tile_targets[lane] = ht;
        for (int k = kHeadItems + threadIdx.x; k < n_tt; k += kThreads)
            tile_targets[k] = gload(gbl(a.tgt_pts) + t_lo + k);
    }
    // sin and cos of every heading, carried alongside the cone from sub-step to sub-step, and
    // the second half of the current Philox block
    float2 trig[kConeSlots];
    uint2 spare[kConeSlots];
#pragma unroll
    for (int k = 0; k < kConeSlots; ++k) {
        trig[k] = make_float2(0.0f, 1.0f);
        spare[k] = make_uint2(0u, 0u);
        if (threadIdx.x + k * kThreads < n_cones) sincos_angle(mine[k].z, trig[k].x, trig[k].y);
    }
    if (threadIdx.x < 9) {
        dest_count[threadIdx.x] = 0;
        dest_fill[threadIdx.x] = 0;
    }
    __syncthreads();
    // every wavefront of this workgroup has the launch state by now; the answer is looked at
    // only after the sub-steps
    int order = -1;
    if (!LISTED && threadIdx.x == 0) order = arrive(lists.ls);
    // last launch's input count becomes the next launch's output
    if (first_part && threadIdx.x == 0) count_next[tile] = 0;

    // Strips of the tile's rows inside the grid, [r0, r1), per wavefront, balanced against
    // the cone work: a wavefront stepping cones in k register slots gives up
    // k * cone_rows rows to the others, so that every wavefront does about the same work
    // between two barriers.  Boundaries are computed for every wavefront in scalar registers
    // and kept monotone.  Rows outside the grid are never computed: no cell inside the grid
    // reads them (at the grid's first and last row the missing neighbour is the row itself).
    const int r0 = max(0, -y0), r1 = min(HL, a.ny - y0);
    int ybeg = 0, yend = 0;
    {
        int cw[kConeSlots];   // wavefronts holding a cone in slot k
        int slots = 0;
#pragma unroll
        for (int k = 0; k < kConeSlots; ++k) {
            cw[k] = min(WAVES, (max(n_cones - k * kThreads, 0) + 63) / 64);
            slots += cw[k];
        }
        const float per = (float)(r1 - r0 + a.cone_rows * slots) / WAVES;
        int prev = r0;
        for (int w = 1; w <= WAVES; ++w) {
            int used = 0;
#pragma unroll
            for (int k = 0; k < kConeSlots; ++k) used += a.cone_rows * min(w, cw[k]);
            const int b = w == WAVES ? r1 : min(max(r0 + (int)rintf(w * per) - used, prev), r1);
            if (w == wave) ybeg = b;       // wavefront w's strip is [b(w), b(w + 1))
            if (w == wave + 1) yend = b;
            prev = b;
        }
        if (wave == 0) ybeg = r0;
    }
    const int src_at = W + (hs.x >> 24) * plane + (hs.x & 0xffffff);   // LDS word
    const int src_row = lane < n_src ? (hs.x & 0xffffff) / W : -1;
    const float src_q = __int_as_float(hs.y);
    const ConeRules& rules = a.rules;
    const int cols = x0 > 0 && x0 + W < a.nx ? kNoWall : aligned ? kWallAligned : kWallAny;
    for (int b = 0; b < steps; ++b) {
        // 2. stencil + decay, in place or into the other copy, strip per wavefront.  After this
        //    sub-step only rows [b + 1, HL - b - 1) are still valid (each sub-step loses one row
        //    at either edge of the tile), so rows outside that band are not computed.
        const int lo = max(ybeg, b + 1), hi = min(yend, HL - b - 1);
        const bool top = lo == -y0, bottom = hi == a.ny - y0;
        float* const from = lds + (TWO && (b & 1) ? NS * plane : 0);
        float* const to = lds + (TWO && !(b & 1) ? NS * plane : 0);
        StripEdges<CPL> edge[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (lo < hi) {
                const float* const L = from + s * plane + W;
                float* const T = to + s * plane + W;
                if (cols == kNoWall)
                    edge[s] = strip_update<CPL, kNoWall>(L, T, lo, hi, cx, gx0, a.nx, top,
                                                         bottom, a.coef[s]);
                else if (cols == kWallAligned)
                    edge[s] = strip_update<CPL, kWallAligned>(L, T, lo, hi, cx, gx0, a.nx, top,
                                                              bottom, a.coef[s]);
                else
                    edge[s] = strip_update<CPL, kWallAny>(L, T, lo, hi, cx, gx0, a.nx, top,
                                                          bottom, a.coef[s]);
            }
        }
        if (!TWO) __syncthreads();
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (lo < hi) *(V*)&to[s * plane + (lo + 1) * W + cx] = edge[s].first;
            if (hi - 1 > lo) *(V*)&to[s * plane + hi * W + cx] = edge[s].last;
        }
        // 3. sources in this wavefront's rows [lo, hi) (entries are unique cells per
        //    species; rows no wavefront computes are not valid after this sub-step), added
        //    after its own edge rows: a wavefront's LDS operations take effect in order, and
        //    the barrier below publishes them with the rest of the sub-step
        if (n_src > 0 && lo < hi) {
            if (src_row >= lo && src_row < hi) to[src_at] += src_q;
            for (int e = src_lo + kHeadItems + lane; e < src_lo + n_src; e += 64) {
                const int2 ent = gload(gbl(a.src_entry) + e);
                const int row = ent.x / W;
                if (row >= lo && row < hi) to[ent.y * plane + W + ent.x] += gbl(a.src_amount)[e];
            }
        }
        __syncthreads();
        // recording a run: the state after this sub-step goes to the tape (read from LDS
        // before the next sub-step's in-place update, hence the barrier)
        if (RECORD && first_part) {
            const size_t cells = (size_t)a.nx * a.ny;
            const size_t at = (size_t)(first_step + (uint32_t)b + 1u - a.record_n0) * NS;
            float* tape[SIM_MAX_SPECIES] = {a.record + at * cells,
                                            a.record + (at + (NS - 1)) * cells};
            store_core<NS, CPL, WAVES, true>(tape, to, a, tx, ty, plane, cx, wave, aligned);
            if (!TWO && n_cones == 0) __syncthreads();   // else that after the cones' reads
        }
        // 4. cones against the updated field.  In place, every read of the field (the
        //    gradients) happens before the barrier; the cones then finish their step after
        //    it, overlapping the next sub-step's stencil.  With two copies the next sub-step
        //    writes the other one, which was last read before this sub-step's barrier.
        const uint32_t step = first_step + (uint32_t)b;
        const size_t rec = RECORD ? step - a.record_n0 : 0;
        if (n_cones > 0) {
            const LdsField2D f0{to + W, x0, y0, W, HL};
            const LdsField2D f1{to + (NS > 1 ? plane : 0) + W, x0, y0, W, HL};
            float3 g[kConeSlots];
#pragma unroll
            for (int k = 0; k < kConeSlots; ++k)
                g[k] = tile_cone_gradient<NS, RECORD>(mine[k], f0, f1, rules, a.cone_record, rec);
            if (!TWO) __syncthreads();
#pragma unroll
            for (int k = 0; k < kConeSlots; ++k)
                tile_cone_advance<RECORD>(mine[k], trig[k], spare[k], g[k], rules, step, b == 0,
                                          contact, a.cones, a.cone_record, rec);
        }
    }

    // 5. write the core back (one part per tile does)
    if (first_part)
        store_core<NS, CPL, WAVES>(out, lds + (TWO && (steps & 1) ? NS * plane : 0), a, tx, ty,
                                   plane, cx, wave, aligned);

    // 6. re-bucket surviving cones, straight from registers, into the tile that now holds
    //    their tip (one of the 3 x 3 tiles around this one)
    int dest[kConeSlots];
#pragma unroll
    for (int k = 0; k < kConeSlots; ++k) {
        dest[k] = -1;
        if (threadIdx.x + k * kThreads < n_cones && __float_as_int(mine[k].w) >= 0) {
            const int2 nt = next_tile(mine[k], tx, ty, a.tiles_x, tiles_y, rules.inv_dx, a.nx,
                                      a.ny, a.tx_core, a.ty_core);
            dest[k] = (nt.y - ty + 1) * 3 + (nt.x - tx + 1);
            atomicAdd(&dest_count[dest[k]], 1);
        }
    }
    __syncthreads();
    if (threadIdx.x < 9 && dest_count[threadIdx.x] > 0) {
        const int dtx = tx + threadIdx.x % 3 - 1, dty = ty + threadIdx.x / 3 - 1;
        const int to = dty * a.tiles_x + dtx, n = dest_count[threadIdx.x];
        const int before = atomicAdd(&count_out[to], n);
        dest_base[threadIdx.x] = before;
        list_parts(lists, to, before, before + n);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kConeSlots; ++k) {
        const int d = dest[k];
        if (d < 0) continue;
        const int ntx = tx + d % 3 - 1, nty = ty + d / 3 - 1;
        const int slot = dest_base[d] + atomicAdd(&dest_fill[d], 1);
        gstore(gbl(bucket_out) + (size_t)(nty * a.tiles_x + ntx) * a.capacity + slot, mine[k]);
    }
    if (!LISTED && order == (int)gridDim.x - 1)
        advance_launch(lists.ls, first_step + (uint32_t)steps, par, w.phase);
}

// The step kernel: one workgroup per tile (part 0) and one per listed further part of a
// crowded tile.  The launch state (step counter, ping-pong parity, count phase) is read by
// every workgroup at its start and advanced by the last one to have read it, so launches
// need no host-side bookkeeping and can be captured in a graph and replayed.
//
// Tiles are dealt to the dies in contiguous stretches: the hardware deals workgroup b to die
// b % kXcds, which takes tile (b % kXcds) * per + b / kXcds, per = ceil(n_tiles / kXcds), so
// that the overlapping halo rows and columns of neighbouring tiles are fetched once into that
// die's L2.  The further parts follow: of the candidate sizes the smallest whose list still
// fits beside the tiles (`room`: workgroups resident at once), so that the spare places carry
// the crowded tiles' cones in more, smaller parts and every workgroup still starts at once.
// The lists were filled when the cones were put into their buckets (list_parts).  Earlier the
// last workgroup to finish scanned every tile's count and laid out a list of work items: a
// serial tail of 3-4 us on every launch, and an item to be read before anything else.
//
// What the launch reads that other workgroups change while it runs is the launch state's
// first group alone, which is written after all have read it; counts, lists and buckets are
// read by the next launch, after the kernel boundary.
template <int NS, int CPL, bool RECORD, int SHAPE>
__global__ __launch_bounds__(64 * waves_of(SHAPE)) void k_tiled2d(TiledArgs2D a, int tile_wgs, int steps,
                                                      LaunchState* ls, int4* extra,
                                                      int extra_cap, int room) {
    const int4 head = *(const int4*)ls;   // step, parity, phase
    const int par = head.y, phase = head.z;
    const int next_phase = phase == 2 ? 0 : phase + 1;
    const PartLists lists{ls, extra + (size_t)(par ^ 1) * kPartSizes * extra_cap, extra_cap,
                          next_phase, kPartSizes, 0, part_units(SHAPE)};
    int chosen = 0, chosen_n = min(ls->extra_n[phase][0], extra_cap);
#pragma unroll
    for (int j = 1; j < kPartSizes; ++j) {   // the counts grow with j: keep the last that fits
        const int n = ls->extra_n[phase][j];
        if (n <= room) {
            chosen = j;
            chosen_n = n;
        }
    }
    TileWork w{-1, 0, chosen, steps, (uint32_t)head.x, par, phase};
    const int b = blockIdx.x;
    if (b < tile_wgs) {
        const int t = (b % kXcds) * (tile_wgs / kXcds) + b / kXcds;
        if (t < a.n_tiles) w.tile = t;
    } else if (b - tile_wgs < chosen_n) {
        const int4 it = extra[((size_t)par * kPartSizes + chosen) * extra_cap + b - tile_wgs];
        w.tile = it.y;
        w.part = it.z;
    }
    // the third of the list lengths that last launch read is the next launch's output
    if (b == 0 && threadIdx.x < kPartSizes) ls->extra_n[3 - phase - next_phase][threadIdx.x] = 0;
    if (w.tile >= 0) {
        tile_body<NS, CPL, SHAPE, RECORD, false>(a, w, lists);
    } else {
        __syncthreads();   // every wavefront has read the launch state
        if (threadIdx.x == 0 && arrive(ls) == (int)gridDim.x - 1)
            advance_launch(ls, w.first_step + (uint32_t)steps, par, phase);
    }
}

// The persistent form for a batch: a fixed grid pulls items (a tile of a simulation, then
// the further parts of crowded ones) from an atomic queue until it runs dry.
template <int NS, int CPL>
__global__ __launch_bounds__(512) void k_tiled2d_batch(
    const TiledArgs2D* __restrict__ table, const int2* __restrict__ base, int n_base, int steps,
    LaunchState* ls, int4* extra, int extra_cap) {
    __shared__ int item_idx;
    const int4 head = *(const int4*)ls;   // step, parity, phase
    const int par = head.y, phase = head.z;
    const int next_phase = phase == 2 ? 0 : phase + 1;
    const int n_items = n_base + min(ls->extra_n[phase][0], extra_cap);
    const int4* const listed = extra + (size_t)par * extra_cap;
    if (blockIdx.x == 0 && threadIdx.x == 0) ls->extra_n[3 - phase - next_phase][0] = 0;
    // the next item is taken from the queue while the current one runs, so the queue's
    // round trip is hidden behind the item's work
    if (threadIdx.x == 0) item_idx = atomicAdd(&ls->next, 1);
    __syncthreads();
    int i = item_idx;
    while (i < n_items) {
        int next = 0;
        if (threadIdx.x == 0) next = atomicAdd(&ls->next, 1);
        int sim, tile, part = 0;
        if (i < n_base) {
            const int2 it = base[i];
            sim = it.x;
            tile = it.y;
        } else {
            const int4 it = listed[i - n_base];
            sim = it.x;
            tile = it.y;
            part = it.z;
        }
        const PartLists lists{ls, extra + (size_t)(par ^ 1) * extra_cap, extra_cap, next_phase,
                              kBatchPartLists, sim, part_units(kPair)};
        const TileWork w{tile, part, 0, steps, (uint32_t)head.x, par, phase};
        tile_body<NS, CPL, kPair, false, true>(table[sim], w, lists);
        // every thread read item_idx before tile_body's first barrier
        if (threadIdx.x == 0) item_idx = next;
        __syncthreads();   // the item is done with LDS; item_idx holds the next index
        i = item_idx;
    }
    // the last workgroup to run out of items has the queue and the launch state to itself
    if (threadIdx.x == 0 && arrive(ls) == (int)gridDim.x - 1) {
        ls->next = 0;
        advance_launch(ls, (uint32_t)head.x + (uint32_t)steps, par, phase);
    }
}

// Initial bucketing from the caller-order arrays (active cones only).
__global__ void k_bucket2d(ConeArrays c, int nx, int ny, int tx_core, int ty_core, int tiles_x,
                           float inv_dx, float4* bucket, int32_t* count, int capacity,
                           PartLists lists) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= c.n || c.status[i] != kActive) return;
    const float x = c.pos[2 * i], y = c.pos[2 * i + 1];
    const int t = cell_of(y, inv_dx, ny) / ty_core * tiles_x + cell_of(x, inv_dx, nx) / tx_core;
    const int slot = atomicAdd(&count[t], 1);
    list_parts(lists, t, slot, slot + 1);
    bucket[(size_t)t * capacity + slot] = make_float4(x, y, c.dir[i], __int_as_float(i));
}

// Active cones from the buckets back into the caller-order arrays; with `drop` the tile's
// counts (and the lists of further parts) start over at none.
__global__ void k_sync_cones2d(ConeArrays c, const float4* bucket, int32_t* count0,
                               int32_t* count1, int32_t* count2, int phase, int capacity,
                               bool drop, LaunchState* ls) {
    const int t = blockIdx.x;
    const int n = (phase == 0 ? count0 : phase == 1 ? count1 : count2)[t];
    for (int k = threadIdx.x; k < n; k += blockDim.x) {
        const float4 st = bucket[(size_t)t * capacity + k];
        const int id = __float_as_int(st.w);
        if (id < 0) continue;
        c.pos[2 * id] = st.x;
        c.pos[2 * id + 1] = st.y;
        c.dir[id] = st.z;
    }
    if (!drop) return;
    __syncthreads();   // every thread has the count
    if (threadIdx.x == 0) count0[t] = count1[t] = count2[t] = 0;
    if (t == 0 && threadIdx.x < 3 * 8) (&ls->extra_n[0][0])[threadIdx.x] = 0;
}

int ceil_div(int a, int b) { return (a + b - 1) / b; }

// The kernel variant for a species count, row width and shape; `record` selects the one that
// also writes every sub-step's state to the run tape (only a recording run launches it).
template <bool RECORD>
const void* kernel_of(const TiledPlan& p) {
    if (p.cpl == 4) {
        if (p.n_species > 1) return (const void*)k_tiled2d<2, 4, RECORD, kPair>;
        return p.shape == kWide ? (const void*)k_tiled2d<1, 4, RECORD, kWide>
                                : (const void*)k_tiled2d<1, 4, RECORD, kPair>;
    }
    if (p.shape == kTwo)
        return p.n_species > 1 ? (const void*)k_tiled2d<2, 2, RECORD, kTwo>
                               : (const void*)k_tiled2d<1, 2, RECORD, kTwo>;
    if (p.shape == kTwoPair)
        return p.n_species > 1 ? (const void*)k_tiled2d<2, 2, RECORD, kTwoPair>
                               : (const void*)k_tiled2d<1, 2, RECORD, kTwoPair>;
    return p.n_species > 1 ? (const void*)k_tiled2d<2, 2, RECORD, kPair>
                           : (const void*)k_tiled2d<1, 2, RECORD, kPair>;
}

const void* kernel_for(const TiledPlan& p, bool record = false) {
    return record ? kernel_of<true>(p) : kernel_of<false>(p);
}

const void* batch_kernel_for(int n_species, int cpl) {
    if (n_species == 1)
        return cpl == 4 ? (const void*)k_tiled2d_batch<1, 4> : (const void*)k_tiled2d_batch<1, 2>;
    return cpl == 4 ? (const void*)k_tiled2d_batch<2, 4> : (const void*)k_tiled2d_batch<2, 2>;
}

}  // namespace

namespace {

// Cells a tile is loaded with on each side of its core at depth B: B sub-steps of shrinkage,
// cone travel before the last sub-step and the gradient footprint (two cells); the small epsilon
// covers FP32 rounding of travel.  Rounded up to the lane segment, which keeps every segment of
// the tile and its core aligned: whole-segment vector loads and stores.
int halo_for(int B, double step_cells, int cpl) {
    const int travel = (int)std::ceil((B - 1) * step_cells + 1e-3);
    return (B + travel + 2 + cpl - 1) / cpl * cpl;
}

// Workgroups of `lds` bytes of dynamic LDS that share a CU (two at most).
int sharing(size_t lds) {
    return std::max(1, std::min(2, (int)(kCuLds / (lds + kStaticLds))));
}

// Shape for `tiles` tiles whose single copy takes `lds` bytes (alone: not in a batch, whose
// queue steps more tiles than start at once).  kTwo leaves a CU to each tile and so fewer for the
// further parts of crowded ones: not where evenly spread cones would already be split (900 x 700,
// 228 tiles, 40,000 cones: 2.29 us per step against 2.73; 60,000: 3.64 against 2.89).
TileShape shape_for(int n_species, int cpl, int height, int tiles, int n_cones, size_t lds,
                    bool alone) {
    if (!alone) return kPair;
    if (cpl == 4) return n_species == 1 && height >= kWideRows ? kWide : kPair;
    const int at_once = ceil_div(tiles, kXcds) * kXcds;
    if (sharing(2 * lds) == 2 && at_once <= 512) return kTwoPair;
    const bool sparse = n_cones <= (int64_t)kSmallest * tiles;
    return 2 * lds <= kLdsBudget && at_once <= 256 && sparse ? kTwo : kPair;
}

// Threads of a launch (at most: the parts' list is as long as every cone can make it), of which the
// runtime takes fewer than 2^32: grids of some hundred million columns and few rows need wide tiles.
int64_t launch_threads(int tiles, int n_cones, TileShape shape) {
    const int64_t parts = std::max(tiled_extra_capacity(n_cones), 512);
    return ((int64_t)ceil_div(tiles, kXcds) * kXcds + parts) * 64 * waves_of(shape);
}

// Microseconds per step of a plan, for the choice of the depth: a launch takes 7 us besides its
// sub-steps, a sub-step 1.1 us (1.0 with two copies of the tile) and 3.2 ns per row of each
// two-column species plane in its CU (a quarter more for 8 wavefronts alone there, which hide
// latency poorly), and tiles past those that start at once wait.  Per step, measured with one
// copy at depths 4 / 8 / 12 / 16 / 20 / 24: 128 x 128 3.0 / 2.1 / 1.84 / 1.73 / 1.68 / 1.72 us;
// 777 x 389, two species 4.1 / 3.1 / 2.93 / 2.89 / 3.1 / 3.2; 1000 x 600 3.2 / 2.3 / 2.01 /
// 1.97 / 1.94 / 2.0; 1500 x 1100 4.0 / 3.0 / 2.69 / 2.65 / 2.70 / 2.9.  Depths past 16 gain
// nothing, and calls of few steps pay for their halo.
constexpr int kDeepest = 16;

double step_time(const TiledPlan& p) {
    const int per_cu = ceil_div(p.n_tiles, 256), fit = sharing(p.lds_bytes);
    const double rows = (double)p.height * std::min(per_cu, fit) * p.n_species * p.cpl / 2;
    const double sub = ((two_copies(p.shape) ? 1.0 : 1.1) + 0.0032 * rows) *
                       (fit < 2 && p.shape == kPair ? 1.25 : 1.0);
    return ceil_div(per_cu, fit) * (7.0 / p.block_steps + sub);
}

// Best tile plan by the cost model, restricted to row width 64 * only_cpl and loaded height
// only_height when those are non-zero.  Depth: the deepest that fits up to block_steps, or with
// block_steps 0 the fastest up to kDeepest.
TiledPlan plan_search(int dim, int nx, int ny, int nz, int n_species, double step_cells,
                      int block_steps, int n_cones, int only_cpl, int only_height, bool alone) {
    TiledPlan best, fastest;
    const bool any_depth = block_steps == 0;
    if (any_depth) block_steps = kDeepest;
    best.dim = dim;
    best.nx = nx;
    best.ny = ny;
    best.nz = nz;
    best.n_species = n_species;
    best.block_steps = 1;
    if (dim != 2 || block_steps < 2) return best;
    fastest = best;
    double best_cost = 1e300;
    for (int B = block_steps; B >= 2; --B) {
        const int move = (int)std::ceil(B * step_cells + 1e-3);
        for (int cpl : {2, 4}) {
            if (only_cpl && cpl != only_cpl) continue;
            const int H = halo_for(B, step_cells, cpl);
            const int W = 64 * cpl;
            const int TX = W - 2 * H;
            if (TX < 16 || TX <= move) continue;
            const int max_height =
                (int)(kLdsBudget / ((size_t)n_species * W * sizeof(float))) - kGuardRows;
            for (int HL = 2 * H + 16; HL <= max_height; ++HL) {
                if (only_height && HL != only_height) continue;
                const int TY = HL - 2 * H;
                if (TY <= move) continue;
                const size_t lds = (size_t)n_species * W * (HL + kGuardRows) * sizeof(float);
                const int tiles = ceil_div(nx, TX) * ceil_div(ny, TY);
                const int per_cu = ceil_div(tiles, 256);
                const TileShape shape = shape_for(n_species, cpl, HL, tiles, n_cones, lds,
                                                  alone);
                if (launch_threads(tiles, n_cones, shape) > UINT32_MAX) continue;
                const size_t used = two_copies(shape) ? 2 * lds : lds;
                const int resident = sharing(used);
                // per-step cost in cell-updates per compute unit: each tile's loaded area
                // per sub-step plus its load/store per launch; one tile of 8 wavefronts per
                // CU hides latency poorly.  Cones gather (attracted to the sources), and a tile
                // holding more than a part's of them takes extra workgroups: keep room
                // for a quarter of the cones in full parts beside one workgroup per tile,
                // or the launch runs in two generations.
                const int spare =
                    std::min(tiles, ceil_div(n_cones, 4 * kPartCones * part_units(shape)));
                double cost = (double)per_cu * W * HL * (1.0 + 2.0 / B) / B;
                if ((resident < 2 && shape == kPair) || ceil_div(tiles + spare, 256) > resident)
                    cost *= 1.25;
                if (cost < best_cost * 0.999) {
                    best_cost = cost;
                    best.block_steps = B;
                    best.move = move;
                    best.halo = H;
                    best.cpl = cpl;
                    best.shape = shape;
                    best.core_x = TX;
                    best.core_y = TY;
                    best.tiles_x = ceil_div(nx, TX);
                    best.tiles_y = ceil_div(ny, TY);
                    best.n_tiles = best.tiles_x * best.tiles_y;
                    best.lds_bytes = used;
                    best.height = HL;
                    // one cone step costs about as much as a stencil row of ~30 cells per
                    // lane-slot pair: 15 rows of two-cell segments for one species
                    best.cone_rows = std::max(1, 30 / (cpl * n_species));
                }
            }
        }
        if (best.block_steps <= 1) continue;
        if (!any_depth) return best;
        if (fastest.block_steps <= 1 || step_time(best) < step_time(fastest)) fastest = best;
        best.block_steps = 1;
        best_cost = 1e300;
    }
    return any_depth ? fastest : best;
}

}  // namespace

TiledPlan tiled_plan(int dim, int nx, int ny, int nz, int n_species, double step_cells,
                     int block_steps, int n_cones, int force_cpl, int force_height,
                     bool alone) {
    if (force_cpl != 0 || force_height != 0) {
        const TiledPlan forced = plan_search(dim, nx, ny, nz, n_species, step_cells,
                                             block_steps, n_cones, force_cpl, force_height,
                                             alone);
        if (forced.block_steps > 1) return forced;
    }
    return plan_search(dim, nx, ny, nz, n_species, step_cells, block_steps, n_cones,
                       alone ? 0 : force_cpl, 0, alone);
}

// Whether a loaded height leaves a core that holds every cone for a launch of depth B, the tile in
// LDS (the conditions of plan_search).
static bool height_fits(const sim_params& p, int B, int cpl, int height) {
    const double step_cells = p.step_len / p.dx;
    const int H = halo_for(B, step_cells, cpl), W = 64 * cpl;
    const int move = (int)std::ceil(B * step_cells + 1e-3);
    const size_t row = (size_t)p.n_species * W * sizeof(float);
    return W - 2 * H >= std::max(16, move + 1) && height - 2 * H >= std::max(16, move + 1) &&
           height <= (int)(kLdsBudget / row) - kGuardRows;
}

// A launch of a batch takes its items' time over the workgroups that run at once.  An item of
// height h takes T = 6 us + h (0.125 + 0.0118 B) us where two share a CU (fit over batches of
// heights 56 .. 144 at depths 8 .. 16, two-column rows of one species), and 7 + B (1.1 + 0.0032 h)
// where it has a CU to itself.  Planned as if it had the chip to itself, every simulation took
// the smallest cores, 16 rows of 44 loaded: 128 simulations of side 64 .. 512 took 33.6 us per
// step, with 144 rows at depth 8 13.9 and at depth 12 13.3.
// A member's tile_height is its height, at depths where it fits; one that fits at no depth is
// ignored.
int tiled_batch_shape(const sim_params* const* params, int n, int cpl,
                      std::vector<int>& height) {
    const int n_species = params[0]->n_species, fixed = params[0]->block_steps;
    const int row_bytes = n_species * 64 * cpl * (int)sizeof(float);
    const int tallest = (int)(80 * 1024 - kStaticLds) / row_bytes - kGuardRows;   // two per CU
    const double planes = n_species * cpl / 2.0;
    double best = 1e300;
    int depth = 0;
    height.assign(n, 0);
    std::vector<int> hint(n, 0);
    for (int i = 0; i < n; ++i)
        for (int B = fixed != 0 ? fixed : kDeepest; B >= 2 && hint[i] == 0; --B)
            if (height_fits(*params[i], B, cpl, params[i]->tile_height))
                hint[i] = params[i]->tile_height;
    for (const int B : {16, 12, 8}) {
        if (fixed != 0 && B != 16) break;
        const int b = fixed != 0 ? fixed : B;
        for (int cap = 32; cap <= tallest; cap += 8) {
            std::vector<int> h(n, 0);
            double work = 0.0, longest = 0.0, alone = 0.0;
            int64_t items = 0;
            bool fits = true;
            for (int i = 0; i < n && fits; ++i) {
                const sim_params& p = *params[i];
                const double step_cells = p.step_len / p.dx;
                const int H = halo_for(b, step_cells, cpl), TX = 64 * cpl - 2 * H;
                const int least = std::max(16, (int)std::ceil(b * step_cells + 1e-3) + 1);
                fits = hint[i] ? height_fits(p, b, cpl, hint[i])
                               : TX >= least && 2 * H + least <= cap;
                if (!fits) break;
                if (hint[i]) {
                    h[i] = hint[i];
                } else {
                    const int tiles_y = ceil_div(p.ny, cap - 2 * H);
                    h[i] = 2 * H + std::max(least, ceil_div(p.ny, tiles_y));
                }
                const int tiles = ceil_div(p.nx, TX) * ceil_div(p.ny, h[i] - 2 * H);
                const double t = 6.0 + h[i] * planes * (0.125 + 0.0118 * b);
                items += tiles;
                work += tiles * t;
                longest = std::max(longest, t);
                alone = std::max(alone, 7.0 + b * (1.1 + 0.0032 * h[i] * planes));
            }
            if (!fits) continue;
            const double t = (items <= 256   ? alone
                              : items <= 512 ? longest
                                             : work / 512 + 0.5 * longest) / b;
            if (t < best) {
                best = t;
                depth = b;
                height = h;
            }
        }
    }
    return depth;
}

// (the other row width where the one asked for, or two columns per lane, leaves no common shape:
// steps of 31 cells fit 256 columns at depth 2 and 128 at none)
int tiled_batch_plan(const sim_params* const* params, int n, BatchPlan& plan) {
    const int asked = params[0]->tile_cols_per_lane ? params[0]->tile_cols_per_lane : 2;
    int misfit = -1;
    for (const int cpl : {asked, 6 - asked}) {
        std::vector<int> height;
        std::vector<TiledPlan> members;
        const int depth = tiled_batch_shape(params, n, cpl, height);
        int common = 0, i = 0;
        for (; i < n; ++i) {
            const sim_params& p = *params[i];
            const int b = p.block_steps ? p.block_steps : depth ? depth : kDefaultBlockSteps;
            const TiledPlan t = tiled_plan(p.dim, p.nx, p.ny, 1, p.n_species, p.step_len / p.dx, b,
                                           p.n_cones, cpl, depth ? height[i] : p.tile_height,
                                           false);
            if (i == 0) common = t.block_steps;
            if (t.block_steps <= 1 || t.block_steps != common) break;
            members.push_back(t);
        }
        if (i == n) {
            plan = BatchPlan{cpl, common, members};
            return -1;
        }
        if (cpl == asked) misfit = i;
    }
    return misfit;
}

hipError_t tiled_allocate(const TiledPlan& plan, TiledState& st, int n_cones,
                          const ConeRules& rules, const sim_params* p, float* const fields[][2],
                          ConeArrays cones, hipStream_t stream) {
    hipError_t e;
    const int W = 64 * plan.cpl;
    st.capacity = std::max(1, n_cones);
    const size_t slots = (size_t)plan.n_tiles * st.capacity;
    if ((e = device_malloc((void**)&st.bucket[0], 2 * slots * sizeof(float4))) != hipSuccess) return e;
    st.bucket[1] = st.bucket[0] + slots;
    st.cur = 0;
    st.phase = 0;
    // per-tile source entries: every unique source cell inside a tile's loaded region
    std::vector<std::vector<std::pair<int2, float>>> per_tile(plan.n_tiles);
    const double vol = std::pow(p->dx, p->dim);
    for (int s = 0; s < p->n_species; ++s) {
        std::map<int32_t, double> merged;
        for (int m = 0; m < p->n_sources[s]; ++m)
            merged[p->source_cell[s][m]] += (double)p->source_q[s][m] / vol;
        for (auto& kv : merged) {
            const int gx = kv.first % plan.nx, gy = kv.first / plan.nx;
            for (int ty = 0; ty < plan.tiles_y; ++ty) {
                const int y0 = ty * plan.core_y - plan.halo;
                if (gy < y0 || gy >= y0 + plan.height) continue;
                for (int tx = 0; tx < plan.tiles_x; ++tx) {
                    const int x0 = tx * plan.core_x - plan.halo;
                    if (gx < x0 || gx >= x0 + W) continue;
                    const int local = (gy - y0) * W + (gx - x0);
                    per_tile[ty * plan.tiles_x + tx].push_back({make_int2(local, s), (float)kv.second});
                }
            }
        }
    }
    std::vector<int4> head(plan.n_tiles, make_int4(0, 0, 0, 0));
    std::vector<int2> head_src((size_t)plan.n_tiles * kHeadItems, make_int2(0, 0));
    std::vector<float4> head_tgt((size_t)plan.n_tiles * kHeadItems);
    std::vector<int2> entry;
    std::vector<float> amount;
    for (int t = 0; t < plan.n_tiles; ++t) {
        head[t].z = (int)entry.size();
        head[t].w = (int)per_tile[t].size();
        for (size_t k = 0; k < per_tile[t].size(); ++k) {
            const auto& en = per_tile[t][k];
            entry.push_back(en.first);
            amount.push_back(en.second);
            if (k >= kHeadItems) continue;
            int2& h = head_src[(size_t)t * kHeadItems + k];
            h.x = en.first.x | en.first.y << 24;   // a tile holds fewer than 2^24 cells
            std::memcpy(&h.y, &en.second, sizeof h.y);
        }
    }
    // per-tile target lists: every target within reach of a tip that starts the launch in
    // the tile core (core grown by the launch's travel, plus the contact radius)
    std::vector<float4> tpts;
    {
        const double reach = (plan.move + 1) * p->dx + p->contact_radius;
        std::vector<std::vector<float4>> lists(plan.n_tiles);
        for (int t = 0; t < p->n_targets; ++t) {
            const float tx_ = p->target_pos[2 * t], ty_ = p->target_pos[2 * t + 1];
            for (int ty = 0; ty < plan.tiles_y; ++ty) {
                const double ylo = ty * plan.core_y * p->dx - reach;
                const double yhi = (ty + 1) * plan.core_y * p->dx + reach;
                if (ty_ < ylo || ty_ > yhi) continue;
                for (int tx = 0; tx < plan.tiles_x; ++tx) {
                    const double xlo = tx * plan.core_x * p->dx - reach;
                    const double xhi = (tx + 1) * plan.core_x * p->dx + reach;
                    if (tx_ < xlo || tx_ > xhi) continue;
                    float4 v = make_float4(tx_, ty_, 0.0f, 0.0f);
                    int32_t idx = t;
                    std::memcpy(&v.w, &idx, sizeof idx);
                    lists[ty * plan.tiles_x + tx].push_back(v);
                }
            }
        }
        for (int t = 0; t < plan.n_tiles; ++t) {
            head[t].x = (int)tpts.size();
            head[t].y = (int)lists[t].size();
            tpts.insert(tpts.end(), lists[t].begin(), lists[t].end());
            std::copy_n(lists[t].begin(), std::min<size_t>(lists[t].size(), kHeadItems),
                        head_tgt.begin() + (size_t)t * kHeadItems);
        }
    }
    // further parts of crowded tiles: full parts always fit their list; smaller ones are used
    // only when they fit beside the tiles
    // (workgroups are dealt to the dies round-robin, idle ones of the last round included: a
    // part past this count would wait for a CU of its die; 220 tiles and 36 parts took 6.0 us per
    // step instead of 4.0)
    st.room = std::max(0, tiled_persistent_grid(plan.lds_bytes) -
                              ceil_div(plan.n_tiles, kXcds) * kXcds);
    st.extra_cap = std::max(tiled_extra_capacity(n_cones),
                            std::min(st.room, ceil_div(n_cones, kSmallest)));
    st.room = std::min(st.room, st.extra_cap);
    // one allocation: the launch state, counts and lists (zeroed), then the tables (one copy)
    size_t bytes = 0;
    auto place = [&](size_t n) {
        const size_t at = bytes;
        bytes += (n + 255) / 256 * 256;
        return at;
    };
    const size_t n_t = (size_t)plan.n_tiles;
    const size_t at_launch = place(sizeof(LaunchState));
    size_t at_count[3];
    for (size_t& c : at_count) c = place(n_t * sizeof(int32_t));
    const size_t at_extra = place((size_t)2 * kPartSizes * st.extra_cap * sizeof(int4));
    const size_t zeroed = bytes;
    std::vector<char> tables;
    auto table = [&](const auto& v) {
        const size_t n = v.size() * sizeof(v[0]), at = place(n);
        tables.resize(bytes - zeroed);
        if (n) std::memcpy(tables.data() + (at - zeroed), v.data(), n);
        return at;
    };
    const size_t at_head = table(head), at_entry = table(entry), at_amount = table(amount),
                 at_tgt = table(tpts), at_hsrc = table(head_src), at_htgt = table(head_tgt);
    if ((e = device_malloc((void**)&st.memory, bytes)) != hipSuccess ||
        (e = hipMemsetAsync(st.memory, 0, zeroed, stream)) != hipSuccess ||
        (e = hipMemcpy(st.memory + zeroed, tables.data(), tables.size(),
                       hipMemcpyHostToDevice)) != hipSuccess)
        return e;
    st.launch = (LaunchState*)(st.memory + at_launch);
    for (int b = 0; b < 3; ++b) st.count[b] = (int32_t*)(st.memory + at_count[b]);
    st.extra = (int4*)(st.memory + at_extra);
    // the kernel's arguments and the launch state
    st.args = new (std::nothrow) TiledArgs2D();
    if (!st.args) return hipErrorOutOfMemory;
    TiledArgs2D& a = *st.args;
    for (int s = 0; s < plan.n_species; ++s) {
        a.field[s][0] = fields[s][0];
        a.field[s][1] = fields[s][1];
        a.coef[s] = plan.coef[s];
    }
    a.nx = plan.nx;
    a.ny = plan.ny;
    a.tiles_x = plan.tiles_x;
    a.n_tiles = plan.n_tiles;
    a.tx_core = plan.core_x;
    a.ty_core = plan.core_y;
    a.halo = plan.halo;
    a.height = plan.height;
    a.head = (const int4*)(st.memory + at_head);
    a.src_entry = (const int2*)(st.memory + at_entry);
    a.src_amount = (const float*)(st.memory + at_amount);
    a.tgt_pts = (const float4*)(st.memory + at_tgt);
    a.head_src = (const int2*)(st.memory + at_hsrc);
    a.head_tgt = (const float4*)(st.memory + at_htgt);
    a.bucket[0] = st.bucket[0];
    a.bucket[1] = st.bucket[1];
    a.count[0] = st.count[0];
    a.count[1] = st.count[1];
    a.count[2] = st.count[2];
    a.capacity = st.capacity;
    a.cone_rows = plan.cone_rows;
    a.cones = cones;
    a.rules = rules;
    for (bool record : {false, true})
        if ((e = hipFuncSetAttribute(kernel_for(plan, record),
                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)plan.lds_bytes)) != hipSuccess)
            return e;
    return hipSuccess;
}

void tiled_set_record(TiledState& st, float* tape, const ConeTape& cones, uint32_t n0) {
    st.args->record = tape;
    st.args->cone_record = cones;
    st.args->record_n0 = n0;
}

hipError_t tiled_set_launch_state(TiledState& st, uint32_t step, int parity, hipStream_t stream) {
    const int32_t head[2] = {(int32_t)step, parity};   // step and parity; items untouched
    st.cur = parity;
    hipError_t e = hipMemcpyAsync(st.launch, head, sizeof head, hipMemcpyHostToDevice, stream);
    if (e != hipSuccess) return e;
    return hipStreamSynchronize(stream);
}

hipError_t tiled_get_launch_state(TiledState& st) {
    int32_t head[3];   // step, parity, phase
    const hipError_t e = hipMemcpy(head, st.launch, sizeof head, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return e;
    st.cur = head[1];
    st.phase = head[2];
    return hipSuccess;
}

int tiled_extra_capacity(int64_t n_cones) {
    // a tile of c cones has ceil(c / kPartCones) - 1 < c / kPartCones further full parts
    return (int)(n_cones / kPartCones) + 1;
}

void tiled_release(TiledState& st) {
    device_free(st.bucket[0]);
    device_free(st.memory);
    delete st.args;
    st = TiledState();
}

hipError_t tiled_bucket_batch(const TiledPlan& plan, TiledState& st, ConeArrays cones, int sim,
                              LaunchState* launch, int4* extra, int extra_cap,
                              hipStream_t stream) {
    if (cones.n == 0) return hipSuccess;
    const int sizes = launch == st.launch ? kPartSizes : kBatchPartLists;
    const PartLists lists{launch, extra + (size_t)st.cur * sizes * extra_cap, extra_cap,
                          st.phase, sizes, sim, part_units(plan.shape)};
    hipLaunchKernelGGL(k_bucket2d, dim3(ceil_div(cones.n, 256)), dim3(256), 0, stream, cones,
                       plan.nx, plan.ny, plan.core_x, plan.core_y, plan.tiles_x, plan.inv_dx,
                       st.bucket[st.cur], st.count[st.phase], st.capacity, lists);
    return hipGetLastError();
}

hipError_t tiled_bucket(const TiledPlan& plan, TiledState& st, ConeArrays cones,
                        hipStream_t stream) {
    return tiled_bucket_batch(plan, st, cones, 0, st.launch, st.extra, st.extra_cap, stream);
}

hipError_t tiled_sync_cones(const TiledPlan& plan, TiledState& st, ConeArrays cones,
                            hipStream_t stream, bool drop) {
    hipLaunchKernelGGL(k_sync_cones2d, dim3(plan.n_tiles), dim3(256), 0, stream, cones,
                       st.bucket[st.cur], st.count[0], st.count[1], st.count[2], st.phase,
                       st.capacity, drop, st.launch);
    return hipGetLastError();
}

hipError_t tiled_launch(const TiledPlan& plan, TiledState& st, int steps, hipStream_t stream,
                        hipEvent_t start, hipEvent_t stop) {
    int tile_wgs = ceil_div(plan.n_tiles, kXcds) * kXcds;
    void* args[] = {st.args, &tile_wgs, &steps, &st.launch, &st.extra, &st.extra_cap, &st.room};
    const hipError_t e = hipExtLaunchKernel(
        kernel_for(plan, st.args->record != nullptr),
        dim3(tile_wgs + st.extra_cap), dim3(64 * waves_of(plan.shape)), args, plan.lds_bytes,
        stream, start, stop, 0);
    if (e == hipSuccess) tiled_advanced(st, 1);
    return e;
}

void tiled_advanced(TiledState& st, int launches) {
    st.cur ^= launches & 1;
    st.phase = (st.phase + launches) % 3;
}

size_t tiled_table_entry_bytes() { return sizeof(TiledArgs2D); }

int tiled_persistent_grid(size_t lds_bytes) {
    return 256 * sharing(lds_bytes);
}

hipError_t tiled_launch_batch(const TiledArgs2D* table, int4* extra, const int2* base,
                              int n_base, int extra_cap, int n_species, int cpl,
                              size_t lds_bytes, int steps, LaunchState* launch,
                              hipStream_t stream) {
    void* args[] = {&table, &base, &n_base, &steps, &launch, &extra, &extra_cap};
    return hipLaunchKernel(batch_kernel_for(n_species, cpl),
                           dim3(tiled_persistent_grid(lds_bytes)), dim3(512), args,
                           lds_bytes, stream);
}

hipError_t tiled_prepare_batch(int n_species, int cpl, size_t lds_bytes) {
    return hipFuncSetAttribute(batch_kernel_for(n_species, cpl),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
}

}  // namespace cuesim
