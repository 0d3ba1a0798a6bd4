// kernels_reverse2d.hip -- the reverse field steps of the gradient sweep, up to kRevSteps per
// launch: with b^t = a^{t+1} + e^t (e: the cone samples' adjoints of run step t),
//   a^t = b + r Lap b - k dt b    (the zero-flux Laplacian is symmetric),
// FP64 sums of b Lap c^t (for dL/dD) and b c^t (for dL/dk) over all cells, and b at every
// source cell (for dL/dq).
//
// One workgroup takes one tile of one species: a core of kTX x kTY cells and a halo of
// kRevSteps cells on every side, a^{t+1} loaded into LDS once; each sub-step adds the cones'
// adjoints into the tile, updates it in place (the valid region shrinks by one cell) and adds
// the core's share of the two sums, reading c^t from the run's recorded states, one sub-step
// ahead of its use; the core's a goes back to memory after the last.
//
// The cones' adjoints of a step are added per cell as 64-bit fixed-point numbers (LDS integer
// atomics, value = q 2^(e - kFixedBits), 2^e from the step's largest contribution) and enter
// the tile as one float: integer additions, so the sum in a cell does not depend on the order
// in which the contributions arrive and the gradient is bitwise reproducible.  Which cones can
// touch a tile's loaded region during a launch is listed beforehand, per launch of a segment
// (k_tile_lists); a contribution is rebuilt where it is needed from the cone's tip and the
// adjoint of its sampled gradient (20 bytes per cone and step, against a 96-byte record of the
// 12 cells and values).
//
// Before, each step's contributions went into a buffer of sums over the whole grid in HBM by
// global 64-bit atomics (3.9 us per step at 1024^2 and 8192 cones), which the reverse step
// then read (8 B per cell and step), at two steps per launch (6.6 us per step).
// HBM bytes per cell and step now: c^t once (4 B), and a in and out once per launch.
// Bound: the VALU (about 12 instructions per row of two cells for the stencil, 22 for the
// sums) and the barriers between sub-steps.
//
// The cones' chain of the segment before (cone_adjoint.hpp) needs no field adjoint: eight of its
// steps per launch run in workgroups past the tiles', on CUs that the tiles leave free.  1024^2,
// 8192 cones: 0.7 us more per launch (22.3 with it), against 55 us per 100 steps for the chain alone
// (gradient of 2000 steps 14.27 -> 13.6 ms; now 13.1).
#include <algorithm>
#include <type_traits>

#include "cone_adjoint.hpp"
#include "rows.hpp"

namespace cuesim {

namespace {

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kCPL = 2;
constexpr int kW = 64 * kCPL;             // loaded tile width
constexpr int kH = kRevSteps;             // halo
// Rows per wavefront, all in registers during a sub-step.  A core row costs three times a halo
// row (the two sums), so the first and the last wavefront take the halo's rows and two of the
// core's, the others three core rows each: tiles of 112 x 22 cells, 470 of them at 1024^2, so
// that every workgroup of that grid is resident at once (two per CU).
constexpr int kEdgeCore = 2, kMidCore = 3;
constexpr int kTX = kW - 2 * kH, kTY = 2 * kEdgeCore + (kWaves - 2) * kMidCore;
constexpr int kHL = kTY + 2 * kH;         // loaded height
constexpr int kXcds = 8;                  // (ReverseGrid)
constexpr int kTileCones = kThreads / 4;  // cones of a tile whose steps are held in LDS: one
                                          // cone per four threads
constexpr int kListThreads = 1024;
constexpr int kListTiles = 24 * 1024;     // most tiles counted in LDS
static_assert(kTX > 0 && kTY > 0 && kH % kCPL == 0, "tile shape");

using V = float2;

struct ReverseArgs {
    const float* a_in[2];
    float* a_out[2];
    StencilCoef coef[2];
    ConeRules rules;
    const float* fields;       // c^t of species s: fields + (t * n_species + s) * cells
    size_t cells;
    int n_species, nx, ny, tiles_x, n_tiles;
    ReverseGrid grid;
    int t_hi, steps;           // segment steps t_hi, t_hi - 1, .. are reversed
    int M;
    const float4* tips;        // [t][M]: tip (x, y, ..) at the start of step t
    const float2* ag;          // [t][M]: the adjoint of the cone's sampled gradient
    const uint32_t* step_max;  // [t]
    const int32_t* list_end;   // [tile]: where the tile's cones end in the list
    const int32_t* list;
    double* acc_D;             // [species][tile]
    double* acc_k;
    const int32_t* q_start;    // [species][tile + 1] into q_entry
    const int2* q_entry;       // (LDS cell in its tile, source number)
    double* acc_q;
    ConeChain chain;           // kRevSteps steps of it, by the workgroups past the tiles'
};

// Sum of v over the wavefront, valid in lane 63: shifts within rows of 16 lanes, then the row
// totals broadcast to the rows after them, without a trip through LDS.
template <int CTRL, int ROWS>
__device__ __forceinline__ double plus_dpp(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xF, false);
    return v + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_sum(double v) {
    v = plus_dpp<0x111, 0xF>(v);   // row_shr:1, 2, 4, 8
    v = plus_dpp<0x112, 0xF>(v);
    v = plus_dpp<0x114, 0xF>(v);
    v = plus_dpp<0x118, 0xF>(v);
    v = plus_dpp<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
    return plus_dpp<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3
}

// Three of the 12 cells of the sample of a cone p = (x, y, agx, agy), cells 3 q .. 3 q + 2: as
// LDS cells of the tile (-1: outside the loaded region) and their adjoints.
struct Share {
    int at[3];
    float v[3];
};
constexpr int kShares = kThreads / kTileCones;   // threads per cone
static_assert(kShares == 4, "four threads share 12 cells");

__device__ __forceinline__ Share share_of(const ConeRules& r, float sign, const float4& p, int q,
                                          int x0, int y0) {
    const Scatter2D s = sample_adjoint_2d(r, p.x, p.y, sign * p.z, sign * p.w);
    Share c;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        int i = s.i[k], j = s.j[k];
        c.v[k] = s.v[k];
#pragma unroll
        for (int m = 1; m < kShares; ++m) {
            i = q == m ? s.i[3 * m + k] : i;
            j = q == m ? s.j[3 * m + k] : j;
            c.v[k] = q == m ? s.v[3 * m + k] : c.v[k];
        }
        const int lx = i - x0, ly = j - y0;
        const bool in = (unsigned)lx < (unsigned)kW && (unsigned)ly < (unsigned)kHL;
        c.at[k] = in ? ly * kW + lx : -1;
    }
    return c;
}

// One wavefront's strip of a tile: N rows from loaded row LY0, of which rows CORE0 ..
// CORE0 + CORES - 1 of the strip belong to the core.  EDGE: the tile meets a wall of the grid,
// so rows and columns outside it are skipped, clamped or replaced (else no test is needed).
template <int N, int CORE0, int CORES, bool ALIGNED, bool EDGE>
struct Strip {
    V row[N + 2];        // b on the strip and a row to either side
    V c[CORES + 2];      // c^t on the strip's core rows and a row to either side

    __device__ __forceinline__ void load_c(GlobalPtr<const float> f, int nx, int ny, int gy0,
                                           int gx0) {
#pragma unroll
        for (int r = 0; r < CORES + 2; ++r) {
            const int gy = gy0 + CORE0 + r - 1;
            if (EDGE || !ALIGNED) {
                const RowVec<kCPL> v = load_row<kCPL, ALIGNED>(f, nx, ny, gy, gx0);
                c[r] = make_float2(v[0], v[1]);
            } else {
                const RowVec<kCPL> v = *(GlobalPtr<const RowVec<kCPL>>)(f + (size_t)gy * nx + gx0);
                c[r] = make_float2(v[0], v[1]);
            }
        }
    }
    __device__ __forceinline__ void read(const float* L, int ly0) {
#pragma unroll
        for (int r = 0; r < N + 2; ++r) row[r] = *(const V*)&L[(ly0 + r - 1) * kW];
    }
    // Sub-step k: the strip's new rows into the tile (rows that later sub-steps need) and the
    // core rows' share of the sums.
    __device__ __forceinline__ void step(float* L, int ly0, int k, int gy0, int gx0, int nx,
                                         int ny, const StencilCoef& coef, bool core_col,
                                         double& pD, double& pk) {
        constexpr int COLS = EDGE ? kWallAny : kNoWall;
#pragma unroll
        for (int r = 0; r < N; ++r) {
            const bool core = r >= CORE0 && r < CORE0 + CORES;
            const int ly = ly0 + r, gy = gy0 + r;
            if (!core && (ly <= k || ly >= kHL - 1 - k)) continue;
            if (EDGE && (gy < 0 || gy >= ny)) continue;
            const V mid = row[r + 1];
            const V below = EDGE && gy == 0 ? mid : row[r];
            const V above = EDGE && gy == ny - 1 ? mid : row[r + 2];
            *(V*)&L[ly * kW] = row_update<kCPL, COLS>(below, mid, above, gx0, nx, coef);
            if (!core) continue;
            // c's rows are clamped into the grid: the zero-flux rule at its first and last
            const int m = r - CORE0 + 1;
            const V lap = row_laplacian<kCPL, COLS>(c[m - 1], c[m], c[m + 1], gx0, nx);
            if (core_col && (!EDGE || gx0 < nx)) {
                pD = fma((double)mid.x, (double)lap.x, pD);
                pk = fma((double)mid.x, (double)c[m].x, pk);
                if (!EDGE || ALIGNED || gx0 + 1 < nx) {
                    pD = fma((double)mid.y, (double)lap.y, pD);
                    pk = fma((double)mid.y, (double)c[m].y, pk);
                }
            }
        }
    }
    // The strip's core rows of the finished tile to memory.
    __device__ __forceinline__ void store(const float* L, GlobalPtr<float> out, int ly0, int gy0,
                                          int gx0, int nx, int ny, bool core_col) const {
        if (!core_col) return;
#pragma unroll
        for (int r = CORE0; r < CORE0 + CORES; ++r) {
            const int gy = gy0 + r;
            if (EDGE && gy >= ny) continue;
            const V v = *(const V*)&L[(ly0 + r) * kW];
            const GlobalPtr<float> dst = out + (size_t)gy * nx + gx0;
            if (ALIGNED) {
                if (!EDGE || gx0 < nx) *(GlobalPtr<RowVec<2>>)dst = RowVec<2>{v.x, v.y};
            } else {
                if (!EDGE || gx0 < nx) dst[0] = v.x;
                if (!EDGE || gx0 + 1 < nx) dst[1] = v.y;
            }
        }
    }
};

// ALIGNED: nx is even, so that a lane's two cells lie inside the grid's columns together and
// are loaded and stored as one 8-byte value.  CROWDED: many cones for the grid (crowded_grid).
template <bool ALIGNED, bool CROWDED>
__global__ __launch_bounds__(kThreads, 4) void k_field_reverse2d(ReverseArgs a) {
    __shared__ __align__(16) float tile_a[(kHL + 2) * kW];     // row ly at (ly + 1) * kW
    __shared__ __align__(16) unsigned long long sums[kHL * kW];
    __shared__ float4 cones[kRevSteps][kTileCones];   // (x, y, agx, agy), step t_hi - k in row k
    __shared__ double part[2][kWaves];
    if ((int)blockIdx.x >= a.grid.per_slice) {   // whole workgroup
        const int i = (blockIdx.x - a.grid.per_slice) * kThreads + threadIdx.x;
        if (i >= a.chain.tape.M || blockIdx.y > 0 || blockIdx.z > 0) return;
        if (a.n_species > 1)
            cone_chain<2, 2>(a.rules, a.chain, i, kRevSteps);
        else
            cone_chain<1, 2>(a.rules, a.chain, i, kRevSteps);
        return;
    }
    const int tile = a.grid.tile(blockIdx.x, blockIdx.z), s = blockIdx.y;
    if (tile >= a.n_tiles) return;   // whole workgroup: the barriers stay uniform
    const int2 place = tile_place(tile, a.tiles_x);
    const int tx = place.x, ty = place.y;
    const int x0 = tx * kTX - kH, y0 = ty * kTY - kH;
    const int nx = a.nx, ny = a.ny, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cx = kCPL * lane, gx0 = x0 + cx;
    const StencilCoef coef = a.coef[s];
    const float sign = s == 0 ? a.rules.sign0 : a.rules.sign1;
    float* const L = tile_a + kW + cx;   // the lane's cells of row 0

    // the ranges of the tile's cones and sources, and the tile's a (indices clamped into the
    // grid: cells outside are never read by cells inside)
    const int list_lo = tile > 0 ? a.list_end[tile - 1] : 0;
    const int n_list = a.list_end[tile] - list_lo;
    const int q_lo = a.q_start[s * (a.n_tiles + 1) + tile];
    const int n_q = a.q_start[s * (a.n_tiles + 1) + tile + 1] - q_lo;
    // the steps' scales, step t_hi - k in lane k
    const int max_bits = lane < a.steps ? (int)a.step_max[a.t_hi - lane] : 0;
    constexpr int kLoad = (kHL + kWaves - 1) / kWaves;
    RowVec<kCPL> in[kLoad];
#pragma unroll
    for (int r = 0; r < kLoad; ++r)
        in[r] = load_row<kCPL, ALIGNED>(gbl(a.a_in[s]), nx, ny,
                                        y0 + min(wave + r * kWaves, kHL - 1), gx0);
    for (int k = tid; k < kHL * kW / 2; k += kThreads)
        *(ulonglong2*)&sums[2 * k] = make_ulonglong2(0, 0);
    // a cone's tip and sample adjoint at step t, as (x, y, agx, agy)
    auto load_cone = [&](int i, int t) {
        const size_t at = (size_t)t * a.M + i;
        const float2 g = a.ag[at], x = *(const float2*)(a.tips + at);
        return make_float4(x.x, x.y, g.x, g.y);
    };
    // every step of the tile's first kTileCones cones, and this thread's source
    const int m0 = tid % kTileCones, k0 = tid / kTileCones;
    const int cone = m0 < n_list ? a.list[list_lo + m0] : -1;
    const int2 src = tid < n_q ? a.q_entry[q_lo + tid] : make_int2(-1, 0);
    double q_sum = 0.0;
    if (cone >= 0) {
        float4 p[kRevSteps / kShares];
#pragma unroll
        for (int u = 0; u < kRevSteps / kShares; ++u)
            p[u] = load_cone(cone, max(a.t_hi - (u * kShares + k0), 0));
#pragma unroll
        for (int u = 0; u < kRevSteps / kShares; ++u) cones[u * kShares + k0][m0] = p[u];
    }
#pragma unroll
    for (int r = 0; r < kLoad; ++r)   // (past the tile: its last row again)
        *(V*)&L[min(wave + r * kWaves, kHL - 1) * kW] = make_float2(in[r][0], in[r][1]);

    // the cones' contributions of sub-step k's step into the sums, and from there into the
    // tile: of all contributions to a cell the first to take its sum adds it, the others find
    // zero
    auto exponent = [&](int k) {
        return fixed_exponent((uint32_t)__builtin_amdgcn_readlane(max_bits, k));
    };
    // cells with a contribution of this thread waiting in the sums
    int mine[3] = {-1, -1, -1};
    const int my_cone = tid / kShares, my_share = tid % kShares;
    auto add = [&](const float4& p, int q, double scale, int (&at)[3]) {
        const Share c = share_of(a.rules, sign, p, q, x0, y0);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            // (a non-finite contribution, possible only from non-finite fields, adds nothing
            // rather than an undefined conversion)
            const double x = (double)c.v[k] * scale;
            const long long n = isfinite(x) ? (long long)rint(x) : 0;
            at[k] = n != 0 ? c.at[k] : -1;
            if (at[k] >= 0) atomicAdd(&sums[at[k]], (unsigned long long)n);
        }
    };
    auto add_cone = [&](const float4& p, double scale) __attribute__((always_inline)) {
        const Scatter2D c = sample_adjoint_2d(a.rules, p.x, p.y, sign * p.z, sign * p.w);
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            const int lx = c.i[k] - x0, ly = c.j[k] - y0;
            const double x = (double)c.v[k] * scale;
            const long long n = isfinite(x) ? (long long)rint(x) : 0;
            if (n != 0 && (unsigned)lx < (unsigned)kW && (unsigned)ly < (unsigned)kHL)
                atomicAdd(&sums[ly * kW + lx], (unsigned long long)n);
        }
    };
    auto take = [&](const int (&at)[3], double inv) {
        long long n[3];
        float v[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) n[k] = at[k] >= 0 ? (long long)atomicExch(&sums[at[k]], 0ull) : 0;
#pragma unroll
        for (int k = 0; k < 3; ++k) v[k] = n[k] != 0 ? tile_a[kW + at[k]] : 0.0f;
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (n[k] != 0) tile_a[kW + at[k]] = v[k] + (float)((double)n[k] * inv);
    };
    auto moving = [](const float4& p) { return p.z != 0.0f || p.w != 0.0f; };
    auto add_step = [&](int k) __attribute__((always_inline)) {
        const double scale = ldexp(1.0, kFixedBits - exponent(k));
        mine[0] = mine[1] = mine[2] = -1;
        if (my_cone < n_list) {
            const float4 p = cones[k][my_cone];
            if (moving(p)) add(p, my_share, scale, mine);
        }
        if (!CROWDED) {   // the tile's further cones, four threads each as well
            for (int m = kTileCones * kShares + tid; m < n_list * kShares; m += kThreads) {
                const float4 p = load_cone(a.list[list_lo + m / kShares], a.t_hi - k);
                int at[3];
                if (moving(p)) add(p, m % kShares, scale, at);
            }
        } else if (n_list > kTileCones + (tid & ~63)) {   // a thread each (whole wavefronts)
            // the next one's record and the number of the one after it travel meanwhile
            auto number = [&](int m) { return a.list[list_lo + min(m, n_list - 1)]; };
            int m = kTileCones + tid;
            float4 p = load_cone(number(m), a.t_hi - k);
            int i = number(m + kThreads);
            for (; m < n_list; m += kThreads) {
                const float4 q = load_cone(i, a.t_hi - k);
                i = number(m + 2 * kThreads);
                if (moving(p)) add_cone(p, scale);
                p = q;
            }
        }
    };
    auto take_step = [&](int k) __attribute__((always_inline)) {
        const double inv = ldexp(1.0, exponent(k) - kFixedBits);
        if (n_list <= kTileCones) {
            take(mine, inv);
            return;
        }
        // more cones than that: every cell of the tile is looked at
        for (int c = tid; c < kHL * kW / 2; c += kThreads) {
            const longlong2 n = *(longlong2*)&sums[2 * c];
            if (n.x == 0 && n.y == 0) continue;
            *(ulonglong2*)&sums[2 * c] = make_ulonglong2(0, 0);
            V v = *(V*)&tile_a[kW + 2 * c];
            if (n.x != 0) v.x += (float)((double)n.x * inv);
            if (n.y != 0) v.y += (float)((double)n.y * inv);
            *(V*)&tile_a[kW + 2 * c] = v;
        }
    };
    const bool core_col = cx >= kH && cx < kH + kTX;   // both cells (kH and kTX are even)
    double pD = 0.0, pk = 0.0;
    auto fields_at = [&](int t) {
        return gbl(a.fields + ((size_t)t * a.n_species + s) * a.cells);
    };
    // the sub-steps on this wavefront's strip, `ly0` its first row; every wavefront passes the
    // same barriers
    auto sweep = [&](auto strip, int ly0) __attribute__((always_inline)) {
        const int gy0 = y0 + ly0;
        strip.load_c(fields_at(a.t_hi), nx, ny, gy0, gx0);
        __syncthreads();
        for (int k = 0; k < a.steps; ++k) {
            const int t = a.t_hi - k;
            // the cones' adjoints of the step; the barrier also ends the strips' sub-step before
            if (n_list > 0) {
                add_step(k);
                __syncthreads();
                take_step(k);
                __syncthreads();
            } else if (k > 0) {
                __syncthreads();
            }
            // b^t is complete in the tile: its source cells, and this strip's rows
            if (src.x >= 0) q_sum += (double)tile_a[kW + src.x];
            for (int m = tid + kThreads; m < n_q; m += kThreads) {
                const int2 e = a.q_entry[q_lo + m];
                unsafeAtomicAdd(&a.acc_q[e.y], (double)tile_a[kW + e.x]);
            }
            strip.read(L, ly0);
            __syncthreads();
            strip.step(L, ly0, k, gy0, gx0, nx, ny, coef, core_col, pD, pk);
            // one sub-step ahead of its use
            if (k + 1 < a.steps) strip.load_c(fields_at(t - 1), nx, ny, gy0, gx0);
        }
        strip.store(L, gbl(a.a_out[s]), ly0, gy0, gx0, nx, ny, core_col);
    };
    auto by_wave = [&](auto edge) {
        constexpr bool EDGE = decltype(edge)::value;
        constexpr int kEdgeRows = kH + kEdgeCore;
        if (wave == 0)
            sweep(Strip<kEdgeRows, kH, kEdgeCore, ALIGNED, EDGE>{}, 0);
        else if (wave == kWaves - 1)
            sweep(Strip<kEdgeRows, 0, kEdgeCore, ALIGNED, EDGE>{}, kHL - kEdgeRows);
        else
            sweep(Strip<kMidCore, 0, kMidCore, ALIGNED, EDGE>{},
                  kEdgeRows + (wave - 1) * kMidCore);
    };
    if (x0 > 0 && x0 + kW < nx && y0 > 0 && y0 + kHL < ny)
        by_wave(std::false_type{});
    else
        by_wave(std::true_type{});
    pD = wave_sum(pD);
    pk = wave_sum(pk);
    if (lane == 63) {
        part[0][wave] = pD;
        part[1][wave] = pk;
    }
    __syncthreads();
    // every accumulator has one writer at a time (its tile, or its source's tile)
    if (tid < 2) {
        double sum = 0.0;
        for (int w = 0; w < kWaves; ++w) sum += part[tid][w];
        unsafeAtomicAdd(&(tid == 0 ? a.acc_D : a.acc_k)[s * a.n_tiles + tile], sum);
    }
    if (src.x >= 0) unsafeAtomicAdd(&a.acc_q[src.y], q_sum);
}

// -- which cones can touch a tile during a launch -----------------------------------------
// Launch g of a segment reverses its steps len - 1 - g kRevSteps downwards.

struct ListArgs {
    ConeRules rules;
    int M, len, tiles_x, tiles_y, cap;
    bool boxed;            // list the tiles of a cone's box (else of each of its samples)
    const float4* tips;    // [t][M]
    const float2* ag;      // [t][M]
    const float4* boxes;   // [launch][M]
    int32_t* list_end;     // [launch][tile]
    int32_t* list;         // [launch][cap]
};

// Tiles x1 .. x2 by y1 .. y2.
struct TileBox {
    int x1, x2, y1, y2;
    __device__ bool has(int tx, int ty) const {
        return tx >= x1 && tx <= x2 && ty >= y1 && ty <= y2;
    }
};

// Tiles along one axis whose loaded region holds a cell of [lo, hi].
__device__ __forceinline__ void tile_range(int lo, int hi, int core, int tiles, int& first,
                                           int& last) {
    first = max(lo - kH, 0) / core;
    last = min((hi + kH) / core, tiles - 1);
}

// Tiles whose loaded region meets the samples of tips from (xa, ya) to (xb, yb).
__device__ __forceinline__ TileBox tiles_of(const ListArgs& a, float xa, float xb, float ya,
                                            float yb) {
    int i0, i1, j0, j1;
    float f;
    corner(xa, a.rules.inv_dx, a.rules.nx, i0, f);
    corner(xb, a.rules.inv_dx, a.rules.nx, i1, f);
    corner(ya, a.rules.inv_dx, a.rules.ny, j0, f);
    corner(yb, a.rules.inv_dx, a.rules.ny, j1, f);
    TileBox b;
    tile_range(max(i0 - 1, 0), min(i1 + 2, a.rules.nx - 1), kTX, a.tiles_x, b.x1, b.x2);
    tile_range(max(j0 - 1, 0), min(j1 + 2, a.rules.ny - 1), kTY, a.tiles_y, b.y1, b.y2);
    return b;
}

// Calls each(tile) once for every tile that a sample of cone i touches in launch g (where cones
// move so far that a box would cover many tiles that no sample touches).
template <class Each>
__device__ __forceinline__ void for_touched_tiles(const ListArgs& a, int i, int g,
                                                  const Each& each) {
    const int t_hi = a.len - 1 - g * kRevSteps;
    TileBox seen[kRevSteps];
#pragma unroll
    for (int k = 0; k < kRevSteps; ++k) {
        seen[k] = TileBox{1, 0, 1, 0};
        if (t_hi - k < 0) continue;
        const size_t at = (size_t)(t_hi - k) * a.M + i;
        const float2 ag = a.ag[at], p = *(const float2*)(a.tips + at);
        if (ag.x == 0.0f && ag.y == 0.0f) continue;
        const TileBox b = tiles_of(a, p.x, p.x, p.y, p.y);
        seen[k] = b;
        for (int ty = b.y1; ty <= b.y2; ++ty)
            for (int tx = b.x1; tx <= b.x2; ++tx) {
                bool before = false;
#pragma unroll
                for (int m = 0; m < kRevSteps; ++m)
                    if (m < k) before = before || seen[m].has(tx, ty);
                if (!before) each(ty * a.tiles_x + tx);
            }
    }
}

// The lists of launch blockIdx.x, by one workgroup: cones counted per tile (in LDS where the
// tiles fit: device-wide atomics and a scan of their own took 37 us per 100-step segment at
// 8192 cones, this 16), the counts scanned to where each tile's cones start, and the cones put
// there; a tile's start becomes its end (the next tile's start).  A thread requests the boxes of
// kKeep cones together and keeps their tiles for the second pass (one cone after the other, read
// twice: 22 us).  The order of a tile's cones
// does not matter: their contributions are added as integers.
template <bool LDS>
__global__ __launch_bounds__(kListThreads) void k_tile_lists(ListArgs a) {
    extern __shared__ int32_t lds_count[];
    __shared__ int32_t wave_total[kListThreads / 64];
    const int g = blockIdx.x, n = a.tiles_x * a.tiles_y, tid = threadIdx.x;
    int32_t* const out = a.list_end + (size_t)g * n;
    int32_t* const count = LDS ? lds_count : out;
    int32_t* const list = a.list + (size_t)g * a.cap;
    auto get = [&](int k) {
        return LDS ? count[k]
                   : __hip_atomic_load(count + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto set = [&](int k, int32_t v) {
        if (LDS)
            count[k] = v;
        else
            __hip_atomic_store(count + k, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    for (int k = tid; k < n; k += kListThreads) set(k, 0);
    __syncthreads();
    // the tiles of the boxes of cones base + u * kListThreads + tid
    constexpr int kKeep = 8, kChunk = kKeep * kListThreads;
    TileBox kept[kKeep];
    auto keep = [&](int base) {
        float4 p[kKeep];
#pragma unroll
        for (int u = 0; u < kKeep; ++u)
            p[u] = a.boxes[(size_t)g * a.M + min(base + u * kListThreads + tid, a.M - 1)];
#pragma unroll
        for (int u = 0; u < kKeep; ++u) {
            const bool any = base + u * kListThreads + tid < a.M && p[u].x <= p[u].y;
            kept[u] = any ? tiles_of(a, p[u].x, p[u].y, p[u].z, p[u].w) : TileBox{1, 0, 1, 0};
        }
    };
    auto for_kept = [&](int base, auto each) {   // each(cone, tile)
#pragma unroll
        for (int u = 0; u < kKeep; ++u)
            for (int ty = kept[u].y1; ty <= kept[u].y2; ++ty)
                for (int tx = kept[u].x1; tx <= kept[u].x2; ++tx)
                    each(base + u * kListThreads + tid, ty * a.tiles_x + tx);
    };
    const int last = a.M > 0 ? (a.M - 1) / kChunk * kChunk : -1;   // the last chunk's first cone
    if (a.boxed) {
        for (int base = 0; base <= last; base += kChunk) {
            keep(base);
            for_kept(base, [&](int, int tile) { atomicAdd(&count[tile], 1); });
        }
    } else {
        for (int i = tid; i < a.M; i += kListThreads)
            for_touched_tiles(a, i, g, [&](int tile) { atomicAdd(&count[tile], 1); });
    }
    __syncthreads();
    const int lane = tid & 63, wave = tid >> 6;
    int32_t carry = 0;
    for (int base = 0; base < n; base += kListThreads) {
        const int k = base + tid;
        const int32_t v = k < n ? get(k) : 0;
        int32_t incl = v;
        for (int off = 1; off < 64; off <<= 1) {
            const int32_t y = __shfl_up(incl, off, 64);
            if (lane >= off) incl += y;
        }
        if (lane == 63) wave_total[wave] = incl;
        __syncthreads();
        int32_t at = carry + incl - v, total = 0;
        for (int w = 0; w < kListThreads / 64; ++w) {
            at += w < wave ? wave_total[w] : 0;
            total += wave_total[w];
        }
        if (k < n) set(k, at);
        carry += total;
        __syncthreads();   // every thread has read wave_total
    }
    auto put = [&](int i, int tile) {
        const int at = atomicAdd(&count[tile], 1);
        if (at < a.cap) list[at] = i;   // (the capacity holds every cone's most tiles)
    };
    if (a.boxed) {
        for (int base = last; base >= 0; base -= kChunk) {
            if (base != last) keep(base);
            for_kept(base, put);
        }
    } else {
        for (int i = tid; i < a.M; i += kListThreads)
            for_touched_tiles(a, i, g, [&](int tile) { put(i, tile); });
    }
    // (within the list's memory, whatever the tips: no entry past it was written)
    __syncthreads();
    for (int k = tid; k < n; k += kListThreads) out[k] = min(get(k), a.cap);
}

int tiles_along(int n, int core) { return (n + core - 1) / core; }

// Most tiles along one axis whose loaded regions meet a stretch of `cells` cells.
int tiles_touched(double cells, int core, int tiles) {
    const double n = (cells - 1.0 + 2.0 * kH) / core + 2.0;
    return n < tiles ? (int)n : tiles;
}

}  // namespace

int reverse_tiles(int nx, int ny) { return tiles_along(nx, kTX) * tiles_along(ny, kTY); }

// Whether a tile's loaded region holds so many cones on average that one thread should do all of a
// cone past the first kTileCones: four threads work out its share of the weights four times, but
// are done sooner where only the tiles at the sources hold that many.  Launch of eight steps, four
// threads / one: 1024^2 with 8192 cones 22.3 / 23.6 us, 27,000 (128 to a tile) 39.0 / 40.2, 55,000
// (255) 50.1 / 45.7, 110,000 79 / 59; 256^2 with 3500 23.9 / 24.3, 7000 (520) 35.5 / 31.2, 65,536
// 131 / 54.  (One kernel with both takes 24.3 us for the first of these.)  While such cones were
// added four threads each and taken from the sums by the same threads again: 23.0, 40.4, 60.6, 108,
// 25.6, 42.1 and 195; the sums in HBM before that needed 130 for the last.
static bool crowded_grid(int nx, int ny, int M) {
    return (double)M * kHL * kW > 1.5 * kTileCones * nx * ny;
}

ReverseGrid reverse_grid(int n_tiles) {
    constexpr int kSlice = 1 << 20;
    if (n_tiles <= kSlice) return ReverseGrid{1, (n_tiles + kXcds - 1) / kXcds * kXcds};
    return ReverseGrid{(n_tiles + kSlice - 1) / kSlice, kSlice};
}

int reverse_launches(int len) { return (len + kRevSteps - 1) / kRevSteps; }

// Most tiles a cone is listed for in one launch: the tiles that kRevSteps footprints of 4 x 4
// cells touch, each on its own (apart), or their box, which covers at most span + 6 cells
// along an axis (one for rounding) when the cone moves `span` cells.  The FP32 rounding of the
// kRevSteps - 1 moves and of both ends' cells, half a unit in the last place each, is up to
// (kRevSteps + 1) n 2^-24 cells on an axis of n: a tile more from some millions of cells on.
static void tiles_per_cone(int nx, int ny, double step_cells, size_t& apart, size_t& boxed) {
    const int tx = tiles_along(nx, kTX), ty = tiles_along(ny, kTY);
    const double cells = (kRevSteps - 1) * step_cells + 6;
    const double rounding = (kRevSteps + 1) * 0x1p-24;
    apart = (size_t)kRevSteps * tiles_touched(4, kTX, tx) * tiles_touched(4, kTY, ty);
    boxed = (size_t)tiles_touched(cells + nx * rounding, kTX, tx) *
            tiles_touched(cells + ny * rounding, kTY, ty);
}

size_t reverse_list_capacity(int nx, int ny, int M, double step_cells) {
    size_t apart, boxed;
    tiles_per_cone(nx, ny, step_cells, apart, boxed);
    return (size_t)M * std::min(apart, boxed);
}

void reverse_sources(int nx, int ny, const std::vector<int32_t>& cells, int first,
                     std::vector<int32_t>& start, std::vector<int2>& entry) {
    const int tiles_x = tiles_along(nx, kTX), n = reverse_tiles(nx, ny);
    std::vector<int32_t> at(n + 1, 0);
    auto tile_of = [&](int32_t cell) { return cell / nx / kTY * tiles_x + cell % nx / kTX; };
    for (int32_t cell : cells) at[tile_of(cell) + 1] += 1;
    for (int t = 0; t < n; ++t) at[t + 1] += at[t];
    const size_t base = entry.size();
    for (int t = 0; t <= n; ++t) start.push_back((int32_t)base + at[t]);
    entry.resize(base + cells.size());
    for (size_t m = 0; m < cells.size(); ++m) {
        const int x = cells[m] % nx % kTX + kH, y = cells[m] / nx % kTY + kH;
        entry[base + at[tile_of(cells[m])]++] = make_int2(y * kW + x, first + (int32_t)m);
    }
}

hipError_t launch_reverse_lists(const ReverseSegment& g, double step_cells, hipStream_t stream) {
    const int launches = reverse_launches(g.len);
    if (launches == 0) return hipSuccess;
    size_t apart, boxed;
    tiles_per_cone(g.nx, g.ny, step_cells, apart, boxed);
    ListArgs a = {};
    a.rules = g.rules;
    a.M = g.M;
    a.len = g.len;
    a.tiles_x = tiles_along(g.nx, kTX);
    a.tiles_y = tiles_along(g.ny, kTY);
    a.cap = (int)g.list_cap;
    a.boxed = boxed <= apart;
    a.tips = g.tape.base;   // plane 0
    a.ag = g.ag;
    a.boxes = g.boxes;
    a.list_end = g.list_end;
    a.list = g.list;
    const int n = a.tiles_x * a.tiles_y;
    if (n <= kListTiles) {
        const size_t bytes = (size_t)n * sizeof(int32_t);
        const hipError_t e = hipFuncSetAttribute((const void*)k_tile_lists<true>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 (int)(kListTiles * sizeof(int32_t)));
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_tile_lists<true>, dim3(launches), dim3(kListThreads), bytes, stream,
                           a);
    } else {
        hipLaunchKernelGGL(k_tile_lists<false>, dim3(launches), dim3(kListThreads), 0, stream, a);
    }
    return hipGetLastError();
}

hipError_t launch_field_reverse2d(const ReverseSegment& g, int launch, const float* const* a_in,
                                  float* const* a_out, const ConeChain* chain,
                                  hipStream_t stream) {
    ReverseArgs a = {};
    a.tiles_x = tiles_along(g.nx, kTX);
    a.n_tiles = reverse_tiles(g.nx, g.ny);
    for (int s = 0; s < g.n_species; ++s) {
        a.a_in[s] = a_in[s];
        a.a_out[s] = a_out[s];
        a.coef[s] = g.coef[s];
    }
    a.rules = g.rules;
    a.fields = g.fields;
    a.cells = (size_t)g.nx * g.ny;
    a.n_species = g.n_species;
    a.nx = g.nx;
    a.ny = g.ny;
    a.grid = reverse_grid(a.n_tiles);
    a.t_hi = g.len - 1 - launch * kRevSteps;
    a.steps = std::min(kRevSteps, a.t_hi + 1);
    a.M = g.M;
    a.tips = g.tape.base;   // plane 0
    a.ag = g.ag;
    a.step_max = g.step_max;
    a.list_end = g.list_end + (size_t)launch * a.n_tiles;
    a.list = g.list + (size_t)launch * g.list_cap;
    a.acc_D = g.acc_D;
    a.acc_k = g.acc_k;
    a.q_start = g.q_start;
    a.q_entry = g.q_entry;
    a.acc_q = g.acc_q;
    int chain_wgs = 0;
    if (chain) {
        a.chain = *chain;
        chain_wgs = (chain->tape.M + kThreads - 1) / kThreads;
    }
    const dim3 grid(a.grid.per_slice + chain_wgs, g.n_species, a.grid.slices);
    const bool crowded = crowded_grid(g.nx, g.ny, g.M);
    auto* const kernel = g.nx % 2 == 0 ? crowded ? k_field_reverse2d<true, true>
                                                 : k_field_reverse2d<true, false>
                         : crowded     ? k_field_reverse2d<false, true>
                                       : k_field_reverse2d<false, false>;
    hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, stream, a);
    return hipGetLastError();
}

}  // namespace cuesim
