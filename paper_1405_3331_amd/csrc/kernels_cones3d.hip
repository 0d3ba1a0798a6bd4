// kernels_cones3d.hip -- the 3D cone step over cones held in spatial order.
//
// A 3D cone samples 32 cells per species around its tip (Sec. 3.5 gradient steering; trilinear).  In
// the caller's order neighbouring threads sit anywhere in the volume, so a wavefront touches
// a separate set of cache lines per cone and uses a few bytes of each.  Here the active
// cones are kept sorted by where their tips are (order_key): a workgroup then covers one
// compact region, its gathers share lines in L1/L2, and the cone state itself streams as two
// aligned float4 per cone (tip x, y, z, id; heading).
// Cones move at most step_len per step, so the order is refreshed every few steps (the
// project's stable counting sort of the keys, kernels_sort.hip, then a gather of the state),
// not every step.
//
// Stopped cones leave the order: the step writes their final tip, heading, status, target
// and event step straight into the caller-order arrays and marks the ordered copy id = -1;
// a refresh moves them behind the active ones.  The caller-order tips and headings of the
// active cones are brought up to date only when the state is read (order3d_end).
//
// Times below are pairs (or more) of variants from one state each, and states differ: as the cones
// gather and stop, a 256^3 step with two species and 262,144 cones takes 114 us over a run's first
// 100 steps, 105 over its fourth and 110 over its eighth; 97 x 64 x 51 with 3000 cones 14.8 down to
// 10.7 over six.
#include "field_step.hpp"
#include "internal.hpp"
#include "memory.hpp"

namespace cuesim {

namespace {

constexpr int kThreads = 256;
// The cone step's workgroups are single wavefronts (nothing is shared between them), eight per
// CU (32 CUs per die), each walking several blocks of its die's stretch, so that a die works
// on a region of the fields its L2 can hold.  Per 256^3 step (field 49 us): 108-110 us, against
// 112 with four, 112 with twelve and 115 with sixteen per CU, and 112 with two workgroups of
// four wavefronts per CU.
constexpr int kConeThreads = 64;
constexpr int kConeWgsPerXcd = 32 * 8;

// Order key of a tip: the Morton code of its (y, z) block of 8 x 8 cells, then its 32-cell run
// along x, a line of the field: a wavefront's cones share lines.  Step against 8-cell Morton
// cubes: 128^3, two species, 262,144 cones 28.5 us (30.4), 160^3 39.1 (41.3), 256^3 95.3 (95.8);
// with 64-cell runs 30.3, 40.2 and 95.3.  Bits past kXBits, kYZBits are dropped: the order of
// a larger volume is only less compact.
constexpr int kRunShift = 5, kBlockShift = 3, kXBits = 6, kYZBits = 12;

__host__ __device__ __forceinline__ uint32_t spread2(uint32_t v) {   // kYZBits bits -> every second bit
    v &= (1u << kYZBits) - 1u;
    v = (v | (v << 8)) & 0x00ff00ffu;
    v = (v | (v << 4)) & 0x0f0f0f0fu;
    v = (v | (v << 2)) & 0x33333333u;
    v = (v | (v << 1)) & 0x55555555u;
    return v;
}

__host__ __device__ __forceinline__ uint32_t cell_key(uint32_t x, uint32_t y, uint32_t z,
                                                      int x_bits) {
    return (spread2(y >> kBlockShift) | spread2(z >> kBlockShift) << 1) << x_bits |
           ((x >> kRunShift) & ((1u << x_bits) - 1u));
}

// Cell of a coordinate, clamped to the grid (as a float first: a NaN tip maps to cell 0).
__device__ __forceinline__ uint32_t cell_coord(float p, float inv_dx, int n) {
    return (uint32_t)fminf(fmaxf(floorf(p * inv_dx), 0.0f), (float)(n - 1));
}

__device__ __forceinline__ uint32_t order_key(const ConeRules& r, float x, float y, float z,
                                              int x_bits) {
    return cell_key(cell_coord(x, r.inv_dx, r.nx), cell_coord(y, r.inv_dx, r.ny),
                    cell_coord(z, r.inv_dx, r.nz), x_bits);
}

// Caller order -> (tip, heading) with keys; inactive cones get id -1 and the key past every
// active one.
__global__ __launch_bounds__(kThreads) void k_pack3d(ConeRules r, ConeArrays c, float4* tip,
                                                     float4* dir, uint32_t* key, int32_t* slot,
                                                     int x_bits, uint32_t inactive) {
    const int i = blockIdx.x * kThreads + threadIdx.x;
    if (i >= c.n) return;
    const float x = c.pos[3 * i], y = c.pos[3 * i + 1], z = c.pos[3 * i + 2];
    const bool active = c.status[i] == kActive;
    tip[i] = make_float4(x, y, z, __int_as_float(active ? i : -1));
    dir[i] = make_float4(c.dir[3 * i], c.dir[3 * i + 1], c.dir[3 * i + 2], 0.0f);
    key[i] = active ? order_key(r, x, y, z, x_bits) : inactive;
    slot[i] = i;
}

__global__ __launch_bounds__(kThreads) void k_keys3d(ConeRules r, const float4* __restrict__ tip,
                                                     int n, uint32_t* key, int32_t* slot,
                                                     int x_bits, uint32_t inactive) {
    const int t = blockIdx.x * kThreads + threadIdx.x;
    if (t >= n) return;
    const float4 p = tip[t];
    key[t] = __float_as_int(p.w) >= 0 ? order_key(r, p.x, p.y, p.z, x_bits) : inactive;
    slot[t] = t;
}

__global__ __launch_bounds__(kThreads) void k_gather3d(const int32_t* __restrict__ slot, int n,
                                                       const float4* __restrict__ tip_in,
                                                       const float4* __restrict__ dir_in,
                                                       float4* __restrict__ tip_out,
                                                       float4* __restrict__ dir_out) {
    const int t = blockIdx.x * kThreads + threadIdx.x;
    if (t >= n) return;
    const int s = slot[t];
    tip_out[t] = tip_in[s];
    dir_out[t] = dir_in[s];
}

struct Global3D {
    const float* f;
    int nx, ny;
    __device__ float operator()(int i, int j, int l) const { return f[(l * ny + j) * nx + i]; }
};

// The 3D gradient footprint of one species read row by row: each of the four rows
// (j0 + b, l0 + c) with four cells (im, i0, i0 + 1, ip) is one 16-byte load of the cells
// [s, s + 4), s = clamp(i0 - 1, 0, nx - 4), from which the four values are picked (at a wall
// the clamped indices repeat a cell, exactly as the per-cell accessor reads it); the other
// eight rows hold two adjacent cells each.  Needs nx >= 4.
__device__ __forceinline__ Footprint3D load_footprint_3d_rows(const float* __restrict__ f,
                                                              const ConeRules& r,
                                                              const Corner3D& k) {
    Footprint3D p;
    const size_t nx = (size_t)r.nx, plane = nx * (size_t)r.ny;
    const int s = min(max(k.i0 - 1, 0), r.nx - 4);
    const int am = k.im - s, a0 = k.i0 - s, ap = k.ip - s;
    auto row4 = [&](int j, int l) {
        float4 v;
        __builtin_memcpy(&v, f + (size_t)l * plane + (size_t)j * nx + s, sizeof v);
        return v;
    };
    auto pick = [](const float4& v, int i) {
        return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w;
    };
    auto row2 = [&](int j, int l) {
        float2 v;
        __builtin_memcpy(&v, f + (size_t)l * plane + (size_t)j * nx + k.i0, sizeof v);
        return v;
    };
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const float4 v = row4(k.j0 + b, k.l0 + c);
            p.xm[b][c] = pick(v, am);
            p.blk[0][b][c] = pick(v, a0);
            p.blk[1][b][c] = pick(v, a0 + 1);
            p.xp[b][c] = pick(v, ap);
        }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const float2 ym = row2(k.jm, k.l0 + c), yp = row2(k.jp, k.l0 + c);
        p.ym[0][c] = ym.x;
        p.ym[1][c] = ym.y;
        p.yp[0][c] = yp.x;
        p.yp[1][c] = yp.y;
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const float2 zm = row2(k.j0 + b, k.lm), zp = row2(k.j0 + b, k.lp);
        p.zm[0][b] = zm.x;
        p.zm[1][b] = zm.y;
        p.zp[0][b] = zp.x;
        p.zp[1][b] = zp.y;
    }
    return p;
}

// One step of ordered cone t against the updated fields.
template <int NS>
__device__ __forceinline__ void step_ordered_cone(const ConeRules& r, const float* f0,
                                                  const float* f1, float4* tip, float4* dir,
                                                  const ConeArrays& c, uint32_t step, int t) {
    const float4 p = tip[t];
    const int id = __float_as_int(p.w);
    if (id < 0) return;
    const float4 h = dir[t];
    float x = p.x, y = p.y, z = p.z, hx = h.x, hy = h.y, hz = h.z;
    const Corner3D k = corner_3d(r, x, y, z);
    // The deviates need the cone's id only: with one species they are worked out while the
    // footprint travels (97 x 64 x 51: 11.0 -> 10.7 us per step).  With two, keeping them through
    // both gradients costs registers and spills (256^3: 103.5 -> 105.2), so they come last.
    float gx, gy, gz, zn[3];
    if (r.nx >= 4) {
        const Footprint3D fp = load_footprint_3d_rows(f0, r, k);
        if (NS == 1) {
            normals<3>(r.key, (uint32_t)id, step, zn);
            __builtin_amdgcn_sched_barrier(0);
        }
        gradient_from_3d(r, k, fp, gx, gy, gz);
    } else {
        if (NS == 1) normals<3>(r.key, (uint32_t)id, step, zn);
        gradient_from_3d(r, k, load_footprint_3d(Global3D{f0, r.nx, r.ny}, k), gx, gy, gz);
    }
    gx *= r.sign0;
    gy *= r.sign0;
    gz *= r.sign0;
    if (NS > 1) {
        float ax, ay, az;
        if (r.nx >= 4)
            gradient_from_3d(r, k, load_footprint_3d_rows(f1, r, k), ax, ay, az);
        else
            gradient_from_3d(r, k, load_footprint_3d(Global3D{f1, r.nx, r.ny}, k), ax, ay,
                             az);
        gx = fmaf(r.sign1, ax, gx);
        gy = fmaf(r.sign1, ay, gy);
        gz = fmaf(r.sign1, az, gz);
    }
    if (NS > 1) normals<3>(r.key, (uint32_t)id, step, zn);
    const ConeEvent ev = cone_step_3d(r, gx, gy, gz, zn, x, y, z, hx, hy, hz,
                                      GridContact{&r.targets});
    dir[t] = make_float4(hx, hy, hz, 0.0f);
    if (ev.status == kActive) {
        tip[t] = make_float4(x, y, z, p.w);
        return;
    }
    tip[t] = make_float4(x, y, z, __int_as_float(-1));
    c.pos[3 * id] = x;
    c.pos[3 * id + 1] = y;
    c.pos[3 * id + 2] = z;
    c.dir[3 * id] = hx;
    c.dir[3 * id + 1] = hy;
    c.dir[3 * id + 2] = hz;
    c.status[id] = ev.status;
    c.target[id] = ev.target;
    c.event_step[id] = (int32_t)(step + 1);
}

// One step of every ordered cone.  The blocks of kConeThreads cones are split into one
// contiguous stretch of the order per accelerator die (workgroups are dealt to the dies
// round-robin), so a die works on one compact region of the fields; when there are more
// blocks than workgroups, the workgroups of a die walk its stretch block after block.  (Loading
// both species' footprints before combining either was measured slower: the wider register
// live range costs more than the extra loads in flight gain.)
template <int NS>
__global__ __launch_bounds__(kConeThreads) void k_cones3d_ordered(ConeRules r,
                                                              const float* __restrict__ f0,
                                                              const float* __restrict__ f1,
                                                              float4* tip, float4* dir, int n,
                                                              int per_xcd, ConeArrays c,
                                                              uint32_t step) {
    const int xcd = blockIdx.x % kXcds;
    const int wgs_per_xcd = gridDim.x / kXcds;
    for (int b = blockIdx.x / kXcds; b < per_xcd; b += wgs_per_xcd) {
        const int t = (xcd * per_xcd + b) * kConeThreads + threadIdx.x;
        if (t < n) step_ordered_cone<NS>(r, f0, f1, tip, dir, c, step, t);
    }
}

// Cones per workgroup of k_step3d: one wavefront of its eight where the cones are few, so that
// every CU gets some (a wavefront's loads go to 64 lines each, and through one CU one after the
// other), or where the fields are past the L2s, which more cones at once would thrash; every
// wavefront where neither holds.  Step with one / eight: 128^3, one species, 32,768 cones 10.9 /
// 13.5 us; 160^3, 65,536 14.6 / 15.3; 128^3, two species, 262,144 34.9 / 30.3; 256^3 98.5 / 108.
constexpr int kSpreadCones = 4 * 256 * 64;
constexpr int64_t kL2Bytes = (int64_t)kXcds * 4 << 20;

// One step's cones and the next field step, which only read the fields as they are between
// them, so one launch and one round of latency serve both.  A die's first cone_wgs workgroups
// take its stretch of the cones, per_wg at a time, and start while all its CUs are free; its
// boxes follow (spread evenly among them they took 120 us of a 256^3 step instead of 107).  At
// 80 registers, for the boxes' occupancy.  Against two launches per step: 97 x 64 x 51, 3000
// cones 12.7 -> 9.7 us; 128^3, one species, 32,768 cones 16.3 -> 10.6; 200^3, 4096 22.5 -> 16.7;
// 256^3, two species, 262,144 100.5 -> 95.3, where the cones are bound by the lines they miss in
// L2 (250 to 330 MB, beside the field's 270 MB).
template <int NS>
__global__ __launch_bounds__(kBoxThreads3D, 6) void k_step3d(ConeRules r, float4* tip,
                                                             float4* dir, int n, int cone_wgs,
                                                             int per_wg, ConeArrays c,
                                                             uint32_t step, Field3DArgs a) {
    const int xcd = blockIdx.x % kXcds, k = blockIdx.x / kXcds;
    if (k < cone_wgs) {
        const int t = (xcd * cone_wgs + k) * per_wg + threadIdx.x;
        if ((int)threadIdx.x < per_wg && t < n)
            step_ordered_cone<NS>(r, a.in[0], a.in[NS - 1], tip, dir, c, step, t);
        return;
    }
    const int box = xcd * a.per_xcd + (k - cone_wgs);
    if (box < a.n_species * a.tx * a.ty * a.tz) field3d_box(a, box, threadIdx.x);
}

__global__ __launch_bounds__(kThreads) void k_unpack3d(const float4* __restrict__ tip,
                                                       const float4* __restrict__ dir, int n,
                                                       ConeArrays c) {
    const int t = blockIdx.x * kThreads + threadIdx.x;
    if (t >= n) return;
    const float4 p = tip[t];
    const int id = __float_as_int(p.w);
    if (id < 0) return;
    const float4 h = dir[t];
    c.pos[3 * id] = p.x;
    c.pos[3 * id + 1] = p.y;
    c.pos[3 * id + 2] = p.z;
    c.dir[3 * id] = h.x;
    c.dir[3 * id + 1] = h.y;
    c.dir[3 * id + 2] = h.z;
}

int blocks_for(int n) { return (n + kThreads - 1) / kThreads; }

int axis_bits(int n, int shift, int most) {
    int bits = 0;
    while (bits < most && ((n - 1) >> shift) >= (1 << bits)) ++bits;
    return bits;
}

// Stable counting sort of (key, slot) (buffers 0 and 1 ping-pong), then the state gather
// into the other half of the state's ping-pong.
hipError_t sort_and_gather(ConeOrder3D& o, hipStream_t stream) {
    bool in_alt = false;
    hipError_t e = sort_pairs(o.key[0], o.slot[0], o.key[1], o.slot[1], o.n, o.end_bit,
                              o.scratch, stream, &in_alt);
    if (e != hipSuccess) return e;
    const int nxt = o.cur ^ 1;
    hipLaunchKernelGGL(k_gather3d, dim3(blocks_for(o.n)), dim3(kThreads), 0, stream,
                       o.slot[in_alt ? 1 : 0], o.n, o.tip[o.cur], o.dir[o.cur], o.tip[nxt],
                       o.dir[nxt]);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    o.cur = nxt;
    return hipSuccess;
}

}  // namespace

hipError_t order3d_allocate(ConeOrder3D& o, int n, int nx, int ny, int nz) {
    o = ConeOrder3D{};
    o.n = n;
    o.x_bits = axis_bits(nx, kRunShift, kXBits);
    // past the far corner's key, the largest where no bits are dropped
    const bool whole = axis_bits(ny, kBlockShift, kYZBits + 1) <= kYZBits &&
                       axis_bits(nz, kBlockShift, kYZBits + 1) <= kYZBits &&
                       axis_bits(nx, kRunShift, kXBits + 1) <= kXBits;
    o.inactive = whole ? cell_key(nx - 1, ny - 1, nz - 1, o.x_bits) + 1
                       : 1u << (2 * kYZBits + o.x_bits);
    for (o.end_bit = 1; o.inactive >> o.end_bit != 0; ++o.end_bit) {
    }
    if (n == 0) return hipSuccess;
    auto padded = [](size_t bytes) { return (bytes + 255) / 256 * 256; };
    const size_t state = padded((size_t)n * sizeof(float4)), word = padded((size_t)n * 4);
    const hipError_t e = device_malloc((void**)&o.memory, 4 * state + 4 * word +
                                                              sort_pairs_scratch_bytes(n));
    if (e != hipSuccess) return e;
    char* at = o.memory;
    for (int b = 0; b < 2; ++b) {
        o.tip[b] = (float4*)at;
        o.dir[b] = (float4*)(at + state);
        at += 2 * state;
    }
    for (int b = 0; b < 2; ++b) {
        o.key[b] = (uint32_t*)at;
        o.slot[b] = (int32_t*)(at + word);
        at += 2 * word;
    }
    o.scratch = (int32_t*)at;
    return hipSuccess;
}

void order3d_release(ConeOrder3D& o) {
    device_free(o.memory);
    o = ConeOrder3D{};
}

hipError_t order3d_begin(ConeOrder3D& o, const ConeRules& r, ConeArrays cones,
                         hipStream_t stream) {
    if (o.n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_pack3d, dim3(blocks_for(o.n)), dim3(kThreads), 0, stream, r, cones,
                       o.tip[o.cur], o.dir[o.cur], o.key[0], o.slot[0], o.x_bits, o.inactive);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return sort_and_gather(o, stream);
}

hipError_t order3d_refresh(ConeOrder3D& o, const ConeRules& r, hipStream_t stream) {
    if (o.n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_keys3d, dim3(blocks_for(o.n)), dim3(kThreads), 0, stream, r,
                       o.tip[o.cur], o.n, o.key[0], o.slot[0], o.x_bits, o.inactive);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return sort_and_gather(o, stream);
}

hipError_t launch_cones3d_ordered(const ConeRules& r, const float* f0, const float* f1,
                                  ConeOrder3D& o, ConeArrays cones, uint32_t step,
                                  hipStream_t stream) {
    if (o.n == 0) return hipSuccess;
    const int blocks = (o.n + kConeThreads - 1) / kConeThreads;
    const int per_xcd = (blocks + kXcds - 1) / kXcds;
    const int wgs_per_xcd = std::min(per_xcd, kConeWgsPerXcd);
    if (r.n_species > 1)
        hipLaunchKernelGGL(k_cones3d_ordered<2>, dim3(wgs_per_xcd * kXcds), dim3(kConeThreads), 0,
                           stream, r, f0, f1, o.tip[o.cur], o.dir[o.cur], o.n, per_xcd, cones,
                           step);
    else
        hipLaunchKernelGGL(k_cones3d_ordered<1>, dim3(wgs_per_xcd * kXcds), dim3(kConeThreads), 0,
                           stream, r, f0, f1, o.tip[o.cur], o.dir[o.cur], o.n, per_xcd, cones,
                           step);
    return hipGetLastError();
}

hipError_t launch_step3d(const ConeRules& r, ConeOrder3D& o, ConeArrays cones, uint32_t step,
                         const Field3DArgs& next, hipStream_t stream) {
    const int64_t bytes = (int64_t)next.n_species * next.nx * next.ny * next.nz * 4;
    // (one wavefront in eight of a launch of fewer than 2^32 threads holds 2^28 cones)
    const bool dense = (o.n > kSpreadCones && bytes <= kL2Bytes) || o.n > 1 << 28;
    const int per_wg = dense ? kBoxThreads3D : 64;
    const int cone_wgs = (o.n + per_wg * kXcds - 1) / (per_wg * kXcds);
    const dim3 grid((next.per_xcd + cone_wgs) * kXcds);
    if (r.n_species > 1)
        hipLaunchKernelGGL(k_step3d<2>, grid, dim3(kBoxThreads3D), 0, stream, r, o.tip[o.cur],
                           o.dir[o.cur], o.n, cone_wgs, per_wg, cones, step, next);
    else
        hipLaunchKernelGGL(k_step3d<1>, grid, dim3(kBoxThreads3D), 0, stream, r, o.tip[o.cur],
                           o.dir[o.cur], o.n, cone_wgs, per_wg, cones, step, next);
    return hipGetLastError();
}

hipError_t order3d_end(const ConeOrder3D& o, ConeArrays cones, hipStream_t stream) {
    if (o.n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_unpack3d, dim3(blocks_for(o.n)), dim3(kThreads), 0, stream,
                       o.tip[o.cur], o.dir[o.cur], o.n, cones);
    return hipGetLastError();
}

}  // namespace cuesim
