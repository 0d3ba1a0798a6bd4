// kernels_plain.hip -- the parts of an un-blocked 2D step besides the field update: the
// cones, one thread each in the caller's order, against the just-updated fields, alone or with
// the next field step in their launch; the near map of a target grid; and the FP64 mass of a
// field.
#include <hip/hip_ext.h>

#include <algorithm>

#include "field_step.hpp"
#include "internal.hpp"

namespace cuesim {

namespace {

struct Global2D {
    const float* f;
    int nx;
    __device__ float operator()(int i, int j) const { return f[j * nx + i]; }
};

// Step of cone i.  RECORD: what the reverse needs of it goes to step t of the run's cone tape.
template <bool RECORD>
__device__ __forceinline__ void step_cone(const ConeRules& r, const float* __restrict__ f0,
                                          const float* __restrict__ f1, const ConeArrays& c,
                                          uint32_t step, const ConeTape& tape, size_t t, int i) {
    if (i >= c.n || c.status[i] != kActive) return;
    float x = c.pos[2 * i], y = c.pos[2 * i + 1], th = c.dir[i];
    float gx, gy, conc = 0.0f;
    const Footprint2D p0 = footprint_2d(Global2D{f0, r.nx}, r, x, y);
    const CornerGradients2D g0 = corner_gradients_2d(p0, r);
    gradient_from_2d(p0, g0, gx, gy, r.turn_law == 1 ? &conc : nullptr);
    if (RECORD) tape.sample(0, t, i, g0);
    gx *= r.sign0;
    gy *= r.sign0;
    if (r.n_species > 1) {
        float hx, hy;
        const Footprint2D p1 = footprint_2d(Global2D{f1, r.nx}, r, x, y);
        const CornerGradients2D g1 = corner_gradients_2d(p1, r);
        gradient_from_2d(p1, g1, hx, hy, nullptr);
        if (RECORD) tape.sample(1, t, i, g1);
        gx = fmaf(r.sign1, hx, gx);
        gy = fmaf(r.sign1, hy, gy);
    }
    if (RECORD) tape.put(2, t, i, make_float4(gx, gy, p0.fx, p0.fy));
    float sn, cs;
    sincos_angle(th, sn, cs);
    const float x0 = x, y0 = y, s0 = sn, c0 = cs;
    float z[2];
    noise_2d(r.key, (uint32_t)i, step, z);
    const ConeEvent ev = cone_step_2d(r, gx, gy, conc, z, x, y, th, sn, cs,
                                      GridContact{&r.targets});
    if (RECORD) record_turn(tape, t, i, r, x0, y0, s0, c0, gx, gy, sn, cs);
    c.pos[2 * i] = x;
    c.pos[2 * i + 1] = y;
    c.dir[i] = th;
    if (ev.status != kActive) {
        c.status[i] = ev.status;
        c.target[i] = ev.target;
        c.event_step[i] = (int32_t)(step + 1);
    }
}

template <bool RECORD>
__global__ __launch_bounds__(256) void k_cones2d(ConeRules r, const float* __restrict__ f0,
                                                 const float* __restrict__ f1, ConeArrays c,
                                                 uint32_t step, ConeTape tape, size_t t) {
    step_cone<RECORD>(r, f0, f1, c, step, tape, t, blockIdx.x * 256 + threadIdx.x);
}

// One step's cones (the first cone_wgs workgroups, a multiple of the dies) and the next field
// step: both only read the fields as they are between them, so one launch and one round of
// latency serve both (1203 x 901, one species, 10.3 -> 6.0 us per step).
__global__ __launch_bounds__(256) void k_step2d(ConeRules r, ConeArrays c, uint32_t step,
                                                int cone_wgs, Field2DStepArgs a) {
    const int wg = blockIdx.x;
    if (wg < cone_wgs) {
        step_cone<false>(r, a.in[0], a.in[r.n_species > 1 ? 1 : 0], c, step, ConeTape{}, 0,
                         wg * 256 + threadIdx.x);
        return;
    }
    const int box = (wg % kXcds) * a.per_xcd + (wg - cone_wgs) / kXcds;
    if (box < a.n_species * a.tx * a.ty) field2d_box(a, box, threadIdx.x);
}

// Marks in the near map every cell that a tip in range of target blockIdx.x * 256 + threadIdx.x
// can lie in: the cells that meet the contact ball, widened by kCellSlack cells for the FP32
// rounding of a tip's cell and distance.
template <int dim>
__global__ __launch_bounds__(256) void k_near_map(TargetGrid tg, uint32_t* near, int n_targets) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= n_targets) return;
    const float4 p = tg.pts[t];
    const double inv = tg.near_inv, reach = (double)tg.r * inv + kCellSlack;
    const double c[3] = {p.x * inv, p.y * inv, dim == 3 ? p.z * inv : 0.0};
    const int n[3] = {tg.near_nx, tg.near_ny, tg.near_nz};
    int lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0};
    for (int a = 0; a < dim; ++a) {
        lo[a] = (int)fmin(fmax(floor(c[a] - reach - kCellSlack), 0.0), (double)n[a]);
        hi[a] = (int)fmin(fmax(floor(c[a] + reach + kCellSlack), -1.0), (double)(n[a] - 1));
    }
    for (int z = lo[2]; z <= hi[2]; ++z)
        for (int y = lo[1]; y <= hi[1]; ++y)
            for (int x = lo[0]; x <= hi[0]; ++x) {
                const int cell[3] = {x, y, z};
                double d2 = 0.0;   // squared distance of the widened cell from the target
                for (int a = 0; a < dim; ++a) {
                    const double d = fmax(fmax(cell[a] - kCellSlack - c[a],
                                               c[a] - (cell[a] + 1 + kCellSlack)), 0.0);
                    d2 += d * d;
                }
                if (d2 > reach * reach) continue;
                uint32_t bit;
                const size_t word = near_word<dim>(tg, x, y, z, bit);
                atomicOr(&near[word], bit);
            }
}

// FP64 sum: each block reduces a grid-stride slice (wavefront shuffles, then LDS), the
// second pass adds the block partials in a fixed order, so the result is deterministic.
constexpr int kMassThreads = 256;

__device__ double block_sum(double v) {
    __shared__ double part[kMassThreads / 64];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) part[wave] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < kMassThreads / 64; ++w) t += part[w];
    return t;
}

__global__ __launch_bounds__(kMassThreads) void k_mass_partial(const float* __restrict__ f,
                                                                int64_t n,
                                                                double* __restrict__ partial) {
    double acc = 0.0;
    for (int64_t x = (int64_t)blockIdx.x * kMassThreads + threadIdx.x; x < n;
         x += (int64_t)gridDim.x * kMassThreads)
        acc += (double)f[x];
    const double t = block_sum(acc);
    if (threadIdx.x == 0) partial[blockIdx.x] = t;
}

// The total goes to *out; a non-finite total also raises *nonfinite (when given).
__global__ __launch_bounds__(kMassThreads) void k_mass_final(const double* __restrict__ partial,
                                                              int n, double* __restrict__ out,
                                                              int32_t* __restrict__ nonfinite) {
    double acc = 0.0;
    for (int x = threadIdx.x; x < n; x += kMassThreads) acc += partial[x];
    const double t = block_sum(acc);
    if (threadIdx.x == 0) {
        *out = t;
        if (nonfinite && !isfinite(t)) *nonfinite = 1;
    }
}

// Several device-to-device copies in one launch (a checkpoint's field and cone arrays):
// word w of the concatenated spans, in 4-byte words, by a grid-stride loop.
__global__ __launch_bounds__(256) void k_copy_spans(CopySpans c) {
    const size_t total = c.word_end[c.n - 1];
    for (size_t w = (size_t)blockIdx.x * 256 + threadIdx.x; w < total;
         w += (size_t)gridDim.x * 256) {
        int k = 0;
        while (w >= c.word_end[k]) ++k;
        const size_t off = w - (k > 0 ? c.word_end[k - 1] : 0);
        ((uint32_t*)c.dst[k])[off] = ((const uint32_t*)c.src[k])[off];
    }
}

}  // namespace

hipError_t launch_copy_spans(const CopySpans& c, hipStream_t stream) {
    if (c.n <= 0 || c.word_end[c.n - 1] == 0) return hipSuccess;
    const size_t total = c.word_end[c.n - 1];
    const int blocks = (int)std::min<size_t>((total + 255) / 256, 2048);
    hipLaunchKernelGGL(k_copy_spans, dim3(blocks), dim3(256), 0, stream, c);
    return hipGetLastError();
}

hipError_t launch_cones2d(const ConeRules& rules, const float* f0, const float* f1,
                          ConeArrays cones, uint32_t step, hipStream_t stream,
                          const ConeTape* tape, size_t t) {
    if (cones.n == 0) return hipSuccess;
    const dim3 grid((cones.n + 255) / 256);
    if (tape)
        hipLaunchKernelGGL(k_cones2d<true>, grid, dim3(256), 0, stream, rules, f0, f1, cones,
                           step, *tape, t);
    else
        hipLaunchKernelGGL(k_cones2d<false>, grid, dim3(256), 0, stream, rules, f0, f1, cones,
                           step, ConeTape{}, (size_t)0);
    return hipGetLastError();
}

hipError_t launch_step2d(const ConeRules& rules, ConeArrays cones, uint32_t step,
                         const Field2DStepArgs& next, hipStream_t stream) {
    const int cone_wgs = (cones.n + 256 * kXcds - 1) / (256 * kXcds) * kXcds;
    hipLaunchKernelGGL(k_step2d, dim3(cone_wgs + next.per_xcd * kXcds), dim3(256), 0, stream,
                       rules, cones, step, cone_wgs, next);
    return hipGetLastError();
}

hipError_t launch_near_map(int dim, const TargetGrid& tg, uint32_t* near, size_t words,
                           int n_targets, hipStream_t stream) {
    hipError_t e = hipMemsetAsync(near, 0, words * sizeof(uint32_t), stream);
    if (e != hipSuccess || n_targets == 0) return e;
    const dim3 grid((n_targets + 255) / 256);
    if (dim == 2)
        hipLaunchKernelGGL(k_near_map<2>, grid, dim3(256), 0, stream, tg, near, n_targets);
    else
        hipLaunchKernelGGL(k_near_map<3>, grid, dim3(256), 0, stream, tg, near, n_targets);
    return hipGetLastError();
}

hipError_t launch_mass(const float* field, int64_t n, double* partial, int n_partial,
                       double* out, hipStream_t stream, int32_t* nonfinite) {
    int blocks = (int)((n + kMassThreads - 1) / kMassThreads);
    if (blocks > n_partial) blocks = n_partial;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(k_mass_partial, dim3(blocks), dim3(kMassThreads), 0, stream, field, n,
                       partial);
    hipLaunchKernelGGL(k_mass_final, dim3(1), dim3(kMassThreads), 0, stream, partial, blocks,
                       out, nonfinite);
    return hipGetLastError();
}

}  // namespace cuesim
