// kernels_adjoint.hip -- reverse pass of the 2D time step, for the gradient of a trajectory
// loss L = sum_i w_i |p_i^N - t_a(i)|^2 with respect to the source amounts, D and k.
//
// The derivative is taken along the forward run's branch: the exit and contact decisions
// and the active side of the turn cap are held as the forward run took them (the cone
// rules of Sec. 3.4-3.5 have no derivative at those switches).
//
// The fields never depend on the cones, so within a checkpoint segment the cones can be
// handled apart from the fields, each cone by one thread over all the segment's steps:
//   the forward run (or, where it did not record its states, k_cones_segments2d, which re-runs
//                             the segment's cone steps against the re-run fields) records what
//                             the reverse of each cone step needs of it (ConeTape);
//   cone_chain                (cone_adjoint.hpp) walks the steps backwards carrying each cone's
//                             adjoint of (p, theta) through advance, capped turn and
//                             interpolated gradient, and records the adjoint of its sampled
//                             gradient (two values per cone and step); here in launches of
//                             its own (k_cone_adjoint_segment2d);
//   k_sample_max              takes each step's largest contribution to a cell, the scale of
//                             its fixed-point sums;
//   kernels_reverse2d.hip     reverses the segment's field steps, eight per launch, adding
//                             the samples' adjoints where the cones were, with the chain of
//                             the segment before beside them where the run recorded it.
#include "cone_adjoint.hpp"
#include "internal.hpp"

namespace cuesim {

namespace {

constexpr int kAdjThreads = 256;
constexpr int kSegThreads = 64;   // segment kernels: one wavefront per workgroup, so that the
                                  // cones of a small run spread over as many CUs as they can

__device__ double adj_block_sum(double v) {
    __shared__ double part[kAdjThreads / 64];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __syncthreads();   // part[] may still be read from a previous call
    if (lane == 0) part[wave] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < kAdjThreads / 64; ++w) t += part[w];
    return t;
}

struct Field2D {
    const float* f;
    int nx;
    __device__ float operator()(int i, int j) const { return f[j * nx + i]; }
};

// Segments of a checkpointed run of n_steps steps from step n0, every `every` steps: run
// step t's field state (after t steps) is fields + ((t - t_base) * n_species + s) * cells;
// the checkpoint arrays hold each segment's cone state at its first step.
struct SegmentSet2D {
    const float* fields;
    size_t cells;
    int n_species;
    int t_base;
    int seg_first, every, n_steps;
    uint32_t n0;
    const float* ckpt_pos;         // [segments][M][2]
    const float* ckpt_dir;         // [segments][M]
    const int32_t* ckpt_status;    // [segments][3][M]: status first
    int M;
    __device__ const float* field(int t, int s) const {
        return fields + ((size_t)(t - t_base) * n_species + s) * cells;
    }
};

// Forward re-run of the cone steps of segments seg_first .. seg_first + gridDim.y - 1, one
// thread per (segment, cone) over all the segment's steps, each starting from its
// checkpoint; the cone's step t is recorded as step t - t_base of the tape while it is active.
// Same arithmetic as the forward step (gradient, turn, noise, advance, exit, contact).
template <int NS>
__global__ __launch_bounds__(kSegThreads) void k_cones_segments2d(ConeRules r, SegmentSet2D set,
                                                                  ConeTape tape) {
    const int i = blockIdx.x * kSegThreads + threadIdx.x;
    if (i >= set.M) return;
    const int seg = set.seg_first + (int)blockIdx.y;
    const int t0 = seg * set.every;
    const int t1 = min(t0 + set.every, set.n_steps);
    const size_t M = (size_t)set.M;
    float x = set.ckpt_pos[((size_t)seg * M + i) * 2];
    float y = set.ckpt_pos[((size_t)seg * M + i) * 2 + 1];
    float th = set.ckpt_dir[(size_t)seg * M + i];
    int status = set.ckpt_status[(size_t)seg * 3 * M + i];
    float sn, cs;
    sincos_angle(th, sn, cs);
    for (int t = t0; t < t1 && status == kActive; ++t) {
        const size_t rec = (size_t)(t - set.t_base);
        float gx, gy;
        const Footprint2D p0 = footprint_2d(Field2D{set.field(t + 1, 0), r.nx}, r, x, y);
        const CornerGradients2D g0 = corner_gradients_2d(p0, r);
        gradient_from_2d(p0, g0, gx, gy, nullptr);
        tape.sample(0, rec, i, g0);
        gx *= r.sign0;
        gy *= r.sign0;
        if (NS > 1) {
            float hx, hy;
            const Footprint2D p1 = footprint_2d(Field2D{set.field(t + 1, NS - 1), r.nx}, r, x, y);
            const CornerGradients2D g1 = corner_gradients_2d(p1, r);
            gradient_from_2d(p1, g1, hx, hy, nullptr);
            tape.sample(1, rec, i, g1);
            gx = fmaf(r.sign1, hx, gx);
            gy = fmaf(r.sign1, hy, gy);
        }
        tape.put(2, rec, i, make_float4(gx, gy, p0.fx, p0.fy));
        const float x0 = x, y0 = y, s0 = sn, c0 = cs;
        float z[2];
        noise_2d(r.key, (uint32_t)i, set.n0 + (uint32_t)t, z);
        const ConeEvent ev = cone_step_2d(r, gx, gy, 0.0f, z, x, y, th, sn, cs,
                                          GridContact{&r.targets});
        record_turn(tape, rec, i, r, x0, y0, s0, c0, gx, gy, sn, cs);
        status = ev.status;
    }
}

template <int NS>
__global__ __launch_bounds__(kSegThreads) void k_cone_adjoint_segment2d(ConeRules r,
                                                                        ConeChain c) {
    const int i = blockIdx.x * kSegThreads + threadIdx.x;
    if (i < c.tape.M) cone_chain<NS, 4>(r, c, i, c.len);
}

// Largest |adjoint| of the cells that one species' sample read.
__device__ __forceinline__ float sample_max(const ConeRules& r, float2 p, float agx, float agy) {
    const Scatter2D c = sample_adjoint_2d(r, p.x, p.y, agx, agy);
    float m = 0.0f;
#pragma unroll
    for (int k = 0; k < 12; ++k) m = fmaxf(m, fabsf(c.v[k]));
    return m;
}

// Largest |contribution| of every step of the segment: a workgroup takes kMaxCones cones of
// one step (kMaxCones / kMaxThreads per thread), reduces their maximum through the wavefronts
// and LDS, and applies one atomic maximum on the step's FP32 bits (non-negative floats order
// like their bits).  Few atomics meet on each step's word: with one per wavefront (128 per
// step at 8192 cones) they queued on those words.
constexpr int kMaxThreads = 256;
constexpr int kMaxCones = 8 * kMaxThreads;

__global__ __launch_bounds__(kMaxThreads) void k_sample_max(ConeRules r,
                                                            const float4* __restrict__ tips,
                                                            const float2* __restrict__ ag,
                                                            uint32_t* __restrict__ step_max,
                                                            int n) {
    const int t = blockIdx.y;
    float m = 0.0f;
    // every cone's loads first (an index past the end reads the last cone again)
    constexpr int kEach = kMaxCones / kMaxThreads;
    float2 gs[kEach], ps[kEach];
#pragma unroll
    for (int k = 0; k < kEach; ++k) {
        const int i = min((int)(blockIdx.x * kMaxCones + k * kMaxThreads + threadIdx.x), n - 1);
        gs[k] = ag[(size_t)t * n + i];
        ps[k] = *(const float2*)(tips + (size_t)t * n + i);
    }
#pragma unroll
    for (int k = 0; k < kEach; ++k) {
        const float2 g = gs[k], p = ps[k];
        if (g.x == 0.0f && g.y == 0.0f) continue;
        m = fmaxf(m, sample_max(r, p, r.sign0 * g.x, r.sign0 * g.y));
        if (r.n_species > 1) m = fmaxf(m, sample_max(r, p, r.sign1 * g.x, r.sign1 * g.y));
    }
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    __shared__ float wave_max[kMaxThreads / 64];
    if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kMaxThreads / 64; ++w) m = fmaxf(m, wave_max[w]);
        if (m > 0.0f) atomicMax(&step_max[t], __float_as_uint(m));
    }
}

// Loss at the final tips and the seed of the cone adjoints: a_p = 2 w (p - t), a_theta = 0.  With
// `stop`, status and event step of the n cones go there.
__global__ __launch_bounds__(kAdjThreads) void k_adjoint_seed2d(
    const float* __restrict__ pos, const int32_t* __restrict__ status,
    const int32_t* __restrict__ event_step, const float* __restrict__ tip_target,
    const float* __restrict__ weight, float* __restrict__ acone, double* __restrict__ partial,
    int32_t* __restrict__ stop, int n) {
    const int i = blockIdx.x * kAdjThreads + threadIdx.x;
    double l = 0.0;
    if (i < n) {
        const float dx = pos[2 * i] - tip_target[2 * i];
        const float dy = pos[2 * i + 1] - tip_target[2 * i + 1];
        const float w = weight[i];
        acone[3 * i] = 2.0f * w * dx;
        acone[3 * i + 1] = 2.0f * w * dy;
        acone[3 * i + 2] = 0.0f;
        l = (double)w * ((double)dx * dx + (double)dy * dy);
        if (stop) {
            stop[i] = status[i];
            stop[n + i] = event_step[i];
        }
    }
    const double t = adj_block_sum(l);
    if (threadIdx.x == 0) partial[blockIdx.x] = t;
}


}  // namespace

int adjoint_cone_blocks(int n) { return (n + kAdjThreads - 1) / kAdjThreads; }

hipError_t launch_cones_segments2d(const ConeRules& rules, const float* fields, size_t cells,
                                   int n_species, int t_base, int seg_first, int n_seg,
                                   int every, int n_steps, uint32_t n0, const float* ckpt_pos,
                                   const float* ckpt_dir, const int32_t* ckpt_int, int M,
                                   const ConeTape& tape, hipStream_t stream) {
    if (M == 0 || n_seg == 0) return hipSuccess;
    const SegmentSet2D set{fields, cells, n_species, t_base, seg_first, every, n_steps, n0,
                           ckpt_pos, ckpt_dir, ckpt_int, M};
    const dim3 grid((M + kSegThreads - 1) / kSegThreads, n_seg);
    if (n_species > 1)
        hipLaunchKernelGGL(k_cones_segments2d<2>, grid, dim3(kSegThreads), 0, stream, rules,
                           set, tape);
    else
        hipLaunchKernelGGL(k_cones_segments2d<1>, grid, dim3(kSegThreads), 0, stream, rules,
                           set, tape);
    return hipGetLastError();
}

hipError_t launch_cone_chain2d(const ConeRules& rules, const ConeChain& c, hipStream_t stream) {
    if (c.t_from < 0 || c.tape.M == 0) return hipSuccess;
    const dim3 grid((c.tape.M + kSegThreads - 1) / kSegThreads);
    if (rules.n_species > 1)
        hipLaunchKernelGGL(k_cone_adjoint_segment2d<2>, grid, dim3(kSegThreads), 0, stream, rules,
                           c);
    else
        hipLaunchKernelGGL(k_cone_adjoint_segment2d<1>, grid, dim3(kSegThreads), 0, stream, rules,
                           c);
    return hipGetLastError();
}

hipError_t launch_sample_max2d(const ReverseSegment& g, hipStream_t stream) {
    const int n = g.M;
    if (g.len == 0 || n == 0) return hipSuccess;
    const dim3 max_grid((n + kMaxCones - 1) / kMaxCones, g.len);
    hipLaunchKernelGGL(k_sample_max, max_grid, dim3(kMaxThreads), 0, stream, g.rules,
                       g.tape.base, g.ag, g.step_max, n);
    return hipGetLastError();
}

hipError_t launch_adjoint_seed2d(const ConeArrays& cones, const float* tip_target,
                                 const float* weight, float* acone, double* partial,
                                 int32_t* stop, hipStream_t stream) {
    const int n = cones.n;
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_adjoint_seed2d, dim3(adjoint_cone_blocks(n)), dim3(kAdjThreads), 0,
                       stream, cones.pos, cones.status, cones.event_step, tip_target, weight,
                       acone, partial, stop, n);
    return hipGetLastError();
}

}  // namespace cuesim
