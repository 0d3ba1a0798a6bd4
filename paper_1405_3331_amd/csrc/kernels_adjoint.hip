// kernels_adjoint.hip -- reverse pass of the 2D time step, for the gradient of a trajectory
// loss L = sum_i w_i |p_i^N - t_a(i)|^2 with respect to the source amounts, D and k.
//
// The derivative is taken along the forward run's branch: the exit and contact decisions
// and the active side of the turn cap are held as the forward run took them (the cone
// rules of Sec. 3.4-3.5 have no derivative at those switches).
//
// The fields never depend on the cones, so within a checkpoint segment the cones can be
// handled apart from the fields, each cone by one thread over all the segment's steps:
//   k_cones_segments2d        re-runs the segment's cone steps against the re-run fields and
//                             records (x, y, theta) of every cone at the start of each step
//                             (when the whole run's fields fit in memory, every segment at
//                             once, one thread per segment and cone);
//   k_cone_adjoint_segment2d  walks the steps backwards carrying each cone's adjoint of
//                             (p, theta) through advance, capped turn and interpolated
//                             gradient, and records the adjoint of its sampled gradient
//                             (two values per cone and step);
//   k_sample_max              takes each step's largest contribution to a cell, the scale of
//                             its fixed-point sums;
//   kernels_reverse2d.hip     reverses the segment's field steps, eight per launch, adding
//                             the samples' adjoints where the cones were.
#include "internal.hpp"

namespace cuesim {

namespace {

constexpr int kAdjThreads = 256;
constexpr int kSegThreads = 64;   // segment kernels: one wavefront per workgroup.  With the
                                  // reverse walk loading footprints a step ahead, a gradient's
                                  // reverse sweep at 1024^2 (8192 cones) takes 21.4-21.6 ms,
                                  // against 21.7-21.8 with 32 threads and 23.0 with 16; half-wave
                                  // workgroups were ~1.5% faster before that prefetch

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

// Reverse of the interpolated central-difference gradient of one species at (x, y) with
// respect to the tip, from the footprint and corner gradients the forward sample used:
// (agx, agy) is the adjoint of the sampled gradient, already weighted by the species sign.
// Adds into (apx, apy) -- the interpolation weights depend on the tip; along an axis where the
// tip is clamped to the outermost centres they do not.  (The field's share is
// sample_adjoint_2d.)
__device__ __forceinline__ void sample_tip_adjoint_2d(const Footprint2D& p,
                                                      const CornerGradients2D& g,
                                                      const ConeRules& r, float x, float y,
                                                      float agx, float agy, float& apx,
                                                      float& apy) {
    const float fx = p.fx, fy = p.fy;
    const float ux = fmaf(x, r.inv_dx, -0.5f), uy = fmaf(y, r.inv_dx, -0.5f);
    const bool free_x = ux > 0.0f && ux < (float)(r.nx - 1);
    const bool free_y = uy > 0.0f && uy < (float)(r.ny - 1);
    // d w / d f along each axis, times d f / d p = 1 / dx where not clamped
    const float aw00 = fmaf(agy, g.gy00, agx * g.gx00), aw10 = fmaf(agy, g.gy10, agx * g.gx10);
    const float aw01 = fmaf(agy, g.gy01, agx * g.gx01), aw11 = fmaf(agy, g.gy11, agx * g.gx11);
    if (free_x) apx = fmaf(r.inv_dx, fmaf(fy, aw11 - aw01, (1.0f - fy) * (aw10 - aw00)), apx);
    if (free_y) apy = fmaf(r.inv_dx, fmaf(fx, aw11 - aw10, (1.0f - fx) * (aw01 - aw00)), apy);
}

struct Field2D {
    const float* f;
    int nx;
    __device__ float operator()(int i, int j) const { return f[j * nx + i]; }
};

// Reverse of one cone step (step index `step`) of cone i from its state (x, y, theta) at
// the start of the step, the footprints p0/p1 of its gradient samples in the fields after
// the step's field update, their corner gradients and the weighted gradient (gx, gy).
// (apx, apy, ath) holds the adjoint of the state after the step on entry and of the state
// before it on exit; (agx, agy) receives the adjoint of the weighted gradient.
template <int NS>
__device__ __forceinline__ void cone_adjoint_step(const ConeRules& r, const Footprint2D& p0,
                                                  const Footprint2D& p1,
                                                  const CornerGradients2D& g0,
                                                  const CornerGradients2D& g1, float gx,
                                                  float gy, float4 st, int i, uint32_t step,
                                                  float& apx, float& apy, float& ath,
                                                  float& agx, float& agy) {
    const float x = st.x, y = st.y, th = st.z;
    float s, c;
    sincos_angle(th, s, c);
    float cross, along;
    turn_terms(r, s, c, gx, gy, cross, along);
    bool capped;
    const float turn = capped_turn(r, cross, along, &capped);
    float z[2];
    noise_2d(r.key, (uint32_t)i, step, z);
    const float thn = wrap_heading(fmaf(r.sigma, z[0], th + turn));
    float sn, cn;
    sincos_angle(thn, sn, cn);

    // reverse: p' = p + s (cos theta', sin theta')
    const float athn = fmaf(r.step_len, fmaf(cn, apy, -(sn * apx)), ath);
    // theta' = theta + turn(theta, g) + noise
    ath = athn;
    agx = agy = 0.0f;
    if (!capped) {
        const float den = fmaf(along, along, cross * cross);
        const float a_cross = athn * along / den, a_along = -athn * cross / den;
        const float dot = fmaf(c, gx, s * gy);
        ath = fmaf(a_cross, -r.gain * dot, fmaf(a_along, cross, ath));
        agx = r.gain * fmaf(a_along, c, -(a_cross * s));
        agy = r.gain * fmaf(a_cross, c, a_along * s);
    }
    sample_tip_adjoint_2d(p0, g0, r, x, y, r.sign0 * agx, r.sign0 * agy, apx, apy);
    if (NS > 1)
        sample_tip_adjoint_2d(p1, g1, r, x, y, r.sign1 * agx, r.sign1 * agy, apx, apy);
}

// The forward gradient sample of a step from its footprints, computed exactly as the
// forward step computes it.
template <int NS>
__device__ __forceinline__ void sample_2d(const ConeRules& r, const Footprint2D& p0,
                                          const Footprint2D& p1, CornerGradients2D& g0,
                                          CornerGradients2D& g1, float& gx, float& gy) {
    g0 = corner_gradients_2d(p0, r);
    g1 = NS > 1 ? corner_gradients_2d(p1, r) : g0;
    gradient_from_2d(p0, g0, gx, gy, nullptr);
    gx *= r.sign0;
    gy *= r.sign0;
    if (NS > 1) {
        float hx, hy;
        gradient_from_2d(p1, g1, hx, hy, nullptr);
        gx = fmaf(r.sign1, hx, gx);
        gy = fmaf(r.sign1, hy, gy);
    }
}

// A checkpoint segment of `len` steps from step seg0: fields[t] (species-major, `cells`
// each) is the field state after t steps of the segment, t = 0..len.
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

struct Segment2D {
    const float* fields;
    size_t cells;
    int n_species;
    uint32_t seg0;
    int len;
    __device__ const float* field(int t, int s) const {
        return fields + ((size_t)t * n_species + s) * cells;
    }
};

// Forward re-run of the cone steps of segments seg_first .. seg_first + gridDim.y - 1, one
// thread per (segment, cone) over all the segment's steps, each starting from its
// checkpoint; the state at the start of run step t goes to tape[t - t_base][i] whether or
// not the cone is still active.  Same arithmetic as the forward step (gradient, turn,
// noise, advance, exit, contact).
template <int NS>
__global__ __launch_bounds__(kSegThreads) void k_cones_segments2d(ConeRules r, SegmentSet2D set,
                                                                  float4* __restrict__ tape) {
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
    for (int t = t0; t < t1; ++t) {
        tape[(size_t)(t - set.t_base) * M + i] = make_float4(x, y, th, 0.0f);
        if (status != kActive) continue;
        const float* f0 = set.field(t + 1, 0);
        float gx, gy;
        gradient_2d(Field2D{f0, r.nx}, r, x, y, gx, gy);
        gx *= r.sign0;
        gy *= r.sign0;
        if (NS > 1) {
            float hx, hy;
            gradient_2d(Field2D{set.field(t + 1, NS - 1), r.nx}, r, x, y, hx, hy);
            gx = fmaf(r.sign1, hx, gx);
            gy = fmaf(r.sign1, hy, gy);
        }
        float sn, cs;
        sincos_angle(th, sn, cs);
        float z[2];
        noise_2d(r.key, (uint32_t)i, set.n0 + (uint32_t)t, z);
        const ConeEvent ev = cone_step_2d(r, gx, gy, 0.0f, z, x, y, th, sn, cs,
                                          GridContact{&r.targets});
        status = ev.status;
    }
}

// Last step of a segment (from step seg0, len steps) in which cone i takes part: status and
// event_step are the run's final ones, and a cone stopped at step n takes part in steps < n
// only (-1: none of the segment's).
__device__ __forceinline__ int last_step(const Segment2D& seg, const int32_t* status,
                                         const int32_t* event_step, int i) {
    const int64_t last = status[i] == kActive ? INT64_MAX : (int64_t)event_step[i];
    return (int)max<int64_t>(min<int64_t>(seg.len - 1, last - 1 - (int64_t)seg.seg0), -1);
}

// Largest |adjoint| of the cells that one species' sample read.
__device__ __forceinline__ float sample_max(const ConeRules& r, float x, float y, float agx,
                                            float agy) {
    const Scatter2D c = sample_adjoint_2d(r, x, y, agx, agy);
    float m = 0.0f;
#pragma unroll
    for (int k = 0; k < 12; ++k) m = fmaxf(m, fabsf(c.v[k]));
    return m;
}

// Reverse of one segment's cone steps, one thread per cone from the last step to the first;
// the adjoint of step t's sampled gradient goes to ag[t * n + i] and the largest adjoint of a
// cell it read to vmax (zero at steps the cone takes no part in).
// The forward states come from the run's cone tape, so the gathers of the step before do
// not wait for this step's adjoint: its footprints are loaded one step ahead and its state
// two.
template <int NS>
__global__ __launch_bounds__(kSegThreads) void k_cone_adjoint_segment2d(
    ConeRules r, Segment2D seg, float2* __restrict__ ag, float* __restrict__ vmax,
    const float4* __restrict__ tape, const int32_t* __restrict__ status,
    const int32_t* __restrict__ event_step, float* __restrict__ acone, int n) {
    const int i = blockIdx.x * kSegThreads + threadIdx.x;
    if (i >= n) return;
    float apx = acone[3 * i], apy = acone[3 * i + 1], ath = acone[3 * i + 2];
    const int t_hi = last_step(seg, status, event_step, i);
    for (int t = seg.len - 1; t > t_hi; --t) {
        ag[(size_t)t * n + i] = make_float2(0.0f, 0.0f);
        vmax[(size_t)t * n + i] = 0.0f;
    }
    if (t_hi >= 0) {
        float4 st = tape[(size_t)t_hi * n + i];
        float4 next = tape[(size_t)max(t_hi - 1, 0) * n + i];
        Footprint2D p0 = footprint_2d(Field2D{seg.field(t_hi + 1, 0), r.nx}, r, st.x, st.y);
        Footprint2D p1 =
            NS > 1 ? footprint_2d(Field2D{seg.field(t_hi + 1, NS - 1), r.nx}, r, st.x, st.y)
                   : p0;
        for (int t = t_hi; t >= 0; --t) {
            // the step before: its state two steps ahead and its footprints one step ahead,
            // requested before this step's arithmetic (the samples do not depend on it)
            const float4 next2 = tape[(size_t)max(t - 2, 0) * n + i];
            Footprint2D q0 = p0, q1 = p1;
            if (t > 0) {
                q0 = footprint_2d(Field2D{seg.field(t, 0), r.nx}, r, next.x, next.y);
                q1 = NS > 1 ? footprint_2d(Field2D{seg.field(t, NS - 1), r.nx}, r, next.x,
                                           next.y)
                            : q0;
            }
            CornerGradients2D g0, g1;
            float gx, gy, agx, agy;
            sample_2d<NS>(r, p0, p1, g0, g1, gx, gy);
            cone_adjoint_step<NS>(r, p0, p1, g0, g1, gx, gy, st, i, seg.seg0 + (uint32_t)t,
                                  apx, apy, ath, agx, agy);
            float m = sample_max(r, st.x, st.y, r.sign0 * agx, r.sign0 * agy);
            if (NS > 1) m = fmaxf(m, sample_max(r, st.x, st.y, r.sign1 * agx, r.sign1 * agy));
            ag[(size_t)t * n + i] = make_float2(agx, agy);
            vmax[(size_t)t * n + i] = m;
            st = next;
            next = next2;
            p0 = q0;
            p1 = q1;
        }
    }
    acone[3 * i] = apx;
    acone[3 * i + 1] = apy;
    acone[3 * i + 2] = ath;
}

// Largest |contribution| of every step of the segment: a workgroup takes kMaxCones cones of
// one step (kMaxCones / kMaxThreads per thread), reduces their maximum through the wavefronts
// and LDS, and applies one atomic maximum on the step's FP32 bits (non-negative floats order
// like their bits).  Few atomics meet on each step's word: with one per wavefront (128 per
// step at 8192 cones) they queued on those words.
constexpr int kMaxThreads = 256;
constexpr int kMaxCones = 8 * kMaxThreads;

__global__ __launch_bounds__(kMaxThreads) void k_sample_max(const float* __restrict__ vmax,
                                                            uint32_t* __restrict__ step_max,
                                                            int n) {
    const int t = blockIdx.y;
    float m = 0.0f;
#pragma unroll
    for (int k = 0; k < kMaxCones / kMaxThreads; ++k) {
        const int i = blockIdx.x * kMaxCones + k * kMaxThreads + threadIdx.x;
        if (i < n) m = fmaxf(m, vmax[(size_t)t * n + i]);
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

// Loss at the final tips and the seed of the cone adjoints: a_p = 2 w (p - t), a_theta = 0.
__global__ __launch_bounds__(kAdjThreads) void k_adjoint_seed2d(
    const float* __restrict__ pos, const float* __restrict__ tip_target,
    const float* __restrict__ weight, float* __restrict__ acone, double* __restrict__ partial,
    int n) {
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
                                   float4* tape, hipStream_t stream) {
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

hipError_t launch_cone_adjoint_segment2d(const ReverseSegment& g, const int32_t* status,
                                         const int32_t* event_step, float* acone,
                                         hipStream_t stream) {
    const int n = g.M;
    if (g.len == 0 || n == 0) return hipSuccess;
    const Segment2D seg{g.fields, (size_t)g.nx * g.ny, g.n_species, g.seg0, g.len};
    const dim3 grid((n + kSegThreads - 1) / kSegThreads);
    const dim3 max_grid((n + kMaxCones - 1) / kMaxCones, g.len);
    if (g.n_species > 1)
        hipLaunchKernelGGL(k_cone_adjoint_segment2d<2>, grid, dim3(kSegThreads), 0, stream,
                           g.rules, seg, g.ag, g.vmax, g.tips, status, event_step, acone, n);
    else
        hipLaunchKernelGGL(k_cone_adjoint_segment2d<1>, grid, dim3(kSegThreads), 0, stream,
                           g.rules, seg, g.ag, g.vmax, g.tips, status, event_step, acone, n);
    hipLaunchKernelGGL(k_sample_max, max_grid, dim3(kMaxThreads), 0, stream, g.vmax, g.step_max,
                       n);
    return hipGetLastError();
}

hipError_t launch_adjoint_seed2d(const float* pos, const float* tip_target, const float* weight,
                                 float* acone, double* partial, int n, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_adjoint_seed2d, dim3(adjoint_cone_blocks(n)), dim3(kAdjThreads), 0,
                       stream, pos, tip_target, weight, acone, partial, n);
    return hipGetLastError();
}


}  // namespace cuesim
