// cone_adjoint.hpp -- the reverse of a cone's steps: the chain of one thread per cone, in launches
// of its own (kernels_adjoint.hip) or beside the reverse field steps of the segment after
// (kernels_reverse2d.hip).
#pragma once

#include "internal.hpp"

namespace cuesim {

// Reverse of the interpolated central-difference gradient of one species at (x, y) with
// respect to the tip, from the fractions and corner gradients of the forward sample:
// (agx, agy) is the adjoint of the sampled gradient, already weighted by the species sign.
// Adds into (apx, apy) -- the interpolation weights depend on the tip; along an axis where the
// tip is clamped to the outermost centres they do not.  (The field's share is
// sample_adjoint_2d.)
__device__ __forceinline__ void sample_tip_adjoint_2d(float fx, float fy, const float4& gx,
                                                      const float4& gy, const ConeRules& r,
                                                      float x, float y, float agx, float agy,
                                                      float& apx, float& apy) {
    const float ux = fmaf(x, r.inv_dx, -0.5f), uy = fmaf(y, r.inv_dx, -0.5f);
    const bool free_x = ux > 0.0f && ux < (float)(r.nx - 1);
    const bool free_y = uy > 0.0f && uy < (float)(r.ny - 1);
    // d w / d f along each axis, times d f / d p = 1 / dx where not clamped
    const float aw00 = fmaf(agy, gy.x, agx * gx.x), aw10 = fmaf(agy, gy.y, agx * gx.y);
    const float aw01 = fmaf(agy, gy.z, agx * gx.z), aw11 = fmaf(agy, gy.w, agx * gx.w);
    if (free_x) apx = fmaf(r.inv_dx, fmaf(fy, aw11 - aw01, (1.0f - fy) * (aw10 - aw00)), apx);
    if (free_y) apy = fmaf(r.inv_dx, fmaf(fx, aw11 - aw10, (1.0f - fx) * (aw01 - aw00)), apy);
}

// A cone step's record (ConeTape).
template <int NS>
struct ConeTerms {
    float4 v[kConePlanes + 2 * NS];
    __device__ __forceinline__ void load(const ConeTape& tape, int t, int i) {
#pragma unroll
        for (int j = 0; j < kConePlanes + 2 * NS; ++j)
            v[j] = tape.base[j * tape.plane + (size_t)t * tape.M + i];
    }
};

// Reverse of one cone step from its record.  (apx, apy, ath) holds the adjoint of the state
// after the step on entry and of the state before it on exit; (agx, agy) receives the adjoint
// of the weighted gradient.
template <int NS>
__device__ __forceinline__ void cone_adjoint_step(const ConeRules& r, const ConeTerms<NS>& m,
                                                  float& apx, float& apy, float& ath,
                                                  float& agx, float& agy) {
    const float x = m.v[0].x, y = m.v[0].y, sn = m.v[0].z, cn = m.v[0].w;
    const float cross = m.v[1].x, along = m.v[1].y, s = m.v[1].z, c = m.v[1].w;
    const float gx = m.v[2].x, gy = m.v[2].y, fx = m.v[2].z, fy = m.v[2].w;
    // reverse: p' = p + s (cos theta', sin theta')
    const float athn = fmaf(r.step_len, fmaf(cn, apy, -(sn * apx)), ath);
    // theta' = theta + turn(theta, g) + noise
    ath = athn;
    agx = agy = 0.0f;
    if (!turn_capped(r, cross, along)) {
        const float den = fmaf(along, along, cross * cross);
        const float a_cross = athn * along / den, a_along = -athn * cross / den;
        const float dot = fmaf(c, gx, s * gy);
        ath = fmaf(a_cross, -r.gain * dot, fmaf(a_along, cross, ath));
        agx = r.gain * fmaf(a_along, c, -(a_cross * s));
        agy = r.gain * fmaf(a_cross, c, a_along * s);
    }
    sample_tip_adjoint_2d(fx, fy, m.v[3], m.v[4], r, x, y, r.sign0 * agx, r.sign0 * agy, apx,
                          apy);
    if (NS > 1)
        sample_tip_adjoint_2d(fx, fy, m.v[kConePlanes + 2 * NS - 2],
                              m.v[kConePlanes + 2 * NS - 1], r, x, y, r.sign1 * agx,
                              r.sign1 * agy, apx, apy);
}

// Last step of a segment (from step seg0, len steps) in which cone i takes part (-1: none):
// none if it had stopped before the segment; a cone stopped at step n takes part in steps < n only,
// by the run's end and by the handle's state.
__device__ __forceinline__ int last_step(const ConeChain& c, int i) {
    if (c.start_status[i] != kActive) return -1;
    const int64_t now = c.status[i] == kActive ? INT64_MAX : (int64_t)c.event_step[i];
    const int64_t run = c.run_status[i] == kActive ? INT64_MAX : (int64_t)c.run_event[i];
    return (int)max<int64_t>(
        min<int64_t>(c.len - 1, min<int64_t>(now, run) - 1 - (int64_t)c.seg0), -1);
}

// Reverse of cone i's steps c.t_from, c.t_from - 1, .., at most `most` of them; the adjoint of step
// t's sampled gradient goes to ag[t * n + i] (zero at steps the cone takes no part in).  The
// forward steps come from the cone tape, a streaming read AHEAD steps ahead, so that only what
// depends on the adjoint is left in the chain from step to step: 65 VALU instructions, two of them
// divisions.  (Before, each step gathered its 12 cells per species from the run's fields, a
// 128-byte line for a few bytes, and computed the forward step again: 115 us per 100 steps of
// 8192 cones, against 55.)
// For every reverse launch (kRevSteps steps, from the segment's end) the box of the tips whose
// samples have an adjoint goes to boxes[launch * n + i] (empty: x from above x to).
template <int NS, int AHEAD>
__device__ __forceinline__ void cone_chain(const ConeRules& r, const ConeChain& c, int i,
                                           int most) {
    const int n = c.tape.M, t_from = c.t_from, t_to = max(t_from - most + 1, 0);
    float apx = c.acone[3 * i], apy = c.acone[3 * i + 1], ath = c.acone[3 * i + 2];
    const int t_hi = last_step(c, i);
    const float4 none = make_float4(INFINITY, -INFINITY, INFINITY, -INFINITY);
    float4 box = none;   // x from, x to, y from, y to
    ConeTerms<NS> terms[AHEAD];
#pragma unroll
    for (int a = 0; a < AHEAD; ++a) terms[a].load(c.tape, max(t_from - a, 0), i);
    // every cone walks all the steps (t is the same for the whole wavefront, so addresses are
    // scalar work); a step it takes no part in leaves its adjoint alone
    for (int t0 = t_from; t0 >= t_to; t0 -= AHEAD) {
#pragma unroll
        for (int a = 0; a < AHEAD; ++a) {
            const int t = t0 - a;
            if (t < t_to) break;
            const ConeTerms<NS> here = terms[a];
            terms[a].load(c.tape, max(t - AHEAD, 0), i);
            float agx = 0.0f, agy = 0.0f;
            if (t <= t_hi) {
                cone_adjoint_step<NS>(r, here, apx, apy, ath, agx, agy);
                if (agx != 0.0f || agy != 0.0f)
                    box = make_float4(fminf(box.x, here.v[0].x), fmaxf(box.y, here.v[0].x),
                                      fminf(box.z, here.v[0].y), fmaxf(box.w, here.v[0].y));
            }
            c.ag[(size_t)t * n + i] = make_float2(agx, agy);
            const int k = c.len - 1 - t;
            if (k % kRevSteps == kRevSteps - 1 || t == 0) {
                c.boxes[(size_t)(k / kRevSteps) * n + i] = box;
                box = none;
            }
        }
    }
    c.acone[3 * i] = apx;
    c.acone[3 * i + 1] = apy;
    c.acone[3 * i + 2] = ath;
}

}  // namespace cuesim
