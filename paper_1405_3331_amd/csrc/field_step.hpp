// field_step.hpp -- one explicit field step of one box of one species, sources included: the
// work of one workgroup of the marching field kernels, alone in their launch or beside the cones
// of the step before (k_step2d, k_step3d).  kernels_field2d.hip and kernels_field3d.hip say how
// boxes and their source lists are laid out.
#pragma once

#include "internal.hpp"

namespace cuesim {

constexpr int kXcds = 8;   // workgroups are dealt to the accelerator dies round-robin

// 2D boxes: 256 columns x 8 rows, all 8 rows' loads at once (measured best)
constexpr int kRX = 256, kRY = 8, kRUnroll = 8;
// 3D boxes: 64 x 8 columns, planes kUnroll3D at a time
constexpr int kTX = 64, kTY = 8, kUnroll3D = 4;
constexpr int kBoxThreads3D = kTX * kTY;

__device__ __forceinline__ float stencil2d(float c, float w, float e, float s, float n,
                                           const StencilCoef& k) {
    const float lap = fmaf(-4.0f, c, (w + e) + (s + n));
    return fmaf(k.r, lap, fmaf(-k.kdt, c, c));
}

__device__ __forceinline__ void field2d_box(const Field2DStepArgs& a, int box, int tid) {
    const int bx = box % a.tx, by = (box / a.tx) % a.ty, s = box / (a.tx * a.ty);
    int e = a.src_start[box];
    const int e_end = a.src_start[box + 1];
    const int i = bx * kRX + tid;
    if (i >= a.nx) return;   // no barriers below
    const StencilCoef k = a.coef[s];
    const int nx = a.nx, ny = a.ny;
    const float* col = a.in[s] + i;
    float* dst = a.out[s] + i;
    const int dw = i > 0 ? -1 : 0, de = i < nx - 1 ? 1 : 0;
    const int j0 = by * kRY, j1 = min(j0 + kRY, ny);
    float c = col[(size_t)j0 * nx];
    float below = col[(size_t)max(j0 - 1, 0) * nx];
    int j = j0;
    auto finish = [&](float v, int row) {
        while (e < e_end && a.src_row[e] == row) {
            if (a.src_col[e] == tid) v += a.src_q[e];
            ++e;
        }
        dst[(size_t)row * nx] = v;
    };
    for (; j + kRUnroll <= j1; j += kRUnroll) {
        float up[kRUnroll], w[kRUnroll], ea[kRUnroll];
#pragma unroll
        for (int u = 0; u < kRUnroll; ++u) {
            const float* p = col + (size_t)(j + u) * nx;
            up[u] = col[(size_t)min(j + u + 1, ny - 1) * nx];
            w[u] = p[dw];
            ea[u] = p[de];
        }
#pragma unroll
        for (int u = 0; u < kRUnroll; ++u) {
            finish(stencil2d(c, w[u], ea[u], below, up[u], k), j + u);
            below = c;
            c = up[u];
        }
    }
    for (; j < j1; ++j) {
        const float* p = col + (size_t)j * nx;
        const float above = col[(size_t)min(j + 1, ny - 1) * nx];
        finish(stencil2d(c, p[dw], p[de], below, above, k), j);
        below = c;
        c = above;
    }
}

__device__ __forceinline__ float stencil3d(float c, float w, float e, float s, float n,
                                           float below, float above, const StencilCoef& k) {
    const float lap = fmaf(-6.0f, c, ((w + e) + (s + n)) + (below + above));
    return fmaf(k.r, lap, fmaf(-k.kdt, c, c));
}

__device__ __forceinline__ void field3d_box(const Field3DArgs& a, int box, int tid) {
    int rest = box;
    const int bx = rest % a.tx;
    rest /= a.tx;
    const int by = rest % a.ty;
    rest /= a.ty;
    const int bz = rest % a.tz;
    const int s = rest / a.tz;
    // this workgroup's slice of the source list
    int e = a.src_start[box];
    const int e_end = a.src_start[box + 1];

    const int i = bx * kTX + tid % kTX;
    const int j = by * kTY + tid / kTX;
    if (i >= a.nx || j >= a.ny) {
        return;   // no barriers below: idle threads may leave
    }
    const StencilCoef k = a.coef[s];
    const size_t plane = (size_t)a.nx * a.ny;
    const float* col = a.in[s] + (size_t)j * a.nx + i;
    float* dst = a.out[s] + (size_t)j * a.nx + i;
    const int dw = i > 0 ? -1 : 0, de = i < a.nx - 1 ? 1 : 0;
    const int ds = j > 0 ? -a.nx : 0, dn = j < a.ny - 1 ? a.nx : 0;
    const int nz = a.nz;
    const int z0 = bz * a.planes, z1 = min(z0 + a.planes, nz);

    float c = col[(size_t)z0 * plane];
    float below = col[(size_t)max(z0 - 1, 0) * plane];
    int l = z0;
    for (; l + kUnroll3D <= z1; l += kUnroll3D) {
        float up[kUnroll3D], w[kUnroll3D], ea[kUnroll3D], so[kUnroll3D], no[kUnroll3D];
#pragma unroll
        for (int u = 0; u < kUnroll3D; ++u) {
            const float* p = col + (size_t)(l + u) * plane;
            up[u] = col[(size_t)min(l + u + 1, nz - 1) * plane];
            w[u] = p[dw];
            ea[u] = p[de];
            so[u] = p[ds];
            no[u] = p[dn];
        }
#pragma unroll
        for (int u = 0; u < kUnroll3D; ++u) {
            float v = stencil3d(c, w[u], ea[u], so[u], no[u], below, up[u], k);
            while (e < e_end && a.src_plane[e] == l + u) {
                if (a.src_thread[e] == tid) v += a.src_q[e];
                ++e;
            }
            dst[(size_t)(l + u) * plane] = v;
            below = c;
            c = up[u];
        }
    }
    for (; l < z1; ++l) {
        const float* p = col + (size_t)l * plane;
        const float above = col[(size_t)min(l + 1, nz - 1) * plane];
        float v = stencil3d(c, p[dw], p[de], p[ds], p[dn], below, above, k);
        while (e < e_end && a.src_plane[e] == l) {
            if (a.src_thread[e] == tid) v += a.src_q[e];
            ++e;
        }
        dst[(size_t)l * plane] = v;
        below = c;
        c = above;
    }
}

}  // namespace cuesim
