// kernels_field2d.hip -- one explicit 2D field step per launch (every species, sources
// included), marching up the rows.
//
// A workgroup owns kRX columns x kRY rows of one species; each thread
// keeps the rows below, at and above its cell in registers and reads its two row neighbours
// from lines the workgroup has just brought into L1, so a cell is fetched from HBM about
// once.  Rows are taken in groups with every load of a group issued before the arithmetic.  A
// missing neighbour at a wall is the cell itself (clamped index).  The stencil expression
// is term for term the one of the temporally blocked kernel, so both paths give the same
// bits.  Boxes are dealt to the accelerator dies in contiguous stretches.
//
// Step (Sec. 3.4 cue field: diffusion with first-order decay and point sources):
//   c' = c + r ((w + e) + (s + n) - 4c) - k dt c, then c' += q / dx^2 at each source cell
//   (a separate FP32 add, the rounding of a source pass), from a per-box list built once.
//   Where every state is kept (the gradient sweep's re-run), k_field2d_pair takes two steps
//   per launch: a box of 256 x 4 cells holds c^n on the box and a two-cell ring in LDS,
//   steps the box and a one-cell ring (with the sources there), writes c^{n+1}, steps the
//   box again and writes c^{n+2}: 12 instead of 16 B per cell and two steps, same bits.
#include <hip/hip_ext.h>

#include <algorithm>
#include <vector>

#include "field_step.hpp"
#include "internal.hpp"
#include "memory.hpp"

namespace cuesim {

namespace {

// two steps per launch: boxes of 256 x kPY cells held with a two-cell
// ring (kPW x kPH) for the first step and a one-cell ring (kQW x kQH) for the second; 4 rows
// measured best (2, 6 and 8 rows slower)
constexpr int kPY = 4;
constexpr int kPW = kRX + 4, kPH = kPY + 4;
constexpr int kQW = kRX + 2, kQH = kPY + 2;

struct Tiles2D {
    int tx, ty;
};

Tiles2D tiles_for(int nx, int ny, int rows = kRY) {
    return Tiles2D{(nx + kRX - 1) / kRX, (ny + rows - 1) / rows};
}

// Logical box of this workgroup (die-contiguous stretches of the box order).
__device__ __forceinline__ int box_of(int per_xcd) {
    return (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
}

__global__ __launch_bounds__(kRX) void k_field2d_rows(Field2DStepArgs a) {
    const int box = box_of(a.per_xcd);
    if (box >= a.n_species * a.tx * a.ty) return;
    field2d_box(a, box, threadIdx.x);
}

// Two forward steps of one species per box; the stencil and the separate source add are
// those of the single step, and neighbour indices are clamped grid indices mapped into the
// tile, so the result has the single step's bits.
struct Field2DPairArgs {
    const float* in[2];
    float* out1[2];
    float* out2[2];
    StencilCoef coef[2];
    int nx, ny, n_species, tx, ty, per_xcd;
    const int32_t* src_start;   // [boxes + 1]
    const int32_t* src_pos;     // row * (kRX + 2) + column in the box with its one-cell ring
    const float* src_q;
};


__global__ __launch_bounds__(kRX) void k_field2d_pair(Field2DPairArgs a) {
    const int box = box_of(a.per_xcd);
    if (box >= a.n_species * a.tx * a.ty) return;   // whole workgroup
    const int bx = box % a.tx, by = (box / a.tx) % a.ty, s = box / (a.tx * a.ty);
    const int x0 = bx * kRX, y0 = by * kPY;
    const int nx = a.nx, ny = a.ny;
    const int tid = threadIdx.x;
    const StencilCoef k = a.coef[s];
    __shared__ float T0[kPH][kPW];   // c^n: box and a two-cell ring
    __shared__ float T1[kQH][kQW];   // c^{n+1}: box and a one-cell ring
    __shared__ float T2[kPY][kRX];   // c^{n+2}: box
    auto t0 = [&](int i, int j) { return T0[j - y0 + 2][i - x0 + 2]; };
    auto t1 = [&](int i, int j) { return T1[j - y0 + 1][i - x0 + 1]; };

    // c^n (clamped into the grid; ring copies outside it are never read), this thread's
    // column and, for threads 0..3, the ring columns x0 - 2, x0 - 1, x0 + 256, x0 + 257
    const float* src = a.in[s];
    const int i = x0 + tid;
    const int ci = min(i, nx - 1);
    const int xcol = tid < 2 ? tid : kRX + tid;
    const int xi = min(max(x0 - 2 + xcol, 0), nx - 1);
    float v[kPH], xv[kPH];
#pragma unroll
    for (int u = 0; u < kPH; ++u)
        v[u] = src[(size_t)min(max(y0 - 2 + u, 0), ny - 1) * nx + ci];
    if (tid < 4) {
#pragma unroll
        for (int u = 0; u < kPH; ++u)
            xv[u] = src[(size_t)min(max(y0 - 2 + u, 0), ny - 1) * nx + xi];
    }
#pragma unroll
    for (int u = 0; u < kPH; ++u) T0[u][tid + 2] = v[u];
    if (tid < 4) {
#pragma unroll
        for (int u = 0; u < kPH; ++u) T0[u][xcol] = xv[u];
    }
    __syncthreads();

    // first step on the box and a one-cell ring (in-grid cells)
    auto step1 = [&](int ii, int col) {
        const int w = max(ii - 1, 0), e = min(ii + 1, nx - 1);
#pragma unroll
        for (int r = 0; r < kQH; ++r) {
            const int j = y0 - 1 + r;
            if (j < 0 || j >= ny) continue;
            const int js = max(j - 1, 0), jn = min(j + 1, ny - 1);
            T1[r][col] = stencil2d(t0(ii, j), t0(w, j), t0(e, j), t0(ii, js), t0(ii, jn), k);
        }
    };
    if (i < nx) step1(i, tid + 1);
    if (tid < 2) {
        const int ri = tid == 0 ? x0 - 1 : x0 + kRX;
        if (ri >= 0 && ri < nx) step1(ri, tid == 0 ? 0 : kRX + 1);
    }
    __syncthreads();
    // its sources (every listed cell is in the grid and appears once)
    const int q0 = a.src_start[box], q1 = a.src_start[box + 1];
    for (int q = q0 + tid; q < q1; q += kRX) (&T1[0][0])[a.src_pos[q]] += a.src_q[q];
    __syncthreads();

    // c^{n+1} out, then the second step on the box
    if (i < nx) {
        const int w = max(i - 1, 0), e = min(i + 1, nx - 1);
        const int rows = min(kPY, ny - y0);
        float* out1 = a.out1[s];
#pragma unroll
        for (int r = 0; r < kPY; ++r) {
            if (r >= rows) break;
            const int j = y0 + r;
            const int js = max(j - 1, 0), jn = min(j + 1, ny - 1);
            out1[(size_t)j * nx + i] = T1[r + 1][tid + 1];
            T2[r][tid] = stencil2d(t1(i, j), t1(w, j), t1(e, j), t1(i, js), t1(i, jn), k);
        }
    }
    __syncthreads();
    for (int q = q0 + tid; q < q1; q += kRX) {
        const int r = a.src_pos[q] / kQW, col = a.src_pos[q] % kQW;
        if (r >= 1 && r <= kPY && col >= 1 && col <= kRX) T2[r - 1][col - 1] += a.src_q[q];
    }
    __syncthreads();
    if (i < nx) {
        const int rows = min(kPY, ny - y0);
        float* out2 = a.out2[s];
#pragma unroll
        for (int r = 0; r < kPY; ++r) {
            if (r >= rows) break;
            out2[(size_t)(y0 + r) * nx + i] = T2[r][tid];
        }
    }
}

}  // namespace

hipError_t field2d_prepare(Field2DStep& f, int nx, int ny, int n_species,
                           const std::vector<int32_t>* cells, const std::vector<float>* q) {
    field2d_release(f);
    const Tiles2D t = tiles_for(nx, ny);
    const int n_boxes = n_species * t.tx * t.ty;
    // source entries per box, in row order (cells are unique per species)
    std::vector<std::vector<std::pair<int64_t, float>>> per_box(n_boxes);
    for (int s = 0; s < n_species; ++s)
        for (size_t m = 0; m < cells[s].size(); ++m) {
            const int i = cells[s][m] % nx, j = cells[s][m] / nx;
            const int box = (s * t.ty + j / kRY) * t.tx + i / kRX;
            per_box[box].push_back({(int64_t)j * kRX + i % kRX, q[s][m]});
        }
    std::vector<int32_t> start(n_boxes + 1, 0), row_of, col_of;
    std::vector<float> amount;
    for (int box = 0; box < n_boxes; ++box) {
        auto& v = per_box[box];
        std::sort(v.begin(), v.end(),
                  [](const std::pair<int64_t, float>& x, const std::pair<int64_t, float>& y) {
                      return x.first < y.first;
                  });
        for (auto& en : v) {
            row_of.push_back((int32_t)(en.first / kRX));
            col_of.push_back((int32_t)(en.first % kRX));
            amount.push_back(en.second);
        }
        start[box + 1] = (int32_t)row_of.size();
    }
    // two-step boxes: the sources on each box and its one-cell ring (a cell near a box edge
    // is listed by up to four boxes)
    const Tiles2D p = tiles_for(nx, ny, kPY);
    const int n_pair = n_species * p.tx * p.ty;
    std::vector<std::vector<std::pair<int32_t, float>>> per_pair(n_pair);
    for (int s = 0; s < n_species; ++s)
        for (size_t m = 0; m < cells[s].size(); ++m) {
            const int i = cells[s][m] % nx, j = cells[s][m] / nx;
            for (int by = std::max(j / kPY - 1, 0); by <= std::min(j / kPY + 1, p.ty - 1); ++by)
                for (int bx = std::max(i / kRX - 1, 0); bx <= std::min(i / kRX + 1, p.tx - 1);
                     ++bx) {
                    const int r = j - (by * kPY - 1), c = i - (bx * kRX - 1);
                    if (r < 0 || r >= kQH || c < 0 || c >= kQW) continue;
                    per_pair[(s * p.ty + by) * p.tx + bx].push_back({r * kQW + c, q[s][m]});
                }
        }
    std::vector<int32_t> pstart(n_pair + 1, 0), ppos;
    std::vector<float> pq;
    for (int b = 0; b < n_pair; ++b) {
        for (auto& en : per_pair[b]) {
            ppos.push_back(en.first);
            pq.push_back(en.second);
        }
        pstart[b + 1] = (int32_t)ppos.size();
    }
    UploadBlock up;
    const size_t at_start = up.add(start), at_row = up.add(row_of), at_col = up.add(col_of),
                 at_q = up.add(amount), at_pstart = up.add(pstart), at_ppos = up.add(ppos),
                 at_pq = up.add(pq);
    const hipError_t e = up.upload(&f.memory);
    if (e != hipSuccess) return e;
    f.src_start = (int32_t*)(f.memory + at_start);
    f.src_row = (int32_t*)(f.memory + at_row);
    f.src_col = (int32_t*)(f.memory + at_col);
    f.src_q = (float*)(f.memory + at_q);
    f.pair_start = (int32_t*)(f.memory + at_pstart);
    f.pair_pos = (int32_t*)(f.memory + at_ppos);
    f.pair_q = (float*)(f.memory + at_pq);
    f.n_pair_boxes = n_pair;
    f.nx = nx;
    f.ny = ny;
    f.n_species = n_species;
    f.n_boxes = n_boxes;
    return hipSuccess;
}

void field2d_release(Field2DStep& f) {
    device_free(f.memory);
    f = Field2DStep{};
}

Field2DStepArgs field2d_args(const Field2DStep& f, const float* const* in, float* const* out,
                             const StencilCoef* coef) {
    const Tiles2D t = tiles_for(f.nx, f.ny);
    Field2DStepArgs a = {};
    for (int s = 0; s < f.n_species; ++s) {
        a.in[s] = in[s];
        a.out[s] = out[s];
        a.coef[s] = coef[s];
    }
    a.nx = f.nx;
    a.ny = f.ny;
    a.n_species = f.n_species;
    a.tx = t.tx;
    a.ty = t.ty;
    a.per_xcd = (f.n_boxes + kXcds - 1) / kXcds;
    a.src_start = f.src_start;
    a.src_row = f.src_row;
    a.src_col = f.src_col;
    a.src_q = f.src_q;
    return a;
}

hipError_t launch_field2d_rows(const Field2DStep& f, const float* const* in, float* const* out,
                               const StencilCoef* coef, hipStream_t stream, hipEvent_t start,
                               hipEvent_t stop) {
    Field2DStepArgs a = field2d_args(f, in, out, coef);
    void* args[] = {&a};
    if (!start && !stop)   // a plain launch (also what a graph capture records)
        return hipLaunchKernel((const void*)k_field2d_rows, dim3(a.per_xcd * kXcds), dim3(kRX),
                               args, 0, stream);
    return hipExtLaunchKernel((const void*)k_field2d_rows, dim3(a.per_xcd * kXcds), dim3(kRX),
                              args, 0, stream, start, stop, 0);
}

hipError_t launch_field2d_pair(const Field2DStep& f, const float* const* in, float* const* out1,
                               float* const* out2, const StencilCoef* coef, hipStream_t stream) {
    const Tiles2D t = tiles_for(f.nx, f.ny, kPY);
    Field2DPairArgs a = {};
    for (int s = 0; s < f.n_species; ++s) {
        a.in[s] = in[s];
        a.out1[s] = out1[s];
        a.out2[s] = out2[s];
        a.coef[s] = coef[s];
    }
    a.nx = f.nx;
    a.ny = f.ny;
    a.n_species = f.n_species;
    a.tx = t.tx;
    a.ty = t.ty;
    a.per_xcd = (f.n_pair_boxes + kXcds - 1) / kXcds;
    a.src_start = f.pair_start;
    a.src_pos = f.pair_pos;
    a.src_q = f.pair_q;
    hipLaunchKernelGGL(k_field2d_pair, dim3(a.per_xcd * kXcds), dim3(kRX), 0, stream, a);
    return hipGetLastError();
}

}  // namespace cuesim
