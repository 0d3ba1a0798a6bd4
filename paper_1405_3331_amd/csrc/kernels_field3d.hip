// kernels_field3d.hip -- one explicit step of every species of a 3D field, sources included.
//
// 7-point stencil with first-order decay, zero-flux walls (a missing neighbour is the cell
// itself), then the point sources of the step (c' += q / dx^3).  One launch covers every
// species.  A workgroup owns a box of kTX x kTY columns and 8 or 4 consecutive planes of one
// species and marches up the planes; each thread keeps the planes below, at and above its cell in
// registers and reads the four in-plane neighbours from lines the workgroup has just brought into
// L1/L2, so a cell is fetched from HBM about once per step: 8 algorithmic bytes per
// species-cell-update.
// Planes are taken kUnroll3D at a time with every load of the group issued before the
// arithmetic, which keeps kUnroll3D times more reads in flight than a plane-by-plane march.
// Walls are handled by clamping the neighbour index, which reads the cell itself exactly
// where the ghost value is the cell's own.
//
// Boxes are dealt to the accelerator dies in contiguous stretches (workgroups are assigned
// to dies round-robin), so boxes that share halo rows usually share an L2.
//
// The sources of a box are a short list (plane, thread, amount) built once on the host and
// sorted by plane; every thread walks it with the march and adds the amounts of its own
// cells after the stencil, as a separate FP32 add (the same rounding as a source pass).
#include <hip/hip_ext.h>

#include <algorithm>
#include <vector>

#include "field_step.hpp"
#include "internal.hpp"
#include "memory.hpp"

namespace cuesim {

namespace {

// Planes per box: kDeep, or kUnroll3D where that leaves CUs without a box.  More planes per box
// read fewer planes twice, fewer put more boxes in flight and keep a die's boxes closer
// together.  Per step, 4 / 8 / 16 planes: 97 x 64 x 51 4.0 / 4.3 / 5.6 us; 128^3 6.4 / 6.1 /
// 6.3; 160^3 10.1 / 8.5 / 9.0; 200^3 17.3 / 13.5 / 15.6; 256^3 25.5 / 21.5 / 23.5, with two
// species 50.4 / 41.4 / 43.4.
constexpr int kDeep = 8;
constexpr int kDeepBoxes = 256;   // CUs
constexpr int64_t kMostBoxes = 1 << 22;

struct Boxes {
    int tx, ty, tz, planes;   // boxes per axis, planes per box
    int per_species() const { return tx * ty * tz; }
};

Boxes boxes_for(int nx, int ny, int nz, int n_species) {
    Boxes b{(nx + kTX - 1) / kTX, (ny + kTY - 1) / kTY, (nz + kDeep - 1) / kDeep, kDeep};
    if (n_species * b.per_species() < kDeepBoxes) {
        b.planes = kUnroll3D;
        b.tz = (nz + kUnroll3D - 1) / kUnroll3D;
    }
    // (a launch holds fewer than 2^32 threads: thin volumes of tens of millions of planes)
    while (b.tz > 1 && (int64_t)n_species * b.tx * b.ty * b.tz > kMostBoxes) {
        b.planes *= 2;
        b.tz = (nz + b.planes - 1) / b.planes;
    }
    return b;
}

__global__ __launch_bounds__(kBoxThreads3D) void k_field3d(Field3DArgs a) {
    const int n_boxes = a.n_species * a.tx * a.ty * a.tz;
    const int box = (blockIdx.x % kXcds) * a.per_xcd + blockIdx.x / kXcds;
    if (box >= n_boxes) return;
    field3d_box(a, box, threadIdx.x);
}

}  // namespace

hipError_t field3d_prepare(Field3D& f, int nx, int ny, int nz, int n_species,
                           const std::vector<int32_t>* cells, const std::vector<float>* q) {
    field3d_release(f);
    const Boxes b = boxes_for(nx, ny, nz, n_species);
    const int n_boxes = n_species * b.per_species();
    // source entries per box, in plane order (cells are unique per species)
    std::vector<std::vector<std::pair<int64_t, float>>> per_box(n_boxes);
    for (int s = 0; s < n_species; ++s)
        for (size_t m = 0; m < cells[s].size(); ++m) {
            const int64_t cell = cells[s][m];
            const int i = (int)(cell % nx), j = (int)((cell / nx) % ny),
                      l = (int)(cell / ((int64_t)nx * ny));
            const int box = ((s * b.tz + l / b.planes) * b.ty + j / kTY) * b.tx + i / kTX;
            const int tid = (j % kTY) * kTX + i % kTX;
            per_box[box].push_back({(int64_t)l * kBoxThreads3D + tid, q[s][m]});
        }
    std::vector<int32_t> start(n_boxes + 1, 0), plane_of, thread_of;
    std::vector<float> amount;
    for (int box = 0; box < n_boxes; ++box) {
        auto& v = per_box[box];
        std::sort(v.begin(), v.end(),
                  [](const std::pair<int64_t, float>& x, const std::pair<int64_t, float>& y) {
                      return x.first < y.first;
                  });
        for (auto& en : v) {
            plane_of.push_back((int32_t)(en.first / kBoxThreads3D));
            thread_of.push_back((int32_t)(en.first % kBoxThreads3D));
            amount.push_back(en.second);
        }
        start[box + 1] = (int32_t)plane_of.size();
    }
    UploadBlock up;
    const size_t at_start = up.add(start), at_plane = up.add(plane_of),
                 at_thread = up.add(thread_of), at_q = up.add(amount);
    const hipError_t e = up.upload(&f.memory);
    if (e != hipSuccess) return e;
    f.src_start = (int32_t*)(f.memory + at_start);
    f.src_plane = (int32_t*)(f.memory + at_plane);
    f.src_thread = (int32_t*)(f.memory + at_thread);
    f.src_q = (float*)(f.memory + at_q);
    f.nx = nx;
    f.ny = ny;
    f.nz = nz;
    f.n_species = n_species;
    f.n_boxes = n_boxes;
    return hipSuccess;
}

void field3d_release(Field3D& f) {
    device_free(f.memory);
    f = Field3D{};
}

Field3DArgs field3d_args(const Field3D& f, const float* const* in, float* const* out,
                         const StencilCoef* coef) {
    const Boxes b = boxes_for(f.nx, f.ny, f.nz, f.n_species);
    Field3DArgs a = {};
    for (int s = 0; s < f.n_species; ++s) {
        a.in[s] = in[s];
        a.out[s] = out[s];
        a.coef[s] = coef[s];
    }
    a.nx = f.nx;
    a.ny = f.ny;
    a.nz = f.nz;
    a.n_species = f.n_species;
    a.tx = b.tx;
    a.ty = b.ty;
    a.tz = b.tz;
    a.planes = b.planes;
    a.per_xcd = (f.n_boxes + kXcds - 1) / kXcds;
    a.src_start = f.src_start;
    a.src_plane = f.src_plane;
    a.src_thread = f.src_thread;
    a.src_q = f.src_q;
    return a;
}

hipError_t launch_field3d(const Field3D& f, const float* const* in, float* const* out,
                          const StencilCoef* coef, hipStream_t stream, hipEvent_t start,
                          hipEvent_t stop) {
    Field3DArgs a = field3d_args(f, in, out, coef);
    void* args[] = {&a};
    return hipExtLaunchKernel((const void*)k_field3d, dim3(a.per_xcd * kXcds), dim3(kBoxThreads3D),
                              args, 0, stream, start, stop, 0);
}

}  // namespace cuesim
