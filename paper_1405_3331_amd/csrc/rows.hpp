// rows.hpp -- rows of cells held one segment per lane of a wavefront: access through
// global-address-space pointers, lane shifts, and the 2D stencil of one row.  Shared by the
// temporally blocked forward step and its reverse.
#pragma once

#include <hip/hip_runtime.h>

#include "internal.hpp"

namespace cuesim {

template <int CPL>
struct Row;
template <>
struct Row<2> {
    using T = float2;
};
template <>
struct Row<4> {
    using T = float4;
};

__device__ __forceinline__ float comp(const float2& v, int k) { return k == 0 ? v.x : v.y; }
__device__ __forceinline__ float comp(const float4& v, int k) {
    return k == 0 ? v.x : (k == 1 ? v.y : (k == 2 ? v.z : v.w));
}
__device__ __forceinline__ void set_comp(float2& v, int k, float x) {
    if (k == 0) v.x = x; else v.y = x;
}
__device__ __forceinline__ void set_comp(float4& v, int k, float x) {
    if (k == 0) v.x = x; else if (k == 1) v.y = x; else if (k == 2) v.z = x; else v.w = x;
}

// Global-address-space view of a pointer held in a table: loads and stores through it are
// global (vector-memory only) rather than flat accesses, which would also count against
// the LDS wait counter.
template <class T>
using GlobalPtr = __attribute__((address_space(1))) T*;
template <class T>
__device__ __forceinline__ GlobalPtr<T> gbl(T* p) {
    return (GlobalPtr<T>)p;
}
// HIP's vector structs do not bind to address-space-qualified references: move them as
// clang vectors.
using f4v = float __attribute__((ext_vector_type(4)));
using i2v = int __attribute__((ext_vector_type(2)));
using i4v = int __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 gload(GlobalPtr<const float4> p) {
    const f4v v = *(GlobalPtr<const f4v>)p;
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ int2 gload(GlobalPtr<const int2> p) {
    const i2v v = *(GlobalPtr<const i2v>)p;
    return make_int2(v.x, v.y);
}
__device__ __forceinline__ void gstore(GlobalPtr<float4> p, float4 v) {
    *(GlobalPtr<f4v>)p = f4v{v.x, v.y, v.z, v.w};
}

// One tile row segment of CPL floats per lane: row gy, columns gx0 .. gx0 + CPL - 1 of the
// field, read at indices clamped into the grid, so every lane loads and nothing branches
// between the loads of a batch; cells outside the grid are zeroed when the segment is
// stored (store_row).  With ALIGNED (the segment starts at a multiple of CPL and the row
// length is one) the segment lies wholly inside or wholly outside the grid's columns and is
// one naturally aligned vector load.
template <int CPL>
using RowVec = float __attribute__((ext_vector_type(CPL)));

template <int CPL, bool ALIGNED>
__device__ __forceinline__ RowVec<CPL> load_row(GlobalPtr<const float> f, int nx, int ny,
                                                int gy, int gx0) {
    const size_t at = (size_t)min(max(gy, 0), ny - 1) * nx;
    if (ALIGNED) return *(GlobalPtr<const RowVec<CPL>>)(f + at + min(max(gx0, 0), nx - CPL));
    RowVec<CPL> v;
#pragma unroll
    for (int k = 0; k < CPL; ++k) v[k] = f[at + min(max(gx0 + k, 0), nx - 1)];
    return v;
}

// Value held by the lane below (lane_from_left) or above (lane_from_right) in the
// wavefront: a whole-wave DPP shift by one lane, which moves data between lanes inside the
// VALU instead of through the LDS crossbar.  Lane 0 (resp. 63) receives 0; it holds the
// tile's outermost column, which is never valid after the first sub-step.  That 0 comes from
// the shift's own bound control and not from a zeroed destination, so the compiler folds the
// shift into the addition that takes its result: 12 instead of 16 VALU instructions per row
// of two cells, and the stencil is bound by them.
__device__ __forceinline__ float lane_from_left(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138 /* wave_shr:1 */,
                                                      0xF, 0xF, true));
}
__device__ __forceinline__ float lane_from_right(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130 /* wave_shl:1 */,
                                                      0xF, 0xF, true));
}

// How a tile meets the grid's first and last column (the zero-flux rule: a missing
// neighbour is the cell itself).  kWallAligned: every lane's segment starts at a multiple of
// CPL and so does nx, so column 0 can only be a segment's first cell and column nx - 1 a
// segment's last, and only the neighbours taken from the adjacent lanes need the rule.
enum ColumnWalls { kNoWall = 0, kWallAligned = 1, kWallAny = 2 };

// Laplacian sum (the four neighbours minus four times the cell) of the CPL cells of one row
// from the rows above (s), at (c) and below (n).  Horizontal neighbours across lanes come
// from the adjacent lanes' registers.  COLS applies the zero-flux rule at the grid's first
// and last column; at the first and last row the caller passes the row itself as the missing
// neighbour.
template <int CPL, int COLS>
__device__ __forceinline__ typename Row<CPL>::T row_laplacian(const typename Row<CPL>::T& s,
                                                              const typename Row<CPL>::T& c,
                                                              const typename Row<CPL>::T& n,
                                                              int gx0, int nx) {
    using V = typename Row<CPL>::T;
    float left = lane_from_left(comp(c, CPL - 1));   // column cx - 1
    float right = lane_from_right(comp(c, 0));       // column cx + CPL
    if (COLS == kWallAligned) {
        if (gx0 == 0) left = comp(c, 0);
        if (gx0 + CPL == nx) right = comp(c, CPL - 1);
    }
    V lap;
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
        const float ck = comp(c, k);
        float w = k == 0 ? left : comp(c, k - 1);
        float e = k == CPL - 1 ? right : comp(c, k + 1);
        if (COLS == kWallAny) {
            if (gx0 + k == 0) w = ck;
            if (gx0 + k == nx - 1) e = ck;
        }
        set_comp(lap, k, fmaf(-4.0f, ck, (w + e) + (comp(s, k) + comp(n, k))));
    }
    return lap;
}

// New value of the CPL cells of one row: diffusion and decay from the old rows.
template <int CPL, int COLS>
__device__ __forceinline__ typename Row<CPL>::T row_update(const typename Row<CPL>::T& s,
                                                           const typename Row<CPL>::T& c,
                                                           const typename Row<CPL>::T& n,
                                                           int gx0, int nx, StencilCoef cf) {
    using V = typename Row<CPL>::T;
    const V lap = row_laplacian<CPL, COLS>(s, c, n, gx0, nx);
    V nv;
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
        const float ck = comp(c, k);
        set_comp(nv, k, fmaf(cf.r, comp(lap, k), fmaf(-cf.kdt, ck, ck)));
    }
    return nv;
}

}  // namespace cuesim
