// Rows of a scalar operator on a structured grid of 8-node bricks: 27 values per node, slot by
// slot, with the columns implied by the grid (multigrid.hip, pcg.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "mf.h"

namespace mf {

// Slot k = (dx+1) + 3 (dy+1) + 9 (dz+1) of node i holds its entry for the neighbour at
// (dx, dy, dz), at v[k * n + i]; 0 where the grid has none.  Slots ascend with the columns, so a
// row's products are summed in the order of its CSR row.
struct Stencil {
    int32_t sx = 0, sy = 0, sz = 0;  // nodes per axis
    const double* v = nullptr;
};

// Position of node i on each axis.
__device__ __forceinline__ void stencil_node(const Stencil& S, uint32_t i, int& ix, int& iy, int& iz)
{
    const uint32_t r = i / (uint32_t)S.sx;
    ix = (int)(i - r * (uint32_t)S.sx);
    iz = (int)(r / (uint32_t)S.sy);
    iy = (int)(r - (uint32_t)iz * (uint32_t)S.sy);
}

// sum over the row of node i; a slot past the grid's side reads a neighbour that the row has, with
// weight 0
__device__ __forceinline__ double stencil_dot(const Stencil& S, int32_t i, const double* __restrict__ x)
{
    int ix, iy, iz;
    stencil_node(S, (uint32_t)i, ix, iy, iz);
    const int64_t n = (int64_t)S.sx * S.sy * S.sz;
    const int dx[3] = {ix > 0 ? -1 : 0, 0, ix + 1 < S.sx ? 1 : 0};
    const int dy[3] = {iy > 0 ? -S.sx : 0, 0, iy + 1 < S.sy ? S.sx : 0};
    const int dz[3] = {iz > 0 ? -S.sx * S.sy : 0, 0, iz + 1 < S.sz ? S.sx * S.sy : 0};
    double v[27], in[27];
#pragma unroll
    for (int k = 0; k < 27; ++k) {
        v[k] = S.v[k * n + i];
        in[k] = x[i + dz[k / 9] + dy[k / 3 % 3] + dx[k % 3]];
    }
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 27; ++k) s = fma(v[k], in[k], s);
    return s;
}

// The level's values from its CSR rows, with the inverse diagonal when dinv is given (0 where the
// diagonal is 0).
void stencil_values(const Stencil& S, const int32_t* row_ptr, const double* A, double* v, double* dinv, hipStream_t s);

// Whether S.v holds the values of the CSR rows, bit for bit (sync; flag: device scratch).
mf_status stencil_holds(const Stencil& S, const int32_t* row_ptr, const double* A, int* flag, hipStream_t s, bool* same);

}  // namespace mf
