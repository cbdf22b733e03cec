// Shared by the owner-computes kernels (assemble_rows.hip, assemble_quadratic.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "element.h"
#include "mf_internal.h"

namespace mf {

constexpr int kXcds = 8;

// Workgroups are dealt to the eight XCDs in turn; the renumbered block index gives each XCD
// one contiguous eighth of the nodes, whose shared elements then come from one L2.
__device__ __forceinline__ unsigned xcd_block(unsigned b, unsigned n)
{
    const unsigned per = n / kXcds, rest = n % kXcds, x = b % kXcds, k = b / kXcds;
    return x * per + (x < rest ? x : rest) + k;
}

// Which elements have a constrained DOF (one byte each), so that the waves that sum
// the rows look up Dirichlet flags only around those.
struct ElemMask {
    const uint8_t* mask;  // [n_rows] or nullptr
    uint8_t* flag;        // [n_elems]
    int64_t n_nodes;
    int field_major;
    template <int NF>
    __device__ __forceinline__ bool node(int64_t v) const
    {
        bool on = false;
#pragma unroll
        for (int j = 0; j < NF; ++j) on |= mask[field_major ? j * n_nodes + v : NF * v + j] != 0;
        return on;
    }
};

// K and d from the blocks (and residual entries) of all elements in the workspace, in A's
// precision; emask: the elements' flags (with A.dirichlet).  Ke [e][a][i][b][j] (elasticity:
// E int dN_a,i dN_b,j, combined by the gather), fe [e][a][i].  Eliminates the Dirichlet rows.
mf_status gather_blocks(const AssembleArgs& A, int nen, int nf, const void* Ke, const void* fe, const uint8_t* emask);

}  // namespace mf
