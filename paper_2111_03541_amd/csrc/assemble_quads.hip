// Owner-computes rows of 4-node quadrilaterals on any mesh (Sec. 2.2 D-2, D-3), in one launch.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "element.h"
#include "mf_internal.h"

namespace mf {
namespace {

constexpr int kWave = 64;
constexpr int kSlots = 4;                 // lanes of a row
constexpr int kRows = kWave / kSlots;     // rows of a wave
// Few rows go as one workgroup that resets the status itself, in one launch: 9.5 us with all host work
// (1 x 1 to 15 x 15 conduction; 18 x 18 9.8, with constrained sides 11.4) against 12.4 in two (12.6).  More
// rows go as one wave per workgroup after the reset's launch, so that they spread over the chip: in
// one workgroup 21 x 21 take 12.8 and 15.0 us, and elasticity on 6 x 6, of 98 rows, in two passes of four
// waves 15.5.
template <int FORM>
struct Alone {
    static constexpr bool SCALAR = FORM == MF_FORM_MASS || FORM == MF_FORM_POISSON;
    static constexpr int WAVES = SCALAR ? 16 : 4;  // of the workgroup
    static constexpr int MOST = SCALAR ? 24 : 4;   // passes of a wave over kRows rows, in all waves
};

struct QuadParams {
    mf_form form;
    int64_t n_el, n_nodes, n_rows;
    const int32_t* conn;
    const double* coords;
    const int32_t* row_ptr;
    const int32_t* col_idx;
    const int32_t* adj_ptr;
    const int32_t* adj;
    const uint8_t* rank_t;
    const void* elem_param;
    const void* src;  // nodal sources (mass, conduction, elasticity) or state (flow)
    const uint8_t* mask;
    int field_major, max_deg;
    void* K;
    void* d;
    unsigned long long* status;
};

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Lane (row, slot): integrates the row over every fourth element around its node, in T; the
// slots take turns to add onto the row's FP64 sums in LDS, so each entry is the sum over the
// elements in ascending order.  The wave's rows are consecutive, and their values one run of K.
// Small meshes are a latency chain (incidence, connectivity, coordinates, the sums, the stores):
// conduction on 32^2 12 us a call, of which the launches take most, against 37 in one workgroup
// colour by colour; flow 32^2 13 against 654.  Large ones are bound by the FP64 geometry, formed
// for each row: conduction 1024^2 119 us against 332, flow 1620 against 3309.
template <int FORM, typename T, bool ALONE>
__global__ void __launch_bounds__((ALONE ? Alone<FORM>::WAVES : 1) * kWave) k_quad_rows(QuadParams p)
{
    constexpr int NEN = 4;
    constexpr int NF = FormTraits<FORM, 2>::NF;
    constexpr int NSRC = FormTraits<FORM, 2>::NSRC;
    extern __shared__ double lds[];
    if constexpr (ALONE) {
        if (threadIdx.x < 3) p.status[threadIdx.x] = ~0ull;
        __syncthreads();
    }
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave, slot = lane % kSlots;
    // [values of the wave's rows], then [kRows] of d
    double* const buf = lds + wave * kRows * (NF * p.max_deg + 1);
    const int n_waves = blockDim.x / kWave;
    for (int64_t r0 = ((int64_t)blockIdx.x * n_waves + wave) * kRows; r0 < p.n_rows; r0 += (int64_t)gridDim.x * n_waves * kRows) {
        const int64_t r1 = min(r0 + kRows, p.n_rows);
        const int64_t r = min(r0 + lane / kSlots, r1 - 1);
        const bool live = r0 + lane / kSlots < r1;
        const int64_t va = p.field_major ? r % p.n_nodes : r / NF;
        const int i = (int)(p.field_major ? r / p.n_nodes : r % NF);
        const int a0 = p.adj_ptr[va], n_adj = live ? p.adj_ptr[va + 1] - a0 : 0;
        const int64_t k0 = p.row_ptr[r0], rs = p.row_ptr[r];
        const int len = (int)(p.row_ptr[r + 1] - rs), deg = len / NF, total = (int)(p.row_ptr[r1] - k0);
        double* const row = buf + (rs - k0);
        double* const dsum = buf + kRows * NF * p.max_deg;
        for (int k = lane; k < total; k += kWave) buf[k] = 0.0;
        if (lane < kRows) dsum[lane] = 0.0;
        wave_sync();
        const T* src = (const T*)p.src;
        for (int s0 = 0; __any(s0 < n_adj); s0 += kSlots) {
            const bool on = s0 + slot < n_adj;
            T krow[NEN * NF];
            T rrow = T(0);
#pragma unroll
            for (int k = 0; k < NEN * NF; ++k) krow[k] = T(0);
            int at[NEN] = {0, 0, 0, 0};
            if (on) {
                const int32_t ent = p.adj[a0 + s0 + slot];
                const int64_t e = ent / NEN;
                const int a = ent % NEN;
                const uint32_t rk = *(const uint32_t*)(p.rank_t + (int64_t)ent * NEN);
                double x[NEN][2];
                T U[NEN][NSRC];
#pragma unroll
                for (int b = 0; b < NEN; ++b) {
                    const int64_t node = p.conn[b * p.n_el + e];
#pragma unroll
                    for (int m = 0; m < 2; ++m) x[b][m] = p.coords[m * p.n_nodes + node];
#pragma unroll
                    for (int s = 0; s < NSRC; ++s) U[b][s] = src ? src[s * p.n_nodes + node] : T(0);
                    at[b] = (int)(rk >> 8 * b & 255u) * (p.field_major ? 1 : NF);
                }
                const Coef<T> C = make_coef<T>(FORM, p.form, p.elem_param ? (double)((const T*)p.elem_param)[e] : 1.0);
                bool bad = false;
#pragma unroll
                for (int q = 0; q < NEN; ++q) {  // 2 x 2 Gauss points, unit weights
                    double gd[NEN][2];
                    const double det = geometry_at<2>(x, q, gd);
                    bad |= !(det > 0.0);
                    T N[NEN], g[NEN][2];
#pragma unroll
                    for (int b = 0; b < NEN; ++b) {
                        N[b] = (T)ref_N<2>(b, q);
#pragma unroll
                        for (int m = 0; m < 2; ++m) g[b][m] = (T)gd[b][m];
                    }
                    row_update<FORM, 2, T>(a, i, C, N, g, (T)det, U, krow, rrow);
                }
                T chk = rrow;
#pragma unroll
                for (int k = 0; k < NEN * NF; ++k) chk += krow[k];
                if (bad) atomicMin(p.status, (unsigned long long)e);
                else if (!isfinite(chk)) atomicMin(p.status + 2, (unsigned long long)e);
                if (bad) {  // such an element adds nothing
#pragma unroll
                    for (int k = 0; k < NEN * NF; ++k) krow[k] = T(0);
                    rrow = T(0);
                }
            }
            const int step = p.field_major ? deg : 1;
            for (int turn = 0; turn < kSlots; ++turn) {
                if (on && turn == slot) {
#pragma unroll
                    for (int b = 0; b < NEN; ++b)
#pragma unroll
                        for (int j = 0; j < NF; ++j) row[at[b] + j * step] += (double)krow[b * NF + j];
                    dsum[lane / kSlots] -= (double)rrow;
                }
                wave_sync();
            }
        }
        // homogeneous Dirichlet elimination: a constrained row becomes a unit row with d = 0, a
        // constrained column is zeroed in the other rows
        if (p.mask && live) {
            const bool fixed = p.mask[r] != 0;
            for (int k = slot; k < len; k += kSlots) {
                const int32_t c = p.col_idx[rs + k];
                if (fixed) row[k] = c == r ? 1.0 : 0.0;
                else if (p.mask[c]) row[k] = 0.0;
            }
            if (fixed && slot == 0) dsum[lane / kSlots] = 0.0;
        }
        wave_sync();
        T* K = (T*)p.K + k0;
        for (int k = lane; k < total; k += kWave) K[k] = (T)buf[k];
        if (lane < (int)(r1 - r0)) ((T*)p.d)[r0 + lane] = (T)dsum[lane];
        wave_sync();
    }
}

template <int FORM, typename T>
mf_status launch_quads(const AssembleArgs& A)
{
    const mf_pattern_s* P = A.P;
    QuadParams p{};
    p.form = *A.form;
    p.n_el = P->n_elems;
    p.n_nodes = P->n_nodes;
    p.n_rows = P->n_rows;
    p.conn = P->conn;
    p.coords = A.coords;
    p.row_ptr = P->row_ptr;
    p.col_idx = P->col_idx;
    p.adj_ptr = P->adj_ptr;
    p.adj = P->adj;
    p.rank_t = P->rank_t;
    p.elem_param = A.elem_param;
    p.src = FORM == MF_FORM_NS_SUPG ? A.lin_state : A.nodal_src;
    p.mask = A.dirichlet;
    p.field_major = P->numbering == MF_FIELD_MAJOR;
    p.max_deg = std::max(1, P->max_deg);
    p.K = A.K;
    p.d = A.d;
    p.status = P->status;
    const size_t lds = sizeof(double) * kRows * ((size_t)P->nf * p.max_deg + 1);  // a wave's
    if (lds > 65536) return MF_ERR_UNSUPPORTED;
    const int64_t waves = (P->n_rows + kRows - 1) / kRows;
    const int64_t alone = std::min<int64_t>(waves, Alone<FORM>::WAVES);
    if (waves <= Alone<FORM>::MOST && lds * (size_t)alone <= 65536) {
        k_quad_rows<FORM, T, true><<<1, (unsigned)alone * kWave, lds * (size_t)alone, A.stream>>>(p);
    } else {
        const mf_status st = reset_status(P, A.stream);
        if (st != MF_OK) return st;
        k_quad_rows<FORM, T, false><<<(unsigned)waves, kWave, lds, A.stream>>>(p);
    }
    MF_HIP(hipGetLastError());
    return MF_OK;
}

template <typename T>
mf_status dispatch_quads(const AssembleArgs& A)
{
    switch (A.form->kind) {
        case MF_FORM_MASS: return launch_quads<MF_FORM_MASS, T>(A);
        case MF_FORM_POISSON: return launch_quads<MF_FORM_POISSON, T>(A);
        case MF_FORM_ELASTICITY: return launch_quads<MF_FORM_ELASTICITY, T>(A);
        case MF_FORM_NS_SUPG: return launch_quads<MF_FORM_NS_SUPG, T>(A);
    }
    return MF_ERR_UNSUPPORTED;
}

}  // namespace

mf_status assemble_quads(const AssembleArgs& A)
{
    const mf_pattern_s* P = A.P;
    if (P->dim != 2 || P->nen != 4 || P->n_elems == 0 || !P->full_coupling) return MF_ERR_UNSUPPORTED;
    return A.prec == MF_F64 ? dispatch_quads<double>(A) : dispatch_quads<float>(A);
}

}  // namespace mf
