// Internal declarations shared by the host API and the HIP kernels of libmf.so.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>
#include <string>
#include <vector>

#include "mf.h"

// Library-owned state of one pattern (Sec. 2.2 Block B).
struct mf_pattern_s {
    int dim = 0, nen = 0, nf = 0;
    int order = 1;  // element order: 2 for the serendipity elements
    mf_numbering numbering = MF_NODE_MAJOR;
    int64_t n_nodes = 0, n_elems = 0, n_rows = 0, nnz = 0, n_pairs = 0;
    uint8_t coupling[16] = {0};
    bool full_coupling = false;
    // device arrays, in two allocations (pattern.hip)
    void* mem[2] = {nullptr, nullptr};
    int32_t* conn = nullptr;     // [nen][n_elems] copy of the caller's connectivity
    int32_t* nbr_ptr = nullptr;  // [n_nodes+1] node graph offsets
    int32_t* nbr = nullptr;      // [n_pairs] sorted neighbours N(v)
    int32_t* row_ptr = nullptr;  // [n_rows+1]
    int32_t* col_idx = nullptr;  // [nnz]
    uint8_t* rank = nullptr;     // [nen*nen][n_elems]
    // node-element incidence: entry e*nen + a for every element e with node v at local
    // position a, ascending within adj[adj_ptr[v] .. adj_ptr[v+1])
    int32_t* adj_ptr = nullptr;  // [n_nodes+1]
    int32_t* adj = nullptr;      // [nen*n_elems]
    uint8_t* rank_t = nullptr;   // rank element by element: [n_elems][nen][nen]
    int max_deg = 0;             // largest neighbour count of a node
    bool scattered = false;      // many consecutive nodes have elements far apart
    // assembly workspace, grown on first use and owned by the pattern: per-element records
    // written by one kernel of a call and read by its next.  ws_done marks the end of the
    // last call that used it, so that a call on another stream waits for it.
    char* ws = nullptr;
    size_t ws_bytes = 0;
    hipEvent_t ws_done = nullptr;
    // held from a call's first kernel that uses the workspace to its last, and while the
    // colouring is made
    std::mutex ws_mu;
    // workspaces of captured calls: at least one for each capture and stream in it
    struct Captured {
        char* p;
        size_t bytes;
        unsigned long long id;
        hipStream_t s;
    };
    std::vector<Captured> cap_ws;
    unsigned long long* status = nullptr;  // [3] first element with det J <= 0, first bad face, first element
                                           // with a non-finite input or coefficient (each ~0 when none)
    // element colouring (no two elements of one colour share a node), made on first use:
    // the elements of colour c are color_elems[color_ptr[c] .. color_ptr[c+1])
    int32_t* color_elems = nullptr;  // device [n_elems]
    int32_t* elem_color = nullptr;   // device [n_elems]: colour of each element
    std::vector<int64_t> color_ptr;
    int64_t* color_at = nullptr;  // device copy of color_ptr
    // face lists (boundary.hip) of the captured calls that come after kCaptured captures
    uint32_t* shared_faces = nullptr;
    // structured lexicographic grid detection
    int is_grid = 0;
    int64_t gx = 0, gy = 0, gz = 0;
    hipStream_t last_stream = nullptr;
};

namespace mf {

// While it lives, this thread may allocate and copy although a stream is being captured.
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    RelaxedCapture();
    ~RelaxedCapture();
};

// A stream of its own for setup that ends before the call goes on, also under capture.
struct SideStream : RelaxedCapture {
    hipStream_t s = nullptr;
    hipError_t status = hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
    ~SideStream()
    {
        if (s) (void)hipStreamDestroy(s);
    }
};

mf_status set_error(mf_status s, const char* fmt, ...);
mf_status hip_error(hipError_t e, const char* what);
void clear_error();  // empties the thread's last-error message

// The error that a pattern's status words stand for.
mf_status status_of(const unsigned long long (&v)[3], int64_t* first_bad_elem);

#define MF_HIP(call)                                            \
    do {                                                        \
        hipError_t e_ = (call);                                 \
        if (e_ != hipSuccess) return ::mf::hip_error(e_, #call); \
    } while (0)

// pattern.hip
mf_status build_pattern(mf_pattern_s* P, const int32_t* conn_in, hipStream_t s);
// greedy element colouring, cached in the pattern (sync on first call)
mf_status ensure_coloring(const mf_pattern_s* P);

struct PcgArgs;
// mf_bicgstab; with P (the pattern whose CSR structure A uses) the SpMV of node-major
// 4-field rows reads its columns from P's node graph
mf_status bicgstab_on_pattern(const mf_csr* A, const mf_pattern_s* P, const double* b, double* x,
                              const mf_pcg_opts* opts, mf_pcg_result* res, void* stream);
mf_status nn_bind_pcg(const mf_nn_t* net, int64_t n_rows, PcgArgs* a);
// multigrid.hip: one V-cycle as the external preconditioner of a solve on `values`
mf_status mg_bind_pcg(const mf_mg_t* mg, int64_t n_rows, const double* values, PcgArgs* a);
// the cycle for A = wa Ka + wb Kb (scalar forms; fa with elem_param) with the Dirichlet
// elimination on every level, A0 the level-0 operator (sync)
mf_status mg_update_combined(mf_mg_t* mg, const mf_form* fa, const double* elem_param, double wa,
                             const mf_form* fb, double wb, const double* coords, const uint8_t* dirichlet,
                             const mf_quadrature* quad, const double* A0, hipStream_t s);

// assemble.hip
struct AssembleArgs {
    const mf_pattern_s* P;
    const mf_form* form;
    const double* coords;
    const void* elem_param;
    const void* nodal_src;
    const void* lin_state;
    const uint8_t* dirichlet;
    mf_precision prec;
    void* K;
    void* d;
    hipStream_t stream;
};
// element-parallel scatter: hardware atomics, or colour by colour with plain adds
// (deterministic sums)
mf_status assemble_atomic(const AssembleArgs& a, bool coloured);
// assemble_quads.hip: owner-computes rows on any mesh of 4-node quadrilaterals, with the
// status reset and the Dirichlet elimination.  MF_ERR_UNSUPPORTED (nothing launched, no error recorded) for other
// elements and for meshes with hundreds of neighbours at a node.
mf_status assemble_quads(const AssembleArgs& a);
// assemble_quadratic.hip: the quadratic elements, and the flow form on 8-node bricks where it
// goes colour by colour; *eliminated: the Dirichlet elimination is done
mf_status assemble_quadratic(const AssembleArgs& a, bool* eliminated);
mf_status assemble_column(const AssembleArgs& a);
// assemble_rows.hip: owner-computes rows on any mesh of 8-node bricks, from element records
// in the pattern's workspace; applies the Dirichlet elimination.  MF_ERR_UNSUPPORTED (nothing
// launched, no error recorded) for other elements and where no workspace can be had.
mf_status assemble_rows(const AssembleArgs& a);
// The pattern's workspace of at least `bytes` for kernels queued on the stream during its
// lifetime (calls that are being captured get one of their own).  p is nullptr when there is
// no memory for it, or kCaptured captures have one already.  Those stay until the pattern goes: a
// graph may be replayed for as long, and nothing that HIP offers tells when it no longer can be (a
// user object of the graph is not kept by an executable graph that was updated from it).
struct Workspace {
    static constexpr size_t kCaptured = 8;
    mf_pattern_s* P;
    hipStream_t s;
    std::unique_lock<std::mutex> lock;
    char* p = nullptr;
    bool record = false;
    bool full = false;  // kCaptured other captures have one: that is why p is nullptr
    Workspace(const mf_pattern_s* P, size_t bytes, hipStream_t stream);
    ~Workspace();
    Workspace(const Workspace&) = delete;
};
mf_status apply_dirichlet(const AssembleArgs& a);
mf_status reset_status(const mf_pattern_s* P, hipStream_t s);

// batched persistent launch (assemble_column.hip)
mf_status batch_check(const AssembleArgs& a);
// chunks[k]: problem k's columns are cut into that many work items along z (the tile
// height); xw[k]: their cross-section, 4 (4x2 nodes) or 2 (2x4); *dev_probs and
// *dev_status are allocated on the first call, reused after
mf_status batch_upload(const std::vector<AssembleArgs>& probs, const std::vector<int>& chunks,
                       const std::vector<int>& xw, void** dev_probs, void** dev_status);
int64_t batch_units_of(const mf_pattern_s* P, int chunks, int xw);
// items [0, n_first) belong to one kernel (elasticity when first_elastic), the rest to the
// other (mass and Poisson); counter holds two ints
mf_status batch_launch(const void* dev_probs, void* dev_status, int n_probs, const int2* items, int n_first,
                       int n_items, bool first_elastic, int* counter, int n_wg, mf_precision prec, bool masked,
                       hipStream_t s);
// workgroups per CU the batched kernel is built for
int batch_max_wg_per_cu(mf_precision prec);

inline unsigned blocks_for(int64_t n, int threads) {
    return (unsigned)((n + threads - 1) / threads);
}

}  // namespace mf
