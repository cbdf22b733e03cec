// Boundary forms: the physics one dimension lower (Sec. 2.2 opening of the algorithm),
// integrated over element faces and added into an assembled K and d.  The forms are the
// ones of Sec. 4.1 (convection, radiation, penalty fix with its flux term), Sec. 4.2
// (load traction, penalty fix) and Sec. 4.3 (flow inflow, outflow and fix), with the sign
// reading of the domain forms: R = -d_paper for the thermal and elastic physics,
// R = +d_paper for the flow, K = dR/dU, exported d = -R(U).
//
// Penalty, convection, radiation, traction and flux go in two steps:
//   rows    one thread per (listed face, row node of the face, field) integrates its row
//           (a, i) of the face tangent and residual with the face rule and stores it in
//           the pattern's workspace;
//   gather  one wave per node of a listed face adds the rows of the faces around the node
//           (its incidence list, faces in local order) in LDS, and then each value of K and
//           d is read, added to and written once.
// The first workgroups of the rows' launch meanwhile find which faces are listed (a face listed n
// times counts n times) and their nodes; a call that names more faces than there are makes the
// distinct ones a list first, which bounds the workspace.  No atomics on K and nothing ordered by
// them, so the sums are the same on every run, and nothing waits on the host.
// All three launches are latency chains (a face reads its element's nodes, their coordinates and
// state, then a node its incidence list, counts and rows), so what helps is to have the loads of a
// step in flight together.  Conduction on 64^3 bricks, 8192 faces and 16384 faces a call, mean:
// clear 5 us, rows 14, gather 14; with the listing in a launch of its own and a node's rows read
// one after another 5, 12, 14 and 17; the eight colour launches took 132 and their marking 20.
// 15288 tetrahedra with all 2240 boundary faces: 4 + 11 + 7 us, before 4, 10, 26 and 10, where 41
// bucket launches took 1242.
//
// The flow forms on 8-node hexahedra carry the test gradient: all eight nodes get rows of
// four fields, 8 kB per face.  They go element by element, one launch per element colour:
// elements of one colour share no node, so each row is added by a single thread of the launch
// with plain stores.  The other forms on these elements go the same way when there is no memory
// for a workspace.
//
// A face whose element id or local face is out of range is skipped and its index
// recorded in the pattern's second status word.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "element.h"
#include "mf_internal.h"
#include "serendipity.h"

namespace mf {
namespace {

constexpr int kThreads = 256;

// The faces of a call.  A key is element * local faces + local face.
struct FaceLists {
    const int32_t* elem;
    const uint8_t* fid;
    int64_t n, n_el;
    const int32_t* conn;
    uint32_t* cnt;   // [keys] how often each face is listed
    int32_t* slot;   // [keys] where the rows of a listed face are
    int32_t* list;   // distinct faces (keys), or nullptr: the call's own order
    uint32_t* node_on;  // [n_nodes]
    int32_t* nodes;     // distinct nodes of the listed faces
    uint32_t* counts;   // distinct faces (with a list) and nodes
    uint32_t blocks;    // without a list: workgroups of the row kernel that list the faces
    unsigned long long* status;
};

struct BParams {
    mf_bform form;
    int64_t n_el, n_nodes, n_faces;
    const int32_t* conn;
    const double* coords;
    const int32_t* row_ptr;
    const int32_t* nbr_ptr;
    const uint8_t* rank;
    const int32_t* face_elem;
    const uint8_t* face_id;
    const void* state;   // [nf][n_nodes] or null (zero)
    const void* target;  // [nf][n_nodes] or null (the constant form->value)
    int field_major;
    void* K;
    void* d;
    unsigned long long* status;
    // colour by colour: per element, the listed local faces (bit fid), and how often each is
    const uint32_t* face_mask;  // [n_el]
    const uint32_t* face_cnt;   // [n_el][local faces]
    // rows and gather: the rows [slot of the face][row node][field][columns + 1], the residual
    // entry last
    FaceLists lists;
    double* rows;
};

// Local faces (edges in 2D) of an element type: their nodes in ascending local order, and a
// node's position among them (-1: not on the face).
template <int NEN>
struct FaceTable {
    static constexpr int NLOC = NEN == 8 || NEN == 20 ? 6 : 4;
    static constexpr int NFN = NEN == 20 ? 8 : NEN == 10 ? 6 : 4;
    int8_t node[NLOC][NFN];
    int8_t at[NLOC][NEN];
    constexpr FaceTable() : node{}, at{}
    {
        for (int f = 0; f < NLOC; ++f) {
            int n = 0;
            for (int a = 0; a < NEN; ++a) {
                bool on = false;
                if (NEN == 10) {  // face k: the vertices but k, and the edges without vertex k
                    constexpr int EI[6] = {0, 1, 2, 0, 1, 2}, EJ[6] = {1, 2, 0, 3, 3, 3};
                    on = a < 4 ? a != f : EI[a - 4] != f && EJ[a - 4] != f;
                } else {
                    const int axis = f >> 1, side = f & 1;
                    if (a < 8) {
                        on = ((a >> axis) & 1) == side;
                    } else {  // midpoint of an edge along ax, at the bits of the other two axes
                        const int ax = (a - 8) >> 2, k = (a - 8) & 3, o0 = ax == 0 ? 1 : 0;
                        on = ax != axis && (axis == o0 ? (k & 1) : (k >> 1)) == side;
                    }
                }
                at[f][a] = on ? (int8_t)n : (int8_t)-1;
                if (on) node[f][n++] = (int8_t)a;
            }
        }
    }
};
// edges of the 4- and 8-node quadrilaterals
template <int NEN>
struct EdgeTable {
    static constexpr int NLOC = 4, NFN = NEN == 8 ? 3 : 2;
    int8_t node[NLOC][NFN];
    int8_t at[NLOC][NEN];
    constexpr EdgeTable() : node{}, at{}
    {
        for (int f = 0; f < NLOC; ++f) {
            const int axis = f >> 1, side = f & 1;
            int n = 0;
            for (int a = 0; a < NEN; ++a) {
                const bool on = a < 4 ? ((a >> axis) & 1) == side : a == (axis == 0 ? 6 + side : 4 + side);
                at[f][a] = on ? (int8_t)n : (int8_t)-1;
                if (on) node[f][n++] = (int8_t)a;
            }
        }
    }
};
__constant__ constexpr FaceTable<8> kFaces8{};
__constant__ constexpr FaceTable<20> kFaces20{};
__constant__ constexpr FaceTable<10> kFaces10{};
__constant__ constexpr EdgeTable<4> kEdges4{};
__constant__ constexpr EdgeTable<8> kEdges8{};

// Per element type: its table, and the columns of a face's rows (8-node hexahedra: all nodes of
// the element, as the flux form needs them; else the nodes of the face).
template <int DIM, int NEN>
struct Faces;
template <>
struct Faces<3, 8> {
    static constexpr int NLOC = 6, NFN = 4, COLS = 8;
    static __device__ __forceinline__ int at(int f, int a) { return kFaces8.at[f][a]; }
    static __device__ __forceinline__ int node(int f, int k) { return kFaces8.node[f][k]; }
    static __device__ __forceinline__ int col(int f, int b) { return b; }
};
template <>
struct Faces<3, 20> {
    static constexpr int NLOC = 6, NFN = 8, COLS = 8;
    static __device__ __forceinline__ int at(int f, int a) { return kFaces20.at[f][a]; }
    static __device__ __forceinline__ int node(int f, int k) { return kFaces20.node[f][k]; }
    static __device__ __forceinline__ int col(int f, int b) { return kFaces20.node[f][b]; }
};
template <>
struct Faces<3, 10> {
    static constexpr int NLOC = 4, NFN = 6, COLS = 6;
    static __device__ __forceinline__ int at(int f, int a) { return kFaces10.at[f][a]; }
    static __device__ __forceinline__ int node(int f, int k) { return kFaces10.node[f][k]; }
    static __device__ __forceinline__ int col(int f, int b) { return kFaces10.node[f][b]; }
};
template <>
struct Faces<2, 4> {
    static constexpr int NLOC = 4, NFN = 2, COLS = 2;
    static __device__ __forceinline__ int at(int f, int a) { return kEdges4.at[f][a]; }
    static __device__ __forceinline__ int node(int f, int k) { return kEdges4.node[f][k]; }
    static __device__ __forceinline__ int col(int f, int b) { return kEdges4.node[f][b]; }
};
template <>
struct Faces<2, 8> {
    static constexpr int NLOC = 4, NFN = 3, COLS = 3;
    static __device__ __forceinline__ int at(int f, int a) { return kEdges8.at[f][a]; }
    static __device__ __forceinline__ int node(int f, int k) { return kEdges8.node[f][k]; }
    static __device__ __forceinline__ int col(int f, int b) { return kEdges8.node[f][b]; }
};

// Counts listed face f of the call under its key (element * NLOC + local face); the first of a key
// takes slot[key], and appends the face's nodes, each once, to the node list.  With a list, faces
// are appended to it, and their slot is the place; else it is f.  Every lane of the wave takes part
// (f >= n: no face).  Returns whether the face is in range.
template <class F>
__device__ __forceinline__ bool list_face(const FaceLists& L, int64_t f, int64_t& e, int& lf)
{
    const int lane = (int)(threadIdx.x & 63);
    // one counter update per wave: the lanes that append take consecutive places
    auto place = [&](bool take, uint32_t* counter) -> uint32_t {
        const unsigned long long group = __ballot(take);
        uint32_t base = 0;
        if (lane == 0 && group) base = atomicAdd(counter, (uint32_t)__popcll(group));
        base = (uint32_t)__shfl((int)base, 0, 64);
        return base + (uint32_t)__popcll(group & ((1ull << lane) - 1ull));
    };
    e = -1;
    lf = 0;
    if (f < L.n) {
        e = L.elem[f];
        lf = L.fid[f];
        if (e < 0 || e >= L.n_el || lf >= F::NLOC) {
            atomicMin(L.status + 1, (unsigned long long)f);
            e = -1;
        }
    }
    const int32_t key = (int32_t)(e * F::NLOC + lf);
    const bool first = e >= 0 && atomicAdd(L.cnt + key, 1u) == 0u;
    if (L.list) {
        const uint32_t at = place(first, L.counts);
        if (first) {
            L.list[at] = key;
            L.slot[key] = (int32_t)at;
        }
    } else if (first) {
        L.slot[key] = (int32_t)f;
    }
    int32_t v[F::NFN];
    bool fresh[F::NFN];
#pragma unroll
    for (int k = 0; k < F::NFN; ++k) v[k] = first ? L.conn[(int64_t)F::node(lf, k) * L.n_el + e] : 0;
#pragma unroll
    for (int k = 0; k < F::NFN; ++k) fresh[k] = first && atomicExch(L.node_on + v[k], 1u) == 0u;
#pragma unroll
    for (int k = 0; k < F::NFN; ++k) {
        const uint32_t w = place(fresh[k], L.counts + 1);
        if (fresh[k]) L.nodes[w] = v[k];
    }
    return e >= 0;
}

// One thread of the row kernels: its face's slot, element, local face, row node (position on
// the face) and field.  Without a list the first workgroups list the faces meanwhile.
struct RowItem {
    int64_t slot, e;
    int fid, k, i;
    bool live;
};
template <class F, int NF, int LANES = 1>
__device__ __forceinline__ RowItem row_item(const BParams& p)  // LANES threads have one item
{
    RowItem r{};
    const FaceLists& L = p.lists;
    if (blockIdx.x < L.blocks) {
        list_face<F>(L, (int64_t)blockIdx.x * kThreads + threadIdx.x, r.e, r.fid);
        return r;
    }
    const int64_t t = ((int64_t)(blockIdx.x - L.blocks) * kThreads + threadIdx.x) / LANES;
    const int64_t n = L.list ? (int64_t)*L.counts : L.n;
    r.live = t < n * F::NFN * NF;
    if (!r.live) return r;
    r.slot = t % n;
    const int ki = (int)(t / n);
    r.k = ki / NF;
    r.i = ki % NF;
    if (L.list) {
        const int key = L.list[r.slot];
        r.e = key / F::NLOC;
        r.fid = key % F::NLOC;
        return r;
    }
    r.e = L.elem[r.slot];
    r.fid = L.fid[r.slot];
    r.live = r.e >= 0 && r.e < L.n_el && r.fid < F::NLOC;
    return r;
}
template <class F, int NF>
__device__ __forceinline__ void store_row(const BParams& p, const RowItem& r, const double (&krow)[F::COLS], double rrow)
{
    double* out = p.rows + ((r.slot * F::NFN + r.k) * NF + r.i) * (F::COLS + 1);
#pragma unroll
    for (int b = 0; b < F::COLS; ++b) out[b] = krow[b];
    out[F::COLS] = -rrow;
}

__device__ __forceinline__ double lin1(int s, double xi) { return 0.5 * (1.0 + (s ? xi : -xi)); }

// (J^-1)[n][m] = dxi_n / dx_m by cofactors; false when det J <= 0
__device__ __forceinline__ bool inverse_jacobian(const double (&J)[3][3], double (&Ji)[3][3])
{
    const double c00 = J[1][1] * J[2][2] - J[1][2] * J[2][1];
    const double c01 = J[1][2] * J[2][0] - J[1][0] * J[2][2];
    const double c02 = J[1][0] * J[2][1] - J[1][1] * J[2][0];
    const double det = J[0][0] * c00 + J[0][1] * c01 + J[0][2] * c02;
    if (!(det > 0.0)) return false;
    const double r = 1.0 / det;
    Ji[0][0] = c00 * r;
    Ji[0][1] = (J[0][2] * J[2][1] - J[0][1] * J[2][2]) * r;
    Ji[0][2] = (J[0][1] * J[1][2] - J[0][2] * J[1][1]) * r;
    Ji[1][0] = c01 * r;
    Ji[1][1] = (J[0][0] * J[2][2] - J[0][2] * J[2][0]) * r;
    Ji[1][2] = (J[0][2] * J[1][0] - J[0][0] * J[1][2]) * r;
    Ji[2][0] = c02 * r;
    Ji[2][1] = (J[0][1] * J[2][0] - J[0][0] * J[2][1]) * r;
    Ji[2][2] = (J[0][0] * J[1][1] - J[0][1] * J[1][0]) * r;
    return true;
}

// Row (a, i) of one face (local face fid) of an 8-node hexahedron by the 2x2 Gauss rule,
// times mult, added to krow and rrow, for the forms that do not couple fields: only field i of the
// state and target and the (a, i) x (b, i) block are held.  Returns false (status set) on a
// degenerate face or element.
template <typename T>
__device__ __forceinline__ bool face_integral(const BParams& p, int64_t e, int fid, double mult, int a, int i,
                                              const double (&x)[8][3], const double (&U)[8][1],
                                              const double (&G)[8][1], double (&krow)[8][1], double& rrow)
{
    const T* tg = (const T*)p.target;
    const mf_bform_kind kind = p.form.kind;
    const double c = p.form.coef;
    const int axis = fid >> 1, side = fid & 1;
    const int u = (axis + 1) % 3, v = (axis + 2) % 3;
    for (int q = 0; q < 4; ++q) {
        double xi[3];
        xi[axis] = side ? 1.0 : -1.0;
        xi[u] = (q & 1) ? kGaussPt : -kGaussPt;
        xi[v] = (q >> 1) ? kGaussPt : -kGaussPt;
        double N[8], dN[8][3];
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const int bx = b & 1, by = (b >> 1) & 1, bz = b >> 2;
            const double Fx = lin1(bx, xi[0]), Fy = lin1(by, xi[1]), Fz = lin1(bz, xi[2]);
            N[b] = Fx * Fy * Fz;
            dN[b][0] = (bx ? 0.5 : -0.5) * Fy * Fz;
            dN[b][1] = (by ? 0.5 : -0.5) * Fx * Fz;
            dN[b][2] = (bz ? 0.5 : -0.5) * Fx * Fy;
        }
        double J[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};  // J[m][n] = dx_m / dxi_n
#pragma unroll
        for (int b = 0; b < 8; ++b)
#pragma unroll
            for (int m = 0; m < 3; ++m)
#pragma unroll
                for (int n = 0; n < 3; ++n) J[m][n] = fma(x[b][m], dN[b][n], J[m][n]);
        const double tu[3] = {J[0][u], J[1][u], J[2][u]}, tv[3] = {J[0][v], J[1][v], J[2][v]};
        const double sg = side ? 1.0 : -1.0;
        double nr[3] = {sg * (tu[1] * tv[2] - tu[2] * tv[1]), sg * (tu[2] * tv[0] - tu[0] * tv[2]),
                        sg * (tu[0] * tv[1] - tu[1] * tv[0])};
        const double dS = sqrt(nr[0] * nr[0] + nr[1] * nr[1] + nr[2] * nr[2]);
        if (!(dS > 0.0)) {
            atomicMin(p.status, (unsigned long long)e);
            return false;
        }
        const double nv[3] = {nr[0] / dS, nr[1] / dS, nr[2] / dS};
        const double w = mult * dS;  // unit Gauss weights on [-1, 1]^2, times the face's count
        const double Na = N[a];
        double uq = 0.0, gq = 0.0;
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            uq = fma(N[b], U[b][0], uq);
            gq = fma(N[b], G[b][0], gq);
        }
        if (kind == MF_BFORM_PENALTY || kind == MF_BFORM_CONVECTION) {
            // R = int c N_a (u_i - g_i)
#pragma unroll
            for (int b = 0; b < 8; ++b) krow[b][0] += c * w * Na * N[b];
            rrow += c * w * Na * (uq - gq);
        } else if (kind == MF_BFORM_RADIATION) {
            // R = int c N_a (T^4 - T_env^4), c = e_m sigma
            const double T1 = uq, Te = gq;
#pragma unroll
            for (int b = 0; b < 8; ++b) krow[b][0] += c * w * Na * 4.0 * T1 * T1 * T1 * N[b];
            rrow += c * w * Na * (T1 * T1 * T1 * T1 - Te * Te * Te * Te);
        } else if (kind == MF_BFORM_TRACTION) {
            // R = -int N_a t_i, t = sigma^l n or the interpolated nodal traction
            const double* S = p.form.value;
            const double ti = tg ? gq : S[3 * i] * nv[0] + S[3 * i + 1] * nv[1] + S[3 * i + 2] * nv[2];
            rrow -= w * Na * ti;
        } else {  // MF_BFORM_FLUX: R = -int c N_a n . grad T
            double Ji[3][3];
            if (!inverse_jacobian(J, Ji)) {
                atomicMin(p.status, (unsigned long long)e);
                return false;
            }
            double ngT = 0.0;
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                double ng = 0.0;  // n . grad N_b,  grad N_b = J^-T grad_xi N_b
#pragma unroll
                for (int m = 0; m < 3; ++m)
                    ng += nv[m] * (Ji[0][m] * dN[b][0] + Ji[1][m] * dN[b][1] + Ji[2][m] * dN[b][2]);
                krow[b][0] -= c * w * Na * ng;
                ngT = fma(ng, U[b][0], ngT);
            }
            rrow -= c * w * Na * ngT;
        }
    }
    return true;
}

// Row (a, FI) of one face for the flow forms (value: u^w [0..3), rho [3], mu [4]; coef = tau^b), which
// carry the test gradient: any node of the element, all four columns.  Field and kind are known at
// compile time, so that every index of a register array is static.  Basis and gradients of the nodes are
// formed twice, before and after the geometry, as held between they would not fit the registers with
// the element's data and the row.  Bound by the instructions of few waves, whose lanes have different
// faces: the six sides of 32^3 bricks 337 us (inflow) and 359 (outflow), 410 and 405 with the kind
// looked up and the basis held; 1000 single faces 588 and 772, 822 and 900 so.  Returns false (status set) on a
// degenerate face or element.
template <int FI, int KIND, typename T>
__device__ __forceinline__ bool flow_face(const BParams& p, int64_t e, int fid, double mult, int a,
                                          const double (&x)[8][3], const double (&U)[8][4], const double (&G)[8][4],
                                          double (&krow)[8][4], double& rrow)
{
    constexpr bool kWall = KIND != MF_BFORM_NS_OUTFLOW;
    const double rho = p.form.value[3], mu = p.form.value[4], tau = p.form.coef;
    const int axis = fid >> 1, side = fid & 1;
    const int u = (axis + 1) % 3, v = (axis + 2) % 3;
#pragma unroll 1
    for (int q = 0; q < 4; ++q) {
        double xi[3];
        xi[axis] = side ? 1.0 : -1.0;
        xi[u] = (q & 1) ? kGaussPt : -kGaussPt;
        xi[v] = (q >> 1) ? kGaussPt : -kGaussPt;
        // N_b and its reference gradient
        auto basis = [&](int b, double (&dN)[3]) {
            const int bx = b & 1, by = (b >> 1) & 1, bz = b >> 2;
            const double Fx = lin1(bx, xi[0]), Fy = lin1(by, xi[1]), Fz = lin1(bz, xi[2]);
            dN[0] = (bx ? 0.5 : -0.5) * (Fy * Fz);
            dN[1] = (by ? 0.5 : -0.5) * (Fx * Fz);
            dN[2] = (bz ? 0.5 : -0.5) * (Fx * Fy);
            return Fx * Fy * Fz;
        };
        double J[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};  // J[m][n] = dx_m / dxi_n
        double uq[4] = {0, 0, 0, 0}, uw[3] = {0, 0, 0};
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            double dN[3];
            const double N = basis(b, dN);
#pragma unroll
            for (int m = 0; m < 3; ++m)
#pragma unroll
                for (int n = 0; n < 3; ++n) J[m][n] = fma(x[b][m], dN[n], J[m][n]);
#pragma unroll
            for (int j = 0; j < 4; ++j) uq[j] = fma(N, U[b][j], uq[j]);
            if constexpr (KIND == MF_BFORM_NS_INFLOW)
#pragma unroll
                for (int m = 0; m < 3; ++m) uw[m] = fma(N, G[b][m], uw[m]);
        }
        const double tu[3] = {J[0][u], J[1][u], J[2][u]}, tv[3] = {J[0][v], J[1][v], J[2][v]};
        const double sg = side ? 1.0 : -1.0;
        const double nr[3] = {sg * (tu[1] * tv[2] - tu[2] * tv[1]), sg * (tu[2] * tv[0] - tu[0] * tv[2]),
                              sg * (tu[0] * tv[1] - tu[1] * tv[0])};
        const double dS = sqrt(nr[0] * nr[0] + nr[1] * nr[1] + nr[2] * nr[2]);
        double Ji[3][3];
        if (!(dS > 0.0) || !inverse_jacobian(J, Ji)) {
            atomicMin(p.status, (unsigned long long)e);
            return false;
        }
        const double nv[3] = {nr[0] / dS, nr[1] / dS, nr[2] / dS};
        double g[3];  // n . grad N_b = g . dN_b
#pragma unroll
        for (int n = 0; n < 3; ++n) g[n] = nv[0] * Ji[n][0] + nv[1] * Ji[n][1] + nv[2] * Ji[n][2];
        asm volatile("" : "+v"(xi[0]), "+v"(xi[1]), "+v"(xi[2]));  // (formed again from here on)
        double da[3];
        const double Na = basis(a, da), gna = g[0] * da[0] + g[1] * da[1] + g[2] * da[2];
        const double w = mult * dS, wN = w * Na;  // unit Gauss weights on [-1, 1]^2, times the face's count
        if constexpr (FI == 3) {
            rrow += wN * ((uw[0] - uq[0]) * nv[0] + (uw[1] - uq[1]) * nv[1] + (uw[2] - uq[2]) * nv[2]);
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                double dN[3];
                const double N = basis(b, dN);
#pragma unroll
                for (int k = 0; k < 3; ++k) krow[b][k] = fma(-wN * nv[k], N, krow[b][k]);
            }
        } else {
            const double un = uq[0] * nv[0] + uq[1] * nv[1] + uq[2] * nv[2];
            const double wall = w * (tau * rho * Na - mu * gna);
            double gu = 0.0, t[3];  // base: p n_i - mu u_i,j n_j
#pragma unroll
            for (int k = 0; k < 3; ++k) t[k] = rho * wN * ((k == FI ? un : 0.0) + uq[FI] * nv[k]);
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                double dN[3];
                const double N = basis(b, dN), gn = g[0] * dN[0] + g[1] * dN[1] + g[2] * dN[2];
                gu = fma(gn, U[b][FI], gu);
                krow[b][3] = fma(wN * nv[FI], N, krow[b][3]);
                krow[b][FI] = fma(-mu * wN, gn, krow[b][FI]);
                if constexpr (kWall) {
                    krow[b][FI] = fma(wall, N, krow[b][FI]);
                } else {
#pragma unroll
                    for (int k = 0; k < 3; ++k) krow[b][k] = fma(N, t[k], krow[b][k]);
                }
            }
            rrow += wN * (uq[3] * nv[FI] - mu * gu);
            if constexpr (kWall) {
                const double uwn = uw[0] * nv[0] + uw[1] * nv[1] + uw[2] * nv[2];
                rrow += w * (rho * Na * uw[FI] * uwn + mu * gna * (uw[FI] - uq[FI]) + tau * rho * Na * (uq[FI] - uw[FI]));
            } else {
                rrow += rho * wN * uq[FI] * un;
            }
        }
    }
    return true;
}

// Coordinates of the element's nodes, and the state and target there: all four fields for the
// flow forms, else field i alone.
template <int NF, typename T>
__device__ __forceinline__ void load_element(const BParams& p, int64_t e, int i, int32_t (&node)[8], double (&x)[8][3],
                                             double (&U)[8][NF == 4 ? 4 : 1], double (&G)[8][NF == 4 ? 4 : 1])
{
    constexpr int NL = NF == 4 ? 4 : 1;
    const T* st = (const T*)p.state;
    const T* tg = (const T*)p.target;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        node[b] = p.conn[(int64_t)b * p.n_el + e];
#pragma unroll
        for (int m = 0; m < 3; ++m) x[b][m] = p.coords[(int64_t)m * p.n_nodes + node[b]];
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const int j = NL == 1 ? i : l;
            U[b][l] = st ? (double)st[(int64_t)j * p.n_nodes + node[b]] : 0.0;
            G[b][l] = tg ? (double)tg[(int64_t)j * p.n_nodes + node[b]] : p.form.value[j];
        }
    }
}

// Rows of the listed faces of 8-node hexahedra (penalty, convection, radiation, traction, flux).
template <int NF, typename T>
__global__ void __launch_bounds__(kThreads) k_face_rows8(BParams p)
{
    using F = Faces<3, 8>;
    const RowItem r = row_item<F, NF>(p);
    if (!r.live) return;
    int32_t node[8];
    double x[8][3], U[8][1], G[8][1], krow[8][1], out[8], rrow = 0.0;
    load_element<NF, T>(p, r.e, r.i, node, x, U, G);
#pragma unroll
    for (int b = 0; b < 8; ++b) krow[b][0] = 0.0;
    const bool ok = face_integral<T>(p, r.e, r.fid, 1.0, F::node(r.fid, r.k), r.i, x, U, G, krow, rrow);
#pragma unroll
    for (int b = 0; b < 8; ++b) out[b] = ok ? krow[b][0] : 0.0;
    store_row<F, NF>(p, r, out, ok ? rrow : 0.0);
}

// Row (a, i) of element e over the listed faces of e (local faces in `fmask`, each
// counted cnt[6 e + fid] times), for 8-node hexahedra.  The caller runs one element colour
// per launch: no other thread of the launch touches row a, so the row is added with plain
// stores.
template <int NF, int FI, int KIND, typename T>
__device__ __forceinline__ void boundary_row(const BParams& p, int64_t e, uint32_t fmask, int a, int fi)
{
    const int i = FI >= 0 ? FI : fi;
    constexpr int NL = NF == 4 ? 4 : 1;
    int32_t node[8];
    double x[8][3];
    double U[8][NL], G[8][NL];
    load_element<NF, T>(p, e, i, node, x, U, G);
    constexpr int KC = NL;  // columns held per node: all fields, or field i alone (slot 0)
    double krow[8][KC];
#pragma unroll
    for (int b = 0; b < 8; ++b)
#pragma unroll
        for (int j = 0; j < KC; ++j) krow[b][j] = 0.0;
    double rrow = 0.0;
    for (int fid = 0; fid < 6; ++fid) {
        if (!((fmask >> fid) & 1)) continue;
        // the row nodes of a face are its four nodes (every node of the element for the
        // flow forms, whose terms carry the test gradient)
        if (NF != 4 && ((a >> (fid >> 1)) & 1) != (fid & 1)) continue;
        const double mult = (double)p.face_cnt[6 * e + fid];
        if constexpr (NF == 4) {
            if (!flow_face<FI, KIND, T>(p, e, fid, mult, a, x, U, G, krow, rrow)) return;
        } else {
            if (!face_integral<T>(p, e, fid, mult, a, fi, x, U, G, krow, rrow)) return;
        }
    }

    const int64_t va = node[a];
    const int64_t row = p.field_major ? (int64_t)i * p.n_nodes + va : (int64_t)NF * va + i;
    const int64_t rs = p.row_ptr[row];
    const int64_t deg = p.nbr_ptr[va + 1] - p.nbr_ptr[va];
    T* K = (T*)p.K;
    T* d = (T*)p.d;
    // nonzero entries only; every old value is loaded before the first store, so the
    // thread's read-modify-writes overlap instead of running one after another
    int rk[8];
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        bool any = false;
#pragma unroll
        for (int l = 0; l < KC; ++l) any = any || krow[b][l] != 0.0;
        rk[b] = any ? (int)p.rank[(int64_t)(a * 8 + b) * p.n_el + e] : 0;
    }
    auto pos_of = [&](int b, int l) -> int64_t {
        const int j = KC == 1 ? i : l;
        return p.field_major ? rs + j * deg + rk[b] : rs + (int64_t)rk[b] * NF + j;
    };
    T old[8][KC];
#pragma unroll
    for (int b = 0; b < 8; ++b)
#pragma unroll
        for (int l = 0; l < KC; ++l) old[b][l] = krow[b][l] != 0.0 ? K[pos_of(b, l)] : T(0);
    const T dold = rrow != 0.0 ? d[row] : T(0);
#pragma unroll
    for (int b = 0; b < 8; ++b)
#pragma unroll
        for (int l = 0; l < KC; ++l)
            if (krow[b][l] != 0.0) K[pos_of(b, l)] = old[b][l] + (T)krow[b][l];
    if (rrow != 0.0) d[row] = dold + (T)(-rrow);
}

// Items (element with listed faces of the colour, element node a, field i), strided over
// the grid; the colour's element list and its length come from k_face_mark.
template <int NF, int KIND, typename T>
__global__ void __launch_bounds__(kThreads) k_boundary(BParams p, const int32_t* __restrict__ elems,
                                                       const uint32_t* __restrict__ n_el_c)
{
    const int64_t nc = *n_el_c;
    const int64_t n = nc * 8 * NF;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t e = elems[t % nc];
        const uint32_t fmask = p.face_mask[e];
        const int ki = (int)(t / nc);
        const int a = ki / NF, i = ki % NF;
        if constexpr (NF == 4) {
            switch (i) {
                case 0: boundary_row<NF, 0, KIND, T>(p, e, fmask, a, i); break;
                case 1: boundary_row<NF, 1, KIND, T>(p, e, fmask, a, i); break;
                case 2: boundary_row<NF, 2, KIND, T>(p, e, fmask, a, i); break;
                default:  // (the outflow form has no continuity rows)
                    if constexpr (KIND != MF_BFORM_NS_OUTFLOW) boundary_row<NF, 3, KIND, T>(p, e, fmask, a, i);
            }
        } else {
            boundary_row<NF, -1, KIND, T>(p, e, fmask, a, i);
        }
    }
}

// Faces of 20-node hexahedra: one thread per (face f, face node k, field i), with the
// eight nodes of the face (the other twelve basis functions vanish on it, with their
// tangential derivatives) and the 3x3 Gauss rule of the face; penalty, convection,
// radiation and traction as above.
template <int NF, typename T>
__global__ void __launch_bounds__(kThreads) k_face_rows20(BParams p)
{
    using F = Faces<3, 20>;
    const RowItem r = row_item<F, NF>(p);
    if (!r.live) return;
    const int64_t e = r.e;
    const int i = r.i;
    const int kf = r.k, axis = r.fid >> 1, side = r.fid & 1;
    const int u = (axis + 1) % 3, v = (axis + 2) % 3;
    int loc[8];  // local ids of the face nodes, ascending
#pragma unroll
    for (int b = 0; b < 8; ++b) loc[b] = F::node(r.fid, b);
    double x[8][3], U[8], G[8];  // coordinates, and field i of the state and target
    int32_t node[8];
    const T* st = (const T*)p.state;
    const T* tg = (const T*)p.target;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        node[b] = p.conn[(int64_t)loc[b] * p.n_el + e];
#pragma unroll
        for (int m = 0; m < 3; ++m) x[b][m] = p.coords[(int64_t)m * p.n_nodes + node[b]];
        U[b] = st ? (double)st[(int64_t)i * p.n_nodes + node[b]] : 0.0;
        G[b] = tg ? (double)tg[(int64_t)i * p.n_nodes + node[b]] : p.form.value[i];
    }
    const mf_bform_kind kind = p.form.kind;
    const double c = p.form.coef;
    double krow[8];
#pragma unroll
    for (int b = 0; b < 8; ++b) krow[b] = 0.0;
    double rrow = 0.0;
    const double gp = 0.7745966692414834;  // sqrt(3/5)
    for (int q = 0; q < 9; ++q) {
        const int qu = q % 3, qv = q / 3;
        double xi[3];
        xi[axis] = side ? 1.0 : -1.0;
        xi[u] = (qu - 1) * gp;
        xi[v] = (qv - 1) * gp;
        const double wq = (qu == 1 ? 8.0 : 5.0) * (qv == 1 ? 8.0 : 5.0) / 81.0;
        double N[8], tu[3] = {0, 0, 0}, tv[3] = {0, 0, 0};
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            double dN[3];
            shape20(loc[b], xi, N[b], dN);
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                tu[m] = fma(x[b][m], dN[u], tu[m]);
                tv[m] = fma(x[b][m], dN[v], tv[m]);
            }
        }
        const double sg = side ? 1.0 : -1.0;
        const double nr[3] = {sg * (tu[1] * tv[2] - tu[2] * tv[1]), sg * (tu[2] * tv[0] - tu[0] * tv[2]),
                              sg * (tu[0] * tv[1] - tu[1] * tv[0])};
        const double dS = sqrt(nr[0] * nr[0] + nr[1] * nr[1] + nr[2] * nr[2]);
        if (!(dS > 0.0)) {
            atomicMin(p.status, (unsigned long long)e);
            double none[F::COLS] = {};
            store_row<F, NF>(p, r, none, 0.0);
            return;
        }
        const double w = wq * dS;
        const double Na = N[kf];
        double uq = 0.0, gq = 0.0;
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            uq = fma(N[b], U[b], uq);
            gq = fma(N[b], G[b], gq);
        }
        if (kind == MF_BFORM_PENALTY || kind == MF_BFORM_CONVECTION) {
#pragma unroll
            for (int b = 0; b < 8; ++b) krow[b] += c * w * Na * N[b];
            rrow += c * w * Na * (uq - gq);
        } else if (kind == MF_BFORM_RADIATION) {
#pragma unroll
            for (int b = 0; b < 8; ++b) krow[b] += c * w * Na * 4.0 * uq * uq * uq * N[b];
            rrow += c * w * Na * (uq * uq * uq * uq - gq * gq * gq * gq);
        } else {  // MF_BFORM_TRACTION
            const double* S = p.form.value;
            const double ti = tg ? gq : (S[3 * i] * nr[0] + S[3 * i + 1] * nr[1] + S[3 * i + 2] * nr[2]) / dS;
            rrow -= w * Na * ti;
        }
    }
    store_row<F, NF>(p, r, krow, rrow);
}

constexpr int kTetLanes = 4;
// Faces of 10-node tetrahedra: four threads per (face f, face node m, field i), one for each first
// coordinate of the rule (2240 faces are 210 waves with one thread each: 26 us
// against 11).  Face k is
// the face opposite vertex k: its three vertices and the three edge midpoints among them.
// The face is the reference triangle p0 + s (p1 - p0) + t (p2 - p0) over its vertices,
// integrated with the collapsed 4 x 4 Gauss rule of the triangle; the normal points away
// from vertex k.  Penalty, convection, radiation and traction as above.
template <int NF, typename T>
__global__ void __launch_bounds__(kThreads) k_face_rows10(BParams p)
{
    using F = Faces<3, 10>;
    const RowItem r = row_item<F, NF, kTetLanes>(p);
    if (!r.live) return;
    const int64_t e = r.e;
    const int i = r.i, sub = threadIdx.x % kTetLanes;
    const int mf = r.k, k = r.fid;
    // face nodes: the vertices other than k, then the edges among them
    int loc[6];
#pragma unroll
    for (int b = 0; b < 6; ++b) loc[b] = F::node(k, b);
    double pv[3][3];  // reference coordinates of the face vertices
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int m = 0; m < 3; ++m) pv[c][m] = loc[c] == m + 1 ? 1.0 : 0.0;
    double x[6][3], U[6], G[6], xk[3];
    int32_t node[6];
    const T* st = (const T*)p.state;
    const T* tg = (const T*)p.target;
#pragma unroll
    for (int b = 0; b < 6; ++b) {
        node[b] = p.conn[(int64_t)loc[b] * p.n_el + e];
#pragma unroll
        for (int m = 0; m < 3; ++m) x[b][m] = p.coords[(int64_t)m * p.n_nodes + node[b]];
        U[b] = st ? (double)st[(int64_t)i * p.n_nodes + node[b]] : 0.0;
        G[b] = tg ? (double)tg[(int64_t)i * p.n_nodes + node[b]] : p.form.value[i];
    }
    {
        const int32_t vk = p.conn[(int64_t)k * p.n_el + e];
#pragma unroll
        for (int m = 0; m < 3; ++m) xk[m] = p.coords[(int64_t)m * p.n_nodes + vk];
    }
    const mf_bform_kind kind = p.form.kind;
    const double c = p.form.coef;
    double krow[6];
#pragma unroll
    for (int b = 0; b < 6; ++b) krow[b] = 0.0;
    double rrow = 0.0;
    const double g4[4] = {0.5 * (1.0 - 0.8611363115940526), 0.5 * (1.0 - 0.3399810435848563),
                          0.5 * (1.0 + 0.3399810435848563), 0.5 * (1.0 + 0.8611363115940526)};
    const double w4[4] = {0.5 * 0.3478548451374538, 0.5 * 0.6521451548625461, 0.5 * 0.6521451548625461,
                          0.5 * 0.3478548451374538};
    const double s_ = g4[sub], ws = w4[sub] * (1.0 - s_);
    bool ok = true;
#pragma unroll 1
    for (int q = 0; q < 4; ++q) {
        const double t_ = g4[q] * (1.0 - s_);
        const double wq = ws * w4[q];
        double xi[3], e1[3], e2[3];
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            e1[m] = pv[1][m] - pv[0][m];
            e2[m] = pv[2][m] - pv[0][m];
            xi[m] = pv[0][m] + s_ * e1[m] + t_ * e2[m];
        }
        double N[6], ts[3] = {0, 0, 0}, tt[3] = {0, 0, 0}, xq[3] = {0, 0, 0};
#pragma unroll
        for (int b = 0; b < 6; ++b) {
            double dN[3];
            shape10(loc[b], xi, N[b], dN);
            const double ds = dN[0] * e1[0] + dN[1] * e1[1] + dN[2] * e1[2];
            const double dt = dN[0] * e2[0] + dN[1] * e2[1] + dN[2] * e2[2];
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                ts[m] = fma(x[b][m], ds, ts[m]);
                tt[m] = fma(x[b][m], dt, tt[m]);
                xq[m] = fma(x[b][m], N[b], xq[m]);
            }
        }
        double nr[3] = {ts[1] * tt[2] - ts[2] * tt[1], ts[2] * tt[0] - ts[0] * tt[2], ts[0] * tt[1] - ts[1] * tt[0]};
        if (nr[0] * (xq[0] - xk[0]) + nr[1] * (xq[1] - xk[1]) + nr[2] * (xq[2] - xk[2]) < 0.0) {
#pragma unroll
            for (int m = 0; m < 3; ++m) nr[m] = -nr[m];
        }
        const double dS = sqrt(nr[0] * nr[0] + nr[1] * nr[1] + nr[2] * nr[2]);
        ok &= dS > 0.0;
        const double w = wq * dS;
        const double Na = N[mf];
        double uq = 0.0, gq = 0.0;
#pragma unroll
        for (int b = 0; b < 6; ++b) {
            uq = fma(N[b], U[b], uq);
            gq = fma(N[b], G[b], gq);
        }
        if (kind == MF_BFORM_PENALTY || kind == MF_BFORM_CONVECTION) {
#pragma unroll
            for (int b = 0; b < 6; ++b) krow[b] += c * w * Na * N[b];
            rrow += c * w * Na * (uq - gq);
        } else if (kind == MF_BFORM_RADIATION) {
#pragma unroll
            for (int b = 0; b < 6; ++b) krow[b] += c * w * Na * 4.0 * uq * uq * uq * N[b];
            rrow += c * w * Na * (uq * uq * uq * uq - gq * gq * gq * gq);
        } else {  // MF_BFORM_TRACTION
            const double* S = p.form.value;
            const double ti = tg ? gq : (S[3 * i] * nr[0] + S[3 * i + 1] * nr[1] + S[3 * i + 2] * nr[2]) / dS;
            rrow -= w * Na * ti;
        }
    }
#pragma unroll
    for (int off = 1; off < kTetLanes; off *= 2) {
#pragma unroll
        for (int b = 0; b < 6; ++b) krow[b] += __shfl_xor(krow[b], off, kTetLanes);
        rrow += __shfl_xor(rrow, off, kTetLanes);
        ok &= __shfl_xor((int)ok, off, kTetLanes) != 0;
    }
    if (sub != 0) return;
    if (!ok) {  // such a face adds nothing
        atomicMin(p.status, (unsigned long long)e);
        rrow = 0.0;
#pragma unroll
        for (int b = 0; b < 6; ++b) krow[b] = 0.0;
    }
    store_row<F, NF>(p, r, krow, rrow);
}

// Edges of quadrilaterals (NEN = 4 or 8): one thread per (edge, edge node, field).  Edge
// eid = 2 * axis + side is xi_axis = -1 or +1, with its two corners and, for the 8-node
// element, its midpoint; Gauss rule with 2 or 3 points along the edge; ds = |dx/dt| and n
// the unit normal pointing away from the element's centre.  Penalty, convection,
// radiation and traction (sigma^l: the leading 2x2 block of value, or a nodal target).
template <int NEN, int NF, typename T>
__global__ void __launch_bounds__(kThreads) k_edge_rows(BParams p)
{
    using F = Faces<2, NEN>;
    const RowItem r = row_item<F, NF>(p);
    if (!r.live) return;
    const int64_t e = r.e;
    const int i = r.i;
    constexpr int NE = F::NFN;  // nodes per edge, and Gauss points
    const int me = r.k, axis = r.fid >> 1, side = r.fid & 1, other = 1 - axis;
    int loc[NE];
#pragma unroll
    for (int b = 0; b < NE; ++b) loc[b] = F::node(r.fid, b);
    double x[NE][2], U[NE], G[NE], centre[2] = {0.0, 0.0};
    int32_t node[NE];
    const T* st = (const T*)p.state;
    const T* tg = (const T*)p.target;
#pragma unroll
    for (int b = 0; b < NE; ++b) {
        node[b] = p.conn[(int64_t)loc[b] * p.n_el + e];
#pragma unroll
        for (int m = 0; m < 2; ++m) x[b][m] = p.coords[(int64_t)m * p.n_nodes + node[b]];
        U[b] = st ? (double)st[(int64_t)i * p.n_nodes + node[b]] : 0.0;
        G[b] = tg ? (double)tg[(int64_t)i * p.n_nodes + node[b]] : p.form.value[i];
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const int32_t v = p.conn[(int64_t)a * p.n_el + e];
#pragma unroll
        for (int m = 0; m < 2; ++m) centre[m] += 0.25 * p.coords[(int64_t)m * p.n_nodes + v];
    }
    const mf_bform_kind kind = p.form.kind;
    const double c = p.form.coef;
    double krow[NE];
#pragma unroll
    for (int b = 0; b < NE; ++b) krow[b] = 0.0;
    double rrow = 0.0;
    const double g3 = 0.7745966692414834;  // sqrt(3/5)
#pragma unroll
    for (int q = 0; q < NE; ++q) {
        const double tq = NE == 3 ? (q - 1) * g3 : (q ? kGaussPt : -kGaussPt);
        const double wq = NE == 3 ? (q == 1 ? 8.0 / 9.0 : 5.0 / 9.0) : 1.0;
        double xi[2];
        xi[axis] = side ? 1.0 : -1.0;
        xi[other] = tq;
        double N[NE], tang[2] = {0.0, 0.0}, xq[2] = {0.0, 0.0};
#pragma unroll
        for (int b = 0; b < NE; ++b) {
            double dN[2];
            if constexpr (NEN == 8) {
                shape8(loc[b], xi, N[b], dN);
            } else {
                const int bx = loc[b] & 1, by = loc[b] >> 1;
                const double fx = 0.5 * (1.0 + (bx ? xi[0] : -xi[0])), fy = 0.5 * (1.0 + (by ? xi[1] : -xi[1]));
                N[b] = fx * fy;
                dN[0] = (bx ? 0.5 : -0.5) * fy;
                dN[1] = (by ? 0.5 : -0.5) * fx;
            }
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                tang[m] = fma(x[b][m], dN[other], tang[m]);
                xq[m] = fma(x[b][m], N[b], xq[m]);
            }
        }
        const double ds = sqrt(tang[0] * tang[0] + tang[1] * tang[1]);
        if (!(ds > 0.0)) {
            atomicMin(p.status, (unsigned long long)e);
            double none[F::COLS] = {};
            store_row<F, NF>(p, r, none, 0.0);
            return;
        }
        double nv[2] = {tang[1] / ds, -tang[0] / ds};
        if (nv[0] * (xq[0] - centre[0]) + nv[1] * (xq[1] - centre[1]) < 0.0) {
            nv[0] = -nv[0];
            nv[1] = -nv[1];
        }
        const double w = wq * ds;
        const double Na = N[me];
        double uq = 0.0, gq = 0.0;
#pragma unroll
        for (int b = 0; b < NE; ++b) {
            uq = fma(N[b], U[b], uq);
            gq = fma(N[b], G[b], gq);
        }
        if (kind == MF_BFORM_PENALTY || kind == MF_BFORM_CONVECTION) {
#pragma unroll
            for (int b = 0; b < NE; ++b) krow[b] += c * w * Na * N[b];
            rrow += c * w * Na * (uq - gq);
        } else if (kind == MF_BFORM_RADIATION) {
#pragma unroll
            for (int b = 0; b < NE; ++b) krow[b] += c * w * Na * 4.0 * uq * uq * uq * N[b];
            rrow += c * w * Na * (uq * uq * uq * uq - gq * gq * gq * gq);
        } else {  // MF_BFORM_TRACTION
            const double* S = p.form.value;
            const double ti = tg ? gq : S[3 * i] * nv[0] + S[3 * i + 1] * nv[1];
            rrow -= w * Na * ti;
        }
    }
    store_row<F, NF>(p, r, krow, rrow);
}

__global__ void k_face_zero(uint32_t* __restrict__ w, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) w[i] = 0u;
}

// per element: bit fid of mask[e] for each listed local face, cnt[6 e + fid] its count;
// an element's first face appends it to the list of its colour (list of colour c at
// clist[cptr[c] ..], length ccount[c]; the order within a list does not matter, as
// elements of one colour write disjoint rows).  A face out of range is skipped and
// reported through the second status word.
__global__ void k_face_mark(const int32_t* __restrict__ fe, const uint8_t* __restrict__ fid, int64_t n,
                            int64_t n_el, const int32_t* __restrict__ ecol, const int64_t* __restrict__ cptr,
                            uint32_t* __restrict__ mask, uint32_t* __restrict__ cnt, int32_t* __restrict__ clist,
                            uint32_t* __restrict__ ccount, unsigned long long* __restrict__ status)
{
    const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t e = -1;
    int c = -1;  // colour of an element this face touches first
    if (f < n) {
        e = fe[f];
        const int lf = fid[f];
        if (e < 0 || e >= n_el || lf > 5) {
            atomicMin(status + 1, (unsigned long long)f);
        } else {
            atomicAdd(cnt + 6 * e + lf, 1u);
            if (atomicOr(mask + e, 1u << lf) == 0u) c = ecol[e];
        }
    }
    // append to the colour lists with one counter update per (wave, colour): the lanes
    // of one colour take consecutive slots after the leader's atomic add
    const int lane = (int)(threadIdx.x & 63);
    unsigned long long pending = __ballot(c >= 0);
    while (pending) {
        const int leader = __ffsll((long long)pending) - 1;
        const int cc = __shfl(c, leader, 64);
        const unsigned long long group = __ballot(c == cc);
        uint32_t base = 0;
        if (lane == leader) base = atomicAdd(ccount + cc, (uint32_t)__popcll(group));
        base = (uint32_t)__shfl((int)base, leader, 64);
        if (c == cc) {
            const uint32_t below = (uint32_t)__popcll(group & ((1ull << lane) - 1ull));
            clist[cptr[cc] + base + below] = (int32_t)e;
        }
        pending &= ~group;
    }
}

// (More faces in the call than there are: the distinct ones, as a list.)
template <class F>
__global__ void __launch_bounds__(kThreads) k_face_list(FaceLists L)
{
    int64_t e;
    int lf;
    list_face<F>(L, (int64_t)blockIdx.x * kThreads + threadIdx.x, e, lf);
}

constexpr int kMaxAt = 3;  // listed faces of an element around one of its nodes

struct FaceGather {
    const int32_t* adj_ptr;
    const int32_t* adj;
    const int32_t* nbr_ptr;
    const uint8_t* rank_t;
    const uint32_t* cnt;
    const int32_t* slot;
    const int32_t* nodes;
    const uint32_t* n_nodes_on;
    const double* rows;
    int64_t n_nodes, n_pairs;
    int field_major, buf_len;
    void* K;
    void* d;
};

// One wave per listed node (strided over the grid): the rows of the faces around it, several at
// once, then its values of K and d.  The (i, i) blocks only: these forms do not couple fields.
template <int DIM, int NEN, int NF, typename T>
__global__ void __launch_bounds__(kThreads) k_face_gather(FaceGather p)
{
    using F = Faces<DIM, NEN>;
    constexpr int ROW = F::COLS + 1, RL = NF * ROW, G = 64 / RL, UN = 2;
    extern __shared__ __align__(16) double sh[];
    const int lane = threadIdx.x & 63, waves = blockDim.x / 64, wave = threadIdx.x / 64;
    int4* list = (int4*)(sh + wave * p.buf_len);  // rows of 64 entries: place, entry, count, local face
    double* buf = (double*)(list + 64 * kMaxAt);  // [i][r], then the residual entries
    double* dbuf = sh + (wave + 1) * p.buf_len - 4;
    const int n = (int)*p.n_nodes_on;
    const int grp = lane / RL, l = lane - grp * RL, li = l / ROW, lb = l - li * ROW;
    for (int w = blockIdx.x * waves + wave; w < n; w += gridDim.x * waves) {
        const int64_t v = p.nodes[w];
        const int k0 = p.adj_ptr[v], k1 = p.adj_ptr[v + 1];
        const int64_t P = p.nbr_ptr[v];
        const int deg = p.nbr_ptr[v + 1] - (int)P;
        for (int t = lane; t < NF * deg; t += 64) buf[t] = 0.0;
        if (lane < NF) dbuf[lane] = 0.0;
        for (int kb = k0; kb < k1; kb += 64) {
            const bool in = kb + lane < k1;
            const int code = in ? p.adj[kb + lane] : 0;
            const int e = code / NEN, a = code - e * NEN;
            uint32_t cnt[F::NLOC];
            int slot[F::NLOC];
#pragma unroll
            for (int f = 0; f < F::NLOC; ++f) {
                cnt[f] = p.cnt[(int64_t)e * F::NLOC + f];
                slot[f] = p.slot[(int64_t)e * F::NLOC + f];  // (anything where cnt is 0)
            }
            // the rows, by local face and entry: the order of their sums
            int total = 0;
#pragma unroll
            for (int f = 0; f < F::NLOC; ++f) {
                const int at = in ? F::at(f, a) : -1;
                const bool on = at >= 0 && cnt[f] != 0u;
                const unsigned long long group = __ballot(on);
                if (on)
                    list[total + __popcll(group & ((1ull << lane) - 1ull))] =
                        make_int4(slot[f] * F::NFN + at, code, (int)cnt[f], f);
                total += __popcll(group);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            for (int j0 = 0; j0 < total; j0 += G * UN) {
                double x[UN];
                int r[UN];
                bool on[UN];
#pragma unroll
                for (int u = 0; u < UN; ++u) {
                    const int j = j0 + u * G + grp;
                    on[u] = grp < G && j < total;
                    const int4 it = list[on[u] ? j : 0];
                    x[u] = p.rows[(int64_t)it.x * RL + l] * (double)it.z;
                    r[u] = lb < F::COLS ? p.rank_t[(int64_t)it.y * NEN + F::col(it.w, lb < F::COLS ? lb : 0)] : 0;
                }
#pragma unroll
                for (int u = 0; u < UN; ++u)
                    if (on[u]) unsafeAtomicAdd(lb < F::COLS ? buf + li * deg + r[u] : dbuf + li, x[u]);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        T* K = (T*)p.K;
        T* d = (T*)p.d;
        for (int t = lane; t < NF * deg; t += 64) {
            const int i = t / deg, r = t - i * deg;
            const int64_t at = p.field_major ? (int64_t)i * NF * p.n_pairs + NF * P + i * deg + r
                                             : P * (NF * NF) + i * NF * deg + r * NF + i;
            if (buf[t] != 0.0) K[at] = (T)((double)K[at] + buf[t]);
        }
        if (lane < NF && dbuf[lane] != 0.0) {
            const int64_t row = p.field_major ? lane * p.n_nodes + v : NF * v + lane;
            d[row] = (T)((double)d[row] + dbuf[lane]);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

template <int DIM, int NEN, int NF, typename T>
void launch_rows(const BParams& p, unsigned blocks, hipStream_t s)
{
    if constexpr (DIM == 2) k_edge_rows<NEN, NF, T><<<blocks, kThreads, 0, s>>>(p);
    else if constexpr (NEN == 8) k_face_rows8<NF, T><<<blocks, kThreads, 0, s>>>(p);
    else if constexpr (NEN == 20) k_face_rows20<NF, T><<<blocks, kThreads, 0, s>>>(p);
    else k_face_rows10<NF, T><<<blocks, kThreads, 0, s>>>(p);
}

// Marking, rows and gather; *done is false (nothing launched) when no workspace can be had.
template <int DIM, int NEN, int NF, typename T>
mf_status launch_faces(BParams p, const mf_pattern_s* P, hipStream_t s, bool* done)
{
    using F = Faces<DIM, NEN>;
    *done = true;
    if (p.n_faces == 0 || P->n_elems == 0) return MF_OK;
    const int64_t keys = P->n_elems * F::NLOC, most = std::min(p.n_faces, keys), nodes_most = std::min(most * F::NFN, P->n_nodes);
    if (most * F::NFN * NF > (int64_t)0x7fffffff * kThreads) return set_error(MF_ERR_ARG, "too many faces for one launch");
    // cnt [keys], node flags [n_nodes], two counters; slot [keys], list [most] where the call names
    // more faces than there are, nodes [most]; rows
    const bool listed = p.n_faces > keys;
    const int64_t clear = keys + P->n_nodes + 2, words = clear + keys + (listed ? most : 0) + nodes_most;
    const size_t rows_at = (sizeof(uint32_t) * (size_t)words + 255) / 256 * 256;
    const size_t rows = sizeof(double) * (size_t)most * F::NFN * NF * (F::COLS + 1);
    const Workspace held(P, rows_at + rows, s);
    char* ws = held.p;
    *done = ws != nullptr;
    if (held.full && (DIM != 3 || NEN != 8))
        return set_error(MF_ERR_UNSUPPORTED,
                         "captured boundary forms on one pattern: %d captures have a workspace (until the pattern is "
                         "destroyed), and this form has no other way",
                         (int)Workspace::kCaptured);
    if (!ws) return MF_OK;
    uint32_t* cnt = (uint32_t*)ws;
    uint32_t* node_on = cnt + keys;
    uint32_t* counts = node_on + P->n_nodes;
    int32_t* slot = (int32_t*)(counts + 2);
    int32_t* nodes = slot + keys;
    p.lists = {p.face_elem, p.face_id, p.n_faces, P->n_elems, P->conn, cnt, slot, listed ? nodes + nodes_most : nullptr,
               node_on, nodes, counts, listed ? 0u : (uint32_t)((p.n_faces + kThreads - 1) / kThreads), P->status};
    p.rows = (double*)(ws + rows_at);
    k_face_zero<<<(unsigned)((clear + kThreads - 1) / kThreads), kThreads, 0, s>>>(cnt, clear);
    if (listed) k_face_list<F><<<(unsigned)((p.n_faces + kThreads - 1) / kThreads), kThreads, 0, s>>>(p.lists);
    const int64_t threads = most * F::NFN * NF * (NEN == 10 ? kTetLanes : 1);
    launch_rows<DIM, NEN, NF, T>(p, p.lists.blocks + (unsigned)((threads + kThreads - 1) / kThreads), s);
    FaceGather g{};
    g.adj_ptr = P->adj_ptr;
    g.adj = P->adj;
    g.nbr_ptr = P->nbr_ptr;
    g.rank_t = P->rank_t;
    g.cnt = cnt;
    g.slot = slot;
    g.nodes = nodes;
    g.n_nodes_on = counts + 1;
    g.rows = p.rows;
    g.n_nodes = P->n_nodes;
    g.n_pairs = P->n_pairs;
    g.field_major = p.field_major;
    g.buf_len = (2 * 64 * kMaxAt + NF * std::max(1, P->max_deg) + 4 + 1) & ~1;  // 16-byte aligned
    g.K = p.K;
    g.d = p.d;
    // at most 255 neighbours and 3 fields: 37 kB for the four waves
    const unsigned blocks = (unsigned)std::min<int64_t>(8192, (nodes_most + 3) / 4);
    k_face_gather<DIM, NEN, NF, T><<<blocks, kThreads, sizeof(double) * 4 * (size_t)g.buf_len, s>>>(g);
    MF_HIP(hipGetLastError());
    return MF_OK;
}

// 8-node hexahedra: mark the listed faces per element, then one launch per element
// colour (elements of a colour share no node, so each row is added by one thread of the
// launch, and the colours follow each other in the stream: the sums do not depend on
// the run).  The face lists are in the pattern's workspace; past kCaptured captures in one buffer
// that those captured calls share.
template <int NF, typename T>
mf_status launch_boundary(BParams p, const mf_pattern_s* Pc, hipStream_t s)
{
    mf_pattern_s* P = const_cast<mf_pattern_s*>(Pc);
    if (p.n_faces == 0 || P->n_elems == 0) return MF_OK;
    mf_status st = ensure_coloring(P);
    if (st != MF_OK) return st;
    const int n_col = (int)P->color_ptr.size() - 1;
    // workspace: mask [n_el], counts [6 n_el], list lengths [n_col], colour lists [n_el]
    const int64_t n_el = P->n_elems;
    const size_t bytes = sizeof(uint32_t) * (size_t)(8 * n_el + n_col);
    const Workspace held(P, bytes, s);
    uint32_t* mask = (uint32_t*)held.p;
    if (held.full) {
        const RelaxedCapture relaxed;
        if (!P->shared_faces) MF_HIP(hipMalloc(&P->shared_faces, bytes));
        mask = P->shared_faces;
    }
    if (!mask) return set_error(MF_ERR_OOM, "no memory for the boundary faces' workspace");
    uint32_t* cnt = mask + n_el;
    uint32_t* ccount = cnt + 6 * n_el;
    int32_t* clist = (int32_t*)(ccount + n_col);
    const int64_t clear = 7 * n_el + n_col;
    k_face_zero<<<(unsigned)((clear + kThreads - 1) / kThreads), kThreads, 0, s>>>(mask, clear);
    k_face_mark<<<(unsigned)((p.n_faces + kThreads - 1) / kThreads), kThreads, 0, s>>>(
        p.face_elem, p.face_id, p.n_faces, n_el, P->elem_color, P->color_at, mask, cnt, clist, ccount, P->status);
    p.face_mask = mask;
    p.face_cnt = cnt;
    for (int c = 0; c < n_col; ++c) {
        // at most min(colour size, faces) elements of the colour carry faces
        const int64_t bound = std::min<int64_t>(P->color_ptr[c + 1] - P->color_ptr[c], p.n_faces) * 8 * NF;
        if (bound == 0) continue;
        const unsigned blocks = (unsigned)std::min<int64_t>(2048, (bound + kThreads - 1) / kThreads);
        auto run = [&](auto kernel) { kernel<<<blocks, kThreads, 0, s>>>(p, clist + P->color_ptr[c], ccount + c); };
        if constexpr (NF == 4) {
            switch (p.form.kind) {
                case MF_BFORM_NS_INFLOW: run(k_boundary<4, MF_BFORM_NS_INFLOW, T>); break;
                case MF_BFORM_NS_OUTFLOW: run(k_boundary<4, MF_BFORM_NS_OUTFLOW, T>); break;
                default: run(k_boundary<4, MF_BFORM_NS_FIX, T>);
            }
        } else {
            run(k_boundary<NF, -1, T>);
        }
    }
    MF_HIP(hipGetLastError());
    return MF_OK;
}

}  // namespace
}  // namespace mf

using namespace mf;

extern "C" mf_status mf_assemble_boundary(const mf_pattern_t* P, const mf_bform* form, const double* coords,
                                          int64_t n_faces, const int32_t* face_elem, const uint8_t* face_id,
                                          const void* state, const void* target, mf_precision prec, void* K,
                                          void* d, void* stream)
{
    clear_error();
    if (!P || !form) return set_error(MF_ERR_ARG, "pattern or form is NULL");
    const bool two_d = P->dim == 2;
    if (two_d ? (P->nen != 4 && P->nen != 8) : (P->nen != 8 && P->nen != 20 && P->nen != 10))
        return set_error(MF_ERR_UNSUPPORTED, "boundary forms need quadrilaterals, hexahedra or tetrahedra");
    const bool quad = P->order == 2;
    const bool tet = P->nen == 10;
    if (prec != MF_F64 && prec != MF_F32) return set_error(MF_ERR_ARG, "unknown precision %d", (int)prec);
    if (n_faces < 0 || n_faces > ((int64_t)1 << 28)) return set_error(MF_ERR_ARG, "n_faces out of range");
    if (n_faces > 0 && (!face_elem || !face_id || !coords || !K || !d))
        return set_error(MF_ERR_ARG, "NULL faces, coords, K or d");
    if (!P->full_coupling) return set_error(MF_ERR_ARG, "boundary forms need a fully coupled pattern");
    const int nf = P->nf;
    switch (form->kind) {
        case MF_BFORM_PENALTY:
            if (nf != 1 && nf != P->dim)
                return set_error(MF_ERR_ARG, "penalty needs 1 or %d fields, pattern has %d", P->dim, nf);
            break;
        case MF_BFORM_CONVECTION:
        case MF_BFORM_RADIATION:
        case MF_BFORM_FLUX:
            if (nf != 1) return set_error(MF_ERR_ARG, "this boundary form is scalar; pattern has %d fields", nf);
            break;
        case MF_BFORM_TRACTION:
            if (nf != P->dim) return set_error(MF_ERR_ARG, "traction needs %d fields, pattern has %d", P->dim, nf);
            break;
        case MF_BFORM_NS_INFLOW:
        case MF_BFORM_NS_OUTFLOW:
        case MF_BFORM_NS_FIX:
            if (nf != 4) return set_error(MF_ERR_ARG, "flow boundary forms need 4 fields, pattern has %d", nf);
            break;
        default: return set_error(MF_ERR_ARG, "unknown boundary form %d", (int)form->kind);
    }
    if ((quad || two_d) && (form->kind == MF_BFORM_FLUX || nf == 4))
        return set_error(MF_ERR_UNSUPPORTED, "the flux and flow boundary forms need 8-node hexahedra");
    if (tet && n_faces > 0 && !face_id) return set_error(MF_ERR_ARG, "NULL face_id");
    hipStream_t s = (hipStream_t)stream;
    BParams p{};
    p.form = *form;
    p.n_el = P->n_elems;
    p.n_nodes = P->n_nodes;
    p.n_faces = n_faces;
    p.conn = P->conn;
    p.coords = coords;
    p.row_ptr = P->row_ptr;
    p.nbr_ptr = P->nbr_ptr;
    p.rank = P->rank;
    p.face_elem = face_elem;
    p.face_id = face_id;
    p.state = state;
    p.target = target;
    p.field_major = P->numbering == MF_FIELD_MAJOR;
    p.K = K;
    p.d = d;
    p.status = P->status;
    const_cast<mf_pattern_s*>(P)->last_stream = s;
    if (two_d && nf != 1 && nf != 2) return set_error(MF_ERR_ARG, "edge forms need 1 or 2 fields, pattern has %d", nf);
    const bool f64 = prec == MF_F64;
    if (nf == 4) return f64 ? launch_boundary<4, double>(p, P, s) : launch_boundary<4, float>(p, P, s);
    bool done = false;
    auto run = [&](auto zero) -> mf_status {
        using T = decltype(zero);
        if (two_d && P->nen == 8)
            return nf == 1 ? launch_faces<2, 8, 1, T>(p, P, s, &done) : launch_faces<2, 8, 2, T>(p, P, s, &done);
        if (two_d) return nf == 1 ? launch_faces<2, 4, 1, T>(p, P, s, &done) : launch_faces<2, 4, 2, T>(p, P, s, &done);
        if (tet) return nf == 1 ? launch_faces<3, 10, 1, T>(p, P, s, &done) : launch_faces<3, 10, 3, T>(p, P, s, &done);
        if (quad) return nf == 1 ? launch_faces<3, 20, 1, T>(p, P, s, &done) : launch_faces<3, 20, 3, T>(p, P, s, &done);
        return nf == 1 ? launch_faces<3, 8, 1, T>(p, P, s, &done) : launch_faces<3, 8, 3, T>(p, P, s, &done);
    };
    const mf_status st = f64 ? run(0.0) : run(0.0f);
    if (st != MF_OK || done) return st;
    if (P->nen != 8 || two_d)
        return set_error(MF_ERR_OOM, "no memory for the boundary faces' workspace");
    if (nf == 1) return f64 ? launch_boundary<1, double>(p, P, s) : launch_boundary<1, float>(p, P, s);
    return f64 ? launch_boundary<3, double>(p, P, s) : launch_boundary<3, float>(p, P, s);
}
