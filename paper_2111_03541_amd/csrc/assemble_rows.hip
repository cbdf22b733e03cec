// Owner-computes assembly for meshes of any numbering (Sec. 2.2 D-2, D-3): every row of K
// and d is summed and written once, by the wave that owns its node, mostly from element data
// that a first kernel has left in the pattern's workspace.  No atomics on K, no clearing pass, no
// colours, and the sums do not depend on the run.
//
//  rows with the geometry (k_scalar_rows; scalar forms on 8-node bricks, up to some 40^3): the
//     wave that owns the node forms everything, without a first kernel.
//  element blocks (k_gather_blocks; scalar forms on larger meshes of 8-node bricks here,
//     every form on the quadratic elements in assemble_quadratic.hip): the first kernel
//     stores the element's rows [e][a][i][b][j]; the wave of node v adds the row blocks of its incidence list
//     (entry e*nen + a is the block's index) in LDS and writes its rows.
//  point records (k_brick_points, k_brick_rows; elasticity and the flow form on 8-node
//     bricks): a block is 4.6 kB (elasticity) or 8 kB (flow) and would cross HBM twice, so
//     the first kernel stores only the geometry (and the flow state) of the 8 Gauss points,
//     and the wave that owns the node forms the products.
//
// The workspace holds the data of all elements (up to about three times K), so that each row is
// summed once, in FP64 to the end.  (In chunks of 1 GiB, a node at a cut read and wrote its rows
// twice, FP32 rows were rounded between, and every node had to look for its entries and constrained
// neighbours again: mass 128^3 FP64 1344 us against 1043 in one, with constrained sides 1828 against
// 1150.)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "mf_internal.h"
#include "rows.h"

namespace mf {

RelaxedCapture::RelaxedCapture()
{
    if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) (void)hipGetLastError();
}

RelaxedCapture::~RelaxedCapture()
{
    if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) (void)hipGetLastError();
}

Workspace::Workspace(const mf_pattern_s* Pc, size_t bytes, hipStream_t stream)
    : P(const_cast<mf_pattern_s*>(Pc)), s(stream), lock(P->ws_mu)
{
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    unsigned long long id = 0;
    if (hipStreamGetCaptureInfo(s, &cap, &id) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    auto alloc = [&]() -> char* {
        void* q = nullptr;
        if (hipMalloc(&q, bytes) == hipSuccess) return (char*)q;
        (void)hipGetLastError();
        return nullptr;
    };
    if (cap != hipStreamCaptureStatusNone) {
        // calls in a capture share a workspace with their own stream's calls in that capture
        // only: a replay may overlap any later call, and a fork of it the other branches
        for (const auto& w : P->cap_ws)
            if (w.id == id && w.s == s && w.bytes >= bytes) {
                p = w.p;
                return;
            }
        // (a capture may hold several: other streams, a later and larger call)
        std::vector<unsigned long long> others;
        for (const auto& w : P->cap_ws)
            if (w.id != id && std::find(others.begin(), others.end(), w.id) == others.end()) others.push_back(w.id);
        full = others.size() >= kCaptured;
        if (full) return;
        RelaxedCapture relaxed;
        p = alloc();
        if (p) P->cap_ws.push_back({p, bytes, id, s});
        return;
    }
    // (the thread may be capturing another stream, which an allocation would end)
    const RelaxedCapture relaxed;
    if (!P->ws_done && hipEventCreateWithFlags(&P->ws_done, hipEventDisableTiming) != hipSuccess) {
        (void)hipGetLastError();
        P->ws_done = nullptr;
        return;
    }
    if (P->ws_bytes < bytes) {
        if (P->ws) {
            (void)hipEventSynchronize(P->ws_done);
            (void)hipFree(P->ws);
            P->ws = nullptr;
            P->ws_bytes = 0;
        }
        P->ws = alloc();
        if (!P->ws) return;
        P->ws_bytes = bytes;
    }
    // (an event that was never recorded counts as complete)
    if (hipStreamWaitEvent(s, P->ws_done, 0) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    p = P->ws;
    record = true;
}

Workspace::~Workspace()
{
    if (record && hipEventRecord(P->ws_done, s) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipStreamSynchronize(s);
    }
}

namespace {

constexpr int kWave = 64;

// ---------------------------------------------------------------- writing a node's rows

struct RowOut {
    const int32_t* nbr;
    const uint8_t* mask;  // Dirichlet flags or nullptr
    int64_t n_nodes, n_pairs;
};

// Entry (i, c) of a node's rows, c = r * NF + j node-major and j * deg + r field-major (r: the
// neighbour's rank, P: the node's offset in the node graph): its place in K.
template <int NF, bool FM>
__device__ __forceinline__ int64_t row_entry(const RowOut& o, int64_t P, int deg, int i, int c)
{
    return FM ? (int64_t)i * NF * o.n_pairs + NF * P + c : P * (NF * NF) + i * NF * deg + c;
}

// Homogeneous elimination (structure kept) in the row buffers of a wave's nodes, before they
// are written: a constrained column is zeroed, a constrained row becomes a unit row.  The nodes'
// neighbours are consecutive in the node graph, [P0, P0 + n): lane l looks at l, l + 64, ...
template <int NF, bool FM>
__device__ __forceinline__ uint32_t elim_flag(const RowOut& o, int64_t w)
{
    uint32_t f = 0;
#pragma unroll
    for (int j = 0; j < NF; ++j) f |= (uint32_t)(o.mask[FM ? j * o.n_nodes + w : NF * w + j] != 0) << j;
    return f;
}

// v0 .. v0 + nodes: the wave's nodes, P and deg lane n's (n < nodes) offset and neighbour count;
// `part` (lane n): the node takes part.  buf: the wave's row buffers, [i][c], or [i][j][r] (SPLIT).
template <int NF, bool FM, bool SPLIT>
__device__ __forceinline__ void eliminate(const RowOut& o, int64_t v0, int nodes, int P0, int n, int P, int deg, bool part,
                                          double* buf, int lane)
{
    for (int t0 = 0; t0 < n; t0 += kWave) {
        const int t = t0 + lane;
        const uint32_t f = t < n ? elim_flag<NF, FM>(o, o.nbr[P0 + t]) : 0;
        if (!__ballot(f != 0)) continue;
        int own = 0, ownP = P0, ownDeg = 0;  // the node whose neighbour this is
        for (int m = 0; m < nodes; ++m) {
            const int Pm = __shfl(P, m), dm = __shfl(deg, m);
            if (t >= Pm - P0 && t < Pm - P0 + dm) own = m, ownP = Pm, ownDeg = dm;
        }
        if (!__shfl((int)part, own) || f == 0) continue;
        const int r = t - (ownP - P0);
#pragma unroll
        for (int j = 0; j < NF; ++j)
            if ((f >> j) & 1)
#pragma unroll
                for (int i = 0; i < NF; ++i)
                    buf[(ownP - P0) * NF * NF + i * NF * ownDeg + (SPLIT ? j * ownDeg + r : r * NF + j)] = 0.0;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const uint32_t rows = lane < nodes && part ? elim_flag<NF, FM>(o, v0 + lane) : 0;
    for (unsigned long long left = __ballot(rows != 0); left; left &= left - 1) {
        const int m = __ffsll((long long)left) - 1;
        const int Pm = __shfl(P, m), dm = __shfl(deg, m);
        const uint32_t f = __shfl(rows, m);
        for (int r = lane; r < dm; r += kWave) {
            const bool self = o.nbr[Pm + r] == v0 + m;
#pragma unroll
            for (int i = 0; i < NF; ++i)
                if ((f >> i) & 1)
#pragma unroll
                    for (int j = 0; j < NF; ++j)
                        buf[(Pm - P0) * NF * NF + i * NF * dm + (SPLIT ? j * dm + r : r * NF + j)] =
                            self && i == j ? 1.0 : 0.0;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// The rows of one node from LDS to K by one wave.  buf: [i][c], or [i][j][r] when SPLIT.
template <int NF, bool FM, bool SPLIT, typename T>
__device__ __forceinline__ void write_rows(const RowOut& o, int64_t P, int deg, const double* buf, T* K, int lane)
{
    const int n = NF * deg;
    for (int c = lane; c < n; c += kWave) {
        const int r = c / NF, j = c - r * NF;
#pragma unroll
        for (int i = 0; i < NF; ++i)
            __builtin_nontemporal_store((T)buf[i * n + (SPLIT && !FM ? j * deg + r : c)],
                                        K + row_entry<NF, FM>(o, P, deg, i, c));
    }
}

// ------------------------------------------------------------------------ element blocks

struct GatherParams {
    const int32_t* adj_ptr;
    const int32_t* adj;
    const int32_t* nbr_ptr;
    const uint8_t* rank_t;
    RowOut out;
    const void* Ke;  // [n_elems * NEN][NF][NEN][NF] row blocks of the incidence entries
    const void* fe;  // [n_elems * NEN][NF] residual entries (d = sum)
    const uint8_t* emask;  // flags of the elements (with out.mask)
    int buf_len;     // doubles of LDS per wave
    double lam, mu;  // Lame parameters of E = 1
    void* K;
    void* d;
};

// One wave takes NPW nodes next to each other, whose incidence lists and neighbours are consecutive
// too: it reads the entries of all of them at once, so that the chain offsets - entries - blocks
// is paid once for many blocks.  A block row is contiguous (NF * NEN * NF values), so a wave
// reads whole lines, each once: CH values per lane of one block row, or one value per lane of SPP
// short ones, UN such passes in flight.  The wave's own LDS additions run in program order:
// ascending incidence entry, whatever the run.  Bound by the reads of the element blocks:
// conduction 64^3 FP64 55 us for 151 MB of blocks and 57 MB of rows (3.8 TB/s), elasticity on
// 24^3 20-node bricks 190 us for 401 MB and 300 MB (3.7 TB/s).  The nodes run from last to first,
// since the end of the blocks is what the first kernel left in the last-level cache.  LAME: the blocks hold E int dN_a,i dN_b,j, and
// the elastic combination is formed once per node pair, from the sums.
template <int NEN, int NF>
struct GatherShape {
    static constexpr int RB = NF * NEN * NF;
    static constexpr int SPP = RB >= kWave ? 1 : kWave / RB, CH = RB >= kWave ? (RB + kWave - 1) / kWave : 1;
    static constexpr int UN = CH >= 4 ? 2 : CH >= 2 ? 4 : 8;
    // nodes per wave on large meshes: short rows leave lanes and loads to spare
    static constexpr int NPW = RB >= kWave ? 1 : 8;
    // a node has at most 255 neighbours
    static_assert(sizeof(double) * NPW * (NF * NF * 255 + NF) <= 65536, "a wave's row buffers exceed the LDS");
};

template <int NEN, int NF, int NPW, typename T, bool FM, bool LAME>
__global__ void __launch_bounds__(256) k_gather_blocks(GatherParams p)
{
    using G = GatherShape<NEN, NF>;
    constexpr int RB = G::RB, SPP = G::SPP, CH = G::CH, UN = G::UN;
    extern __shared__ double sh[];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, n_nodes = (int)p.out.n_nodes;
    // from the last node to the first: the blocks written last are the ones still in the cache
    const int v0 = ((int)(gridDim.x - 1 - xcd_block(blockIdx.x, gridDim.x)) * (blockDim.x / kWave) + wave) * NPW;
    if (v0 >= n_nodes) return;
    double* buf = sh + wave * p.buf_len;  // row buffers of the nodes, one after another
    double* dbuf = buf + p.buf_len - NPW * NF;
    T* K = (T*)p.K;
    T* d = (T*)p.d;
    // lane n (mod NPW): node v0 + n (nodes past the end: no entries, no neighbours)
    const int v = v0 + lane % NPW, vc = min(v, n_nodes), vn = min(v + 1, n_nodes);
    const int a0 = p.adj_ptr[vc], a1 = p.adj_ptr[vn], P = p.nbr_ptr[vc], deg = p.nbr_ptr[vn] - P;
    const int A0 = __shfl(a0, 0), A1 = __shfl(a1, NPW - 1), P0 = __shfl(P, 0);
    const int n_nbr = __shfl(P + deg, NPW - 1) - P0;
    const bool on = v < n_nodes;
    int touched = 0;  // an element around a node has a constrained DOF
    for (int t = lane; t < n_nbr * NF * NF; t += kWave) buf[t] = 0.0;
    for (int t = lane; t < NPW * NF; t += kWave) dbuf[t] = 0.0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // the lane's values of a block row: column node, row and column field
    const int sl = SPP > 1 ? lane / RB : 0;
    int tb[CH], ti[CH], tj[CH];
#pragma unroll
    for (int u = 0; u < CH; ++u) {
        const int t = SPP > 1 ? lane - sl * RB : lane + u * kWave;
        const int i = t / (NEN * NF), c = t - i * (NEN * NF), b = c / NF;
        tb[u] = (SPP > 1 ? sl < SPP : t < RB) ? b : -1;
        ti[u] = i;
        tj[u] = c - b * NF;
        if (NPW == 1) ti[u] = i * NF * deg + (FM ? tj[u] * deg : tj[u]);  // its place but for the rank
    }
    for (int kb = A0; kb < A1; kb += kWave) {
        const int m = min(kWave, A1 - kb);
        // lane's entry (-1: none), its node's buffer and width
        const int k = kb + lane, mine = lane < m ? p.adj[k] : -1;
        int at = 0, width = 0, mydb = 0;
        double fd[NF];
        {
            int nd = 0;
#pragma unroll
            for (int n = 1; n < NPW; ++n) nd += k >= __shfl(a0, n);
            at = (__shfl(P, nd) - P0) * NF * NF;
            width = __shfl(deg, nd);
            if (p.out.mask && mine >= 0) touched |= p.emask[mine / NEN];
#pragma unroll
            for (int j = 0; j < NF; ++j) fd[j] = mine >= 0 ? (double)((const T*)p.fe)[(int64_t)mine * NF + j] : 0.0;
            mydb = nd * NF;
        }
        for (int s0 = 0; s0 < m; s0 += SPP * UN) {
            // (loads without conditions, past the end from entry 0: all of them in flight together)
            double val[UN][CH];
            int rk[UN][CH], base[UN], dg[UN];
            bool live[UN];
#pragma unroll
            for (int w = 0; w < UN; ++w) {
                const int s = s0 + w * SPP + sl, sc = s < m ? s : 0;
                const int c = SPP > 1 ? __shfl(mine, sc) : __builtin_amdgcn_readlane(mine, sc);
                base[w] = NPW > 1 ? __shfl(at, sc) : 0;
                dg[w] = NPW > 1 ? __shfl(width, sc) : 0;
                live[w] = s < m && c >= 0;
                const int64_t code = c >= 0 ? c : 0;
#pragma unroll
                for (int u = 0; u < CH; ++u) {
                    const int t = SPP > 1 ? lane - sl * RB : min(lane + u * kWave, RB - 1);
                    rk[w][u] = p.rank_t[code * NEN + (tb[u] >= 0 ? tb[u] : 0)];
                    val[w][u] = (double)__builtin_nontemporal_load((const T*)p.Ke + code * RB + t);
                }
            }
#pragma unroll
            for (int w = 0; w < UN; ++w)
#pragma unroll
                for (int u = 0; u < CH; ++u) {
                    const int r = rk[w][u];
                    const int pos = NPW == 1 ? ti[u] + (FM ? r : r * NF)
                                             : base[w] + ti[u] * NF * dg[w] + (FM ? tj[u] * dg[w] + r : r * NF + tj[u]);
                    if (live[w] && tb[u] >= 0) unsafeAtomicAdd(buf + pos, val[w][u]);
                }
        }
        if (mine >= 0)
#pragma unroll
            for (int j = 0; j < NF; ++j) unsafeAtomicAdd(dbuf + mydb + j, fd[j]);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if constexpr (LAME) {
        // K_ij = lam T_ij + mu T_ji + mu delta_ij tr T, in place, a node pair per lane
        for (int t0 = 0; t0 < n_nbr; t0 += kWave) {
            const int t = t0 + lane;
            int nd = 0;  // (every lane takes part in the exchanges)
#pragma unroll
            for (int n = 1; n < NPW; ++n) nd += t >= __shfl(P, n) - P0;
            const int Pn = __shfl(P, nd), dg = __shfl(deg, nd);
            if (t >= n_nbr) continue;
            double* pair = buf + (Pn - P0) * NF * NF;
            const int r = t - (Pn - P0);
            double x[NF][NF], tr = 0.0;
#pragma unroll
            for (int i = 0; i < NF; ++i) {
#pragma unroll
                for (int j = 0; j < NF; ++j) x[i][j] = pair[i * NF * dg + (FM ? j * dg + r : r * NF + j)];
                tr = fma(p.mu, x[i][i], tr);
            }
#pragma unroll
            for (int i = 0; i < NF; ++i)
#pragma unroll
                for (int j = 0; j < NF; ++j)
                    pair[i * NF * dg + (FM ? j * dg + r : r * NF + j)] =
                        fma(p.lam, x[i][j], p.mu * x[j][i]) + (i == j ? tr : 0.0);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    if (p.out.mask && __any(touched)) eliminate<NF, FM, FM>(p.out, v0, NPW, P0, n_nbr, P, deg, on, buf, lane);
    for (int t = lane; t < NPW * NF; t += kWave) {
        const int m = t / NF, j = t - m * NF;
        const int64_t row = FM ? (int64_t)j * n_nodes + v0 + m : (int64_t)NF * (v0 + m) + j;
        if (v0 + m < n_nodes) d[row] = (T)(p.out.mask && p.out.mask[row] ? 0.0 : dbuf[t]);
    }
    if constexpr (!FM) {
        T* out = K + (int64_t)P0 * (NF * NF);
#pragma unroll 4
        for (int t = lane; t < n_nbr * NF * NF; t += kWave) __builtin_nontemporal_store((T)buf[t], out + t);
        return;
    }
#pragma unroll 1
    for (int n = 0; n < NPW; ++n) {
        if (v0 + n >= n_nodes) break;
        const int Pn = __shfl(P, n);
        write_rows<NF, FM, FM, T>(p.out, Pn, __shfl(deg, n), buf + (Pn - P0) * (NF * NF), K, lane);
    }
}

template <int NEN, int NF, typename T, bool LAME = false>
mf_status launch_gather(const AssembleArgs& A, const void* Ke, const void* fe, const uint8_t* emask)
{
    const mf_pattern_s* P = A.P;
    GatherParams p{};
    p.adj_ptr = P->adj_ptr;
    p.adj = P->adj;
    p.nbr_ptr = P->nbr_ptr;
    p.rank_t = P->rank_t;
    p.out = {P->nbr, A.dirichlet, P->n_nodes, P->n_pairs};
    p.Ke = Ke;
    p.fe = fe;
    p.emask = emask;
    const double nu = A.form->nu;
    p.lam = nu / ((1.0 + nu) * (1.0 - 2.0 * nu));
    p.mu = 1.0 / (2.0 * (1.0 + nu));
    p.K = A.K;
    p.d = A.d;
    auto run = [&](auto npw) {
        constexpr int NPW = decltype(npw)::value;
        p.buf_len = NPW * (NF * NF * std::max(1, P->max_deg) + NF);
        const size_t per_wave = sizeof(double) * (size_t)p.buf_len;
        const int waves = per_wave * 4 <= 65536 ? 4 : per_wave * 2 <= 65536 ? 2 : 1;
        const unsigned blocks = (unsigned)((P->n_nodes + waves * NPW - 1) / (waves * NPW));
        const size_t lds = per_wave * waves;
        if (P->numbering == MF_FIELD_MAJOR)
            k_gather_blocks<NEN, NF, NPW, T, true, LAME><<<blocks, waves * kWave, lds, A.stream>>>(p);
        else
            k_gather_blocks<NEN, NF, NPW, T, false, LAME><<<blocks, waves * kWave, lds, A.stream>>>(p);
    };
    // 64^3 conduction: 55 us with eight nodes a wave, 95 with one; on 25 thousand nodes of
    // tetrahedra 24 against 19 (too few waves)
    constexpr int kMany = GatherShape<NEN, NF>::NPW;
    if (kMany > 1 && P->n_nodes >= 30000) run(std::integral_constant<int, kMany>{});
    else run(std::integral_constant<int, 1>{});
    MF_HIP(hipGetLastError());
    return MF_OK;
}

// ------------------------------------------------------- geometry of an 8-node brick point

constexpr double kHi = 0.5 * (1.0 + kGaussPt), kLo = 0.5 * (1.0 - kGaussPt);  // Q1 factors at a Gauss point

// N_a at Gauss point q: one factor per axis, kHi where the bits of a and q agree
__device__ __forceinline__ double brick_N(int a, int q)
{
    const int d = a ^ q;
    return ((d & 1) ? kLo : kHi) * ((d & 2) ? kLo : kHi) * ((d & 4) ? kLo : kHi);
}

__device__ __forceinline__ void brick_dN(int a, int q, double (&g)[3])
{
    const int d = a ^ q;
    const double fx = (d & 1) ? kLo : kHi, fy = (d & 2) ? kLo : kHi, fz = (d & 4) ? kLo : kHi;
    g[0] = ((a & 1) ? 0.5 : -0.5) * fy * fz;
    g[1] = ((a & 2) ? 0.5 : -0.5) * fx * fz;
    g[2] = ((a & 4) ? 0.5 : -0.5) * fx * fy;
}

// det J and its cofactors, C[n][m] = det J * dxi_n/dx_m.
__device__ __forceinline__ double cofactors(const double (&J)[3][3], double (&C)[3][3])
{
    C[0][0] = J[1][1] * J[2][2] - J[1][2] * J[2][1];
    C[0][1] = J[0][2] * J[2][1] - J[0][1] * J[2][2];
    C[0][2] = J[0][1] * J[1][2] - J[0][2] * J[1][1];
    C[1][0] = J[1][2] * J[2][0] - J[1][0] * J[2][2];
    C[1][1] = J[0][0] * J[2][2] - J[0][2] * J[2][0];
    C[1][2] = J[0][2] * J[1][0] - J[0][0] * J[1][2];
    C[2][0] = J[1][0] * J[2][1] - J[1][1] * J[2][0];
    C[2][1] = J[0][1] * J[2][0] - J[0][0] * J[2][1];
    C[2][2] = J[0][0] * J[1][1] - J[0][1] * J[1][0];
    return J[0][0] * C[0][0] + J[0][1] * C[1][0] + J[0][2] * C[2][0];
}

// det J and the cofactors of J at Gauss point q: C[n][m] = det J * dxi_n/dx_m.  X [8][3] in LDS.
__device__ __forceinline__ double brick_cofactors(const double* X, int q, double (&C)[3][3])
{
    double J[3][3];
#pragma unroll
    for (int m = 0; m < 3; ++m)
#pragma unroll
        for (int n = 0; n < 3; ++n) J[m][n] = 0.0;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        double g[3];
        brick_dN(b, q, g);
#pragma unroll
        for (int m = 0; m < 3; ++m)
#pragma unroll
            for (int n = 0; n < 3; ++n) J[m][n] = fma(X[b * 3 + m], g[n], J[m][n]);
    }
    return cofactors(J, C);
}

// Two layouts of the records.  By values, [NR / 2][8 points][elements][2], then the last
// value [8 points][elements]: the lanes of consecutive elements load one run.  By elements,
// [elements][8 points][NR]: a lane's loads are one run, for meshes whose consecutive nodes have
// elements anywhere, where a run of lanes would use 16 bytes of each line.  41x40x37 bricks, by
// values against by elements: renumbered at random elasticity 324 us against 143, flow 970 against
// 271; nodes shuffled among 64 neighbours 85 against 101 and 211 against 245; 64^3 in grid order 275
// against 328 and 982 against 1054.  Elements some thousand apart still meet in the L2 (4 MB), so
// the line lies at a quarter of the nodes with a first element more than 1024 from the next node's.
//
// Byte offsets in the records: pair m of point q of element e at e * pe + q * pq + m * pm, the last
// value at last + e * le + q * lq; residual entry (a, j) of element e at e * fe + a * fa + j * fj
// values.
struct RecLayout {
    int64_t pe, pq, pm, last, le, lq, fe, fa, fj;
};
typedef double f64x2 __attribute__((ext_vector_type(2), aligned(8)));

struct BrickParams {
    ElemMask em;
    mf_form form;
    int64_t n_el, n_nodes;
    const int32_t* conn;
    const double* coords;
    const void* elem_param;
    const void* src;  // nodal sources, or the flow state
    void* Ke;         // element blocks (scalar forms) or point records
    void* fe;
    RecLayout lay;    // of point records and their fe
    unsigned long long* status;
};

// Coordinates and sources of node b of element e into LDS, and whether it has a constrained DOF
// into *masked (cleared before, behind a barrier).  Returns the sum of the sources read,
// non-finite when one is.
template <int NSRC, typename T>
__device__ __forceinline__ double brick_load(const BrickParams& p, int64_t e, int b, bool live, double* X, double* S,
                                             int* masked)
{
    const int64_t node = live ? p.conn[(int64_t)b * p.n_el + e] : 0;
#pragma unroll
    for (int m = 0; m < 3; ++m) X[b * 3 + m] = live ? p.coords[(int64_t)m * p.n_nodes + node] : 0.0;
    double chk = 0.0;
#pragma unroll
    for (int j = 0; j < NSRC; ++j) {
        const double s = live && p.src ? (double)((const T*)p.src)[(int64_t)j * p.n_nodes + node] : 0.0;
        S[b * NSRC + j] = s;
        chk += s;
    }
    if (p.em.mask && live && p.em.node<NSRC>(node)) *masked = 1;
    return chk;
}

// Blocks of kBE elements: thread (point or node q, element el), elements fastest, so that the
// connectivity, the records and the blocks move in runs of kBE values.
constexpr int kBE = 32;

// Flags a bad Jacobian or a non-finite value of element el in LDS (cleared by the caller
// before a barrier; the caller's next barrier makes the flags visible) and in the status.
__device__ __forceinline__ void brick_flag(const BrickParams& p, int64_t e, bool live, double det, double chk, int* bad)
{
    if (!live) return;
    if (!(det > 0.0)) {
        *bad = 1;
        atomicMin(p.status, (unsigned long long)e);
    }
    if (!isfinite(chk)) atomicMin(p.status + 2, (unsigned long long)e);
}

// Mass and conduction on 8-node bricks: the element block.  Thread (point, element) forms the
// metric W c J^-1 J^-T (W c for the mass form) and W f in LDS, then thread (node a, element)
// sums row a over the points; the rows leave through LDS as whole lines.  Conduction 64^3 FP64:
// 63 us, of which 151 MB of stores take 23; the rest is the FP64 geometry and two barriers, with
// five waves per SIMD to hide them.  With the gather 118 us, where the column kernel, which
// forms the elements between two columns in both, took 272.
template <int FORM, typename T>
__global__ void __launch_bounds__(8 * kBE, 5) k_brick_scalar(BrickParams p)
{
    constexpr int NG = FORM == MF_FORM_MASS ? 2 : 7;  // metric, then W f
    // metrics [8 NG][kBE], then the blocks [kBE][64] (padded: elements on different banks)
    constexpr int kLen = 8 * NG * kBE > kBE * 65 ? 8 * NG * kBE : kBE * 65;
    __shared__ double sX[kBE][25], sS[kBE][9], sW[kLen];
    double(*sG)[kBE] = (double(*)[kBE])sW;
    __shared__ int sBad[kBE], sMask[kBE];
    const int el = threadIdx.x % kBE, q = threadIdx.x / kBE;
    const int64_t e = (int64_t)blockIdx.x * kBE + el;
    const bool live = e < p.n_el;
    if (q == 0) sBad[el] = sMask[el] = 0;
    if (p.em.mask) __syncthreads();
    double chk = brick_load<1, T>(p, e, q, live, sX[el], sS[el], &sMask[el]);
    const double c = p.form.coef * (live && p.elem_param ? (double)((const T*)p.elem_param)[e] : 1.0);
    __syncthreads();
    double C[3][3], f = 0.0;
    const double det = brick_cofactors(sX[el], q, C);
#pragma unroll
    for (int b = 0; b < 8; ++b) f = fma(brick_N(b, q), sS[el][b], f);
    brick_flag(p, e, live, det, chk + c + f, &sBad[el]);
    double g[NG];
    if constexpr (FORM == MF_FORM_MASS) {
        g[0] = det * c;
        g[1] = det * c * f;
    } else {
        const double s = c / det;  // W c (1/det)^2
#pragma unroll
        for (int n = 0, k = 0; n < 3; ++n)
#pragma unroll
            for (int m = n; m < 3; ++m, ++k)
                g[k] = s * (C[n][0] * C[m][0] + C[n][1] * C[m][1] + C[n][2] * C[m][2]);
        g[6] = det * f;
    }
#pragma unroll
    for (int k = 0; k < NG; ++k) sG[q * NG + k][el] = g[k];
    __syncthreads();
    const int a = q;
    double row[8], load = 0.0;
#pragma unroll
    for (int b = 0; b < 8; ++b) row[b] = 0.0;
#pragma unroll 2
    for (int k = 0; k < 8; ++k) {
        double h[NG];
#pragma unroll
        for (int m = 0; m < NG; ++m) h[m] = sG[k * NG + m][el];
        load = fma(brick_N(a, k), h[NG - 1], load);
        if constexpr (FORM == MF_FORM_MASS) {
            const double wa = h[0] * brick_N(a, k);
#pragma unroll
            for (int b = 0; b < 8; ++b) row[b] = fma(wa, kRefHex.N[k][b], row[b]);
        } else {
            double da[3];
            brick_dN(a, k, da);
            const double v0 = h[0] * da[0] + h[1] * da[1] + h[2] * da[2];
            const double v1 = h[1] * da[0] + h[3] * da[1] + h[4] * da[2];
            const double v2 = h[2] * da[0] + h[4] * da[1] + h[5] * da[2];
#pragma unroll
            for (int b = 0; b < 8; ++b)
                row[b] = fma(v0, kRefHex.dN[k][b][0], fma(v1, kRefHex.dN[k][b][1], fma(v2, kRefHex.dN[k][b][2], row[b])));
        }
    }
    const bool bad = sBad[el] != 0;  // such an element adds nothing
    __syncthreads();
#pragma unroll
    for (int b = 0; b < 8; ++b) sW[el * 65 + a * 8 + b] = bad ? 0.0 : row[b];
    if (live) {
        if (p.em.mask && q == 0) p.em.flag[e] = (uint8_t)sMask[el];
        ((T*)p.fe)[e * 8 + a] = bad ? T(0) : (T)load;
    }
    __syncthreads();
    // the blocks of the workgroup's elements are one contiguous range
    const int64_t e0 = (int64_t)blockIdx.x * kBE;
    const int n = (int)(p.n_el - e0 < kBE ? p.n_el - e0 : kBE) * 64;
    T* K = (T*)p.Ke + e0 * 64;
#pragma unroll
    for (int t = threadIdx.x; t < kBE * 64; t += 8 * kBE)
        if (t < n) K[t] = (T)sW[t / 64 * 65 + t % 64];
}

// ------------------------------------------------------------------------- point records

// Per form: fields, values of a record, column nodes per lane and workgroups per CU of the
// row kernel.  Records are read in pairs of values, 16 bytes a load.
template <int FORM>
struct Rec;

// elasticity: sqrt(det J) J^-1 (so that a product of two gradients carries the weight)
template <>
struct Rec<MF_FORM_ELASTICITY> {
    static constexpr int NF = 3, NR = 9, BPL = 8, WG = 2;
};
// flow: J^-1, W, u, c_0, grad u (row i, column l), c_1, c_2 with c = W (tau_m rho Rm - rho u);
// the first 14 are what a point's first products need
template <>
struct Rec<MF_FORM_NS_SUPG> {
    static constexpr int NF = 4, NR = 25, BPL = 4, WG = 2;
};

// Thread (point, element): the geometry once per element instead of once per row, as records
// of value pairs so that the lanes' stores and the row waves' loads are 16 bytes.  Bound by the
// latency of the node gathers and the stores: elasticity 64^3 60 us for 201 MB, flow 48^3 72 us
// for 205 MB.
template <int FORM, typename T>
__global__ void __launch_bounds__(8 * kBE) k_brick_points(BrickParams p)
{
    constexpr int NF = Rec<FORM>::NF, NR = Rec<FORM>::NR;
    constexpr bool NS = FORM == MF_FORM_NS_SUPG;
    // LDS per point: W f, or the record and W(tau_c div - p), W div, W tau_m Rm
    constexpr int NL = NS ? NR + 5 : 3;
    __shared__ double sX[kBE][25], sS[kBE][8 * NF + 1], sL[8 * NL][kBE];
    __shared__ int sBad[kBE], sMask[kBE];
    const int el = threadIdx.x % kBE, q = threadIdx.x / kBE;
    const int64_t e = (int64_t)blockIdx.x * kBE + el;
    const bool live = e < p.n_el;
    const double* S = sS[el];
    if (q == 0) sBad[el] = sMask[el] = 0;
    if (p.em.mask) __syncthreads();
    double chk = brick_load<NF, T>(p, e, q, live, sX[el], sS[el], &sMask[el]);
    if (NS) chk += p.form.rho + p.form.mu + p.form.tau_m + p.form.tau_c;
    else chk += p.form.coef * (live && p.elem_param ? (double)((const T*)p.elem_param)[e] : 1.0);
    __syncthreads();
    double C[3][3], u[NF], R[NR];
    const double det = brick_cofactors(sX[el], q, C);
#pragma unroll
    for (int j = 0; j < NF; ++j) u[j] = 0.0;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const double N = brick_N(b, q);
#pragma unroll
        for (int j = 0; j < NF; ++j) u[j] = fma(N, S[b * NF + j], u[j]);
    }
    double* L = &sL[q * NL][el];  // value k at L[k * kBE]
    if constexpr (!NS) {
        const double s = rsqrt(det);
#pragma unroll
        for (int n = 0; n < 3; ++n)
#pragma unroll
            for (int m = 0; m < 3; ++m) R[n * 3 + m] = s * C[n][m];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            chk += u[j];
            L[j * kBE] = det * u[j];
        }
    } else {
        const double r = 1.0 / det;
        double dU[4][3];
#pragma unroll
        for (int n = 0; n < 3; ++n)
#pragma unroll
            for (int m = 0; m < 3; ++m) R[n * 3 + m] = C[n][m] * r;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            double d[3] = {0.0, 0.0, 0.0};
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                double g[3];
                brick_dN(b, q, g);
#pragma unroll
                for (int n = 0; n < 3; ++n) d[n] = fma(g[n], S[b * 4 + j], d[n]);
            }
#pragma unroll
            for (int m = 0; m < 3; ++m) dU[j][m] = d[0] * R[m] + d[1] * R[3 + m] + d[2] * R[6 + m];
        }
        const double rho = p.form.rho, tm = p.form.tau_m, W = det;
        const double div = dU[0][0] + dU[1][1] + dU[2][2];
        R[9] = W;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const double Rm = rho * (u[0] * dU[i][0] + u[1] * dU[i][1] + u[2] * dU[i][2]) + dU[3][i];
            chk += Rm;
            R[10 + i] = u[i];
#pragma unroll
            for (int l = 0; l < 3; ++l) R[14 + 3 * i + l] = dU[i][l];
            R[i == 0 ? 13 : 22 + i] = W * rho * (tm * Rm - u[i]);
            L[(NR + 2 + i) * kBE] = W * tm * Rm;
        }
        chk += div;
        L[NR * kBE] = W * (p.form.tau_c * div - u[3]);
        L[(NR + 1) * kBE] = W * div;
#pragma unroll
        for (int k = 0; k < NR; ++k) L[k * kBE] = R[k];
    }
    brick_flag(p, e, live, det, chk, &sBad[el]);
    __syncthreads();
    if (!live) return;
    if (p.em.mask && q == 0) p.em.flag[e] = (uint8_t)sMask[el];
    const bool bad = sBad[el] != 0;  // such an element adds nothing
    char* rec = (char*)p.Ke + e * p.lay.pe + q * p.lay.pq;
#pragma unroll
    for (int k = 0; k < NR / 2; ++k) {
        const f64x2 x = {bad ? 0.0 : R[2 * k], bad ? 0.0 : R[2 * k + 1]};
        *(f64x2*)(rec + k * p.lay.pm) = x;
    }
    *(double*)((char*)p.Ke + p.lay.last + e * p.lay.le + q * p.lay.lq) = bad ? 0.0 : R[NR - 1];
    // residual entries of node a
    const int a = q;
    double f[NF];
#pragma unroll
    for (int j = 0; j < NF; ++j) f[j] = 0.0;
#pragma unroll 2
    for (int k = 0; k < 8; ++k) {
        const double* x = &sL[k * NL][el];
        const double N = brick_N(a, k);
        if constexpr (!NS) {
#pragma unroll
            for (int j = 0; j < 3; ++j) f[j] = fma(N, x[j * kBE], f[j]);
        } else {
            double da[3], g[3], adv = 0.0;
            brick_dN(a, k, da);
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                g[m] = da[0] * x[m * kBE] + da[1] * x[(3 + m) * kBE] + da[2] * x[(6 + m) * kBE];
                adv = fma(x[(10 + m) * kBE], g[m], adv);
            }
            const double muW = p.form.mu * x[9 * kBE];
#pragma unroll
            for (int i = 0; i < 3; ++i)
                f[i] -= adv * x[(i == 0 ? 13 : 22 + i) * kBE] + g[i] * x[NR * kBE] +
                        muW * (g[0] * x[(14 + 3 * i) * kBE] + g[1] * x[(15 + 3 * i) * kBE] + g[2] * x[(16 + 3 * i) * kBE]);
            f[3] -= N * x[(NR + 1) * kBE] + g[0] * x[(NR + 2) * kBE] + g[1] * x[(NR + 3) * kBE] + g[2] * x[(NR + 4) * kBE];
        }
    }
    T* fe = (T*)p.fe + e * p.lay.fe + a * p.lay.fa;
#pragma unroll
    for (int j = 0; j < NF; ++j) fe[j * p.lay.fj] = bad ? T(0) : (T)f[j];
}

// x and y factors of the trilinear basis at a point: the value, and the two derivatives
struct RefTablesQuad {
    double N[4][4];
    double dN[4][4][2];
    constexpr RefTablesQuad() : N{}, dN{}
    {
        for (int q = 0; q < 4; ++q)
            for (int a = 0; a < 4; ++a) {
                N[q][a] = ref_N<2>(a, q);
                for (int d = 0; d < 2; ++d) dN[q][a][d] = ref_dN<2>(a, q, d);
            }
    }
};
__constant__ constexpr RefTablesQuad kRefQuad{};

struct RowParams {
    mf_form form;
    const int32_t* adj_ptr;
    const int32_t* adj;
    const int32_t* nbr_ptr;
    const uint8_t* rank_t;
    RowOut out;
    const void* elem_param;
    const double* rec;
    RecLayout lay;
    const void* fe;
    const uint8_t* emask;  // flags of the elements (with out.mask)
    int buf_len, wave_len;  // doubles of LDS per node and per wave
    uint32_t plane, slots, shift;  // nodes of a grid plane (0: nodes in order), workgroups of a band in it; 2^shift nodes a workgroup
    void* K;
    void* d;
};

// The workgroup's nodes, in units of 2^shift, or -1.  A record is read by the eight nodes around
// its element.  In node order an XCD has passed a whole plane of the grid before the next reads it
// again, and a plane above some 2.5 MB of records has left the XCD's 4 MB of L2 by then, with all of K
// streaming through: each record was fetched twice (elasticity 64^3: 400 MB for 201).  So each XCD
// takes a band of an eighth of every plane, and goes through the planes: 255 MB fetched.  Whole calls,
// nodes in order against bands: flow 48^3 FP64 411 against 383 us, FP32 405 against 388, 40^3 FP64 226
// against 225, with constrained DOFs 255 against 250; elasticity 64^3 318 against 311, 62^3 313 against
// 285, 58^3 263 against 247.  Below, where the records stay, the bands' uneven ends only cost: flow 36^3 168
// against 175 (FP32, constrained 182 against 193), elasticity 48^3 137 against 140 (constrained 176
// against 180, FP32 162 against 167), 56^3 FP32 252 against 264.
__device__ __forceinline__ int row_block(const RowParams& p)
{
    if (p.plane == 0) return (int)xcd_block(blockIdx.x, gridDim.x);
    const uint32_t band = blockIdx.x % kXcds, r = blockIdx.x / kXcds, z = r / p.slots, plane = p.plane;
    const uint32_t part = plane / kXcds, rest = plane % kXcds, up = (1u << p.shift) - 1;
    const uint32_t lo = z * plane + band * part + band * rest / kXcds;  // (node ids have 31 bits)
    const uint32_t hi = z * plane + (band + 1) * part + (band + 1) * rest / kXcds;
    const uint32_t b = ((lo + up) >> p.shift) + (r - z * p.slots);
    return b < (hi + up) >> p.shift ? (int)b : -1;
}

// Products of one Gauss point: adds the blocks (a, b) of the lane's BPL column nodes.
// Elasticity: acc_ij += h_a,i h_b,j (the Lame combination follows once per block).
template <int BPL>
__device__ __forceinline__ void point_elasticity(int a, int q, const double (&h)[9], double (&acc)[BPL][3][3])
{
    double da[3], ga[3];
    brick_dN(a, q, da);
#pragma unroll
    for (int m = 0; m < 3; ++m) ga[m] = da[0] * h[m] + da[1] * h[3 + m] + da[2] * h[6 + m];
#pragma unroll
    for (int bb = 0; bb < BPL; ++bb) {
        const double* db = kRefHex.dN[q][bb];  // uniform: scalar loads
        double gb[3];
#pragma unroll
        for (int m = 0; m < 3; ++m) gb[m] = db[0] * h[m] + db[1] * h[3 + m] + db[2] * h[6 + m];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) acc[bb][i][j] = fma(ga[i], gb[j], acc[bb][i][j]);
    }
}

// Flow: with the factors of the row node gathered first, every entry is a combination of
// N_b, grad N_b, u . grad N_b and one scalar product.  Column node bb + 4 half: the z factor is
// the lane's, the others are uniform.
struct FlowPoint {
    double ga[3], Pg[3], tAr, rWadv, c0, zf;  // what the second part needs of the first
};

// First part, from the first 14 values of the record: all entries but the products with c
// and grad u.
template <int BPL, typename Issue>
__device__ __forceinline__ void point_flow_head(const mf_form& fm, int a, int half, int q, const double (&h)[14],
                                                FlowPoint& f, double (&acc)[BPL][4][4], const Issue& issue)
{
    double da[3];
    brick_dN(a, q, da);
#pragma unroll
    for (int m = 0; m < 3; ++m) f.ga[m] = da[0] * h[m] + da[1] * h[3 + m] + da[2] * h[6 + m];
    const double W = h[9], rtm = fm.rho * fm.tau_m;
    const double Wadv = W * (h[10] * f.ga[0] + h[11] * f.ga[1] + h[12] * f.ga[2]);
    const double tA = rtm * Wadv;  // W tau_m rho (u . grad N_a)
    const double WN = W * brick_N(a, q);
    const double zf = (half == (q >> 2)) ? kHi : kLo, sz = half ? 1.0 : -1.0;
    f.tAr = fm.rho * tA;
    f.rWadv = fm.rho * Wadv;
    f.c0 = h[13];
    f.zf = zf;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        f.Pg[i] = W * f.ga[i];
    }
#pragma unroll
    for (int bb = 0; bb < BPL; ++bb) {
        if (bb == BPL - 1) issue();  // the second part's loads
        const double cN = kRefQuad.N[q & 3][bb], c0 = kRefQuad.dN[q & 3][bb][0], c1 = kRefQuad.dN[q & 3][bb][1];
        const double c0z = c0 * zf, c1z = c1 * zf, c2z = (0.5 * cN) * sz, Nb = cN * zf;
        double gb[3];
#pragma unroll
        for (int m = 0; m < 3; ++m) gb[m] = c0z * h[m] + c1z * h[3 + m] + c2z * h[6 + m];
        const double ug = h[10] * gb[0] + h[11] * gb[1] + h[12] * gb[2], ub = rtm * ug;
        const double pb = f.Pg[0] * gb[0] + f.Pg[1] * gb[1] + f.Pg[2] * gb[2];
        const double yb = fma(fm.mu, pb, f.tAr * ug);
        const double tcg[3] = {fm.tau_c * gb[0], fm.tau_c * gb[1], fm.tau_c * gb[2]};
#pragma unroll
        for (int i = 0; i < 3; ++i) {
#pragma unroll
            for (int l = 0; l < 3; ++l) acc[bb][i][l] = fma(f.Pg[i], tcg[l], acc[bb][i][l]);
            acc[bb][i][i] += yb;
            acc[bb][i][3] = fma(tA, gb[i], fma(-f.Pg[i], Nb, acc[bb][i][3]));
            acc[bb][3][i] = fma(WN, gb[i], fma(f.Pg[i], ub, acc[bb][3][i]));
        }
        acc[bb][3][3] = fma(fm.tau_m, pb, acc[bb][3][3]);
    }
}

// Second part: r holds grad u (9), c_1, c_2.
template <int BPL>
__device__ __forceinline__ void point_flow_tail(const mf_form& fm, int q, const double (&r)[11], const FlowPoint& f,
                                                double (&acc)[BPL][4][4])
{
    const double rtm = fm.rho * fm.tau_m;
    double Nb[BPL];
#pragma unroll
    for (int bb = 0; bb < BPL; ++bb) Nb[bb] = kRefQuad.N[q & 3][bb] * f.zf;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            double X = fma(i == 0 ? f.c0 : r[8 + i], f.ga[l], f.tAr * r[3 * i + l]);
            if (l == i) X -= f.rWadv;
#pragma unroll
            for (int bb = 0; bb < BPL; ++bb) acc[bb][i][l] = fma(X, Nb[bb], acc[bb][i][l]);
        }
        __builtin_amdgcn_sched_barrier(0);  // row by row: the factors of all rows would not fit the registers
    }
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        const double S = rtm * (f.Pg[0] * r[l] + f.Pg[1] * r[3 + l] + f.Pg[2] * r[6 + l]);
#pragma unroll
        for (int bb = 0; bb < BPL; ++bb) acc[bb][3][l] = fma(S, Nb[bb], acc[bb][3][l]);
    }
}

// Lane (node, slot of its incidence list, group of BPL column nodes): the lane reads its
// element's records (consecutive nodes have consecutive elements on a mesh numbered with
// some locality, so a wave's load is a few runs), sums its BPL node blocks over the 8 points
// in registers, adds them to the node's row buffer in LDS, and the rows of the wave's nodes
// leave as one contiguous run.  Two waves per SIMD (the node blocks take half the registers),
// the next point's record is in flight during the products of the present one.  Elasticity 64^3
// FP64: 256 us, VALU busy 48 %; with k_brick_points 315 us, the column kernel 356; 41x40x37 renumbered
// bricks 143 us, the coloured scatter 1600.  Flow 48^3 FP64: 359 + 74 us, the coloured kernel 1540.
// FP32 builds sum in FP64 too: without packed math the rates are the same.
template <int FORM, typename T, bool FM>
__global__ void __launch_bounds__(256, (Rec<FORM>::WG)) k_brick_rows(RowParams p)
{
    using R = Rec<FORM>;
    constexpr int NF = R::NF, NR = R::NR, BPL = R::BPL;
    constexpr int GRP = 8 / BPL, LPN = 8 * GRP, NPW = kWave / LPN;
    constexpr int NH = FORM == MF_FORM_NS_SUPG ? 14 : NR;  // values of a record read together
    static_assert(BPL == 8 || BPL == 4, "the column node's z bit is a literal or the lane's group");
    // row buffers as K has them, or [i][j][r]: four values per neighbour next to each other
    // would put all lanes' additions into a quarter of the LDS banks
    constexpr bool SPLIT = FM || NF == 4;
    extern __shared__ __align__(16) double sh[];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    // lanes: node fastest, then group of column nodes, then slot
    const int grp = lane % NPW, half = lane / NPW % GRP, slot = lane / (NPW * GRP), sub = lane / NPW;
    const int n_nodes = (int)p.out.n_nodes, blk = row_block(p);
    const int v0 = (blk << p.shift) + wave * NPW, v = v0 + grp;
    if (blk < 0 || v0 >= n_nodes) return;
    const int wbase = wave * p.wave_len;  // the wave's row buffers, one after another
    double* dbuf = sh + wbase + NPW * p.buf_len + grp * NF;
    // (nodes past the end read the last offset: no entries, no neighbours)
    const int vc = min(v, n_nodes), vn = min(v + 1, n_nodes);
    const int a0 = p.adj_ptr[vc], a1 = p.adj_ptr[vn], P = p.nbr_ptr[vc], deg = p.nbr_ptr[vn] - P;
    const int P0 = __shfl(P, 0), n_wave = (__shfl(P + deg, NPW - 1) - P0) * NF * NF;
    const bool on = v < n_nodes;
    const int base = wbase + (P - P0) * (NF * NF);
    const int64_t drow = FM ? (int64_t)sub * n_nodes + v : (int64_t)NF * v + sub;
    T* K = (T*)p.K;
    T* d = (T*)p.d;
    int touched = 0;  // an element around the node has a constrained DOF
    for (int t = 2 * lane; t < n_wave; t += 2 * kWave) *(double2*)(sh + wbase + t) = make_double2(0.0, 0.0);
    if (sub < NF) dbuf[sub] = 0.0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    for (int k = a0 + slot; k < a1; k += 8) {
        const int code = p.adj[k];  // element * 8 + local node
        const int a = code & 7;
        const uint32_t e = (uint32_t)code >> 3;
        // value pairs [m0, m1) of the record at point q: uniform bases, 32-bit lane offset
        auto load_pairs = [&](int q, int m0, int m1, double* h) {
            uint32_t eo = e * (uint32_t)p.lay.pe;
            asm volatile("" : "+v"(eo));  // (a 64-bit lane address per value would not fit the registers)
            const char* b2 = (const char*)p.rec + q * p.lay.pq;
#pragma unroll
            for (int m = m0; m < m1; ++m) {
                const f64x2 x = *(const f64x2*)(b2 + m * p.lay.pm + eo);
                h[2 * (m - m0)] = x.x;
                h[2 * (m - m0) + 1] = x.y;
            }
        };
        auto load_last = [&](int q) {
            uint32_t eo = e * (uint32_t)p.lay.le;
            asm volatile("" : "+v"(eo));
            return *(const double*)((const char*)p.rec + p.lay.last + q * p.lay.lq + eo);
        };
        auto load_head = [&](int q, double (&h)[NH]) {
            load_pairs(q, 0, NH / 2, h);
            if constexpr (NH % 2) h[NH - 1] = load_last(q);
        };
        double acc[BPL][NF][NF];
#pragma unroll
        for (int bb = 0; bb < BPL; ++bb)
#pragma unroll
            for (int i = 0; i < NF; ++i)
#pragma unroll
                for (int j = 0; j < NF; ++j) acc[bb][i][j] = 0.0;
        double h0[NH];
        load_head(0, h0);
        // the next point's record is on its way while this one's products are formed
        if constexpr (FORM == MF_FORM_ELASTICITY) {
            double h1[NH];
#pragma unroll 1
            for (int q = 0; q < 8; q += 2) {
                load_head(q + 1, h1);
                point_elasticity<BPL>(a, q, h0, acc);
                load_head(q < 6 ? q + 2 : 7, h0);
                point_elasticity<BPL>(a, q + 1, h1, acc);
            }
        } else {
#pragma unroll 1
            for (int q = 0; q < 8; ++q) {
                double r[11];
                FlowPoint f;
                point_flow_head<BPL>(p.form, a, half, q, h0, f, acc, [&] {
                    load_pairs(q, 7, 12, r);
                    r[10] = load_last(q);
                });
                load_head(q < 7 ? q + 1 : 7, h0);
                point_flow_tail<BPL>(p.form, q, r, f, acc);
            }
        }
        // (here, as the wait for it would come before the first record's loads)
        if (p.out.mask) touched |= p.emask[code >> 3];
        uint32_t ranks[BPL / 4];
#pragma unroll
        for (int u = 0; u < BPL / 4; ++u) ranks[u] = *(const uint32_t*)(p.rank_t + (int64_t)code * 8 + (half + u) * 4);
        const T* fe = (const T*)p.fe + e * p.lay.fe + a * p.lay.fa;
        double fd[NF];
#pragma unroll
        for (int j = 0; j < NF; ++j) fd[j] = half == 0 ? (double)fe[j * p.lay.fj] : 0.0;
        double lam = 0.0, mu = 0.0;
        if constexpr (FORM == MF_FORM_ELASTICITY) {
            const double ep = p.elem_param ? (double)((const T*)p.elem_param)[code >> 3] : 1.0;
            const double E = p.form.coef * ep, nu = p.form.nu;
            lam = E * nu / ((1.0 + nu) * (1.0 - 2.0 * nu));
            mu = E / (2.0 * (1.0 + nu));
        }
#pragma unroll
        for (int bb = 0; bb < BPL; ++bb) {
            const int r = (ranks[bb >> 2] >> (8 * (bb & 3))) & 0xff;
            double tr = 0.0;
            if constexpr (FORM == MF_FORM_ELASTICITY) tr = mu * (acc[bb][0][0] + acc[bb][1][1] + acc[bb][2][2]);
#pragma unroll
            for (int i = 0; i < NF; ++i) {
                double* row = sh + base + i * NF * deg + (SPLIT ? r : r * NF);
#pragma unroll
                for (int j = 0; j < NF; ++j) {
                    double x = acc[bb][i][j];
                    if constexpr (FORM == MF_FORM_ELASTICITY) {
                        x = fma(lam, x, mu * acc[bb][j][i]);
                        if (i == j) x += tr;
                    }
                    unsafeAtomicAdd(row + (SPLIT ? j * deg : j), x);
                }
            }
        }
        if (half == 0)
#pragma unroll
            for (int j = 0; j < NF; ++j) unsafeAtomicAdd(dbuf + j, fd[j]);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (on && sub < NF) d[drow] = (T)(p.out.mask && p.out.mask[drow] ? 0.0 : dbuf[sub]);
    // (every lane takes part from here on)
    if (p.out.mask && __any(touched))
        eliminate<NF, FM, SPLIT>(p.out, v0, NPW, P0, n_wave / (NF * NF), P, deg, on, sh + wbase, lane);
    if constexpr (!SPLIT) {
        T* out = K + (int64_t)P0 * (NF * NF);
#pragma unroll 4
        for (int t = lane; t < n_wave; t += kWave) __builtin_nontemporal_store((T)sh[wbase + t], out + t);
        return;
    }
#pragma unroll 1
    for (int n = 0; n < NPW; ++n) {
        if (v0 + n >= n_nodes) break;
        const int Pn = __shfl(P, n);
        write_rows<NF, FM, SPLIT, T>(p.out, Pn, __shfl(deg, n), sh + wbase + (Pn - P0) * (NF * NF), K, lane);
    }
}

struct ScalarParams {
    mf_form form;
    int64_t n_el;
    const int32_t* conn;
    const double* coords;
    const int32_t* adj_ptr;
    const int32_t* adj;
    const int32_t* nbr_ptr;
    const uint8_t* rank_t;
    RowOut out;
    const void* elem_param;
    const void* src;
    int wave_len;  // doubles of LDS per wave: row buffers, then d
    void* K;
    void* d;
    unsigned long long* status;
};

// Mass and conduction without element data: lane (node, slot of its incidence list) forms its
// element's geometry and its row over the 8 points in registers, and adds the row to the node's in
// LDS.  Eight times the geometry of k_brick_scalar, but one launch, no workspace and nothing read
// back: bound by the FP64 instructions (1717 a wave for conduction, VALU busy 70 %) at three waves
// per SIMD; four spill (64^3 177 us against 126), and so does sharing the columns of J between the
// points (30 % fewer instructions, 350 us).  Conduction 28^3 18 us, where the column kernel took 35.
template <int FORM, typename T>
__global__ void __launch_bounds__(256, 3) k_scalar_rows(ScalarParams p)
{
    constexpr int NPW = 8;
    extern __shared__ __align__(16) double sh[];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int grp = lane % NPW, slot = lane / NPW;
    const int waves = blockDim.x / kWave, n_nodes = (int)p.out.n_nodes;
    const int v0 = ((int)xcd_block(blockIdx.x, gridDim.x) * waves + wave) * NPW, v = v0 + grp;
    if (v0 >= n_nodes) return;
    const int wbase = wave * p.wave_len;
    double* dbuf = sh + wbase + p.wave_len - NPW;
    const int vc = min(v, n_nodes), vn = min(v + 1, n_nodes);
    const int a0 = p.adj_ptr[vc], a1 = p.adj_ptr[vn], P = p.nbr_ptr[vc], deg = p.nbr_ptr[vn] - P;
    const int P0 = __shfl(P, 0), n_wave = __shfl(P + deg, NPW - 1) - P0;
    const int base = wbase + P - P0;
    int touched = 0;  // an element around the node has a constrained DOF
    for (int t = lane; t < n_wave; t += kWave) sh[wbase + t] = 0.0;
    if (lane < NPW) dbuf[lane] = 0.0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const T* src = (const T*)p.src;
    for (int k = a0 + slot; k < a1; k += 8) {
        const int code = p.adj[k];  // element * 8 + local node
        const int a = code & 7;
        const uint32_t e = (uint32_t)code >> 3;
        const uint2 ranks = *(const uint2*)(p.rank_t + (int64_t)code * 8);
        const double c = p.form.coef * (p.elem_param ? (double)((const T*)p.elem_param)[e] : 1.0);
        double x[8][3], S[8], chk = c;
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint32_t node = (uint32_t)p.conn[b * p.n_el + e];
            if (p.out.mask) touched |= p.out.mask[node];
#pragma unroll
            for (int m = 0; m < 3; ++m) x[b][m] = p.coords[(int64_t)m * n_nodes + node];
            S[b] = src ? (double)src[node] : 0.0;
            chk += S[b];
        }
        double row[8], load = 0.0;
        bool bad = false;
#pragma unroll
        for (int b = 0; b < 8; ++b) row[b] = 0.0;
#pragma unroll 1
        for (int q = 0; q < 8; ++q) {
            double J[3][3], C[3][3], u = 0.0;
#pragma unroll
            for (int m = 0; m < 3; ++m)
#pragma unroll
                for (int n = 0; n < 3; ++n) J[m][n] = 0.0;
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const double* g = kRefHex.dN[q][b];  // uniform: scalar loads
#pragma unroll
                for (int m = 0; m < 3; ++m)
#pragma unroll
                    for (int n = 0; n < 3; ++n) J[m][n] = fma(x[b][m], g[n], J[m][n]);
                u = fma(kRefHex.N[q][b], S[b], u);
            }
            const double det = cofactors(J, C), N = brick_N(a, q);
            bad |= !(det > 0.0);
            if constexpr (FORM == MF_FORM_MASS) {
                const double wN = det * c * N;
                load = fma(wN, u, load);
#pragma unroll
                for (int b = 0; b < 8; ++b) row[b] = fma(wN, kRefHex.N[q][b], row[b]);
            } else {
                const double s = c / det;
                double da[3], t[3], w[3];
                brick_dN(a, q, da);
#pragma unroll
                for (int m = 0; m < 3; ++m) t[m] = s * (da[0] * C[0][m] + da[1] * C[1][m] + da[2] * C[2][m]);
#pragma unroll
                for (int n = 0; n < 3; ++n) w[n] = t[0] * C[n][0] + t[1] * C[n][1] + t[2] * C[n][2];
                load = fma(det * N, u, load);
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    const double* g = kRefHex.dN[q][b];
                    row[b] = fma(w[0], g[0], fma(w[1], g[1], fma(w[2], g[2], row[b])));
                }
            }
        }
        if (bad) atomicMin(p.status, (unsigned long long)e);
        if (!isfinite(chk)) atomicMin(p.status + 2, (unsigned long long)e);
        if (!bad) {  // (such an element adds nothing)
#pragma unroll
            for (int b = 0; b < 8; ++b)
                unsafeAtomicAdd(sh + base + (((b < 4 ? ranks.x : ranks.y) >> (8 * (b & 3))) & 0xff), row[b]);
            unsafeAtomicAdd(dbuf + grp, load);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (lane < NPW && v0 + lane < n_nodes) ((T*)p.d)[v0 + lane] = (T)(p.out.mask && p.out.mask[v0 + lane] ? 0.0 : dbuf[lane]);
    if (p.out.mask && __any(touched)) eliminate<1, false, false>(p.out, v0, NPW, P0, n_wave, P, deg, v < n_nodes, sh + wbase, lane);
    T* out = (T*)p.K + P0;
    for (int t = lane; t < n_wave; t += kWave) __builtin_nontemporal_store((T)sh[wbase + t], out + t);
}

template <int FORM, typename T>
mf_status launch_scalar_rows(const AssembleArgs& A)
{
    const mf_pattern_s* P = A.P;
    ScalarParams p{};
    p.form = *A.form;
    p.n_el = P->n_elems;
    p.conn = P->conn;
    p.coords = A.coords;
    p.adj_ptr = P->adj_ptr;
    p.adj = P->adj;
    p.nbr_ptr = P->nbr_ptr;
    p.rank_t = P->rank_t;
    p.out = {P->nbr, A.dirichlet, P->n_nodes, P->n_pairs};
    p.elem_param = A.elem_param;
    p.src = A.nodal_src;
    p.wave_len = 8 * std::max(1, P->max_deg) + 8;  // at most 255 neighbours: 64 kB for four waves
    p.K = A.K;
    p.d = A.d;
    p.status = P->status;
    constexpr int kWaves = 4;
    const unsigned blocks = (unsigned)((P->n_nodes + kWaves * 8 - 1) / (kWaves * 8));
    k_scalar_rows<FORM, T><<<blocks, kWaves * kWave, sizeof(double) * kWaves * (size_t)p.wave_len, A.stream>>>(p);
    MF_HIP(hipGetLastError());
    return MF_OK;
}

template <typename T>
BrickParams brick_params(const AssembleArgs& A, void* Ke, void* fe, uint8_t* emask)
{
    const mf_pattern_s* P = A.P;
    BrickParams p{};
    p.form = *A.form;
    p.n_el = P->n_elems;
    p.n_nodes = P->n_nodes;
    p.conn = P->conn;
    p.coords = A.coords;
    p.elem_param = A.elem_param;
    p.src = A.form->kind == MF_FORM_NS_SUPG ? A.lin_state : A.nodal_src;
    p.Ke = Ke;
    p.fe = fe;
    p.em = {A.dirichlet, emask, P->n_nodes, P->numbering == MF_FIELD_MAJOR};
    p.status = P->status;
    return p;
}

template <int FORM, typename T>
mf_status launch_scalar(const AssembleArgs& A)
{
    const mf_pattern_s* P = A.P;
    const size_t per = sizeof(T) * (64 + 8) + 1, n = (size_t)P->n_elems;
    const Workspace ws(P, per * n, A.stream);
    char* w = ws.p;
    if (!w) return MF_ERR_UNSUPPORTED;
    void* fe = w + sizeof(T) * 64 * n;
    uint8_t* emask = (uint8_t*)w + sizeof(T) * 72 * n;
    const BrickParams p = brick_params<T>(A, w, fe, emask);
    k_brick_scalar<FORM, T><<<(unsigned)((P->n_elems + kBE - 1) / kBE), 8 * kBE, 0, A.stream>>>(p);
    MF_HIP(hipGetLastError());
    return launch_gather<8, 1, T>(A, w, fe, emask);
}

constexpr int64_t kPlaneBytes = 2500000;  // records of a grid plane that stay in an XCD's L2

template <int FORM, typename T>
mf_status launch_rows(const AssembleArgs& A)
{
    using R = Rec<FORM>;
    constexpr int NPW = kWave * R::BPL / 64;
    const mf_pattern_s* P = A.P;
    const int buf_len = R::NF * R::NF * std::max(1, P->max_deg);
    const int wave_len = (buf_len + R::NF) * NPW + 2 & ~1;  // 16-byte aligned, one double of slack
    const size_t per_wave = sizeof(double) * (size_t)wave_len;
    if (per_wave > 65536) return MF_ERR_UNSUPPORTED;  // hundreds of neighbours: the scatter
    const int waves = 4 * per_wave <= 65536 ? 4 : 2 * per_wave <= 65536 ? 2 : 1;
    const size_t rec = sizeof(double) * 8 * R::NR, per = rec + sizeof(T) * 8 * R::NF + 1;
    const int64_t n = P->n_elems;
    const Workspace ws(P, per * (size_t)n, A.stream);
    char* w = ws.p;
    if (!w) return MF_ERR_UNSUPPORTED;
    void* fe = w + rec * (size_t)n;
    uint8_t* emask = (uint8_t*)w + (per - 1) * (size_t)n;
    // by elements on a scattered mesh (lane offsets have 32 bits)
    const bool by_elem = P->scattered && n * 64 * R::NR < ((int64_t)1 << 32);
    const RecLayout lay = by_elem ? RecLayout{64 * R::NR, 8 * R::NR, 16, 8 * (R::NR - 1), 64 * R::NR, 8 * R::NR, 8 * R::NF, R::NF, 1}
                                  : RecLayout{16, 16 * n, 128 * n, 64 * (R::NR - 1) * n, 8, 8 * n, 1, R::NF * n, n};
    BrickParams b = brick_params<T>(A, w, fe, emask);
    b.lay = lay;
    k_brick_points<FORM, T><<<(unsigned)((n + kBE - 1) / kBE), 8 * kBE, 0, A.stream>>>(b);
    MF_HIP(hipGetLastError());
    RowParams p{};
    p.form = *A.form;
    p.adj_ptr = P->adj_ptr;
    p.adj = P->adj;
    p.nbr_ptr = P->nbr_ptr;
    p.rank_t = P->rank_t;
    p.out = {P->nbr, A.dirichlet, P->n_nodes, P->n_pairs};
    p.elem_param = A.elem_param;
    p.rec = (const double*)w;
    p.fe = fe;
    p.emask = emask;
    p.lay = lay;
    p.buf_len = buf_len;
    p.wave_len = wave_len;
    p.K = A.K;
    p.d = A.d;
    const int64_t per_block = (int64_t)waves * NPW;  // a power of two
    while ((int64_t)1 << p.shift < per_block) ++p.shift;
    unsigned blocks = (unsigned)((P->n_nodes + per_block - 1) / per_block);
    if (P->is_grid && (int64_t)per * P->gx * P->gy > kPlaneBytes) {
        p.plane = (uint32_t)((P->gx + 1) * (P->gy + 1));
        p.slots = (uint32_t)((p.plane / kXcds + per_block) / per_block) + 1;
        blocks = (unsigned)(kXcds * (P->gz + 1) * p.slots);
    }
    if (P->numbering == MF_FIELD_MAJOR) k_brick_rows<FORM, T, true><<<blocks, waves * kWave, per_wave * waves, A.stream>>>(p);
    else k_brick_rows<FORM, T, false><<<blocks, waves * kWave, per_wave * waves, A.stream>>>(p);
    MF_HIP(hipGetLastError());
    return MF_OK;
}

// Rows with the geometry, in one launch without a workspace, against element blocks and their gather
// (us; "fixed": with constrained sides).  Conduction 12^3 12 against 16, 28^3 17 against 35, 40^3 36
// against 44 (FP32 37 against 43, fixed 45 against 48, FP32 fixed 47 both), 48^3 56 against 59 (57
// against 56, 69 against 64, 71 against 63).  Mass, with half the work, 48^3 43 against 56, 52^3 55
// against 68 (FP32 59 to 64 against 62), 56^3 71 against 81 (81 against 74); fixed, where each lane
// looks up its element's flags, 46^3 53 against 58 (53 against 54), 48^3 60 against 62 (61 against 59),
// 50^3 71 against 68 (72 against 65), 52^3 79 against 74 (81 against 70).  On a scattered mesh each of a
// node's elements reads its 24 coordinates from anywhere: conduction 24^3 26 against 30 (FP32 26
// against 27), 27^3 32 against 36 (34 against 33), 30^3 41 both (44 against 38), 41x40x37 86 against 55;
// fixed 20^3 26 both (26 against 24), 24^3 32 both (31 against 29), 27^3 41 against 39 (43 against 37).
bool direct_wins(const AssembleArgs& A)
{
    const bool f32 = A.prec == MF_F32, fixed = A.dirichlet != nullptr;
    const int64_t n = A.P->n_elems;
    if (A.P->scattered) return n < (fixed ? (f32 ? 8000 : 14000) : f32 ? 16000 : 20000);
    if (A.form->kind == MF_FORM_MASS) return n < (!fixed ? 150000 : f32 ? 100000 : 115000);
    return n < 70000;
}

template <typename T>
mf_status dispatch_rows(const AssembleArgs& A)
{
    switch (A.form->kind) {
        case MF_FORM_MASS: return direct_wins(A) ? launch_scalar_rows<MF_FORM_MASS, T>(A) : launch_scalar<MF_FORM_MASS, T>(A);
        case MF_FORM_POISSON: return direct_wins(A) ? launch_scalar_rows<MF_FORM_POISSON, T>(A) : launch_scalar<MF_FORM_POISSON, T>(A);
        case MF_FORM_ELASTICITY: return launch_rows<MF_FORM_ELASTICITY, T>(A);
        case MF_FORM_NS_SUPG: return launch_rows<MF_FORM_NS_SUPG, T>(A);
    }
    return MF_ERR_UNSUPPORTED;
}

}  // namespace

mf_status gather_blocks(const AssembleArgs& A, int nen, int nf, const void* Ke, const void* fe, const uint8_t* emask)
{
    auto run = [&](auto zero) -> mf_status {
        using T = decltype(zero);
        switch (nen * 8 + nf) {
            case 20 * 8 + 1: return launch_gather<20, 1, T>(A, Ke, fe, emask);
            case 20 * 8 + 3: return launch_gather<20, 3, T, true>(A, Ke, fe, emask);
            case 20 * 8 + 4: return launch_gather<20, 4, T>(A, Ke, fe, emask);
            case 10 * 8 + 1: return launch_gather<10, 1, T>(A, Ke, fe, emask);
            case 10 * 8 + 3: return launch_gather<10, 3, T, true>(A, Ke, fe, emask);
            case 10 * 8 + 4: return launch_gather<10, 4, T>(A, Ke, fe, emask);
            case 8 * 8 + 1: return launch_gather<8, 1, T>(A, Ke, fe, emask);
            case 8 * 8 + 2: return launch_gather<8, 2, T, true>(A, Ke, fe, emask);
            case 8 * 8 + 3: return launch_gather<8, 3, T>(A, Ke, fe, emask);
        }
        return set_error(MF_ERR_ARG, "no gather for %d nodes and %d fields", nen, nf);
    };
    return A.prec == MF_F64 ? run(0.0) : run(0.0f);
}

mf_status assemble_rows(const AssembleArgs& A)
{
    const mf_pattern_s* P = A.P;
    if (P->dim != 3 || P->nen != 8 || P->n_elems == 0 || !P->full_coupling) return MF_ERR_UNSUPPORTED;
    return A.prec == MF_F64 ? dispatch_rows<double>(A) : dispatch_rows<float>(A);
}

}  // namespace mf
