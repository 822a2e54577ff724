// Finite-element assembly of the thermoelastic system (weak form wf_elastic,
// Sec. 3.1) into 3x3-block compressed rows, and Dirichlet elimination; and
// the residual and Newton Jacobian of the heat equation (weak form
// wf_thermal) in scalar compressed rows.
//
// Gather formulation, nothing is scattered: the stiffness rows of a node are
// built by one wave that walks the cells containing the node (ascending cell
// id, so the summation order is fixed and the result deterministic): the
// element blocks of a chunk of cells go through LDS and each lane adds them
// to the row blocks it owns, which are written once.  The load vectors take
// one thread per node, several load cases at a time.  Element integrals:
//   stiffness  P1: constant gradients; P2: degree-2 integrand, the integrals
//              of the products of barycentric coordinates in closed form;
//   thermal    P1: centroid rule (degree 1 exact); P2: degree-3 integrand,
//              5-point rule with barycentric points (1/4,...) weight -4/5 and
//              the permutations of (1/2,1/6,1/6,1/6) weight 9/20 (exact for
//              degree 3);
//   body force consistent mass: P1 |K|(1+delta_ac)/20; P2 the closed-form
//              10-node mass matrix (|K|/420: 6/1 vertex-vertex, -4/-6
//              vertex-edge, 32/16/8 edge-edge).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <numeric>

#include "te_dev.h"
#include "te_internal.h"
#include "te_thermal.h"

namespace te {

constexpr int ABLK = 64;
constexpr int PCAP = 192;  // maximum distinct neighbours of one node

__constant__ int c_edge[6][2] = {{0, 1}, {0, 2}, {0, 3}, {1, 2}, {1, 3}, {2, 3}};

// ---------------------------------------------------------------------------
// node -> (cell, local index) incidence
// ---------------------------------------------------------------------------
// bad: the first entry that is no node (initially all ones)
__global__ void k_check_cells(const int32_t *__restrict__ cells, int64_t n_entries, int64_t n_nodes,
                              unsigned long long *__restrict__ bad) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n_entries; t += (int64_t)gridDim.x * blockDim.x) {
        int32_t v = cells[t];
        if (v < 0 || v >= n_nodes) atomicMin(bad, (unsigned long long)t);
    }
}

// entries t = cell * npe + local node, local nodes below a0 left out
__global__ void k_inc_count(const int32_t *__restrict__ cells, int64_t n_entries, int npe, int a0,
                            int32_t *__restrict__ cnt) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n_entries; t += (int64_t)gridDim.x * blockDim.x)
        if (a0 == 0 || t % npe >= a0) atomicAdd(&cnt[cells[t]], 1);
}

__global__ void k_inc_fill(const int32_t *__restrict__ cells, int64_t n_entries, int npe, int a0,
                           const int64_t *__restrict__ start, int32_t *__restrict__ fill, int64_t *__restrict__ inc) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n_entries; t += (int64_t)gridDim.x * blockDim.x) {
        if (a0 != 0 && t % npe < a0) continue;
        int32_t v = cells[t];
        int32_t k = atomicAdd(&fill[v], 1);
        inc[start[v] + k] = t;
    }
}

// Per node: its entries in ascending order.  Lists of at most CAP entries go
// through registers, every entry placed by the number of smaller ones; longer
// ones are sorted by insertion.  524,576 P2 nodes: insertion alone 0.169 ms
// (a serial chain of loads and stores), now 0.040.
template <int CAP>
__device__ __forceinline__ void sort_list(int64_t *__restrict__ inc, int64_t lo, int len) {
    int64_t v[CAP];
#pragma unroll
    for (int a = 0; a < CAP; ++a) v[a] = a < len ? inc[lo + a] : INT64_MAX;
#pragma unroll
    for (int a = 0; a < CAP; ++a) {
        int r = 0;
#pragma unroll
        for (int b = 0; b < CAP; ++b) r += v[b] < v[a] ? 1 : 0;
        if (a < len) inc[lo + r] = v[a];
    }
}
__global__ void k_inc_sort(const int64_t *__restrict__ start, int64_t *__restrict__ inc, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t lo = start[i], hi = start[i + 1];
        if (hi - lo <= 8) {
            sort_list<8>(inc, lo, (int)(hi - lo));
        } else if (hi - lo <= 24) {
            sort_list<24>(inc, lo, (int)(hi - lo));
        } else {
            for (int64_t a = lo + 1; a < hi; ++a) {
                int64_t v = inc[a];
                int64_t b = a - 1;
                while (b >= lo && inc[b] > v) {
                    inc[b + 1] = inc[b];
                    --b;
                }
                inc[b + 1] = v;
            }
        }
    }
}

// Exclusive scan of int32 counts into int64 offsets (out[0] = 0, out[n] = total),
// three phases with fixed-size blocks.
__global__ void k_scan_block(const int32_t *__restrict__ in, int64_t *__restrict__ out, int64_t n,
                             int64_t *__restrict__ block_sums) {
    __shared__ int64_t s[1024];
    int64_t base = (int64_t)blockIdx.x * 1024;
    int64_t i = base + threadIdx.x;
    s[threadIdx.x] = (i < n) ? (int64_t)in[i] : 0;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        int64_t v = (threadIdx.x >= (unsigned)o) ? s[threadIdx.x - o] : 0;
        __syncthreads();
        s[threadIdx.x] += v;
        __syncthreads();
    }
    if (i < n) out[i + 1] = s[threadIdx.x];  // inclusive -> shifted
    if (threadIdx.x == 1023) block_sums[blockIdx.x] = s[1023];
}
// exclusive prefix sums of the block sums, in place: one workgroup
__global__ void __launch_bounds__(1024) k_scan_sums(int64_t nb, int64_t *__restrict__ bs) {
    __shared__ int64_t s[1024];
    int64_t base = 0;
    for (int64_t b0 = 0; b0 < nb; b0 += 1024) {
        const int64_t i = b0 + threadIdx.x;
        const int64_t own = i < nb ? bs[i] : 0;
        s[threadIdx.x] = own;
        __syncthreads();
        for (int o = 1; o < 1024; o <<= 1) {
            const int64_t v = (threadIdx.x >= (unsigned)o) ? s[threadIdx.x - o] : 0;
            __syncthreads();
            s[threadIdx.x] += v;
            __syncthreads();
        }
        if (i < nb) bs[i] = base + s[threadIdx.x] - own;
        base += s[1023];
        __syncthreads();
    }
}
__global__ void k_scan_add(int64_t *__restrict__ out, int64_t n, const int64_t *__restrict__ block_off) {
    int64_t i = (int64_t)blockIdx.x * 1024 + threadIdx.x;
    if (i < n) out[i + 1] += block_off[blockIdx.x];
    if (i == 0) out[0] = 0;
}

// bs: scratch of (n + 1023) / 1024 sums, kept by the caller until the stream has run
static void scan_counts(const int32_t *cnt, int64_t *out, int64_t n, DBuf<int64_t> &bs, hipStream_t s) {
    const int64_t nb = (n + 1023) / 1024;   // n > 0
    bs.alloc(nb);
    hipLaunchKernelGGL(k_scan_block, dim3((unsigned)nb), dim3(1024), 0, s, cnt, out, n, bs.p);
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(1024), 0, s, nb, bs.p);
    hipLaunchKernelGGL(k_scan_add, dim3((unsigned)nb), dim3(1024), 0, s, out, n, bs.p);
    TE_CHECK_HIP(hipGetLastError());
}

// the first of n_entries node numbers outside [0, n_nodes), -1 if there is none
static int64_t first_bad_node(const int32_t *nodes, int64_t n_entries, int64_t n_nodes, hipStream_t s) {
    DBuf<unsigned long long> bad(1);
    TE_CHECK_HIP(hipMemsetAsync(bad.p, 0xFF, sizeof(unsigned long long), s));
    const unsigned g = (unsigned)std::min<int64_t>((n_entries + 255) / 256 + 1, 1 << 20);
    hipLaunchKernelGGL(k_check_cells, dim3(g), dim3(256), 0, s, nodes, n_entries, n_nodes, bad.p);
    TE_CHECK_HIP(hipGetLastError());
    int64_t hb = -1;
    TE_CHECK_HIP(hipMemcpyAsync(&hb, bad.p, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    TE_CHECK_HIP(hipStreamSynchronize(s));
    return hb;
}

// node -> entries of `cells` (n_cells x npe node numbers, checked) whose local
// node is a0 or above, ascending if `sorted`.  Returns after the launches; cnt and bs are
// scratch that the caller keeps until the stream has run.
static void entry_lists(const int32_t *cells, int64_t n_cells, int npe, int a0, int64_t n, bool sorted,
                        Incidence &I, DBuf<int32_t> &cnt, DBuf<int64_t> &bs, hipStream_t s) {
    const int64_t ne = n_cells * (int64_t)npe;
    const unsigned g = (unsigned)std::min<int64_t>((ne + 255) / 256 + 1, 1 << 20);
    cnt.alloc(n);
    I.start.alloc(n + 1);
    I.inc.alloc(std::max<int64_t>(ne, 1));
    TE_CHECK_HIP(hipMemsetAsync(cnt.p, 0, n * sizeof(int32_t), s));
    hipLaunchKernelGGL(k_inc_count, dim3(g), dim3(256), 0, s, cells, ne, npe, a0, cnt.p);
    scan_counts(cnt.p, I.start.p, n, bs, s);
    TE_CHECK_HIP(hipMemsetAsync(cnt.p, 0, n * sizeof(int32_t), s));
    hipLaunchKernelGGL(k_inc_fill, dim3(g), dim3(256), 0, s, cells, ne, npe, a0, I.start.p, cnt.p, I.inc.p);
    unsigned gn = (unsigned)std::min<int64_t>((n + 255) / 256 + 1, 1 << 20);
    if (sorted) hipLaunchKernelGGL(k_inc_sort, dim3(gn), dim3(256), 0, s, I.start.p, I.inc.p, n);
    TE_CHECK_HIP(hipGetLastError());
}

// (a pattern needs the cells of a node in no particular order)
static void build_incidence(const te_mesh *m, int npe, Incidence &I, hipStream_t s, bool sorted = true) {
    const int64_t n = m->n_nodes, ne = m->n_cells * (int64_t)npe;
    TE_REQUIRE(first_bad_node(m->cells, ne, n, s) < 0, TE_EINVAL,
               "cells reference a node index outside [0, n_nodes)");
    DBuf<int32_t> cnt;
    DBuf<int64_t> bs;
    entry_lists(m->cells, m->n_cells, npe, 0, n, sorted, I, cnt, bs, s);
    TE_CHECK_HIP(hipStreamSynchronize(s));
}

// ---------------------------------------------------------------------------
// sparsity pattern
// ---------------------------------------------------------------------------
// The distinct nodes of one node's cells, found by one wave: hashed into LDS
// with linear probing, then each one's rank among them by counting.
constexpr int PTAB = 256;  // slots, more than PCAP
struct RowSet {
    int32_t key[PTAB];     // node, -1 = empty
    int16_t pos[PTAB];     // its position in the ascending row (after rank)
    union {
        struct {
            int32_t lst[PTAB];   // the nodes in the order of their arrival
            int16_t at[PTAB];    // and their slots
        };
        unsigned long long hit[PCAP];   // k_stiff, once the ranks are known
    };
    int32_t num, over;
};
__device__ __forceinline__ uint32_t row_hash(int32_t v) { return ((uint32_t)v * 2654435761u) >> 24; }

// the slot of a node, which the set has to hold
__device__ __forceinline__ int row_find(const RowSet &R, int32_t v) {
    uint32_t h = row_hash(v);
    for (int probe = 0; probe < PTAB && R.key[h] != v; ++probe) h = (h + 1) & (PTAB - 1);
    return (int)h;
}
__device__ __forceinline__ void row_clear(RowSet &R) {
    for (int t = threadIdx.x; t < PTAB; t += 64) R.key[t] = -1;
    if (threadIdx.x == 0) R.num = R.over = 0;
    __syncthreads();
}
// puts a node into the set -> its slot
__device__ __forceinline__ int row_insert(RowSet &R, int32_t v) {
    uint32_t h = row_hash(v);
    for (int probe = 0; probe < PTAB; ++probe) {
        const int32_t old = atomicCAS(&R.key[h], -1, v);
        if (old == -1) {
            const int k = atomicAdd(&R.num, 1);
            R.lst[k] = v;
            R.at[k] = (int16_t)h;
        }
        if (old == -1 || old == v) return (int)h;
        h = (h + 1) & (PTAB - 1);
    }
    R.over = 1;
    return 0;
}
// -> the number of distinct nodes, PCAP + 1 if there are more than PCAP
__device__ __forceinline__ int row_count(const RowSet &R) {
    __syncthreads();
    return R.over || R.num > PCAP ? PCAP + 1 : R.num;
}
// Sorted distinct neighbours of a node, one wave per node.  col null: their
// number to cnt[i]; otherwise the list to col[row_ptr[i] ..].
//   An insertion into a sorted list of one thread per node (48 KB of LDS for 64
// nodes) took 1.19 ms on 524,576 P2 nodes; now 0.151 ms.
__global__ void __launch_bounds__(64) k_pattern(const int32_t *__restrict__ cells, int npe,
                                                const int64_t *__restrict__ start, const int64_t *__restrict__ inc,
                                                int64_t n, int32_t *__restrict__ cnt,
                                                const int64_t *__restrict__ row_ptr, int32_t *__restrict__ col,
                                                int32_t *__restrict__ overflow) {
    __shared__ RowSet R;
    const int lane = threadIdx.x;
    for (int64_t i = xcd_logical_block(blockIdx.x, gridDim.x); i < n; i += gridDim.x) {
        const int64_t e0 = start[i];
        const int total = (int)(start[i + 1] - e0) * npe;
        row_clear(R);
        for (int t = lane; t < total; t += 64) {
            const int e = t / npe;
            row_insert(R, cells[inc[e0 + e] / npe * npe + (t - e * npe)]);
        }
        const int m = row_count(R);
        if (m > PCAP) {
            if (lane == 0) *overflow = 1;
        } else if (!col) {
            if (lane == 0) cnt[i] = m;
        } else if (row_ptr[i + 1] - row_ptr[i] != m) {
            // row_ptr comes from the caller: never write past its row
            if (lane == 0) *overflow = 2;
        } else {
            for (int x = lane; x < m; x += 64) {
                const int32_t v = R.lst[x];
                int r = 0;
                for (int y = 0; y < m; ++y) r += R.lst[y] < v ? 1 : 0;
                col[row_ptr[i] + r] = v;
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// element integrals
// ---------------------------------------------------------------------------
struct Geo {
    double G[4][3];  // gradient of barycentric coordinate k
    double vol;
};

// x: the four vertices
__device__ __forceinline__ Geo vertex_geo(const double *x) {
    double J[3][3];
    for (int k = 0; k < 3; ++k)
        for (int c = 0; c < 3; ++c) J[c][k] = x[(k + 1) * 3 + c] - x[c];  // columns = edges
    // inverse via cofactors: rows of J^-1 are the gradients of l1..l3
    double det = J[0][0] * (J[1][1] * J[2][2] - J[1][2] * J[2][1]) - J[0][1] * (J[1][0] * J[2][2] - J[1][2] * J[2][0]) +
                 J[0][2] * (J[1][0] * J[2][1] - J[1][1] * J[2][0]);
    double id = 1.0 / det;
    Geo g;
    g.G[1][0] = (J[1][1] * J[2][2] - J[1][2] * J[2][1]) * id;
    g.G[1][1] = (J[0][2] * J[2][1] - J[0][1] * J[2][2]) * id;
    g.G[1][2] = (J[0][1] * J[1][2] - J[0][2] * J[1][1]) * id;
    g.G[2][0] = (J[1][2] * J[2][0] - J[1][0] * J[2][2]) * id;
    g.G[2][1] = (J[0][0] * J[2][2] - J[0][2] * J[2][0]) * id;
    g.G[2][2] = (J[0][2] * J[1][0] - J[0][0] * J[1][2]) * id;
    g.G[3][0] = (J[1][0] * J[2][1] - J[1][1] * J[2][0]) * id;
    g.G[3][1] = (J[0][1] * J[2][0] - J[0][0] * J[2][1]) * id;
    g.G[3][2] = (J[0][0] * J[1][1] - J[0][1] * J[1][0]) * id;
    for (int c = 0; c < 3; ++c) g.G[0][c] = -(g.G[1][c] + g.G[2][c] + g.G[3][c]);
    g.vol = fabs(det) / 6.0;
    return g;
}
__device__ __forceinline__ Geo cell_geo(const double *__restrict__ X, const int32_t *__restrict__ cv) {
    double x[12];
    for (int k = 0; k < 4; ++k)
        for (int c = 0; c < 3; ++c) x[k * 3 + c] = X[(int64_t)cv[k] * 3 + c];
    return vertex_geo(x);
}

// Element tables are indexed by runtime node numbers; to keep them out of
// private (scratch) memory, the barycentric values are selected from
// registers and the gradients are read from LDS (G: [4][3] row-major).
__device__ __forceinline__ double sel4(double v0, double v1, double v2, double v3, int k) {
    return k == 0 ? v0 : (k == 1 ? v1 : (k == 2 ? v2 : v3));
}

// gradient of the P2 basis function a at the barycentric point (l0..l3)
__device__ __forceinline__ void p2_grad(int a, double l0, double l1, double l2, double l3, const double *G,
                                        double out[3]) {
    if (a < 4) {
        const double s = 4.0 * sel4(l0, l1, l2, l3, a) - 1.0;
        for (int c = 0; c < 3; ++c) out[c] = s * G[a * 3 + c];
    } else {
        const int i = c_edge[a - 4][0], j = c_edge[a - 4][1];
        const double li = sel4(l0, l1, l2, l3, i), lj = sel4(l0, l1, l2, l3, j);
        for (int c = 0; c < 3; ++c) out[c] = 4.0 * (lj * G[i * 3 + c] + li * G[j * 3 + c]);
    }
}

// closed-form P2 mass matrix times 420/|K|
__device__ __forceinline__ double p2_mass420(int a, int c) {
    if (a < 4 && c < 4) return a == c ? 6.0 : 1.0;
    if (a >= 4 && c >= 4) {
        if (a == c) return 32.0;
        int i0 = c_edge[a - 4][0], i1 = c_edge[a - 4][1], j0 = c_edge[c - 4][0], j1 = c_edge[c - 4][1];
        bool share = (i0 == j0) || (i0 == j1) || (i1 == j0) || (i1 == j1);
        return share ? 16.0 : 8.0;
    }
    int v = a < 4 ? a : c, e = a < 4 ? c : a;
    bool contains = (c_edge[e - 4][0] == v) || (c_edge[e - 4][1] == v);
    return contains ? -4.0 : -6.0;
}

struct AsmArgs {
    const double *X;
    const int32_t *cells;
    int npe;
    const int64_t *start;
    const int64_t *inc;
    int64_t n;
    double lam, mu, calpha, T_ref;
    const double *coef;  // per cell (lam, mu, (3 lam + 2 mu) alpha) [C][3], or null: the scalars above
    const double *T;   // [nrhs][N]
    const double *f;   // [nrhs][N][3] or null
    const int64_t *row_ptr;
    int32_t *col;      // columns and values of the stiffness (k_stiff)
    double *val;
    double *b;         // [N][3][nrhs]
    int nrhs;
};

// Loads of node i for the JT right-hand sides j0 = JT * blockIdx.y ... (thermal
// strain and body force), one thread per node over its cells in ascending
// order.  A cell's contribution is linear in its nodal temperatures and
// forces: its coefficients (the geometry, and for P2 the quadrature sum) are
// formed once and applied to all JT cases, whose nodal values are read row by
// row of T and f (neighbouring lanes read neighbouring nodes).  With many
// cases the geometry of a node's cells is thus formed nrhs / 8 times instead
// of nrhs times.  The workgroups of one XCD take neighbouring nodes, whose values
// then come from its L2.  64 cases with body forces on
// 334,368 P1 nodes 23.0 -> 7.4 -> 5.9 ms (what is left is the nodal reads
// through the L1), one case on 524,576 P2 nodes 0.31 -> 0.18 ms.
template <int DEG, int JT>
__global__ void __launch_bounds__(ABLK) k_load(AsmArgs A) {
    const int64_t i = xcd_logical_block(blockIdx.x, gridDim.x) * ABLK + threadIdx.x;
    if (i >= A.n) return;
    constexpr int NPE = DEG == 1 ? 4 : 10;
    const int j0 = JT * blockIdx.y;
    double bi[JT][3];
#pragma unroll
    for (int t = 0; t < JT; ++t)
#pragma unroll
        for (int c = 0; c < 3; ++c) bi[t][c] = 0.0;
    for (int64_t e = A.start[i]; e < A.start[i + 1]; ++e) {
        const int64_t cell = A.inc[e] / NPE;
        const int a = (int)(A.inc[e] % NPE);
        const int32_t *cv = A.cells + cell * NPE;
        int64_t nd[NPE];
#pragma unroll
        for (int c = 0; c < NPE; ++c) nd[c] = cv[c];
        const Geo g = cell_geo(A.X, cv);
        const double calpha = A.coef ? A.coef[cell * 3 + 2] : A.calpha;
        double cT[DEG == 1 ? 1 : NPE][3];   // b_c += sum over nodes of cT[node][c] dT[node] (P1: of cT[0][c] dT)
        if (DEG == 1) {
            // thermal: (3 lam + 2 mu) alpha |K| mean(dT) grad l_a
#pragma unroll
            for (int c = 0; c < 3; ++c)
                cT[0][c] = 0.25 * calpha * g.vol * sel4(g.G[0][c], g.G[1][c], g.G[2][c], g.G[3][c], a);
        } else {
            // thermal load, degree-3 exact 5-point rule
#pragma unroll
            for (int k = 0; k < NPE; ++k)
#pragma unroll
                for (int c = 0; c < 3; ++c) cT[k % (DEG == 1 ? 1 : NPE)][c] = 0.0;
            // gradient of phi_a: (4 l_a - 1) grad l_a, or 4 (l_j grad l_i + l_i grad l_j)
            const int ei = a < 4 ? a : c_edge[a - 4][0], ej = a < 4 ? a : c_edge[a - 4][1];
            double gi[3], gj[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                gi[c] = sel4(g.G[0][c], g.G[1][c], g.G[2][c], g.G[3][c], ei);
                gj[c] = sel4(g.G[0][c], g.G[1][c], g.G[2][c], g.G[3][c], ej);
            }
#pragma unroll
            for (int qp = 0; qp < 5; ++qp) {
                // (1/4,1/4,1/4,1/4), then the permutations of (1/2,1/6,1/6,1/6)
                const double l[4] = {qp == 0 ? 0.25 : (qp == 1 ? 0.5 : 1.0 / 6.0),
                                     qp == 0 ? 0.25 : (qp == 2 ? 0.5 : 1.0 / 6.0),
                                     qp == 0 ? 0.25 : (qp == 3 ? 0.5 : 1.0 / 6.0),
                                     qp == 0 ? 0.25 : (qp == 4 ? 0.5 : 1.0 / 6.0)};
                const double li = sel4(l[0], l[1], l[2], l[3], ei), lj = sel4(l[0], l[1], l[2], l[3], ej);
                const double w = calpha * (qp == 0 ? -0.8 : 0.45) * g.vol;
                double gr[3];
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    gr[c] = w * (a < 4 ? (4.0 * li - 1.0) * gi[c] : 4.0 * (lj * gi[c] + li * gj[c]));
#pragma unroll
                for (int k = 0; k < NPE; ++k) {
                    constexpr int E0[6] = {0, 0, 0, 1, 1, 2}, E1[6] = {1, 2, 3, 2, 3, 3};
                    const double phi = k < 4 ? l[k & 3] * (2.0 * l[k & 3] - 1.0)
                                             : 4.0 * l[E0[(k + 2) % 6]] * l[E1[(k + 2) % 6]];
#pragma unroll
                    for (int c = 0; c < 3; ++c) cT[k % (DEG == 1 ? 1 : NPE)][c] += phi * gr[c];
                }
            }
        }
#pragma unroll
        for (int t = 0; t < JT; ++t) {
            const int j = j0 + t < A.nrhs ? j0 + t : A.nrhs - 1;   // a spare case repeats the last, and is not stored
            const double *T = A.T + (int64_t)j * A.n;
            if (DEG == 1) {
                double s = 0.0;
#pragma unroll
                for (int k = 0; k < NPE; ++k) s += T[nd[k]] - A.T_ref;
#pragma unroll
                for (int c = 0; c < 3; ++c) bi[t][c] += cT[0][c] * s;
            } else {
#pragma unroll
                for (int k = 0; k < NPE; ++k) {
                    const double dT = T[nd[k]] - A.T_ref;
#pragma unroll
                    for (int c = 0; c < 3; ++c) bi[t][c] += cT[k % (DEG == 1 ? 1 : NPE)][c] * dT;
                }
            }
        }
        if (A.f) {
            double m[NPE];   // row a of the consistent mass matrix
#pragma unroll
            for (int k = 0; k < NPE; ++k)
                m[k] = DEG == 1 ? g.vol * (k == a ? 2.0 : 1.0) / 20.0 : g.vol * p2_mass420(a, k) / 420.0;
#pragma unroll
            for (int t = 0; t < JT; ++t) {
                const int j = j0 + t < A.nrhs ? j0 + t : A.nrhs - 1;
                const double *f = A.f + (int64_t)j * A.n * 3;
#pragma unroll
                for (int k = 0; k < NPE; ++k)
#pragma unroll
                    for (int c = 0; c < 3; ++c) bi[t][c] += m[k] * f[nd[k] * 3 + c];
            }
        }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int t = 0; t < JT; ++t)
            if (j0 + t < A.nrhs) A.b[(i * 3 + c) * A.nrhs + j0 + t] = bi[t][c];
}

// one case: one pass; more: LOAD_JT cases per pass
constexpr int LOAD_JT = 8;
static void launch_load(const AsmArgs &a, int degree, hipStream_t s) {
    const dim3 g((unsigned)((a.n + ABLK - 1) / ABLK), a.nrhs == 1 ? 1 : (a.nrhs + LOAD_JT - 1) / LOAD_JT);
    if (a.nrhs == 1) {
        if (degree == 1) hipLaunchKernelGGL((k_load<1, 1>), g, dim3(ABLK), 0, s, a);
        else hipLaunchKernelGGL((k_load<2, 1>), g, dim3(ABLK), 0, s, a);
    } else {
        if (degree == 1) hipLaunchKernelGGL((k_load<1, LOAD_JT>), g, dim3(ABLK), 0, s, a);
        else hipLaunchKernelGGL((k_load<2, LOAD_JT>), g, dim3(ABLK), 0, s, a);
    }
    TE_CHECK_HIP(hipGetLastError());
}

// coefficients of the integral of grad phi_a (x) grad phi_b over a P2 cell,
// divided by its volume.  A basis gradient is 4 l_m1 G_k1 + 4 l_m2 G_k2 for an
// edge (k1, k2) = (m2, m1), and (4 l_a - 1) G_a for a vertex; with
// int l_i l_j = (1 + d_ij) |K| / 20 and int l_i = |K| / 4.
struct P2Grad {
    int k1, k2, m1, m2;
    double c, w;   // the constant term of G_k1 and whether there is a G_k2 term
};
__device__ __forceinline__ P2Grad p2_terms(int a) {
    // the six edges (0,1) (0,2) (0,3) (1,2) (1,3) (2,3), four bits each
    const int e = 4 * (a < 4 ? 0 : a - 4), i = (0x211000 >> e) & 15, j = (0x332321 >> e) & 15;
    if (a < 4) return {a, a, a, a, -1.0, 0.0};
    return {i, j, j, i, 0.0, 1.0};
}

// Stiffness rows and their columns, one wave per node row.  The distinct nodes
// of the row's cells are its columns.  The cells are then taken CH
// at a time: lanes compute their geometries, then one lane per (cell, b) the
// element block K_e[a][b]; the chunk's cells that meet a row block, and the b of
// each, are gathered in four bits per cell.  Lane q owns blocks q, q + 64,
// q + 128 of the row (at most PCAP) and adds the chunk's blocks to them in cell
// order: block q in registers, the others, which few rows have, in place.
//   Bound by the latency of the dependent steps (cells of the row, their nodes,
// coordinates, blocks), so by the waves in flight: CH is what one pass over the
// lanes takes.  With the columns written by a kernel before, 16 cells in LDS,
// every block looked for in every cell and P2 integrals by quadrature: 3.03 +
// 1.19 ms on 524,576 P2 nodes; now 1.41 ms for both, half of it the issue of 810
// vector instructions per row.
template <int DEG>
__global__ void __launch_bounds__(64, 4) k_stiff(AsmArgs A, int64_t nnzb, int32_t *__restrict__ overflow) {
    constexpr int NPE = DEG == 1 ? 4 : 10, CH = 64 / NPE;
    static_assert(CH <= 16, "four bits per cell");
    __shared__ RowSet R;
    __shared__ double s_geo[CH][15];  // the vertices, then the gradients of the 4 barycentric coordinates, volume, lam, mu
    __shared__ double s_k[64][9];
    __shared__ int32_t s_dup;
    const int lane = threadIdx.x, c = lane / NPE, bb = lane - c * NPE;   // lane (c, bb): cell, local node
    for (int64_t i = xcd_logical_block(blockIdx.x, gridDim.x); i < A.n; i += gridDim.x) {
        const int64_t r0 = A.row_ptr[i], r1 = A.row_ptr[i + 1];
        const int64_t e0 = A.start[i];
        const int ne = (int)(A.start[i + 1] - e0);
        int64_t ent = 0;   // of the lane's cell in the current chunk
        int32_t v = 0;     // the node and its coordinates
        double x[3] = {0.0, 0.0, 0.0};
        int slot = 0;
        auto fetch = [&](int cb) {
            if (c < CH && cb + c < ne) {
                ent = A.inc[e0 + cb + c];
                v = A.cells[ent / NPE * NPE + bb];
            }
        };
        auto fetch_x = [&](int cb) {
            if (c < CH && cb + c < ne && bb < 4)
                for (int k = 0; k < 3; ++k) x[k] = A.X[(int64_t)v * 3 + k];
        };
        row_clear(R);
        // the first chunk last: what it fetched is what the loop below starts with
        for (int cb = ne > 0 ? (ne - 1) / CH * CH : -1; cb >= 0; cb -= CH) {
            fetch(cb);
            if (cb == 0) fetch_x(0);
            if (c < CH && cb + c < ne) slot = row_insert(R, v);
        }
        const int len = row_count(R);
        // row_ptr comes from the caller: never write past its row
        const int bad = len > PCAP ? 1 : r1 - r0 != len || r0 < 0 || r1 > nnzb ? 2 : 0;
        if (bad) {
            if (lane == 0) *overflow = bad;
            __syncthreads();
            continue;
        }
        for (int y0 = lane; y0 < len; y0 += 64) {
            const int32_t w = R.lst[y0];
            int r = 0;
            for (int y = 0; y < len; ++y) r += R.lst[y] < w ? 1 : 0;
            A.col[r0 + r] = w;
            R.pos[R.at[y0]] = (int16_t)r;
        }
        if (lane == 0) s_dup = 0;
        double acc[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) acc[k] = 0.0;
        for (int cb = 0; cb < ne; cb += CH) {
            const int nc = ne - cb < CH ? ne - cb : CH;
            const int a = (int)(ent % NPE);
            __syncthreads();   // the ranks are taken, the last chunk is added
            for (int t = lane; t < len; t += 64) R.hit[t] = 0;
            if (c < nc && bb < 4)
                for (int k = 0; k < 3; ++k) s_geo[c][bb * 3 + k] = x[k];
            if (c < nc && bb < 2) {
                const int64_t cell = ent / NPE;
                s_geo[c][13 + bb] = A.coef ? A.coef[cell * 3 + bb] : bb ? A.mu : A.lam;
            }
            if (cb > 0 && c < nc) slot = row_find(R, v);
            int p = R.pos[slot];
            if (cb + CH < ne) {   // the next chunk's nodes meanwhile
                fetch(cb + CH);
                fetch_x(cb + CH);
            }
            __syncthreads();
            if (lane < nc) {
                const Geo g = vertex_geo(s_geo[lane]);
                for (int k = 0; k < 4; ++k)
                    for (int d = 0; d < 3; ++d) s_geo[lane][k * 3 + d] = g.G[k][d];
                s_geo[lane][12] = g.vol;
            }
            __syncthreads();
            if (c < nc) {
                const double *G = s_geo[c];
                const double vol = G[12], lam = G[13], mu = G[14];
                double H[3][3];   // int grad phi_a (x) grad phi_b / |K|
                if (DEG == 1) {
#pragma unroll
                    for (int d = 0; d < 3; ++d)
#pragma unroll
                        for (int y = 0; y < 3; ++y) H[d][y] = G[a * 3 + d] * G[bb * 3 + y];
                } else {
                    const P2Grad u = p2_terms(a), w = p2_terms(bb);
                    auto mass = [](int x, int y) { return x == y ? 1.6 : 0.8; };   // 16 int l_x l_y / |K|
                    const double m11 = mass(u.m1, w.m1) + u.c + w.c + u.c * w.c, m12 = w.w * (mass(u.m1, w.m2) + u.c);
                    const double m21 = u.w * (mass(u.m2, w.m1) + w.c), m22 = u.w * w.w * mass(u.m2, w.m2);
#pragma unroll
                    for (int y = 0; y < 3; ++y) {
                        const double b1 = G[w.k1 * 3 + y], b2 = G[w.k2 * 3 + y];
                        const double h1 = m11 * b1 + m12 * b2, h2 = m21 * b1 + m22 * b2;
#pragma unroll
                        for (int d = 0; d < 3; ++d) H[d][y] = G[u.k1 * 3 + d] * h1 + G[u.k2 * 3 + d] * h2;
                    }
                }
                const double dot = mu * (H[0][0] + H[1][1] + H[2][2]);
#pragma unroll
                for (int d = 0; d < 3; ++d)
#pragma unroll
                    for (int y = 0; y < 3; ++y)
                        s_k[lane][d * 3 + y] = vol * (lam * H[d][y] + mu * H[y][d] + (d == y ? dot : 0.0));
                const unsigned long long old = atomicOr(&R.hit[p], (unsigned long long)(bb + 1) << (4 * c));
                if ((old >> (4 * c)) & 15) s_dup = 1;
            }
            __syncthreads();
            if (s_dup) {   // a cell names a node twice: the later local node counts
                if (c < nc) atomicAnd(&R.hit[p], ~(15ull << (4 * c)));
                __syncthreads();
                for (int b = 0; b < NPE; ++b) {
                    if (c < nc && bb == b) {
                        atomicAnd(&R.hit[p], ~(15ull << (4 * c)));
                        atomicOr(&R.hit[p], (unsigned long long)(bb + 1) << (4 * c));
                    }
                    __syncthreads();
                }
            }
            auto add = [&](int blk, double (&v)[9]) {
                unsigned long long hit = R.hit[blk];
                while (hit) {   // cells ascending
                    const int cc = __builtin_ctzll(hit) >> 2;
                    const double *K = s_k[cc * NPE + (int)((hit >> (4 * cc)) & 15) - 1];
#pragma unroll
                    for (int k = 0; k < 9; ++k) v[k] += K[k];
                    hit &= ~(15ull << (4 * cc));
                }
            };
            if (lane < len) add(lane, acc);
            for (int blk = lane + 64; blk < len; blk += 64) {
                double o[9], *dst = A.val + (r0 + blk) * 9;
#pragma unroll
                for (int k = 0; k < 9; ++k) o[k] = cb == 0 ? 0.0 : dst[k];
                add(blk, o);
#pragma unroll
                for (int k = 0; k < 9; ++k) dst[k] = o[k];
            }
        }
        if (lane < len)
#pragma unroll
            for (int k = 0; k < 9; ++k) A.val[(r0 + lane) * 9 + k] = acc[k];
        __syncthreads();
    }
}

// Columns and values of the rows of a pattern whose row pointer the caller holds.
// A refused row pointer is found on the way: rows that match are written by then,
// so the caller writes its other outputs after this.
static void stiffness_rows(const AsmArgs &a, int degree, int64_t nnzb, hipStream_t s) {
    DBuf<int32_t> ovf(1);
    TE_CHECK_HIP(hipMemsetAsync(ovf.p, 0, sizeof(int32_t), s));
    const unsigned gs = (unsigned)std::min<int64_t>(a.n, 1 << 18);
    if (degree == 1) hipLaunchKernelGGL(k_stiff<1>, dim3(gs), dim3(64), 0, s, a, nnzb, ovf.p);
    else hipLaunchKernelGGL(k_stiff<2>, dim3(gs), dim3(64), 0, s, a, nnzb, ovf.p);
    TE_CHECK_HIP(hipGetLastError());
    int32_t h = 0;
    TE_CHECK_HIP(hipMemcpyAsync(&h, ovf.p, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    TE_CHECK_HIP(hipStreamSynchronize(s));
    TE_REQUIRE(h == 0, TE_EINVAL, h == 1 ? "a node couples to more than 192 nodes"
                                         : "row_ptr does not match this mesh's sparsity pattern");
}

// Dirichlet elimination, eight lanes per row.  Lifting with the unconstrained
// values first (every eighth block per lane, the eight sums added in a fixed
// order), then rows/columns of constrained DOFs zeroed, unit diagonal,
// b_D = u_D.  One thread per row strode over the columns and values of 64 rows
// at a time: 0.273 ms on 524,576 P2 nodes (14.3 M blocks); now 0.080.
__global__ void __launch_bounds__(256) k_dirichlet(int64_t n, const int64_t *__restrict__ row_ptr,
                                                   const int32_t *__restrict__ col, double *__restrict__ val,
                                                   double *__restrict__ b, const uint8_t *__restrict__ mask,
                                                   const double *__restrict__ ubc) {
    const int l = threadIdx.x & 7;
    for (int64_t i0 = blockIdx.x * (int64_t)32; i0 < n; i0 += (int64_t)gridDim.x * 32) {
        const int64_t i = i0 + (threadIdx.x >> 3);
        double lift[3] = {0.0, 0.0, 0.0};
        bool mi[3] = {false, false, false};
        if (i < n) {
            for (int p = 0; p < 3; ++p) mi[p] = mask[i * 3 + p] != 0;
            for (int64_t k = row_ptr[i] + l; k < row_ptr[i + 1]; k += 8) {
                const int64_t J = col[k];
                const bool mj[3] = {mask[J * 3] != 0, mask[J * 3 + 1] != 0, mask[J * 3 + 2] != 0};
                if (!(mi[0] || mi[1] || mi[2] || mj[0] || mj[1] || mj[2])) continue;
                double *blk = val + k * 9;
                for (int q = 0; q < 3; ++q) {
                    if (!mj[q]) continue;
                    const double u = ubc ? ubc[J * 3 + q] : 0.0;
                    for (int p = 0; p < 3; ++p) lift[p] += blk[p * 3 + q] * u;
                }
                for (int p = 0; p < 3; ++p)
                    for (int q = 0; q < 3; ++q)
                        if (mi[p] || mj[q]) blk[p * 3 + q] = (J == i && p == q) ? 1.0 : 0.0;
            }
        }
        for (int o = 4; o > 0; o >>= 1)
            for (int p = 0; p < 3; ++p) lift[p] += __shfl_xor(lift[p], o, 64);
        if (i < n && l < 3) {
            const double bi = b[i * 3 + l] - (l == 0 ? lift[0] : l == 1 ? lift[1] : lift[2]);
            const bool m = l == 0 ? mi[0] : l == 1 ? mi[1] : mi[2];
            b[i * 3 + l] = m ? (ubc ? ubc[i * 3 + l] : 0.0) : bi;
        }
    }
}

// load-only variant: constrained entries set to zero (u_bc = 0, no lifting needed)
__global__ void k_zero_masked(int64_t n, int nrhs, double *__restrict__ b, const uint8_t *__restrict__ mask) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n * 3 * nrhs; t += (int64_t)gridDim.x * blockDim.x)
        if (mask[t / nrhs]) b[t] = 0.0;
}

// ---------------------------------------------------------------------------
// Temperature-dependent materials and boundary pressure
// ---------------------------------------------------------------------------
// Value of one table (n samples at temperatures Tt, ascending) at Tm: linear
// between samples, constant beyond the ends.
__device__ __forceinline__ double table_at(const double *Tt, const double *v, int n, double Tm) {
    if (n == 1 || Tm <= Tt[0]) return v[0];
    if (Tm >= Tt[n - 1]) return v[n - 1];
    int k = 0;
    while (k + 2 < n && Tm >= Tt[k + 1]) ++k;
    const double slope = (v[k + 1] - v[k]) / (Tt[k + 1] - Tt[k]);
    return slope * (Tm - Tt[k]) + v[k];
}

// Per cell: mean of T_h over the cell (P1: vertex average; P2: -1/20 of each
// vertex value plus 1/5 of each edge value, the exact cell integrals of the
// basis), the material's E, nu, alpha there, and (lam, mu, (3 lam + 2 mu) alpha).
// tab = [T | E | nu | alpha], each [nmat][npts].
template <int DEG>
__global__ void k_cell_coef(int64_t nc, const int32_t *__restrict__ cells, const double *__restrict__ T,
                            const int32_t *__restrict__ cmat, int nmat, int npts, const double *__restrict__ tab,
                            double *__restrict__ coef, int32_t *__restrict__ bad) {
    constexpr int NPE = DEG == 1 ? 4 : 10;
    for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < nc; c += (int64_t)gridDim.x * blockDim.x) {
        const int32_t *cv = cells + c * NPE;
        double Tm;
        if (DEG == 1) {
            Tm = 0.25 * (T[cv[0]] + T[cv[1]] + T[cv[2]] + T[cv[3]]);
        } else {
            double sv = 0.0, se = 0.0;
            for (int k = 0; k < 4; ++k) sv += T[cv[k]];
            for (int k = 4; k < 10; ++k) se += T[cv[k]];
            Tm = -0.05 * sv + 0.2 * se;
        }
        int m = cmat[c];
        if (m < 0 || m >= nmat) {
            *bad = 1;
            m = 0;
        }
        const int64_t so = (int64_t)nmat * npts, mo = (int64_t)m * npts;
        const double *Tt = tab + mo;
        const double E = table_at(Tt, tab + so + mo, npts, Tm);
        const double nu = table_at(Tt, tab + 2 * so + mo, npts, Tm);
        const double al = table_at(Tt, tab + 3 * so + mo, npts, Tm);
        const double lam = E * nu / ((1.0 + nu) * (1.0 - 2.0 * nu));
        const double mu = E / (2.0 * (1.0 + nu));
        coef[c * 3] = lam;
        coef[c * 3 + 1] = mu;
        coef[c * 3 + 2] = (3.0 * lam + 2.0 * mu) * al;
    }
}

// Pressure load, one thread per node: b_i += p_f |F| w_a n_f over the node's
// (face, local node) entries in face order (w_a = 1/3 for P1 nodes and P2
// edge nodes; P2 vertices have none).
__global__ void k_pressure(int64_t n, const int64_t *__restrict__ ptr, const int64_t *__restrict__ ent, int npf,
                           const int32_t *__restrict__ faces, const double *__restrict__ p,
                           const double *__restrict__ X, double *__restrict__ b) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        if (ptr[i] == ptr[i + 1]) continue;
        double acc[3] = {0.0, 0.0, 0.0};
        for (int64_t e = ptr[i]; e < ptr[i + 1]; ++e) {
            const int64_t f = ent[e] / npf;
            const int32_t *fv = faces + f * npf;
            double x0[3], d1[3], d2[3];
            for (int k = 0; k < 3; ++k) {
                x0[k] = X[(int64_t)fv[0] * 3 + k];
                d1[k] = X[(int64_t)fv[1] * 3 + k] - x0[k];
                d2[k] = X[(int64_t)fv[2] * 3 + k] - x0[k];
            }
            const double nv[3] = {d1[1] * d2[2] - d1[2] * d2[1], d1[2] * d2[0] - d1[0] * d2[2],
                                  d1[0] * d2[1] - d1[1] * d2[0]};
            // p |F| / 3 * n = p * |nv| / 2 / 3 * nv / |nv| = p nv / 6
            const double s = p[f] / 6.0;
            for (int k = 0; k < 3; ++k) acc[k] += s * nv[k];
        }
        for (int k = 0; k < 3; ++k) b[i * 3 + k] += acc[k];
    }
}

// ---------------------------------------------------------------------------
// heat equation (eq. wf_thermal): residual and Newton Jacobian
// ---------------------------------------------------------------------------
// F_i = sum over cells of kappa_c (K_c T)_i + rho c_c / dt (M_c (T - T_old))_i
//     + sum over heat-transfer faces of h_f ((M_f T)_i - T_bc,f int_f phi_i),
// kappa_c and c_c the cell's material tables at the cell mean Tbar_c of T_h
// (weights w: P1 1/4; P2 -1/20 vertices, 1/5 edges); J = dF/dT adds the
// rank-one terms kappa'(Tbar) (K_c T) w^T and rho c'(Tbar)/dt (M_c dT) w^T.
struct ThArgs {
    const double *X;
    const int32_t *cells;
    int64_t n;
    const int64_t *start, *inc;
    const int32_t *cmat;
    const double *tab;  // [3][nm][np]
    int nm, np;
    const double *rho;
    const int64_t *fptr, *fent;
    const int32_t *faces;
    const double *h, *Tbc;
    const double *T, *Told;
    double inv_dt;      // 0: steady
    const int64_t *ptr;
    const int32_t *col;
    double *J, *F;
};

// piecewise-linear table, constant beyond its ends: value at x and the slope
// of the segment [T_k, T_k+1) holding x (0 outside)
__device__ __forceinline__ void table_eval(const double *Tt, const double *v, int np, double x, double &val,
                                           double &slope) {
    int k = -1;
    for (int j = 0; j < np; ++j)
        if (Tt[j] <= x) k = j;
    if (k < 0) {
        val = v[0];
        slope = 0.0;
    } else if (k >= np - 1) {
        val = v[np - 1];
        slope = 0.0;
    } else {
        slope = (v[k + 1] - v[k]) / (Tt[k + 1] - Tt[k]);
        val = slope * (x - Tt[k]) + v[k];
    }
}

__device__ __forceinline__ int64_t row_pos(const int32_t *__restrict__ col, int64_t r0, int64_t r1, int32_t c) {
    int64_t lo = r0, hi = r1;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (col[mid] < c) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// P2 triangle mass matrix times 180/|F| (vertices, then edges 01, 02, 12)
__device__ __forceinline__ double p2_face_mass180(int a, int b) {
    if (a < 3 && b < 3) return a == b ? 6.0 : -1.0;
    if (a >= 3 && b >= 3) return a == b ? 32.0 : 16.0;
    const int v = a < 3 ? a : b, e = a < 3 ? b : a;
    // edge 3 = (0,1), 4 = (0,2), 5 = (1,2): the vertex opposite is 2, 1, 0
    return (5 - e) == v ? -4.0 : 0.0;
}

template <int DEG>
__global__ void __launch_bounds__(ABLK) k_thermal(ThArgs A) {
    const int64_t i = (int64_t)blockIdx.x * ABLK + threadIdx.x;
    if (i >= A.n) return;
    constexpr int NPE = DEG == 1 ? 4 : 10;
    constexpr int NPF = DEG == 1 ? 3 : 6;
    __shared__ double s_g[ABLK][12];
    double *G = s_g[threadIdx.x];
    const int64_t r0 = A.ptr[i], r1 = A.ptr[i + 1];
    for (int64_t k = r0; k < r1; ++k) A.J[k] = 0.0;
    double Fi = 0.0;
    for (int64_t e = A.start[i]; e < A.start[i + 1]; ++e) {
        const int64_t cell = A.inc[e] / NPE;
        const int a = (int)(A.inc[e] % NPE);
        const int32_t *cv = A.cells + cell * NPE;
        const Geo g = cell_geo(A.X, cv);
        for (int k = 0; k < 4; ++k)
            for (int c = 0; c < 3; ++c) G[k * 3 + c] = g.G[k][c];
        double Tc[NPE], w[NPE];
        double Tbar = 0.0;
        for (int c = 0; c < NPE; ++c) {
            Tc[c] = A.T[cv[c]];
            w[c] = DEG == 1 ? 0.25 : (c < 4 ? -0.05 : 0.2);
            Tbar += w[c] * Tc[c];
        }
        const int m = A.cmat[cell];
        double kap, dkap, cvv = 0.0, dcv = 0.0;
        table_eval(A.tab + (int64_t)m * A.np, A.tab + (int64_t)(A.nm + m) * A.np, A.np, Tbar, kap, dkap);
        if (A.inv_dt > 0.0)
            table_eval(A.tab + (int64_t)m * A.np, A.tab + (int64_t)(2 * A.nm + m) * A.np, A.np, Tbar, cvv, dcv);
        // row a of the reference stiffness int grad phi_a . grad phi_b and mass
        double Kab[NPE], Mab[NPE];
        if (DEG == 1) {
            for (int b = 0; b < NPE; ++b) {
                Kab[b] = g.vol * (G[a * 3] * G[b * 3] + G[a * 3 + 1] * G[b * 3 + 1] + G[a * 3 + 2] * G[b * 3 + 2]);
                Mab[b] = g.vol * (a == b ? 2.0 : 1.0) / 20.0;
            }
        } else {
            for (int b = 0; b < NPE; ++b) Kab[b] = 0.0;
            const double qa = 0.5854101966249685, qb = 0.1381966011250105;
            for (int q = 0; q < 4; ++q) {
                const double l0 = q == 0 ? qa : qb, l1 = q == 1 ? qa : qb, l2 = q == 2 ? qa : qb,
                             l3 = q == 3 ? qa : qb;
                double ga[3];
                p2_grad(a, l0, l1, l2, l3, G, ga);
                for (int b = 0; b < NPE; ++b) {
                    double gb[3];
                    p2_grad(b, l0, l1, l2, l3, G, gb);
                    Kab[b] += 0.25 * g.vol * (ga[0] * gb[0] + ga[1] * gb[1] + ga[2] * gb[2]);
                }
            }
            for (int b = 0; b < NPE; ++b) Mab[b] = g.vol * p2_mass420(a, b) / 420.0;
        }
        double KT = 0.0, MdT = 0.0;
        for (int b = 0; b < NPE; ++b) KT += Kab[b] * Tc[b];
        Fi += kap * KT;
        const double rc = A.inv_dt > 0.0 ? A.rho[m] * A.inv_dt : 0.0;
        if (A.inv_dt > 0.0) {
            for (int b = 0; b < NPE; ++b) MdT += Mab[b] * (Tc[b] - A.Told[cv[b]]);
            Fi += rc * cvv * MdT;
        }
        for (int b = 0; b < NPE; ++b) {
            double v = kap * Kab[b] + dkap * w[b] * KT;
            if (A.inv_dt > 0.0) v += rc * (cvv * Mab[b] + dcv * w[b] * MdT);
            A.J[row_pos(A.col, r0, r1, cv[b])] += v;
        }
    }
    if (A.fptr) {
        for (int64_t e = A.fptr[i]; e < A.fptr[i + 1]; ++e) {
            const int64_t f = A.fent[e] / NPF;
            const int a = (int)(A.fent[e] % NPF);
            const int32_t *fv = A.faces + f * NPF;
            double d1[3], d2[3];
            for (int k = 0; k < 3; ++k) {
                const double x0 = A.X[(int64_t)fv[0] * 3 + k];
                d1[k] = A.X[(int64_t)fv[1] * 3 + k] - x0;
                d2[k] = A.X[(int64_t)fv[2] * 3 + k] - x0;
            }
            const double nx = d1[1] * d2[2] - d1[2] * d2[1], ny = d1[2] * d2[0] - d1[0] * d2[2],
                         nz = d1[0] * d2[1] - d1[1] * d2[0];
            const double area = 0.5 * sqrt(nx * nx + ny * ny + nz * nz);
            const double hf = A.h[f];
            double MT = 0.0;
            for (int b = 0; b < NPF; ++b) {
                const double mf = DEG == 1 ? area * (a == b ? 2.0 : 1.0) / 12.0 : area * p2_face_mass180(a, b) / 180.0;
                MT += mf * A.T[fv[b]];
                A.J[row_pos(A.col, r0, r1, fv[b])] += hf * mf;
            }
            const double fint = DEG == 1 ? area / 3.0 : (a < 3 ? 0.0 : area / 3.0);
            Fi += hf * (MT - A.Tbc[f] * fint);
        }
    }
    A.F[i] = Fi;
}

static void pattern_impl(const te_mesh *m, Incidence &I, int64_t *row_ptr, int32_t *col, hipStream_t s);

void thermal_asm_init(ThermalAsm &ta, const te_mesh *m, const te_thermal_tables *tab, const int32_t *cell_material,
                      const te_robin *robin, hipStream_t s) {
    TE_REQUIRE(m && tab && cell_material, TE_EINVAL, "NULL argument");
    TE_REQUIRE(m->degree == 1 || m->degree == 2, TE_EINVAL, "degree must be 1 or 2 (got %d)", m->degree);
    TE_REQUIRE(m->n_nodes > 0 && m->n_cells > 0 && m->coords && m->cells, TE_EINVAL, "empty mesh");
    TE_REQUIRE(m->n_nodes < (int64_t)INT32_MAX, TE_EINVAL, "too many nodes for 32-bit indices");
    const int nm = tab->n_materials, np = tab->n_points;
    TE_REQUIRE(nm >= 1 && np >= 1 && tab->T && tab->kappa && tab->cv && tab->rho, TE_EINVAL,
               "thermal tables are empty or NULL");
    std::vector<double> h((size_t)3 * nm * np);
    const size_t so = (size_t)nm * np;
    for (int mm = 0; mm < nm; ++mm) {
        TE_REQUIRE(tab->rho[mm] > 0.0, TE_EINVAL, "material %d: density must be positive", mm);
        for (int k = 0; k < np; ++k) {
            const size_t q = (size_t)mm * np + k;
            TE_REQUIRE(k == 0 || tab->T[q] > tab->T[q - 1], TE_EINVAL, "material %d: temperatures not ascending", mm);
            TE_REQUIRE(tab->kappa[q] > 0.0 && tab->cv[q] > 0.0, TE_EINVAL,
                       "material %d: conductivity and specific heat must be positive", mm);
            h[q] = tab->T[q];
            h[so + q] = tab->kappa[q];
            h[2 * so + q] = tab->cv[q];
        }
    }
    ta.n = m->n_nodes;
    ta.nc = m->n_cells;
    ta.degree = m->degree;
    ta.npe = m->degree == 1 ? 4 : 10;
    ta.npf = m->degree == 1 ? 3 : 6;
    ta.nm = nm;
    ta.np = np;
    upload(ta.tab, h, s);
    upload(ta.rho, std::vector<double>(tab->rho, tab->rho + nm), s);
    ta.coords.alloc(ta.n * 3);
    ta.cells.alloc(ta.nc * ta.npe);
    ta.cell_material.alloc(ta.nc);
    TE_CHECK_HIP(hipMemcpyAsync(ta.coords.p, m->coords, ta.n * 3 * sizeof(double), hipMemcpyDeviceToDevice, s));
    TE_CHECK_HIP(hipMemcpyAsync(ta.cells.p, m->cells, ta.nc * ta.npe * sizeof(int32_t), hipMemcpyDeviceToDevice, s));
    TE_CHECK_HIP(hipMemcpyAsync(ta.cell_material.p, cell_material, ta.nc * sizeof(int32_t), hipMemcpyDeviceToDevice, s));
    te_mesh mc{ta.n, ta.nc, ta.degree, ta.coords.p, ta.cells.p};
    build_incidence(&mc, ta.npe, ta.I, s);  // rejects node ids outside the mesh
    {
        std::vector<int32_t> cm;
        download(cm, ta.cell_material.p, (size_t)ta.nc, s);
        for (int32_t v : cm) TE_REQUIRE(v >= 0 && v < nm, TE_EINVAL, "a cell material id is outside 0..%d", nm - 1);
    }
    ta.n_faces = robin ? robin->n_faces : 0;
    TE_REQUIRE(ta.n_faces >= 0, TE_EINVAL, "negative face count");
    if (ta.n_faces > 0) {
        TE_REQUIRE(robin->faces && robin->h && robin->T_bc, TE_EINVAL, "heat-transfer face arrays are NULL");
        const int npf = ta.npf;
        std::vector<int32_t> fh;
        download(fh, robin->faces, (size_t)ta.n_faces * npf, s);
        std::vector<double> hh, tb;
        download(hh, robin->h, (size_t)ta.n_faces, s);
        download(tb, robin->T_bc, (size_t)ta.n_faces, s);
        for (double v : hh) TE_REQUIRE(v >= 0.0, TE_EINVAL, "heat-transfer coefficients must be >= 0");
        std::vector<int64_t> cnt(ta.n + 1, 0);
        for (int64_t q = 0; q < (int64_t)fh.size(); ++q) {
            TE_REQUIRE(fh[q] >= 0 && fh[q] < ta.n, TE_EINVAL, "face %lld has a node outside the mesh",
                       (long long)(q / npf));
            ++cnt[fh[q] + 1];
        }
        for (int64_t i = 0; i < ta.n; ++i) cnt[i + 1] += cnt[i];
        std::vector<int64_t> ent(cnt[ta.n]), fill(cnt.begin(), cnt.end() - 1);
        for (int64_t q = 0; q < (int64_t)fh.size(); ++q) ent[fill[fh[q]]++] = q;
        upload(ta.fptr, cnt, s);
        upload(ta.fent, ent, s);
        upload(ta.faces, fh, s);
        upload(ta.h, hh, s);
        upload(ta.T_bc, tb, s);
    }
    ta.ptr.alloc(ta.n + 1);
    pattern_impl(&mc, ta.I, ta.ptr.p, nullptr, s);
    TE_CHECK_HIP(hipMemcpyAsync(&ta.nnz, ta.ptr.p + ta.n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    TE_CHECK_HIP(hipStreamSynchronize(s));
    ta.col.alloc(std::max<int64_t>(ta.nnz, 1));
    pattern_impl(&mc, ta.I, ta.ptr.p, ta.col.p, s);
}

void thermal_asm_run(const ThermalAsm &ta, const double *T, const double *T_old, double dt, double *Jval, double *F,
                     hipStream_t s) {
    const bool transient = T_old != nullptr && dt > 0.0;
    ThArgs a{ta.coords.p, ta.cells.p, ta.n, ta.I.start.p, ta.I.inc.p, ta.cell_material.p, ta.tab.p, ta.nm, ta.np,
             ta.rho.p, ta.n_faces > 0 ? ta.fptr.p : nullptr, ta.fent.p, ta.faces.p, ta.h.p, ta.T_bc.p, T,
             transient ? T_old : nullptr, transient ? 1.0 / dt : 0.0, ta.ptr.p, ta.col.p, Jval, F};
    const unsigned g = (unsigned)((ta.n + ABLK - 1) / ABLK);
    if (ta.degree == 1) hipLaunchKernelGGL(k_thermal<1>, dim3(g), dim3(ABLK), 0, s, a);
    else hipLaunchKernelGGL(k_thermal<2>, dim3(g), dim3(ABLK), 0, s, a);
    TE_CHECK_HIP(hipGetLastError());
}

static void check_mesh(const te_mesh *m) {
    TE_REQUIRE(m, TE_EINVAL, "mesh is NULL");
    TE_REQUIRE(m->degree == 1 || m->degree == 2, TE_EINVAL, "degree must be 1 or 2 (got %d)", m->degree);
    TE_REQUIRE(m->n_nodes > 0 && m->n_cells > 0, TE_EINVAL, "empty mesh");
    TE_REQUIRE(m->n_nodes < (int64_t)INT32_MAX, TE_EINVAL, "too many nodes for 32-bit indices");
    TE_REQUIRE(m->coords && m->cells, TE_EINVAL, "mesh arrays are NULL");
}

static void pattern_impl(const te_mesh *m, Incidence &I, int64_t *row_ptr, int32_t *col, hipStream_t s) {
    const int npe = m->degree == 1 ? 4 : 10;
    const int64_t n = m->n_nodes;
    DBuf<int32_t> ovf(1), cnt;
    DBuf<int64_t> bs;
    TE_CHECK_HIP(hipMemsetAsync(ovf.p, 0, sizeof(int32_t), s));
    if (!col) cnt.alloc(n);
    hipLaunchKernelGGL(k_pattern, dim3((unsigned)std::min<int64_t>(n, 1 << 18)), dim3(64), 0, s, m->cells, npe,
                       I.start.p, I.inc.p, n, cnt.p, row_ptr, col, ovf.p);
    TE_CHECK_HIP(hipGetLastError());
    int32_t h = 0;
    TE_CHECK_HIP(hipMemcpyAsync(&h, ovf.p, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    TE_CHECK_HIP(hipStreamSynchronize(s));
    TE_REQUIRE(h == 0, TE_EINVAL, h == 1 ? "a node couples to more than 192 nodes"
                                         : "row_ptr does not match this mesh's sparsity pattern");
    if (!col) {
        scan_counts(cnt.p, row_ptr, n, bs, s);
        TE_CHECK_HIP(hipStreamSynchronize(s));
    }
}

}  // namespace te

using namespace te;

extern "C" int fe_assemble_pattern(const te_mesh *mesh, int64_t *row_ptr, int64_t *nnzb_out, hipStream_t stream) {
    return guarded([&]() -> int {
        check_mesh(mesh);
        TE_REQUIRE(row_ptr && nnzb_out, TE_EINVAL, "row_ptr / nnzb_out is NULL");
        Incidence I;
        build_incidence(mesh, mesh->degree == 1 ? 4 : 10, I, stream, false);
        pattern_impl(mesh, I, row_ptr, nullptr, stream);
        TE_CHECK_HIP(hipMemcpyAsync(nnzb_out, row_ptr + mesh->n_nodes, sizeof(int64_t), hipMemcpyDeviceToHost, stream));
        TE_CHECK_HIP(hipStreamSynchronize(stream));
        return TE_OK;
    });
}

static void material_consts(const te_material *mat, double &lam, double &mu, double &calpha) {
    TE_REQUIRE(mat, TE_EINVAL, "material is NULL");
    TE_REQUIRE(mat->E > 0 && mat->nu > -1.0 && mat->nu < 0.5, TE_EINVAL, "invalid E / nu");
    lam = mat->E * mat->nu / ((1.0 + mat->nu) * (1.0 - 2.0 * mat->nu));
    mu = mat->E / (2.0 * (1.0 + mat->nu));
    calpha = (3.0 * lam + 2.0 * mu) * mat->alpha;
}

extern "C" int fe_assemble_thermoelastic(const te_mesh *mesh, const te_material *mat, const double *T,
                                         const double *f, const uint8_t *dir_mask, const double *u_bc, te_bsr *A,
                                         double *b, hipStream_t stream) {
    return guarded([&]() -> int {
        check_mesh(mesh);
        TE_REQUIRE(T && b && A && A->row_ptr && A->col_idx && A->val, TE_EINVAL, "NULL array argument");
        TE_REQUIRE(A->n_brows == mesh->n_nodes, TE_EINVAL, "A.n_brows != n_nodes");
        double lam, mu, calpha;
        material_consts(mat, lam, mu, calpha);
        const int npe = mesh->degree == 1 ? 4 : 10;
        Incidence I;
        build_incidence(mesh, npe, I, stream);
        int64_t nnzb = 0;
        TE_CHECK_HIP(hipMemcpyAsync(&nnzb, A->row_ptr + mesh->n_nodes, sizeof(int64_t), hipMemcpyDeviceToHost, stream));
        TE_CHECK_HIP(hipStreamSynchronize(stream));
        TE_REQUIRE(nnzb == A->nnzb, TE_EINVAL, "A.nnzb (%lld) != row_ptr[N] (%lld)", (long long)A->nnzb,
                   (long long)nnzb);
        AsmArgs a{mesh->coords, mesh->cells, npe, I.start.p, I.inc.p, mesh->n_nodes, lam, mu, calpha, mat->T_ref,
                  nullptr, T, f, A->row_ptr, A->col_idx, A->val, b, 1};
        stiffness_rows(a, mesh->degree, nnzb, stream);
        launch_load(a, mesh->degree, stream);
        if (dir_mask) {
            unsigned gd = (unsigned)std::min<int64_t>((mesh->n_nodes + 31) / 32, 1 << 20);
            hipLaunchKernelGGL(k_dirichlet, dim3(gd), dim3(256), 0, stream, mesh->n_nodes, A->row_ptr, A->col_idx,
                               A->val, b, dir_mask, u_bc);
            TE_CHECK_HIP(hipGetLastError());
        }
        TE_CHECK_HIP(hipStreamSynchronize(stream));
        return TE_OK;
    });
}

extern "C" int fe_assemble_load(const te_mesh *mesh, const te_material *mat, const double *T, const double *f,
                                const uint8_t *dir_mask, int32_t nrhs, double *b, hipStream_t stream) {
    return guarded([&]() -> int {
        check_mesh(mesh);
        TE_REQUIRE(T && b, TE_EINVAL, "NULL array argument");
        TE_REQUIRE(nrhs >= 1 && nrhs <= 64, TE_EINVAL, "nrhs must be in 1..64");
        double lam, mu, calpha;
        material_consts(mat, lam, mu, calpha);
        const int npe = mesh->degree == 1 ? 4 : 10;
        Incidence I;
        build_incidence(mesh, npe, I, stream);
        AsmArgs a{mesh->coords, mesh->cells, npe, I.start.p, I.inc.p, mesh->n_nodes, lam, mu, calpha, mat->T_ref,
                  nullptr, T, f, nullptr, nullptr, nullptr, b, nrhs};
        launch_load(a, mesh->degree, stream);
        if (dir_mask) {
            unsigned gd = (unsigned)std::min<int64_t>((mesh->n_nodes * 3 * nrhs + 255) / 256, 1 << 20);
            hipLaunchKernelGGL(k_zero_masked, dim3(gd), dim3(256), 0, stream, mesh->n_nodes, nrhs, b, dir_mask);
            TE_CHECK_HIP(hipGetLastError());
        }
        TE_CHECK_HIP(hipStreamSynchronize(stream));
        return TE_OK;
    });
}

extern "C" int fe_assemble_thermoelastic_materials(const te_mesh *mesh, const te_material_tables *mat,
                                                   const int32_t *cell_material, const double *T, const double *f,
                                                   const te_pressure *pressure, const uint8_t *dir_mask,
                                                   const double *u_bc, te_bsr *A, double *b, hipStream_t stream) {
    return guarded([&]() -> int {
        check_mesh(mesh);
        TE_REQUIRE(mat && cell_material && T && b && A && A->row_ptr && A->col_idx && A->val, TE_EINVAL,
                   "NULL argument");
        TE_REQUIRE(A->n_brows == mesh->n_nodes, TE_EINVAL, "A.n_brows != n_nodes");
        const int nm = mat->n_materials, np = mat->n_points;
        TE_REQUIRE(nm >= 1 && np >= 1 && mat->T && mat->E && mat->nu && mat->alpha, TE_EINVAL,
                   "material tables are empty or NULL");
        std::vector<double> tab((size_t)4 * nm * np);
        for (int m = 0; m < nm; ++m)
            for (int k = 0; k < np; ++k) {
                const size_t q = (size_t)m * np + k, so = (size_t)nm * np;
                const double Tk = mat->T[q], E = mat->E[q], nu = mat->nu[q];
                TE_REQUIRE(k == 0 || Tk > mat->T[q - 1], TE_EINVAL, "material %d: temperatures not ascending", m);
                TE_REQUIRE(E > 0 && nu > -1.0 && nu < 0.5, TE_EINVAL, "material %d: invalid E / nu at sample %d", m, k);
                tab[q] = Tk;
                tab[so + q] = E;
                tab[2 * so + q] = nu;
                tab[3 * so + q] = mat->alpha[q];
            }
        const int npe = mesh->degree == 1 ? 4 : 10;
        const int64_t nc = mesh->n_cells, n = mesh->n_nodes;
        // node -> cell incidence first: it rejects node ids outside the mesh
        // before any kernel reads through them
        Incidence I;
        build_incidence(mesh, npe, I, stream);
        DBuf<double> dtab, coef(nc * 3);
        upload(dtab, tab, stream);
        DBuf<int32_t> bad(1);
        TE_CHECK_HIP(hipMemsetAsync(bad.p, 0, sizeof(int32_t), stream));
        const unsigned gc = (unsigned)std::min<int64_t>((nc + 255) / 256, 1 << 20);
        if (mesh->degree == 1)
            hipLaunchKernelGGL(k_cell_coef<1>, dim3(gc), dim3(256), 0, stream, nc, mesh->cells, T, cell_material, nm,
                               np, dtab.p, coef.p, bad.p);
        else
            hipLaunchKernelGGL(k_cell_coef<2>, dim3(gc), dim3(256), 0, stream, nc, mesh->cells, T, cell_material, nm,
                               np, dtab.p, coef.p, bad.p);
        TE_CHECK_HIP(hipGetLastError());
        int32_t hb = 0;
        TE_CHECK_HIP(hipMemcpyAsync(&hb, bad.p, sizeof(int32_t), hipMemcpyDeviceToHost, stream));
        int64_t nnzb = 0;
        TE_CHECK_HIP(hipMemcpyAsync(&nnzb, A->row_ptr + n, sizeof(int64_t), hipMemcpyDeviceToHost, stream));
        TE_CHECK_HIP(hipStreamSynchronize(stream));
        TE_REQUIRE(hb == 0, TE_EINVAL, "a cell material id is outside 0..%d", nm - 1);
        TE_REQUIRE(nnzb == A->nnzb, TE_EINVAL, "A.nnzb (%lld) != row_ptr[N] (%lld)", (long long)A->nnzb,
                   (long long)nnzb);
        // node -> (face, local node) entries of the pressure faces, in face order
        const bool has_p = pressure && pressure->n_faces > 0;
        Incidence PF;
        DBuf<int32_t> fcnt;
        DBuf<int64_t> fbs;
        const int npf = mesh->degree == 1 ? 3 : 6;
        if (has_p) {
            TE_REQUIRE(pressure->faces && pressure->p, TE_EINVAL, "pressure faces / values are NULL");
            const int64_t q = first_bad_node(pressure->faces, pressure->n_faces * npf, n, stream);
            TE_REQUIRE(q < 0, TE_EINVAL, "pressure face %lld has a node outside the mesh", (long long)(q / npf));
            // P2 vertices carry no pressure load
            entry_lists(pressure->faces, pressure->n_faces, npf, mesh->degree == 1 ? 0 : 3, n, true, PF, fcnt, fbs,
                        stream);
        }
        AsmArgs a{mesh->coords, mesh->cells, npe, I.start.p, I.inc.p, n, 0.0, 0.0, 0.0, mat->T_ref,
                  coef.p, T, f, A->row_ptr, A->col_idx, A->val, b, 1};
        stiffness_rows(a, mesh->degree, nnzb, stream);
        launch_load(a, mesh->degree, stream);
        if (has_p) {
            const unsigned gp = (unsigned)std::min<int64_t>((n + 255) / 256, 1 << 20);
            hipLaunchKernelGGL(k_pressure, dim3(gp), dim3(256), 0, stream, n, PF.start.p, PF.inc.p, npf,
                               pressure->faces, pressure->p, mesh->coords, b);
            TE_CHECK_HIP(hipGetLastError());
        }
        if (dir_mask) {
            const unsigned gd = (unsigned)std::min<int64_t>((n + 31) / 32, 1 << 20);
            hipLaunchKernelGGL(k_dirichlet, dim3(gd), dim3(256), 0, stream, n, A->row_ptr, A->col_idx, A->val, b,
                               dir_mask, u_bc);
            TE_CHECK_HIP(hipGetLastError());
        }
        TE_CHECK_HIP(hipStreamSynchronize(stream));
        return TE_OK;
    });
}
