// Kernels of block conjugate gradients over the columns of a multi-RHS solve
// (O'Leary 1980; the driver is in te_solve.cpp).  Block vectors are the
// solve's [rows][m] arrays (right-hand sides fastest, m <= 64); small matrices
// are 64 x 64 row-major with zero padding.
//
// The three kernels are tall-skinny dense contractions on the float64 matrix
// cores (v_mfma_f64_16x16x4; lane l of A: row l % 16, inner index l / 16; of B:
// column l % 16, inner index l / 16; register r of D: row 4 r + l / 16, column
// l % 16).  Their rate is that of the vector units, but a block row is read by
// the lanes that need it only, without passing through LDS, and the tiles of 16
// columns follow the block size: T = ceil(m / 16) of them, not 64 columns.
//
//   k_gram      C_t = L_t^T R_t for up to three pairs of block vectors in one
//               pass over the rows: one wave per pair and row range, both
//               operands straight from memory (four rows of 16 columns).  One
//               partial per workgroup, summed in workgroup order (k_gram_sum1/2:
//               deterministic).
//   k_block_xr  X += P alpha, R -= Q alpha, plus per-column partial sums of
//               R^2.  A wave takes 16 block rows; alpha from LDS.
//   k_block_p   P <- Z T1 + P T2 in place, organised as k_block_xr (a wave
//               reads its 16 rows of Z and P whole before it writes them).
//
// 24 columns, 287,000 rows (vectors of 55 MB), with vector FMAs on tiles of 64
// columns before: k_gram 377 -> 51 us, k_block_xr 199 -> 67 us, k_block_p 107 ->
// 37 us; 64 columns, 1,003,104 rows: 1.37 -> 0.72, 1.37 -> 0.85 and 0.93 -> 0.59
// ms, the last two within 1.4 of their traffic at the rate of a copy.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "te_dev.h"

namespace te {
namespace {

constexpr int GM = 64;      // largest block size
constexpr int GBLKS = 1024; // most workgroups of the Gram pass
constexpr int GSPLIT = 16;  // first-stage slices of the Gram partial sum
constexpr int UBLK = 256;   // threads of the update kernels (4 waves)
constexpr int TRW = 16;     // block rows per wave in the updates

using f64x4 = __attribute__((__vector_size__(4 * sizeof(double)))) double;

struct GramArgs {
    const double *mat[3];   // distinct block vectors [rows][m]
    int li[3], ri[3];       // pair t: mat[li[t]]^T mat[ri[t]]
    int npair;
    int64_t rows;
    int m;
    double *partials;       // [gridDim.x][npair][16 T][16 T]
};

// Row ranges of a workgroup, each with one wave per pair: four where the
// accumulators are few, to have the loads of as many waves in flight.
constexpr int gram_split(int T) { return T <= 2 ? 4 : 1; }

// blockDim = 64 * npair * gram_split(T)
template <int T>
__global__ void __launch_bounds__(192 * gram_split(T)) k_gram(GramArgs g) {
    constexpr int S = gram_split(T), U = 4, C = 16 * T;
    __shared__ double s_acc[S > 1 ? 3 * C * C : 1];
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE, p = w / S, part = w - p * S;
    const int m = g.m, c = lane & 15, k = lane >> 4;
    const double *__restrict__ L = g.mat[g.li[p]], *__restrict__ R = g.mat[g.ri[p]];
    f64x4 acc[T][T] = {};
    const int64_t chunk = (g.rows + (int64_t)gridDim.x * S - 1) / ((int64_t)gridDim.x * S);
    const int64_t lo = ((int64_t)blockIdx.x * S + part) * chunk, hi = min(g.rows, lo + chunk);
    for (int64_t r0 = lo; r0 < hi; r0 += 4 * U) {
        double l[U][T], r[U][T];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t row = r0 + 4 * u + k;
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const bool ok = row < hi && 16 * t + c < m;
                l[u][t] = ok ? L[row * m + 16 * t + c] : 0.0;
                r[u][t] = ok ? R[row * m + 16 * t + c] : 0.0;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int a = 0; a < T; ++a)
#pragma unroll
                for (int b = 0; b < T; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(l[u][a], r[u][b], acc[a][b], 0, 0, 0);
    }
    // the ranges of the workgroup in order
    auto at = [&](int a, int b, int q) { return (16 * a + 4 * q + k) * C + 16 * b + c; };
    if constexpr (S > 1) {
        double *mine = s_acc + p * C * C;
        for (int v = 0; v < S; ++v) {
            if (part == v)
#pragma unroll
                for (int a = 0; a < T; ++a)
#pragma unroll
                    for (int b = 0; b < T; ++b)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            if (v > 0) acc[a][b][q] += mine[at(a, b, q)];
                            if (v < S - 1) mine[at(a, b, q)] = acc[a][b][q];
                        }
            __syncthreads();
        }
    }
    if (part == S - 1) {
        double *out = g.partials + ((int64_t)blockIdx.x * g.npair + p) * C * C;
#pragma unroll
        for (int a = 0; a < T; ++a)
#pragma unroll
            for (int b = 0; b < T; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q) out[at(a, b, q)] = acc[a][b][q];
    }
}

// Partial sums over the workgroups in a fixed order: slice y of them into
// out2[y], then the GSPLIT slices in order, into 64 x 64 matrices.
__global__ void __launch_bounds__(256) k_gram_sum1(const double *__restrict__ partials, int nb, int64_t n,
                                                   double *__restrict__ out2) {
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (e >= n) return;
    const int per = (nb + GSPLIT - 1) / GSPLIT, b1 = min(nb, (int)(blockIdx.y + 1) * per);
    double s = 0.0;
#pragma unroll 8
    for (int b = blockIdx.y * per; b < b1; ++b) s += partials[(int64_t)b * n + e];
    out2[(int64_t)blockIdx.y * n + e] = s;
}
// C = 16 T columns of a partial; n = npair * C * C
__global__ void __launch_bounds__(256) k_gram_sum2(const double *__restrict__ out2, int C, int64_t n,
                                                   double *__restrict__ out) {
    const int p = blockIdx.y, e = blockIdx.x * blockDim.x + threadIdx.x, a = e / GM, b = e % GM;
    double s = 0.0;
    if (a < C && b < C)
#pragma unroll
        for (int y = 0; y < GSPLIT; ++y) s += out2[(int64_t)y * n + ((int64_t)p * C + a) * C + b];
    out[(int64_t)p * GM * GM + e] = s;
}

// A small matrix in LDS: rows of LD doubles, the 16-column halves of each 32
// swapped in odd rows, so that the four rows a wave reads meet every bank twice.
template <int T>
struct SmallMat {
    static constexpr int LD = T <= 2 ? 32 : 64;
    double v[16 * T][LD];
    __device__ __forceinline__ double &at(int k, int c) { return v[k][c ^ ((k & 1) << 4)]; }
    __device__ __forceinline__ void load(const double *__restrict__ src) {
        for (int e = threadIdx.x; e < 16 * T * LD; e += blockDim.x)
            if (e % LD < 16 * T || T == 1) at(e / LD, e % LD) = src[(e / LD) * GM + e % LD];
    }
};
// row `row` of a block vector as A operand: inner indices 4 s + l / 16
template <int T>
__device__ __forceinline__ void load_rows(const double *A, int64_t row, int64_t rows, int m, double (&a)[4 * T]) {
    const int k = (threadIdx.x & (WAVE - 1)) >> 4;
#pragma unroll
    for (int s = 0; s < 4 * T; ++s) a[s] = row < rows && 4 * s + k < m ? A[row * m + 4 * s + k] : 0.0;
}
// acc += (16 rows) * C
template <int T>
__device__ __forceinline__ void times(const double (&a)[4 * T], int m, SmallMat<T> &C, f64x4 (&acc)[T]) {
    const int c = threadIdx.x & 15, k = (threadIdx.x & (WAVE - 1)) >> 4;
#pragma unroll
    for (int s = 0; s < 4 * T; ++s)
        if (4 * s < m)   // uniform
#pragma unroll
            for (int t = 0; t < T; ++t)
                acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], C.at(4 * s + k, 16 * t + c), acc[t], 0, 0, 0);
}

// X += P alpha, R -= Q alpha; a wave takes TRW rows.
template <int T>
__global__ void __launch_bounds__(UBLK) k_block_xr(int64_t rows, int m, const double *__restrict__ alpha,
                                                   const double *__restrict__ P, const double *__restrict__ Q,
                                                   double *__restrict__ X, double *__restrict__ R,
                                                   double *__restrict__ partials) {
    __shared__ SmallMat<T> s_a;
    __shared__ double s_col[UBLK / WAVE][4][16 * T];
    s_a.load(alpha);
    __syncthreads();
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE, c = lane & 15, k = lane >> 4;
    double rr[T];
#pragma unroll
    for (int t = 0; t < T; ++t) rr[t] = 0.0;
    const int64_t step = (int64_t)gridDim.x * (UBLK / WAVE) * TRW;
    for (int64_t row0 = ((int64_t)blockIdx.x * (UBLK / WAVE) + w) * TRW; row0 < rows; row0 += step) {
        double p[4 * T], q[4 * T];
        load_rows<T>(P, row0 + c, rows, m, p);
        load_rows<T>(Q, row0 + c, rows, m, q);
        f64x4 ap[T] = {}, aq[T] = {};
        times<T>(p, m, s_a, ap);
        times<T>(q, m, s_a, aq);
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t row = row0 + 4 * u + k, e = row * m + 16 * t + c;
                if (row < rows && 16 * t + c < m) {
                    X[e] += ap[t][u];
                    const double r = R[e] - aq[t][u];
                    R[e] = r;
                    rr[t] += r * r;
                }
            }
    }
    // per-column partial of this workgroup: (wave, row group) in order
#pragma unroll
    for (int t = 0; t < T; ++t) s_col[w][k][16 * t + c] = rr[t];
    __syncthreads();
    if ((int)threadIdx.x < m) {
        double tot = 0.0;
        for (int v = 0; v < UBLK / WAVE; ++v)
            for (int gq = 0; gq < 4; ++gq) tot += s_col[v][gq][threadIdx.x];
        partials[(int64_t)blockIdx.x * m + threadIdx.x] = tot;
    }
}

// P <- Z T1 + P T2 in place; rows as in k_block_xr.
template <int T>
__global__ void __launch_bounds__(UBLK) k_block_p(int64_t rows, int m, const double *__restrict__ T1,
                                                  const double *__restrict__ T2, const double *__restrict__ Z,
                                                  double *P) {
    __shared__ SmallMat<T> s_1, s_2;
    s_1.load(T1);
    s_2.load(T2);
    __syncthreads();
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE, c = lane & 15, k = lane >> 4;
    const int64_t step = (int64_t)gridDim.x * (UBLK / WAVE) * TRW;
    for (int64_t row0 = ((int64_t)blockIdx.x * (UBLK / WAVE) + w) * TRW; row0 < rows; row0 += step) {
        double z[4 * T], p[4 * T];
        load_rows<T>(Z, row0 + c, rows, m, z);
        load_rows<T>(P, row0 + c, rows, m, p);
        f64x4 acc[T] = {};
        times<T>(z, m, s_1, acc);
        times<T>(p, m, s_2, acc);
        // every product above has taken the wave's rows of P whole
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t row = row0 + 4 * u + k;
                if (row < rows && 16 * t + c < m) P[row * m + 16 * t + c] = acc[t][u];
            }
    }
}

// f(integral_constant<int, T>) for T = 1 .. 4 column tiles
template <typename F>
void with_tiles(int T, F &&f) {
    switch (T) {
        case 1: f(std::integral_constant<int, 1>()); break;
        case 2: f(std::integral_constant<int, 2>()); break;
        case 3: f(std::integral_constant<int, 3>()); break;
        default: f(std::integral_constant<int, 4>()); break;
    }
}

inline unsigned update_grid(int64_t rows) {
    const int64_t per = (int64_t)(UBLK / WAVE) * TRW;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>((rows + per - 1) / per, 2048));
}

}  // namespace

int block_gram_nblocks() { return GBLKS + GSPLIT; }
int block_xr_nblocks(int64_t rows) { return (int)update_grid(rows); }

void block_gram(const double *const *mats, int nmat, const int *li, const int *ri, int npair, int64_t rows, int m,
                double *partials, double *out, hipStream_t s) {
    TE_REQUIRE(nmat >= 1 && nmat <= 3 && npair >= 1 && npair <= 3 && m >= 1 && m <= GM, TE_EINVAL,
               "block Gram: bad arguments");
    for (int p = 0; p < npair; ++p)
        TE_REQUIRE(li[p] >= 0 && li[p] < nmat && ri[p] >= 0 && ri[p] < nmat, TE_EINVAL, "block Gram: bad pair");
    GramArgs g{};
    for (int i = 0; i < nmat; ++i) g.mat[i] = mats[i];
    for (int p = 0; p < npair; ++p) {
        g.li[p] = li[p];
        g.ri[p] = ri[p];
    }
    g.npair = npair;
    g.rows = rows;
    g.m = m;
    g.partials = partials;
    const int T = (m + 15) / 16, C = 16 * T;
    // a workgroup at least a few steps of 16 rows per wave
    const int64_t per = (int64_t)gram_split(T) * 64;
    const int nb = (int)std::max<int64_t>(1, std::min<int64_t>((rows + per - 1) / per, T <= 2 ? GBLKS / 2 : GBLKS));
    with_tiles(T, [&](auto t) {
        constexpr int TT = decltype(t)::value;
        hipLaunchKernelGGL(k_gram<TT>, dim3(nb), dim3(64 * npair * gram_split(TT)), 0, s, g);
    });
    const int64_t n = (int64_t)npair * C * C;
    double *out2 = partials + (int64_t)nb * n;
    hipLaunchKernelGGL(k_gram_sum1, dim3((unsigned)((n + 255) / 256), GSPLIT), dim3(256), 0, s, partials, nb, n, out2);
    hipLaunchKernelGGL(k_gram_sum2, dim3(GM * GM / 256, npair), dim3(256), 0, s, out2, C, n, out);
    TE_CHECK_HIP(hipGetLastError());
}

void block_xr(int64_t rows, int m, const double *alpha, const double *P, const double *Q, double *X, double *R,
              double *partials, hipStream_t s) {
    TE_REQUIRE(m >= 1 && m <= GM, TE_EINVAL, "block update: m = %d", m);
    with_tiles((m + 15) / 16, [&](auto t) {
        hipLaunchKernelGGL(k_block_xr<decltype(t)::value>, dim3(update_grid(rows)), dim3(UBLK), 0, s, rows, m, alpha, P,
                           Q, X, R, partials);
    });
    TE_CHECK_HIP(hipGetLastError());
}

void block_p(int64_t rows, int m, const double *T1, const double *T2, const double *Z, double *P, hipStream_t s) {
    TE_REQUIRE(m >= 1 && m <= GM, TE_EINVAL, "block update: m = %d", m);
    with_tiles((m + 15) / 16, [&](auto t) {
        hipLaunchKernelGGL(k_block_p<decltype(t)::value>, dim3(update_grid(rows)), dim3(UBLK), 0, s, rows, m, T1, T2, Z,
                           P);
    });
    TE_CHECK_HIP(hipGetLastError());
}

}  // namespace te
