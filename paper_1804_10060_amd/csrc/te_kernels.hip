// Sparse and vector kernels of the PCG / V-cycle hot loop (gfx950, wave64).
//
// Every sparse product runs on the SELL-64 block layout of te_internal.h:
// one lane per block row, 64 rows per wave, entry k of all 64 lanes stored
// contiguously so each value plane is one fully coalesced 512-byte (float64)
// load per wave.  Rows inside a slice are sorted by descending length, so the
// per-lane length mask switches off whole cache lines of padding at the tail.
// The x gathers hit L2: node numbering is lexicographic, and the block index
// is remapped so that each XCD streams one contiguous range of slices and
// keeps its own L2 window of x.
//
// Multi-RHS products (nrhs > 1, vectors laid out [row][comp][rhs]) of SELL
// operators take several block rows per wave, each with a group of lanes over
// its columns (k_sellm); above 32 columns one wave per block row with the
// right-hand sides on the lanes and the block values through the scalar cache
// (k_sellw).  Wave-per-row operators put slots of entries times columns on the
// lanes (k_rowm).
//
// Epilogues fuse the vector work of the Chebyshev smoother (Saad, Alg. 12.1),
// the residual of the V-cycle and the dot products of CG into the product.
// All reductions are deterministic: per-block partials in a fixed order,
// then summed in a fixed order (by one workgroup, or, for large partial
// tables, by fixed chunks and then the chunk sums).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "te_dev.h"

namespace te {
// Single right-hand side, lane per row: each wave handles `spw` consecutive
// slices, a workgroup blockDim/64 waves (both chosen by the autotuner);
// `remap` turns the XCD-contiguous block order on.
template <int BR, int BC, typename VT, typename XT, typename AT, class Epi, bool NT>
__global__ void __launch_bounds__(512) k_sell1(SellView<VT> A, const XT *__restrict__ x, Epi epi,
                                               double *__restrict__ partials, int spw, int remap) {
    __shared__ double lds[16];
    const int64_t nb = gridDim.x;
    const int64_t lb = remap ? xcd_logical_block(blockIdx.x, nb) : (int64_t)blockIdx.x;
    const int lane = threadIdx.x & (WAVE - 1);
    const int64_t w0 = (lb * (blockDim.x / WAVE) + threadIdx.x / WAVE) * spw;
    double red = 0.0;
    for (int u = 0; u < spw; ++u)
        if (w0 + u < A.nslices) sell1_body<BR, BC, VT, XT, AT, Epi, NT>(A, x, epi, w0 + u, lane, red);
    if (Epi::kReduce) {
        double t = block_sum(red, lds);
        if (threadIdx.x == 0) partials[lb] = t;
    }
}

// Single right-hand side on an operator of too few slices to fill the device
// (sell_split): a workgroup of W waves per slice, XCD-contiguous.
template <int BR, int BC, typename VT, typename XT, typename AT, class Epi, bool NT>
__global__ void __launch_bounds__(512) k_sell1s(SellView<VT> A, const XT *__restrict__ x, Epi epi,
                                                double *__restrict__ partials) {
    __shared__ AT buf[8 * BR * WAVE];
    __shared__ double lds[16];
    const int64_t slice = xcd_logical_block(blockIdx.x, gridDim.x);
    const int lane = threadIdx.x & (WAVE - 1), W = blockDim.x / WAVE;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
    double red = 0.0;
    sell1_split<BR, BC, VT, XT, AT, Epi, NT>(A, x, epi, slice, lane, w, W, buf, red);
    if (Epi::kReduce) {
        const double t = block_sum(red, lds);   // waves past the first add zero
        if (threadIdx.x == 0) partials[slice] = t;
    }
}

// Several right-hand sides on the SELL layout, one wave per block row with
// the right-hand sides on the lanes (at most 64); the block values are
// wave-uniform (scalar loads), the row's column indices come 64 at a time
// and are taken by readlane, and the x rows of 4 entries are loaded before
// any of them is used.  The default above 32 columns; the tuner may pick
// the row groups below instead.
//   Bound by the walk over a row's blocks (dependent loads, eight waves per SIMD
// at most), not by memory: 64 columns on 334,368 P1 nodes gather 7.4 GB of x a
// product, of which 1.6 GB come from memory.  More entries in flight, at fewer
// waves, and a last batch padded with repeated entries took longer (0.75 to 1.1
// ms).  The epilogue's inputs are loaded before the entries: Chebyshev start and
// steps 875, 806 and 765 us -> 781, 757 and 726 there.
template <int BR, int BC, typename VT, typename XT, typename AT, class Epi>
__global__ void __launch_bounds__(512) k_sellw(SellView<VT> A, const XT *__restrict__ x, Epi epi, int nrhs,
                                               double *__restrict__ partials, int wpb) {
    constexpr int MU = BC <= 3 ? 4 : 2;
    __shared__ double lds[8 * WAVE];
    const int64_t nb = gridDim.x;
    const int64_t lb = xcd_logical_block(blockIdx.x, nb);
    const int lane = threadIdx.x & (WAVE - 1);
    const int64_t row = (int64_t)__builtin_amdgcn_readfirstlane((int)(lb * wpb + threadIdx.x / WAVE));
    double red = 0.0;
    if (row < A.nrows) {
        const int rl = (int)(row % WAVE);
        const int off = A.slice_off[row / WAVE];
        const int len = A.rowlen[row];
        const int64_t out = A.rowmap ? (int64_t)A.rowmap[row] : row;
        typename Epi::template Pre<BR> pre{};
        if (lane < nrhs) pre = epi.template load_m<BR>(out, lane, nrhs);
        AT acc[BR];
#pragma unroll
        for (int i = 0; i < BR; ++i) acc[i] = AT(0);
        auto entry = [&](int k, const AT *xv) {
            const VT *vk = A.val + (int64_t)(off + k) * (BR * BC * WAVE);
#pragma unroll
            for (int i = 0; i < BR; ++i)
#pragma unroll
                for (int j = 0; j < BC; ++j)
                    acc[i] += AT(vk[sell_val_off<sell_vw<VT>()>(i * BC + j, BR * BC, rl)]) * xv[j];
        };
        for (int k0 = 0; k0 < len; k0 += WAVE) {
            const int cnt = min(WAVE, len - k0);
            const int cl = k0 + lane < len ? A.col[(int64_t)(off + k0 + lane) * WAVE + rl] : 0;
            if (lane < nrhs) {
                int u = 0;
                for (; u + MU <= cnt; u += MU) {
                    AT xv[MU][BC];
#pragma unroll
                    for (int t = 0; t < MU; ++t) {
                        const int64_t c = __builtin_amdgcn_readlane(cl, u + t);
#pragma unroll
                        for (int j = 0; j < BC; ++j) xv[t][j] = AT(x[(c * BC + j) * nrhs + lane]);
                    }
#pragma unroll
                    for (int t = 0; t < MU; ++t) entry(k0 + u + t, xv[t]);
                }
                for (; u < cnt; ++u) {
                    const int64_t c = __builtin_amdgcn_readlane(cl, u);
                    AT xv[BC];
#pragma unroll
                    for (int j = 0; j < BC; ++j) xv[j] = AT(x[(c * BC + j) * nrhs + lane]);
                    entry(k0 + u, xv);
                }
            }
        }
        if (lane < nrhs) epi.template apply_m<BR>(out, lane, nrhs, acc, red, pre);
    }
    if (Epi::kReduce) {
        lds[threadIdx.x] = red;
        __syncthreads();
        if (threadIdx.x < WAVE && threadIdx.x < nrhs) {
            double t = 0.0;
            for (int w = 0; w < wpb; ++w) t += lds[w * WAVE + threadIdx.x];
            partials[lb * nrhs + threadIdx.x] = t;
        }
    }
}

// Several right-hand sides on the SELL layout in row groups: R consecutive
// block rows of one slice per wave, T = 64 / R lanes per row, each lane S
// right-hand sides
// (c0 + j, c0 + j + T, ...) of the column tile c0 = blockIdx.y * T * S.  A
// lane loads its row's block values (vector loads: the R rows of a wave
// share each 16-byte value piece line) and reuses them for its S columns;
// the x rows of MU entries are loaded before any is used.  Column tiles are
// the slowest grid dimension, so the whole matrix runs for one tile before
// the next and the x rows an XCD gathers (tile width x 24 bytes per node)
// stay in its L2; the matrix is read once per tile.  The rows of a slice are
// sorted by descending length, so the first row of the wave bounds the
// entry loop; shorter rows run over their zero padding blocks (valid
// columns).  `wpb` waves per workgroup.  With split_tiles > 0 the column
// tiles are spread over the XCDs instead (see the kernel).
template <int BC, int S>
constexpr int multi_unroll() {
    return BC <= 3 && S <= 2 ? 2 : 1;
}

template <int BR, int BC, typename VT, typename XT, typename AT, class Epi, int R, int S>
__global__ void __launch_bounds__(512) k_sellm(SellView<VT> A, const XT *__restrict__ x, Epi epi, int nrhs,
                                                double *__restrict__ partials, int wpb, int split_tiles,
                                                int64_t split_chunk, int64_t nrb) {
    constexpr int T = WAVE / R, E = BR * BC, MU = multi_unroll<BC, S>();
    constexpr int VW = sell_vw<VT>(), G = E / VW;
    typedef VT vec_t __attribute__((ext_vector_type(VW)));
    __shared__ double lds[16 * WAVE];
    int64_t lb;
    int c0;
    if (split_tiles) {
        // workgroup b runs on XCD b % 8: the XCDs are split_tiles column tiles
        // times 8 / split_tiles row ranges, so the XCDs of one range stream the
        // same rows (and value lines) at the same time, each for its tile
        const int xcd = (int)(blockIdx.x & 7);
        const int64_t i = blockIdx.x >> 3;
        lb = (int64_t)(xcd / split_tiles) * split_chunk + i;
        if (i >= split_chunk || lb >= nrb) return;   // the whole workgroup
        c0 = (xcd % split_tiles) * (T * S);
    } else {
        lb = xcd_logical_block(blockIdx.x, gridDim.x);
        c0 = blockIdx.y * (T * S);
    }
    const int lane = threadIdx.x & (WAVE - 1);
    const int q = lane / T, w = threadIdx.x / WAVE;
    const int j = c0 + lane % T;      // first column of the lane
    const int64_t row0 = (lb * wpb + w) * R;
    const int64_t row = row0 + q;
    double red[S];
#pragma unroll
    for (int t = 0; t < S; ++t) red[t] = 0.0;
    if (row0 < A.nrows) {
        // rows past the end (last slice) compute on row0's entries, store nothing
        const bool live = row < A.nrows;
        const int64_t rr = live ? row : row0;
        const int rl = (int)(rr % WAVE);
        const int off = A.slice_off[rr / WAVE];
        const int lmax = __builtin_amdgcn_readfirstlane(A.rowlen[row0]);
        const int64_t out = A.rowmap ? (int64_t)A.rowmap[rr] : rr;
        typename Epi::template Pre<BR> pre[S];
#pragma unroll
        for (int t = 0; t < S; ++t) pre[t] = epi.template load_m<BR>(out, min(j + t * T, nrhs - 1), nrhs);
        AT acc[S][BR];
#pragma unroll
        for (int t = 0; t < S; ++t)
#pragma unroll
            for (int i = 0; i < BR; ++i) acc[t][i] = AT(0);
        for (int k = 0; k < lmax; k += MU) {
            VT v[MU][E];
            AT xv[MU][S][BC];
#pragma unroll
            for (int u = 0; u < MU; ++u) {
                const int kk = min(k + u, lmax - 1);   // a repeated entry is not accumulated
                const int64_t c = A.col[(int64_t)(off + kk) * WAVE + rl];
                const VT *vk = A.val + (int64_t)(off + kk) * (E * WAVE);
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const vec_t t = *reinterpret_cast<const vec_t *>(vk + (int64_t)(g * WAVE + rl) * VW);
#pragma unroll
                    for (int e = 0; e < VW; ++e) v[u][g * VW + e] = t[e];
                }
#pragma unroll
                for (int e = G * VW; e < E; ++e) v[u][e] = vk[(int64_t)(G * VW) * WAVE + (e - G * VW) * WAVE + rl];
#pragma unroll
                for (int t = 0; t < S; ++t) {
                    const int jj = j + t * T;
#pragma unroll
                    for (int b = 0; b < BC; ++b) xv[u][t][b] = jj < nrhs ? AT(x[(c * BC + b) * nrhs + jj]) : AT(0);
                }
            }
#pragma unroll
            for (int u = 0; u < MU; ++u) {
                if (k + u >= lmax) break;
#pragma unroll
                for (int t = 0; t < S; ++t)
#pragma unroll
                    for (int i = 0; i < BR; ++i)
#pragma unroll
                        for (int b = 0; b < BC; ++b) acc[t][i] += AT(v[u][i * BC + b]) * xv[u][t][b];
            }
        }
        if (live) {
#pragma unroll
            for (int t = 0; t < S; ++t)
                if (j + t * T < nrhs) epi.template apply_m<BR>(out, j + t * T, nrhs, acc[t], red[t], pre[t]);
        }
    }
    if (Epi::kReduce) {
        // per column: the R rows of the wave by a fixed shuffle tree, then the
        // waves of the block in order
#pragma unroll
        for (int t = 0; t < S; ++t) {
            double v = red[t];
#pragma unroll
            for (int o = T; o < WAVE; o <<= 1) v += __shfl_xor(v, o, WAVE);
            if (q == 0) lds[w * WAVE + (j - c0) + t * T] = v;
        }
        __syncthreads();
        if (threadIdx.x < T * S && c0 + (int)threadIdx.x < nrhs) {
            double t = 0.0;
            for (int ww = 0; ww < wpb; ++ww) t += lds[ww * WAVE + threadIdx.x];
            partials[lb * nrhs + c0 + threadIdx.x] = t;
        }
    }
}

template <int BR, int BC, typename VT, typename XT, typename AT, class Epi, bool NT>
__global__ void __launch_bounds__(512) k_roww(RowView<VT> A, const XT *__restrict__ x, Epi epi,
                                              double *__restrict__ partials, int spw, int remap, int xb) {
    __shared__ double rlds[16];
    __shared__ AT wb[512];
    const int64_t nb = gridDim.x;
    const int64_t lb = remap ? xcd_logical_block(blockIdx.x, nb) : (int64_t)blockIdx.x;
    const int lane = threadIdx.x & (WAVE - 1);
    const int64_t w0 = (lb * (blockDim.x / WAVE) + threadIdx.x / WAVE) * spw;
    AT *wbuf = wb + (threadIdx.x / WAVE) * WAVE;
    double red = 0.0;
    if constexpr (BC <= BR) {
        if (xb) {
            for (int u = 0; u < spw; ++u)
                if (w0 + u < A.nrows)
                    roww_body<BR, BC, VT, XT, AT, Epi, NT, true>(A, x, epi, w0 + u, lane, red, wbuf);
        } else {
            for (int u = 0; u < spw; ++u)
                if (w0 + u < A.nrows) roww_body<BR, BC, VT, XT, AT, Epi, NT>(A, x, epi, w0 + u, lane, red, wbuf);
        }
    } else {
        for (int u = 0; u < spw; ++u)
            if (w0 + u < A.nrows) roww_body<BR, BC, VT, XT, AT, Epi, NT>(A, x, epi, w0 + u, lane, red, wbuf);
    }
    if (Epi::kReduce) {
        double t = block_sum(red, rlds);
        if (threadIdx.x == 0) partials[lb] = t;
    }
}

// Few long rows (roww_split): a workgroup of W waves per row, the partial sums
// added slot by slot in wave order.
template <int BR, int BC, typename VT, typename XT, typename AT, class Epi, bool NT>
__global__ void __launch_bounds__(512) k_rowws(RowView<VT> A, const XT *__restrict__ x, Epi epi,
                                               double *__restrict__ partials, int xb) {
    constexpr int NB = WAVE / BR;
    __shared__ AT wb[512];
    __shared__ double rlds[16];
    const int64_t row = xcd_logical_block(blockIdx.x, gridDim.x);
    const int lane = threadIdx.x & (WAVE - 1), W = blockDim.x / WAVE;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
    wb[threadIdx.x] = xb ? roww_sum<BR, BC, VT, XT, AT, NT, true>(A, x, row, lane, w, W)
                         : roww_sum<BR, BC, VT, XT, AT, NT>(A, x, row, lane, w, W);
    __syncthreads();
    double red = 0.0;
    if (threadIdx.x < BR) {
        AT t[1] = {AT(0)};
        for (int v = 0; v < W; ++v)
#pragma unroll
            for (int sl = 0; sl < NB; ++sl) t[0] += wb[v * WAVE + sl * BR + threadIdx.x];
        const int64_t out = A.rowmap ? (int64_t)A.rowmap[row] : row;
        epi.template apply<1>(out * BR + threadIdx.x, t, red);
    }
    if (Epi::kReduce) {
        const double t = block_sum(red, rlds);
        if (threadIdx.x == 0) partials[row] = t;
    }
}

// Format 1 with several right-hand sides.  A wave takes S = 64 / C entries of
// a row at once: lane (slot, column), C the power of two that holds the
// columns (so up to 32 columns leave no lane without work); wpr waves share a
// row, wave w its entries w, w + wpr, ... (of slots), and their partial sums
// meet in LDS, where BR * C threads each add one entry's in a fixed order and
// run the epilogue.  With C = 64 the block values are wave-uniform and come
// through the scalar cache, MU blocks' x rows loaded before they are used;
// with slots every lane loads its block (16-byte pieces, one address per slot).
// What bounds it: a row is a serial walk over its blocks, so rows x waves in
// flight must cover the latency.  Against one wave per row with a lane per
// column for any number of columns: level products at 5 columns (5,000 rows of
// 46 blocks) 85 -> 35 us, the restrictions to levels of a few hundred long
// rows 196 -> 16 us at 5 columns and 304 -> 85 us at 64.  Two slots of 32
// columns measured slower than a lane per column with wave-uniform values
// (24 columns: 116 against 80 us), so slots end at 16 columns.
template <int BR, int BC, typename VT, typename XT, typename AT, class Epi, int C>
__global__ void __launch_bounds__(1024) k_rowm(RowView<VT> A, const XT *__restrict__ x, Epi epi, int nrhs, int wpr) {
    constexpr int S = WAVE / C, E = BR * BC;
    constexpr int VW = sizeof(VT) == 8 ? 2 : (E % 4 == 0 ? 4 : 2);
    static_assert(E % VW == 0, "block of whole 8- or 16-byte pieces");
    typedef VT vec_t __attribute__((ext_vector_type(VW)));
    extern __shared__ __align__(16) char rowm_lds[];   // [waves][BR][C] partial sums
    AT *buf = reinterpret_cast<AT *>(rowm_lds);
    const int lane = threadIdx.x & (WAVE - 1);
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
    const int grp = wv / wpr, ws = wv % wpr, rpg = blockDim.x / WAVE / wpr;
    const int64_t row = xcd_logical_block(blockIdx.x, gridDim.x) * rpg + grp;
    const bool live = row < A.nrows;   // uniform in the wave
    const int slot = lane / C, j = lane % C;
    const int jj = j < nrhs ? j : nrhs - 1;   // a spare column repeats the last, and is not stored
    AT acc[BR];
#pragma unroll
    for (int i = 0; i < BR; ++i) acc[i] = AT(0);
    if (live) {
        // the entries [lo, hi) of one list, col/idx its columns and blocks (idx
        // null: block k of entry k); TR: the block is stored transposed
        auto walk = [&](int64_t lo, int64_t hi, const int32_t *__restrict__ col, const int32_t *__restrict__ idx,
                        auto tr) {
            constexpr bool TR = decltype(tr)::value;
            if constexpr (S == 1) {
                constexpr int MU = BC <= 3 ? 4 : 2;
                const int64_t cntw = hi - lo > ws ? (hi - lo - ws + wpr - 1) / wpr : 0;   // this wave's entries
                for (int64_t t0 = 0; t0 < cntw; t0 += WAVE) {
                    const int cnt = (int)min((int64_t)WAVE, cntw - t0);
                    const int64_t kl = lo + ws + (t0 + (lane < cnt ? lane : 0)) * wpr;
                    const int cl = col[kl];
                    const int il = idx ? idx[kl] : 0;
                    auto one = [&](int u, const AT *xv) {
                        const VT *v = A.val + (idx ? (int64_t)__builtin_amdgcn_readlane(il, u)
                                                   : lo + ws + (t0 + u) * wpr) * E;
#pragma unroll
                        for (int i = 0; i < BR; ++i)
#pragma unroll
                            for (int b = 0; b < BC; ++b) acc[i] += AT(TR ? v[b * BC + i] : v[i * BC + b]) * xv[b];
                    };
                    auto load = [&](int u, AT *xv) {
                        const int64_t c = __builtin_amdgcn_readlane(cl, u);
#pragma unroll
                        for (int b = 0; b < BC; ++b) xv[b] = AT(x[(c * BC + b) * nrhs + jj]);
                    };
                    int u = 0;
                    for (; u + MU <= cnt; u += MU) {
                        AT xv[MU][BC];
#pragma unroll
                        for (int t = 0; t < MU; ++t) load(u + t, xv[t]);
#pragma unroll
                        for (int t = 0; t < MU; ++t) one(u + t, xv[t]);
                    }
                    for (; u < cnt; ++u) {
                        AT xv[BC];
                        load(u, xv);
                        one(u, xv);
                    }
                }
            } else {
                for (int64_t k = lo + ws * S + slot; k < hi; k += (int64_t)wpr * S) {
                    const int64_t c = col[k];
                    const vec_t *v = reinterpret_cast<const vec_t *>(A.val + (idx ? (int64_t)idx[k] : k) * E);
                    AT xv[BC];
#pragma unroll
                    for (int b = 0; b < BC; ++b) xv[b] = AT(x[(c * BC + b) * nrhs + jj]);
                    VT e[E];
#pragma unroll
                    for (int g = 0; g < E / VW; ++g) {
                        const vec_t t = v[g];
#pragma unroll
                        for (int h = 0; h < VW; ++h) e[g * VW + h] = t[h];
                    }
#pragma unroll
                    for (int i = 0; i < BR; ++i)
#pragma unroll
                        for (int b = 0; b < BC; ++b) acc[i] += AT(TR ? e[b * BC + i] : e[i * BC + b]) * xv[b];
                }
            }
        };
        walk(A.rptr[row], A.rptr[row + 1], A.col, (const int32_t *)nullptr, std::false_type{});
        if constexpr (BR == BC)
            if (A.lptr) walk(A.lptr[row], A.lptr[row + 1], A.lcol, A.lidx, std::true_type{});
    }
    double red = 0.0;
    if (S == 1 && wpr == 1) {
        if (live && j < nrhs) {
            const int64_t out = A.rowmap ? (int64_t)A.rowmap[row] : row;
            epi.template apply_m<BR>(out, j, nrhs, acc, red, epi.template load_m<BR>(out, j, nrhs));
        }
        return;
    }
#pragma unroll
    for (int o = C; o < WAVE; o <<= 1)
#pragma unroll
        for (int i = 0; i < BR; ++i) acc[i] += __shfl_xor(acc[i], o, WAVE);
    if (slot == 0)
#pragma unroll
        for (int i = 0; i < BR; ++i) buf[(wv * BR + i) * C + j] = acc[i];
    __syncthreads();
    if (!live) return;
    const int64_t out = A.rowmap ? (int64_t)A.rowmap[row] : row;
    for (int o = ws * WAVE + lane; o < BR * C; o += wpr * WAVE) {
        const int i = o / C, jo = o % C;
        if (jo >= nrhs) continue;
        AT t[1] = {AT(0)};
        for (int w = 0; w < wpr; ++w) t[0] += buf[((grp * wpr + w) * BR + i) * C + jo];
        epi.template apply_m<1>(out * BR + i, jo, nrhs, t, red, epi.template load_m<1>(out * BR + i, jo, nrhs));
    }
}

// ---------------------------------------------------------------------------
// Launch helpers
// ---------------------------------------------------------------------------
template <typename T>
static inline const Tune &tune_of(const Sell &A) {
    return sizeof(T) == 4 ? A.tune32 : A.tune64;
}

// Block rows per wave of the SELL multi-RHS product for nrhs columns: 16
// rows (4 lanes each) for at most 4 columns, 8 rows of 8 lanes for at most 8,
// else 4 rows of 16 lanes; one row per wave for the lane-per-column kernel
// (tile 0, above 32 columns).  Five columns on 95,700 P1 nodes: 93 to 120 us a
// product with 16 lanes per row, 54 to 76 with 8 (four entries in flight instead
// of two: no faster).
static inline int multi_rows(int nrhs, int mtile) {
    if (mtile == 0 && nrhs > 32) return 1;   // k_sellw
    return nrhs <= 4 ? 16 : nrhs <= 8 ? 8 : 4;
}
// Columns per lane: the column tile (16, 32 or 64 columns per pass over the
// matrix, tuned; 32 where tile 0 does not mean a lane per column) over the 16
// lanes of a row.  24 columns on 95,700 P1 nodes with a lane per column: 145 to
// 203 us a product, with two columns on each of 16 lanes 142 to 188, with one on
// each of 32 194 to 234.
static inline int multi_cols(int nrhs, int mtile) {
    if (nrhs <= 8) return 1;
    const int need = (nrhs + 15) / 16;   // 1..4
    const int s = std::min(need, (mtile == 0 ? 32 : mtile) / 16);
    return s >= 4 ? 4 : (s >= 2 ? 2 : 1);
}

// Waves per slice (SELL) or row (one wave per row) of the single-RHS products.
// An operator whose slices or rows leave the device's wave slots empty (4096
// at four waves of the float64 product per SIMD) takes more waves for each,
// while every wave keeps three entries of a lane's row, or two steps of its
// row's blocks.  The operator alone decides, so the sums do not depend on the
// tuned launch shape.  Products of 1115 slices of 27 blocks (the
// 214,000-DOF P2 disc) 0.056 -> 0.027 ms, restriction to 155 rows of 122
// blocks 9.6 -> 6.4 us, the 77 slices of the 14,739-DOF cube 8 -> 5 us.
static int launch_split(const Sell &A) {
    const int64_t units = A.format == FMT_SELL ? A.nslices : A.nrows;
    if (units == 0) return 1;
    const int64_t blocks = A.sym() ? 2 * A.nnzb - A.nrows : A.nnzb;
    const int64_t steps = A.format == FMT_SELL ? blocks / (3 * A.nrows) : blocks / (2 * (WAVE / A.br) * A.nrows);
    int w = 1;
    while (w < 8 && units * w < 4096 && 2 * w <= steps) w *= 2;
    return w;
}

static inline int64_t sell_grid(const Sell &A, int nrhs, const Tune &t) {
    if (nrhs == 1) {
        if (launch_split(A) > 1) return A.format == FMT_SELL ? A.nslices : A.nrows;
        const int64_t units = A.format == FMT_SELL ? A.nslices : A.nrows;
        const int64_t per = (int64_t)t.wpb * t.spw;
        return (units + per - 1) / per;
    }
    const int64_t per = (int64_t)t.mwpb * (A.format == FMT_SELL ? multi_rows(nrhs, t.mtile) : 1);
    return (A.nrows + per - 1) / per;
}

int sell_partials_count(const Sell &A, int nrhs) { return (int)sell_grid(A, nrhs, A.tune64); }

// Waves per row of k_rowm: one where the rows alone fill the device (8192
// waves, eight per SIMD), else doubled until they do, while each wave keeps at
// least two steps of its slots (a restriction to 96 rows of 300 blocks at 64
// columns takes 263 us with one wave per row).
static int rowm_waves(const Sell &A, int slots) {
    const int64_t blocks = A.sym() ? 2 * A.nnzb - A.nrows : A.nnzb;
    const int64_t steps = blocks / (A.nrows * slots);
    int w = 1;
    while (w < 16 && A.nrows * w < 8192 && steps >= 4 * w) w *= 2;
    return w;
}

static inline int rowm_cols(int nrhs) { return nrhs <= 2 ? 2 : nrhs <= 4 ? 4 : nrhs <= 8 ? 8 : nrhs <= 16 ? 16 : WAVE; }

// column tiles of the row-group product, and whether they can go to different XCDs
static inline unsigned multi_tiles(int nrhs, int R, int S) {
    const int tile = (WAVE / R) * S;
    return (unsigned)((nrhs + tile - 1) / tile);
}
static inline bool splits_over_xcds(unsigned tiles) { return tiles == 2 || tiles == 4 || tiles == 8; }

Tune effective_tune(const Sell &A, int nrhs, Tune c, const Tune &d) {
    if (nrhs == 1) {
        if (launch_split(A) > 1) {
            c.wpb = d.wpb;
            c.spw = d.spw;
            c.remap = d.remap;
        }
        if (A.format == FMT_SELL) c.xb = d.xb;
        c.mwpb = d.mwpb;
        c.mtile = d.mtile;
        c.msplit = d.msplit;
        return c;
    }
    c.wpb = d.wpb;
    c.spw = d.spw;
    c.remap = d.remap;
    c.nt = d.nt;
    c.xb = d.xb;
    if (A.format == FMT_ROWWAVE) {
        const int cols = rowm_cols(nrhs);
        if (cols < WAVE || rowm_waves(A, 1) > 1) c.mwpb = d.mwpb;
        c.mtile = d.mtile;
        c.msplit = d.msplit;
        return c;
    }
    const int R = multi_rows(nrhs, c.mtile), S = multi_cols(nrhs, c.mtile);
    if (R == 1 || !splits_over_xcds(multi_tiles(nrhs, R, S))) c.msplit = d.msplit;
    if (R == multi_rows(nrhs, d.mtile) && (R == 1 || S == multi_cols(nrhs, d.mtile))) c.mtile = d.mtile;
    else if (R > 1) c.mtile = 16 * S;
    return c;
}

template <int BR, int BC, typename VT, typename XT, typename AT, class Epi>
static void launch_rowm(const Sell &A, const VT *val, const XT *x, const Epi &epi, int nrhs, int mwpb, hipStream_t s) {
    auto go = [&](auto kern, int c) {
        const int wpr = rowm_waves(A, WAVE / c);
        const int waves = c == WAVE && wpr == 1 ? mwpb : std::max(4, wpr);
        const int64_t g = (A.nrows + waves / wpr - 1) / (waves / wpr);
        const size_t lds = c == WAVE && wpr == 1 ? 0 : (size_t)waves * BR * c * sizeof(AT);
        hipLaunchKernelGGL(kern, dim3((unsigned)g), dim3(waves * WAVE), lds, s, rview(A, val), x, epi, nrhs, wpr);
    };
    switch (rowm_cols(nrhs)) {
        case 2: go(k_rowm<BR, BC, VT, XT, AT, Epi, 2>, 2); break;
        case 4: go(k_rowm<BR, BC, VT, XT, AT, Epi, 4>, 4); break;
        case 8: go(k_rowm<BR, BC, VT, XT, AT, Epi, 8>, 8); break;
        case 16: go(k_rowm<BR, BC, VT, XT, AT, Epi, 16>, 16); break;
        default: go(k_rowm<BR, BC, VT, XT, AT, Epi, WAVE>, WAVE);
    }
    TE_CHECK_HIP(hipGetLastError());
}

template <int BR, int BC, typename VT, typename XT, typename AT, class Epi>
static void launch_t(const Sell &A, const VT *val, const XT *x, const Epi &epi, int nrhs, double *partials,
                     hipStream_t s) {
    const Tune &t = tune_of<VT>(A);
    // the partial-sum tables hold one entry per 4 block rows at most; the SELL
    // multi-RHS kernel runs at most 8 waves per workgroup
    TE_REQUIRE(nrhs == 1 || t.mwpb == 4 || t.mwpb == 8 || (t.mwpb == 16 && A.format == FMT_ROWWAVE), TE_EINVAL,
               "bad waves per workgroup %d", t.mwpb);
    int64_t g = sell_grid(A, nrhs, t);
    if (g == 0) return;
    const dim3 blk(64 * (nrhs == 1 ? t.wpb : t.mwpb));
    TE_REQUIRE(A.format == (BR == 6 ? FMT_ROWWAVE : FMT_SELL), TE_EINVAL, "no %dx%d-block operator in layout %d", BR,
               BC, A.format);
    if (const int split = nrhs == 1 ? launch_split(A) : 1; split > 1) {
        const dim3 gs((unsigned)g), bs(WAVE * split);
        if constexpr (BR == 6) {
            if (t.nt) hipLaunchKernelGGL((k_rowws<BR, BC, VT, XT, AT, Epi, true>), gs, bs, 0, s, rview(A, val), x, epi,
                                         partials, t.xb);
            else hipLaunchKernelGGL((k_rowws<BR, BC, VT, XT, AT, Epi, false>), gs, bs, 0, s, rview(A, val), x, epi,
                                    partials, t.xb);
        } else {
            if (t.nt) hipLaunchKernelGGL((k_sell1s<BR, BC, VT, XT, AT, Epi, true>), gs, bs, 0, s, view(A, val), x,
                                         epi, partials);
            else hipLaunchKernelGGL((k_sell1s<BR, BC, VT, XT, AT, Epi, false>), gs, bs, 0, s, view(A, val), x, epi,
                                    partials);
        }
    } else if (nrhs == 1) {
        if constexpr (BR == 6) {
            if (t.nt)
                hipLaunchKernelGGL((k_roww<BR, BC, VT, XT, AT, Epi, true>), dim3((unsigned)g), blk, 0, s,
                                   rview(A, val), x, epi, partials, t.spw, t.remap, t.xb);
            else
                hipLaunchKernelGGL((k_roww<BR, BC, VT, XT, AT, Epi, false>), dim3((unsigned)g), blk, 0, s,
                                   rview(A, val), x, epi, partials, t.spw, t.remap, t.xb);
        } else {
            if (t.nt)
                hipLaunchKernelGGL((k_sell1<BR, BC, VT, XT, AT, Epi, true>), dim3((unsigned)g), blk, 0, s,
                                   view(A, val), x, epi, partials, t.spw, t.remap);
            else
                hipLaunchKernelGGL((k_sell1<BR, BC, VT, XT, AT, Epi, false>), dim3((unsigned)g), blk, 0, s,
                                   view(A, val), x, epi, partials, t.spw, t.remap);
        }
    } else if constexpr (BR == 6) {
        // sums over the rows are formed on the mesh level only (3-row blocks)
        if constexpr (!Epi::kReduce) launch_rowm<BR, BC, VT, XT, AT, Epi>(A, val, x, epi, nrhs, t.mwpb, s);
        else TE_REQUIRE(false, TE_EINVAL, "no reducing product of %dx%d blocks for several columns", BR, BC);
        return;
    } else {
        const int R = multi_rows(nrhs, t.mtile);
        if (R == 1) {
            hipLaunchKernelGGL((k_sellw<BR, BC, VT, XT, AT, Epi>), dim3((unsigned)g), blk, 0, s, view(A, val), x,
                               epi, nrhs, partials, t.mwpb);
            TE_CHECK_HIP(hipGetLastError());
            return;
        }
        const int S = multi_cols(nrhs, t.mtile);
        const unsigned tiles = multi_tiles(nrhs, R, S);
        dim3 grid((unsigned)g, tiles);
        int split = 0;
        int64_t chunk = 0;
        if (t.msplit && splits_over_xcds(tiles)) {
            split = (int)tiles;
            chunk = (g + 8 / split - 1) / (8 / split);
            grid = dim3((unsigned)(8 * chunk), 1);
        }
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, grid, blk, 0, s, view(A, val), x, epi, nrhs, partials, t.mwpb, split, chunk,
                               g);
        };
        if (R == 16) go(k_sellm<BR, BC, VT, XT, AT, Epi, 16, 1>);
        else if (R == 8) go(k_sellm<BR, BC, VT, XT, AT, Epi, 8, 1>);
        else if (S == 1) go(k_sellm<BR, BC, VT, XT, AT, Epi, 4, 1>);
        else if (S == 2) go(k_sellm<BR, BC, VT, XT, AT, Epi, 4, 2>);
        else go(k_sellm<BR, BC, VT, XT, AT, Epi, 4, 4>);
    }
    TE_CHECK_HIP(hipGetLastError());
}

template <typename T, class Epi>
static void dispatch(const Sell &A, const T *x, const Epi &epi, int nrhs, double *partials, hipStream_t s) {
    const T *val;
    if constexpr (sizeof(T) == 4) {
        TE_REQUIRE(A.val32.p, TE_EINVAL, "float32 operator copy not built");
        val = A.val32.p;
    } else {
        val = A.val.p;
    }
    const int key = A.br * 10 + A.bc;
    switch (key) {
        case 33: launch_t<3, 3, T, T, T>(A, val, x, epi, nrhs, partials, s); break;
        case 66: launch_t<6, 6, T, T, T>(A, val, x, epi, nrhs, partials, s); break;
        case 36: launch_t<3, 6, T, T, T>(A, val, x, epi, nrhs, partials, s); break;
        case 63: launch_t<6, 3, T, T, T>(A, val, x, epi, nrhs, partials, s); break;
        default: TE_REQUIRE(false, TE_EINVAL, "unsupported block shape %dx%d", A.br, A.bc);
    }
}

template <typename T>
void sell_apply(const Sell &A, const T *x, T *y, const T *g, int mode, int nrhs, hipStream_t s) {
    if (mode == 0) dispatch(A, x, EpiSet<T>{y}, nrhs, nullptr, s);
    else if (mode == 1) dispatch(A, x, EpiAdd<T>{y}, nrhs, nullptr, s);
    else dispatch(A, x, EpiResid<T, false>{g, y}, nrhs, nullptr, s);
}
template void sell_apply<double>(const Sell &, const double *, double *, const double *, int, int, hipStream_t);
template void sell_apply<float>(const Sell &, const float *, float *, const float *, int, int, hipStream_t);

void sell_resid_norm(const Sell &A, const double *x, const double *g, double *y, int nrhs, double *partials,
                     hipStream_t s) {
    dispatch(A, x, EpiResid<double, true>{g, y}, nrhs, partials, s);
}

void sell_dot(const Sell &A, const double *p, double *q, int nrhs, double *partials, hipStream_t s) {
    dispatch(A, p, EpiDot{p, q}, nrhs, partials, s);
}

template <typename T>
void cheb_init(const Sell &A, const T *x, const T *g, const T *dinv, T *r, T *d, double inv_theta, int nrhs,
               hipStream_t s) {
    dispatch(A, x, EpiChebInit<T>{g, dinv, r, d, T(inv_theta)}, nrhs, nullptr, s);
}
template void cheb_init<double>(const Sell &, const double *, const double *, const double *, double *, double *,
                                double, int, hipStream_t);
template void cheb_init<float>(const Sell &, const float *, const float *, const float *, float *, float *, double,
                               int, hipStream_t);

template <typename T>
void cheb_step(const Sell &A, const T *d, const T *rin, const T *dinv, T *rout, T *dout, T *x, double c1, double c2,
               bool last, bool xzero, int nrhs, hipStream_t s) {
    if (last && xzero)
        dispatch(A, d, EpiChebStep<T, true, true>{rin, d, dinv, rout, dout, x, T(c1), T(c2)}, nrhs, nullptr, s);
    else if (last)
        dispatch(A, d, EpiChebStep<T, true, false>{rin, d, dinv, rout, dout, x, T(c1), T(c2)}, nrhs, nullptr, s);
    else if (xzero)
        dispatch(A, d, EpiChebStep<T, false, true>{rin, d, dinv, rout, dout, x, T(c1), T(c2)}, nrhs, nullptr, s);
    else
        dispatch(A, d, EpiChebStep<T, false, false>{rin, d, dinv, rout, dout, x, T(c1), T(c2)}, nrhs, nullptr, s);
}
template void cheb_step<double>(const Sell &, const double *, const double *, const double *, double *, double *,
                                double *, double, double, bool, bool, int, hipStream_t);
template void cheb_step<float>(const Sell &, const float *, const float *, const float *, float *, float *, float *,
                               double, double, bool, bool, int, hipStream_t);

// ---------------------------------------------------------------------------
// Element-wise kernels
// ---------------------------------------------------------------------------
static inline unsigned egrid(int64_t n) {
    int64_t g = (n + BLK - 1) / BLK;
    if (g > (1 << 20)) g = 1 << 20;
    return (unsigned)(g < 1 ? 1 : g);
}

// d = D^-1 g / theta  (pre-smoothing start, x0 = 0); rows*bs*nrhs entries
template <typename T>
__global__ void k_jacobi_scale(const T *__restrict__ g, const T *__restrict__ dinv, T *__restrict__ d, T inv_theta,
                               int64_t n, int nrhs) {
    for (int64_t i = blockIdx.x * (int64_t)BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK)
        d[i] = dinv[i / nrhs] * g[i] * inv_theta;
}
template <typename T>
void jacobi_scale(const T *g, const T *dinv, T *d, double inv_theta, int64_t n, int nrhs, hipStream_t s) {
    if (n == 0) return;
    hipLaunchKernelGGL(k_jacobi_scale<T>, dim3(egrid(n)), dim3(BLK), 0, s, g, dinv, d, T(inv_theta), n, nrhs);
    TE_CHECK_HIP(hipGetLastError());
}
template void jacobi_scale<double>(const double *, const double *, double *, double, int64_t, int, hipStream_t);
template void jacobi_scale<float>(const float *, const float *, float *, double, int64_t, int, hipStream_t);

template <typename T>
__global__ void k_axpy(T *__restrict__ y, const T *__restrict__ x, T a, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK) y[i] += a * x[i];
}
template <typename T>
void axpy(T *y, const T *x, double a, int64_t n, hipStream_t s) {
    if (n == 0) return;
    hipLaunchKernelGGL(k_axpy<T>, dim3(egrid(n)), dim3(BLK), 0, s, y, x, T(a), n);
    TE_CHECK_HIP(hipGetLastError());
}
template void axpy<double>(double *, const double *, double, int64_t, hipStream_t);
template void axpy<float>(float *, const float *, double, int64_t, hipStream_t);

template <typename A, typename B>
__global__ void k_cast(const A *__restrict__ x, B *__restrict__ y, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK) y[i] = B(x[i]);
}
void cast_f64_f32(const double *x, float *y, int64_t n, hipStream_t s) {
    if (n == 0) return;
    hipLaunchKernelGGL((k_cast<double, float>), dim3(egrid(n)), dim3(BLK), 0, s, x, y, n);
    TE_CHECK_HIP(hipGetLastError());
}
void cast_f32_f64(const float *x, double *y, int64_t n, hipStream_t s) {
    if (n == 0) return;
    hipLaunchKernelGGL((k_cast<float, double>), dim3(egrid(n)), dim3(BLK), 0, s, x, y, n);
    TE_CHECK_HIP(hipGetLastError());
}

// dst[i] = src[map[i]] per node (bs*nrhs contiguous values per node)
__global__ void k_perm_gather(const double *__restrict__ src, double *__restrict__ dst, const int32_t *__restrict__ map,
                              int64_t n, int per) {
    for (int64_t t = blockIdx.x * (int64_t)BLK + threadIdx.x; t < n * per; t += (int64_t)gridDim.x * BLK) {
        int64_t i = t / per, k = t % per;
        dst[t] = src[(int64_t)map[i] * per + k];
    }
}
__global__ void k_perm_scatter(const double *__restrict__ src, double *__restrict__ dst,
                               const int32_t *__restrict__ map, int64_t n, int per) {
    for (int64_t t = blockIdx.x * (int64_t)BLK + threadIdx.x; t < n * per; t += (int64_t)gridDim.x * BLK) {
        int64_t i = t / per, k = t % per;
        dst[(int64_t)map[i] * per + k] = src[t];
    }
}
void permute_gather(const double *src, double *dst, const int32_t *map, int64_t n_nodes, int bs, int nrhs,
                    hipStream_t s) {
    if (n_nodes == 0) return;
    hipLaunchKernelGGL(k_perm_gather, dim3(egrid(n_nodes * bs * nrhs)), dim3(BLK), 0, s, src, dst, map, n_nodes,
                       bs * nrhs);
    TE_CHECK_HIP(hipGetLastError());
}
void permute_scatter(const double *src, double *dst, const int32_t *map, int64_t n_nodes, int bs, int nrhs,
                     hipStream_t s) {
    if (n_nodes == 0) return;
    hipLaunchKernelGGL(k_perm_scatter, dim3(egrid(n_nodes * bs * nrhs)), dim3(BLK), 0, s, src, dst, map, n_nodes,
                       bs * nrhs);
    TE_CHECK_HIP(hipGetLastError());
}

// ---------------------------------------------------------------------------
// Deterministic dot products (per right-hand side column)
// ---------------------------------------------------------------------------
constexpr int DOT_BLOCKS = 1024;

int dot_nblocks(int64_t n) {
    int64_t g = (n + BLK - 1) / BLK;
    return (int)(g < 1 ? 1 : (g > DOT_BLOCKS ? DOT_BLOCKS : g));
}

// The vector kernels below give every workgroup a contiguous chunk of rows and
// every thread entries of one column only: the first 256 / nrhs * nrhs threads
// walk the chunk's entries in turn (column = thread % nrhs), so few columns
// leave no lane without work (a lane per column measured 66 us for the CG
// update at 5 columns on 287,000 rows, now 14), four entries in flight.
// The threads of a column are then added in a fixed order.
constexpr int VU = 4;

// sums of NV values per column over the workgroup, out[c * NV + v]
template <int NV>
__device__ __forceinline__ void column_sums(const double (&t)[NV], int nrhs, double *__restrict__ out) {
    __shared__ double lds[NV][BLK];
    if (nrhs == 1) {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const double s = block_sum(t[v], lds[v]);
            if (threadIdx.x == 0) out[v] = s;
        }
        return;
    }
    const int per = BLK / nrhs;
#pragma unroll
    for (int v = 0; v < NV; ++v) lds[v][threadIdx.x] = t[v];
    __syncthreads();
    for (int e = threadIdx.x; e < NV * nrhs; e += BLK) {
        const int c = e / NV, v = e % NV;
        double s = 0.0;
        for (int k = 0; k < per; ++k) s += lds[v][k * nrhs + c];
        out[e] = s;
    }
}

// f(i, act, cnt): entries i, i + act, ... (cnt of them, VU or 1) of this
// workgroup's chunk, in the thread's column
template <class F>
__device__ __forceinline__ void chunk_entries(int64_t rows, int nrhs, F f) {
    const int64_t chunk = (rows + gridDim.x - 1) / gridDim.x;
    const int64_t lo = blockIdx.x * chunk * nrhs, hi = min(rows, (blockIdx.x + 1) * chunk) * nrhs;
    const int act = BLK / nrhs * nrhs;
    if ((int)threadIdx.x >= act) return;
    int64_t i = lo + threadIdx.x;
    for (; i + (int64_t)(VU - 1) * act < hi; i += (int64_t)VU * act) f(i, act, VU);
    for (; i < hi; i += act) f(i, act, 1);
}

__global__ void __launch_bounds__(BLK) k_dot(const double *__restrict__ a, const double *__restrict__ b, int64_t rows,
                                             int nrhs, double *__restrict__ partials) {
    double t[1] = {0.0};
    chunk_entries(rows, nrhs, [&](int64_t i, int act, int cnt) {
        if (cnt == VU) {
            double x[VU], y[VU];
#pragma unroll
            for (int u = 0; u < VU; ++u) {
                x[u] = a[i + (int64_t)u * act];
                y[u] = b[i + (int64_t)u * act];
            }
#pragma unroll
            for (int u = 0; u < VU; ++u) t[0] += x[u] * y[u];
        } else {
            t[0] += a[i] * b[i];
        }
    });
    column_sums<1>(t, nrhs, partials + blockIdx.x * (int64_t)nrhs);
}

void dot_partials(const double *a, const double *b, int64_t n, int nrhs, double *partials, hipStream_t s) {
    const int64_t rows = n / nrhs;
    hipLaunchKernelGGL(k_dot, dim3(dot_nblocks(rows)), dim3(BLK), 0, s, a, b, rows, nrhs, partials);
    TE_CHECK_HIP(hipGetLastError());
}

// Column sums of a [nparts][ncols] table of partials in a fixed order, the
// scalar bookkeeping of the CG recurrence done by the same launch.
//   RED_STORE  out[c] = sum
//   RED_ALPHA  sum = (p, A p): alpha = active ? rz / pq : 0; flag if pq <= 0
//   RED_BETA   sum pairs ((r, z), (z, r - r_old)): beta; rz = (r, z); flag if <= 0
//   RED_RZ0    sum pairs: rz; flag if <= 0
// One workgroup: thread (r, c) adds every Rth part of its column, R the
// largest power of two of rows that fit 1024 threads, then a tree over r.  Long
// tables are cut to G chunks first (k_reduce_chunks, coalesced).  The former
// one-workgroup forms walked the columns one after the other, or the chunk
// sums in one thread per column: at 64 columns 166 us ((r, z) pairs), 84 us
// (|r|^2) and 233 us ((p, A p)) per launch, now 8 to 15 us.
enum { RED_STORE = 0, RED_ALPHA = 1, RED_BETA = 2, RED_RZ0 = 3 };
constexpr int RBLK = 1024;

template <int FIN>
__global__ void __launch_bounds__(RBLK) k_reduce(const double *__restrict__ partials, int nparts, int ncols, int R,
                                                 double *__restrict__ out, CgScalars *S, int flexible) {
    __shared__ double lds[RBLK];
    const int r = threadIdx.x / ncols, c = threadIdx.x % ncols;
    double t = 0.0;
    if (r < R)
#pragma unroll 8
        for (int b = r; b < nparts; b += R) t += partials[(int64_t)b * ncols + c];
    lds[threadIdx.x] = t;
    __syncthreads();
    for (int o = R / 2; o > 0; o >>= 1) {
        if (r < o) lds[threadIdx.x] += lds[threadIdx.x + o * ncols];
        __syncthreads();
    }
    const int j = threadIdx.x;
    if (FIN == RED_STORE) {
        if (j < ncols) out[j] = lds[j];
    } else if (FIN == RED_ALPHA) {
        if (j >= ncols) return;
        const double pq = lds[j];
        double a = 0.0;
        if (S->active[j]) {
            if (!(pq > 0.0)) S->flag[j] = (pq != pq) ? 3 : 1;
            else a = S->rz[j] / pq;
        }
        S->pq[j] = pq;
        S->alpha[j] = a;
    } else {
        if (2 * j >= ncols) return;
        const double rzn = lds[2 * j], fl = lds[2 * j + 1];
        const bool bad = S->active[j] && !(rzn > 0.0);
        if (bad) S->flag[j] = (rzn != rzn) ? 3 : 2;
        if (FIN == RED_BETA) {
            double b = 0.0;
            if (S->active[j] && !bad) {
                b = flexible ? fl / S->rz[j] : rzn / S->rz[j];
                S->rz[j] = rzn;
            }
            S->beta[j] = b;
        } else {
            S->rz[j] = rzn;
        }
    }
}

// chunk sums of a long table: workgroup g adds parts [g*chunk, (g+1)*chunk)
__global__ void __launch_bounds__(BLK) k_reduce_chunks(const double *__restrict__ partials, int nparts, int ncols,
                                                       int chunk, double *__restrict__ out2) {
    __shared__ double lds[BLK];
    const int R = BLK / ncols;  // rows per pass
    const int r = threadIdx.x / ncols, c = threadIdx.x % ncols;
    const int lo = blockIdx.x * chunk, hi = min(nparts, lo + chunk);
    double t = 0.0;
    if (r < R)
#pragma unroll 4
        for (int b = lo + r; b < hi; b += R) t += partials[(int64_t)b * ncols + c];
    lds[threadIdx.x] = t;
    __syncthreads();
    if ((int)threadIdx.x < ncols) {
        double u = 0.0;
        for (int k = 0; k < R; ++k) u += lds[k * ncols + threadIdx.x];
        out2[(int64_t)blockIdx.x * ncols + threadIdx.x] = u;
    }
}

// One pass up to 64 parts per thread; above, min(512, nparts / 64) chunk sums
// go behind the table.
template <int FIN>
static void reduce_fin(const double *partials, int nparts, int ncols, double *out, CgScalars *S, int flexible,
                       hipStream_t s) {
    TE_REQUIRE(ncols >= 1 && ncols <= 128, TE_EINVAL, "reduction over %d columns", ncols);
    int R = 1;
    while (2 * R * ncols <= RBLK) R *= 2;
    if ((int64_t)nparts > (int64_t)64 * R) {
        const int G = std::min(512, std::max(1, nparts / 64));
        const int chunk = (nparts + G - 1) / G;
        double *out2 = const_cast<double *>(partials) + (int64_t)nparts * ncols;
        hipLaunchKernelGGL(k_reduce_chunks, dim3(G), dim3(BLK), 0, s, partials, nparts, ncols, chunk, out2);
        partials = out2;
        nparts = G;
    }
    hipLaunchKernelGGL(k_reduce<FIN>, dim3(1), dim3(RBLK), 0, s, partials, nparts, ncols, R, out, S, flexible);
    TE_CHECK_HIP(hipGetLastError());
}

void reduce_partials(const double *partials, int nparts, int nrhs, double *out, hipStream_t s) {
    reduce_fin<RED_STORE>(partials, nparts, nrhs, out, nullptr, 0, s);
}
void reduce_alpha(const double *partials, int nparts, int nrhs, void *S, hipStream_t s) {
    reduce_fin<RED_ALPHA>(partials, nparts, nrhs, nullptr, (CgScalars *)S, 0, s);
}
void reduce_beta(const double *partials, int nparts, int nrhs, void *S, int flexible, hipStream_t s) {
    reduce_fin<RED_BETA>(partials, nparts, 2 * nrhs, nullptr, (CgScalars *)S, flexible, s);
}
void reduce_rz0(const double *partials, int nparts, int nrhs, void *S, hipStream_t s) {
    reduce_fin<RED_RZ0>(partials, nparts, 2 * nrhs, nullptr, (CgScalars *)S, 0, s);
}

// ---------------------------------------------------------------------------
// CG vector updates (float64), per-column scalars on the device
// ---------------------------------------------------------------------------
// u += alpha_j p; r_old = r (if keep_old); r -= alpha_j q; red_j += r^2
template <bool OLD>
__global__ void __launch_bounds__(BLK) k_cg_update(double *__restrict__ u, double *__restrict__ r,
                                                   double *__restrict__ r_old, const double *__restrict__ p,
                                                   const double *__restrict__ q, const double *__restrict__ alpha,
                                                   int64_t rows, int nrhs, double *__restrict__ partials) {
    double t[1] = {0.0};
    const double a = alpha[nrhs == 1 ? 0 : threadIdx.x % nrhs];
    chunk_entries(rows, nrhs, [&](int64_t i0, int act, int cnt) {
        auto part = [&](auto n) {
            constexpr int N = decltype(n)::value;
            double uv[N], pv[N], rv[N], qv[N];
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const int64_t i = i0 + (int64_t)k * act;
                uv[k] = u[i];
                pv[k] = p[i];
                rv[k] = r[i];
                qv[k] = q[i];
            }
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const int64_t i = i0 + (int64_t)k * act;
                u[i] = uv[k] + a * pv[k];
                if (OLD) r_old[i] = rv[k];
                const double rn = rv[k] - a * qv[k];
                r[i] = rn;
                t[0] += rn * rn;
            }
        };
        if (cnt == VU) part(std::integral_constant<int, VU>{});
        else part(std::integral_constant<int, 1>{});
    });
    column_sums<1>(t, nrhs, partials + blockIdx.x * (int64_t)nrhs);
}
void cg_update(double *u, double *r, double *r_old, const double *p, const double *q, const double *alpha,
               int64_t rows, int nrhs, double *partials, hipStream_t s) {
    auto kern = r_old ? k_cg_update<true> : k_cg_update<false>;
    hipLaunchKernelGGL(kern, dim3(dot_nblocks(rows)), dim3(BLK), 0, s, u, r, r_old, p, q, alpha, rows, nrhs,
                       partials);
    TE_CHECK_HIP(hipGetLastError());
}

// (r, z) and, for the flexible variant, (z, r - r_old) per column
template <bool OLD>
__global__ void __launch_bounds__(BLK) k_dot_rz(const double *__restrict__ r, const double *__restrict__ z,
                                                const double *__restrict__ r_old, int64_t rows, int nrhs,
                                                double *__restrict__ partials) {
    double t[2] = {0.0, 0.0};
    chunk_entries(rows, nrhs, [&](int64_t i0, int act, int cnt) {
        auto part = [&](auto n) {
            constexpr int N = decltype(n)::value;
            double rv[N], zv[N], ov[N];
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const int64_t i = i0 + (int64_t)k * act;
                rv[k] = r[i];
                zv[k] = z[i];
                ov[k] = OLD ? r_old[i] : 0.0;
            }
#pragma unroll
            for (int k = 0; k < N; ++k) {
                t[0] += rv[k] * zv[k];
                if (OLD) t[1] += zv[k] * (rv[k] - ov[k]);
            }
        };
        if (cnt == VU) part(std::integral_constant<int, VU>{});
        else part(std::integral_constant<int, 1>{});
    });
    column_sums<2>(t, nrhs, partials + blockIdx.x * (int64_t)nrhs * 2);
}
void dot_rz(const double *r, const double *z, const double *r_old, int64_t rows, int nrhs, double *partials,
            hipStream_t s) {
    auto kern = r_old ? k_dot_rz<true> : k_dot_rz<false>;
    hipLaunchKernelGGL(kern, dim3(dot_nblocks(rows)), dim3(BLK), 0, s, r, z, r_old, rows, nrhs, partials);
    TE_CHECK_HIP(hipGetLastError());
}

// p = z + beta_j p
__global__ void k_p_update(double *__restrict__ p, const double *__restrict__ z, const double *__restrict__ beta,
                           int64_t n, int nrhs) {
    for (int64_t i = blockIdx.x * (int64_t)BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK)
        p[i] = z[i] + beta[i % nrhs] * p[i];
}
void p_update(double *p, const double *z, const double *beta, int64_t n, int nrhs, hipStream_t s) {
    hipLaunchKernelGGL(k_p_update, dim3(egrid(n)), dim3(BLK), 0, s, p, z, beta, n, nrhs);
    TE_CHECK_HIP(hipGetLastError());
}

size_t cg_scalars_bytes() { return sizeof(CgScalars); }

// Column select: r[:, j] = t[:, j] where sel[j] != 0
__global__ void k_copy_cols(double *__restrict__ r, const double *__restrict__ t, const int32_t *__restrict__ sel,
                            int64_t n, int nrhs) {
    for (int64_t i = blockIdx.x * (int64_t)BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK)
        if (sel[i % nrhs]) r[i] = t[i];
}
void copy_cols(double *r, const double *t, const int32_t *sel, int64_t n, int nrhs, hipStream_t s) {
    hipLaunchKernelGGL(k_copy_cols, dim3(egrid(n)), dim3(BLK), 0, s, r, t, sel, n, nrhs);
    TE_CHECK_HIP(hipGetLastError());
}

// ---------------------------------------------------------------------------
// Dense coarse solve: y = Ainv x (Ainv symmetric n x n, float64)
// ---------------------------------------------------------------------------
// One column: one wave per row, the row's entries in pairs (16-byte loads when
// the rows start on 16 bytes: n even), four pairs per lane in flight (one entry
// at a time: 17 us at n = 2800, now 11).
template <typename T>
__global__ void __launch_bounds__(BLK) k_dense_mv(const double *__restrict__ Ainv, const T *__restrict__ x,
                                                  T *__restrict__ y, int n) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int64_t row = (int64_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * WPB + threadIdx.x / WAVE));
    if (row >= n) return;
    const double *a = Ainv + row * (int64_t)n;
    typedef double d2 __attribute__((ext_vector_type(2)));
    double t = 0.0;
    if ((n & 1) == 0) {
        const d2 *a2 = reinterpret_cast<const d2 *>(a);
#pragma unroll 4
        for (int j = lane; j < n / 2; j += WAVE) {
            const d2 v = a2[j];
            t += v[0] * double(x[2 * j]) + v[1] * double(x[2 * j + 1]);
        }
    } else {
#pragma unroll 4
        for (int j = lane; j < n; j += WAVE) t += a[j] * double(x[j]);
    }
    t = wave_sum(t);
    if (lane == 0) y[row] = T(t);
}

// Several columns: y[16 rows][nrhs] per workgroup on the float64 matrix cores
// (v_mfma_f64_16x16x4, column tiles of 16).  The eight waves take every eighth
// step of eight inner indices (lane (q, i): entries 8 s + 2 q and + 1 of row i
// and of column i's vector) and add their tiles in order through LDS.  One
// wave per row with a lane per column walked n inner indices serially: 139 us
// at n = 570 (64 columns), 32 us at n = 738 (5 columns); now 11 and 5 us.
constexpr int DW = 8;   // waves
template <typename T, int NT>
__global__ void __launch_bounds__(DW *WAVE) k_dense_mm(const double *__restrict__ Ainv, const T *__restrict__ x,
                                                       T *__restrict__ y, int n, int nrhs) {
    typedef double d4 __attribute__((ext_vector_type(4)));
    __shared__ double part[DW][16][16 * NT];
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE, i = lane & 15, q = lane >> 4;
    const int r0 = blockIdx.x * 16;
    const double *a = Ainv + (int64_t)min(r0 + i, n - 1) * n;   // a spare row repeats the last, and is not stored
    d4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
    for (int k0 = 8 * w; k0 < n; k0 += 8 * DW) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int k = k0 + 2 * q + h;
            const bool ok = k < n;
            const int kk = ok ? k : n - 1;
            const double av = a[kk];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const double xv = double(x[(int64_t)kk * nrhs + min(16 * t + i, nrhs - 1)]);
                acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(ok ? av : 0.0, ok ? xv : 0.0, acc[t], 0, 0, 0);
            }
        }
    }
    // register r of lane (q, i) is row 4 r + q, column i of the tile
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) part[w][4 * r + q][16 * t + i] = acc[t][r];
    __syncthreads();
    for (int e = threadIdx.x; e < 16 * 16 * NT; e += DW * WAVE) {
        const int r = e / (16 * NT), c = e % (16 * NT);
        if (r0 + r >= n || c >= nrhs) continue;
        double s = 0.0;
#pragma unroll
        for (int v = 0; v < DW; ++v) s += part[v][r][c];
        y[(int64_t)(r0 + r) * nrhs + c] = T(s);
    }
}
template <typename T>
void dense_mv(const double *Ainv, const T *x, T *y, int n, int nrhs, hipStream_t s) {
    if (n == 0) return;
    const dim3 g((n + 15) / 16), b(DW * WAVE);
    TE_REQUIRE(nrhs >= 1 && nrhs <= 64, TE_EINVAL, "dense product with %d columns", nrhs);
    if (nrhs == 1)
        hipLaunchKernelGGL(k_dense_mv<T>, dim3((n + WPB - 1) / WPB), dim3(BLK), 0, s, Ainv, x, y, n);
    else if (nrhs <= 16)
        hipLaunchKernelGGL((k_dense_mm<T, 1>), g, b, 0, s, Ainv, x, y, n, nrhs);
    else if (nrhs <= 32)
        hipLaunchKernelGGL((k_dense_mm<T, 2>), g, b, 0, s, Ainv, x, y, n, nrhs);
    else if (nrhs <= 48)
        hipLaunchKernelGGL((k_dense_mm<T, 3>), g, b, 0, s, Ainv, x, y, n, nrhs);
    else
        hipLaunchKernelGGL((k_dense_mm<T, 4>), g, b, 0, s, Ainv, x, y, n, nrhs);
    TE_CHECK_HIP(hipGetLastError());
}
template void dense_mv<double>(const double *, const double *, double *, int, int, hipStream_t);
template void dense_mv<float>(const double *, const float *, float *, int, int, hipStream_t);

// ---------------------------------------------------------------------------
// Lanczos helpers (setup)
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
    // Steele, Lea & Flood 2014: one step of the generator on input x
    uint64_t z = x + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// v[new*bs + c] = U(splitmix64(seed ^ natural_dof)) - 0.5
__global__ void k_lanczos_start(double *__restrict__ v, const int32_t *__restrict__ perm, int64_t n, int bs,
                                uint64_t seed) {
    for (int64_t t = blockIdx.x * (int64_t)BLK + threadIdx.x; t < n * bs; t += (int64_t)gridDim.x * BLK) {
        int64_t i = t / bs, c = t % bs;
        uint64_t nat = (uint64_t)perm[i] * (uint64_t)bs + (uint64_t)c;
        uint64_t z = splitmix64(seed ^ nat);
        v[t] = (double)(z >> 11) * 0x1.0p-53 - 0.5;
    }
}
void lanczos_start(double *v, const int32_t *perm, int64_t n, int bs, uint64_t seed, hipStream_t s) {
    hipLaunchKernelGGL(k_lanczos_start, dim3(egrid(n * bs)), dim3(BLK), 0, s, v, perm, n, bs, seed);
    TE_CHECK_HIP(hipGetLastError());
}

// y = a*x + b*y element-wise, then helpers for D^{1/2} scaling
__global__ void k_scale_mul(const double *__restrict__ x, const double *__restrict__ s, double *__restrict__ y,
                            int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK) y[i] = s[i] * x[i];
}
void scale_mul(const double *x, const double *sc, double *y, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_scale_mul, dim3(egrid(n)), dim3(BLK), 0, s, x, sc, y, n);
    TE_CHECK_HIP(hipGetLastError());
}
// w = sc * w - beta * vprev  (in place on w)
__global__ void k_lanczos_w(double *__restrict__ w, const double *__restrict__ sc, const double *__restrict__ vprev,
                            double beta, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK)
        w[i] = sc[i] * w[i] - beta * vprev[i];
}
void lanczos_w(double *w, const double *sc, const double *vprev, double beta, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_lanczos_w, dim3(egrid(n)), dim3(BLK), 0, s, w, sc, vprev, beta, n);
    TE_CHECK_HIP(hipGetLastError());
}
__global__ void k_scal(double *__restrict__ x, double a, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK) x[i] *= a;
}
void scal(double *x, double a, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_scal, dim3(egrid(n)), dim3(BLK), 0, s, x, a, n);
    TE_CHECK_HIP(hipGetLastError());
}

}  // namespace te

