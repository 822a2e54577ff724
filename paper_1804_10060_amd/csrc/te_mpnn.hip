// Message-passing network for the learned initial displacement guess:
// forward, backward (hand-written adjoints) and Adam, float32, on the vertex
// graph of a P1 mesh.  The paper starts each transient solve from the previous
// step's displacement (Sec. 5.3); here the starting guess comes from the load.
//
//   h0   = relu(X W_in + b_in)                               X: [N, 10]
//   for l < 4:  m = mean_{u in N(v)} h_u;  g = mean_v h_v
//               d_k = sum_{u in N(v)} w^k_vu h_u   (k = x, y, z)
//               h = h + relu(h W_s + m W_n + g W_g + d_x W_dx + d_y W_dy + d_z W_dz + b)
//   y    = (h W_out + b_out) * (1 - mask)                    [N, 3]
// with the direction weights w^k_vu = (x_u - x_v)_k / (deg_v l_v), l_v the
// mean length of the edges at v (a first-difference stencil).
//
// Layouts: activations [N][64] row-major, the directional sums [N][3][64];
// parameters one float array in the order W_in[10][64], b_in[64], per layer
// {W_s, W_n, W_g, W_dx, W_dy, W_dz}[64][64], b[64], W_out[64][3], b_out[3]
// (weights [in][out]), so the three directional weights of a layer form one
// [192][64] matrix against the [N][192] sums.
//
// The dense products run on the float32 matrix cores: a layer forward and
// backward is one [N][320] x [320][64] product whose rows are gathered into
// LDS by the workgroup that multiplies them (k_mp_layer), its weight gradient
// one [320][N] x [N][64] product (k_wgrad).  The graph is symmetric, so the
// adjoints of the neighbour mean and of the directional sums are gathers too:
//   dL/dh_u gains (sum_{v in N(u)} ga_v / deg_v) W_n^T
//                 + sum_k (sum_{v in N(u)} w^k_vu ga_v) W_dk^T.
// Sums over the vertices are per-workgroup partials added in a fixed order in
// double: deterministic, no atomics.  A workgroup forms its part of the means,
// of the bias gradients and of the loss in double too, its part of the weight
// gradients in float32 chains whose length does not grow with the mesh
// (WCHAIN).  On 334,368 vertices a training step (forward, backward, Adam) went
// from 22.8 to 4.8 ms.
#include <hip/hip_runtime.h>

#include <cmath>
#include <memory>

#include "te_amg.h"
#include "te_internal.h"

namespace te {

constexpr int MH = 64, ML = 4, MF = 10, MO = 3, MD = 3 * MH;
constexpr int64_t OFF_WIN = 0, OFF_BIN = MF * MH;
constexpr int64_t LAYER0 = OFF_BIN + MH;
constexpr int64_t LAYER_SZ = 6 * MH * MH + MH;
constexpr int64_t OFF_WOUT = LAYER0 + ML * LAYER_SZ;
constexpr int64_t OFF_BOUT = OFF_WOUT + MH * MO;
constexpr int64_t NPARAM = OFF_BOUT + MO;
constexpr float S_T = 500.f, S_F = 2.0e9f, S_X = 0.5f;
constexpr double S_U = 1.0e-3;
constexpr int MB = 256, MW = MB / 64;
constexpr int MK = 5 * MH;        // concatenated layer input: own row, neighbour mean, three directional sums
constexpr int LROW = MK + 4;      // its LDS row, padded so that 16 rows read 16 bytes each without bank conflicts
constexpr int RED_BLOCKS = 512;   // workgroups of the weight-gradient passes, more on meshes beyond 524,288 vertices
constexpr int WCHAIN = 32;        // vertices whose products are added in one float32 chain
constexpr int LAYER_BLOCKS = 768; // workgroups of a layer: the three a CU holds at once (LDS), on 256 CUs

typedef float f32x4 __attribute__((ext_vector_type(4)));

__host__ __device__ constexpr int64_t off_ws(int l) { return LAYER0 + l * LAYER_SZ; }
__host__ __device__ constexpr int64_t off_wn(int l) { return LAYER0 + l * LAYER_SZ + MH * MH; }
__host__ __device__ constexpr int64_t off_wg(int l) { return LAYER0 + l * LAYER_SZ + 2 * MH * MH; }
__host__ __device__ constexpr int64_t off_wd(int l) { return LAYER0 + l * LAYER_SZ + 3 * MH * MH; }
__host__ __device__ constexpr int64_t off_b(int l) { return LAYER0 + l * LAYER_SZ + 6 * MH * MH; }
// weight matrix of slab p of the concatenated layer input
__host__ __device__ constexpr int64_t off_slab(int l, int p) {
    return p == 0 ? off_ws(l) : (p == 1 ? off_wn(l) : off_wd(l) + (p - 2) * MH * MH);
}

__device__ __forceinline__ float lane_val(float v, int k) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k));
}

// The block's double per channel and wave (one value per lane group of 16,
// channel 16 w + lane % 16) into part[blockIdx][64]: the four lanes of a
// channel added in a fixed order.
__device__ __forceinline__ void store_colsum(double cs, double *__restrict__ part) {
    cs += __shfl_xor(cs, 16, 64);
    cs += __shfl_xor(cs, 32, 64);
    const int lane = threadIdx.x & 63, w = threadIdx.x / 64;
    if (lane < 16) part[blockIdx.x * (int64_t)MH + 16 * w + lane] = cs;
}

// ---------------------------------------------------------------------------
// forward
// ---------------------------------------------------------------------------
// features: X[v] = [dT/S_T, f/S_F, mask, xc/S_X]
__global__ void k_features(int64_t n, const double *__restrict__ xc, const double *__restrict__ T, double T_ref,
                           const double *__restrict__ f, const uint8_t *__restrict__ mask, float *__restrict__ X) {
    for (int64_t v = blockIdx.x * (int64_t)MB + threadIdx.x; v < n; v += (int64_t)gridDim.x * MB) {
        float *o = X + v * MF;
        o[0] = float((T[v] - T_ref) / S_T);
        for (int c = 0; c < 3; ++c) {
            o[1 + c] = f ? float(f[v * 3 + c] / S_F) : 0.f;
            o[4 + c] = mask[v * 3 + c] ? 1.f : 0.f;
            o[7 + c] = float(xc[v * 3 + c] / S_X);
        }
    }
}

// h0 = relu(X W_in + b_in), one wave per vertex, lane = channel; the block's
// column sums of h0 for the first layer's mean over the vertices; and the
// handle's copies of X and the mask, which the backward pass reads.
__global__ void __launch_bounds__(MB) k_in(int64_t n, const float *__restrict__ P, const float *__restrict__ X,
                                           const uint8_t *__restrict__ mask, float *__restrict__ Xc,
                                           uint8_t *__restrict__ maskc, float *__restrict__ h0,
                                           double *__restrict__ part) {
    __shared__ double lds[MB];
    const int c = threadIdx.x & 63, w = threadIdx.x / 64;
    float win[MF];
#pragma unroll
    for (int k = 0; k < MF; ++k) win[k] = P[OFF_WIN + k * MH + c];
    const float b = P[OFF_BIN + c];
    double cs = 0.0;
    for (int64_t v = blockIdx.x * (int64_t)MW + w; v < n; v += (int64_t)gridDim.x * MW) {
        const float xv = c < MF ? X[v * MF + c] : 0.f;
        if (c < MF) Xc[v * MF + c] = xv;
        if (c < 3) maskc[v * 3 + c] = mask[v * 3 + c];
        double ad = b;   // added in double: the layers amplify what is rounded here
#pragma unroll
        for (int k = 0; k < MF; ++k) ad += double(lane_val(xv, k)) * win[k];
        const float a = ad > 0.0 ? float(ad) : 0.f;
        h0[v * MH + c] = a;
        cs += a;
    }
    lds[threadIdx.x] = cs;
    __syncthreads();
    if (threadIdx.x < 64) {
        double t = 0.0;
        for (int k = 0; k < MW; ++k) t += lds[k * 64 + threadIdx.x];
        part[blockIdx.x * (int64_t)MH + threadIdx.x] = t;
    }
}

// Sums of the [nparts][64] partials per channel: 16 lane groups take every
// 16th part, their sums are added in order.  Valid in threads 0..63.
constexpr int SB = 1024;
__device__ __forceinline__ double sum_parts64(int nparts, const double *__restrict__ part, double *lds) {
    const int c = threadIdx.x & 63, y = threadIdx.x / 64;
    double s = 0.0;
#pragma unroll 4
    for (int b = y; b < nparts; b += SB / 64) s += part[(int64_t)b * MH + c];
    lds[threadIdx.x] = s;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x < 64)
#pragma unroll
        for (int k = 0; k < SB / 64; ++k) t += lds[k * 64 + threadIdx.x];
    return t;
}

// out[c] = sum_k v[k] M(k, c) over 64 k, the 16 lane groups taking 4 k each;
// M row-major [k][c], or its transpose.  Valid in threads 0..63; v in LDS.
// Added in double: every vertex receives the result, so its rounding does not
// average out.
template <bool TRANS, typename V>
__device__ __forceinline__ double vec_mat64(const V *v, const float *__restrict__ M, double *lds) {
    const int c = threadIdx.x & 63, y = threadIdx.x / 64;
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int k = 4 * y + q;
        t += double(v[k]) * (TRANS ? M[c * MH + k] : M[k * MH + c]);
    }
    lds[threadIdx.x] = t;
    __syncthreads();
    double o = 0.0;
    if (threadIdx.x < 64)
#pragma unroll
        for (int k = 0; k < SB / 64; ++k) o += lds[k * 64 + threadIdx.x];
    return o;
}

// g = colsum/n (from partials), gw = g W_g + b (forward) as two floats, the value
// and what its rounding left; one workgroup
__global__ void __launch_bounds__(SB) k_global(int nparts, const double *__restrict__ part, int64_t n,
                                               const float *__restrict__ P, int l, float *__restrict__ g,
                                               float *__restrict__ gw) {
    __shared__ double lds[SB];
    __shared__ double gs[64];
    const int c = threadIdx.x;
    const double s = sum_parts64(nparts, part, lds);
    if (c < 64) {
        gs[c] = s / double(n);
        g[c] = float(gs[c]);
    }
    __syncthreads();
    const double a = vec_mat64<false>(gs, P + off_wg(l), lds);
    if (c < 64) {
        const double v = P[off_b(l) + c] + a;
        gw[c] = float(v);
        gw[MH + c] = float(v - double(float(v)));
    }
}

// One message-passing layer, forward or backward.  Both are one product of
// the concatenated rows [s | m | d_x | d_y | d_z] (320 wide) with the layer's
// five 64 x 64 matrices:
//   forward   s = h, m = mean of the neighbours' h, d_k = sum_u w^k_vu h_u;
//             a = [..] W + gw,  h' = h + relu(a); m, d and a are kept for the
//             backward pass
//   backward  s = ga, m = sum_u ga_u / deg_u, d_k = sum_u w^k_uv ga_u: the
//             adjoint gathers commute with the transposed matrices, so only
//             the 64 channels of ga are gathered, not the 256 of their images;
//             gh' = gh + [..] W^T + gg / n, then ga' = gh' where the gate of
//             the layer below is open
// A workgroup takes tiles of 16 MT vertices (contiguous, in XCD order: the
// gathered rows of a tile stay in one L2).  Each wave gathers 4 MT of them
// with its 64 lanes on the channels: the wave's neighbour entries are one
// list, each lane looks up one entry's vertex and weights, the rows of 20
// entries are loaded together.  The rows meet in LDS, and each wave multiplies
// them by its 16 output channels' weights, which stay in 80 registers for
// all tiles (v_mfma_f32_16x16x4: lane (q, i) holds channels 16 kb + 4 q + s of
// row i, so one 16-byte LDS read feeds four instructions).
// Bound: 2 * 320 * 64 flop per vertex (0.09 ms on 334,368 vertices at the
// float32 matrix rate) and about 1.5 KB of rows per vertex (0.10 ms); what is
// left is the latency of the gather's dependent loads.  334,368 vertices, per
// layer: forward 1.72 -> 0.40 ms, backward (two kernels) 1.62 -> 0.41 ms, with
// one wave per vertex and vector FMAs before; with the rows of eight entries 0.42
// and 0.44 ms.
template <int MT, bool BWD>
__global__ void __launch_bounds__(MB, 2) k_mp_layer(int64_t n, int64_t ntiles, const int64_t *__restrict__ gp,
                                                    const int32_t *__restrict__ gi, const float *__restrict__ xf,
                                                    const float *__restrict__ invdl, const float *__restrict__ P, int l,
                                                    const float *__restrict__ gvec, const float *__restrict__ src,
                                                    float *__restrict__ mout, float *__restrict__ dout,
                                                    float *__restrict__ aout, const float *__restrict__ gate,
                                                    float *__restrict__ hout, float *__restrict__ gout,
                                                    double *__restrict__ part) {
    constexpr int VT = 16 * MT, VW = VT / MW, EU = 20;
    __shared__ float T[VT][LROW];
    const int lane = threadIdx.x & 63, w = threadIdx.x / 64;
    const int i16 = lane & 15, q = lane >> 4, col = 16 * w + i16;
    float wr[MK / 4];
#pragma unroll
    for (int kb = 0; kb < MK / 16; ++kb) {
        const float *M = P + off_slab(l, kb / 4);
        const int k0 = (kb % 4) * 16 + 4 * q;
#pragma unroll
        for (int t = 0; t < 4; ++t) wr[kb * 4 + t] = BWD ? M[col * MH + k0 + t] : M[(k0 + t) * MH + col];
    }
    // forward: the rounding of gw is the same for every vertex and would not
    // average out, so its remainder goes in first and its value last
    const float gv = BWD ? gvec[col] / float(n) : gvec[MH + col], ghi = BWD ? 0.f : gvec[col];
    double cs = 0.0;
    const int64_t nb = gridDim.x, x = blockIdx.x & 7, xi = blockIdx.x >> 3;
    const int64_t lb = x * (nb >> 3) + (x < (nb & 7) ? x : (nb & 7)) + xi;   // workgroups of one XCD adjacent
    const int64_t t_lo = ntiles * lb / nb, t_hi = ntiles * (lb + 1) / nb;
    for (int64_t tile = t_lo; tile < t_hi; ++tile) {
        const int64_t v0 = tile * VT + w * VW;
        const int r0 = w * VW;
        const int nv = (int)(v0 < n ? (n - v0 < VW ? n - v0 : VW) : 0);   // the wave's vertices inside the mesh
        for (int i = 0; i < VW; ++i) T[r0 + i][lane] = i < nv ? src[(v0 + i) * MH + lane] : 0.f;
        const int64_t e0 = nv > 0 ? gp[v0] : 0;
        // lane i: end of vertex i's entries in the wave's list
        int pe = 0;
        if (nv > 0) pe = (int)(gp[v0 + (lane + 1 < nv ? lane + 1 : nv)] - e0);
        const int tot = __builtin_amdgcn_readlane(pe, VW - 1);
        int cur = 0, beg = 0, end = __builtin_amdgcn_readlane(pe, 0);
        float s = 0.f, d0 = 0.f, d1 = 0.f, d2 = 0.f;
        auto flush = [&]() {
            const float m = BWD ? s : (end > beg ? s / float(end - beg) : 0.f);
            float *row = T[r0 + cur];
            row[MH + lane] = m;
            row[2 * MH + lane] = d0;
            row[3 * MH + lane] = d1;
            row[4 * MH + lane] = d2;
            if (!BWD && cur < nv) {
                const int64_t v = v0 + cur;
                mout[v * MH + lane] = m;
                dout[v * MD + lane] = d0;
                dout[v * MD + MH + lane] = d1;
                dout[v * MD + 2 * MH + lane] = d2;
            }
            s = d0 = d1 = d2 = 0.f;
            ++cur;
            beg = end;
            end = cur < VW ? __builtin_amdgcn_readlane(pe, cur) : tot;
        };
        for (int c0 = 0; c0 < tot; c0 += 64) {
            const int e = c0 + lane, cnt = tot - c0 < 64 ? tot - c0 : 64;
            int u = 0;
            float w0 = 0.f, w1 = 0.f, w2 = 0.f, wm = 1.f;
            int vi = 0;   // the vertex an entry belongs to
#pragma unroll
            for (int i = 0; i + 1 < VW; ++i) vi += e >= __builtin_amdgcn_readlane(pe, i) ? 1 : 0;
            if (e < tot) {
                u = gi[e0 + e];
                const int64_t v = v0 + vi;
                const float *xu = xf + (int64_t)u * 3, *xv = xf + v * 3;
                if (BWD) {
                    const float iu = invdl[u];
                    w0 = (xv[0] - xu[0]) * iu;
                    w1 = (xv[1] - xu[1]) * iu;
                    w2 = (xv[2] - xu[2]) * iu;
                    const int64_t du = gp[u + 1] - gp[u];
                    wm = du > 0 ? 1.f / float(du) : 0.f;
                } else {
                    const float iv = invdl[v];
                    w0 = (xu[0] - xv[0]) * iv;
                    w1 = (xu[1] - xv[1]) * iv;
                    w2 = (xu[2] - xv[2]) * iv;
                }
            }
            for (int b = 0; b < cnt; b += EU) {
                float hr[EU];
#pragma unroll
                for (int t = 0; t < EU; ++t) {
                    const int k = b + t < cnt ? b + t : cnt - 1;
                    hr[t] = src[(int64_t)__builtin_amdgcn_readlane(u, k) * MH + lane];
                }
#pragma unroll
                for (int t = 0; t < EU; ++t) {
                    if (b + t >= cnt) break;
                    while (c0 + b + t >= end) flush();
                    if (BWD) s += lane_val(wm, b + t) * hr[t];
                    else s += hr[t];
                    d0 += lane_val(w0, b + t) * hr[t];
                    d1 += lane_val(w1, b + t) * hr[t];
                    d2 += lane_val(w2, b + t) * hr[t];
                }
            }
        }
        while (cur < VW) flush();
        __syncthreads();
        // a slab's 64 terms in a sum of their own: shorter float32 sums than one
        // over all 320 (relative error of the network's output 2.3e-7 -> 1.5e-7)
        f32x4 acc[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[m][r] = gv;
#pragma unroll
        for (int p = 0; p < MK / MH; ++p) {
            f32x4 sl[MT] = {};
#pragma unroll
            for (int kb = p * (MH / 16); kb < (p + 1) * (MH / 16); ++kb)
#pragma unroll
                for (int m = 0; m < MT; ++m) {
                    const f32x4 a = *reinterpret_cast<const f32x4 *>(&T[16 * m + i16][16 * kb + 4 * q]);
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        sl[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t], wr[kb * 4 + t], sl[m], 0, 0, 0);
                }
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[m] += sl[m];
        }
        if (!BWD)
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[m] += ghi;
        // lane (q, i) holds rows 4 q + r of channel col
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * m + 4 * q + r;
                const int64_t v = tile * VT + row;
                if (v >= n) continue;
                const int64_t o = v * MH + col;
                const float av = acc[m][r];
                if (BWD) {
                    const float gh = hout[o] + av;
                    const float ga = gate[o] > 0.f ? gh : 0.f;
                    hout[o] = gh;
                    gout[o] = ga;
                    cs += ga;
                } else {
                    const float hv = T[row][col] + (av > 0.f ? av : 0.f);
                    aout[o] = av;
                    hout[o] = hv;
                    cs += hv;
                }
            }
        __syncthreads();   // the next tile overwrites T
    }
    store_colsum(cs, part);
}

// The output layer's rows: four lanes per vertex, lane j of them the 16
// channels 16 i + 4 j + r.  hv[4 i + r] and the three weights of each.
constexpr int OV = MB / 4;   // vertices per workgroup step
__device__ __forceinline__ void out_weights(const float *__restrict__ P, int j, float (&wo)[16][MO]) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < MO; ++c) wo[4 * i + r][c] = P[OFF_WOUT + (16 * i + 4 * j + r) * MO + c];
}
__device__ __forceinline__ void load_row16(const float *__restrict__ h, int64_t v, int j, float (&hv)[16]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const f32x4 t = *reinterpret_cast<const f32x4 *>(h + v * MH + 16 * i + 4 * j);
#pragma unroll
        for (int r = 0; r < 4; ++r) hv[4 * i + r] = t[r];
    }
}

// y = (h W_out + b_out) * keep, into the handle's copy and, if given, the caller's
__global__ void __launch_bounds__(MB) k_out(int64_t n, const float *__restrict__ P, const float *__restrict__ h,
                                            const uint8_t *__restrict__ mask, float *__restrict__ y,
                                            float *__restrict__ yuser) {
    const int j = threadIdx.x & 3;
    float wo[16][MO];
    out_weights(P, j, wo);
    for (int64_t v = blockIdx.x * (int64_t)OV + threadIdx.x / 4; v < n; v += (int64_t)gridDim.x * OV) {
        float hv[16];
        double t[MO] = {0.0, 0.0, 0.0};   // the kernel is bound by the rows: the sums cost nothing in double
        load_row16(h, v, j, hv);
#pragma unroll
        for (int k = 0; k < 16; ++k)
#pragma unroll
            for (int c = 0; c < MO; ++c) t[c] += double(hv[k]) * wo[k][c];
#pragma unroll
        for (int c = 0; c < MO; ++c) {
            t[c] += __shfl_xor(t[c], 1, 64);
            t[c] += __shfl_xor(t[c], 2, 64);
        }
        if (j < MO) {
            const float o = float((j == 0 ? t[0] : (j == 1 ? t[1] : t[2])) + P[OFF_BOUT + j]);
            const float yv = mask[v * 3 + j] ? o * 0.f : o;
            y[v * MO + j] = yv;
            if (yuser) yuser[v * MO + j] = yv;
        }
    }
}

// ---------------------------------------------------------------------------
// backward
// ---------------------------------------------------------------------------
// dL/dy (MSE against a target: 2 (y - t) / 3n; or given) with constrained
// entries zero, gh = gy W_out^T, ga = gh where the last layer's gate a is open;
// per block: the loss, the output layer's gradients (64 x 3 float partials at
// wpart, the three of the bias in double at bpart) and the column sums of ga.
// Lanes as in k_out.
constexpr int OPART = MH * MO;
template <bool MSE>
__global__ void __launch_bounds__(MB) k_out_bwd(int64_t n, const float *__restrict__ P, const float *__restrict__ h,
                                                const float *__restrict__ a, const uint8_t *__restrict__ mask,
                                                const float *__restrict__ y, const float *__restrict__ in,
                                                float *__restrict__ gh, float *__restrict__ ga,
                                                double *__restrict__ lpart, double *__restrict__ part,
                                                float *__restrict__ wpart, double *__restrict__ bpart) {
    __shared__ double s_cs[MW][MH], s_l[MW], s_b[MW][MO];
    __shared__ float s_w[MW][OPART];
    const int j = threadIdx.x & 3, lane = threadIdx.x & 63, w = threadIdx.x / 64;
    float wo[16][MO], gw[16][MO];
    double cs[16], gb[MO] = {0.0, 0.0, 0.0}, ls = 0.0;
    out_weights(P, j, wo);
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        cs[k] = 0.0;
#pragma unroll
        for (int c = 0; c < MO; ++c) gw[k][c] = 0.f;
    }
    const float inv = 2.f / float(3 * n);
    for (int64_t v = blockIdx.x * (int64_t)OV + threadIdx.x / 4; v < n; v += (int64_t)gridDim.x * OV) {
        float hv[16], av[16], g[MO];
        load_row16(h, v, j, hv);
        load_row16(a, v, j, av);
#pragma unroll
        for (int c = 0; c < MO; ++c) {
            const bool keep = mask[v * 3 + c] == 0;
            if (MSE) {
                const float d = y[v * MO + c] - in[v * MO + c];
                if (j == 0) ls += double(d) * double(d);
                g[c] = keep ? inv * d : 0.f;
            } else {
                g[c] = keep ? in[v * MO + c] : 0.f;
            }
            gb[c] += g[c];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f32x4 t, u;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int k = 4 * i + r;
                float x = 0.f;
#pragma unroll
                for (int c = 0; c < MO; ++c) {
                    x += g[c] * wo[k][c];
                    gw[k][c] += hv[k] * g[c];
                }
                t[r] = x;
                u[r] = av[k] > 0.f ? x : 0.f;
                cs[k] += u[r];
            }
            *reinterpret_cast<f32x4 *>(gh + v * MH + 16 * i + 4 * j) = t;
            *reinterpret_cast<f32x4 *>(ga + v * MH + 16 * i + 4 * j) = u;
        }
    }
    // the wave's 16 vertices in a fixed tree, then the waves in order
#pragma unroll
    for (int o = 4; o < 64; o <<= 1) {
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            cs[k] += __shfl_xor(cs[k], o, 64);
#pragma unroll
            for (int c = 0; c < MO; ++c) gw[k][c] += __shfl_xor(gw[k][c], o, 64);
        }
#pragma unroll
        for (int c = 0; c < MO; ++c) gb[c] += __shfl_xor(gb[c], o, 64);
        ls += __shfl_xor(ls, o, 64);
    }
    if (lane < 4) {
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int ch = 16 * (k / 4) + 4 * j + k % 4;
            s_cs[w][ch] = cs[k];
#pragma unroll
            for (int c = 0; c < MO; ++c) s_w[w][ch * MO + c] = gw[k][c];
        }
        if (j == 0) {
            s_l[w] = ls;
#pragma unroll
            for (int c = 0; c < MO; ++c) s_b[w][c] = gb[c];
        }
    }
    __syncthreads();
    const int t = threadIdx.x;
    if (t < MH) {
        double v = 0.0;
        for (int k = 0; k < MW; ++k) v += s_cs[k][t];
        part[blockIdx.x * (int64_t)MH + t] = v;
    }
    if (t < OPART) {
        float v = 0.f;
        for (int k = 0; k < MW; ++k) v += s_w[k][t];
        wpart[blockIdx.x * (int64_t)OPART + t] = v;
    }
    if (t < MO) {
        double v = 0.0;
        for (int k = 0; k < MW; ++k) v += s_b[k][t];
        bpart[blockIdx.x * (int64_t)MO + t] = v;
    }
    if (MSE && t == 0) {
        double v = 0.0;
        for (int k = 0; k < MW; ++k) v += s_l[k];
        lpart[blockIdx.x] = v;
    }
}

// Weight gradients of a layer, partial over a chunk of vertices:
//   part[b][k][c] = sum_v [h | m | d](v, k) ga(v, c),  k < 320, c < 64
// A wave holds 80 of the 320 rows (20 MFMA tiles of 16 x 16 in 80 registers);
// four vertices per v_mfma_f32_16x16x4, operands straight from global memory
// (16 channels of four rows: 64-byte pieces), two steps in flight.  The tiles
// are closed every WCHAIN vertices and added to 80 registers of their own, and a
// chunk has at most WCHAIN of these chains, so no float32 sum has more than 64
// steps; as one chain per chunk, vertices of equal sign were off by 157 units of
// the last place at 334,368 and by 691 at 1,500,001, now by 12 and 14.
// Bound: the float32 matrix rate and the rows, 0.09 and 0.10 ms per layer on
// 334,368 vertices; 1.31 (three LDS-tiled vector products) -> 0.28 ms, of which
// the second set of registers takes 0.006.
__global__ void __launch_bounds__(MB, 2) k_wgrad(int64_t n, const float *__restrict__ h, const float *__restrict__ m,
                                                 const float *__restrict__ d, const float *__restrict__ ga,
                                                 float *__restrict__ part) {
    constexpr int MTW = MK / 16 / MW;   // row tiles per wave
    const int lane = threadIdx.x & 63, w = threadIdx.x / 64, i16 = lane & 15, q = lane >> 4;
    const float *base[MTW];
    int ld[MTW];
#pragma unroll
    for (int t = 0; t < MTW; ++t) {
        const int tile = w * MTW + t, slab = tile / 4, c0 = (tile % 4) * 16;
        base[t] = (slab == 0 ? h : (slab == 1 ? m : d + (slab - 2) * MH)) + c0 + i16;
        ld[t] = slab < 2 ? MH : MD;
    }
    f32x4 sum[MTW][4];
#pragma unroll
    for (int t = 0; t < MTW; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c) sum[t][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int64_t chunk = ((n + gridDim.x - 1) / gridDim.x + 3) / 4 * 4;
    const int64_t lo = blockIdx.x * chunk, hi = lo + chunk < n ? lo + chunk : n;
    auto load = [&](int64_t r, float (&x)[MTW], float (&g)[4]) {
        const int64_t v = r + q;
        const bool ok = v < hi;
        const int64_t vv = ok ? v : lo;   // inside the chunk
#pragma unroll
        for (int t = 0; t < MTW; ++t) {
            const float z = base[t][vv * ld[t]];
            x[t] = ok ? z : 0.f;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float z = ga[vv * MH + 16 * c + i16];
            g[c] = ok ? z : 0.f;
        }
    };
    if (lo < hi) {
        float x0[MTW], g0[4], x1[MTW], g1[4];
        load(lo, x0, g0);
        for (int64_t r = lo; r < hi;) {
            f32x4 acc[MTW][4];   // a chain of at most WCHAIN vertices
#pragma unroll
            for (int t = 0; t < MTW; ++t)
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[t][c] = f32x4{0.f, 0.f, 0.f, 0.f};
            const int64_t end = r + WCHAIN < hi ? r + WCHAIN : hi;
            for (; r < end; r += 8) {
                load(r + 4, x1, g1);   // past the chunk: zeros
#pragma unroll
                for (int t = 0; t < MTW; ++t)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(x0[t], g0[c], acc[t][c], 0, 0, 0);
                load(r + 8, x0, g0);
#pragma unroll
                for (int t = 0; t < MTW; ++t)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(x1[t], g1[c], acc[t][c], 0, 0, 0);
            }
#pragma unroll
            for (int t = 0; t < MTW; ++t)
#pragma unroll
                for (int c = 0; c < 4; ++c) sum[t][c] += acc[t][c];
        }
    }
    float *o = part + blockIdx.x * (int64_t)(MK * MH);
#pragma unroll
    for (int t = 0; t < MTW; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) o[((w * MTW + t) * 16 + 4 * q + r) * MH + 16 * c + i16] = sum[t][c][r];
}

// The same for the input layer: part[b][k][c] = sum_v X(v, k) ga(v, c),
// k < 10; one 16-row tile, the waves take every fourth step of four vertices.
__global__ void __launch_bounds__(MB) k_wgrad_in(int64_t n, const float *__restrict__ X, const float *__restrict__ ga,
                                                 float *__restrict__ part) {
    __shared__ float s_w[MW][MF * MH];
    const int lane = threadIdx.x & 63, w = threadIdx.x / 64, i16 = lane & 15, q = lane >> 4;
    f32x4 sum[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) sum[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int64_t chunk = ((n + gridDim.x - 1) / gridDim.x + 15) / 16 * 16;
    const int64_t lo = blockIdx.x * chunk, hi = lo + chunk < n ? lo + chunk : n;
    for (int64_t r = lo + 4 * w; r < hi;) {
        f32x4 acc[4];   // a chain of at most WCHAIN vertices
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < WCHAIN / 4; ++t, r += 4 * MW) {
            const int64_t v = r + q;
            const bool ok = v < hi;   // past the chunk: zeros
            const int64_t vv = ok ? v : lo;
            const float z = X[vv * MF + (i16 < MF ? i16 : 0)];
            const float x = ok && i16 < MF ? z : 0.f;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float y = ga[vv * MH + 16 * c + i16];
                acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, ok ? y : 0.f, acc[c], 0, 0, 0);
            }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) sum[c] += acc[c];
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (4 * q + r < MF) s_w[w][(4 * q + r) * MH + 16 * c + i16] = sum[c][r];
    __syncthreads();
    for (int e = threadIdx.x; e < MF * MH; e += MB) {
        float t = 0.f;
        for (int k = 0; k < MW; ++k) t += s_w[k][e];
        part[blockIdx.x * (int64_t)(MF * MH) + e] = t;
    }
}

// Sums over the parts of nel-element partial tables, in double: a workgroup
// takes 64 elements, its four waves a quarter of the parts each (in order),
// the quarters added in order.  The sum of element e goes to out(e).
template <typename T, class Out>
__device__ __forceinline__ void sum_table(int nparts, int nel, const T *__restrict__ part, int block, Out out) {
    __shared__ double lds[MW][64];
    const int lane = threadIdx.x & 63, y = threadIdx.x / 64;
    const int e = block * 64 + lane;
    const int b0 = nparts * y / MW, b1 = nparts * (y + 1) / MW;
    double s = 0.0;
    if (e < nel)
#pragma unroll 8
        for (int b = b0; b < b1; ++b) s += part[(int64_t)b * nel + e];
    lds[y][lane] = s;
    __syncthreads();
    if (y == 0 && e < nel) {
        double t = 0.0;
#pragma unroll
        for (int k = 0; k < MW; ++k) t += lds[k][lane];
        out(e, t);
    }
}
__global__ void __launch_bounds__(MB) k_sum_parts(int nparts, int nel, const float *__restrict__ part,
                                                  float *__restrict__ out) {
    sum_table(nparts, nel, part, blockIdx.x, [&](int e, double t) { out[e] = float(t); });
}
// the output layer's tables: the last workgroup takes the bias
__global__ void __launch_bounds__(MB) k_sum_out(int nparts, const float *__restrict__ wpart,
                                                const double *__restrict__ bpart, float *__restrict__ grad) {
    if (blockIdx.x < OPART / 64)
        sum_table(nparts, OPART, wpart, blockIdx.x, [&](int e, double t) { grad[OFF_WOUT + e] = float(t); });
    else
        sum_table(nparts, MO, bpart, 0, [&](int e, double t) { grad[OFF_BOUT + e] = float(t); });
}
// the [320][64] table of a layer to its five matrices
__global__ void __launch_bounds__(MB) k_sum_layer(int nparts, const float *__restrict__ part, int l,
                                                  float *__restrict__ grad) {
    sum_table(nparts, MK * MH, part, blockIdx.x, [&](int e, double t) {
        grad[off_slab(l, e / (MH * MH)) + e % (MH * MH)] = float(t);
    });
}

// layer scalars: gb = colsum(ga); gW_g = g^T gb (outer product); gg = gb W_g^T
__global__ void __launch_bounds__(SB) k_layer_small(int nparts, const double *__restrict__ part,
                                                    const float *__restrict__ g, const float *__restrict__ P, int l,
                                                    float *__restrict__ grad, float *__restrict__ gg) {
    __shared__ double lds[SB];
    __shared__ float gb[64];
    const int c = threadIdx.x;
    const double s = sum_parts64(nparts, part, lds);
    if (c < 64) {
        gb[c] = float(s);
        grad[off_b(l) + c] = gb[c];
    }
    __syncthreads();
    for (int t = threadIdx.x; t < MH * MH; t += SB) grad[off_wg(l) + t] = g[t / MH] * gb[t % MH];
    const double t = vec_mat64<true>(gb, P + off_wg(l), lds);
    if (c < 64) gg[c] = float(t);
}

// the input layer's bias gradient from partial column sums
__global__ void __launch_bounds__(SB) k_colsum_out(int nparts, const double *__restrict__ part,
                                                   float *__restrict__ out) {
    __shared__ double lds[SB];
    const double s = sum_parts64(nparts, part, lds);
    if (threadIdx.x < 64) out[threadIdx.x] = float(s);
}

// u = S_U y * keep, u_t = S_U t  (float64, natural order)
__global__ void k_energy_prep(int64_t n, const float *__restrict__ y, const float *__restrict__ t,
                              const uint8_t *__restrict__ mask, double *__restrict__ u, double *__restrict__ ut) {
    for (int64_t i = blockIdx.x * (int64_t)MB + threadIdx.x; i < n * 3; i += (int64_t)gridDim.x * MB) {
        u[i] = mask[i] ? 0.0 : S_U * double(y[i]);
        ut[i] = S_U * double(t[i]);
    }
}
// gy = keep * (ca * A u_t + cb * A u)  (float)
__global__ void k_energy_gy(int64_t n, const double *__restrict__ Aut, const double *__restrict__ Au,
                            const uint8_t *__restrict__ mask, double ca, double cb, float *__restrict__ gy) {
    for (int64_t i = blockIdx.x * (int64_t)MB + threadIdx.x; i < n * 3; i += (int64_t)gridDim.x * MB)
        gy[i] = mask[i] ? 0.f : float(ca * Aut[i] + cb * Au[i]);
}

// Adam (Kingma & Ba 2015) with bias correction
__global__ void k_adam(int64_t n, float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                       float *__restrict__ v, float lr, float b1, float b2, float eps, float c1, float c2) {
    for (int64_t i = blockIdx.x * (int64_t)MB + threadIdx.x; i < n; i += (int64_t)gridDim.x * MB) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.f - b1) * gi;
        const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    }
}

__global__ void k_guess(int64_t n, const float *__restrict__ y, double *__restrict__ u0) {
    for (int64_t t = blockIdx.x * (int64_t)MB + threadIdx.x; t < n * 3; t += (int64_t)gridDim.x * MB)
        u0[t] = S_U * double(y[t]);
}

// 1 / (deg_v l_v), l_v the mean length of the edges at v (0 without edges)
__global__ void k_invdl(int64_t n, const int64_t *__restrict__ gp, const int32_t *__restrict__ gi,
                        const double *__restrict__ xc, float *__restrict__ invdl, float *__restrict__ xf) {
    for (int64_t v = blockIdx.x * (int64_t)MB + threadIdx.x; v < n; v += (int64_t)gridDim.x * MB) {
        double len = 0.0;
        for (int64_t e = gp[v]; e < gp[v + 1]; ++e) {
            const int64_t u = gi[e];
            const double a = xc[u * 3] - xc[v * 3], b = xc[u * 3 + 1] - xc[v * 3 + 1], c = xc[u * 3 + 2] - xc[v * 3 + 2];
            len += sqrt(a * a + b * b + c * c);
        }
        const int64_t deg = gp[v + 1] - gp[v];
        invdl[v] = deg > 0 && len > 0.0 ? float(1.0 / len) : 0.f;   // 1 / (deg * (len / deg))
        for (int k = 0; k < 3; ++k) xf[v * 3 + k] = float(xc[v * 3 + k]);
    }
}

// vertex graph = stiffness pattern without the diagonal
__global__ void k_graph_count(int64_t n, const int64_t *__restrict__ rp, const int32_t *__restrict__ ci,
                              int32_t *__restrict__ cnt) {
    for (int64_t v = blockIdx.x * (int64_t)MB + threadIdx.x; v < n; v += (int64_t)gridDim.x * MB) {
        int c = 0;
        for (int64_t e = rp[v]; e < rp[v + 1]; ++e) c += ci[e] != v;
        cnt[v] = c;
    }
}
__global__ void k_graph_fill(int64_t n, const int64_t *__restrict__ rp, const int32_t *__restrict__ ci,
                             const int64_t *__restrict__ gp, int32_t *__restrict__ gi) {
    for (int64_t v = blockIdx.x * (int64_t)MB + threadIdx.x; v < n; v += (int64_t)gridDim.x * MB) {
        int64_t o = gp[v];
        for (int64_t e = rp[v]; e < rp[v + 1]; ++e)
            if (ci[e] != v) gi[o++] = ci[e];
    }
}

}  // namespace te

// ---------------------------------------------------------------------------
// handle and C ABI
// ---------------------------------------------------------------------------
struct mpnn_handle {
    int64_t n = 0;
    te::DBuf<int64_t> gp;
    te::DBuf<int32_t> gi;
    te::DBuf<double> xc;  // centred coordinates
    te::DBuf<float> xf, invdl;  // float centred coordinates, 1 / (deg l) per vertex
    te::DBuf<float> h[te::ML + 1], m[te::ML], d[te::ML], a[te::ML], g[te::ML], gw;
    te::DBuf<float> y, gh, ga[2], gg, part;
    te::DBuf<double> dpart, lpart, bpart;
    te::DBuf<float> X;     // last forward input (borrowed copy)
    te::DBuf<uint8_t> mask;
    bool have_forward = false;
};

using namespace te;

// Workgroups of the weight-gradient and output passes: 64 vertices each at
// least, and 1024 (WCHAIN chains of WCHAIN) at most
static int nparts_for(int64_t n) {
    const int64_t most = std::max<int64_t>(RED_BLOCKS, (n + WCHAIN * WCHAIN - 1) / (WCHAIN * WCHAIN));
    return (int)std::max<int64_t>(1, std::min<int64_t>(most, (n + 63) / 64));
}

extern "C" int64_t mpnn_param_count(void) { return NPARAM; }

extern "C" int mpnn_create(int64_t n, const int64_t *row_ptr, const int32_t *col_idx, const double *coords,
                           mpnn_handle **out, hipStream_t s) {
    return guarded([&] {
        TE_REQUIRE(n > 0 && row_ptr && col_idx && coords && out, TE_EINVAL, "bad argument");
        auto H = std::make_unique<mpnn_handle>();
        H->n = n;
        DBuf<int32_t> cnt(n);
        const unsigned g = (unsigned)std::min<int64_t>((n + MB - 1) / MB, 65536);
        hipLaunchKernelGGL(k_graph_count, dim3(g), dim3(MB), 0, s, n, row_ptr, col_idx, cnt.p);
        TE_CHECK_HIP(hipGetLastError());
        std::vector<int32_t> hc;
        download(hc, cnt.p, n, s);
        std::vector<int64_t> gp(n + 1, 0);
        for (int64_t v = 0; v < n; ++v) gp[v + 1] = gp[v] + hc[v];
        upload(H->gp, gp, s);
        H->gi.alloc(std::max<int64_t>(gp[n], 1));
        hipLaunchKernelGGL(k_graph_fill, dim3(g), dim3(MB), 0, s, n, row_ptr, col_idx, H->gp.p, H->gi.p);
        TE_CHECK_HIP(hipGetLastError());
        std::vector<double> X;
        download(X, coords, n * 3, s);
        double c[3] = {0, 0, 0};
        for (int64_t v = 0; v < n; ++v)
            for (int k = 0; k < 3; ++k) c[k] += X[v * 3 + k];
        for (int k = 0; k < 3; ++k) c[k] /= double(n);
        for (int64_t v = 0; v < n; ++v)
            for (int k = 0; k < 3; ++k) X[v * 3 + k] -= c[k];
        upload(H->xc, X, s);
        H->xf.alloc(n * 3);
        H->invdl.alloc(n);
        hipLaunchKernelGGL(k_invdl, dim3(g), dim3(MB), 0, s, n, H->gp.p, H->gi.p, H->xc.p, H->invdl.p, H->xf.p);
        TE_CHECK_HIP(hipGetLastError());
        for (int l = 0; l <= ML; ++l) H->h[l].alloc(n * MH);
        for (int l = 0; l < ML; ++l) {
            H->m[l].alloc(n * MH);
            H->d[l].alloc(n * MD);
            H->a[l].alloc(n * MH);
            H->g[l].alloc(MH);
        }
        H->gw.alloc(2 * MH);
        H->y.alloc(n * MO);
        H->gh.alloc(n * MH);
        for (auto &b : H->ga) b.alloc(n * MH);
        H->gg.alloc(MH);
        const size_t np = nparts_for(n);
        H->part.alloc(np * MK * MH);
        H->dpart.alloc(std::max<size_t>(LAYER_BLOCKS, np) * MH);
        H->lpart.alloc(np);
        H->bpart.alloc(np * MO);
        H->X.alloc(n * MF);
        H->mask.alloc(n * 3);
        TE_CHECK_HIP(hipStreamSynchronize(s));
        *out = H.release();
        return TE_OK;
    });
}

extern "C" int mpnn_destroy(mpnn_handle *h) {
    delete h;
    return TE_OK;
}

extern "C" int mpnn_features(mpnn_handle *H, const double *T, double T_ref, const double *f, const uint8_t *mask,
                             float *X, hipStream_t s) {
    return guarded([&] {
        TE_REQUIRE(H && T && mask && X, TE_EINVAL, "bad argument");
        const unsigned g = (unsigned)std::min<int64_t>((H->n + MB - 1) / MB, 65536);
        hipLaunchKernelGGL(k_features, dim3(g), dim3(MB), 0, s, H->n, H->xc.p, T, T_ref, f, mask, X);
        TE_CHECK_HIP(hipGetLastError());
        return TE_OK;
    });
}

// Tiles of 32 vertices; of 16 while tiles of 32 would leave some of the
// LAYER_BLOCKS workgroups without one.  Forward and backward pass with tiles of 16
// and of 32: 4,624 vertices 81, 206 and 98, 219 us; 8,648: 104, 243 and 122, 256;
// 23,808: 166, 353 and 169, 358; 15,600, where 975 tiles of 16 leave some
// workgroups with a second one: 150, 304 and 138, 285.
static bool wide_tiles(int64_t n) { return (n + 31) / 32 > LAYER_BLOCKS; }
static int layer_blocks(int64_t n) {
    const int64_t nt = wide_tiles(n) ? (n + 31) / 32 : (n + 15) / 16;
    return (int)std::max<int64_t>(1, std::min<int64_t>(nt, LAYER_BLOCKS));
}
template <bool BWD>
static void launch_layer(mpnn_handle *H, const float *P, int l, const float *gvec, const float *src, float *m, float *d,
                         float *a, const float *gate, float *hout, float *gout, hipStream_t s) {
    const int64_t n = H->n;
    const dim3 g(layer_blocks(n));
    if (wide_tiles(n))
        hipLaunchKernelGGL((k_mp_layer<2, BWD>), g, dim3(MB), 0, s, n, (n + 31) / 32, H->gp.p, H->gi.p, H->xf.p,
                           H->invdl.p, P, l, gvec, src, m, d, a, gate, hout, gout, H->dpart.p);
    else
        hipLaunchKernelGGL((k_mp_layer<1, BWD>), g, dim3(MB), 0, s, n, (n + 15) / 16, H->gp.p, H->gi.p, H->xf.p,
                           H->invdl.p, P, l, gvec, src, m, d, a, gate, hout, gout, H->dpart.p);
}

extern "C" int mpnn_forward(mpnn_handle *H, const float *P, const float *X, const uint8_t *mask, float *y,
                            hipStream_t s) {
    return guarded([&] {
        TE_REQUIRE(H && P && X && mask, TE_EINVAL, "bad argument");
        const int64_t n = H->n;
        const int gi = (int)std::min<int64_t>((n + MW - 1) / MW, LAYER_BLOCKS);
        hipLaunchKernelGGL(k_in, dim3(gi), dim3(MB), 0, s, n, P, X, mask, H->X.p, H->mask.p, H->h[0].p, H->dpart.p);
        int np = gi;
        for (int l = 0; l < ML; ++l) {
            hipLaunchKernelGGL(k_global, dim3(1), dim3(SB), 0, s, np, H->dpart.p, n, P, l, H->g[l].p, H->gw.p);
            launch_layer<false>(H, P, l, H->gw.p, H->h[l].p, H->m[l].p, H->d[l].p, H->a[l].p, nullptr, H->h[l + 1].p,
                                nullptr, s);
            np = layer_blocks(n);
        }
        hipLaunchKernelGGL(k_out, dim3((unsigned)std::min<int64_t>((n + OV - 1) / OV, 4096)), dim3(MB), 0, s, n, P,
                           H->h[ML].p, H->mask.p, H->y.p, y == H->y.p ? nullptr : y);
        TE_CHECK_HIP(hipGetLastError());
        H->have_forward = true;
        return TE_OK;
    });
}

// Backward pass after the output layer's (gh, ga of the last layer and its
// column sums from np workgroups are in the handle).
static void backward_tail(mpnn_handle *H, const float *P, float *grad, int np, hipStream_t s) {
    const int64_t n = H->n;
    const int nw = nparts_for(n);
    hipLaunchKernelGGL(k_sum_out, dim3(OPART / 64 + 1), dim3(MB), 0, s, np, H->part.p, H->bpart.p, grad);
    int cur = 0;
    for (int l = ML - 1; l >= 0; --l) {
        hipLaunchKernelGGL(k_layer_small, dim3(1), dim3(SB), 0, s, np, H->dpart.p, H->g[l].p, P, l, grad, H->gg.p);
        hipLaunchKernelGGL(k_wgrad, dim3(nw), dim3(MB), 0, s, n, H->h[l].p, H->m[l].p, H->d[l].p, H->ga[cur].p,
                           H->part.p);
        hipLaunchKernelGGL(k_sum_layer, dim3(MK * MH / 64), dim3(MB), 0, s, nw, H->part.p, l, grad);
        // the gate of the layer below; the input layer's is h0 > 0
        launch_layer<true>(H, P, l, H->gg.p, H->ga[cur].p, nullptr, nullptr, nullptr,
                           l > 0 ? H->a[l - 1].p : H->h[0].p, H->gh.p, H->ga[cur ^ 1].p, s);
        np = layer_blocks(n);
        cur ^= 1;
    }
    hipLaunchKernelGGL(k_wgrad_in, dim3(nw), dim3(MB), 0, s, n, H->X.p, H->ga[cur].p, H->part.p);
    hipLaunchKernelGGL(k_sum_parts, dim3((MF * MH + 63) / 64), dim3(MB), 0, s, nw, MF * MH, H->part.p, grad + OFF_WIN);
    hipLaunchKernelGGL(k_colsum_out, dim3(1), dim3(SB), 0, s, np, H->dpart.p, grad + OFF_BIN);
    TE_CHECK_HIP(hipGetLastError());
}

// Loss of the last forward against target (scaled displacement [N][3]) and
// gradients of every parameter into grad[NPARAM].
extern "C" int mpnn_backward(mpnn_handle *H, const float *P, const float *target, float *grad, double *loss,
                             hipStream_t s) {
    return guarded([&] {
        TE_REQUIRE(H && P && target && grad, TE_EINVAL, "bad argument");
        TE_REQUIRE(H->have_forward, TE_EINVAL, "mpnn_backward needs a preceding mpnn_forward");
        const int64_t n = H->n;
        const int np = nparts_for(n);
        hipLaunchKernelGGL(k_out_bwd<true>, dim3(np), dim3(MB), 0, s, n, P, H->h[ML].p, H->a[ML - 1].p, H->mask.p,
                           H->y.p, target, H->gh.p, H->ga[0].p, H->lpart.p, H->dpart.p, H->part.p,
                           H->bpart.p);
        TE_CHECK_HIP(hipGetLastError());
        backward_tail(H, P, grad, np, s);
        std::vector<double> lp;
        download(lp, H->lpart.p, np, s);
        double L = 0.0;
        for (double v : lp) L += v;
        if (loss) *loss = L / double(3 * n);
        return TE_OK;
    });
}

// Gradients of a loss given dL/dy of the last forward (float [N][3]).
extern "C" int mpnn_backward_from(mpnn_handle *H, const float *P, const float *gy, float *grad, hipStream_t s) {
    return guarded([&] {
        TE_REQUIRE(H && P && gy && grad, TE_EINVAL, "bad argument");
        TE_REQUIRE(H->have_forward, TE_EINVAL, "mpnn_backward_from needs a preceding mpnn_forward");
        const int np = nparts_for(H->n);
        hipLaunchKernelGGL(k_out_bwd<false>, dim3(np), dim3(MB), 0, s, H->n, P, H->h[ML].p, H->a[ML - 1].p, H->mask.p,
                           H->y.p, gy, H->gh.p, H->ga[0].p, H->lpart.p, H->dpart.p, H->part.p,
                           H->bpart.p);
        TE_CHECK_HIP(hipGetLastError());
        backward_tail(H, P, grad, np, s);
        return TE_OK;
    });
}

// Relative energy error of the energy-optimally scaled guess of the last
// forward: loss = 1 - c^2 / (a e) with u = S_U y (constrained DOFs zero),
// t = S_U target, a = (u, A u), c = (u, A t), e = (t, A t) (A = level-0
// operator of the AMG handle), and gy = dloss/dy =
// S_U keep (-2c/(a e) A t + 2c^2/(a^2 e) A u).  A zero guess: loss 1, gy 0.
// Uses the AMG handle's solve workspace.
extern "C" int mpnn_energy_grad(mpnn_handle *H, amg_handle *A, const float *target, float *gy, double *loss,
                                hipStream_t s) {
    return guarded([&] {
        TE_REQUIRE(H && A && target && gy, TE_EINVAL, "bad argument");
        TE_REQUIRE(H->have_forward, TE_EINVAL, "mpnn_energy_grad needs a preceding mpnn_forward");
        Level &L0 = A->L[0];
        TE_REQUIRE(L0.n == H->n, TE_EINVAL, "AMG and MPNN sizes differ");
        const int64_t n = H->n, nv = 3 * n;
        const unsigned g = (unsigned)std::min<int64_t>((nv + MB - 1) / MB, 65536);
        // natural-order u and u_t in the AMG's z / p buffers, storage order in t / u
        hipLaunchKernelGGL(k_energy_prep, dim3(g), dim3(MB), 0, s, n, H->y.p, target, H->mask.p, A->z.p, A->p.p);
        permute_gather(A->z.p, A->t.p, L0.perm.p, n, 3, 1, s);
        permute_gather(A->p.p, A->u.p, L0.perm.p, n, 3, 1, s);
        sell_apply<double>(L0.A, A->t.p, A->q.p, nullptr, 0, 1, s);   // A u
        sell_apply<double>(L0.A, A->u.p, A->r.p, nullptr, 0, 1, s);   // A u_t
        double *part = A->partials.p, *sums = A->sums.p;
        dot_partials(A->t.p, A->q.p, nv, 1, part, s);
        reduce_partials(part, dot_nblocks(nv), 1, sums, s);
        dot_partials(A->t.p, A->r.p, nv, 1, part, s);
        reduce_partials(part, dot_nblocks(nv), 1, sums + 1, s);
        dot_partials(A->u.p, A->r.p, nv, 1, part, s);
        reduce_partials(part, dot_nblocks(nv), 1, sums + 2, s);
        std::vector<double> v;
        download(v, sums, 3, s);
        const double aa = v[0], c = v[1], e = v[2];
        TE_REQUIRE(e > 0, TE_EINVAL, "target has no energy");
        double ca = 0.0, cb = 0.0, L = 1.0;
        if (aa > 0) {
            L = 1.0 - c * c / (aa * e);
            ca = -2.0 * c / (aa * e) * S_U;
            cb = 2.0 * c * c / (aa * aa * e) * S_U;
        }
        if (loss) *loss = L;
        permute_scatter(A->q.p, A->z.p, L0.perm.p, n, 3, 1, s);   // A u, natural
        permute_scatter(A->r.p, A->p.p, L0.perm.p, n, 3, 1, s);   // A u_t, natural
        hipLaunchKernelGGL(k_energy_gy, dim3(g), dim3(MB), 0, s, n, A->p.p, A->z.p, H->mask.p, ca, cb, gy);
        TE_CHECK_HIP(hipGetLastError());
        return TE_OK;
    });
}

extern "C" int mpnn_adam_step(int64_t n, float *p, const float *g, float *m, float *v, int32_t step, float lr,
                              float b1, float b2, float eps, hipStream_t s) {
    return guarded([&] {
        TE_REQUIRE(n > 0 && p && g && m && v && step >= 1, TE_EINVAL, "bad argument");
        const float c1 = 1.f - std::pow(b1, (float)step), c2 = 1.f - std::pow(b2, (float)step);
        const unsigned gr = (unsigned)std::min<int64_t>((n + MB - 1) / MB, 65536);
        hipLaunchKernelGGL(k_adam, dim3(gr), dim3(MB), 0, s, n, p, g, m, v, lr, b1, b2, eps, c1, c2);
        TE_CHECK_HIP(hipGetLastError());
        return TE_OK;
    });
}

// u0 = S_U * y of the last forward (float64 [N][3])
extern "C" int mpnn_guess(mpnn_handle *H, double *u0, hipStream_t s) {
    return guarded([&] {
        TE_REQUIRE(H && u0 && H->have_forward, TE_EINVAL, "bad argument or no forward pass");
        const unsigned g = (unsigned)std::min<int64_t>((H->n * 3 + MB - 1) / MB, 65536);
        hipLaunchKernelGGL(k_guess, dim3(g), dim3(MB), 0, s, H->n, H->y.p, u0);
        TE_CHECK_HIP(hipGetLastError());
        return TE_OK;
    });
}
