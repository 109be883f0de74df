// Row x centroid scores in FP32 on the matrix cores (internal): the k-means
// assignment and the routing scores.
//
// score(x, c) = |c|^2 - 2 x.c (L2) or -x.c (IP), each dot product a sequential
// fma over ascending dimensions.  v_mfma_f32_32x32x2_f32 adds its two products
// to the accumulator one after the other, each with one rounding (checked
// against fmaf(a1, b1, fmaf(a0, b0, c)) bit for bit over normal, subnormal and
// signed zero operands), so a chain of them is that sequential fma.
//
// A workgroup scores 64 TB rows x 64 TB centroids, wave w the block (w / 2, w % 2)
// of a quarter of them: TB x TB 32 x 32 accumulators.  TB = 2 for the assignment
// (four independent products in turn, half the operand reads), 1 for the routing
// scores (four times the workgroups: a batch of 10k queries has 2512).  32 dimensions at a time are staged in LDS (two buffers, the
// next step's loads in flight meanwhile), the even and the odd dimensions of
// each eight apart, so that a lane's operands of four products (half g holds
// dimension 2 s + g of product s) are one 16-byte read; rows are 36 floats
// apart, and 16 lanes' reads hit distinct banks.  Bound by the matrix cores.
#pragma once

#include "caps_device.h"
#include "caps_internal.h"

namespace caps {

typedef float f32x16s __attribute__((ext_vector_type(16)));
constexpr int kSK = 32;           // dimensions per step
constexpr int kSS = kSK + 4;      // row stride in LDS, floats

// ARGMIN: out_assign[r] = the centroid with the smallest (score, id), over all b
// (grid.y = 1); else out_scores[r * b + c] (grid.y = centroid tiles), with a row
// list score row r of input row rows[r], r < *nrows.
template <bool ARGMIN, bool VEC, int TB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(TB == 2 ? 2 : 4))) void k_scores_mfma(
    const float *__restrict__ x, int64_t n, int32_t d, const float *__restrict__ cent, const float *__restrict__ cn,
    int32_t b, int32_t metric, int32_t *__restrict__ out_assign, float *__restrict__ out_scores,
    const int32_t *__restrict__ rows, const int32_t *__restrict__ nrows) {
    constexpr int kSM = 64 * TB;      // rows and centroids per tile
    constexpr int NU = kSM / 32;      // staged rows per thread and operand
    __shared__ __align__(16) float xs[2][kSM * kSS], cs[2][kSM * kSS];
    __shared__ __align__(16) float cns[2][kSM];   // |c|^2 of the centroid tile (IP: 0; past b: inf), by tile in turn
    __shared__ uint64_t red[ARGMIN ? kSM : 1];
    const int t = threadIdx.x, w = t >> 6, lane = t & 63, g = lane >> 5, l32 = lane & 31;
    const int wr = (w >> 1) * 32 * TB, wc = (w & 1) * 32 * TB;
    if (!ARGMIN && nrows) n = min(n, (int64_t)*nrows);
    const int64_t r0 = (int64_t)blockIdx.x * kSM;
    if (r0 >= n) return;
    const int nk = (d + kSK - 1) / kSK;
    const int ct0 = ARGMIN ? 0 : blockIdx.y, ct1 = ARGMIN ? (b + kSM - 1) / kSM : ct0 + 1;
    const int total = (ct1 - ct0) * nk;
    // staging: thread t holds columns 4 (t % 8).. of rows t / 8 + 32 u
    const int sc = 4 * (t & 7), sr = t >> 3;
    const float *xrow[NU];
#pragma unroll
    for (int u = 0; u < NU; u++) {
        const int64_t r = min(r0 + sr + 32 * u, n - 1);
        xrow[u] = x + (!ARGMIN && rows ? (int64_t)rows[r] : r) * d;
    }
    auto load4 = [&](const float *row, int j) {
        if (VEC) return j < d ? *reinterpret_cast<const float4 *>(row + j) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        return make_float4(j < d ? row[j] : 0.0f, j + 1 < d ? row[j + 1] : 0.0f, j + 2 < d ? row[j + 2] : 0.0f,
                           j + 3 < d ? row[j + 3] : 0.0f);
    };
    float4 px[NU], pc[NU];
    float pn = 0.0f;
    const float cm = metric == 0 ? -2.0f : -1.0f;   // score = |c|^2 + (cm x.c), the product rounded (2 x.c may overflow)
    auto fetch = [&](int it) {
        const int c0 = (ct0 + it / nk) * kSM, j = it % nk * kSK + sc;
        if (it % nk == 0 && t < kSM) pn = c0 + t >= b ? __builtin_huge_valf() : metric == 0 ? cn[c0 + t] : 0.0f;
#pragma unroll
        for (int u = 0; u < NU; u++) {
            px[u] = load4(xrow[u], j);
            pc[u] = load4(cent + (int64_t)min(c0 + sr + 32 * u, b - 1) * d, j);
        }
    };
    const int so = (sc & ~7) + (sc & 4) / 2;   // of each eight: even dimensions at 0..3, odd ones at 4..7
    auto stage = [&](int buf) {
#pragma unroll
        for (int u = 0; u < NU; u++) {
            float *xd = &xs[buf][(sr + 32 * u) * kSS + so], *cd = &cs[buf][(sr + 32 * u) * kSS + so];
            *reinterpret_cast<float2 *>(xd) = make_float2(px[u].x, px[u].z);
            *reinterpret_cast<float2 *>(xd + 4) = make_float2(px[u].y, px[u].w);
            *reinterpret_cast<float2 *>(cd) = make_float2(pc[u].x, pc[u].z);
            *reinterpret_cast<float2 *>(cd + 4) = make_float2(pc[u].y, pc[u].w);
        }
    };
    f32x16s acc[TB][TB];   // [row block][centroid block]
#pragma unroll
    for (int i = 0; i < TB; i++)
#pragma unroll
        for (int k = 0; k < TB; k++) acc[i][k] = f32x16s{};
    // ARGMIN: the products are centroids x rows, so that a lane's 16 results are
    // centroids of one row (l32 of block i); best so far of each block's row
    float best[TB];
    int bestc[TB];
#pragma unroll
    for (int i = 0; i < TB; i++) {
        best[i] = __builtin_huge_valf();
        bestc[i] = 0;
    }
    fetch(0);
    for (int it = 0; it < total; it++) {
        const int buf = it & 1;
        stage(buf);
        if (it % nk == 0 && t < kSM) cns[it / nk & 1][t] = pn;
        __syncthreads();   // (the other buffer is free: every wave is past its last read of it)
        // (after the barrier, which waits for outstanding loads: they land during
        // the products)
        if (it + 1 < total) fetch(it + 1);
#pragma unroll
        for (int s = 0; s < kSK; s += 8) {
            float4 xv[TB], cv[TB];
#pragma unroll
            for (int i = 0; i < TB; i++) {
                xv[i] = *reinterpret_cast<const float4 *>(&xs[buf][(wr + 32 * i + l32) * kSS + s + 4 * g]);
                cv[i] = *reinterpret_cast<const float4 *>(&cs[buf][(wc + 32 * i + l32) * kSS + s + 4 * g]);
            }
#pragma unroll
            for (int e = 0; e < 4; e++)
#pragma unroll
                for (int i = 0; i < TB; i++)
#pragma unroll
                    for (int k = 0; k < TB; k++) {
                        const float xe = e == 0 ? xv[i].x : e == 1 ? xv[i].y : e == 2 ? xv[i].z : xv[i].w;
                        const float ce = e == 0 ? cv[k].x : e == 1 ? cv[k].y : e == 2 ? cv[k].z : cv[k].w;
                        acc[i][k] = ARGMIN ? __builtin_amdgcn_mfma_f32_32x32x2f32(ce, xe, acc[i][k], 0, 0, 0)
                                           : __builtin_amdgcn_mfma_f32_32x32x2f32(xe, ce, acc[i][k], 0, 0, 0);
                    }
        }
        if ((it + 1) % nk) continue;
        // ---- the centroid tile is summed
        const int c0 = (ct0 + it / nk) * kSM + wc;
        if (ARGMIN) {
#pragma unroll
            for (int k = 0; k < TB; k++)
#pragma unroll
                for (int r4 = 0; r4 < 4; r4++) {   // ascending centroids: a strict test keeps the smallest id of a tie
                    const int cl = 32 * k + 8 * r4 + 4 * g;
                    const float4 nv = *reinterpret_cast<const float4 *>(&cns[it / nk & 1][wc + cl]);
                    const float nc[4] = {nv.x, nv.y, nv.z, nv.w};
#pragma unroll
                    for (int e = 0; e < 4; e++)
#pragma unroll
                        for (int i = 0; i < TB; i++) {
                            const float s = nc[e] + cm * acc[i][k][4 * r4 + e];
                            const bool lt = s < best[i];
                            best[i] = lt ? s : best[i];
                            bestc[i] = lt ? c0 + cl + e : bestc[i];
                            acc[i][k][4 * r4 + e] = 0.0f;
                        }
                }
        } else {
#pragma unroll
            for (int k = 0; k < TB; k++) {
                const int c = c0 + 32 * k + l32;
                if (c >= b) continue;
                const float nc = cns[it / nk & 1][wc + 32 * k + l32];
#pragma unroll
                for (int i = 0; i < TB; i++)
#pragma unroll
                    for (int r = 0; r < 16; r++) {
                        const int64_t row = r0 + wr + 32 * i + 8 * (r >> 2) + 4 * g + (r & 3);
                        if (row < n)
                            out_scores[row * b + c] = canon0(nc + cm * acc[i][k][r]);
                    }
            }
        }
    }
    if (ARGMIN) {
        // join the halves of the lanes, then the two waves of a row
        uint64_t key[TB];
#pragma unroll
        for (int i = 0; i < TB; i++) {
            key[i] = ((uint64_t)f2ord(canon0(best[i])) << 32) | (uint32_t)bestc[i];
            const uint64_t o = __shfl_xor(key[i], 32, 64);
            key[i] = o < key[i] ? o : key[i];
        }
        if ((w & 1) && g == 0)
#pragma unroll
            for (int i = 0; i < TB; i++) red[wr + 32 * i + l32] = key[i];
        __syncthreads();
        if (!(w & 1) && g == 0)
#pragma unroll
            for (int i = 0; i < TB; i++) {
                const uint64_t o = red[wr + 32 * i + l32], v = o < key[i] ? o : key[i];
                const int64_t row = r0 + wr + 32 * i + l32;
                if (row < n) out_assign[row] = (int32_t)(uint32_t)v;
            }
    }
}

template <bool ARGMIN>
inline void launch_scores(const float *x, int64_t n, int32_t d, const float *cent, const float *cn, int32_t b,
                          int32_t metric, int32_t *out_assign, float *out_scores, hipStream_t st,
                          const int32_t *rows = nullptr, const int32_t *nrows = nullptr) {
    constexpr int TB = ARGMIN ? 2 : 1, T = 64 * TB;
    const dim3 grid((unsigned)((n + T - 1) / T), ARGMIN ? 1u : (unsigned)((b + T - 1) / T));
    if (d % 4 == 0)
        hipLaunchKernelGGL((k_scores_mfma<ARGMIN, true, TB>), grid, dim3(256), 0, st, x, n, d, cent, cn, b, metric,
                           out_assign, out_scores, rows, nrows);
    else
        hipLaunchKernelGGL((k_scores_mfma<ARGMIN, false, TB>), grid, dim3(256), 0, st, x, n, d, cent, cn, b, metric,
                           out_assign, out_scores, rows, nrows);
}

}  // namespace caps
