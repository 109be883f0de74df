// Matrix-core scan over the index's low-precision copy.
//
// Build: every CSR vector gets a BF16, FP16 or FP8-E4M3 copy (zero padded to
// 32 x {1, 2, 4, 8} coordinates), its FP32 |x|^2 (sequential fma) and two
// error norms computed in FP64 and rounded up: |x - x~| and |x~| (x~ the
// value the copy represents).  Queries are rounded the same way when a
// search starts, with the matching query-side norms.
//
// Each tile (one partition, up to 64 of the queries probing it) computes
// query x point dot products with MFMA (v_mfma_f32_16x16x32_{bf16,f16,fp8},
// FP32 accumulation) and applies the exact attribute filter to every
// (query, point) pair in the epilogue.  Two uses:
//
// * approximate search (mode 1): each query keeps its best R candidates
//   under the approximate score (L2: |x|^2 - 2 x~.q~, IP: -x~.q~); a merge
//   pass rescores a query's candidates over all probes with the exact FP32
//   arithmetic and keeps the final top k;
// * exact search (mode 0 on an index with a copy): the approximate score,
//   widened by the error norms and a rounding margin, is a lower bound on the
//   exact FP32 distance.  A pair whose bound exceeds its query's current k-th
//   exact key cannot enter the top k; every other pair is rescored exactly
//   (the sequential fma of the plain scan) and competes with its exact key.
//   Results are identical to the plain FP32 scan.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "caps_mfma.h"
#include "caps_query.h"
#include "caps_x32.h"

namespace caps {

// ------------------------------------------------------------------ build
// |x|^2 (sequential fma), rounded copy, FP8 scale and the error norms |x - x~|
// and |x~| (rounded up).  A wave takes 64 rows through LDS, 32 coordinates at a
// time: rows come in and codes go out coalesced, and each lane sums one row in
// order (the sums are defined as sequential).  FP8 rows are read twice, for
// the scale first.  A thread per row straight from memory, each of its loads
// and stores in a line of its own, took 2.5 ms for 0.5M x 128.
constexpr int kQS = 33;   // row stride of the staged step, in floats
__global__ __launch_bounds__(64) void k_quantize(const float *__restrict__ x, int64_t n, int32_t d, int32_t dpad,
                                                 int32_t prec, void *__restrict__ out, float *__restrict__ scale,
                                                 float *__restrict__ xnorm, float *__restrict__ lerr,
                                                 float *__restrict__ lnrm) {
    __shared__ float st[64 * kQS];
    const int lane = threadIdx.x;
    const int64_t r0 = (int64_t)blockIdx.x * 64;
    const int nr = (int)min((int64_t)64, n - r0);
    auto stage = [&](int j0) {   // 32 coordinates of the 64 rows (zeros past d and n), two rows per step
        wave_sync();
        for (int i = 0; i < 64; i += 2) {
            const int r = i + (lane >> 5), j = j0 + (lane & 31);
            st[r * kQS + (lane & 31)] = r < nr && j < d ? x[(r0 + r) * d + j] : 0.0f;
        }
        wave_sync();
    };
    const float *row = st + lane * kQS;
    float s = 1.0f;
    if (prec == CAPS_PREC_FP8) {
        float amax = 0.0f;
        for (int j0 = 0; j0 < d; j0 += 32) {
            stage(j0);
            for (int j = 0; j < 32; j++) amax = fmaxf(amax, fabsf(row[j]));
        }
        s = amax > 0.0f ? amax / 448.0f : 1.0f;
    }
    float acc = 0.0f;
    double e2 = 0.0, a2 = 0.0;
    for (int j0 = 0; j0 < dpad; j0 += 32) {
        stage(j0);
        for (int j = 0; j < 32 && j0 + j < d; j++) {
            const float v = row[j];
            acc = fmaf(v, v, acc);
            double u;
            uint32_t c;
            if (prec == CAPS_PREC_FP8) {
                c = e4m3_rne_sat(v / s);
                u = (double)s * e4m3_value((uint8_t)c);
            } else {
                c = prec == CAPS_PREC_BF16 ? bf16_rne(v) : f16_rne_sat(v);
                u = prec == CAPS_PREC_BF16 ? (double)__uint_as_float(c << 16)
                                           : (double)__builtin_bit_cast(_Float16, (uint16_t)c);
            }
            e2 += ((double)v - u) * ((double)v - u);
            a2 += u * u;
            st[lane * kQS + j] = __uint_as_float(c);   // (the code in the coordinate's place; zeros stay zero codes)
        }
        wave_sync();
        // codes out: 64 two-byte codes of two rows, or 128 one-byte codes of four, at a time
        if (prec == CAPS_PREC_FP8) {
            for (int i = 0; i < 64; i += 8) {
                const int r = i + (lane >> 3), j = 4 * (lane & 7);
                const float *cv = st + r * kQS + j;
                const uint32_t v = __float_as_uint(cv[0]) | __float_as_uint(cv[1]) << 8 | __float_as_uint(cv[2]) << 16 |
                                   __float_as_uint(cv[3]) << 24;
                if (r < nr) *reinterpret_cast<uint32_t *>(reinterpret_cast<uint8_t *>(out) + (r0 + r) * dpad + j0 + j) = v;
            }
        } else {
            for (int i = 0; i < 64; i += 4) {
                const int r = i + (lane >> 4), j = 2 * (lane & 15);
                const float *cv = st + r * kQS + j;
                const uint32_t v = __float_as_uint(cv[0]) | __float_as_uint(cv[1]) << 16;
                if (r < nr) *reinterpret_cast<uint32_t *>(reinterpret_cast<uint16_t *>(out) + (r0 + r) * dpad + j0 + j) = v;
            }
        }
    }
    if (lane < nr) {
        const int64_t i = r0 + lane;
        xnorm[i] = acc;
        if (prec == CAPS_PREC_FP8) scale[i] = s;
        lerr[i] = f32_up(sqrt(e2) * kNormSlack);
        lnrm[i] = f32_up(sqrt(a2) * kNormSlack);
    }
}

// The BF16 copy that a large search on an FP32 index makes in its workspace:
// 16 lanes per row, four coordinates per lane and step, norms in FP32.  The
// error norm is the square root of a sum of d squares, each with at most d + 2
// roundings, and a square below the smallest normal number may come out as 0:
// both are covered by the factor 1 + 2^-10 and the term d 2^-125.  HBM bound
// (4 d + 2 dpad bytes a row): 1M x 128 in 0.19 ms (4.2 TB/s); k_quantize, whose
// sums are sequential and in FP64, takes 0.35 ms for half as many rows.
template <bool VEC>
__global__ __launch_bounds__(256) void k_search_copy(const float *__restrict__ x, int64_t n, int32_t d, int32_t dpad,
                                                     uint16_t *__restrict__ out, float *__restrict__ xnorm,
                                                     float *__restrict__ lerr, float *__restrict__ lnrm) {
    const int l16 = threadIdx.x & 15;
    const int64_t i = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
    if (i >= n) return;   // (whole groups of 16 lanes)
    const float *r = x + i * d;
    uint16_t *o = out + i * dpad;
    float nx = 0.0f, e2 = 0.0f, a2 = 0.0f;
    uint2 code[4];   // dpad <= 256: at most four steps of 64 coordinates
#pragma unroll
    for (int s = 0; s < 4; s++) {
        const int j = 64 * s + 4 * l16;
        float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (VEC) {
            if (j < d) {
                const float4 f = *reinterpret_cast<const float4 *>(r + j);
                v[0] = f.x;
                v[1] = f.y;
                v[2] = f.z;
                v[3] = f.w;
            }
        } else {
#pragma unroll
            for (int c = 0; c < 4; c++)
                if (j + c < d) v[c] = r[j + c];
        }
        uint32_t h[4];
#pragma unroll
        for (int c = 0; c < 4; c++) {
            h[c] = bf16_rne(v[c]);
            const float u = __uint_as_float(h[c] << 16), e = v[c] - u;
            nx = fmaf(v[c], v[c], nx);
            e2 = fmaf(e, e, e2);
            a2 = fmaf(u, u, a2);
        }
        code[s] = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
    }
#pragma unroll
    for (int w = 8; w >= 1; w >>= 1) {
        nx += __shfl_xor(nx, w, 64);
        e2 += __shfl_xor(e2, w, 64);
        a2 += __shfl_xor(a2, w, 64);
    }
    const bool ok = nx < kNormMax && a2 < kNormMax;   // (false for NaN too)
#pragma unroll
    for (int s = 0; s < 4; s++) {
        const int j = 64 * s + 4 * l16;
        if (j < dpad) *reinterpret_cast<uint2 *>(o + j) = ok ? code[s] : make_uint2(0u, 0u);
    }
    if (l16 == 0) {
        const float tiny = (float)d * 0x1p-125f, up = 1.0f + 0x1p-10f;
        xnorm[i] = ok ? nx : 0.0f;
        lerr[i] = ok ? sqrtf(e2 + tiny) * up : __builtin_huge_valf();
        lnrm[i] = ok ? sqrtf(a2 + tiny) * up : __builtin_huge_valf();
    }
}

caps_status search_copy(const float *x, int64_t n, int32_t d, int32_t dpad, uint16_t *lvec, float *xnorm, float *lerr,
                        float *lnrm, hipStream_t st) {
    const dim3 g((unsigned)((n + 15) / 16));
    if (d % 4 == 0)
        hipLaunchKernelGGL(k_search_copy<true>, g, dim3(256), 0, st, x, n, d, dpad, lvec, xnorm, lerr, lnrm);
    else
        hipLaunchKernelGGL(k_search_copy<false>, g, dim3(256), 0, st, x, n, d, dpad, lvec, xnorm, lerr, lnrm);
    CAPS_HIP(hipGetLastError());
    return CAPS_OK;
}

static int esize_of(int prec) { return prec == CAPS_PREC_FP8 ? 1 : 2; }

caps_status quantize_rows(const Index *ix, const float *x, int64_t n, void *lvec, float *scale, float *xnorm,
                          float *lerr, float *lnrm, hipStream_t st) {
    if (n <= 0) return CAPS_OK;
    hipLaunchKernelGGL(k_quantize, dim3((unsigned)((n + 63) / 64)), dim3(64), 0, st, x, n, ix->d, ix->dpad,
                       ix->prec, lvec, scale, xnorm, lerr, lnrm);
    CAPS_HIP(hipGetLastError());
    return CAPS_OK;
}

caps_status build_lowp(Index *ix, hipStream_t st) {
    if (ix->prec == CAPS_PREC_NONE) return CAPS_OK;
    // rows padded to 32 x {1, 2, 4, 8} coordinates: the scan kernels are
    // specialised on the number of 32-wide MFMA K-steps
    int ns = 1;
    while (32 * ns < ix->d) ns <<= 1;
    ix->dpad = 32 * ns;
    const size_t eb = (size_t)esize_of(ix->prec);
    const size_t lbytes = (size_t)ix->n * ix->dpad * eb;
    const size_t fbytes = sizeof(float) * (size_t)ix->n;
    CAPS_HIP(hipMalloc(&ix->lvecs, lbytes));
    ix->bytes += (int64_t)lbytes;
    CAPS_HIP(hipMalloc((void **)&ix->xnorm, fbytes));
    CAPS_HIP(hipMalloc((void **)&ix->lerr, fbytes));
    CAPS_HIP(hipMalloc((void **)&ix->lnrm, fbytes));
    ix->bytes += (int64_t)(3 * fbytes);
    if (ix->prec == CAPS_PREC_FP8) {
        CAPS_HIP(hipMalloc((void **)&ix->lscale, fbytes));
        ix->bytes += (int64_t)fbytes;
    }
    hipLaunchKernelGGL(k_quantize, dim3((unsigned)((ix->n + 63) / 64)), dim3(64), 0, st, ix->vecs, ix->n, ix->d,
                       ix->dpad, ix->prec, ix->lvecs, ix->lscale, ix->xnorm, ix->lerr, ix->lnrm);
    CAPS_HIP(hipGetLastError());
    return build_lowp_centroids(ix, st);
}

// ------------------------------------------------------------------ queries
// One wave per query.
__global__ __launch_bounds__(256) void k_qquant(const float *__restrict__ q, int32_t nq, int32_t d, int32_t dpad,
                                                int32_t prec, bool exact, void *__restrict__ out,
                                                float *__restrict__ scale, float *__restrict__ qaux) {
    const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= nq) return;
    qquant_row(q + i * d, i, d, dpad, prec, exact, out, scale, qaux);
}

// ------------------------------------------------------------------ routing
// Precision-mode routing: query x centroid scores from the low-precision
// copies on the matrix cores (FP32 accumulation).  64 queries x 64
// centroids per workgroup, wave w owning queries 16w..16w+15: per K-step
// one A operand (its query rows) and four B operands (four 16-centroid
// blocks), read straight from global memory (the centroid copy is small and
// stays in cache).  Score: L2 |c|^2 - 2 q~.c~ (|c|^2 of the FP32 centroid,
// sequential fma), IP -q~.c~; FP8 products are scaled by both scales.
template <int PREC, int NS>
__global__ __launch_bounds__(256) void k_route_mfma(const uint8_t *__restrict__ qlow, const float *__restrict__ qscale,
                                                    int32_t nq, const uint8_t *__restrict__ clow,
                                                    const float *__restrict__ cscale, const float *__restrict__ cn,
                                                    int32_t b, int32_t metric, float *__restrict__ scores,
                                                    const int32_t *__restrict__ rows,
                                                    const int32_t *__restrict__ nrows) {
    typedef MfmaOp<PREC> Op;
    typedef typename Op::T VT;
    constexpr int ES = Op::ES;
    constexpr int KSTEP_BYTES = 32 * ES, LANE_BYTES = 8 * ES, ROWB = NS * KSTEP_BYTES;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (nrows) nq = min(nq, *nrows);
    if ((int64_t)blockIdx.x * 64 >= nq) return;
    const int64_t q0 = (int64_t)blockIdx.x * 64 + 16 * w;
    const int c0 = blockIdx.y * 64;
    const int64_t arow = q0 + (lane & 15);
    const bool aok = arow < nq;
    const int64_t asrc_row = aok ? (rows ? (int64_t)rows[arow] : arow) : 0;
    const uint8_t *asrc = qlow + asrc_row * ROWB + (lane >> 4) * LANE_BYTES;
    f32x4 acc[4];
#pragma unroll
    for (int bb = 0; bb < 4; bb++) acc[bb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < NS; s++) {
        const VT a = aok ? Op::load(asrc + s * KSTEP_BYTES) : VT{};
        VT bf[4];
#pragma unroll
        for (int bb = 0; bb < 4; bb++) {
            const int c = c0 + bb * 16 + (lane & 15);
            bf[bb] = c < b ? Op::load(clow + (int64_t)c * ROWB + s * KSTEP_BYTES + (lane >> 4) * LANE_BYTES) : VT{};
        }
#pragma unroll
        for (int bb = 0; bb < 4; bb++) acc[bb] = Op::mma(a, bf[bb], acc[bb]);
    }
#pragma unroll
    for (int bb = 0; bb < 4; bb++) {
        const int c = c0 + bb * 16 + (lane & 15);
        if (c >= b) continue;
        const float cs = PREC == CAPS_PREC_FP8 ? cscale[c] : 1.0f;
#pragma unroll
        for (int rr = 0; rr < 4; rr++) {
            const int64_t q = q0 + (lane >> 4) * 4 + rr;
            if (q >= nq) continue;
            float dd = acc[bb][rr];
            if (PREC == CAPS_PREC_FP8) dd = dd * qscale[rows ? (int64_t)rows[q] : q] * cs;
            scores[q * b + c] = canon0(metric == 0 ? fmaf(-2.0f, dd, cn[c]) : -dd);
        }
    }
}

template <int PREC>
static void launch_route(int ns, dim3 g, hipStream_t st, const uint8_t *qlow, const float *qscale, int32_t nq,
                         const uint8_t *clow, const float *cscale, const float *cn, int32_t b, int32_t metric,
                         float *scores, const int32_t *rows, const int32_t *nrows) {
    switch (ns) {
    case 1: hipLaunchKernelGGL((k_route_mfma<PREC, 1>), g, dim3(256), 0, st, qlow, qscale, nq, clow, cscale, cn, b, metric, scores, rows, nrows); return;
    case 2: hipLaunchKernelGGL((k_route_mfma<PREC, 2>), g, dim3(256), 0, st, qlow, qscale, nq, clow, cscale, cn, b, metric, scores, rows, nrows); return;
    case 4: hipLaunchKernelGGL((k_route_mfma<PREC, 4>), g, dim3(256), 0, st, qlow, qscale, nq, clow, cscale, cn, b, metric, scores, rows, nrows); return;
    default: hipLaunchKernelGGL((k_route_mfma<PREC, 8>), g, dim3(256), 0, st, qlow, qscale, nq, clow, cscale, cn, b, metric, scores, rows, nrows); return;
    }
}

// Scores of nb rounded queries (k_qquant output) against the centroid copy.
// With a row list, score row r belongs to query rows[r], for r < *nrows.
caps_status lowp_route(const Index *ix, const void *qlow, const float *qscale, int32_t nb, float *scores,
                       hipStream_t st, const int32_t *rows, const int32_t *nrows) {
    const dim3 g((unsigned)((nb + 63) / 64), (unsigned)((ix->b + 63) / 64));
    const uint8_t *q = reinterpret_cast<const uint8_t *>(qlow), *c = reinterpret_cast<const uint8_t *>(ix->clow);
    const int ns = ix->dpad / 32;
    if (ix->prec == CAPS_PREC_BF16)
        launch_route<CAPS_PREC_BF16>(ns, g, st, q, qscale, nb, c, ix->cscale, ix->cnorm, ix->b, ix->metric, scores,
                                     rows, nrows);
    else if (ix->prec == CAPS_PREC_FP16)
        launch_route<CAPS_PREC_FP16>(ns, g, st, q, qscale, nb, c, ix->cscale, ix->cnorm, ix->b, ix->metric, scores,
                                     rows, nrows);
    else
        launch_route<CAPS_PREC_FP8>(ns, g, st, q, qscale, nb, c, ix->cscale, ix->cnorm, ix->b, ix->metric, scores,
                                    rows, nrows);
    CAPS_HIP(hipGetLastError());
    return CAPS_OK;
}

// Rounds the queries of a sub-batch into the index's copy format (codes,
// FP8 scale, error norms) for the matrix-core kernels of the exact or the
// approximate search.
caps_status lowp_qquant(const Index *ix, const float *q, int32_t nb, bool exact, void *qlow, float *qscale, float *qaux,
                        hipStream_t st) {
    hipLaunchKernelGGL(k_qquant, dim3((nb + 3) / 4), dim3(256), 0, st, q, nb, ix->d, ix->dpad, ix->prec, exact, qlow,
                       qscale, qaux);
    CAPS_HIP(hipGetLastError());
    return CAPS_OK;
}

// Low-precision copy of the centroids (the same format as the vectors', FP8
// with one scale per centroid) for precision-mode routing.
caps_status build_lowp_centroids(Index *ix, hipStream_t st) {
    if (ix->prec == CAPS_PREC_NONE) return CAPS_OK;
    const size_t eb = (size_t)esize_of(ix->prec), b = (size_t)ix->b;
    if (!ix->clow) {
        CAPS_HIP(hipMalloc(&ix->clow, b * ix->dpad * eb));
        CAPS_HIP(hipMalloc((void **)&ix->cscale, sizeof(float) * b));
        ix->bytes += (int64_t)(b * ix->dpad * eb + sizeof(float) * b);
    }
    float *tmp = nullptr;   // the norms k_quantize also writes (unused here)
    CAPS_HIP(hipMallocAsync((void **)&tmp, sizeof(float) * 3 * b, st));
    hipLaunchKernelGGL(k_quantize, dim3((unsigned)((b + 63) / 64)), dim3(64), 0, st, ix->cent, (int64_t)b, ix->d,
                       ix->dpad, ix->prec, ix->clow, ix->cscale, tmp, tmp + b, tmp + 2 * b);
    const hipError_t e = hipGetLastError();
    (void)hipFreeAsync(tmp, st);
    if (e != hipSuccess) {
        set_error("build_lowp_centroids: %s", hipGetErrorString(e));
        return CAPS_EDEVICE;
    }
    return CAPS_OK;
}

// ------------------------------------------------------------------ merge + rerank
// One wave per query: the best r approximate keys over all probes, rescored
// with the exact FP32 arithmetic, keep k.  They come from the query's deferred
// pairs (dpos: at most dcap pairs at or below the seed bound, whose r smallest
// keys are found by bisection over their scores, then over the positions of
// the tied ones) or, without those lists or where a query's did not fit
// (oflow), from the per-probe lists.  DEFER: there are deferred pairs (their 64
// registers in the other kernel halved its waves: 6141 queries, r = 64, 66 us
// against 49).
constexpr int kMCap = 256;

template <int METRIC, bool DEFER>
__global__ __launch_bounds__(256) void k_merge_rerank(const uint64_t *__restrict__ partials,
                                                      const int32_t *__restrict__ pcnt,
                                                      const uint32_t *__restrict__ sel,
                                                      const int32_t *__restrict__ cand, int32_t nq, int32_t m,
                                                      int32_t r, int32_t k, const float *__restrict__ q,
                                                      int32_t d, const float *__restrict__ vecs,
                                                      const int32_t *__restrict__ perm, int32_t *__restrict__ ids,
                                                      float *__restrict__ dist, int32_t *__restrict__ ncand,
                                                      const uint64_t *__restrict__ dpos,
                                                      const int32_t *__restrict__ dcnt,
                                                      const int32_t *__restrict__ oflow, int32_t dcap) {
    __shared__ uint64_t pool_all[4][kMCap];
    __shared__ int32_t npool_all[4];
    const int wq = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int qq = blockIdx.x * 4 + wq;
    if (qq >= nq) return;
    uint64_t *pool = pool_all[wq];
    int32_t *npool = &npool_all[wq];
    int nr;   // <= r <= 64 candidates in the pool
    if (!DEFER || oflow[qq]) {
        const int nc = gather_best<kMCap>(pool, npool, partials, pcnt, sel, cand, (int64_t)qq * m, 0, m, r, r);
        if (lane == 0) ncand[qq] = nc;
        nr = *npool;
    } else {
        const int n = min(dcnt[qq], dcap);
        const uint64_t *src = dpos + (int64_t)qq * dcap;
        auto select = [&](auto np_c) {
            constexpr int NP = decltype(np_c)::value;   // n <= 64 NP
            uint64_t e[NP];
#pragma unroll
            for (int j = 0; j < NP; j++) e[j] = j * 64 + lane < n ? src[j * 64 + lane] : ~0ull;
            // the r-th smallest key: its score, then its position
            uint64_t T = ~0ull - 1;
            if (n > r) {
                uint32_t ans = 0;
                int below = 0;   // keys of scores below ans
                for (int bit = 31; bit >= 0; bit--) {
                    const uint32_t t = ans | (1u << bit);
                    int c = 0;
#pragma unroll
                    for (int j = 0; j < NP; j++) c += __popcll(__ballot((uint32_t)(e[j] >> 32) < t));
                    if (c < r) {
                        ans = t;
                        below = c;
                    }
                    if (c == r) {   // exactly the keys below t
                        ans = t - 1;
                        below = -1;
                        break;
                    }
                }
                uint32_t pa = ~0u;
                if (below >= 0) {   // r - below of the keys with score ans
                    int eq = 0;
#pragma unroll
                    for (int j = 0; j < NP; j++) eq += __popcll(__ballot((uint32_t)(e[j] >> 32) == ans));
                    if (eq > r - below) {
                        pa = 0;
                        for (int bit = 31; bit >= 0; bit--) {
                            const uint32_t t = pa | (1u << bit);
                            int c = 0;
#pragma unroll
                            for (int j = 0; j < NP; j++)
                                c += __popcll(__ballot((uint32_t)(e[j] >> 32) == ans && (uint32_t)e[j] < t));
                            if (c < r - below) pa = t;
                        }
                    }
                }
                T = ((uint64_t)ans << 32) | pa;
            }
            int at = 0;
#pragma unroll
            for (int j = 0; j < NP; j++) {
                const bool s = e[j] <= T;
                const uint64_t b = __ballot(s);
                if (s) pool[at + __popcll(b & lanemask_lt())] = e[j];
                at += __popcll(b);
            }
            return at;
        };
        nr = n <= 512 ? select(std::integral_constant<int, 8>{}) : select(std::integral_constant<int, 32>{});
        wave_sync();
        int nc = 0;
        for (int i = lane; i < m; i += 64) {
            const int64_t slot = (int64_t)qq * m + i;
            nc += sel[slot] ? cand[slot] : 0;
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) nc += __shfl_xor(nc, o, 64);
        if (lane == 0) ncand[qq] = nc;
    }
    // exact FP32 rescoring, one candidate per lane
    uint64_t key2 = ~0ull;
    if (lane < nr) {
        const int32_t pos = (int32_t)(uint32_t)(pool[lane] & 0xFFFFFFFFu);
        const float kf = exact_score<8>(vecs + (int64_t)pos * d, q + (int64_t)qq * d, d, METRIC == 0);
        key2 = ((uint64_t)f2ord(kf) << 32) | (uint32_t)perm[pos];
    }
    int rank = 0;
    for (int i = 0; i < nr; i++) rank += readlane_u64(key2, i) < key2 ? 1 : 0;
    if (lane < nr && rank < k) {
        const int64_t o = (int64_t)qq * k + rank;
        ids[o] = (int32_t)(uint32_t)(key2 & 0xFFFFFFFFu);
        const float kf = ord2f((uint32_t)(key2 >> 32));
        dist[o] = METRIC == 0 ? kf : canon0(-kf);
    }
    if (lane >= nr && lane < k) {
        const int64_t o = (int64_t)qq * k + lane;
        ids[o] = -1;
        dist[o] = METRIC == 0 ? __builtin_huge_valf() : -__builtin_huge_valf();
    }
}

// ------------------------------------------------------------------ host
template <int PREC, int KIND>
static LowpFn pick_ns(int ns, bool lab, int r) {
    switch (ns) {
    case 1: return pick_lab<PREC, 1, KIND>(lab, r);
    case 2: return pick_lab<PREC, 2, KIND>(lab, r);
    case 4: return pick_lab<PREC, 4, KIND>(lab, r);
    default: return pick_lab<PREC, 8, KIND>(lab, r);
    }
}

template <int KIND>
static LowpFn pick_prec(int prec, int ns, bool lab, int r) {
    if (prec == CAPS_PREC_BF16) return pick_ns<CAPS_PREC_BF16, KIND>(ns, lab, r);
    if (prec == CAPS_PREC_FP16) return pick_ns<CAPS_PREC_FP16, KIND>(ns, lab, r);
    return pick_ns<CAPS_PREC_FP8, KIND>(ns, lab, r);
}

template <int PREC>
static LowpFn pick_x32_filt(int filt, int ns, int mode) {
    return filt == 0 ? pick_x32<PREC, 0>(ns, mode) : filt == 1 ? pick_x32<PREC, 1>(ns, mode) : pick_x32<PREC, 2>(ns, mode);
}
static LowpFn pick_x32_prec(int prec, int filt, int ns, int mode) {
    if (prec == CAPS_PREC_BF16) return pick_x32_filt<CAPS_PREC_BF16>(filt, ns, mode);
    if (prec == CAPS_PREC_FP16) return pick_x32_filt<CAPS_PREC_FP16>(filt, ns, mode);
    return pick_x32_filt<CAPS_PREC_FP8>(filt, ns, mode);
}

// workgroups of the rescue pass (32 per compute unit): enough to spread a
// long list, few enough that an empty one costs little
constexpr int64_t kRescueWgs = 8192;

size_t lowp_scan_lds(const Index *ix, int r, int kind, bool disj) {
    return LowpLds(kind == 1 || kind == 3 ? 32 : lowp_cb(r), kind, ix->sch.label_vocab > 0 || disj).total + 64;
}

caps_status lowp_scan(const Index *ix, const LowpScan &S, hipStream_t st) {
    LowpArgs A;
    A.tiles = S.tiles;
    A.ntiles = (int32_t)S.max_tiles;
    A.entries = S.entries;
    A.esel = S.esel;
    A.sel = S.sel;
    A.qd = S.qd;
    A.qterms = S.qterms;
    A.offs = ix->offs;
    A.lvecs = reinterpret_cast<const uint8_t *>(ix->lvecs);
    A.lscale = ix->lscale;
    A.xnorm = ix->xnorm;
    A.lerr = ix->lerr;
    A.lnrm = ix->lnrm;
    A.words = ix->words;
    A.sigs = ix->sigs;
    A.slots = ix->slots;
    A.lslots = ix->lslots;
    A.wbits = 0;
    for (int a = 0; a < ix->sch.n_dense; a++) A.wbits += ix->sch.field_bits[a];
    A.qlow = reinterpret_cast<const uint8_t *>(S.qlow);
    A.qscale = S.qscale;
    A.qaux = S.qaux;
    A.vecs = ix->vecs;
    A.q = S.q;
    A.perm = ix->perm;
    A.partials = S.partials;
    A.pcnt = S.pcnt;
    A.tau = S.tau;
    A.nsurv = S.nsurv;
    A.dpos = S.dpos;
    A.dcnt = S.dcnt;
    A.dcap = S.dcap;
    A.split = std::max(1, S.split);
    A.oflow = S.oflow;
    A.rlist = S.rlist;
    A.rcount = S.rcount;
    A.rhalves = S.rhalves ? 1 : 0;
    A.m = S.m;
    A.h = ix->h;
    A.b = ix->b;
    A.r = S.r;
    A.metric = ix->metric;
    A.d = ix->d;
    // Rounding budget of the exact bound, relative to |x|^2 + |q|^2 (+ the
    // bound's own magnitude): the stored |x|^2 (d roundings), the exact
    // distance against its real value (d + 2), the FP32 evaluation of the
    // bound (a dozen) -- about 3 dpad + 24 units of 2^-24, doubled.  The
    // MFMA accumulation (at most dpad additions, each within 2^-23 of the
    // sum of magnitudes) is bounded by gam |x~| |q~|, gam = 8 dpad 2^-24
    // (four times that).
    A.eta = exact_eta(ix);
    A.gam = (float)(8.0 * ix->dpad) * 0x1p-24f;
    // the variant with the filter's slow path: label tests, disjunctions
    const bool lab = ix->sch.label_vocab > 0 || S.disj;
    const int ns = ix->dpad / 32;
    // (the 32 x 32 scan holds its arrays in static LDS)
    const bool x32 = S.kind == 4 || S.kind == 6 || (S.kind == 1 && x32_kernel(ns, lab, S.nsurv != nullptr));
    const int xmode = S.kind == 4 ? (S.seed_mh == 1 ? 2 : 3) : S.kind == 6 ? 4 : S.nsurv ? 1 : 0;
    const LowpFn fn = x32 ? pick_x32_prec(ix->prec, S.disj ? 2 : lab ? 1 : 0, ns, xmode)
                      : S.kind == 0 ? pick_prec<0>(ix->prec, ns, lab, S.r)
                      : S.kind == 1 ? (S.nsurv ? pick_prec<3>(ix->prec, ns, lab, S.r) : pick_prec<1>(ix->prec, ns, lab, S.r))
                      : S.kind == 5 ? pick_prec<5>(ix->prec, ns, lab, S.r)
                                    : pick_prec<2>(ix->prec, ns, lab, S.r);
    const size_t lds = x32 ? 0 : lowp_scan_lds(ix, S.r, S.kind, S.disj);
    {
        const caps_status ls = set_kernel_lds((const void *)fn, lds, ix->device);
        if (ls != CAPS_OK) return ls;
    }
    prof_begin(S.stage, st);
    // the rescue pass walks its (device-side) tile list with a bounded grid
    const int64_t full = (S.max_tiles * (x32 ? A.split : 1) + kXcds - 1) / kXcds * kXcds;
    const int64_t rcap = S.rescue_grid > 0 ? S.rescue_grid : kRescueWgs;
    const int64_t grid = S.kind == 2 || S.kind == 5 ? std::min<int64_t>(full, rcap) : full;
    hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(x32 ? kXW * 64 : kLNT), lds, st, A);
    prof_end(S.stage, st);
    CAPS_HIP(hipGetLastError());
    return CAPS_OK;
}

caps_status lowp_merge(const Index *ix, const float *q, int32_t nb, const uint32_t *sel, int32_t m, int32_t k,
                       int32_t r, const uint64_t *partials, const int32_t *pcnt, const int32_t *cand, int32_t *ncand,
                       int32_t *out_ids, float *out_dist, hipStream_t st, const uint64_t *dpos, const int32_t *dcnt,
                       const int32_t *oflow, int32_t dcap) {
    prof_begin(CAPS_STAGE_MERGE, st);
    const auto fn = ix->metric == 0 ? (dpos ? k_merge_rerank<0, true> : k_merge_rerank<0, false>)
                                    : (dpos ? k_merge_rerank<1, true> : k_merge_rerank<1, false>);
    hipLaunchKernelGGL(fn, dim3((nb + 3) / 4), dim3(256), 0, st, partials, pcnt, sel, cand, nb, m, r, k, q, ix->d, ix->vecs,
                       ix->perm, out_ids, out_dist, ncand, dpos, dcnt, oflow, dcap);
    prof_end(CAPS_STAGE_MERGE, st);
    CAPS_HIP(hipGetLastError());
    return CAPS_OK;
}

int lowp_qb() { return kLQB; }

int lowp_qb_main(const Index *ix, bool disj, bool count) {
    return x32_kernel(ix->dpad / 32, ix->sch.label_vocab > 0 || disj, count) ? kXQB : kLQB;
}

// Keys each lane of the 32 x 32 seed pass keeps (half of a partition's rows
// and one query), or 0 where the seed round runs k_scan_mfma's approximate
// kind; *split: in, how many workgroups may share a tile's rows; out, how many do
// (each fills its own part of the lists of r keys).
// Lists of two keys per seed probe are enough when they hold twice k
// (longer lists cost more insertions than their tighter bound saved: 4 and 10
// keys ran 0.34 and 0.44 ms per 10k-query step against 0.28 ms with the same
// main pass); with fewer seed probes or a longer result list, lists of eight
// keys where those can hold k; else the full lists of r.  The lists of two of
// all workgroups of a tile take the place of lists of eight where together they
// hold 4 k, or, if every probe is a seed (all), 2 k with as many a probe as
// those (or k): with fewer a query finds too few keys in the partitions that
// hold its neighbours (5223 queries over 7 of 98 partitions, k = 10, two
// workgroups a tile: 0.75 ms against 0.48 with lists of eight) or, selective
// ones, fewer than k in all, and then no bound (65 queries over 74 of 97, k = 52:
// 0.25 ms against 0.14).
int lowp_seed_x32(const Index *ix, bool disj, int r, int k, int s_seed, bool all, int *split) {
    const int want = *split;
    *split = 1;
    if (!x32_kernel(ix->dpad / 32, ix->sch.label_vocab > 0 || disj, false) || r < 2) return 0;
    const int s1 = std::max(1, std::min(want, r / 2));   // (two keys each)
    const bool two = s_seed >= k || s1 * s_seed >= 2 * k || (all && s1 * s_seed >= k && 2 * s1 >= std::min(8, k));
    const int mh = two ? 1 : r >= 8 && 8 * s_seed >= k ? 4 : 0;
    if (mh) *split = mh == 1 ? s1 : std::max(1, std::min(want, r / 8));
    return mh;
}

// The approximate search defers its pairs (32 x 32 blocks) where that scan has
// a kernel and the seed lists (eight keys a probe, or two for r < 8) can hold r
// keys.  10k queries x 1M x 128 BF16, r = 40: 1.9 ms main pass against 5.5 ms
// with the per-query key buffers of k_scan_mfma's approximate kind.
bool lowp_approx_x32(int32_t dpad, bool lab, int32_t r, int32_t s_seed) {
    return x32_kernel(dpad / 32, lab, false) && r >= 2 && (r >= 8 ? 8 : 2) * (int64_t)s_seed >= r;
}

}  // namespace caps
